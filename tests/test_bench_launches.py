"""bench.py's count of the launches of a timed run."""
import pytest

import bench


@pytest.mark.parametrize("steps,launches", [(1, 1), (2, 1), (3, 1), (4, 2), (5, 2), (20, 7),
                                            (200, 67), (1000, 334)])
def test_launches_of(steps, launches):
    assert bench.launches_of(steps) == launches


def test_rates_of_bytes_only_where_they_are_moved():
    assert bench.hbm_of(1e9, 1e-3, "fp32") == {} == bench.hbm_of(1e9, 1e-3, "fp64")
    assert bench.hbm_of(4e9, 1e-3, "fp16") == {"gbs": 4000.0, "frac_hbm": 0.5}
