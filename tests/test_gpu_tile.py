"""Small channels advance several steps per launch in regions of one block
(lks_tile): the same bits as single steps (a chosen launch shape), and the
oracle's fields.  Sizes around the plan's: one region for the whole channel,
regions as wide as the channel, overlapping regions in both directions with a
short last one, one column, two rows, widths and heights one off a region."""
import pytest
import torch

import oracle
from oracle import Params

from helpers import TOL, assert_close, field_errors, lib_kwargs, mrt, to_numpy, trt
from paper_2112_13930_amd.channel import Channel
from paper_2112_13930_amd.workloads import random_populations

pytestmark = pytest.mark.gpu

COLL = {"bgk": lambda p: p, "trt": trt, "mrt": mrt}
PRECISIONS = ["fp64", "fp32", "fp16", "fp16_f64"]
SIZES = [(1, 5), (2, 3), (8, 64), (16, 16), (16, 17), (17, 33), (15, 100), (70, 19), (129, 127),
         (257, 65), (3, 3000), (4000, 4)]


def _params(nx, ny, bc, coll):
    return COLL[coll](Params(nx=nx, ny=ny, bc=bc, tau_f=0.7, tau_m=0.9, b0=0.03, fx=1e-5, fy=2e-6,
                             c_lo=0.3, c_hi=1.0, u_lo=-0.01, u_hi=0.04))


@pytest.mark.parametrize("coll", ["bgk", "trt", "mrt"])
@pytest.mark.parametrize("bc", [oracle.LINK, oracle.MOMENT])
@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("nx,ny", SIZES)
def test_equals_single_steps(nx, ny, precision, bc, coll):
    p = _params(nx, ny, bc, coll)
    s0 = torch.from_numpy(random_populations(nx, ny, seed=3, b0=p.b0))
    a, b = (Channel(nx, ny, **lib_kwargs(p, precision)) for _ in range(2))
    b.set_launch_shape(0)
    for ch in (a, b):
        ch.set_rebase(13)  # binary16: a rebase in the middle of a run
        ch.load_state(s0, steps=5)
    for n in (2, 3, 7, 1, 33):
        a.step(n)
        b.step(n)
        assert a.steps_done == b.steps_done
        assert torch.equal(a.save_state(), b.save_state()), n


@pytest.mark.parametrize("coll", ["bgk", "trt", "mrt"])
@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("nx,ny", [(2, 3), (8, 64), (17, 33), (70, 19), (129, 127)])
def test_enclosure_equals_single_steps(nx, ny, precision, coll):
    p = _params(nx, ny, oracle.LINK, coll)
    p.x_walls, p.cx_lo, p.cx_hi = True, 0.5, 2.0
    s0 = torch.from_numpy(random_populations(nx, ny, seed=8, b0=p.b0))
    a, b = (Channel(nx, ny, **lib_kwargs(p, precision)) for _ in range(2))
    b.set_launch_shape(0)
    for ch in (a, b):
        ch.load_state(s0)
        ch.step(2)
        ch.step(25)
    assert torch.equal(a.save_state(), b.save_state())


@pytest.mark.parametrize("precision", PRECISIONS)
def test_two_rows(precision):
    p = _params(37, 2, oracle.LINK, "bgk")
    s0 = torch.from_numpy(random_populations(p.nx, p.ny, seed=4, b0=p.b0))
    a, b = (Channel(p.nx, p.ny, **lib_kwargs(p, precision)) for _ in range(2))
    b.set_launch_shape(0)
    for ch in (a, b):
        ch.load_state(s0)
        ch.step(9)
    assert torch.equal(a.save_state(), b.save_state())


@pytest.mark.parametrize("bc", [oracle.LINK, oracle.MOMENT])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("nx,ny", [(8, 64), (129, 127)])
def test_against_oracle(nx, ny, precision, bc):
    p = _params(nx, ny, bc, "bgk")
    s0 = random_populations(nx, ny, seed=6, b0=p.b0)
    ch = Channel(nx, ny, **lib_kwargs(p, precision))
    ch.load_state(torch.from_numpy(s0))
    ch.step(41)
    s = s0.copy()
    oracle.run(p, s, 41)
    assert_close(field_errors(to_numpy(ch.moments()), oracle.observe(p, s), p.b0), TOL[precision])


@pytest.mark.parametrize("precision,per_graph", [("fp64", 2), ("fp32", 6), ("fp16", 10)])
def test_graphs_and_windows(precision, per_graph):
    """Captured steps replayed several times with eager steps and a
    steady-state window in between."""
    p = _params(61, 47, oracle.LINK, "bgk")
    s0 = torch.from_numpy(random_populations(p.nx, p.ny, seed=7, b0=p.b0))
    a, b = (Channel(p.nx, p.ny, stream=torch.cuda.Stream(), **lib_kwargs(p, precision))
            for _ in range(2))
    a.set_graph(per_graph)
    b.set_launch_shape(0)
    for ch in (a, b):
        ch.load_state(s0)
    for n in (per_graph, 3 * per_graph + 1, 1, 2 * per_graph):
        a.step(n)
        b.step(n)
        assert torch.equal(a.save_state(), b.save_state()), n
    ra, rb = (ch.run_to_steady(tol=0.0, check_every=9, max_steps=18) for ch in (a, b))
    assert ra == rb
    assert torch.equal(a.save_state(), b.save_state())
