"""Several steps per launch (lks_march) against single steps and the oracle.

Large FP64 and FP32 channels advance 2 to 4 steps per launch by default; a
chosen launch shape (set_launch_shape) keeps single steps.  Both give the same
bits, whatever the sizes leave over: strips of columns narrower than a
wavefront, one row chunk, walls two rows apart, step counts that are no
multiple of the launch's, graphs, and load/save in between."""
import numpy as np
import pytest
import torch

import oracle
from oracle import Params

from helpers import TOL, assert_close, field_errors, lib_kwargs, mrt, to_numpy, trt
from paper_2112_13930_amd.channel import Channel
from paper_2112_13930_amd.workloads import random_populations

pytestmark = pytest.mark.gpu

COLL = {"bgk": lambda p: p, "trt": trt, "mrt": mrt}


def _params(nx, ny, bc, coll):
    return COLL[coll](Params(nx=nx, ny=ny, bc=bc, tau_f=0.7, tau_m=0.9, b0=0.03, fx=1e-5, fy=2e-6,
                             c_lo=0.3, c_hi=1.0, u_lo=-0.01, u_hi=0.04))


# widths: one strip not full (47), one strip of one step count and two of
# another (60, 62), a last strip of one column (121); odd ones; heights: two
# and three rows, one chunk, many chunks with a short last one
SIZES = [(60, 8400), (62, 8111), (121, 4200), (47, 10650), (1021, 493), (175001, 3),
         (400, 251), (1500, 701)]


@pytest.mark.parametrize("coll", ["bgk", "trt", "mrt"])
@pytest.mark.parametrize("bc", [oracle.LINK, oracle.MOMENT])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("nx,ny", SIZES)
def test_equals_single_steps(nx, ny, precision, bc, coll):
    p = _params(nx, ny, bc, coll)
    s0 = torch.from_numpy(random_populations(nx, ny, seed=3, b0=p.b0))
    a, b = (Channel(nx, ny, **lib_kwargs(p, precision)) for _ in range(2))
    b.set_launch_shape(0)
    for ch in (a, b):
        ch.load_state(s0, steps=5)
    for n in (2, 3, 4, 5, 1, 11):
        a.step(n)
        b.step(n)
        assert a.steps_done == b.steps_done
        assert torch.equal(a.save_state(), b.save_state()), n


def test_two_rows():
    """Both walls on the two rows of a link channel."""
    p = _params(262145, 2, oracle.LINK, "bgk")
    s0 = torch.from_numpy(random_populations(p.nx, p.ny, seed=4, b0=p.b0))
    a, b = (Channel(p.nx, p.ny, **lib_kwargs(p, "fp64")) for _ in range(2))
    b.set_launch_shape(0)
    for ch in (a, b):
        ch.load_state(s0)
        ch.step(7)
    assert torch.equal(a.save_state(), b.save_state())


@pytest.mark.parametrize("bc", [oracle.LINK, oracle.MOMENT])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_against_oracle(precision, bc):
    p = _params(1021, 493, bc, "bgk")
    s0 = random_populations(p.nx, p.ny, seed=6, b0=p.b0)
    ch = Channel(p.nx, p.ny, **lib_kwargs(p, precision))
    ch.load_state(torch.from_numpy(s0))
    ch.step(13)
    s = s0.copy()
    oracle.run(p, s, 13, nthreads=4)
    assert_close(field_errors(to_numpy(ch.moments()), oracle.observe(p, s), p.b0), TOL[precision])


@pytest.mark.parametrize("precision,per_graph", [("fp64", 2), ("fp64", 6), ("fp32", 4)])
def test_graphs_and_windows(precision, per_graph):
    """Captured steps, whose launches may be odd in number, replayed several
    times with eager steps and a steady-state window in between."""
    p = _params(1021, 493, oracle.LINK, "bgk")
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
    ma, mb = a.moments(), b.moments()
    assert all(np.array_equal(ma[k].cpu(), mb[k].cpu()) for k in ma)
