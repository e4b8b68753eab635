"""Single channels keep their rows padded to cache lines (or not): the same
bits as a batch, whose rows are packed, in every precision, and the oracle's
fields for the walls a batch does not take.  Widths around the padding rules:
one off a line, half lines, packed."""
import numpy as np
import pytest
import torch

import oracle
from oracle import Params

from helpers import TOL, assert_close, field_errors, lib_kwargs, to_numpy
from paper_2112_13930_amd._lib import make_params
from paper_2112_13930_amd.batch import Batch
from paper_2112_13930_amd.channel import Channel
from paper_2112_13930_amd.workloads import random_populations

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bc", [oracle.LINK, oracle.MOMENT])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16", "fp16_f64"])
@pytest.mark.parametrize("nx", [13, 60, 125, 223, 255, 257, 999])
def test_padded_equals_packed(nx, precision, bc):
    p = Params(nx=nx, ny=9, bc=bc, tau_f=0.7, tau_m=0.9, b0=0.03, fx=1e-5, c_lo=0.3, c_hi=1.0,
               u_hi=0.04)
    ch = Channel(nx, 9, **lib_kwargs(p, precision))
    ch.set_launch_shape(0)
    ch.set_rebase(5)
    b = Batch(precision, max_channels=2, max_nodes=nx * 9 + 64)
    s = b.admit(make_params(nx, 9, **lib_kwargs(p, precision)))
    for _ in range(2):
        b.step_check(5)
        ch.step(5)
    assert torch.equal(b.save_state(s), ch.save_state())
    m, n = b.moments(s), ch.moments()
    assert all(torch.equal(m[k], n[k]) for k in m)
    b.close()


@pytest.mark.parametrize("case", ["x_walls", "cut", "disc"])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("nx", [60, 125, 257])
def test_other_walls_against_oracle(nx, precision, case):
    kw = dict(nx=nx, ny=31, bc=oracle.LINK, tau_f=0.7, tau_m=0.9, b0=0.03, fx=1e-5, c_lo=0.3,
              c_hi=1.0, u_hi=0.04)
    if case == "x_walls":
        kw.update(x_walls=True, cx_lo=0.5, cx_hi=2.0)
    elif case == "cut":
        kw.update(q_lo=0.3, q_hi=0.8)
    else:
        kw.update(solids=((oracle.DISC, 20.3, 15.2, 6.4, 0.002, 0.0),))
    p = Params(**kw)
    s0 = random_populations(nx, 31, seed=5, b0=p.b0)
    if case == "disc":  # solid nodes rest
        s0[:, oracle.solid_mask(p)] = oracle.init_state(p)[:, oracle.solid_mask(p)]
    ch = Channel(nx, 31, **lib_kwargs(p, precision))
    ch.load_state(torch.from_numpy(s0))
    ch.step(7)
    s = s0.copy()
    oracle.run(p, s, 7)
    assert_close(field_errors(to_numpy(ch.moments()), oracle.observe(p, s), p.b0), TOL[precision])
    assert np.isfinite(s).all()
