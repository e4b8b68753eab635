"""autotune on a batch that takes several steps per launch: its trials, which
time the tiles of single steps, are real steps, and the batch goes back to
several steps per launch after them."""
import pytest
import torch

import oracle
from oracle import Params

from helpers import lib_kwargs
from paper_2112_13930_amd._lib import make_params
from paper_2112_13930_amd.batch import Batch
from paper_2112_13930_amd.channel import Channel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("graph", [True, False])
def test_bits_after_autotune(graph):
    sizes = [(501, 401), (9, 200), (130, 33)]
    ps = [Params(nx=nx, ny=ny, bc=oracle.LINK, tau_f=0.7, tau_m=0.9, b0=0.03, fx=1e-5, c_lo=0.3,
                 c_hi=1.0, u_hi=0.04) for nx, ny in sizes]
    b = Batch("fp64", max_channels=4, max_nodes=400_000)
    slots = [b.admit(make_params(p.nx, p.ny, **lib_kwargs(p, "fp64"))) for p in ps]
    b.step(7, graph=graph)
    b.autotune(trial_steps=4)
    b.step(50, graph=graph)
    b.step_check(8, graph=graph)
    for s, p in zip(slots, ps):
        ch = Channel(p.nx, p.ny, **lib_kwargs(p, "fp64"))
        ch.set_launch_shape(0)
        ch.step(b.steps_done(s))
        assert torch.equal(b.save_state(s), ch.save_state()), (p.nx, p.ny)
    b.close()
