"""A batch that grows and shrinks over the size from which it takes several
steps per launch, with its graphs on: every channel's bits stay those of its
solo run, also where a slot is taken by a channel of another width."""
import pytest
import torch

import oracle
from oracle import Params

from helpers import lib_kwargs, trt
from paper_2112_13930_amd._lib import make_params
from paper_2112_13930_amd.batch import Batch
from paper_2112_13930_amd.channel import Channel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,big", [("fp64", (501, 401)), ("fp32", (1501, 1401))])
def test_over_the_threshold_and_back(precision, big):
    b = Batch(precision, max_channels=8, max_nodes=4_400_000)
    held = {}

    def admit(nx, ny, coll=lambda p: p):
        p = coll(Params(nx=nx, ny=ny, bc=oracle.LINK, tau_f=0.7, tau_m=0.9, b0=0.03, fx=1e-5,
                        c_lo=0.3, c_hi=1.0, u_hi=0.04))
        s = b.admit(make_params(nx, ny, **lib_kwargs(p, precision)))
        held[s] = p
        return s

    def retire(s):
        held.pop(s)
        b.retire(s)

    def advance_and_check():
        b.step(50)      # the long graph and what is left over
        b.step_check(9)
        b.step(7)
        for s, p in held.items():
            ch = Channel(p.nx, p.ny, **lib_kwargs(p, precision))
            ch.set_launch_shape(0)
            ch.step(b.steps_done(s))
            assert torch.equal(b.save_state(s), ch.save_state()), (p.nx, p.ny, b.steps_done(s))

    first, other = admit(*big), admit(33, 47)
    admit(7, 90)
    advance_and_check()          # several steps per launch
    retire(other)
    admit(200, 61)               # same slot, another width and tile count
    advance_and_check()
    retire(first)
    admit(120, 88)               # single steps
    advance_and_check()
    admit(big[0] + 40, big[1])   # several again
    advance_and_check()
    admit(64, 64, trt)           # another kernel
    advance_and_check()
    b.close()
