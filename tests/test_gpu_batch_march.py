"""Large FP32 and FP64 batches advance three steps per launch: every channel's
bits equal those of a solo run in single steps, over widths that share a
wavefront's lanes in different numbers (1, 3, 4, 29, 30, 60, 61, 130 columns),
two and three rows, both wall schemes, pools with and without TRT and MRT
channels, channels admitted at an odd step and retired, and graphs on and off."""
import pytest
import torch

import oracle
from oracle import Params

from helpers import lib_kwargs, mrt, trt
from paper_2112_13930_amd._lib import make_params
from paper_2112_13930_amd.batch import Batch
from paper_2112_13930_amd.channel import Channel

pytestmark = pytest.mark.gpu

COLL = {"bgk": lambda p: p, "trt": trt, "mrt": mrt}
# the first is large enough for the multi-step launches of either precision
MIX = [(1501, 1401), (1, 300), (3, 517), (4, 33), (29, 64), (30, 129), (60, 95), (61, 41),
       (130, 77), (256, 3), (257, 2), (2, 2)]


def _params(i, pool):
    nx, ny = MIX[i]
    bc = oracle.LINK if i % 2 == 0 or ny < 3 else oracle.MOMENT
    coll = "bgk" if pool == "bgk" else ("bgk", "trt", "mrt")[i % 3]
    return COLL[coll](Params(nx=nx, ny=ny, bc=bc, tau_f=0.7, tau_m=0.9, b0=0.03, fx=1e-5,
                             c_lo=0.3, c_hi=1.0, u_lo=-0.01, u_hi=0.04))


def _admit(b, i, pool, precision):
    p = _params(i, pool)
    return b.admit(make_params(p.nx, p.ny, **lib_kwargs(p, precision)))


@pytest.mark.parametrize("graph", [True, False])
@pytest.mark.parametrize("pool", ["bgk", "mixed"])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_equals_solo_single_steps(precision, pool, graph):
    b = Batch(precision, max_channels=16, max_nodes=2_400_000)
    slots = {i: _admit(b, i, pool, precision) for i in range(7)}
    b.step(5, graph=graph)
    for i in range(7, len(MIX)):
        slots[i] = _admit(b, i, pool, precision)
    b.step(61, graph=graph)
    b.retire(slots.pop(5))
    b.step_check(12, graph=graph)
    b.step(8, graph=graph)
    for i, s in slots.items():
        n = b.steps_done(s)
        assert n == (86 if i < 7 else 81)
        p = _params(i, pool)
        ch = Channel(p.nx, p.ny, **lib_kwargs(p, precision))
        ch.set_launch_shape(0)
        ch.step(n)
        assert torch.equal(b.save_state(s), ch.save_state()), (i, MIX[i])
    b.close()
