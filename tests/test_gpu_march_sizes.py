"""FP64 channels of medium size march two or three steps per launch, by their
nodes and width: the bits of single steps on both sides of those lines."""
import pytest
import torch

import oracle
from oracle import Params

from helpers import lib_kwargs, mrt, trt
from paper_2112_13930_amd.channel import Channel
from paper_2112_13930_amd.workloads import random_populations

pytestmark = pytest.mark.gpu

COLL = {"bgk": lambda p: p, "trt": trt, "mrt": mrt}


# 100k, 125k and 350k nodes; powers of two; one column more
@pytest.mark.parametrize("coll", ["bgk", "trt", "mrt"])
@pytest.mark.parametrize("nx,ny", [(256, 391), (257, 391), (512, 200), (1024, 122), (128, 977),
                                   (26, 4400), (333, 500), (700, 499), (701, 500)])
def test_equals_single_steps(nx, ny, coll):
    p = COLL[coll](Params(nx=nx, ny=ny, bc=oracle.LINK if nx % 2 else oracle.MOMENT, tau_f=0.7,
                          tau_m=0.9, b0=0.03, fx=1e-5, fy=2e-6, c_lo=0.3, c_hi=1.0, u_hi=0.04))
    s0 = torch.from_numpy(random_populations(nx, ny, seed=3, b0=p.b0))
    a, b = (Channel(nx, ny, **lib_kwargs(p, "fp64")) for _ in range(2))
    b.set_launch_shape(0)
    for ch in (a, b):
        ch.load_state(s0)
    for n in (2, 3, 4, 11):
        a.step(n)
        b.step(n)
        assert torch.equal(a.save_state(), b.save_state()), n
