"""Plain steps captured in a graph of the caller's: an even number of them ends
in the buffer it starts from however many steps a launch takes, so every
replay goes on from the one before it, bit for bit as eager steps do."""
import pytest
import torch

import oracle
from oracle import Params

from helpers import lib_kwargs
from paper_2112_13930_amd.channel import Channel
from paper_2112_13930_amd.workloads import random_populations

pytestmark = pytest.mark.gpu


# marches of 4, 3 and 2 steps a launch, regions, single steps
@pytest.mark.parametrize("nx,ny,precision", [(1021, 493, "fp64"), (1500, 701, "fp32"),
                                             (1021, 493, "fp32"), (61, 33, "fp64"),
                                             (61, 33, "fp16"), (512, 512, "fp16")])
@pytest.mark.parametrize("steps", [2, 4, 6, 10])
def test_replays_of_a_callers_graph(nx, ny, precision, steps):
    p = Params(nx=nx, ny=ny, bc=oracle.LINK, tau_f=0.7, tau_m=0.9, b0=0.03, fx=1e-5, c_lo=0.3,
               c_hi=1.0, u_hi=0.04)
    s0 = torch.from_numpy(random_populations(nx, ny, seed=3, b0=p.b0))
    stream = torch.cuda.Stream()
    captured = Channel(nx, ny, stream=stream, **lib_kwargs(p, precision))
    eager = Channel(nx, ny, **lib_kwargs(p, precision))
    for ch in (captured, eager):
        ch.load_state(s0)
        ch.step(steps)
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        captured.step(steps)
    for replay in range(4):
        with torch.cuda.stream(stream):
            graph.replay()
        eager.step(steps)
        assert torch.equal(captured.save_state(), eager.save_state()), replay
