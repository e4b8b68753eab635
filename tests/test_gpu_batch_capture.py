"""Batched steps in a caller's graph: replays go on after channels have come
and gone, whether the batch is large enough for several steps per launch or
not at that moment, and each channel's bits stay those of its solo run."""
import pytest
import torch

import oracle
from oracle import Params

from helpers import lib_kwargs
from paper_2112_13930_amd._lib import make_params
from paper_2112_13930_amd.batch import Batch
from paper_2112_13930_amd.channel import Channel

pytestmark = pytest.mark.gpu


def _params(nx, ny):
    return Params(nx=nx, ny=ny, bc=oracle.LINK if nx % 2 else oracle.MOMENT, tau_f=0.7, tau_m=0.9,
                  b0=0.03, fx=1e-5, c_lo=0.3, c_hi=1.0, u_hi=0.04)


@pytest.mark.parametrize("graph", [True, False])
def test_replays_after_changes_of_the_list(graph):
    stream = torch.cuda.Stream()
    b = Batch("fp64", max_channels=8, max_nodes=400_000, stream=stream)
    held = {}  # slot -> (sizes, steps taken)

    def admit(nx, ny):
        p = _params(nx, ny)
        s = b.admit(make_params(nx, ny, **lib_kwargs(p, "fp64")))
        held[s] = [(nx, ny), 0]
        return s

    def count(n):
        for v in held.values():
            v[1] += n

    def check():
        for s, ((nx, ny), n) in held.items():
            ch = Channel(nx, ny, **lib_kwargs(_params(nx, ny), "fp64"))
            ch.set_launch_shape(0)
            ch.step(n)
            assert torch.equal(b.save_state(s), ch.save_state()), (nx, ny, n)

    big, small, _ = admit(501, 401), admit(60, 40), admit(9, 50)
    b.step(4, graph=graph)
    count(4)
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=stream):
        b.step(6, graph=graph)

    def replay():
        with torch.cuda.stream(stream):
            g.replay()
        count(6)
        check()

    replay()
    b.retire(small)
    held.pop(small)
    admit(130, 77)
    b.step(2, graph=graph)
    count(2)
    replay()
    b.retire(big)  # too few nodes for several steps per launch
    held.pop(big)
    b.step(8, graph=graph)
    count(8)
    replay()
    admit(250, 640)
    b.step(8, graph=graph)
    count(8)
    replay()
    b.close()
