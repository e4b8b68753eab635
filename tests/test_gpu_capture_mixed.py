"""A caller's graph and eager calls on one channel, in turn.  The graph holds
the buffer its first step reads, so an even number of eager steps (plain, from
a private graph, or a steady-state window) has to end in the buffer it starts
from, however many steps a launch takes: replays then go on from the eager
steps, bit for bit, and a captured read of the fields reads the state."""
import pytest
import torch

import oracle
from oracle import Params

from helpers import lib_kwargs
from paper_2112_13930_amd.channel import Channel
from paper_2112_13930_amd.workloads import random_populations

pytestmark = pytest.mark.gpu

# marches of 4, 3 and 2 steps a launch, regions, single steps
SIZES = [(1021, 493, "fp64"), (1500, 701, "fp32"), (1021, 493, "fp32"), (61, 33, "fp64"),
         (61, 33, "fp16"), (512, 512, "fp16")]


def _pair(nx, ny, precision, stream):
    p = Params(nx=nx, ny=ny, bc=oracle.LINK, tau_f=0.7, tau_m=0.9, b0=0.03, fx=1e-5, c_lo=0.3,
               c_hi=1.0, u_hi=0.04)
    s0 = torch.from_numpy(random_populations(nx, ny, seed=3, b0=p.b0))
    pair = (Channel(nx, ny, stream=stream, **lib_kwargs(p, precision)),
            Channel(nx, ny, **lib_kwargs(p, precision)))
    for ch in pair:
        ch.load_state(s0)
        ch.step(2)
    return pair


@pytest.mark.parametrize("private", [0, 2, 4, 10])
@pytest.mark.parametrize("nx,ny,precision", SIZES)
def test_eager_steps_between_replays(nx, ny, precision, private):
    stream = torch.cuda.Stream()
    ch, ref = _pair(nx, ny, precision, stream)
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        ch.step(4)
    ch.set_graph(private)
    for n in (0, 4, 2, 10, 20):
        ch.step(n)
        ref.step(n)
        with torch.cuda.stream(stream):
            graph.replay()
        ref.step(4)
        assert torch.equal(ch.save_state(), ref.save_state()), n
    if precision == "fp16":  # (its rebases draw by the host's step count, which replays leave)
        return
    a, b = (c.run_to_steady(tol=0.0, check_every=10, max_steps=10) for c in (ch, ref))
    assert a[2:] == b[2:]
    with torch.cuda.stream(stream):
        graph.replay()
    ref.step(4)
    assert torch.equal(ch.save_state(), ref.save_state())


@pytest.mark.parametrize("nx,ny,precision", SIZES)
def test_captured_reads(nx, ny, precision):
    stream = torch.cuda.Stream()
    ch, ref = _pair(nx, ny, precision, stream)
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        m = ch.moments()
        s = ch.save_state()
    for n in (4, 2, 10):
        ch.step(n)
        ref.step(n)
        with torch.cuda.stream(stream):
            graph.replay()
        torch.cuda.synchronize()
        want = ref.moments()
        assert all(torch.equal(m[k], want[k]) for k in want), n
        assert torch.equal(s, ref.save_state()), n


@pytest.mark.parametrize("per_graph", [2, 4, 50])
@pytest.mark.parametrize("nx,ny,precision", SIZES)
def test_captured_with_private_graphs(nx, ny, precision, per_graph):
    """set_graph before the caller's capture: an eager call may have left the
    channel in the buffer that no private graph starts from yet."""
    stream = torch.cuda.Stream()
    ch, ref = _pair(nx, ny, precision, stream)
    ch.set_graph(per_graph)
    ch.step(per_graph)
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        ch.step(per_graph)
    ref.step(per_graph)
    for replay in range(3):
        with torch.cuda.stream(stream):
            graph.replay()
        ch.step(2 * per_graph)
        ref.step(3 * per_graph)
        assert torch.equal(ch.save_state(), ref.save_state()), replay
