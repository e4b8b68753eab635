"""Three-dimensional steps captured by a caller while the channel has private
graphs: they go into the caller's graph as plain launches."""
import pytest
import torch

from paper_2112_13930_amd.channel3 import Channel3
from paper_2112_13930_amd.workloads import random_populations3

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("per_graph", [2, 6])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_captured_with_private_graphs(precision, per_graph):
    kw = dict(bc="link", precision=precision, tau_f=0.7, tau_m=0.9, b0=0.03, fx=1e-5, c_lower=0.3,
              c_upper=1.0, u_upper=0.04)
    stream = torch.cuda.Stream()
    ch, ref = Channel3(33, 20, 9, stream=stream, **kw), Channel3(33, 20, 9, **kw)
    ch.set_graph(per_graph)
    s0 = torch.from_numpy(random_populations3(33, 20, 9, seed=2, b0=0.03))
    for c in (ch, ref):
        c.load_state(s0)
        c.step(per_graph)
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        ch.step(per_graph)
    for replay in range(3):
        with torch.cuda.stream(stream):
            graph.replay()
        ch.step(per_graph)
        ref.step(2 * per_graph)
        assert torch.equal(ch.save_state(), ref.save_state()), replay
