"""Several steps per launch only where they are not slower: the launches a
channel or batch takes by default against single steps, at sizes near the
lines of the dispatch.  Times are the least of several runs taken in turn; the
margin is far above what two such times differ by."""
import pytest
import torch

from paper_2112_13930_amd._lib import make_params
from paper_2112_13930_amd.batch import Batch
from paper_2112_13930_amd.channel import Channel

pytestmark = pytest.mark.gpu

KW = dict(tau_f=0.7, tau_m=0.9, b0=0.03, fx=1e-5, c_lower=0.3, c_upper=1.0, u_upper=0.04)
MARGIN = 1.12


def _least(streams_and_calls, reps=8):
    best = [1e9] * len(streams_and_calls)
    for _, call in streams_and_calls:
        call()
    for _ in range(reps):
        for i, (stream, call) in enumerate(streams_and_calls):
            torch.cuda.synchronize()
            e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            with torch.cuda.stream(stream):
                e0.record()
                call()
                e1.record()
            e1.synchronize()
            best[i] = min(best[i], e0.elapsed_time(e1))
    return best


def _against_single(nx, ny, shape=0, **kw):
    stream = torch.cuda.Stream()
    a, b = (Channel(nx, ny, stream=stream, **KW, **kw) for _ in range(2))
    b.set_launch_shape(shape)
    return _least([(stream, lambda: a.step(96)), (stream, lambda: b.step(96))])


@pytest.mark.parametrize("nx,ny", [(64, 1600), (64, 2048), (128, 1024), (256, 512), (300, 333)])
@pytest.mark.parametrize("bc", ["link", "moment"])
def test_fp64_march(nx, ny, bc):
    several, single = _against_single(nx, ny, bc=bc, precision="fp64")
    assert several <= MARGIN * single, (several, single)


@pytest.mark.parametrize("nx,ny,precision,kw", [
    (256, 256, "fp32", dict()), (256, 256, "fp16", dict(collision="mrt", bc="moment")),
    (256, 256, "fp16_f64", dict()), (512, 128, "fp16", dict(collision="trt")),
    (200, 200, "fp32", dict()), (200, 200, "fp16", dict(collision="mrt"))])
def test_regions(nx, ny, precision, kw):
    several, single = _against_single(nx, ny, precision=precision, **kw)
    assert several <= MARGIN * single, (several, single)


@pytest.mark.parametrize("nx,ny,precision,kw", [
    (1024, 512, "fp16", dict()), (384, 1197, "fp16", dict()), (300, 1747, "fp16", dict()),
    (300, 1747, "fp16", dict(collision="mrt")), (384, 1822, "fp16_f64", dict()),
    (700, 700, "fp16", dict()), (512, 1367, "fp16", dict(bc="moment")),
    (1024, 512, "fp16", dict(collision="mrt", q=(0.3, 0.8))),
    (448, 1026, "fp16", dict(x_walls=True, c_x=(0.5, 1.0)))])
def test_binary16_nodes_per_thread(nx, ny, precision, kw):
    """The default launch against both one and two nodes per thread."""
    for shape in (0, 5):
        default, given = _against_single(nx, ny, shape, precision=precision, **kw)
        assert default <= 1.07 * given, (shape, default, given)


@pytest.mark.parametrize("count,nx,ny,precision,kw", [
    (600, 4, 1000, "fp32", dict()), (1000, 8, 256, "fp32", dict(bc="moment")),
    (2000, 32, 32, "fp32", dict(collision="mrt")), (700, 61, 61, "fp32", dict(collision="trt")),
    (1250, 4, 200, "fp64", dict(collision="mrt")), (64, 256, 128, "fp32", dict())])
def test_batches(count, nx, ny, precision, kw):
    """Steps as the batch takes them against single steps, which a caller's
    graph records."""
    stream = torch.cuda.Stream()
    b = Batch(precision, max_channels=count, max_nodes=count * nx * ny, stream=stream)
    p = make_params(nx, ny, precision=precision, **KW, **kw)
    for _ in range(count):
        b.admit(p)
    b.step(96)
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        b.step(96)
    default, single = _least([(stream, lambda: b.step(96)), (stream, graph.replay)], reps=4)
    b.close()
    assert default <= MARGIN * single, (default, single)
