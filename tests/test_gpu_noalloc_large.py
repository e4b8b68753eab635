"""lks_mhd_advance_noalloc at the size of its static array: channels whose
padded rows do not fit it run with packed ones, and large FP64 ones march; the
bits are those of the entry points that pad."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SCRATCH = 64 << 20


@pytest.mark.parametrize("nx,ny,precision,padded_fits", [
    (225, 1733, "fp32", False), (225, 3100, "fp16", False), (225, 900, "fp64", True)])
@pytest.mark.parametrize("bc", ["link", "moment"])
def test_equals_existing_entry_points(nx, ny, precision, padded_fits, bc):
    from paper_2112_13930_amd import _lib as L
    from paper_2112_13930_amd.channel import Channel
    from paper_2112_13930_amd.workloads import random_populations
    params = L.make_params(nx, ny, bc=bc, precision=precision, tau_f=0.75, tau_m=0.85, b0=0.02,
                           fx=1e-5, c_lower=0.3, c_upper=float("inf"), u_upper=0.04)
    assert L.lib().lks_mhd_least_bytes(ctypes.byref(params)) <= SCRATCH
    assert (L.lib().lks_mhd_state_bytes(ctypes.byref(params)) <= SCRATCH) == padded_fits
    pops = torch.from_numpy(random_populations(nx, ny, seed=nx, b0=0.02)).cuda()
    stream = torch.cuda.current_stream()
    ch = Channel(params=params, stream=stream)
    ch.load_state(pops, steps=995)
    ch.step(12)
    want = ch.save_state()
    got = pops.clone()
    rc = L.lib().lks_mhd_advance_noalloc(ctypes.byref(params), ctypes.c_void_p(got.data_ptr()),
                                         995, 12, ctypes.c_void_p(stream.cuda_stream))
    assert rc == L.LKS_OK, L.last_error()
    torch.cuda.synchronize()
    assert torch.equal(got, want)
