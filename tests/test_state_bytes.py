"""Channels go on fitting the memory they have fitted: create takes a buffer
without room for padded rows, and the Python classes fall back to one."""
import ctypes

import pytest
import torch

import oracle
from oracle import Params

from helpers import lib_kwargs
from paper_2112_13930_amd import channel
from paper_2112_13930_amd._lib import LksParams3, lib, make_params
from paper_2112_13930_amd.channel import Channel
from paper_2112_13930_amd.channel3 import Channel3
from paper_2112_13930_amd.workloads import random_populations, random_populations3


# marches and, but in FP64, regions, which gain little or nothing by padded rows
@pytest.mark.parametrize("nx,ny,precision", [
    (333, 333, "fp64"), (1021, 493, "fp32"), (26, 4000, "fp64"), (2500, 300, "fp64"),
    (5000, 1111, "fp32"), (13, 900, "fp32"), (257, 65, "fp32"), (129, 127, "fp16"),
    (55, 60, "fp16_f64")])
def test_several_steps_per_launch_pad_little(nx, ny, precision):
    p = make_params(nx, ny, precision=precision)
    least = lib().lks_mhd_least_bytes(ctypes.byref(p))
    assert lib().lks_mhd_state_bytes(ctypes.byref(p)) <= 1.02 * least


# bytes of the packed layout, which buffers may have been sized by
@pytest.mark.parametrize("nx,ny,precision,size", [
    (13, 900, "fp64", 4228096), (257, 65, "fp32", 3153920), (1021, 493, "fp64", 161602816),
    (1023, 513, "fp32", 88702208), (3001, 2110, "fp16", 585480960),
    (999, 40, "fp16_f64", 4022528), (333, 333, "fp32", 19040256)])
def test_least_bytes(nx, ny, precision, size):
    p = make_params(nx, ny, precision=precision)
    least = lib().lks_mhd_least_bytes(ctypes.byref(p))
    assert least <= size and least <= lib().lks_mhd_state_bytes(ctypes.byref(p))


@pytest.mark.parametrize("nx,ny,nz,precision,size", [
    (250, 130, 100, "fp32", 1015187712), (90, 61, 47, "fp64", 157455872),
    (33, 5, 4, "fp32", 239872)])
def test_least_bytes_3d(nx, ny, nz, precision, size):
    p = LksParams3()
    p.base = make_params(nx, ny, precision=precision)
    p.nz = nz
    least = lib().lks_mhd3_least_bytes(ctypes.byref(p))
    assert least <= size and least <= lib().lks_mhd3_state_bytes(ctypes.byref(p))


def _only(least, monkeypatch):
    """Allocations of more than `least` bytes fail while a channel is made."""
    empty = torch.empty

    def limited(*size, **kw):
        if kw.get("dtype") is torch.uint8 and size[0] > least:
            raise torch.OutOfMemoryError
        return empty(*size, **kw)

    monkeypatch.setattr(channel.torch, "empty", limited)


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16", "fp16_f64"])
@pytest.mark.parametrize("nx,ny", [(61, 33), (223, 300), (333, 700), (125, 1000), (1021, 493)])
def test_packed_equals_padded(nx, ny, precision, monkeypatch):
    p = Params(nx=nx, ny=ny, bc=oracle.LINK, tau_f=0.7, tau_m=0.9, b0=0.03, fx=1e-5, c_lo=0.3,
               c_hi=1.0, u_hi=0.04)
    if nx == 125:
        p.x_walls, p.cx_lo, p.cx_hi = True, 0.5, 2.0
    full = Channel(nx, ny, **lib_kwargs(p, precision))
    least = lib().lks_mhd_least_bytes(ctypes.byref(full.params))
    with monkeypatch.context() as m:
        _only(least, m)
        packed = Channel(nx, ny, **lib_kwargs(p, precision))
    assert packed._buf.numel() == least
    s0 = torch.from_numpy(random_populations(nx, ny, seed=5, b0=p.b0))
    for ch in (full, packed):
        ch.load_state(s0)
        ch.set_rebase(5)
        ch.step(11)
        ch.run_to_steady(tol=0.0, check_every=4, max_steps=8)
    assert torch.equal(full.save_state(), packed.save_state())
    a, b = full.moments(), packed.moments()
    assert all(torch.equal(a[k], b[k]) for k in a)


@pytest.mark.gpu
@pytest.mark.parametrize("side", [False, True])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_packed_equals_padded_3d(precision, side, monkeypatch):
    kw = dict(side_walls=side, c_side=0.5, bc="link", precision=precision, tau_f=0.7, tau_m=0.9,
              b0=0.03, fx=1e-5, c_lower=0.3, c_upper=1.0, u_upper=0.04)
    full = Channel3(90, 9, 7, **kw)
    least = lib().lks_mhd3_least_bytes(ctypes.byref(full.params))
    with monkeypatch.context() as m:
        _only(least, m)
        packed = Channel3(90, 9, 7, **kw)
    assert packed._buf.numel() == least < full._buf.numel()
    s0 = torch.from_numpy(random_populations3(90, 9, 7, seed=5, b0=0.03))
    for ch in (full, packed):
        ch.load_state(s0)
        ch.step(7)
    assert torch.equal(full.save_state(), packed.save_state())
