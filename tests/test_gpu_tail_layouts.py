"""Automatic launch shapes with one-column tail strips, into every kind of
destination: float rows whose address is not a multiple of 4, planes with
spread columns and packed bytes hold the bits of an aligned planar destination
down to the last column, which is checked against the FP64 oracle, and nothing
around the destination's elements is written."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2312_00229_amd import _lib
from paper_2312_00229_amd._lib import WenoParams, WenoTensor

pytestmark = pytest.mark.gpu

# tails of 40, 1, 55 and 10 columns; one round of waves and (48 planes) several
SHAPES = [(12, 512, 512), (48, 512, 512), (64, 512, 473), (40, 300, 173), (30, 200, 291), (3, 1500, 954)]


def _zoom(x, dst, dtype, n, h, w, sc, sh, sw):
    """weno_zoom2x of the planes x (n, h, w) into memory at the address dst;
    the launch's tail rows."""
    L = _lib.lib()
    src = WenoTensor(x.data_ptr(), _lib.WENO_U8 if x.dtype == torch.uint8 else _lib.WENO_F32, 1, n, h, w, n * h * w,
                     h * w, w, 1)
    out = WenoTensor(dst, dtype, 1, n, 2 * h, 2 * w, n * sc, sc, sh, sw)
    tail = ctypes.c_int32()
    assert L.weno_query_launch_config(ctypes.byref(src), ctypes.byref(out), None, None, ctypes.byref(tail)) == 0
    p = WenoParams(2.0, 1e-8, 1.0, -1.0, _lib.WENO_BOUNDARY_CLAMP)
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert L.weno_zoom2x(ctypes.byref(src), ctypes.byref(out), ctypes.byref(p), stream) == _lib.WENO_OK
    return tail.value


@pytest.mark.parametrize("u8_in", [False, True])
@pytest.mark.parametrize("n,h,w", SHAPES)
def test_tails_in_every_layout(gpu, n, h, w, u8_in):
    gpu.set_launch_config(0, 0)
    gen = torch.Generator(device="cuda").manual_seed(w)
    x = torch.rand((n, h, w), device="cuda", generator=gen)
    if u8_in:
        x = (255 * x).round().to(torch.uint8)
    H, W = 2 * h, 2 * w
    ref = torch.full((n, H, W), -7.0, device="cuda")
    assert _zoom(x, ref.data_ptr(), _lib.WENO_F32, n, h, w, H * W, W, 1) > 0
    V = x[-1].double().cpu().numpy() / (255.0 if u8_in else 1.0)
    assert np.abs(ref[-1].double().cpu().numpy() - oracle.zoom2x(V)).max() <= 1e-5
    # float rows 2 bytes past a multiple of 4
    buf = torch.full((ref.numel() * 4 + 4,), 77, dtype=torch.uint8, device="cuda")
    assert _zoom(x, buf.data_ptr() + 2, _lib.WENO_F32, n, h, w, H * W, W, 1) > 0
    assert torch.equal(buf[2:-2].clone().view(torch.float32).view(n, H, W), ref)
    assert bool((buf[:2] == 77).all()) and bool((buf[-2:] == 77).all())
    # every second column of wider planes
    wide = torch.full((n, H, 2 * W), -7.0, device="cuda")
    assert _zoom(x, wide.data_ptr() + 4, _lib.WENO_F32, n, h, w, 2 * H * W, 2 * W, 2) > 0
    assert torch.equal(wide[..., 1::2], ref) and bool((wide[..., ::2] == -7.0).all())
    # bytes, packed and spread
    ref8 = torch.full((n, H, W), 77, dtype=torch.uint8, device="cuda")
    assert _zoom(x, ref8.data_ptr(), _lib.WENO_U8, n, h, w, H * W, W, 1) > 0
    if not u8_in:   # the same scale either way
        assert torch.equal(ref8, (255 * ref).round().clamp(0, 255).to(torch.uint8))
    wide8 = torch.full((n, H, 2 * W), 77, dtype=torch.uint8, device="cuda")
    tail8 = _zoom(x, wide8.data_ptr() + 1, _lib.WENO_U8, n, h, w, 2 * H * W, 2 * W, 2)
    assert tail8 > 0 or w == 473   # there one column per lane is cheaper for spread bytes
    assert torch.equal(wide8[..., 1::2], ref8) and bool((wide8[..., ::2] == 77).all())
