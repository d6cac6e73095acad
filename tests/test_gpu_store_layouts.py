"""Destination layouts of the doubling, at the edges of its strips: float rows
with spread columns (interleaved channels, every second column of a wider
tensor), float rows at every 4-byte alignment and byte rows give the same bits
as an aligned planar destination, which is checked against the FP64 oracle;
nothing outside the destination's elements is written."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

# one- and two-column strips own 55 and 118 columns
WIDTHS = (1, 2, 7, 31, 32, 33, 54, 55, 56, 64, 117, 118, 119, 173, 237)


def _dest(layout, n, c, h, w, dtype):
    """(destination view, its whole storage) filled with a value no result has."""
    fill = 77 if dtype == torch.uint8 else -7.0
    if layout == "planar":
        base = torch.full((n, c, h, w), fill, dtype=dtype, device="cuda")
        return base, base
    if layout == "hwc":
        base = torch.full((n, h, w, c), fill, dtype=dtype, device="cuda")
        return base.permute(0, 3, 1, 2), base
    if layout == "spread":
        base = torch.full((n, c, h, 2 * w + 1), fill, dtype=dtype, device="cuda")
        return base[..., 1::2], base
    off = int(layout[-1])   # "offK": rows start K elements past an aligned pitch of odd length
    base = torch.full((n, c, h, w + off + 1), fill, dtype=dtype, device="cuda")
    return base[..., off:off + w], base


@pytest.mark.parametrize("cols", [1, 2])
@pytest.mark.parametrize("w", WIDTHS)
def test_layouts_give_the_same_bits(gpu, w, cols):
    rng = np.random.default_rng(w)
    gpu.set_launch_config(7, cols)
    try:
        for n, c, h, u8_in in ((1, 3, 23, False), (2, 3, 9, True), (1, 4, 1, False)):
            x8 = torch.tensor(rng.integers(0, 256, size=(n, c, h, w)).astype(np.uint8), device="cuda")
            x = x8 if u8_in else x8.float() / 255.0
            ref, _ = _dest("planar", n, c, 2 * h, 2 * w, torch.float32)
            gpu.zoom2x_(x, ref)
            V = x8.double().cpu().numpy() / 255.0 if u8_in else x.double().cpu().numpy()
            assert np.abs(ref.double().cpu().numpy() - oracle.zoom2x(V)).max() <= 1e-5
            ref8 = None
            for layout in ("hwc", "spread", "off1", "off2", "off3"):
                out, base = _dest(layout, n, c, 2 * h, 2 * w, torch.float32)
                gpu.zoom2x_(x, out)
                assert torch.equal(out, ref), (layout, n, c, h)
                out.fill_(-7.0)
                assert bool((base == -7.0).all()), (layout, n, c, h)
            for layout in ("planar", "hwc", "spread", "off1", "off2", "off3"):
                out, base = _dest(layout, n, c, 2 * h, 2 * w, torch.uint8)
                gpu.zoom2x_(x, out)
                if ref8 is None:
                    ref8 = out.clone()
                assert torch.equal(out, ref8), (layout, n, c, h)
                out.fill_(77)
                assert bool((base == 77).all()), (layout, n, c, h)
    finally:
        gpu.set_launch_config(0, 0)


@pytest.mark.parametrize("shape", [(1, 3, 300, 500), (2, 4, 61, 700), (1, 2, 1000, 130), (3, 3, 64, 64)])
def test_interleaved_automatic_shapes(gpu, shape):
    # the launch order of interleaved planes, at automatic launch shapes
    x = torch.rand(shape, device="cuda")
    n, c, h, w = shape
    ref, _ = _dest("planar", n, c, 2 * h, 2 * w, torch.float32)
    gpu.zoom2x_(x, ref)
    out, _ = _dest("hwc", n, c, 2 * h, 2 * w, torch.float32)
    gpu.zoom2x_(x.contiguous(memory_format=torch.channels_last), out)
    assert torch.equal(out, ref)


@pytest.mark.parametrize("beta", [2.0, 1.5])
def test_batch_of_mixed_layouts(gpu, beta):
    # one queue per layout and type: each image as alone, on every run of the plan
    kinds = [("hwc", torch.uint8, torch.uint8), ("planar", torch.float32, torch.float32),
             ("hwc", torch.uint8, torch.float32), ("planar", torch.uint8, torch.uint8),
             ("spread", torch.float32, torch.float32), ("planar", torch.float32, torch.uint8),
             ("hwc", torch.float32, torch.uint8), ("planar", torch.uint8, torch.float32)]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    xs, outs, refs = [], [], []
    for i in range(3 * len(kinds)):
        layout, src, dst = kinds[i % len(kinds)]
        h, w = 9 + 13 * i, 200 - 7 * i
        v = torch.rand((1, 3, h, w), generator=gen, device="cuda")
        xs.append((255 * v).round().to(torch.uint8) if src == torch.uint8 else v)
        outs.append(_dest(layout, 1, 3, 2 * h, 2 * w, dst)[0])
        refs.append(gpu.zoom2x(xs[-1], beta=beta, out_dtype=dst))
    plan = gpu.BatchedZoom(xs, outs, gpu.Params(beta=beta))
    for _ in range(3):
        for o in outs:
            o.zero_()
        plan.run()
        assert all(torch.equal(o, r) for o, r in zip(outs, refs))
