"""Batches that mix contiguous and spread destinations of one pair of types: all
in one launch (bytes always, floats while the batch is small), or a launch for
each; every image as alone either way."""
import pytest
import torch

pytestmark = pytest.mark.gpu

U8, F32 = torch.uint8, torch.float32


def _image(planar, h, w, dtype, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    v = torch.rand((3, h, w) if planar else (h, w, 3), generator=gen, device="cuda")
    v = (255 * v).round().to(U8) if dtype == U8 else v
    return v if planar else v.permute(2, 0, 1)


def _dest(planar, h, w, dtype):
    if planar:
        return torch.zeros((3, 2 * h, 2 * w), dtype=dtype, device="cuda")
    return torch.zeros((2 * h, 2 * w, 3), dtype=dtype, device="cuda").permute(2, 0, 1)


def _plan(gpu, images):
    gpu.set_launch_config(0, 0)
    xs = [_image(p, h, w, s, i) for i, (p, s, _, h, w) in enumerate(images)]
    outs = [_dest(p, h, w, d) for p, _, d, h, w in images]
    return xs, outs, gpu.BatchedZoom(xs, outs)


def _check(gpu, xs, outs, plan):
    for _ in range(2):
        for o in outs:
            o.zero_()
        plan.run()
        for x, o in zip(xs, outs):
            assert torch.equal(o, gpu.zoom2x(x, out_dtype=o.dtype))


@pytest.mark.parametrize("src,dst", [(U8, U8), (F32, U8), (U8, F32), (F32, F32)])
@pytest.mark.parametrize("h,w,count", [(5, 7, 2), (61, 173, 9), (300, 200, 6)])
def test_small_batches_take_one_launch(gpu, src, dst, h, w, count):
    xs, outs, plan = _plan(gpu, [(i % 2 == 0, src, dst, h + i, w + 3 * i) for i in range(count)])
    assert bin(plan.plan.reserved).count("1") == 1
    _check(gpu, xs, outs, plan)


@pytest.mark.parametrize("src,dst,launches", [(U8, U8, 1), (U8, F32, 2), (F32, F32, 2)])
def test_large_batches(gpu, src, dst, launches):
    # 8 x 3591 strips of 16 rows: over six rounds of 16 waves on 256 compute units
    xs, outs, plan = _plan(gpu, [(i % 2 == 0, src, dst, 1000, 1000) for i in range(8)])
    assert bin(plan.plan.reserved).count("1") == launches
    _check(gpu, xs, outs, plan)


def test_planar_batches_stay_contiguous(gpu):
    xs, outs, plan = _plan(gpu, [(True, U8, U8, 40, 50), (True, F32, F32, 40, 50)])
    assert plan.plan.reserved == (1 << 4) | (1 << 0)
    _check(gpu, xs, outs, plan)
