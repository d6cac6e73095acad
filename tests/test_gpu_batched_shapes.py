"""The automatic strip shape of a batch with float destinations: short strips
where interleaved float destinations hold most of the pixels or the batch is a
few rounds of waves, the cost model's elsewhere; the same bits either way."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _image(interleaved, h, w, dtype, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    v = torch.rand((3, h, w), generator=gen, device="cuda")
    if dtype == torch.uint8:
        v = (255 * v).round().to(torch.uint8)
    return v.permute(1, 2, 0).contiguous().permute(2, 0, 1) if interleaved else v


def _dest(interleaved, h, w):
    shape = (2 * h, 2 * w, 3) if interleaved else (3, 2 * h, 2 * w)
    out = torch.full(shape, -7.0, device="cuda")
    return out.permute(2, 0, 1) if interleaved else out


# images as (source interleaved, destination interleaved, height), all uint8 to float32
@pytest.mark.parametrize("images,short", [
    ([(True, False, 1000)] * 24, False),                             # a network's input, many rounds
    ([(True, False, 200)] * 8, True),                                # the same, a few rounds
    ([(False, True, 1000)] + [(False, False, 1000)] * 23, False),    # one interleaved destination decides nothing
    ([(False, True, 1000)] * 12 + [(False, False, 1000)] * 12, True),
])
def test_shape_of_float_batches(gpu, images, short):
    gpu.set_launch_config(0, 0)
    xs = [_image(s, h, 1000, torch.uint8, i) for i, (s, _, h) in enumerate(images)]
    outs = [_dest(d, h, 1000) for _, d, h in images]
    plan = gpu.BatchedZoom(xs, outs)
    assert (plan.plan.rows_per_strip <= 16) == short
    plan.run()
    for i in (0, len(xs) - 1):
        assert torch.equal(outs[i], gpu.zoom2x(xs[i], out_dtype=torch.float32))
