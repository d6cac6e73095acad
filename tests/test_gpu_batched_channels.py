"""Batches whose images differ in their channel counts and layouts: the units of
the persistent launch then come in runs of 1 to 16 planes, images of more
channels in several groups.  Every image as alone, nothing beside the outputs
written."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _layout(shape, dtype, interleaved):
    n, c, h, w = shape
    if interleaved:
        return torch.full((n, h, w, c), 77, dtype=dtype, device="cuda").permute(0, 3, 1, 2)
    return torch.full(shape, 77, dtype=dtype, device="cuda")


def _batch(seed, channels, count, dtypes, mixed):
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    xs, outs = [], []
    for i in range(count):
        c, n = int(channels[i % len(channels)]), int(rng.integers(1, 3))
        h, w = (int(rng.integers(1, 90)) for _ in range(2))
        src, dst = dtypes[i % len(dtypes)]
        v = torch.rand((n, c, h, w), generator=gen, device="cuda")
        x = _layout(v.shape, src, not mixed or rng.random() < 0.6)
        x.copy_((255 * v).round() if src == torch.uint8 else v)
        xs.append(x)
        outs.append(_layout((n, c, 2 * h, 2 * w), dst, not mixed or rng.random() < 0.6))
    return xs, outs


U8, F32 = torch.uint8, torch.float32


@pytest.mark.parametrize("rows,cols", [(0, 0), (4, 1), (32, 2)])
@pytest.mark.parametrize("channels,count,dtypes,mixed", [
    ((64, 3), 24, [(U8, U8)], False),
    ((3, 1, 17, 16, 2, 33), 40, [(U8, U8)], True),
    ((1, 40, 3, 5), 40, [(F32, F32)], True),
    ((100,), 3, [(F32, F32)], False),
    ((1, 3, 20), 60, [(U8, U8), (U8, F32), (F32, U8), (F32, F32)], True),
    ((3,), 1, [(U8, U8)], False),
])
def test_channel_counts(gpu, channels, count, dtypes, mixed, rows, cols):
    xs, outs = _batch(count + len(channels), channels, count, dtypes, mixed)
    refs = [gpu.zoom2x_(x, torch.empty_like(o)) for x, o in zip(xs, outs)]
    gpu.set_launch_config(rows, cols)
    try:
        plan = gpu.BatchedZoom(xs, outs)
        for _ in range(2):
            for o in outs:
                o.fill_(77)
            plan.run()
            for k, (o, r) in enumerate(zip(outs, refs)):
                assert torch.equal(o, r), (k, tuple(o.shape), o.stride())
    finally:
        gpu.set_launch_config(0, 0)
