"""Launches of one round that read and write more than 256 MiB in float rows
(written back from the L2) against the same planes one by one (written
through): the same bits, with and without a narrow last strip, on both sides
of the limit."""
import pytest
import torch

pytestmark = pytest.mark.gpu


# 3 x 4 planes: reads + writes in MiB: float32 20 px bytes, uint8 -> float32 17
@pytest.mark.parametrize("h,w,src", [
    (1081, 1090, torch.float32),   # 270: ragged, odd rows
    (1024, 1097, torch.float32),   # 257: just above
    (1024, 1088, torch.float32),   # 255: just below (written through)
    (700, 1800, torch.float32),    # 288
    (1500, 954, torch.float32),    # 327: 8 strips of 118 columns and 10 more
    (1200, 1219, torch.uint8),     # 284
])
def test_large_paced_launch_is_planewise(gpu, h, w, src):
    gen = torch.Generator(device="cuda").manual_seed(h + w)
    x = torch.rand(4, 3, h, w, device="cuda", generator=gen)
    if src == torch.uint8:
        x = (x * 255).to(torch.uint8)
    y = torch.full((4, 3, 2 * h, 2 * w), -1.0, device="cuda")
    gpu.zoom2x_(x, y)
    for n in range(4):
        for c in range(3):
            assert torch.equal(y[n, c], gpu.zoom2x(x[n, c], out_dtype=torch.float32)), (n, c)
