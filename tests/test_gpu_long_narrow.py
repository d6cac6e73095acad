"""Planes so long and narrow that short runs and strips would need more than the
2^32 work-items of a launch: interleaved as planar, and planar as a few of its
rows alone."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _column(c, h):
    gen = torch.Generator(device="cuda").manual_seed(c)
    return torch.randint(0, 256, (h, 1, c), generator=gen, dtype=torch.uint8, device="cuda").permute(2, 0, 1)


def test_resample_interleaved(gpu):
    # 8 interleaved channels: runs of 18 rows, 4 to a workgroup, would be 29.8 million workgroups
    c, h_in, h_out = 8, 1 << 10, (1 << 28) - 1
    x = _column(c, h_in)
    out = torch.zeros((h_out, 1, c), dtype=torch.uint8, device="cuda").permute(2, 0, 1)
    gpu.resample(x, h_out, 1, out=out)
    planar = torch.zeros((c, h_out, 1), dtype=torch.uint8, device="cuda")
    assert torch.equal(out, gpu.resample(x.contiguous(), h_out, 1, out=planar))


def test_resample_planar(gpu):
    # 1.6 billion rows of one column against the first and last intervals of a smaller target of the same positions
    h_in, step = 1 << 10, 1_600_000
    x = _column(1, h_in)
    h_out = (h_in - 1) * step + 1
    out = torch.zeros((1, h_out, 1), dtype=torch.uint8, device="cuda")
    gpu.resample(x, h_out, 1, out=out)
    assert torch.equal(out[:, ::step], x)   # nodes are copied
    coarse = gpu.resample(x, (h_in - 1) * 1000 + 1, 1)
    assert torch.equal(out[:, ::step // 1000], coarse)


@pytest.mark.parametrize("c", [8, 1])
def test_doubling(gpu, c):
    # 4-row strips, 4 to a workgroup, would be 33 million workgroups
    h = (1 << 29) // c - 1
    x = _column(c, h)
    out = torch.zeros((2 * h, 2, c), dtype=torch.uint8, device="cuda").permute(2, 0, 1)
    gpu.set_launch_config(4, 1)
    try:
        gpu.zoom2x_(x, out)
    finally:
        gpu.set_launch_config(0, 0)
    for at in (0, h // 3, h // 2, h - 1000):
        ref = gpu.zoom2x(x[:, at:at + 1000].contiguous())
        assert torch.equal(out[:, 2 * at + 20:2 * at + 1980], ref[:, 20:1980])   # away from the part's clamped ends
