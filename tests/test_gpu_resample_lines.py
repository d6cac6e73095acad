"""The resampler's tiles of whole 128-byte lines (large float32 launches whose
output rows start on lines): the same bits as an output that starts inside a
line, whose tiles are cut evenly, and the FP64 oracle's values."""
import numpy as np
import pytest
import torch

from oracle import resample as R

pytestmark = pytest.mark.gpu

# 24 planes of 3000 rows: over 64 rows of tiles for each SIMD, whatever the width
WIDTHS = [(40, 32), (100, 64), (61, 96), (300, 192), (190, 256), (259, 256), (400, 288), (250, 320), (333, 576),
          (1100, 288), (700, 704)]


@pytest.mark.parametrize("w,ow", WIDTHS)
def test_whole_line_tiles(gpu, w, ow):
    h, oh, shape = 1500, 3000, (8, 3, 3000, ow)
    gen = torch.Generator(device="cuda").manual_seed(w)
    x = torch.rand(8, 3, h, w, device="cuda", generator=gen)
    size = 24 * oh * ow
    line = torch.full((size,), -1.0, device="cuda").view(shape)
    inside = torch.full((size + 2,), -1.0, device="cuda")
    assert line.data_ptr() % 128 == 0
    gpu.resample(x, oh, ow, out=line)
    gpu.resample(x, oh, ow, out=inside[1:-1].view(shape))
    assert torch.equal(line.view(-1), inside[1:-1])
    assert inside[0] == -1.0 and inside[-1] == -1.0
    ref = R.tensor_resample(x[7, 2:].cpu().numpy().astype(np.float64), oh, ow, beta=2.0)
    assert np.abs(line[7, 2:].cpu().numpy() - ref).max() <= 1e-5
