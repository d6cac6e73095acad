"""The resampler at the edges of its launch shapes, against the FP64 oracle:
tiles of 64 to 256 columns and 64 to 256 input columns, width and height
ratios on both sides of 4 (where the kernel changes), single rows and columns,
nodes, every pair of types, planar and interleaved."""
import numpy as np
import pytest
import torch

import oracle
from conftest import check_u8
from oracle import resample as R

pytestmark = pytest.mark.gpu

SHAPES = [
    (1, 1, 7, 9), (1, 40, 3, 333), (40, 1, 90, 2), (2, 2, 2, 2), (17, 300, 17, 300),      # lines, copies
    (9, 61, 30, 1000), (30, 100, 61, 257), (30, 190, 29, 256), (30, 189, 31, 255),        # up: 256-column tiles
    (33, 254, 25, 190), (33, 255, 25, 191), (33, 256, 25, 192), (40, 700, 31, 525),       # 4/3: 190-column tiles
    (64, 253, 16, 64), (65, 256, 16, 64), (68, 257, 17, 65), (64, 300, 17, 74),           # ratios about 4
    (400, 90, 99, 90), (300, 61, 40, 183), (57, 500, 200, 40), (129, 129, 65, 257),       # nodes at every second row
]


@pytest.mark.parametrize("shape", SHAPES)
def test_shapes_against_oracle(gpu, shape):
    h, w, oh, ow = shape
    rng = np.random.default_rng(h * 1000 + ow)
    codes = rng.integers(0, 256, size=(3, h, w)).astype(np.uint8)
    V8, V32 = codes.astype(np.float64) / 255.0, rng.random((3, h, w), dtype=np.float32)
    for beta in (2.0, 1.5):
        p = gpu.Params(beta=beta)
        x = torch.tensor(V32, device="cuda")
        ref = R.tensor_resample(V32.astype(np.float64), oh, ow, beta=beta)
        got = gpu.resample(x, oh, ow, p).cpu().numpy()
        assert np.abs(got - ref).max() <= 1e-5
        # interleaved: the same bits
        xi = x.permute(1, 2, 0).contiguous().permute(2, 0, 1)
        assert np.array_equal(gpu.resample(xi, oh, ow, p).cpu().numpy(), got)
        check_u8(gpu.resample(x, oh, ow, p, out_dtype=torch.uint8).cpu().numpy(), ref, "f32 -> u8 %s" % (shape,))
        x8 = torch.tensor(codes, device="cuda")
        ref8 = R.tensor_resample(V8, oh, ow, beta=beta)
        got8 = gpu.resample(x8, oh, ow, p).cpu().numpy()
        check_u8(got8, ref8, "u8 %s" % (shape,))
        assert np.abs(gpu.resample(x8, oh, ow, p, out_dtype=torch.float32).cpu().numpy() - ref8).max() <= 1e-5
        x8i = x8.permute(1, 2, 0).contiguous().permute(2, 0, 1)
        assert np.array_equal(gpu.resample(x8i, oh, ow, p).cpu().numpy(), got8)
