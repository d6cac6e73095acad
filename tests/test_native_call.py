"""The binding's native call path against its general one: the same outputs,
layouts and errors with and without it."""
import numpy as np
import pytest
import torch

import paper_2312_00229_amd as wz


@pytest.fixture(params=["native", "general"])
def path(request, monkeypatch):
    if request.param == "general":
        monkeypatch.setattr(wz, "_native", None)
    else:
        assert wz._native is not None, "build the package: _native.so is missing"
    return request.param


def test_errors_on_the_cpu(path):
    x = torch.zeros(3, 8, 8)
    for call in (lambda: wz.zoom2x(x), lambda: wz.zoom2x_(x, torch.zeros(3, 16, 16)),
                 lambda: wz.zoom2x_backward(x, torch.zeros(3, 16, 16))):
        with pytest.raises(ValueError, match="tensors must live on the GPU"):
            call()
    with pytest.raises(IndexError):
        wz.zoom2x(torch.zeros(4))
    with pytest.raises(ValueError):
        wz.zoom2x(x, boundary="wrap")


class _Tagged(torch.Tensor):
    pass


@pytest.mark.gpu
def test_same_outputs_and_layouts(gpu, monkeypatch):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    base = torch.rand((4, 3, 40, 52), generator=gen, device="cuda")
    xs = [base[0, 0], base[0], base, base[:, :, 3:30, 1:40:2], base[0].permute(1, 2, 0).contiguous().permute(2, 0, 1),
          base.contiguous(memory_format=torch.channels_last), base[1, 1].t(), base[0, :1], (255 * base[2]).byte(),
          (255 * base[0, 0]).byte(), base[0].as_subclass(_Tagged), torch.nn.Parameter(base[3])]
    for x in xs:
        for dtype in (None, torch.uint8, torch.float32):
            with torch.no_grad():
                got = wz.zoom2x(x, out_dtype=dtype, beta=1.5)
                into = torch.empty_like(got)
                assert wz.zoom2x_(x, into, beta=1.5) is into
                with monkeypatch.context() as m:
                    m.setattr(wz, "_native", None)
                    ref = wz.zoom2x(x, out_dtype=dtype, beta=1.5)
            assert (got.shape, got.stride(), got.dtype) == (ref.shape, ref.stride(), ref.dtype)
            assert torch.equal(got, ref) and torch.equal(into, ref)
        if x.dtype == torch.float32:
            g = torch.rand(ref.shape, generator=gen, device="cuda")
            with torch.no_grad():
                gx = wz.zoom2x_backward(x, g)
                with monkeypatch.context() as m:
                    m.setattr(wz, "_native", None)
                    assert torch.equal(wz.zoom2x_backward(x, g), gx)


@pytest.mark.gpu
def test_same_errors(gpu, path):
    x = torch.rand((3, 8, 8), device="cuda")
    with pytest.raises(ValueError, match="dtype must be uint8 or float32"):
        gpu.zoom2x(x.double())
    with pytest.raises(ValueError, match="2, 3 or 4 dims"):
        gpu.zoom2x(x[None, None])
    for call in (lambda: gpu.zoom2x_(x, torch.empty((3, 16, 15), device="cuda")), lambda: gpu.zoom2x(x[:, :0]),
                 lambda: gpu.zoom2x(x, beta=-1.0), lambda: gpu.zoom2x_backward(x, x)):
        with pytest.raises(gpu.WenoError) as e:
            call()
        assert e.value.status == -1
    buf = torch.rand((3, 24, 24), device="cuda")
    with pytest.raises(gpu.WenoError) as e:
        gpu.zoom2x_(buf[:, :8, :8], buf[:, :16, :16])
    assert e.value.status == -3


@pytest.mark.gpu
def test_current_stream(gpu, path):
    # the call goes to torch's current stream: ordered after the work on it
    side = torch.cuda.Stream()
    big = torch.rand((4096, 4096), device="cuda")
    x = torch.zeros((3, 64, 64), device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        for _ in range(4):
            big = big @ big * 1e-3
        x += 0.25
        out = gpu.zoom2x(x)
    side.synchronize()
    assert np.array_equal(out.cpu().numpy(), np.full((3, 128, 128), 0.25, np.float32))
