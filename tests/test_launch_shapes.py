"""The automatic launch shape on the host: spread byte destinations weigh a
two-column iteration alike with and without tail strips, and a shape that is
set grows where its grid would not fit a launch."""
import ctypes

import pytest

from paper_2312_00229_amd import _lib
from paper_2312_00229_amd._lib import WenoTensor


def _shape(n, h, w, dtype, sw=1, interleaved=False):
    """(rows, columns per lane, tail rows) of n planes h x w (bytes if interleaved) into dtype, columns sw apart."""
    if interleaved:
        src = WenoTensor(1 << 20, _lib.WENO_U8, 1, n, h, w, n * h * w, 1, n * w, n)
        dst = WenoTensor(1 << 40, dtype, 1, n, 2 * h, 2 * w, 4 * n * h * w, 1, 2 * n * w, n)
    else:
        src = WenoTensor(1 << 20, _lib.WENO_F32, 1, n, h, w, n * h * w, h * w, w, 1)
        dst = WenoTensor(1 << 40, dtype, 1, n, 2 * h, 2 * w, 4 * n * h * w * sw, 4 * h * w * sw, 2 * w * sw, sw)
    out = [ctypes.c_int32() for _ in range(3)]
    rc = _lib.lib().weno_query_launch_config(ctypes.byref(src), ctypes.byref(dst), *[ctypes.byref(v) for v in out])
    assert rc == _lib.WENO_OK
    return tuple(v.value for v in out)


@pytest.mark.parametrize("n,h,w", [(1, 1080, 1920), (3, 480, 640), (3, 512, 512), (12, 700, 355)])
def test_spread_bytes_with_and_without_tails(n, h, w):
    # one column per lane is cheaper by the measured cost of an iteration, tail strips or not
    _, cols, tail = _shape(n, h, w, _lib.WENO_U8, sw=2)
    assert (cols, tail) == (1, 0)
    assert _shape(n, h, w, _lib.WENO_F32, sw=2)[1] == 2


def test_rows_grow_to_fit_a_launch():
    L = _lib.lib()
    assert L.weno_set_launch_config(4, 1) == _lib.WENO_OK
    try:
        assert _shape(3, 1000, 1000, _lib.WENO_U8)[0] == 4
        for n in (1, 8):   # 2^29 rows of one column in all: 2^25 workgroups of 4-row strips, 2^23 of 16-row ones
            assert _shape(n, (1 << 29) // n - 1, 1, _lib.WENO_U8, interleaved=n > 1)[0] == 16
    finally:
        L.weno_set_launch_config(0, 0)
