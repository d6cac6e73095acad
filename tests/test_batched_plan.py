"""Batched plans on the host: what a run refuses, and a plan that runs out of host
memory."""
import ctypes
import os
import subprocess
import sys

import pytest

from paper_2312_00229_amd import _lib
from paper_2312_00229_amd._lib import WenoBatchPlan


@pytest.mark.parametrize("modes", [0, -1, 1 << 8, 1 << 62])
def test_run_refuses_a_plan_without_modes(modes):
    # all other fields as a plan leaves them; nothing is launched
    plan = WenoBatchPlan(0x300000, 4096, 10, 2, 32, 2, 2, modes)
    assert _lib.lib().weno_zoom2x_batched_run(ctypes.byref(plan), None) == _lib.WENO_EINVAL


_SHORT_OF_MEMORY = """
import ctypes, resource, sys
from paper_2312_00229_amd import _lib
from paper_2312_00229_amd._lib import WenoBatchPlan, WenoParams, WenoTensor
L, n = _lib.lib(), 1 << 18
src, dst = (WenoTensor * n)(), (WenoTensor * n)()
for i in range(n):
    src[i] = WenoTensor((1 << 30) + 256 * i, 1, 1, 1, 2, 2, 4, 4, 2, 1)
    dst[i] = WenoTensor((1 << 40) + 256 * i, 1, 1, 1, 4, 4, 16, 16, 4, 1)
p, plan = WenoParams(2.0, 1e-8, 1.0, -1.0, 0), WenoBatchPlan()
ws = L.weno_zoom2x_batched_workspace(n)
args = (src, dst, n, ctypes.byref(p), 1 << 29, ws, None, ctypes.byref(plan))
used = int(open("/proc/self/statm").read().split()[0]) * resource.getpagesize()
resource.setrlimit(resource.RLIMIT_AS, (used + (int(sys.argv[1]) << 20),) * 2)
print(L.weno_zoom2x_batched_plan(*args), _lib.status_string(_lib.WENO_EHIP))
"""


@pytest.mark.parametrize("mib", [6, 30])   # short in the checks, and in the table
def test_host_memory_that_runs_out_is_an_error(mib):
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    res = subprocess.run([sys.executable, "-c", _SHORT_OF_MEMORY, str(mib)], cwd=root, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    assert res.stdout.startswith("%d " % _lib.WENO_EHIP) and "host memory" in res.stdout
