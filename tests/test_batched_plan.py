"""Batched plans on the host: what a run refuses."""
import ctypes

import pytest

from paper_2312_00229_amd import _lib
from paper_2312_00229_amd._lib import WenoBatchPlan


@pytest.mark.parametrize("modes", [0, -1, 1 << 8, 1 << 62])
def test_run_refuses_a_plan_without_modes(modes):
    # all other fields as a plan leaves them; nothing is launched
    plan = WenoBatchPlan(0x300000, 4096, 10, 2, 32, 2, 2, modes)
    assert _lib.lib().weno_zoom2x_batched_run(ctypes.byref(plan), None) == _lib.WENO_EINVAL
