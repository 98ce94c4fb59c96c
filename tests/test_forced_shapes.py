"""Kernel shapes forced through the environment: an index that a pass cannot
run is refused when the plan is made, before any HIP call."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


# 2^22 = 2048 x 2048: the first pass multiplies by the four-step factors, which
# the 64-point shapes (the last two of the 2048-point columns) do not do
@pytest.mark.parametrize("n,variant,refused", [(1 << 22, 0, False), (1 << 22, 2, False), (1 << 22, 3, True),
                                               (1 << 22, 4, True), (1 << 22, 5, True), (1 << 21, 3, True),
                                               (1 << 18, 1, False), (1 << 18, 2, True)])
def test_forced_column_shape_of_a_long_transform(n, variant, refused):
    code = ("import ctypes\n"
            "from paper_2609_32237_amd import _lib as L\n"
            "p = ctypes.c_void_p()\n"
            f"print(L.lib.fft_plan_create({n}, 1, 1, {n}, 0, -1, ctypes.byref(p)))\n")
    # the allocation that follows the checks is made to fail (-3)
    env = dict(os.environ, MI355FFT_COL_VARIANT=str(variant), MI355FFT_TEST_FAIL_ALLOC="1")
    res = subprocess.run([sys.executable, "-c", code], cwd=ROOT, env=env, capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res.stderr
    assert int(res.stdout.split()[0]) == (-1 if refused else -3)
