"""The kernel shape that a call takes changes with its size: parity against
the fp64 oracle on both sides of each line, at odd sizes and at the smallest.

Tolerances as in the other parity tests: relative L2 1e-5 with FP32 storage,
3e-3 with FP16.
"""
import numpy as np
import pytest

import oracle
import workloads
from gpu_util import log, rel_rows, to_dev, to_host, widen

pytestmark = pytest.mark.gpu

TOL = {0: 1e-5, 1: 3e-3}


@pytest.fixture(scope="module")
def api():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2609_32237_amd import torch_api

    return torch_api


def run_columns(api, n, count, pad, storage, direction=-1):
    """The first `count` columns of an n x (count + pad) matrix, and the oracle's."""
    import torch

    x = workloads.uniform_complex(n, count + pad, 31 + count, "fp16" if storage else "fp32")
    xd = to_dev(x)
    out = torch.full_like(xd, 7.0)
    plan = api.Plan(n, count, count + pad, 1, storage, direction)
    plan.execute(xd, out)
    torch.cuda.synchronize()
    plan.close()
    got = widen(to_host(out))
    assert np.all(got[:, count:] == (7.0 + 7.0j if storage else 7.0)), "columns outside the batch were written"
    ref = oracle.fft(np.ascontiguousarray(np.moveaxis(x[:, :count], 0, 1)), direction)
    return got[:, :count].T, ref


@pytest.mark.parametrize("storage", [0, 1])
@pytest.mark.parametrize("count,pad", [(1, 0), (5, 3), (1023, 1), (1024, 0), (1025, 2)])
def test_few_columns_of_4096(api, storage, count, pad):
    """Up to 1024 columns of 4096 points take the 4-column strips, more the
    8-column ones; a strip's last columns may be missing."""
    got, ref = run_columns(api, 4096, count, pad, storage)
    e = rel_rows(got, ref).max()
    log(f"columns 4096 x {count} storage {storage}: rel {e:.2e}")
    assert e < TOL[storage]
