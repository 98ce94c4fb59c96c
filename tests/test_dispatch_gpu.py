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


def run_columns(api, n, count, pad, storage, direction=-1, in_place=False):
    """The first `count` columns of an n x (count + pad) matrix, and the
    oracle's: all of them, or the first, the last and 14 more."""
    import torch

    x = workloads.uniform_complex(n, count + pad, 31 + count, "fp16" if storage else "fp32")
    xd = to_dev(x)
    out = xd if in_place else torch.full_like(xd, 7.0)
    plan = api.Plan(n, count, count + pad, 1, storage, direction)
    plan.execute(xd, out)
    torch.cuda.synchronize()
    plan.close()
    y = to_host(out)
    outside = x[:, count:] if in_place else np.full_like(x[:, count:], 7.0)
    assert np.array_equal(y[:, count:], outside), "columns outside the batch were written"
    pick = np.arange(count) if count <= 32 else np.unique(
        np.r_[0, count - 1, np.random.default_rng(count).integers(0, count, 14)])
    ref = oracle.fft(np.ascontiguousarray(np.moveaxis(x[:, pick], 0, 1)), direction)
    return np.ascontiguousarray(widen(np.ascontiguousarray(y[:, pick])).T), ref


@pytest.mark.parametrize("storage", [0, 1])
@pytest.mark.parametrize("n,count,pad", [(1024, 3, 2), (1024, 8191, 1), (1024, 8192, 0),
                                         (2048, 2047, 3), (2048, 2049, 0), (2048, 4095, 1), (2048, 4100, 0),
                                         (2048, 8191, 1), (2048, 8193, 0),
                                         (4096, 1, 0), (4096, 5, 3), (4096, 1023, 1), (4096, 1024, 0), (4096, 1025, 2)])
def test_columns_by_count(api, storage, n, count, pad):
    """The strip width (4, 8 or 16 columns) goes with the number of columns;
    a strip's last columns may be missing."""
    got, ref = run_columns(api, n, count, pad, storage)
    e = rel_rows(got, ref).max()
    log(f"columns {n} x {count} storage {storage}: rel {e:.2e}")
    assert e < TOL[storage]


@pytest.mark.parametrize("storage", [0, 1])
@pytest.mark.parametrize("n,count", [(8192, 1), (8192, 511), (8192, 514), (8192, 1025), (16384, 3), (16384, 255),
                                     (16384, 257)])
def test_long_columns_in_place(api, storage, n, count):
    """8192 and 16384 points in place: single passes of 1, 2 or 4 columns."""
    got, ref = run_columns(api, n, count, 1, storage, 1, True)
    e = rel_rows(got, ref).max()
    log(f"columns in place {n} x {count} storage {storage}: rel {e:.2e}")
    assert e < TOL[storage]


@pytest.mark.parametrize("storage", [0, 1])
@pytest.mark.parametrize("log2n,batch", [(16, 127), (16, 128), (18, 63), (18, 65), (20, 7), (20, 8), (21, 1), (21, 2)])
def test_long_transforms_by_batch(api, storage, log2n, batch):
    """The four-step passes' strips go with the columns of all transforms."""
    import torch

    n = 1 << log2n
    x = workloads.uniform_complex(batch, n, 77 + batch, "fp16" if storage else "fp32")
    xd = to_dev(x)
    plan = api.Plan(n, batch, 1, n, storage, -1, log2n // 2 if storage else 0)
    y = plan.execute(xd, torch.empty_like(xd))
    torch.cuda.synchronize()
    plan.close()
    pick = np.unique([0, batch // 2, batch - 1])
    got = widen(to_host(y[torch.from_numpy(pick).cuda()]))
    ref = oracle.fft(x[pick]) * (2.0 ** -(log2n // 2) if storage else 1.0)
    e = rel_rows(got, ref).max()
    log(f"long 2^{log2n} x {batch} storage {storage}: rel {e:.2e}")
    assert e < TOL[storage]


@pytest.mark.parametrize("inter", [0, 1])
@pytest.mark.parametrize("shape", [(2048, 8192), (1024, 8192), (16384, 4096)])
def test_images_by_shape(api, shape, inter):
    """Azimuth passes whose strips or form go with the image's width (the
    three-pass form at 16384 x 4096 with an FP32 intermediate)."""
    n_az, n_rg = shape
    sc = workloads.sar_scene(n_az=n_az, n_rg=n_rg, n_targets=4, len_rg=256, len_az=128, sigma=0.0, seed=3, min_sep=24)
    import torch

    img = to_host(api.sar_form_image(to_dev(sc.raw), to_dev(sc.range_ref), to_dev(sc.az_ref), inter))
    torch.cuda.synchronize()
    ref = oracle.sar_chain(sc.raw, sc.range_ref, sc.az_ref)
    img -= ref.astype(np.complex64)
    e = np.linalg.norm(img) / np.linalg.norm(ref)
    log(f"sar {n_az}x{n_rg} inter {inter}: rel {e:.2e}")
    assert e < TOL[inter]


@pytest.mark.parametrize("storage", [0, 1])
@pytest.mark.parametrize("n,batch", [(1024, 1), (1024, 1027), (2048, 511), (2048, 513), (4096, 1025), (8192, 1),
                                     (8192, 4096), (8192, 4097), (16384, 17), (16384, 512), (16384, 513)])
def test_rows_by_batch(api, storage, n, batch):
    """Row shapes on both sides of their batch limits, odd batches and one."""
    import torch

    x = workloads.uniform_complex(batch, n, 5 + batch, "fp16" if storage else "fp32")
    y = api.fft(to_dev(x), 1)
    torch.cuda.synchronize()
    pick = np.unique(np.r_[0, batch - 1, np.random.default_rng(batch).integers(0, batch, 10)])
    got = widen(to_host(y[torch.from_numpy(pick).cuda()]))
    e = rel_rows(got, oracle.fft(x[pick], 1)).max()
    log(f"rows {n} x {batch} storage {storage}: rel {e:.2e}")
    assert e < TOL[storage]


@pytest.mark.parametrize("storage", [0, 1])
@pytest.mark.parametrize("n,batch", [(1024, 3072), (1024, 3073), (1024, 4096), (1024, 4097), (1024, 12287),
                                     (1024, 12289), (4096, 2048), (4096, 2049), (16384, 127), (16384, 128)])
def test_rows_by_batch_limits(api, storage, n, batch):
    """Both sides of the remaining batch limits of the row shapes."""
    test_rows_by_batch(api, storage, n, batch)


@pytest.mark.parametrize("storage", [0, 1])
@pytest.mark.parametrize("n,count", [(8192, 512), (8192, 513)])
def test_long_columns_at_the_strip_limit(api, storage, n, count):
    """512 columns of 8192 points: 256 strips of two."""
    test_long_columns_in_place(api, storage, n, count)


@pytest.mark.parametrize("log2n,batch", [(17, 255), (17, 256), (18, 128), (22, 15), (22, 16)])
def test_long_transforms_at_the_strip_limits(api, log2n, batch):
    """FP32 passes of 512-point columns around 65536 of them, and of 2048-point
    columns in rows of 2048 around 32768."""
    import torch

    n = 1 << log2n
    g = torch.Generator(device="cuda").manual_seed(batch)
    x = torch.view_as_complex(torch.empty(batch, n, 2, device="cuda").uniform_(-1.0, 1.0, generator=g))
    plan = api.Plan(n, batch, 1, n, 0, -1)
    y = plan.execute(x, torch.empty_like(x))
    torch.cuda.synchronize()
    plan.close()
    pick = np.unique([0, batch // 2, batch - 1])
    at = torch.from_numpy(pick).cuda()
    e = rel_rows(widen(to_host(y[at])), oracle.fft(to_host(x[at]))).max()
    log(f"long 2^{log2n} x {batch}: rel {e:.2e}")
    assert e < TOL[0]


RD_SHAPES = {
    (1024, 8192): dict(pulse_samples=600, targets=((256, 300, 1.0), (512, 4400, 1.0), (768, 7000, 0.6))),
    (1024, 16384): dict(pulse_samples=600, targets=((256, 300, 1.0), (512, 15000, 1.0))),
    (2048, 4096): dict(prf=250.0, targets=((512, 128, 1.0), (1024, 2640, 1.0), (1536, 3384, 0.8))),
    (2048, 8192): dict(prf=250.0, targets=((512, 128, 1.0), (1024, 5640, 1.0), (1536, 7384, 0.8))),
}


@pytest.mark.parametrize("shape", sorted(RD_SHAPES))
def test_range_doppler_by_shape(api, shape):
    """The scaled azimuth pass, written transposed, on both sides of its strip
    limits (1024 pulses from 8192 range bins, 2048 from 4096 and 8192), and the
    range pass at 8192 and 16384 bins; each with either intermediate."""
    import torch

    n_az, n_rg = shape
    args = dict(prf=125.0)
    args.update(RD_SHAPES[shape])
    sc = workloads.rd_scene_small(n_az=n_az, n_rg=n_rg, **args)
    ref = oracle.rd_chain(sc.raw, sc.range_ref, sc.geometry)
    raw, range_ref = to_dev(sc.raw), to_dev(sc.range_ref)
    for inter in (0, 1):
        got = to_host(api.sar_rd_form_image(raw, range_ref, sc.geometry, inter))
        torch.cuda.synchronize()
        e = np.linalg.norm(got - ref) / np.linalg.norm(ref)
        log(f"rd {n_az} x {n_rg} inter {inter}: rel {e:.2e}")
        assert e < TOL[inter]
        for a, r in zip(sc.targets_az, sc.targets_rg):
            win = np.abs(got[a - 8:a + 9, r - 8:r + 9])
            assert np.unravel_index(np.argmax(win), win.shape) == (8, 8), (a, r)
