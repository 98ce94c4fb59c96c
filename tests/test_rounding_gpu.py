"""What FP32 arithmetic owes its input beyond the parity bounds: outputs that
are finite stay finite, however near the type's limit their neighbours are, and
the rounding error against FP64 stays where the shapes with the most accurate
factors put it, an order of magnitude inside those bounds.
"""
import numpy as np
import pytest

from gpu_util import log, to_dev, to_host

pytestmark = pytest.mark.gpu

FLT_MAX = float(np.finfo(np.float32).max)


@pytest.fixture(scope="module")
def api():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2609_32237_amd import torch_api

    return torch_api


# Two points h = n/2 apart, equal and real, of value 2e38: every odd output is
# their difference, exactly 0, and every even one overflows.  Points 1 and 0
# instead: output k is 2e38 (1 + W^k), of which the part near k = n/2 is small
# although the other overflows half a turn away.  No sum on the way to a
# finite output is larger than that output's terms, so a transform that forms
# each output of a butterfly from its inputs keeps all outputs whose components
# stay below half of FLT_MAX finite and accurate.
@pytest.mark.parametrize("gap", ["half", "one"])
@pytest.mark.parametrize("direction", [-1, 1])
@pytest.mark.parametrize("layout,n,count", [
    ("rows", 1024, 3), ("rows", 1024, 4100), ("rows", 2048, 5), ("rows", 4096, 3), ("rows", 8192, 3),
    ("rows", 8192, 5000), ("rows", 16384, 20), ("rows", 16384, 600), ("rows", 65536, 1), ("cols", 1024, 5), ("cols", 1024, 8200),
    ("cols", 2048, 3), ("cols", 2048, 2100), ("cols", 2048, 4100), ("cols", 4096, 5), ("cols", 4096, 1100),
    ("in", 8192, 3), ("in", 8192, 600), ("in", 8192, 1100), ("in", 16384, 3), ("in", 16384, 300)])
def test_finite_outputs_near_the_limit(api, layout, n, count, direction, gap):
    import torch

    j = n // 2 if gap == "half" else 1
    x = np.zeros((n, 1), np.complex64)
    x[[0, j]] = 2e38
    k = np.arange(n)
    ref = 2e38 * (1.0 + np.exp(direction * 2j * np.pi * (k * j % n) / n))
    if gap == "half":
        ref[1::2] = 0.0
    xd = to_dev(x).expand(n, count).contiguous()
    if layout == "rows":
        xd = xd.t().contiguous()
    out = xd if layout == "in" else torch.empty_like(xd)
    plan = api.Plan(n, count, *((1, n) if layout == "rows" else (count, 1)), 0, direction)
    plan.execute(xd, out)
    torch.cuda.synchronize()
    plan.close()
    y = to_host(out[[0, -1]] if layout == "rows" else out[:, [0, -1]].t().contiguous()).astype(np.complex128)
    safe = np.maximum(abs(ref.real), abs(ref.imag)) < FLT_MAX / 2
    assert safe.sum() >= n // 4
    bad = ~np.isfinite(y[:, safe])
    log(f"{layout} {n} x {count} dir {direction} gap {gap}: {bad.sum()} of {2 * safe.sum()} not finite")
    assert not bad.any()
    # relative to the input's size: log2(n) roundings of 2^-24
    assert np.abs(y[:, safe] - ref[safe]).max() < 2e38 * np.log2(n) * 2.0**-23


@pytest.mark.parametrize("n", [1024, 4096, 16384])
def test_infinite_fp16_input(api, n):
    """An infinite point leaves no finite output in its row and does not touch
    the rows beside it (FP16 data, whose butterflies double)."""
    import torch

    rng = np.random.default_rng(n)
    x = rng.uniform(-1, 1, (20, n, 2)).astype(np.float16)
    y0 = to_host(api.fft(to_dev(x)))
    x[7, 5, 0] = np.inf
    y = to_host(api.fft(to_dev(x)))
    torch.cuda.synchronize()
    assert not np.isfinite(y[7].astype(np.float32)).all(-1).any()
    rest = np.arange(20) != 7
    assert np.array_equal(y[rest].view(np.uint16), y0[rest].view(np.uint16))


# Bounds in 1e-7 on the relative L2 error against FP64: the error measured of
# one shape of each length with its factors read or formed as digit products,
# plus 0.5%.  Over the 2^17 points or more of a case the sample itself spreads
# by less than 0.2%.
@pytest.mark.parametrize("layout,n,count,bound", [
    ("rows", 1024, 1025, 1.313), ("rows", 1024, 4100, 1.313), ("rows", 2048, 513, 1.400), ("rows", 4096, 300, 1.525),
    ("rows", 8192, 100, 1.414), ("rows", 8192, 4100, 1.414), ("rows", 16384, 65, 1.510), ("rows", 16384, 300, 1.510),
    ("cols", 1024, 700, 1.313), ("cols", 1024, 8192, 1.313), ("cols", 2048, 300, 1.400), ("cols", 2048, 2100, 1.400),
    ("cols", 2048, 4100, 1.400), ("cols", 4096, 250, 1.478), ("cols", 4096, 1100, 1.478), ("in", 8192, 100, 1.572),
    ("in", 8192, 700, 1.572), ("in", 8192, 1100, 1.572), ("in", 16384, 64, 1.660), ("in", 16384, 300, 1.660)])
def test_rounding_error(api, layout, n, count, bound):
    import torch

    g = torch.Generator(device="cuda").manual_seed(n + count)
    shape = (count, n) if layout == "rows" else (n, count)
    x = torch.view_as_complex(torch.empty(*shape, 2, device="cuda").uniform_(-1.0, 1.0, generator=g))
    out = x.clone() if layout == "in" else torch.empty_like(x)
    plan = api.Plan(n, count, *((1, n) if layout == "rows" else (count, 1)), 0, -1)
    plan.execute(out if layout == "in" else x, out)
    torch.cuda.synchronize()
    plan.close()
    few = max(1, (1 << 20) // n)  # the first 2^20 points, or all
    x, out = (x[:few], out[:few]) if layout == "rows" else (x[:, :few].t(), out[:, :few].t())
    ref = np.fft.fft(to_host(x.contiguous()).astype(np.complex128), axis=1)
    e = np.linalg.norm(to_host(out.contiguous()) - ref) / np.linalg.norm(ref)
    log(f"{layout} {n} x {count}: {e:.4e}")
    assert e < bound * 1e-7


# The same for SAR images with an FP32 intermediate, whose two transforms per
# axis share their twiddles: a factor's rounding counts twice.  Bounds as
# above, from shapes of the same kind, plus 1.5%: one reference chirp's
# spectrum, of as many values as the axis has points, is in every image point
# (seeds differ by 0.5%).
@pytest.mark.parametrize("n_az,n_rg,bound", [(1024, 1024, 3.99), (1024, 16384, 4.68), (4096, 1024, 4.39),
                                             (8192, 1024, 5.01), (16384, 1024, 4.76)])
def test_rounding_error_of_images(api, n_az, n_rg, bound):
    import torch

    g = torch.Generator(device="cuda").manual_seed(n_az + n_rg)

    def rnd(*shape):
        return torch.view_as_complex(torch.empty(*shape, 2, device="cuda").uniform_(-1.0, 1.0, generator=g))

    raw, h_rg, h_az = rnd(n_az, n_rg), rnd(n_rg), rnd(n_az)
    img = to_host(api.sar_form_image(raw, h_rg, h_az, 0))
    ref = np.fft.fft2(to_host(raw).astype(np.complex128))
    ref *= np.fft.fft(to_host(h_rg).astype(np.complex128)).conj()[None, :]
    ref *= np.fft.fft(to_host(h_az).astype(np.complex128)).conj()[:, None]
    ref = np.fft.ifft2(ref)
    e = np.linalg.norm(img - ref) / np.linalg.norm(ref)
    log(f"sar {n_az} x {n_rg}: {e:.4e}")
    assert e < bound * 1e-7
