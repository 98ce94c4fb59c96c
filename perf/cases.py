"""The work that a program has this library do, as cases that can be timed and checked.

Every case goes through the public entry points: ``torch_api.Plan`` (batched
FFTs of contiguous rows, of strided columns, and of transforms longer than the
chip holds), ``torch_api.sar_form_image`` (the two-pass SAR chain) and
``torch_api.sar_rd_form_image`` (the full range-Doppler chain).  Plans, output
buffers and workspaces are made once, as a program that processes one batch or
image after another keeps them; ``run`` is one call.

``exact`` gives the same results in 64 bits from plain torch, on its own.
"""
import math

import torch

from paper_2609_32237_amd import torch_api as mf

C_LIGHT = 299_792_458.0
FP32, FP16 = 0, 1


def listed():
    return [
        # one small batch, as an interactive or real-time caller issues it: latency and launches count
        dict(name="rows_1024x64_fp32", kind="rows", n=1024, count=64, pad=0, storage=FP32, inverse=False, shift=0),
        # a medium, ragged batch in half storage, inverse, with the block-floating-point output shift
        dict(name="rows_2048x1501_fp16_inv", kind="rows", n=2048, count=1501, pad=0, storage=FP16, inverse=True, shift=6),
        # large batches from device memory: the library's headline sizes, both directions, both storages
        dict(name="rows_4096x32768_fp32", kind="rows", n=4096, count=32768, pad=0, storage=FP32, inverse=False, shift=0),
        dict(name="rows_8192x16384_fp32_inv", kind="rows", n=8192, count=16384, pad=0, storage=FP32, inverse=True, shift=0),
        dict(name="rows_16384x16384_fp16", kind="rows", n=16384, count=16384, pad=0, storage=FP16, inverse=False, shift=0),
        # transforms longer than the chip holds: an odd batch of the shorter ones, inverse, and the benchmark's
        dict(name="rows_65536x333_fp32_inv", kind="rows", n=65536, count=333, pad=0, storage=FP32, inverse=True, shift=0),
        dict(name="rows_1048576x128_fp32", kind="rows", n=1048576, count=128, pad=0, storage=FP32, inverse=False, shift=0),
        # the columns of a row-major matrix (the second axis of a 2-D transform)
        dict(name="cols_4096x4096_fp32", kind="cols", n=4096, count=4096, pad=0, storage=FP32, inverse=False, shift=0),
        # one SAR image from its echo, intermediates in either precision
        dict(name="sar_4096x4096_fp32", kind="sar", n_az=4096, n_rg=4096, inter=FP32, chirp_rg=1024, chirp_az=512),
        dict(name="sar_4096x4096_fp16", kind="sar", n_az=4096, n_rg=4096, inter=FP16, chirp_rg=1024, chirp_az=512),
        # one range-Doppler image with migration correction (L-band stripmap scene)
        dict(name="rd_4096x4096_fp32", kind="rd", n_az=4096, n_rg=4096, inter=FP32, wavelength=0.24, speed=200.0,
             prf=500.0, antenna=8.0, r_near=17500.0, pulse=1200),
        dict(name="rd_4096x4096_fp16", kind="rd", n_az=4096, n_rg=4096, inter=FP16, wavelength=0.24, speed=200.0,
             prf=500.0, antenna=8.0, r_near=17500.0, pulse=1200),
    ]


def draw(rng):
    kind = rng.choice(["rows", "rows", "rows", "long", "cols", "sar", "rd"])
    if kind in ("rows", "long", "cols"):
        storage = rng.choice([FP32, FP16])
        n = 1 << (rng.randint(15, 23) if kind == "long" else rng.randint(10, 14))
        # the whole batch: 2^16 points (one long transform) to 2^27 (2^25 down columns)
        lo, hi = max(16.0, math.log2(n)), 25.0 if kind == "cols" else 27.0
        count = max(1, int(2.0 ** rng.uniform(lo, hi) / n))
        pad = rng.choice([0, 0, 0, rng.randint(1, 40)])
        return dict(kind="cols" if kind == "cols" else "rows", n=n, count=count, pad=pad, storage=storage,
                    inverse=rng.random() < 0.5, shift=rng.choice([0, n.bit_length() // 2]) if storage == FP16 else 0)
    az, rg = rng.randint(10, 14), rng.randint(10, 14)
    while az + rg > 24:
        az, rg = rng.randint(10, 14), rng.randint(10, 14)
    case = dict(kind=kind, n_az=1 << az, n_rg=1 << rg, inter=rng.choice([FP32, FP16]))
    if kind == "sar":
        case.update(chirp_rg=2 * rng.randint(64, case["n_rg"] // 4), chirp_az=2 * rng.randint(64, case["n_az"] // 4))
    else:
        while True:
            wavelength, speed, antenna = rng.choice([0.24, 0.056, 0.031]), rng.uniform(150.0, 250.0), rng.choice([4.0, 8.0, 12.0])
            prf = rng.uniform(1.3, 4.0) * 2.0 * speed / antenna
            if wavelength * prf / (4.0 * speed) < 0.33:
                break
        case.update(wavelength=wavelength, speed=speed, prf=prf, antenna=antenna, r_near=rng.uniform(6e3, 25e3),
                    pulse=rng.randint(100, case["n_rg"] // 3))
    return case


# ---------------------------------------------------------------- inputs


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _batch(case, seed):
    """Uniform complex values on [-1, 1) in the case's layout: one array (rows, row length), padded rows."""
    rows, cols = (case["count"], case["n"]) if case["kind"] == "rows" else (case["n"], case["count"])
    x = torch.empty(rows, cols + case["pad"], 2, device="cuda").uniform_(-1.0, 1.0, generator=_generator(seed))
    return x.half() if case["storage"] == FP16 else torch.view_as_complex(x)


def _chirp(n, length, device="cuda"):
    """Centred linear-FM chirp spanning 0.8 of the band, wrapped to index t mod n."""
    t = torch.arange(-(length // 2), length // 2, dtype=torch.float64, device=device)
    h = torch.zeros(n, dtype=torch.complex128, device=device)
    h[t.long() % n] = torch.polar(torch.ones_like(t), math.pi * 0.8 * t * t / length)
    return h


def _noise(shape, g):
    return torch.view_as_complex(torch.empty(*shape, 2, device="cuda").normal_(0.0, 0.01, generator=g))


def _sar_scene(case, seed):
    """Echo of 32 separable point targets in noise, and the two reference chirps."""
    n_az, n_rg, g = case["n_az"], case["n_rg"], _generator(seed)
    h_rg, h_az = _chirp(n_rg, case["chirp_rg"]), _chirp(n_az, case["chirp_az"])
    at = torch.rand(3, 32, device="cuda", generator=g)
    az, rg, amp = (at[0] * n_az).long(), (at[1] * n_rg).long(), 0.5 + 0.5 * at[2]
    rows = h_az[(torch.arange(n_az, device="cuda")[None, :] - az[:, None]) % n_az].to(torch.complex64)
    cols = h_rg[(torch.arange(n_rg, device="cuda")[None, :] - rg[:, None]) % n_rg].to(torch.complex64)
    raw = _noise((n_az, n_rg), g)
    for k in range(32):
        raw.addcmul_((rows[k] * amp[k])[:, None], cols[k][None, :])
    return raw, h_rg.to(torch.complex64), h_az.to(torch.complex64)


def _rd_scene(case, seed):
    """Broadside stripmap echo of six point targets in noise (start-stop approximation), and the pulse replica."""
    n_az, n_rg, g, fs, bandwidth = case["n_az"], case["n_rg"], _generator(seed), 120e6, 100e6
    dr, pulse = C_LIGHT / (2.0 * fs), case["pulse"]
    t_p = pulse / fs
    rate = bandwidth / t_p
    at = torch.rand(2, 6, device="cuda", generator=g).tolist()
    raw = _noise((n_az, n_rg), g)
    a = torch.arange(n_az, dtype=torch.float64, device="cuda")
    m = torch.arange(n_rg, dtype=torch.float64, device="cuda")
    for k in range(6):
        r0 = case["r_near"] + at[1][k] * 0.7 * n_rg * dr
        x = case["speed"] * (a - at[0][k] * n_az) / case["prf"]
        lit = x.abs() <= case["wavelength"] * r0 / (2.0 * case["antenna"])
        r = torch.sqrt(r0 * r0 + x * x)
        u = (m[None, :] - ((r - case["r_near"]) / dr)[:, None]) / fs
        on = (u >= 0.0) & (u < t_p) & lit[:, None]
        phase = math.pi * rate * (u - t_p / 2) ** 2 - (4.0 * math.pi / case["wavelength"]) * r[:, None]
        raw += torch.polar(on.double(), phase).to(torch.complex64)
    u = m[:pulse] / fs
    ref = torch.zeros(n_rg, dtype=torch.complex128, device="cuda")
    ref[:pulse] = torch.polar(torch.ones_like(u), math.pi * rate * (u - t_p / 2) ** 2)
    geometry = dict(wavelength=case["wavelength"], speed=case["speed"], prf=case["prf"], range_bin=dr,
                    r_near=case["r_near"])
    return raw, ref.to(torch.complex64), geometry


# ---------------------------------------------------------------- the calls


def prepare(case, seed):
    if case["kind"] in ("rows", "cols"):
        x = _batch(case, seed)
        direction = mf.FFT_INVERSE if case["inverse"] else mf.FFT_FORWARD
        stride, dist = (1, x.shape[1]) if case["kind"] == "rows" else (x.shape[1], 1)
        plan = mf.Plan(case["n"], case["count"], stride, dist, case["storage"], direction, case["shift"])
        width = case["n"] if case["kind"] == "rows" else case["count"]
        return dict(kind="fft", plan=plan, x=x, out=torch.zeros_like(x), width=width)
    inter = case["inter"]
    if case["kind"] == "sar":
        raw, range_ref, az_ref = _sar_scene(case, seed)
        nbytes = mf._lib.sar_workspace_bytes(case["n_az"], case["n_rg"], inter)
        return dict(kind="sar", raw=raw, range_ref=range_ref, az_ref=az_ref, inter=inter, out=torch.empty_like(raw),
                    workspace=torch.empty(nbytes, dtype=torch.uint8, device="cuda"))
    raw, range_ref, geometry = _rd_scene(case, seed)
    nbytes = mf._lib.sar_rd_workspace_bytes(case["n_az"], case["n_rg"], inter)
    return dict(kind="rd", raw=raw, range_ref=range_ref, geometry=geometry, inter=inter, out=torch.empty_like(raw),
                workspace=torch.empty(nbytes, dtype=torch.uint8, device="cuda"))


def run(state):
    if state["kind"] == "fft":
        return state["plan"].execute(state["x"], state["out"])[:, :state["width"]]
    if state["kind"] == "sar":
        return mf.sar_form_image(state["raw"], state["range_ref"], state["az_ref"], state["inter"], state["out"],
                                 state["workspace"])
    return mf.sar_rd_form_image(state["raw"], state["range_ref"], state["geometry"], state["inter"], state["out"],
                                state["workspace"])


# ---------------------------------------------------------------- what a pass cannot do without


def work(case):
    """Each input point read once, each output point written once; 5 n log2 n operations a transform.

    The chains' intermediates are no input and no output."""
    if case["kind"] in ("rows", "cols"):
        points = case["n"] * case["count"]
        return dict(bytes=points * (16 if case["storage"] == FP32 else 8), flops=points * 5 * math.log2(case["n"]))
    points = case["n_az"] * case["n_rg"]
    logs = 5 * 2 * (math.log2(case["n_rg"]) + math.log2(case["n_az"]))
    # a complex product with each spectrum, and for the migration 8 complex taps with a real weight and a rotation
    more = 12 if case["kind"] == "sar" else 6 + 8 * 4 + 6
    return dict(bytes=points * 16, flops=points * (logs + more))


def tolerance(case):
    """About four times what another kernel shape (other radices and strips, another order of the sums) differs by.

    Seen: FP32 transforms and chains 1.1e-7 to 2.4e-7, with single image points away from the targets up to 1e-4 of
    the image's root mean square; half storage 6e-6 to 1.2e-5 (a rounding to the neighbour, 2^-10, now and then).
    Where an intermediate is stored in half precision, an order that rounds other values shows the whole rounding
    (2e-4 to 3e-4 against 64 bits), and the migration's positions in FP32 are worth 3.5e-6 at 4096 pulses.
    """
    if case["kind"] in ("rows", "cols"):
        # transforms of several passes (a small batch of 16384 points is split as well)
        stored = case["n"] >= (8192 if case["kind"] == "cols" else 16384)
        if case["storage"] == FP32:
            return dict(rel=1e-6)
        return dict(rel=1e-3) if stored else dict(rel=5e-5, max=4e-3)
    if case["inter"] == FP16:
        return dict(rel=1e-3, max=0.1)
    return dict(rel=1e-6 if case["kind"] == "sar" else 4e-6, max=4e-4)


# ---------------------------------------------------------------- the same in 64 bits


def _wide(x):
    return x.to(torch.complex128) if x.is_complex() else torch.view_as_complex(x.double())


def _exact_rd(raw, range_ref, geometry):
    n_az, n_rg = raw.shape
    y = torch.fft.ifft(torch.fft.fft(_wide(raw), dim=1) * torch.fft.fft(_wide(range_ref)).conj()[None, :], dim=1)
    z = torch.fft.fft(y, dim=0) / n_az
    del y
    k = torch.arange(n_az, dtype=torch.float64, device=raw.device)
    f = torch.where(k < n_az / 2, k, k - n_az) * geometry["prf"] / n_az
    x2 = (geometry["wavelength"] * f / (2.0 * geometry["speed"])) ** 2
    d = torch.sqrt(1.0 - x2)
    n = torch.arange(n_rg, device=raw.device)
    r0 = geometry["r_near"] + n.double() * geometry["range_bin"]
    dn = (x2 / (d * (1.0 + d)) / geometry["range_bin"])[:, None] * r0[None, :]
    s = torch.floor(dn)
    mu = (dn - s) * 128.0
    q = mu.floor().clamp_(max=127.0)
    alpha, q, s = mu - q, q.long(), s.long()
    # 8-tap sinc under a Kaiser window (beta 2.5), 129 shifts, each row of unit sum
    tap = torch.arange(8, dtype=torch.float64, device=raw.device) - 3.0
    at = tap[None, :] - torch.arange(129, dtype=torch.float64, device=raw.device)[:, None] / 128.0
    g = torch.sinc(at) * torch.special.i0(2.5 * torch.sqrt((1.0 - (at / 4.0) ** 2).clamp_(min=0.0)))
    g = g / g.sum(dim=1, keepdim=True)
    out = torch.zeros_like(z)
    for j in range(8):
        at = n[None, :] + s + (j - 3)
        inside = (at >= 0) & (at < n_rg)
        weight = (g[q, j] + alpha * (g[q + 1, j] - g[q, j])) * inside
        out += z.gather(1, at.clamp_(0, n_rg - 1)) * weight
    phase = (-4.0 * math.pi / geometry["wavelength"]) * (x2 / (1.0 + d))[:, None] * r0[None, :]
    out *= torch.polar(torch.ones_like(phase), phase)
    return torch.fft.ifft(out, dim=0, norm="forward")


def exact(case, seed):
    if case["kind"] in ("rows", "cols"):
        x, dim = _wide(_batch(case, seed)), 1 if case["kind"] == "rows" else 0
        x = x[:, :case["n"] if case["kind"] == "rows" else case["count"]]
        y = torch.fft.ifft(x, dim=dim, norm="forward") if case["inverse"] else torch.fft.fft(x, dim=dim)
        del x
        y = y * 2.0 ** -case["shift"] if case["shift"] else y
        return torch.view_as_real(y) if case["storage"] == FP16 else y
    if case["kind"] == "sar":
        raw, range_ref, az_ref = _sar_scene(case, seed)
        y = torch.fft.fft2(_wide(raw))
        y *= torch.fft.fft(_wide(range_ref)).conj()[None, :]
        y *= torch.fft.fft(_wide(az_ref)).conj()[:, None]
        return torch.fft.ifft2(y)
    return _exact_rd(*_rd_scene(case, seed))
