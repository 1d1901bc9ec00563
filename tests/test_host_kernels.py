"""Device functions that also compile for the host, run there by a small
driver (host_kernels.cpp) built from the kernels' own headers."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")

# Boxes on both sides of every line of xcd_map (storage, box, mapping with the
# remap on: 1 eighths, 2 runs of 16 tiles); the small ones step on the GPU with
# and without the remap (test_gpu_parity.py)
REMAP_BOXES = [("f16s", (101, 79, 83), 1), ("f16s", (113, 83, 89), 2), ("f16s", (256, 63, 53), 2),
               ("bf16s", (127, 97, 71), 2), ("f32", (64, 64, 96), 1), ("f32s", (97, 61, 71), 2),
               ("f64", (61, 59, 47), 1), ("f64", (64, 64, 64), 1), ("f64", (64, 64, 65), 2)]
REMAP_LARGE = [("f16s", (128, 128, 128), 2), ("f16s", (128, 128, 248), 2), ("f16s", (128, 128, 254), 1),
               ("f16s", (128, 128, 256), 1), ("bf16s", (128, 128, 260), 1), ("bf16s", (128, 128, 264), 2),
               ("f16s", (512, 512, 384), 2), ("f16s", (512, 512, 512), 2), ("f32", (64, 64, 128), 1),
               ("f32", (128, 128, 63), 2), ("f32", (128, 128, 64), 1), ("f32", (128, 128, 128), 1),
               ("f32", (127, 127, 130), 1), ("f32", (128, 128, 256), 2), ("f32", (512, 512, 512), 2),
               ("f64", (128, 128, 64), 1), ("f64", (256, 256, 256), 2)]


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("ROCm toolchain not found")
    exe = tmp_path_factory.mktemp("host_kernels") / "driver"
    cmd = [HIPCC, "-x", "hip", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-O2", "-std=c++17", os.path.join(ROOT, "tests", "host_kernels.cpp"), "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]

    def run(mode, data):
        r = subprocess.run([str(exe), mode], input=np.ascontiguousarray(data).tobytes(), capture_output=True,
                           timeout=120)
        assert r.returncode == 0, (mode, r.returncode, r.stderr[-500:])
        return r.stdout

    return run


def _round(v, bits, emin, emax):
    """v in FP64 rounded once, to nearest even, to `bits` significant bits with
    least exponent emin (subnormals below) and largest emax (infinity above)."""
    m, e = np.frexp(v)  # 0.5 <= |m| < 1
    q = np.maximum(e, emin + 1) - bits
    with np.errstate(over="ignore", invalid="ignore"):
        r = np.ldexp(np.rint(np.ldexp(v, -q)), q)
        r = np.where(np.abs(r) >= np.ldexp(1.0, emax + 1), np.copysign(np.inf, v), r)
    return np.where(np.isfinite(v), r, v)


@pytest.mark.parametrize("bits,emin,emax", [(11, -14, 15), (8, -126, 127)], ids=["fp16", "bf16"])
def test_round_to_odd_then_to_16_bits_is_one_rounding(driver, bits, emin, emax):
    """FP64 -> FP32 by rounding to odd -> 16 bits to nearest equals one
    rounding of the FP64 value: zeros, values that underflow FP32 from either
    side (their sign kept), subnormals of both formats, ties and their
    neighbours, the ends of the 16-bit and of the FP32 range, infinities,
    NaN, and random values over all exponents."""
    rng = np.random.default_rng(4)
    pos = [0.0, 5e-324, 1e-60, 2.0 ** -151, 2.0 ** -150, 2.0 ** -149, 1.5 * 2.0 ** -149, 2.5 * 2.0 ** -149, 2.0 ** -134,
           2.0 ** -133, 2.0 ** -126, 3.3e-39, 2.0 ** -26, 2.0 ** -25, 2.0 ** -24, 1.5 * 2.0 ** -24, 2.0 ** -14, 1.0,
           1 + 2.0 ** -11, 1 + 3 * 2.0 ** -11, 1 + 2.0 ** -8, 1 + 3 * 2.0 ** -8, 65472.0, 65504.0, 65520.0, 65536.0,
           float(np.finfo(np.float32).max), 2.0 ** 128 * (1 - 2.0 ** -9), 2.0 ** 128 * (1 - 2.0 ** -25), 2.0 ** 128,
           1e60, 1e308]
    pos = np.array(pos)
    near = np.concatenate([pos, np.nextafter(pos, np.inf), np.nextafter(pos, 0), pos * (1 + 1e-9), pos * (1 - 1e-9)])
    wide = rng.uniform(1, 2, 200000) * 2.0 ** rng.integers(-170, 140, 200000)
    ties = (2 * rng.integers(2 ** bits // 2, 2 ** bits, 20000) + 1) * 2.0 ** rng.integers(emin - bits - 3, 5, 20000)
    v = np.concatenate([near, wide, ties, np.nextafter(ties, 0), np.nextafter(ties, np.inf), [np.inf]])
    v = np.concatenate([v, -v])
    odd = np.frombuffer(driver("odd", v), np.float32)
    got, want = _round(odd.astype(np.float64), bits, emin, emax), _round(v, bits, emin, emax)
    bad = (got != want) | (np.signbit(odd) != np.signbit(v))
    assert not bad.any(), list(zip(v[bad][:5], odd[bad][:5], want[bad][:5]))
    # where FP32 does not hold v, its neighbour with the odd last bit
    inexact = np.isfinite(v) & (odd.astype(np.float64) != v)
    assert np.all(odd.view(np.uint32)[inexact] & 1)
    assert np.all(np.isnan(np.frombuffer(driver("odd", [np.nan, -np.nan]), np.float32)))


def _root(f, d):
    """Nontrivial root of dH per node by bisection in FP64, and what FP32
    rounding may move it by: dH's terms f u L, f y and a d log(1 + x) to four
    roundings each, its sum to eight roundings of its terms, over the slope."""
    x = d / f
    cap = np.minimum((1 - 2.0 ** -10) * -1 / x.min(0), 64.0)
    P = np.sum(d * np.log1p(x), 0)

    def terms(a):
        y = a * x
        return f * (1 + y) * np.log1p(y), f * y

    def dh(a):
        s, t = terms(a)
        return np.sum(s - t, 0) - a * P

    lo, hi = np.ones_like(cap), cap.copy()
    for _ in range(60):
        mid = 0.5 * (lo + hi)
        up = dh(mid) > 0
        hi, lo = np.where(up, mid, hi), np.where(up, lo, mid)
    a = np.where(dh(cap) <= 0, cap, lo)
    s, t = terms(a)
    slope = np.abs(np.sum(d * np.log1p(a * x), 0) - P)  # (of either sign where the cap is below 1)
    noise = 4 * np.sum(np.abs(s) + np.abs(t), 0) + 4 * a * np.sum(np.abs(d * np.log1p(x)), 0)
    noise += 8 * np.sum(np.abs(s - t), 0)
    return a, 2.0 ** -24 * noise / slope


@pytest.mark.parametrize("amp", [0.2, 0.35, 0.5, 0.7, 0.9, 0.99, "one", "hole", "wide"])
def test_fp32_path_length_far_from_equilibrium(driver, orc, amp):
    """The entropic path length in FP32 arithmetic, both storage widths, over
    10000 nodes far from equilibrium against bisection in FP64: populations off
    the weights by up to amp, with one of them up to 40 times larger or smaller
    besides, or by factors of any size. Bar per node: the FP32 noise of dH (see
    _root), 2e-7 of alpha for what the iteration leaves (its stop is 1e-7, twice
    that allows for the terms its estimate leaves out) and four roundings of the
    positivity cap."""
    rng = np.random.default_rng(11)
    dims = (50, 20, 5)
    n = 2 * dims[0] * dims[1] * dims[2]
    w = orc.lattice()[1][:, None]
    a = rng.uniform(0, 0.9, n) if isinstance(amp, str) else amp
    f = w * (1 + a * rng.uniform(-1, 1, (41, n)))
    if amp == "wide":
        f = w * np.exp(rng.uniform(0.1, 0.8, n) * rng.standard_normal((41, n)))
    elif isinstance(amp, str):
        f[rng.integers(0, 41, n), np.arange(n)] *= rng.uniform(1, 40, n) ** (1 if amp == "one" else -1)
    f = f.astype(np.float32)
    d = (orc.collide_field(*dims, 1.0, f.astype(np.float64)) - f).astype(np.float32)
    got = np.frombuffer(driver("alpha", np.concatenate([f, d]).T), np.float32).reshape(n, 2)
    f, d = f.astype(np.float64), d.astype(np.float64)
    far = np.max(np.abs(d / f), 0) > 0.0625
    assert far.sum() > 0.9 * n
    ref, noise = _root(f, d)
    for k in range(2):
        excess = (np.abs(got[:, k] - ref) - noise)[far] / ref[far]
        assert np.max(excess) <= 2e-7 + 4 * 2.0 ** -24, (k, np.max(excess), int(np.sum(excess > 2e-7)))


def test_tile_mapping_of_boxes(driver):
    """xcd_map's answer for boxes of every width on both sides of its lines,
    from the bytes of a q-block, of the stride between q-blocks (rounded up to
    256 bytes, a mebibyte and 256 bytes more for 16-bit blocks of whole
    mebibytes) and of both buffers: a block whose stride rounds up to a power
    of two is taken as one; without the remap always dispatch order."""
    def record(storage, nodes, remap=1):
        eb = {"f16s": 2, "bf16s": 2, "f32": 4, "f32s": 4, "f64": 8}[storage]
        stride = -(-nodes * eb // 256) * 256
        if eb == 2 and stride % 2 ** 20 == 0:
            stride += 2 ** 20 + 256
        return remap, nodes * eb, stride, 82 * nodes * eb

    cases = [(s, 2 * x * y * z, m) for s, (x, y, z), m in REMAP_BOXES + REMAP_LARGE]
    cases += [("f32", 2 ** 21 - 6, 1), ("f32", 2 ** 21 - 66, 2), ("f64", 2 ** 20 - 6, 1), ("f64", 2 ** 20 + 2, 2)]
    for remap in (1, 0):
        out = driver("map", np.array([record(s, n, remap) for s, n, _ in cases], np.uint64))
        assert np.frombuffer(out, np.uint32).tolist() == [m if remap else 0 for _, _, m in cases]
    # many boxes: by what both buffers hold
    out = driver("map", np.array([[1, 0, 0, 2 ** 28], [1, 0, 0, 2 ** 28 + 1]], np.uint64))
    assert np.frombuffer(out, np.uint32).tolist() == [1, 2]
