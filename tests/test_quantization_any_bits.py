"""The compressor's three rules for a code give the same one for every bit pattern of a value, NaNs and infinities included:
chunks are sized by one of them and written by another (csrc/compress.hip: quantize_quad sizes rounds in two passes,
quantize_value and quantize_token8 write packs of 8 and of 16), and a chunk that came out larger would not fit its place.
All of them mean clamp(rint(fl((x - min) / scale)), 0, qmax) with 0 for a scale of 0, and qmax where that quotient is no number.
quantize_value is the kernel's own code, compiled for the host; the other two are models in numpy."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

from paper_2512_24449_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))
ALL = np.arange(65536, dtype=np.uint16)


@pytest.fixture(scope="module")
def kernels_rule(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("value") / "quantize_value_check.so")
    subprocess.check_call([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-O2", "-std=c++17", "-ffp-contract=off", "-x", "hip",
                           "--offload-host-only", "-shared", "-fPIC", "-I", build.CSRC, "-o", lib, os.path.join(HERE, "quantize_value_check.cpp")])
    L = C.CDLL(lib)
    L.quantize.argtypes = [C.c_void_p] * 3 + [C.c_int, C.c_int, C.c_void_p]

    def codes(x, s, mn, qmax):
        x, s, mn = (np.ascontiguousarray(v, dtype=np.float32) for v in (x, np.broadcast_to(s, x.shape), np.broadcast_to(mn, x.shape)))
        out = np.empty(x.shape, np.uint8)
        L.quantize(x.ctypes.data, s.ctypes.data, mn.ctypes.data, x.size, qmax, out.ctypes.data)
        return out.astype(np.int64)
    return codes


def _definition(x, s, mn, qmax):
    if s == 0:
        return np.zeros(x.shape, np.int64)
    q = ((x - mn).astype(np.float32) / s).astype(np.float32)
    return np.clip(np.rint(np.where(np.isnan(q), np.float32(qmax), q)), 0, qmax).astype(np.int64)


def _fma(bits, r, c, payload):
    """fl(x * r + c) as bits; x: fp16 bits.  payload: a NaN comes out with its own payload, else as the default NaN."""
    x = bits.view(np.float16).astype(np.float32)
    t = (x.astype(np.float64) * np.float64(r) + np.float64(c)).astype(np.float32)
    out = t.view(np.uint32).copy()
    out[np.isnan(t)] = 0x7FC00000
    if payload and np.isfinite(r) and np.isfinite(c):
        wide = ((bits.astype(np.uint32) & 0x8000) << 16) | 0x7FC00000 | ((bits.astype(np.uint32) & 0x3FF) << 13)
        out = np.where(np.isnan(x), wide, out)
    return out


def _guard(r, mn, least):
    probe = np.float32(np.float64(-mn) * np.float64(r) + 128.5)
    e = ((int(probe.view(np.uint32)) >> 23) & 0xFF) - 127
    g = least + (2 << min(e - 8, 14) if e >= 8 else 0)
    c = np.float32(np.float64(-mn) * np.float64(r) + np.float64(np.float32(128.5 + g / 65536.0)))
    return g, c


def _token8(bits, s, mn, qmax, payload):
    """token_quant, quantize_token8; each value is tested for the divide by itself, which decides no less than all eight together."""
    r = np.float32(1) / s if s != 0 else np.float32(0)
    g, c = _guard(r, mn, 3)
    guard = 2 * g
    if s == 0:
        guard, c = 0xFFFF, np.uint32(0x4300FFFF).view(np.float32)
    t = _fma(bits, r, c, payload)
    fast = np.minimum(t >> 16, 0x4300 + qmax).astype(np.int64) & 0xFF
    return np.where((t & 0xFFFF) < guard, _definition(bits.view(np.float16).astype(np.float32), s, mn, qmax), fast)


def _quad(bits, s, mn, qmax, payload):
    """token_quant_near, quantize_quad: t / 256 clamped to 0 .. 1, a NaN to 0."""
    r = np.float32(1) / s if s != 0 else np.float32(0)
    g, c = _guard(r, mn, 4 if qmax > 15 else 2)
    t = _fma(bits, r, c, payload).view(np.float32)
    with np.errstate(invalid="ignore"):
        unit = np.where(np.isnan(t), np.float32(0), np.clip(t / np.float32(256), np.float32(0), np.float32(1))).astype(np.float32).view(np.uint32)
    fast = (unit >> 16).astype(np.int64) - 0x3F00
    return np.where((unit & 0xFFFF) < 2 * g, _definition(bits.view(np.float16).astype(np.float32), s, mn, qmax), fast)


# tokens as (smallest value, largest value) of those that are numbers
TOKENS = [(-1.0, 1.0), (0.0, 0.0), (3.0, 3.0), (-2.0 ** -24, 2.0 ** -24), (1.0, 1.25), (-65504.0, 65504.0), (0.0, np.inf), (-np.inf, 5.0),
          (-np.inf, np.inf), (-np.inf, -np.inf), (np.inf, np.inf), (2000.0, 2002.0)]


@pytest.mark.parametrize("rel", [0.1, 0.2, 1 / 15, 1.0, 0.05, 1 / 31, 1 / 127])
def test_every_bit_pattern_has_one_code(kernels_rule, rel):
    qmax = int(np.floor(1 / float(np.float32(rel)) + 0.5))
    with np.errstate(over="ignore", invalid="ignore", divide="ignore"):
        for lo, hi in TOKENS:
            mn = np.float32(lo)
            s = np.float32(abs(np.float16(np.float32(rel) * (np.float32(hi) - mn))))
            x = ALL.view(np.float16).astype(np.float32)
            bits = ALL[np.isnan(x) | ((x >= mn) & (x <= np.float32(hi)))]   # what such a token can hold
            x = bits.view(np.float16).astype(np.float32)
            want = _definition(x, s, mn, qmax)
            assert np.array_equal(kernels_rule(x, s, mn, qmax), want), ("quantize_value", lo, hi)
            # (scales below this have every value take the divide)
            if s == 0 or s >= 64 * 2.0 ** -24 or np.isnan(s):
                for payload in (False, True):
                    assert np.array_equal(_quad(bits, s, mn, qmax, payload), want), ("quantize_quad", lo, hi, payload)
                    if qmax < 16:
                        assert np.array_equal(_token8(bits, s, mn, qmax, payload), want), ("quantize_token8", lo, hi, payload)
