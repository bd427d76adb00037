"""Packs of 16: the compressor quantizes with one fused multiply-add per value whose result is a
fixed-point number (csrc/compress.hip, token_quant / quantize_token8): t = fl(x * r + c) with r = 1 / s
up to an ulp and c = fl(128.5 + g * 2^-16 - min * r); the code is the integer part of t - 128, clamped,
unless the 16 fraction bits of t are below 2g, where the IEEE divide decides.  This checks that rule in
numpy for fp16 tokens as the kernel meets them (scale = fp16(rel * (max - min)), min <= x <= max): it
gives exactly the code of clamp(rint(fl((x - min) / scale)), 0, qmax) (PackKV Sec. III-B.2)."""
import numpy as np
import pytest


def _rule(x, mn, s, qmax, ulp_off):
    x, mn, s = (v.astype(np.float32) for v in (x, mn, s))
    exact = np.clip(np.rint(((x - mn).astype(np.float32) / s).astype(np.float32)), 0, qmax)
    r = (np.float32(1.0) / s).astype(np.float32)
    r = (r.view(np.int32) + ulp_off).view(np.float32)                      # the hardware reciprocal: within one ulp
    fma = lambda a, b, c: (a.astype(np.float64) * b.astype(np.float64) + c).astype(np.float32)  # noqa: E731
    probe = fma(-mn, r, 128.5)
    e = ((probe.view(np.uint32) >> 23) & 0xFF).astype(np.int64) - 127
    g = 3 + np.where(e >= 8, 2 << np.minimum(np.maximum(e - 8, 0), 14), 0)
    c = fma(-mn, r, (np.float32(128.5) + (g / 65536.0).astype(np.float32)).astype(np.float32).astype(np.float64))
    t = fma(x, r, c.astype(np.float64)).view(np.uint32)
    divide = (t & 0xFFFF) < 2 * g
    fast = np.minimum(t >> 16, 0x4300 + qmax.astype(np.int64)) & 0xFF
    return exact, np.where(divide, exact, fast), divide


@pytest.mark.parametrize("ulp_off", [0, 1, -1])
@pytest.mark.parametrize("offset", [0.0, 1.0, 40.0, 3000.0])
def test_fixed_point_rule_gives_the_codes_of_the_divide(ulp_off, offset):
    rng = np.random.default_rng(int(offset) * 7 + ulp_off + 11)
    n = 400_000
    near = 0
    with np.errstate(over="ignore", invalid="ignore", divide="ignore"):
        mag = np.float32(2.0) ** rng.integers(-24, 12, n)
        mn = ((rng.standard_normal(n) + offset) * mag).astype(np.float16)
        span = np.abs(rng.standard_normal(n).astype(np.float32) * mag * 4)
        mx = (mn.astype(np.float32) + span).astype(np.float16)             # the token's largest value
        rel = rng.choice([0.1, 0.2, 1 / 15, 1 / 7, 0.3, 1.0, 0.5], n).astype(np.float32)
        s = (rel * (mx.astype(np.float32) - mn.astype(np.float32))).astype(np.float32).astype(np.float16)
        qmax = np.rint(1 / rel)
        ok = (s.astype(np.float32) > 0) & np.isfinite(s.astype(np.float32)) & np.isfinite(mx.astype(np.float32))
        inside = (mn.astype(np.float32) + rng.random(n).astype(np.float32) * (mx.astype(np.float32) - mn.astype(np.float32))).astype(np.float16)
        tie = (mn.astype(np.float32) + (rng.integers(0, 16, n) + np.float32(0.5)) * s.astype(np.float32)).astype(np.float16)
        cases = [inside, mn, mx] + [(tie.view(np.uint16).astype(np.int32) + k).clip(0, 0xFBFF).astype(np.uint16).view(np.float16)
                                    for k in (0, 1, -1, 2, -2)]
        for x in cases:
            xf = x.astype(np.float32)
            use = ok & np.isfinite(xf) & (xf >= mn.astype(np.float32)) & (xf <= mx.astype(np.float32))
            exact, got, divide = _rule(x[use], mn[use], s[use], qmax[use], ulp_off)
            assert np.array_equal(exact, got)
            near += int(divide.sum())
    assert near > 1000, "the tie cases are meant to reach the divide"
