"""Packs of 16, staged rounds: the quantizer's guard and clamp rule (csrc/compress.hip, token_quant_near, quant_range), in
numpy for fp16 tokens as the kernel meets them.  t = fl(x * r + c) with r = 1 / s up to an ulp and c = fl(128.5 +
g * 2^-16 - min * r); the code is the integer part of t - 128, unless the 16 fraction bits of t are below 2g or the
token's scale is below the tensor's small_scale, where the IEEE divide decides; values are clamped on the fast path only
where the tensor's relative scale asks for it.  (The kernel holds t / 256, clamped to 0 .. 1; for numbers that changes the
exponent only.)  The result is the code of clamp(rint(fl((x - min) / scale)), 0, qmax)
(PackKV Sec. III-B.2)."""
import numpy as np
import pytest


def _quant_range(rel, qmax):
    room = (qmax + 0.5 - 4.0 / 65536.0) * float(np.float32(rel)) / (1.0 + 2.0 ** -20) - 1.0
    cap_all = not room > 1.0 / 2048.0
    return cap_all, np.float32(0.0) if cap_all else np.float32(2.0 ** -25 / room * 1.0001)


def _rule(x, mn, s, qmax, rel, ulp_off):
    x, mn, s = (v.astype(np.float32) for v in (x, mn, s))
    exact = np.clip(np.rint(((x - mn).astype(np.float32) / s).astype(np.float32)), 0, qmax)
    r = (np.float32(1.0) / s).astype(np.float32)
    r = (r.view(np.int32) + ulp_off).view(np.float32)                      # the hardware reciprocal: within one ulp
    fma = lambda a, b, c: (a.astype(np.float64) * b.astype(np.float64) + c).astype(np.float32)  # noqa: E731
    probe = fma(-mn, r, 128.5)
    e = ((probe.view(np.uint32) >> 23) & 0xFF).astype(np.int64) - 127
    g = 2 + np.where(e >= 8, 2 << np.minimum(np.maximum(e - 8, 0), 14), 0)
    c = fma(-mn, r, (np.float32(128.5) + (g / 65536.0).astype(np.float32)).astype(np.float32).astype(np.float64))
    t = fma(x, r, c.astype(np.float64)).view(np.uint32)
    cap_all, small = _quant_range(rel, qmax)
    divide = ((t & 0xFFFF) < 2 * g) | (s < small)
    top = (t >> 16).astype(np.int64)
    if cap_all:
        top = np.minimum(top, 0x4300 + qmax)
    return exact, np.where(divide, exact, top - 0x4300), divide


# 2 / 21 and its neighbour below 1 / 10.5: the quotient of a token's largest value reaches qmax + 1/2
@pytest.mark.parametrize("rel", [0.1, 0.2, 1 / 15, 0.07, 1 / 7, 0.3, 1.0, 0.5, 2 / 21, 0.09525, 0.0953, 0.4001, 0.6667])
@pytest.mark.parametrize("ulp_off", [0, 1, -1])
@pytest.mark.parametrize("offset", [0.0, 40.0, 3000.0])
def test_near_rule_gives_the_codes_of_the_divide(rel, ulp_off, offset):
    rng = np.random.default_rng(int(offset) * 7 + ulp_off + 11)
    n = 60_000
    qmax = int(np.floor(1.0 / float(np.float32(rel)) + 0.5))
    near = 0
    with np.errstate(over="ignore", invalid="ignore", divide="ignore"):
        mag = np.float32(2.0) ** rng.integers(-24, 12, n)
        mn = ((rng.standard_normal(n) + offset) * mag).astype(np.float16)
        span = np.abs(rng.standard_normal(n).astype(np.float32) * mag * 4)
        mx = (mn.astype(np.float32) + span).astype(np.float16)             # the token's largest value
        s = (np.float32(rel) * (mx.astype(np.float32) - mn.astype(np.float32))).astype(np.float32).astype(np.float16)
        ok = (s.astype(np.float32) > 0) & np.isfinite(s.astype(np.float32)) & np.isfinite(mx.astype(np.float32))
        inside = (mn.astype(np.float32) + rng.random(n).astype(np.float32) * (mx.astype(np.float32) - mn.astype(np.float32))).astype(np.float16)
        tie = (mn.astype(np.float32) + (rng.integers(0, 16, n) + np.float32(0.5)) * s.astype(np.float32)).astype(np.float16)
        cases = [inside, mn, mx] + [(tie.view(np.uint16).astype(np.int32) + k).clip(0, 0xFBFF).astype(np.uint16).view(np.float16)
                                    for k in (0, 1, -1, 2, -2)]
        for x in cases:
            xf = x.astype(np.float32)
            use = ok & np.isfinite(xf) & (xf >= mn.astype(np.float32)) & (xf <= mx.astype(np.float32))
            exact, got, divide = _rule(x[use], mn[use], s[use], qmax, rel, ulp_off)
            assert np.array_equal(exact, got)
            near += int(divide.sum())
    # (far from zero fp16's own steps are coarse against the scale, and some scales meet no tie there)
    assert near > 100 or offset > 0, "the tie cases are meant to reach the divide"


def test_small_scale_is_rare():
    """The default scales clamp by token only, and only tokens whose range is below fp16's smallest steps."""
    for rel, qmax in ((0.1, 10), (0.2, 5), (1 / 15, 15)):
        cap_all, small = _quant_range(rel, qmax)
        assert not cap_all and small < 64 * 2.0 ** -24
