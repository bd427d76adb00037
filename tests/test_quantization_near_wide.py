"""Wide chunks, staged rounds: the fixed-point rule of the packs of 16 with codes up to 127 and a guard of 4 (+ 2^(e-7)) steps
of 2^-16 (csrc/compress.hip, token_quant_near<true>), in numpy against the IEEE divide of the definition."""
import numpy as np
import pytest


def _fma(a, b, c):
    return (a.astype(np.float64) * b.astype(np.float64) + c.astype(np.float64)).astype(np.float32)


@pytest.mark.parametrize("rel", [1 / 16, 0.05, 0.0333, 1 / 63, 1 / 100, 1 / 100.49, 1 / 127, 0.0079])
@pytest.mark.parametrize("ulp_off", [0, 1, -1])
@pytest.mark.parametrize("offset", [0.0, 40.0, 3000.0])
def test_codes_of_the_divide(rel, ulp_off, offset):
    rng = np.random.default_rng(int(offset) * 7 + ulp_off + 11)
    n = 60_000
    qmax = int(np.floor(1.0 / float(np.float32(rel)) + 0.5))
    assert qmax <= 127
    room = (qmax + 0.5 - 8.0 / 65536.0) * float(np.float32(rel)) / (1.0 + 2.0 ** -20) - 1.0
    cap_all = not room > 1.0 / 2048.0
    small = np.float32(0.0) if cap_all else np.float32(2.0 ** -25 / room * 1.0001)
    near = 0
    with np.errstate(over="ignore", invalid="ignore", divide="ignore"):
        mag = np.float32(2.0) ** rng.integers(-24, 12, n)
        mn = ((rng.standard_normal(n) + offset) * mag).astype(np.float16)
        mx = (mn.astype(np.float32) + np.abs(rng.standard_normal(n).astype(np.float32) * mag * 4)).astype(np.float16)
        s = (np.float32(rel) * (mx.astype(np.float32) - mn.astype(np.float32))).astype(np.float32).astype(np.float16)
        ok = (s.astype(np.float32) > 0) & np.isfinite(s.astype(np.float32)) & np.isfinite(mx.astype(np.float32))
        inside = (mn.astype(np.float32) + rng.random(n).astype(np.float32) * (mx.astype(np.float32) - mn.astype(np.float32))).astype(np.float16)
        tie = (mn.astype(np.float32) + (rng.integers(0, qmax, n) + np.float32(0.5)) * s.astype(np.float32)).astype(np.float16)
        cases = [inside, mn, mx] + [(tie.view(np.uint16).astype(np.int32) + k).clip(0, 0xFBFF).astype(np.uint16).view(np.float16)
                                    for k in (0, 1, -1, 2, -2)]
        for x in cases:
            xf = x.astype(np.float32)
            use = ok & np.isfinite(xf) & (xf >= mn.astype(np.float32)) & (xf <= mx.astype(np.float32))
            x1, m1, s1 = (v[use].astype(np.float32) for v in (x, mn, s))
            exact = np.clip(np.rint(((x1 - m1).astype(np.float32) / s1).astype(np.float32)), 0, qmax)
            r = ((np.float32(1.0) / s1).astype(np.float32).view(np.int32) + ulp_off).view(np.float32)
            e = ((_fma(-m1, r, np.full_like(r, 128.5)).view(np.uint32) >> 23) & 0xFF).astype(np.int64) - 127
            g = 4 + np.where(e >= 8, 2 << np.minimum(np.maximum(e - 8, 0), 14), 0)
            t = _fma(x1, r, _fma(-m1, r, (np.float32(128.5) + (g / 65536.0).astype(np.float32)).astype(np.float32)))
            t = np.clip(np.nan_to_num(t, nan=0.0), 0.0, 256.0).astype(np.float32).view(np.uint32)   # the kernel's clamp, times 256
            divide = ((t & 0xFFFF) < 2 * g) | (s1 < small)
            top = (t >> 16).astype(np.int64) - 0x4300
            if cap_all:
                top = np.minimum(top, qmax)
            assert np.array_equal(exact, np.where(divide, exact, top))
            near += int(divide.sum())
    assert near > 100 or offset > 0, "the tie cases are meant to reach the divide"
