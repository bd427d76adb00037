"""V product over wide chunks against 64 bits, for values on both sides of 0 and for values that are nearly all their token's minimum: the centre of the
codes (csrc/pack8.h, vw_chunk) must not cost the one what it gives the other."""
import numpy as np
import pytest
import torch

import oracle
from paper_2512_24449_amd import binding
from tests import gpu_cases

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hq", [2, 6, 8, 16])
@pytest.mark.parametrize("levels", [16, 31, 32, 255])
@pytest.mark.parametrize("kind", ["normal", "near the minimum"])
def test_error(kind, levels, Hq):
    B, H, blocks = 1, 2, 128
    L = 64 * blocks
    rng = np.random.default_rng(levels + Hq)
    V = rng.standard_normal((B, L, H, 128))
    if kind != "normal":
        V = np.where(rng.random(V.shape) < 0.02, np.abs(V), 0.0)
        V[..., 0] = 0.0
    V = V.astype(np.float16)
    K = np.zeros_like(V)
    cache = binding.PackedKVCache(B, H, Hq, L, k_rel_scale=1 / levels, v_rel_scale=1 / levels, pack_size=8)
    cache.kv_compress_append(torch.from_numpy(K).cuda(), torch.from_numpy(V).cuda())
    n, _, cv = gpu_cases.oracle_cache(K, V, 1 / levels, 1 / levels, 8)
    codes, meta = gpu_cases.full_codes(cv, V.shape, n)
    p = (rng.uniform(0.5, 1.5, (B, Hq, L)) / L).astype(np.float32)
    got = cache.kv_v_matvec(torch.from_numpy(p).cuda()).cpu().numpy()
    want = oracle.v_out(codes, V, meta, n, p)
    scale = meta[0].astype(np.uint32).astype(np.uint16).view(np.float16).astype(np.float64)
    low = (meta[0].astype(np.uint32) >> 16).astype(np.uint16).view(np.float16).astype(np.float64)
    z = np.clip(-low / np.where(scale == 0, 1, scale), 0, levels)
    for r in range(Hq):
        h = r // (Hq // H)
        # A weight is right to 2^-36 (its fp16 residual, subnormal and times 2^11) or, from 2^-14 on, 2^-22 of itself, at random, and is made good for
        # a code of z: the norm over a head's 128 outputs, four times what is to be expected.
        w = p[0, r] * scale
        unit = np.maximum(2.0 ** -36, 2.0 ** -22 * w) / np.sqrt(3) * (scale > 0)
        weights = np.sqrt(((unit[:, None] * (codes[0, :, h].astype(np.float64) - z[:, None])) ** 2).sum())
        # fp32 sums: a wave sums a block's w (code - mid) and p (min + mid scale), each at most S, over 64 tokens, and adds the two; a rounding
        # of S each way, the waves' independent of each other.  What comes behind is of the output's size.
        S = (w * (levels / 2)).reshape(blocks, 64).sum(1)
        sums = 2.0 ** -24 * 2 * np.sqrt(128 * (S ** 2).sum())
        size, error = np.linalg.norm(want[0, r]), np.linalg.norm(got[0, r] - want[0, r])
        print("%s %d %d: error %.2e weights %.2e sums %.2e of %.2e" % (kind, levels, Hq, error, weights, sums, size))
        assert error <= 4 * weights + sums + 2.0 ** -22 * size, (kind, levels, Hq, r)
