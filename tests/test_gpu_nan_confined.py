"""NaNs in the input stay with their own value, whatever their bits: they count for no token's scale or minimum and take
the largest code of their token, so the cache holds what it holds with the token's largest value in their place.  (The
largest value's code is qmax at these scales.)  Packs of 16: rounds that are staged, paged, repacked or done in two passes."""
import numpy as np
import pytest
import torch

from paper_2512_24449_amd import binding, synth

pytestmark = pytest.mark.gpu

# quiet and signalling, low bits of the payload set and not, both signs
FP16_NANS = (0x7E00, 0x7FFF, 0xFFFF, 0x7E01, 0x7C01, 0xFC02, 0x7D04)
BF16_NANS = (0x7FC0, 0x7FFF, 0xFFFF, 0x7FC1, 0x7F81, 0xFF82, 0x7FA0)


def _with_nans(x, rng, patterns):
    """-> (x with NaNs, x with the token's largest value there instead); x: [B, L, H, 128] on the CPU."""
    B, L = x.shape[:2]
    clean = x.clone().view(B, L, -1)
    lo, hi = clean.amin(-1, keepdim=True), clean.amax(-1, keepdim=True)
    at = torch.from_numpy(rng.random(clean.shape) < 0.005)
    at[:, 5, 1:] = True  # nearly all of a token
    at &= (clean != lo) & (clean != hi)
    clean = torch.where(at, hi.expand_as(clean), clean)
    bits = torch.from_numpy(rng.choice(np.array(patterns, np.uint16), clean.shape).view(np.int16))
    nans = torch.where(at, bits, clean.view(torch.int16)).view(x.dtype)
    return nans.view_as(x).cuda(), clean.view_as(x).cuda()


def _contents(cache, n_chunks):
    """Token metadata and the bytes of every chunk."""
    out = []
    for name in ("k", "v"):
        out.append(cache.view(name + "_token_meta", torch.int32).cpu().numpy().reshape(cache.batch, -1)[:, :n_chunks // cache.batch // cache.n_kv_heads * 64])
        words = cache.view(name + "_index", torch.int32).cpu().numpy().view(np.uint32).astype(np.int64) * 16
        ends = words[:2 * n_chunks].reshape(-1, 2) if cache.pool else np.stack([words[:n_chunks], words[1:n_chunks + 1]], 1)
        arena = (cache.pool.pages if cache.pool else cache.tensors[name + "_arena"]).cpu().numpy()
        out += [arena[a:b] for a, b in ends]
    return out


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("H", [1, 2, 3, 8, 65])
@pytest.mark.parametrize("kw", [dict(), dict(paged=True), dict(repack=binding.REPACK_V_MEDIAN), dict(bits_per_element_budget=4.4),
                                dict(k_rel_scale=1 / 15, v_rel_scale=1 / 7)])
def test_a_nan_is_its_tokens_largest_value(kw, H, bf16):
    kw = dict(kw)
    paged = kw.pop("paged", False)
    B, L = 2, 3 * 64
    K, V, _ = synth.make_kv(B, L, H, H, 5)
    rng = np.random.default_rng(H + 100 * bf16)
    dtype, patterns = (torch.bfloat16, BF16_NANS) if bf16 else (torch.float16, FP16_NANS)
    inputs = [_with_nans(x.cpu().to(dtype), rng, patterns) for x in (K, V)]
    got = []
    for which in (0, 1):
        pool = binding.PagePool(400) if paged else None
        cache = binding.PackedKVCache(B, H, H, L, pool=pool, **kw)
        cache.kv_compress_append(inputs[0][which], inputs[1][which])
        assert cache.kv_cache_stats().overflow == 0
        got.append(_contents(cache, 3 * B * H))
        cache.close()
    for nans, clean in zip(*got):
        assert np.array_equal(nans, clean)
