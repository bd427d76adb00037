"""NaNs and infinities in the input through every way a round is compressed: staged, in two passes because the arena may be too full, in
two passes instead of many small parts, in pages beyond the staging area.  All of them give the same metadata and chunks, every chunk fills its
place in the index exactly and nothing is written outside the chunks; with NaNs the cache holds what it holds with the token's largest value in their place."""
import numpy as np
import pytest
import torch

from paper_2512_24449_amd import binding, synth
from tests.test_gpu_nan_confined import BF16_NANS, FP16_NANS, _contents, _with_nans

pytestmark = pytest.mark.gpu
FILL = 0xAA


def _append(B, H, L, K, V, pool_pages=0, **kw):
    pool = binding.PagePool(pool_pages) if pool_pages else None
    cache = binding.PackedKVCache(B, H, H, L, pool=pool, **kw)
    arenas = [pool.pages] if pool else [cache.tensors["k_arena"], cache.tensors["v_arena"]]
    for x in arenas:
        x.fill_(FILL)
    cache.kv_compress_append(K, V)
    st = cache.kv_cache_stats()
    assert st.overflow == 0
    n = L // 64 * B * H
    contents = _contents(cache, n)
    written = [np.zeros(x.numel(), bool) for x in arenas]
    for i, name in enumerate(("k", "v")):
        words = cache.view(name + "_index", torch.int32).cpu().numpy().view(np.uint32).astype(np.int64) * 16
        for a, b in words[:2 * n].reshape(-1, 2) if pool else np.stack([words[:n], words[1:n + 1]], 1):
            written[0 if pool else i][a:b] = True
    for x, w in zip(arenas, written):
        assert (x.cpu().numpy()[~w] == FILL).all(), "bytes outside the chunks"
    rels = (kw.get("k_rel_scale", 0.1), kw.get("v_rel_scale", 0.2))
    for i, rel in enumerate(rels):
        for chunk in contents[i * (n + 1) + 1:(i + 1) * (n + 1)]:
            wide = rel < 1 / 15.5
            header, step = (512, 2) if kw["pack_size"] == 16 else (2048 if wide else 1024, 1)
            widths = chunk[:1024].astype(int) if wide else chunk[:header].astype(int) >> 4
            assert (header + step * widths.sum() + 15) // 16 * 16 == chunk.size, "a chunk and its place in the index"
    cache.close()
    return contents, max(st.k_bytes, st.v_bytes) * 8.0 / (n * 64 * 128)


def _same(a, b, what):
    for x, y in zip(a, b):
        assert np.array_equal(x, y), what


def _one_value(nans, clean, rng):
    """Two tokens of one value, a scale of 0: a NaN is that value there."""
    patterns = np.array(BF16_NANS if nans.dtype == torch.bfloat16 else FP16_NANS, np.uint16)
    for t, value in ((9, 1.5), (70, 0.0)):
        nans[:, t], clean[:, t] = value, value
        some = nans[:, t, :, 1::3]
        nans[:, t, :, 1::3] = torch.from_numpy(rng.choice(patterns, tuple(some.shape)).view(np.int16)).view(nans.dtype).to(nans.device)


def _with_infinities(x, rng):
    B, L = x.shape[:2]
    x = x.clone().view(B, L, -1)
    at = torch.from_numpy((rng.random(x.shape) < 0.004) & (rng.random((B, L, 1)) < 0.5))
    at[:, 3, 1:] = True
    big = torch.tensor([float("inf"), float("-inf"), 1e30 if x.dtype == torch.bfloat16 else float("inf")], dtype=x.dtype)
    return torch.where(at, big[torch.from_numpy(rng.integers(0, 3, x.shape))], x)


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("layout", [dict(pack_size=16), dict(pack_size=8), dict(pack_size=8, k_rel_scale=0.05, v_rel_scale=1 / 31),
                                    dict(pack_size=8, k_rel_scale=0.05), dict(pack_size=8, v_rel_scale=1 / 127)])
@pytest.mark.parametrize("B,H,blocks", [(1, 1, 257), (1, 3, 90), (2, 5, 27)])   # all beyond 256 chunks of a tensor
def test_one_result_by_every_way(B, H, blocks, layout, dtype):
    L = 64 * blocks
    K, V, _ = synth.make_kv(B, L, H, H, 7)
    rng = np.random.default_rng(B + H)
    inputs = {"nan": [], "clean": [], "inf": []}
    for x in (K, V):
        x = x.cpu().to(dtype)
        nans, clean = (y.cpu() for y in _with_nans(x, rng, BF16_NANS if dtype == torch.bfloat16 else FP16_NANS))
        _one_value(nans, clean, rng)
        inputs["nan"].append(nans.cuda()), inputs["clean"].append(clean.cuda())
        inputs["inf"].append(_with_infinities(x, rng).view_as(x).cuda())
    staged = {}
    for kind, (k, v) in inputs.items():
        short, bits = _append(B, H, L, k, v, **layout)   # (1 x 1 and 1 x 3: two passes instead of small parts)
        staged[kind] = short
        _same(short, _append(B, H, L, k, v, bits_per_element_budget=bits + 0.02, **layout)[0], (kind, "nearly full arena"))
        _same(short, _append(B, H, L, k, v, pool_pages=2 * (blocks * B * H // 6 + 8), **layout)[0], (kind, "pages"))
        # block by block: rounds that are staged for sure
        pool = binding.PagePool(2 * (blocks * B * H // 6 + 8))
        cache = binding.PackedKVCache(B, H, H, L, pool=pool, **layout)
        for at in range(0, L, 16 * 64):
            cache.kv_compress_append(k[:, at:at + 16 * 64].contiguous(), v[:, at:at + 16 * 64].contiguous())
        _same(short, _contents(cache, blocks * B * H), (kind, "small rounds"))
        cache.close()
    _same(staged["nan"], staged["clean"], "a NaN and the largest value")


@pytest.mark.parametrize("layout", [dict(pack_size=16), dict(pack_size=8), dict(pack_size=8, k_rel_scale=0.05)])
@pytest.mark.parametrize("bits", [0.0, 4.9])
def test_repacked_tokens(layout, bits):
    """Codes moved into storage order, and the order found first (arenas that may be too full; a wide tensor)."""
    B, H, L = 2, 3, 3 * 64
    K, V, _ = synth.make_kv(B, L, H, H, 8)
    rng = np.random.default_rng(3)
    got = []
    pairs = [_with_nans(x.cpu().half(), rng, FP16_NANS) for x in (K, V)]
    for nans, clean in pairs:
        _one_value(nans, clean, rng)
    wide = 7.5 if bits and "k_rel_scale" in layout else bits
    for which in (0, 1):
        got.append(_append(B, H, L, pairs[0][which], pairs[1][which], repack=binding.REPACK_V_MEDIAN, bits_per_element_budget=wide, **layout)[0])
    _same(*got, "a NaN and the largest value")
