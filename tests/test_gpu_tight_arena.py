"""Packs of 16, an arena that has room for what an append needs but not for its largest chunks: the round is done in two
passes, and nothing is staged for the tensor that is (the bytes of its staging slots are never written).  Either tensor or
both, token metadata found by the first kernel or given, several parts; contents against a cache with room for anything."""
import ctypes as C

import pytest
import torch

from paper_2512_24449_amd import binding, synth

pytestmark = pytest.mark.gpu


def _with_sizes(cache, **sizes):
    """Rebuilds the handle over the same buffers with other sizes."""
    cache.close()
    for name, n in sizes.items():
        setattr(cache.sizes, name, n)
    bufs, handle = binding.kv_buffers_t(), C.c_void_p()
    for name, t in cache.tensors.items():
        setattr(bufs, name, t.data_ptr() if t.numel() else None)
    binding._check(binding.lib().kv_cache_create(C.byref(cache.cfg), C.byref(bufs), C.byref(cache.sizes), C.byref(handle)), "create")
    cache.handle = handle


@pytest.mark.parametrize("tight", ["k", "v", "kv"])
@pytest.mark.parametrize("B,H,blocks", [(1, 1, 3), (2, 2, 5), (1, 3, 2), (2, 8, 1), (1, 20, 5), (2, 65, 2), (1, 2, 300)])
@pytest.mark.parametrize("repack", [binding.REPACK_NONE, binding.REPACK_V_MEDIAN])
def test_nothing_is_staged_for_a_tight_arena(tight, B, H, blocks, repack):
    L = blocks * 64
    K, V, _ = synth.make_kv(B, L, H, H, blocks + H, device="cuda:0")
    full = binding.PackedKVCache(B, H, H, L, repack=repack)
    full.kv_compress_append(K, V)
    want = full.kv_cache_stats()
    cache = binding.PackedKVCache(B, H, H, L, repack=repack)
    nbytes = {"k": want.k_bytes, "v": want.v_bytes}
    assert all(nbytes[t] < blocks * B * H * binding.CHUNK_MAX_BYTES for t in tight)
    _with_sizes(cache, **{t + "_arena": nbytes[t] for t in tight})
    # a part's slots: one of the largest chunk's size for each of its chunks, K's first; behind status words (256 bytes),
    # chunk sizes (65536 words) and partial rows (64 per query head, of 132 floats)
    offset = (256 + 65536 * 4 + 64 * B * H * 132 * 4 + 255) // 256 * 256
    staging = cache.tensors["workspace"][offset:]
    slots, rows = min(max(B * H * 128, 512), 16384, 2 * blocks * B * H), blocks * B
    parts = -(-rows // (slots // 2 // H))
    n = -(-rows // parts) * H
    staging.fill_(0xA5)
    cache.kv_compress_append(K, V)
    got = cache.kv_cache_stats()
    assert (got.overflow, got.k_bytes, got.v_bytes) == (0, want.k_bytes, want.v_bytes)
    for t in "kv":
        assert torch.equal(cache.tensors[t + "_arena"][:nbytes[t]], full.tensors[t + "_arena"][:nbytes[t]])
        for name in ("_index", "_token_meta"):
            words = (blocks * B * H + 1) if name == "_index" else B * L
            assert torch.equal(cache.view(t + name, torch.int32)[:words], full.view(t + name, torch.int32)[:words])
    part = n * binding.CHUNK_MAX_BYTES
    untouched = {"k": bool((staging[:part] == 0xA5).all()), "v": bool((staging[part:2 * part] == 0xA5).all())}
    if parts == 1:
        assert untouched == {"k": "k" in tight, "v": "v" in tight}
    elif tight == "kv":
        assert bool((staging == 0xA5).all())
    for c in (cache, full):
        c.close()
