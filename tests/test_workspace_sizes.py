"""The compressor's staging area in the workspace: never more slots than the cache has chunks, and a workspace of half
as many slots (64 per stream, 256 .. 16384 in all) serves as well, with the same bytes."""
import pytest

from paper_2512_24449_amd import binding

SLOT = binding.CHUNK_MAX_BYTES


def _round256(n):
    return (n + 255) // 256 * 256


def _without_staging(B, Hq):
    return _round256(256 + 65536 * 4 + 64 * B * Hq * 132 * 4)


def _half_staging(B, H):
    return _round256(max(256, min(64 * B * H, 16384)) * SLOT)


@pytest.mark.parametrize("B,H,T", [(1, 1, 64), (1, 1, 1000), (1, 32, 4096), (8, 52, 32000), (1, 8, 20), (2, 3, 131072)])
def test_no_more_staging_slots_than_chunks(B, H, T):
    chunks = -(-T // 64) * B * H
    for query in (binding.kv_query_sizes, binding.kv_query_sizes_paged):
        staging = query(binding.make_config(B, H, H, T)).workspace - _without_staging(B, H)
        assert 0 < staging <= _round256(2 * chunks * SLOT), (staging / SLOT, 2 * chunks)
        assert staging <= 2 * _half_staging(B, H)


@pytest.mark.gpu
@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("B,H,L", [(1, 8, 300 * 64 + 5), (2, 3, 130 * 64), (1, 1, 7 * 64)])
def test_workspace_of_half_the_staging(B, H, L, paged, monkeypatch):
    import torch
    from paper_2512_24449_amd import synth
    name = "kv_query_sizes_paged" if paged else "kv_query_sizes"
    query = getattr(binding, name)
    half = _without_staging(B, H) + min(_half_staging(B, H), _round256(2 * -(-L // 64) * B * H * SLOT))

    def create(workspace=None):
        def sizes(cfg, *bits):
            s = query(cfg, *bits)
            if workspace is not None:
                s.workspace = workspace
            return s
        monkeypatch.setattr(binding, name, sizes)
        pool = binding.PagePool(2 * (-(-L // 64)) * B * H // 14 + 8) if paged else None
        return binding.PackedKVCache(B, H, H, L, pool=pool)

    K, V, q = synth.make_kv(B, L, H, H, 9, device="cuda:0")
    full, small = create(), create(half)
    with pytest.raises(binding.PackKVError):
        create(half - 256)
    for cache in (full, small):
        cache.kv_compress_append(K, V)
    st, st2 = full.kv_cache_stats(), small.kv_cache_stats()
    assert (st2.overflow, st2.k_bytes, st2.v_bytes) == (0, st.k_bytes, st.v_bytes)
    n = L // 64 * B * H
    for t in ("k", "v"):
        words = 2 * n if paged else n + 1
        assert torch.equal(full.view(t + "_index", torch.int32)[:words], small.view(t + "_index", torch.int32)[:words])
        if not paged:
            nbytes = getattr(st, t + "_bytes")
            assert torch.equal(full.tensors[t + "_arena"][:nbytes], small.tensors[t + "_arena"][:nbytes])
    assert torch.equal(full.kv_decode_attention(q, 0.09), small.kv_decode_attention(q, 0.09))
