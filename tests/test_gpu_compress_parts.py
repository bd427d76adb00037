"""The compressor of packs of 16 at the edges of its split: the staging area holds half of its slots
per tensor, a compaction workgroup takes four chunks and adds up the sizes before them; both tensors share
every launch.  Bytes, index and metadata against the oracle, bit for bit."""
import pytest
import torch

from tests import gpu_cases

pytestmark = pytest.mark.gpu


# 1 x 1: 256 chunks of each tensor to a part; 1 x 3: 256; 3 x 4: 768
@pytest.mark.parametrize("B,H,blocks,tail", [(1, 1, 1, 0), (1, 1, 3, 5), (1, 1, 4, 0), (1, 1, 5, 63), (1, 1, 255, 0), (1, 1, 256, 1),
                                             (1, 1, 257, 0), (1, 3, 85, 0), (1, 3, 86, 2), (3, 4, 64, 0), (3, 4, 65, 0)])
def test_parts_and_four_chunk_groups(B, H, blocks, tail):
    gpu_cases.run_case(B, H, H, blocks * 64 + tail, seed=31 * blocks + tail)


@pytest.mark.parametrize("pieces", [[64, 64, 64], [63, 1, 64], [128, 1, 63, 64]])
def test_small_rounds_behind_one_another(pieces):
    gpu_cases.run_case(2, 5, 10, sum(pieces), seed=77, pieces=pieces)


def test_append_behind_restored_contents_in_a_tight_arena():
    """A cache that adopts packed contents and has room for a little more: the append finds that its chunks may
    not fit even though the handle has appended nothing itself, and packs them all the same."""
    from paper_2512_24449_amd import binding, synth
    B, H, T, more = 1, 16, 64 * 64, 64 * 64
    K, V, _ = synth.make_kv(B, T + more, H, H, 5, device="cuda:0")
    full = binding.PackedKVCache(B, H, H, T + more)
    full.kv_compress_append(K, V)
    want = full.kv_cache_stats()
    bits = max(want.k_bytes, want.v_bytes) * 8.0 / (B * H * (T + more) * 128) + 0.01
    tight = binding.PackedKVCache(B, H, H, T + more, bits_per_element_budget=bits)
    first = binding.PackedKVCache(B, H, H, T + more)
    first.kv_compress_append(K[:, :T].contiguous(), V[:, :T].contiguous())
    st = first.kv_cache_stats()
    for name, n in (("k_arena", st.k_bytes), ("v_arena", st.v_bytes), ("k_index", None), ("v_index", None),
                    ("k_token_meta", None), ("v_token_meta", None)):
        tight.tensors[name][:n].copy_(first.tensors[name][:n])
    torch.cuda.synchronize()
    tight.kv_cache_restore(T)
    tight.kv_compress_append(K[:, T:].contiguous(), V[:, T:].contiguous())
    got = tight.kv_cache_stats()
    assert (got.overflow, got.k_bytes, got.v_bytes) == (0, want.k_bytes, want.v_bytes)
    for name, n in (("k_arena", want.k_bytes), ("v_arena", want.v_bytes)):
        assert torch.equal(tight.tensors[name][:n], full.tensors[name][:n])
