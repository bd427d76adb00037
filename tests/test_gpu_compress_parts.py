"""The compressor of packs of 16 at the edges of its split: the staging area holds half of its slots
per tensor, an assembling workgroup takes four chunks and adds up the sizes before them; both tensors share
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


# One read of the input, packs of 16: kv-heads per wave (1, 2, 4 rows), waves per workgroup, workgroups that share an
# item (few items: 1, 2 or 4 per item at 20 heads), more kv-heads than a workgroup holds (token parameters first)
@pytest.mark.parametrize("B,H,blocks", [(1, 1, 2), (3, 1, 5), (2, 2, 3), (1, 3, 2), (1, 4, 1), (2, 5, 1), (1, 16, 1), (1, 17, 2),
                                        (1, 20, 7), (2, 20, 9), (1, 33, 1), (1, 64, 1), (1, 65, 1), (1, 81, 2)])
@pytest.mark.parametrize("repack", [False, True])
def test_heads_per_wave_and_shared_items(B, H, blocks, repack):
    if repack and H > 20 and H != 65:
        pytest.skip("the oracle's order takes long; 17 and 65 heads cover the head sets")
    gpu_cases.run_case(B, H, H, blocks * 64 + 1, seed=blocks + H, repack=repack)


# rel: the largest quotient reaches qmax + 1/2 (every value clamped), and does not
@pytest.mark.parametrize("rel", [0.0953, 2 / 21, 0.1, 1 / 15])
@pytest.mark.parametrize("magnitude", [1.0, 2.0 ** -14, 2.0 ** -20, 2.0 ** -22, 2.0 ** -24])
def test_tiny_scales_and_ties(rel, magnitude):
    """Ranges down to fp16's smallest steps, where a scale's own rounding lets quotients pass qmax, and values on and next
    to rounding ties: bytes against the oracle."""
    import numpy as np
    from paper_2512_24449_amd import binding
    rng = np.random.default_rng(3)
    K = (rng.integers(-12, 13, size=(1, 192, 5, 128)) * magnitude).astype(np.float16)
    V = (rng.standard_normal((1, 192, 5, 128)) * 4 * magnitude).astype(np.float16)
    V[0, 64:128] = (rng.integers(0, 22, size=(64, 5, 128)) * 0.5 * magnitude).astype(np.float16)
    cache = binding.PackedKVCache(1, 5, 5, 192, k_rel_scale=rel, v_rel_scale=rel)
    cache.kv_compress_append(torch.from_numpy(K).cuda(), torch.from_numpy(V).cuda())
    n_packed, ck, cv = gpu_cases.oracle_cache(K, V, rel, rel)
    gpu_cases.check_packed_state(cache, n_packed, ck, cv, 1, 5)


# Token parameters and V-median keys in one kernel: rows of up to 1024, 2048 and 4096 values in registers, longer ones
# read twice; a last piece of 512 values that is not full
@pytest.mark.parametrize("H", [8, 9, 31, 32, 33, 66])
def test_rows_of_keys_and_token_parameters(H):
    gpu_cases.run_case(1, H, H, 64, seed=H, repack=True)
