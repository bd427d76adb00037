"""Fused attention with a workgroup to a stream, tail included: both sides of every line of the rule (blocks, streams, heads),
tails that end inside a wave's share, four-bit V codes, blocks dropped by a full arena.  Against the oracle."""
import pytest
import torch

from paper_2512_24449_amd import binding, synth
from tests import gpu_cases

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G", [1, 2, 3, 4, 8])
@pytest.mark.parametrize("blocks,tail", [(1, 0), (1, 1), (3, 8), (4, 63), (5, 9), (4, 16)])
def test_few_blocks(G, blocks, tail):
    gpu_cases.run_case(1, 3, 3 * G, 64 * blocks + tail, seed=G + tail, v_rel=0.1 if G % 2 else 0.2)


# 127 / 128: half of the chip, 191 / 192: three quarters, 256 / 257: a stream to a compute unit, 384 / 385 and 512: two
@pytest.mark.parametrize("B,H,G,blocks", [(1, 127, 1, 5), (2, 64, 1, 16), (2, 64, 1, 17), (2, 96, 1, 17), (3, 64, 2, 24), (4, 64, 1, 9), (1, 257, 1, 10),
                                          (1, 257, 1, 11), (5, 77, 1, 12), (8, 64, 1, 3), (1, 513, 1, 3), (6, 43, 2, 3)])
def test_stream_counts(B, H, G, blocks):
    gpu_cases.run_case(B, H, H * G, 64 * blocks + 21, seed=H)


@pytest.mark.parametrize("tail", [0, 5])
def test_dropped_blocks_and_empty_rows(tail):
    """An arena that takes the first append only: later blocks have no part in the result."""
    B, H = 1, 4
    K, V, q = synth.make_kv(B, 192 + tail, H, H, 3, device="cuda:0")
    cache = binding.PackedKVCache(B, H, H, 192 + 64, bits_per_element_budget=1.3)
    cache.kv_compress_append(K[:, :64].contiguous(), V[:, :64].contiguous())
    cache.kv_compress_append(K[:, 64:192].contiguous(), V[:, 64:192].contiguous())
    if tail:
        cache.kv_compress_append(K[:, 192:].contiguous(), V[:, 192:].contiguous())
    assert cache.kv_cache_stats().overflow == 1
    p = cache.kv_softmax(cache.kv_k_matvec(q, 0.09))
    kept = [i for i in range(3) if float(p[..., 64 * i:64 * i + 64].sum()) > 0]
    assert kept == [0]
    torch.testing.assert_close(cache.kv_decode_attention(q, 0.09), cache.kv_v_matvec(p), rtol=1e-3, atol=1e-4)


@pytest.mark.parametrize("G", [1, 4])
@pytest.mark.parametrize("blocks", [1, 4])
def test_tail_tokens_of_weight_zero(G, blocks):
    """Tail tokens whose scores are all -inf, in the share of a wave with a block and of waves without: they weigh nothing."""
    B, H, tail = 1, 3, 40
    L = 64 * blocks + tail
    K, V, q = synth.make_kv(B, L, H, H * G, 6, device="cuda:0")
    q[..., 0] = 1.0
    K[:, 64 * blocks:64 * blocks + 32, :, 0] = float("-inf")
    cache = binding.PackedKVCache(B, H, H * G, L)
    cache.kv_compress_append(K, V)
    out = cache.kv_decode_attention(q, 0.09)
    p = cache.kv_softmax(cache.kv_k_matvec(q, 0.09))
    assert float(p[..., 64 * blocks:64 * blocks + 32].abs().max()) == 0.0 and bool(torch.isfinite(out).all())
    for b in range(B):
        gpu_cases.assert_close_vectors(out[b].cpu().numpy(), cache.kv_v_matvec(p)[b].cpu().numpy(), "fused")


@pytest.mark.parametrize("G", [1, 4])
def test_no_block_and_no_tail(G):
    """The only append overflows the arena: every block is dropped, and the output is exactly 0."""
    B, H = 1, 4
    K, V, q = synth.make_kv(B, 128, H, H * G, 3, device="cuda:0")
    cache = binding.PackedKVCache(B, H, H * G, 128, bits_per_element_budget=1.3)
    cache.kv_compress_append(K, V)
    st = cache.kv_cache_stats()
    assert st.overflow == 1 and (st.k_bytes, st.v_bytes) == (0, 0) and cache.tokens == 128
    assert not cache.kv_decode_attention(q, 0.09).any()
