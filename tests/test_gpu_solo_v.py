"""V product with a workgroup to a stream, tail included: both sides of every line of the rule, tails that end inside a wave's share,
four-bit codes, the entry point that allocates nothing.  Against the oracle."""
import pytest
import torch

from paper_2512_24449_amd import binding, synth
from tests import gpu_cases

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G", [1, 2, 3, 4, 8])
@pytest.mark.parametrize("blocks,tail", [(1, 0), (7, 1), (8, 8), (9, 63), (16, 9), (17, 16)])
def test_few_blocks(G, blocks, tail):
    gpu_cases.run_case(1, 3, 3 * G, 64 * blocks + tail, seed=G + tail, v_rel=0.1 if G % 2 else 0.2)


# 127 / 128: half of the chip, 191 / 192: three quarters, 256 / 257: a stream to a compute unit, 384 / 385 and 512: two
@pytest.mark.parametrize("B,H,G,blocks", [(1, 127, 1, 17), (2, 64, 1, 32), (2, 64, 1, 33), (2, 96, 2, 33), (1, 257, 1, 30), (1, 257, 1, 31), (5, 77, 1, 31),
                                          (6, 43, 4, 9), (1, 513, 1, 3)])
def test_stream_counts(B, H, G, blocks):
    gpu_cases.run_case(B, H, H * G, 64 * blocks + 21, seed=H)


@pytest.mark.parametrize("G", [1, 4])
def test_without_workspace_and_around_other_calls(G):
    """The two V entry points and the fused attention, in turn, many times: nothing of one is left for another."""
    B, H, L = 2, 3, 64 * 7 + 11
    K, V, q = synth.make_kv(B, L, H, H * G, 5, device="cuda:0")
    cache = binding.PackedKVCache(B, H, H * G, L)
    cache.kv_compress_append(K, V)
    p = cache.kv_softmax(cache.kv_k_matvec(q, 0.09))
    first = cache.kv_v_matvec(p)
    fused = cache.kv_decode_attention(q, 0.09)
    out = torch.empty_like(first)
    for _ in range(5):
        assert torch.equal(cache.kv_v_matvec_noalloc(p, out), first)
        assert torch.equal(cache.kv_decode_attention(q, 0.09), fused)
        assert torch.equal(cache.kv_v_matvec(p), first)
