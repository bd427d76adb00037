"""How the decode kernels cut the blocks of all streams into workgroups: few blocks per wave (whole numbers of
workgroups per stream), ranges that cross stream boundaries, one block in all, and the fused attention on its
flat plan (from eight blocks per resident wave on)."""
import math

import pytest
import torch

from paper_2512_24449_amd import binding, synth
from tests import gpu_cases

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,Hq,L", [(1, 1, 1, 64), (2, 3, 3, 5 * 64 + 9), (16, 16, 16, 7 * 64), (16, 26, 26, 2 * 64 + 1),
                                      (3, 40, 40, 30 * 64), (2, 10, 20, 41 * 64 + 3), (4, 8, 32, 15 * 64), (1, 2, 6, 300 * 64)])
def test_short_streams(B, H, Hq, L):
    gpu_cases.run_case(B, H, Hq, L, seed=L + H)


# 26 streams of 950 blocks and 5 of 5003: both above eight blocks per wave of 768 workgroups, with ranges across boundaries
@pytest.mark.parametrize("B,H,blocks,tail,v_rel", [(2, 13, 950, 17, 0.2), (2, 13, 950, 0, 0.1), (1, 5, 5003, 1, 0.2)])
def test_fused_attention_on_the_flat_plan_equals_the_three_steps(B, H, blocks, tail, v_rel):
    L = blocks * 64 + tail
    K, V, q = synth.make_kv(B, L, H, H, 3, device="cuda:0")
    cache = binding.PackedKVCache(B, H, H, L, v_rel_scale=v_rel)
    cache.kv_compress_append(K, V)
    sm = 1.0 / math.sqrt(128)
    scores = cache.kv_k_matvec(q, sm)
    p = torch.softmax(scores.double(), -1)
    steps = cache.kv_v_matvec(p.float()).double()
    fused = cache.kv_decode_attention(q, sm)
    again = cache.kv_decode_attention(q, sm)
    assert torch.equal(fused, again)
    # both round the block weights to 20 bits below the block's largest: 2^-20 of it per token and path, and the
    # outputs are a few hundredths of sum(p |v|) at these lengths
    rel = (fused.double() - steps).norm(dim=-1) / steps.norm(dim=-1)
    assert float(rel.max()) < 1e-4, float(rel.max())


# segments in registers (up to 64 of 4096 tokens) and beyond them; a row of 16 segments with an odd stride
@pytest.mark.parametrize("Hq,tokens,ld", [(1, 64 * 4096, 64 * 4096), (1, 64 * 4096 + 1, 64 * 4096 + 3), (3, 8192, 8193),
                                          (3, 12289, 12289), (32, 65537, 65539), (2, 300001, 300001)])
def test_softmax_of_few_long_rows(Hq, tokens, ld):
    cache = binding.PackedKVCache(1, 1, Hq, tokens)
    cache.kv_cache_restore(tokens)
    gen = torch.Generator(device="cuda:0").manual_seed(tokens)
    s = 3.0 * torch.randn(1, Hq, ld, device="cuda:0", generator=gen)
    s[0, 0, 100:5000] = -math.inf   # a dropped range
    s[0, Hq - 1, tokens - 1] = 40.0
    want = torch.softmax(s[..., :tokens].double(), -1)
    rest = s[..., tokens:].clone()
    got = cache.kv_softmax(s)
    # exp2 of an argument rounded to 24 bits: up to 2^-24 * |argument| (under 100) relative, plus the fp32 sum
    assert float(((got[..., :tokens].double() - want).abs() / (want + 1e-30)).max()) < 2e-5
    assert torch.equal(got[..., tokens:], rest)
