"""How the decode kernels cut the blocks of all streams into workgroups: few blocks per wave (whole numbers of
workgroups per stream), one block in all, the fused attention on its flat plan (from eight blocks per resident wave
on), and ranges that cross stream boundaries.  The shapes of CROSSING_STEPS and CROSSING_FUSED do cross, however many
workgroups of a kernel fit a compute unit: test_work_split_plan.py checks that against the rule of the dispatch."""
import math

import pytest
import torch

from paper_2512_24449_amd import binding, synth
from tests import gpu_cases
from tests.test_gpu_fullsize import _check_batch_element

pytestmark = pytest.mark.gpu


# (batch, kv-heads, blocks); streams = batch * kv-heads (times 5 where five queries share a kv-head: they are split
# into as many streams)
CROSSING_STEPS = [(9, 57, 17)]
CROSSING_FUSED = [(9, 25, 150), (9, 15, 257)]
CROSSING_FUSED_SPLIT = [(9, 5, 150)]


@pytest.mark.parametrize("B,H,Hq,L", [(1, 1, 1, 64), (2, 3, 3, 5 * 64 + 9), (16, 16, 16, 7 * 64), (16, 26, 26, 2 * 64 + 1),
                                      (3, 40, 40, 30 * 64), (2, 10, 20, 41 * 64 + 3), (4, 8, 32, 15 * 64), (1, 2, 6, 300 * 64)])
def test_short_streams(B, H, Hq, L):
    gpu_cases.run_case(B, H, Hq, L, seed=L + H)


# 26 streams of 950 blocks and 5 of 5003: both above eight blocks per wave of 768 workgroups, a whole number of workgroups per stream
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


def _decode(B, H, G, blocks, tail, v_rel, elements):
    """Every decode entry point on a filled cache, the named batch elements against the oracle."""
    L = blocks * 64 + tail
    K, V, q = synth.make_kv(B, L, H, H * G, 11 + blocks, device="cuda:0")
    cache = binding.PackedKVCache(B, H, H * G, L, v_rel_scale=v_rel)
    cache.kv_compress_append(K, V)
    sm = 1.0 / math.sqrt(128)
    scores = cache.kv_k_matvec(q, sm)
    p = synth.make_probs(scores)
    out = cache.kv_v_matvec(p)
    attn = cache.kv_decode_attention(q, sm)
    for _ in range(2):
        assert torch.equal(scores, cache.kv_k_matvec(q, sm))
        assert torch.equal(out, cache.kv_v_matvec(p))
        assert torch.equal(attn, cache.kv_decode_attention(q, sm))
    # every output of every stream: both paths round their weights to at least 16 bits below a block's largest
    # and the outputs are some hundredths of sum(p |v|) at these lengths
    gpu_cases.assert_close_vectors(attn.cpu().numpy(), out.cpu().numpy(), "fused against three steps")
    for b in elements:
        _check_batch_element(cache, K, V, q, scores, p, out, b, sm, blocks * 64, attn=attn, v_rel=v_rel)


@pytest.mark.parametrize("v_rel", [0.2, 0.1])
@pytest.mark.parametrize("G", [1, 2, 4])
@pytest.mark.parametrize("B,H,blocks", CROSSING_STEPS)
def test_steps_across_stream_boundaries(B, H, blocks, G, v_rel):
    _decode(B, H, G, blocks, 13 * (G - 1), v_rel, [0, B - 1])


@pytest.mark.parametrize("v_rel", [0.2, 0.1])
@pytest.mark.parametrize("B,H,G,blocks", [(B, H, 1, n) for B, H, n in CROSSING_FUSED] + [(B, H, 5, n) for B, H, n in CROSSING_FUSED_SPLIT])
def test_fused_attention_across_stream_boundaries(B, H, G, blocks, v_rel):
    _decode(B, H, G, blocks, 21, v_rel, [B - 1])
