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
