"""Fused attention: softmax weights down to fp32's subnormals take part in an output that has no larger ones."""
import math

import pytest
import torch

from paper_2512_24449_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("log2_weight", [-120, -128, -131])
@pytest.mark.parametrize("pack,k_rel,v_rel", [(16, 0.1, 0.2), (16, 0.1, 0.1), (8, 0.1, 0.2), (8, 0.05, 0.2), (8, 0.1, 0.05),
                                              (8, 0.05, 0.05)])
@pytest.mark.parametrize("G", [1, 4])
def test_weights_below_the_normal_range(pack, k_rel, v_rel, G, log2_weight):
    """Token 0 holds the row's largest score and a value of zero, the 63 others of its block weigh 2^log2_weight
    of it and hold 30000.  Constant tokens have scale 0: the stored values are exact, and the output is
    63 * 30000 * 2^log2_weight over a weight sum of 1."""
    K = torch.zeros(1, 64, 1, synth.HEAD_DIM, dtype=torch.float16, device="cuda:0")
    V = torch.full_like(K, 30000.0)
    K[0, 0], V[0, 0] = 1.0, 0.0
    q = torch.ones(1, G, synth.HEAD_DIM, dtype=torch.float16, device="cuda:0")
    cache = binding.PackedKVCache(1, 1, G, 64, k_rel_scale=k_rel, v_rel_scale=v_rel, pack_size=pack)
    cache.kv_compress_append(K, V)
    out = cache.kv_decode_attention(q, -log2_weight * math.log(2.0) / synth.HEAD_DIM)
    want = 63 * 30000.0 * 2.0 ** log2_weight
    # the score is around -130: half an ulp of fp32 there (2^-17) and of sm_scale is 2e-5 in the exponent, and a
    # subnormal 2^-131 keeps 18 bits
    assert float((out.double() / want - 1).abs().max()) < 1e-4, out.flatten()[:4]
