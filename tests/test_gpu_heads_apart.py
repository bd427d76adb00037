"""The query heads of a group share matrix-core tiles, but no result: weights or a query that are no numbers spoil the
outputs of their own head only (bitwise: the others are what they are beside a head of zeros)."""
import pytest
import torch

from paper_2512_24449_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G", [2, 3, 4, 5, 8])
@pytest.mark.parametrize("pack_size,rel", [(16, 0.2), (16, 0.1), (8, 0.2), (8, 0.05)])
@pytest.mark.parametrize("tokens", [6 * 64 + 9, 40 * 64])
def test_a_head_without_numbers_stays_alone(G, pack_size, rel, tokens):
    H, Hq = 2, 2 * G
    K, V, q = synth.make_kv(1, tokens, H, Hq, G, device="cuda:0")
    cache = binding.PackedKVCache(1, H, Hq, tokens, k_rel_scale=rel, v_rel_scale=rel, pack_size=pack_size)
    cache.kv_compress_append(K, V)
    p = torch.rand(1, Hq, tokens, device="cuda:0", generator=torch.Generator(device="cuda:0").manual_seed(G))
    for spoilt in (0, G - 1):
        others = [i for i in range(Hq) if i != spoilt]
        got = []
        for bits in (0, 0x7FC00000, -0x400000):  # zeros, and quiet NaNs of either sign
            ps, qs = p.clone(), q.clone()
            ps.view(torch.int32)[0, spoilt] = bits
            qs.view(torch.int16)[0, spoilt] = 0 if bits == 0 else 0x7E00 if bits > 0 else -0x200
            got.append((cache.kv_v_matvec(ps)[0, others], cache.kv_decode_attention(qs, 0.09)[0, others]))
        for v, attention in got[1:]:
            assert torch.equal(v, got[0][0]) and torch.equal(attention, got[0][1])
