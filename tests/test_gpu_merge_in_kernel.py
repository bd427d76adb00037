"""Short contexts of few streams: the last workgroup of a stream merges the partial rows inside the V product and the
fused attention (csrc/last_group.h; up to 32 streams and 128 workgroups, 64 with wide chunks, up to four heads).  Against the oracle on both sides
of that line, with tails that end in every wave's part of it, and replayed from a graph."""
import pytest
import torch

from tests import gpu_cases

pytestmark = pytest.mark.gpu


# heads per kv-head 1 .. 8, tails around 16, 32 and 48 tokens, a context that is all tail or has none
@pytest.mark.parametrize("B,H,Hq,L", [(1, 1, 1, 64), (1, 1, 1, 15 * 64 + 1), (1, 32, 32, 4 * 64 + 16), (1, 33, 33, 4 * 64 + 17),
                                      (2, 16, 16, 17 * 64 + 48), (1, 8, 16, 64 * 17 + 63), (1, 3, 9, 5 * 64 + 31), (2, 2, 8, 9 * 64 + 33),
                                      (1, 2, 10, 3 * 64 + 49), (1, 2, 16, 6 * 64 + 5), (1, 8, 32, 64 * 64), (1, 9, 36, 61 * 64 + 32)])
def test_merged_streams(B, H, Hq, L):
    gpu_cases.run_case(B, H, Hq, L, seed=L + Hq)


@pytest.mark.parametrize("B,H,Hq,L", [(1, 2, 2, 33 * 64 + 20), (1, 4, 12, 16 * 64), (1, 1, 7, 5 * 64 + 63), (1, 8, 40, 33 * 64 + 1), (4, 8, 8, 9 * 64 + 7)])
@pytest.mark.parametrize("k_rel,v_rel", [(0.1, 0.2), (0.05, 0.05), (0.1, 0.05)])
def test_merged_streams_pack8(B, H, Hq, L, k_rel, v_rel):
    gpu_cases.run_case(B, H, Hq, L, seed=L + Hq, pack_size=8, k_rel=k_rel, v_rel=v_rel)


def test_replays_of_a_captured_step():
    """The counters are back at zero after every call: replays with eager calls between them give the eager result."""
    from paper_2512_24449_amd import binding, synth
    B, H, Hq, L = 1, 8, 32, 20 * 64 + 37
    K, V, q = synth.make_kv(B, L, H, Hq, 4, device="cuda:0")
    cache = binding.PackedKVCache(B, H, Hq, L)
    cache.kv_compress_append(K, V)
    out, out_v = torch.empty(B, Hq, 128, device="cuda:0"), torch.empty(B, Hq, 128, device="cuda:0")
    p = torch.empty(B, Hq, L, device="cuda:0")

    def step():
        cache.kv_decode_attention(q, 0.09, out=out)
        cache.kv_k_matvec(q, 0.09, scores=p)
        cache.kv_softmax(p)
        cache.kv_v_matvec(p, out=out_v)

    step()
    torch.cuda.synchronize()
    want, want_v = out.clone(), out_v.clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for _ in range(4):
        out.zero_(), out_v.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want) and torch.equal(out_v, want_v)
        out.zero_(), out_v.zero_()
        step()
        torch.cuda.synchronize()
        assert torch.equal(out, want) and torch.equal(out_v, want_v)
