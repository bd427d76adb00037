"""Wide chunks (packs of 8): codes of up to 31 run in kernels with smaller chunk buffers, two to a wave.  Both sides of that
line, with every pack at its largest width (the largest chunk fills its buffer to the last byte), and mixed layouts."""
import numpy as np
import pytest
import torch

import oracle
from paper_2512_24449_amd import binding
from tests import gpu_cases

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("levels", [16, 31, 32, 255])
@pytest.mark.parametrize("Hq", [2, 8, 16])
def test_largest_chunks(levels, Hq):
    B, H, L = 1, 2, 5 * 64 + 9
    rng = np.random.default_rng(levels)
    codes = rng.integers(0, levels + 1, size=(2, B, L, H, 128))
    # every pack of 8 tokens holds both ends of the range, and so does every token
    low = (np.arange(L)[:, None, None] % 2 == 0) == (np.arange(128)[None, None, :] % 2 == 0)
    codes[:, :, np.arange(L) % 8 < 2] = np.where(low, 0, levels)[None, None, np.arange(L) % 8 < 2]
    codes[:, :, :, :, 0], codes[:, :, :, :, 1] = 0, levels
    codes[:, :, 1::8, :, 0], codes[:, :, 1::8, :, 1] = levels, 0
    K, V = ((codes - levels // 2) / 16.0).astype(np.float16)
    q = (rng.standard_normal((B, Hq, 128))).astype(np.float16)
    rel = 1.0 / levels
    cache = binding.PackedKVCache(B, H, Hq, L, k_rel_scale=rel, v_rel_scale=rel, pack_size=8)
    cache.kv_compress_append(torch.from_numpy(K).cuda(), torch.from_numpy(V).cuda())
    n_packed, ck, cv = gpu_cases.oracle_cache(K, V, rel, rel, 8)
    st = gpu_cases.check_packed_state(cache, n_packed, ck, cv, B, H)
    if levels == 31:
        assert st.k_bytes == st.n_chunks * (2048 + 1024 * 5)
    out = cache.kv_decode_attention(torch.from_numpy(q).cuda(), 0.05).cpu().numpy()
    kcodes, kmeta = gpu_cases.full_codes(ck, K.shape, n_packed)
    vcodes, vmeta = gpu_cases.full_codes(cv, V.shape, n_packed)
    gpu_cases.assert_close_vectors(out, oracle.attention(kcodes, K, kmeta, vcodes, V, vmeta, n_packed, q, 0.05), "fused")
    s = cache.kv_k_matvec(torch.from_numpy(q).cuda(), 0.05)
    gpu_cases.assert_close_vectors(s.cpu().numpy(), oracle.k_scores(kcodes, K, kmeta, n_packed, q, 0.05), "K")
    cache.kv_softmax(s)
    gpu_cases.assert_close_vectors(cache.kv_v_matvec(s).cpu().numpy(), oracle.v_out(vcodes, V, vmeta, n_packed, s.cpu().numpy()), "V")


@pytest.mark.parametrize("k_rel,v_rel", [(1 / 31, 0.2), (0.1, 1 / 31), (1 / 31, 1 / 32), (1 / 32, 0.2), (1 / 20, 1 / 31)])
@pytest.mark.parametrize("H,Hq,L", [(2, 2, 9 * 64 + 1), (1, 5, 4 * 64), (3, 24, 6 * 64 + 63)])
def test_mixed_layouts(k_rel, v_rel, H, Hq, L):
    gpu_cases.run_case(1, H, Hq, L, seed=Hq, pack_size=8, k_rel=k_rel, v_rel=v_rel)


def _workgroups(streams, n_blocks):
    """Workgroups of the K product and of the fused attention (target_workgroups and the splits of csrc)."""
    target = min(max(streams * n_blocks // 32, 512), 4096)
    per_group = max(4, -(-(-(-n_blocks // max(1, target // streams))) // 4) * 4)
    splits = min(-(-target // streams), -(-n_blocks // 4), 64)
    return streams * -(-n_blocks // per_group), streams * -(-n_blocks // -(-n_blocks // splits))


# More workgroups than the kernels with two smaller buffers run at once, two to a compute unit: the other kernels take codes
# of up to 31 as well.  Both batch elements have the same contents, and a cache of one of them stays on the near side of the
# line (all its results depend on its own tokens only).  Heads repeat two base heads, so that the oracle has little to do.
@pytest.mark.parametrize("Hq", [32, 96])
def test_both_sides_of_the_line_between_buffers(Hq):
    B, H, blocks = 2, 32, 400
    L, G = blocks * 64 + 5, Hq // H
    room = 2 * torch.cuda.get_device_properties(0).multi_processor_count
    assert max(_workgroups(H, blocks)) <= room < min(_workgroups(B * H, blocks)), "one kernel on both sides"
    g = torch.Generator(device="cuda:0").manual_seed(Hq)
    K, V = (torch.randn((1, L, 2, 128), generator=g, device="cuda:0").to(torch.float16) for _ in range(2))
    q = torch.randn((1, Hq, 128), generator=g, device="cuda:0").to(torch.float16)
    got = []
    for batch in (1, B):
        cache = binding.PackedKVCache(batch, H, Hq, L, k_rel_scale=1 / 31, v_rel_scale=1 / 31, pack_size=8)
        cache.kv_compress_append(K.repeat(batch, 1, H // 2, 1), V.repeat(batch, 1, H // 2, 1))
        qb = q.expand(batch, -1, -1).contiguous()
        got.append((cache.kv_k_matvec(qb, 0.05)[:, :, :L].cpu().numpy(), cache.kv_decode_attention(qb, 0.05).cpu().numpy()))
        assert cache.kv_cache_stats().overflow == 0
    for b in range(B):
        gpu_cases.assert_close_vectors(got[1][0][b], got[0][0][0], "K", tol=1e-5)
        gpu_cases.assert_close_vectors(got[1][1][b], got[0][1][0], "fused", tol=1e-5)
    K, V = K.cpu().numpy(), V.cpu().numpy()
    n_packed, ck, cv = gpu_cases.oracle_cache(K, V, 1 / 31, 1 / 31, 8)
    (kcodes, kmeta), (vcodes, vmeta) = gpu_cases.full_codes(ck, K.shape, n_packed), gpu_cases.full_codes(cv, V.shape, n_packed)
    by_base = sorted(range(Hq), key=lambda i: i // G % 2)
    qn = q.cpu().numpy()[:, by_base]
    gpu_cases.assert_close_vectors(got[0][0][:, by_base], oracle.k_scores(kcodes, K, kmeta, n_packed, qn, 0.05), "K against the oracle")
    gpu_cases.assert_close_vectors(got[0][1][:, by_base], oracle.attention(kcodes, K, kmeta, vcodes, V, vmeta, n_packed, qn, 0.05),
                                   "fused against the oracle")
