"""Appends that complete the block in the raw tail: packs of 16 read its first tokens from the tail and the others where
the caller has them, leave those in the tail as well and copy what follows the block to its start.  Packed bytes, index and
metadata against the oracle, the tail against the tokens."""
import numpy as np
import pytest
import torch

from paper_2512_24449_amd import binding, synth
from tests import gpu_cases

pytestmark = pytest.mark.gpu


# kv-heads per wave 1, 2, 4; one, two and four workgroups to an item; 65 heads take the copy first, as does
# an arena that is nearly full
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("pieces", [[1, 63], [63, 1], [37, 27 + 63], [37, 27 + 64 * 2 + 5], [16, 48 + 1], [64 + 15, 49 + 16, 48 + 2]])
@pytest.mark.parametrize("B,H,kind", [(1, 1, ""), (3, 1, ""), (2, 2, ""), (1, 3, ""), (2, 5, "paged"), (2, 20, ""), (8, 52, ""), (1, 64, ""),
                                      (1, 65, ""), (2, 5, "repack"), (1, 17, "tight")])
def test_completed_block(B, H, kind, pieces, dtype):
    L = sum(pieces)
    if (H > 20 or kind) and pieces[0] not in (37, 79):
        pytest.skip("the smaller shapes cover the other splits")
    K, V, _ = synth.make_kv(B, L, H, H, seed=H + L, device="cuda:0")
    K, V = K.to(dtype), V.to(dtype)
    K16, V16 = K.half(), V.half()
    Kn, Vn = K16.cpu().numpy(), V16.cpu().numpy()
    if kind == "repack":
        import oracle
        order = oracle.v_median_order(oracle.compress_v(np.ascontiguousarray(Vn[:, :L // 64 * 64]), 0.2, 16).codes)
        Kn, Vn = (np.concatenate([oracle.apply_order(x, order), x[:, L // 64 * 64:]], axis=1) for x in (Kn, Vn))
    n_packed, ck, cv = gpu_cases.oracle_cache(Kn, Vn)
    pool = binding.PagePool(2 * (L // 64) * B * H // 14 + 8) if kind == "paged" else None
    bits = max(ck.arena.size, cv.arena.size) * 8.0 / (B * H * ((L + 63) // 64 * 64) * 128) + 0.01 if kind == "tight" else 0.0
    cache = binding.PackedKVCache(B, H, H, L, pool=pool, bits_per_element_budget=bits,
                                  repack=binding.REPACK_V_MEDIAN if kind == "repack" else binding.REPACK_NONE)
    for name in ("k_tail", "v_tail"):
        cache.tensors[name].zero_()
    want = [torch.zeros(B, 64, H, 128, dtype=torch.float16, device="cuda:0") for _ in "kv"]
    pos = 0
    for n in pieces:
        cache.kv_compress_append(K[:, pos:pos + n].contiguous(), V[:, pos:pos + n].contiguous())
        for w, x in zip(want, (K16, V16)):
            if pos % 64:      # through the tail up to the end of the block
                take = min(n, 64 - pos % 64)
                w[:, pos % 64:pos % 64 + take] = x[:, pos:pos + take]
            rest = (pos + n) % 64
            if rest and rest <= n:
                w[:, :rest] = x[:, pos + n - rest:pos + n]
        pos += n
    assert cache.tokens == L
    (gpu_cases.check_paged_state if pool else gpu_cases.check_packed_state)(cache, n_packed, ck, cv, B, H)
    for name, w in zip(("k_tail", "v_tail"), want):
        assert torch.equal(cache.view(name, torch.float16)[:w.numel()].view(w.shape), w), name
