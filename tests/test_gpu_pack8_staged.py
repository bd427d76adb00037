"""Packs of 8 and wide chunks through the staging area (one read of the input): edges of its split, the layouts side by side,
the largest code it takes and the first it does not, blocks completed in the tail, pages.  Bytes, index and metadata against
the oracle, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2512_24449_amd import binding, synth
from tests import gpu_cases

pytestmark = pytest.mark.gpu

NARROW, WIDE = (0.1, 0.2), (0.05, 0.05)


# 256 chunks of each tensor to a part at 1 x 1; heads per wave 1, 2, 4; shared items; parameters first (65 heads, repacked)
@pytest.mark.parametrize("B,H,blocks,repack", [(1, 1, 1, False), (1, 1, 257, False), (3, 1, 5, True), (2, 2, 3, False), (1, 3, 2, False),
                                               (2, 5, 1, True), (2, 20, 2, False), (1, 64, 1, False), (1, 65, 1, False)])
@pytest.mark.parametrize("rels", [NARROW, WIDE, (0.05, 0.2), (0.1, 0.05)])
def test_bytes(B, H, blocks, repack, rels):
    gpu_cases.run_case(B, H, H, blocks * 64 + 1, seed=blocks + H, pack_size=8, k_rel=rels[0], v_rel=rels[1], repack=repack)


# 127 and 128 levels (7 and 8 bits), 16 levels, a scale whose quotients pass qmax + 1/2 (every value clamped)
@pytest.mark.parametrize("rel", [1 / 127, 1 / 128, 1 / 255, 1 / 16, 2 / 41, 0.0488])
@pytest.mark.parametrize("magnitude", [1.0, 2.0 ** -14, 2.0 ** -22])
def test_levels_and_tiny_scales(rel, magnitude):
    rng = np.random.default_rng(3)
    K = (rng.integers(-130, 131, size=(1, 192, 5, 128)) * magnitude).astype(np.float16)
    V = (rng.standard_normal((1, 192, 5, 128)) * 4 * magnitude).astype(np.float16)
    V[0, 64:128] = (rng.integers(0, 255, size=(64, 5, 128)) * 0.5 * magnitude).astype(np.float16)
    cache = binding.PackedKVCache(1, 5, 5, 192, k_rel_scale=rel, v_rel_scale=rel, pack_size=8)
    cache.kv_compress_append(torch.from_numpy(K).cuda(), torch.from_numpy(V).cuda())
    n_packed, ck, cv = gpu_cases.oracle_cache(K, V, rel, rel, 8)
    gpu_cases.check_packed_state(cache, n_packed, ck, cv, 1, 5)


@pytest.mark.parametrize("rels", [NARROW, (0.1, 0.05)])
@pytest.mark.parametrize("pieces", [[37, 27 + 63], [64 + 15, 49 + 16, 48 + 2]])
@pytest.mark.parametrize("B,H,paged", [(3, 1, False), (2, 2, True), (2, 20, False)])
def test_completed_blocks_and_pages(B, H, paged, pieces, rels):
    pool = binding.PagePool(2 * (sum(pieces) // 64) * B * H // 6 + 8) if paged else None
    gpu_cases.run_case(B, H, H, sum(pieces), seed=9, pieces=pieces, pack_size=8, k_rel=rels[0], v_rel=rels[1], pool=pool)


@pytest.mark.parametrize("spare", [0, 300 * 1024, 1 << 30])
def test_any_workspace_gives_the_same_bytes(spare, monkeypatch):
    """No staging area (two passes), a small one (many parts) and the full one."""
    B, H, L = 2, 5, 40 * 64
    K, V, _ = synth.make_kv(B, L, H, H, 4, device="cuda:0")
    least = (256 + 65536 * 4 + 64 * B * H * 132 * 4 + 255) // 256 * 256
    query = binding.kv_query_sizes

    def sizes(cfg, *bits):
        s = query(cfg, *bits)
        s.workspace = min(s.workspace, least + spare)
        return s
    monkeypatch.setattr(binding, "kv_query_sizes", sizes)
    cache = binding.PackedKVCache(B, H, H, L, pack_size=8, k_rel_scale=0.05)
    cache.kv_compress_append(K, V)
    n_packed, ck, cv = gpu_cases.oracle_cache(K.cpu().numpy(), V.cpu().numpy(), 0.05, 0.2, 8)
    gpu_cases.check_packed_state(cache, n_packed, ck, cv, B, H)
