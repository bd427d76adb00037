"""Rounds in two passes over the input whose metadata and sizes come from the staged path's quantizer: both sides of the lines
of the rule, both pack sizes and layouts, one to three kv-heads per wave, pages through either placement kernel, an arena that turns out too
full.  Bytes, index and metadata against the oracle, bit for bit."""
import pytest
import torch

from paper_2512_24449_amd import binding, synth
from tests import gpu_cases

pytestmark = pytest.mark.gpu


# 256 chunks of each tensor to a part at 1 x 1 .. 1 x 4, 512 at 1 x 8, 576 and 640 at 1 x 9 and 10, 1024 at 2 x 8
@pytest.mark.parametrize("pack,rels", [(16, (0.1, 0.2)), (8, (0.1, 0.2)), (8, (0.05, 0.2)), (8, (0.05, 1 / 127))])
@pytest.mark.parametrize("B,H,blocks", [(1, 1, 256), (1, 1, 257), (1, 2, 200), (3, 1, 90), (1, 3, 90), (1, 8, 64), (1, 8, 65), (1, 10, 65), (2, 8, 129)])
def test_parts_and_passes(B, H, blocks, pack, rels):
    if pack == 8 and rels != (0.05, 0.2) and B * H > 3:
        pytest.skip("the mixed layout covers the larger ones")
    gpu_cases.run_case(B, H, H, 64 * blocks + 3, seed=blocks + H, pack_size=pack, k_rel=rels[0], v_rel=rels[1])


# more than 8192 chunks of a tensor: the placement kernel of large rounds
@pytest.mark.parametrize("pack,rels", [(16, (0.1, 0.2)), (8, (0.05, 0.2))])
@pytest.mark.parametrize("B,H,blocks", [(3, 1, 90), (1, 10, 70), (5, 13, 130)])
def test_pages(B, H, blocks, pack, rels):
    if pack == 8 and blocks == 130:
        pytest.skip("packs of 16 cover the large rounds")
    pool = binding.PagePool(2 * blocks * B * H // (14 if pack == 16 else 6) + 16)
    gpu_cases.run_case(B, H, H, 64 * blocks + 1, seed=H, pack_size=pack, k_rel=rels[0], v_rel=rels[1], pool=pool)


@pytest.mark.parametrize("pack", [16, 8])
def test_arena_turns_out_too_full(pack):
    """K fits, V does not: V's chunks are dropped as a whole, K's are the oracle's."""
    B, H, blocks = 1, 4, 200
    K, V, _ = synth.make_kv(B, 64 * blocks, H, H, 5, device="cuda:0")
    n_packed, ck, cv = gpu_cases.oracle_cache(K.cpu().numpy(), V.cpu().numpy(), 0.1, 0.1, pack)
    cache = binding.PackedKVCache(B, H, H, 64 * blocks, pack_size=pack, v_rel_scale=0.1,
                                  bits_per_element_budget=(ck.arena.size + cv.arena.size) * 4.0 / (B * H * 64 * blocks * 128))
    cache.kv_compress_append(K, V)
    st = cache.kv_cache_stats()
    fits = [c.arena.size <= cache.sizes.k_arena for c in (ck, cv)]
    assert sorted(fits) == [False, True], "the budget lies between the two sizes"
    assert st.overflow == 1 and (st.k_bytes, st.v_bytes) == tuple(c.arena.size if f else 0 for c, f in zip((ck, cv), fits))
    for name, c, f in zip("kv", (ck, cv), fits):
        if f:
            assert torch.equal(cache.tensors[name + "_arena"][:c.arena.size].cpu(), torch.from_numpy(c.arena))
