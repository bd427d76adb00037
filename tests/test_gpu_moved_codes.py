"""Repacked tokens that are quantized in arrival order and whose codes are moved afterwards: a wave and four waves to a token,
several parts, blocks completed in the tail, packs of 8, pages.  Order, bytes, index and metadata against the oracle."""
import pytest

from paper_2512_24449_amd import binding
from tests import gpu_cases

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pack", [16, 8])
@pytest.mark.parametrize("B,H,pieces", [(1, 1, [257 * 64]), (3, 3, [100 * 64 + 5]), (1, 8, [64]), (2, 16, [129]), (1, 17, [30, 40]), (2, 33, [64, 63, 1]),
                                        (1, 64, [100, 28])])
def test_order_and_bytes(B, H, pieces, pack):
    if pack == 8 and H > 17:
        pytest.skip("the rows are those of packs of 16")
    gpu_cases.run_case(B, H, H, sum(pieces), seed=H, pieces=pieces, pack_size=pack, repack=True)


# the largest codes of one-byte pack metadata; constant scales aside, every level occurs
@pytest.mark.parametrize("rels", [(1 / 15, 1 / 15), (0.5, 1.0)])
@pytest.mark.parametrize("paged", [False, True])
def test_levels_and_pages(rels, paged):
    pool = binding.PagePool(40) if paged else None
    gpu_cases.run_case(2, 5, 5, 300, seed=2, pieces=[200, 100], k_rel=rels[0], v_rel=rels[1], repack=True, pool=pool)
