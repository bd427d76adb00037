"""The arithmetic of csrc/flat_plan.h on the host: divisions by a prepared multiplier, the ranges of a flat plan and their
inverse, and that the shapes of the GPU tests of crossing ranges do cross."""
import ctypes as C
import os
import random
import subprocess

import pytest

from paper_2512_24449_amd import build
from tests.test_gpu_work_split import CROSSING_FUSED, CROSSING_FUSED_SPLIT, CROSSING_STEPS

HERE = os.path.dirname(os.path.abspath(__file__))
FULL = 5000   # workgroups up to which a plan is checked whole


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("plan") / "flat_plan_check.so")
    subprocess.check_call([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-O1", "-std=c++17", "-x", "hip", "--offload-host-only",
                           "-shared", "-fPIC", "-I", build.CSRC, "-o", lib, os.path.join(HERE, "flat_plan_check.cpp")])
    L = C.CDLL(lib)
    L.check_divisor.argtypes = [C.c_uint64, C.c_uint64]
    L.groups_for.argtypes = [C.c_int, C.c_int, C.c_int64, C.c_int64]
    return L


def test_divisions_are_exact(plan):
    rng = random.Random(5)
    ds = {1, 2, 3, 5, 7, 52, 64, 416, 500, 641, 768, 1280, 6700417, 10 ** 8}
    for k in range(1, 33):
        ds |= {2 ** k - 1, 2 ** k, 2 ** k + 1}
    for d in sorted(ds - {0}):
        most = (2 ** 64 - 1) // d
        xs = {0, 1, d - 1, d, d + 1, most, most - 1, most // d * d, max(most // d * d - 1, 0)}
        xs |= {rng.randrange(most + 1) for _ in range(50)} | {q * d + e for q in (rng.randrange(most // d + 1) for _ in range(20)) for e in (-1, 0, 1)}
        for x in xs:
            if 0 <= x <= most and x * d < 2 ** 64:
                assert plan.check_divisor(d, x) == 0, (x, d)


# (blocks, batch, heads, workgroups): one chunk, fewer blocks than workgroups, powers of two, primes, the benchmark shapes
@pytest.mark.parametrize("n_blocks,batch,heads,groups", [
    (1, 1, 1, 1), (1, 1, 1, 3), (1, 3, 5, 4), (7, 1, 1, 2), (15, 1, 1, 4), (64, 1, 32, 512), (500, 8, 52, 768), (500, 8, 52, 1280),
    (2048, 1, 8, 496), (5003, 1, 5, 310), (17, 9, 57, 769), (150, 9, 25, 1023), (123, 1, 1, 62), (124, 1, 1, 62), (125, 1, 3, 186),
    (997, 3, 11, 1009), (2, 16, 26, 416), (32767, 1, 1, 62)])
def test_ranges_and_their_inverse(plan, n_blocks, batch, heads, groups):
    assert plan.check_plan(n_blocks, batch, heads, groups, FULL) == 0
    assert bool(plan.uses_estimate(n_blocks, batch, heads, groups)) == (n_blocks * batch * heads == 1)


# chunks * chunks * workgroups on both sides of 1e19, where the workgroup of a chunk comes from a division or an estimate;
# the last ones are the largest an arena of 64 GiB (2^27 chunks) and split heads allow
@pytest.mark.parametrize("n_blocks,batch,heads,groups,estimate", [
    (80000, 8, 125, 1280, False), (100000, 8, 125, 1280, True), (100003, 7, 143, 1021, True), (1 << 17, 1, 1024, 1280, True),
    (1 << 17, 1, 1024, 512, False), (1 << 15, 1, 65535, 768, True), (1 << 15, 5, 13107, 65535, True), (1 << 27, 1, 1, 62, False),
    (3 << 24, 1, 2, 124, False), (1 << 27, 1, 16, 992, True)])
def test_large_plans(plan, n_blocks, batch, heads, groups, estimate):
    assert bool(plan.uses_estimate(n_blocks, batch, heads, groups)) == estimate
    assert plan.check_plan(n_blocks, batch, heads, groups, FULL) == 0


def test_drawn_plans(plan):
    rng = random.Random(11)
    for _ in range(1500):
        n = int(2 ** rng.uniform(0, 12))
        batch, heads = rng.choice([1, 1, 2, 3, 8, 9]), rng.choice([1, 2, 5, 8, 13, 40, 52, 57])
        room = 256 * rng.randint(1, 8)
        for most in (1 << 30, 62 * batch * heads):
            groups = plan.groups_for(n, batch * heads, room, most)
            assert 1 <= groups <= most and groups <= max(n * batch * heads, 1)
            assert plan.check_plan(n, batch, heads, groups, FULL) == 0, (n, batch, heads, groups)


# workgroups of a kernel to a compute unit: 2 to 6
@pytest.mark.parametrize("per_cu", [2, 3, 4, 5, 6])
def test_shapes_of_the_crossing_tests_cross(plan, per_cu):
    room = 256 * per_cu
    for B, H, n in CROSSING_STEPS:      # the K product, and the V product with its row sets
        for most in (1 << 30, 62 * B * H):
            assert plan.crossed_boundaries(n, B * H, plan.groups_for(n, B * H, room, most)) >= 5
    if per_cu > 4:                      # the fused kernel's LDS allows four at most
        return
    for B, H, n, split in [s + (1,) for s in CROSSING_FUSED] + [s + (5,) for s in CROSSING_FUSED_SPLIT]:
        streams = B * H * split
        groups = plan.groups_for(n, streams, room, 62 * streams)
        assert n * streams >= groups * 4 * 8, "below the flat plan's line"
        assert plan.crossed_boundaries(n, streams, groups) >= 5
