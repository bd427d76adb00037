"""Workgroups per stream of the kernels that split every stream alike (csrc/flat_plan.h, stream_splits), on the host."""
import ctypes as C
import os
import random
import subprocess

import pytest

from paper_2512_24449_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def splits(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("splits") / "stream_splits_check.so")
    subprocess.check_call([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-O1", "-std=c++17", "-x", "hip", "--offload-host-only",
                           "-shared", "-fPIC", "-I", build.CSRC, "-o", lib, os.path.join(HERE, "stream_splits_check.cpp")])
    L = C.CDLL(lib)

    def call(n_blocks, streams, per_cu, most=64):
        cost, usual = C.c_int64(), C.c_int()
        n = L.splits(n_blocks, streams, 256, per_cu, most, C.byref(cost), C.byref(usual))
        return n, cost.value, bool(usual.value)
    return call


# the shapes that were measured (blocks, streams, workgroups to a compute unit): kept at the usual number, and not
@pytest.mark.parametrize("n_blocks,streams,per_cu,n,usual", [
    (512, 32, 3, 16, True), (256, 32, 3, 16, True), (128, 32, 3, 16, True), (1000, 32, 3, 24, False), (2000, 32, 3, 24, False),
    (300, 64, 3, 12, False), (160, 40, 3, 12, False), (64, 32, 3, 16, True), (156, 32, 3, 16, True), (1500, 104, 3, 40, True),
    (1000, 128, 3, 32, True), (127, 64, 2, 8, True), (100, 256, 2, 2, False), (3, 1, 3, 1, True), (1, 65535, 2, 1, True)])
def test_measured_shapes(splits, n_blocks, streams, per_cu, n, usual):
    assert (splits(n_blocks, streams, per_cu)[0], splits(n_blocks, streams, per_cu)[2]) == (n, usual)


def test_within_bounds(splits):
    rng = random.Random(3)
    for _ in range(3000):
        nb, streams, per_cu = int(2 ** rng.uniform(0, 15)), int(2 ** rng.uniform(0, 16)), rng.randint(1, 8)
        for most in (64, 1 << 20):
            n, cost, usual = splits(nb, streams, per_cu, most)
            assert 1 <= n <= max(1, min(most, (nb + 3) // 4)) and cost > 0
            assert usual or n * streams <= 256 * per_cu or n == 1


# test_gpu_wide_buffers compares 32 streams of 400 blocks, which take the kernels with two smaller chunk buffers (two workgroups to a compute unit),
# with 64, which must not.  The rules as launch_k_matvec and launch_decode_attention have them, three workgroups of the other kernels to a compute unit.
@pytest.mark.parametrize("streams,small_buffers", [(32, True), (64, False)])
def test_both_sides_of_the_line_between_wide_buffers(splits, streams, small_buffers):
    blocks = 400
    (_, cost, _), (n2, cost2, _) = splits(blocks, streams, 3), splits(blocks, streams, 2)
    assert (n2 * streams <= 512 and cost2 <= cost) == small_buffers, "fused attention"
    _, cost, _ = splits(blocks, streams, 3, 1 << 20)
    n2, cost2, usual2 = splits(blocks, streams, 2, 1 << 20)
    if usual2:
        n2 = max(1, min(max(streams * blocks // 32, 512), 4096) // streams)
    per_group = max(4, -(-(-(-blocks // n2)) // 4) * 4)
    assert (cost2 <= cost and streams * -(-blocks // per_group) <= 512) == small_buffers, "K product"
