"""Which tiles a plan gets by default: the lines of the rules, on the CPU."""
import os
import shutil
import subprocess

import pytest

import oracle

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2004_14020_amd", "csrc")
MIB = 1 << 20
RING, HD, SHUFFLE = oracle.PATTERN_RING, oracle.PATTERN_HALVING_DOUBLING, oracle.PATTERN_SHUFFLE

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")


@pytest.fixture(scope="module")
def shape(tmp_path_factory):
    """(vectors per long tile or 0 if there are none, boundaries per long tile, per small tile)"""
    exe = str(tmp_path_factory.mktemp("shape") / "shape_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(ROOT, "tests", "host", "shape_check.cpp"), os.path.join(CSRC, "plan.cpp"),
                    os.path.join(CSRC, "tiles.cpp"), "-o", exe], check=True)

    def ask(world, dtype, pattern, nbytes, block=1024, few_tiles=0, stream_major=8):
        res = subprocess.run([exe, *map(str, (world, dtype, pattern, nbytes, block, few_tiles, stream_major))], capture_output=True, text=True,
                             check=True)
        return tuple(int(x) for x in res.stdout.split())
    return ask


@pytest.mark.parametrize("W", [1, 2, 3, 4, 5, 7, 8, 9, 12, 16, 24, 64])
def test_128_kib_tiles_where_they_pay(shape, W):
    for pattern in (RING, SHUFFLE):
        assert shape(W, oracle.F32, pattern, 32 * MIB - 4)[0] == 0
        for at in (32, 64, 192, 1024):
            wide = at >= 64 if W in (2, 4, 8) else (at >= 192 and W > 4)
            assert shape(W, oracle.F32, pattern, at * MIB)[0] == (8192 if wide else 4096), (pattern, at)
            assert shape(W, oracle.F32, pattern, at * MIB - 4)[0] != 8192 or at > (64 if W in (2, 4, 8) else 192)
            assert shape(W, oracle.BF16, pattern, at * MIB)[0] == 4096


@pytest.mark.parametrize("W", [2, 8, 16, 32, 64])
def test_trees_without_a_walk_get_small_tiles(shape, W):
    for at in (32, 64, 1024):
        assert shape(W, oracle.BF16, HD, at * MIB)[0] == (4096 if W <= 16 else 0)
        assert shape(W, oracle.F32, HD, at * MIB)[0] == (8192 if W <= 4 and at >= 64 else 4096)
        for block in (256, 512):
            assert shape(W, oracle.BF16, HD, at * MIB, block)[0] == (2048 if W <= 16 else 0)
            assert shape(W, oracle.F32, HD, at * MIB, block)[0] == 4096
        for vectors in (0, 2, 4):      # walks switched off, or shortened
            short = vectors < 4
            assert shape(W, oracle.BF16, HD, at * MIB, stream_major=vectors)[0] == (0 if W > 16 else 2048 if short else 4096)
            assert shape(W, oracle.F32, HD, at * MIB, stream_major=vectors)[0] == (0 if W > 16 and short else 4096)


@pytest.mark.parametrize("W", [1, 3, 5, 8, 16, 32, 64])
def test_few_tiles_where_the_table_space_is_limited(shape, W):
    """The largest tiles that a kernel takes, whatever is fastest."""
    for at in (64, 192, 1024):
        wide = at >= (64 if W == 8 else 192)
        assert shape(W, oracle.F32, RING, at * MIB, few_tiles=1)[0] == (8192 if wide else 4096)
        if W in (8, 16, 32, 64):
            assert shape(W, oracle.BF16, HD, at * MIB, 256, few_tiles=1)[0] == (4096 if W <= 16 else 2048)
