"""Tiles across several segment boundaries: the tables on the CPU, the walk over them on the GPU."""
import os
import shutil
import subprocess

import pytest

import oracle

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2004_14020_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_tables_with_several_boundaries_per_tile(tmp_path):
    exe = str(tmp_path / "splits_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-static-libasan", "-static-libubsan", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(ROOT, "tests", "host", "splits_check.cpp"), os.path.join(CSRC, "plan.cpp"),
                    os.path.join(CSRC, "tiles.cpp"), "-o", exe], check=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0 and "splits_check ok" in res.stdout, res.stdout[-2000:] + res.stderr[-2000:]


@pytest.mark.gpu
@pytest.mark.parametrize("W", [6, 16, 24, 33, 64])
@pytest.mark.parametrize("dtype", [oracle.F32, oracle.BF16])
def test_walk_over_several_boundaries(W, dtype):
    """Rows of lanes 1 .. 8 and their ragged ends, none to four boundaries per tile; the sums of -0.0
    and of infinities and NaN start and end where those of other values do."""
    import paper_2004_14020_amd as cm
    from gpu_util import assert_same_bits, lib_plan, make_inputs, oracle_result
    from paper_2004_14020_amd.device import Replicas
    print(f"case: several boundaries per tile W={W} dtype={dtype}", flush=True)
    cfg = oracle.Config(W, dtype, 0, oracle.SPLIT_NONE, 1, 0, 16, 1)
    elems = [37, 5003, 1024 * 8 + 3, 3000 * 8, 5 * 4096 + 9, 8 * 4096, 200001]
    grads = make_inputs(cfg, elems, seed=77 + W)
    special = [-0.0, float("inf"), float("nan")]
    for w in range(W):
        for i, v in enumerate(special):
            bits = {-0.0: 0x80000000}.get(v) if v == 0 else (0x7F800000 if v > 0 else 0x7FC00000)
            part = grads[w][5][i * 8192:i * 8192 + 4096]
            if i == 0 or w == i:
                part[:] = (part.view("uint32").dtype.type(bits).view("float32") if dtype == oracle.F32 else bits >> 16)
    ref = oracle_result(cfg, elems, grads)
    for opts in ({}, {cm.OPT_TILE_VECS: 8192, cm.OPT_TAIL_TILES: 0}, {cm.OPT_TILE_VECS: 4096, cm.OPT_TAIL_TILES: 2},
                 {cm.OPT_TILE_VECS: 1000, cm.OPT_BLOCK: 256, cm.OPT_TAIL_TILES: 0}, {cm.OPT_STREAM_MAJOR: 2},
                 {cm.OPT_NONTEMPORAL: 0}):
        plan = lib_plan(cfg, elems, {cm.OPT_LONG_RUN_BYTES: 1, **opts})
        dev = Replicas(plan, elems, arena_phase=1280)
        dev.upload(grads)
        plan.allreduce()
        assert_same_bits(dev.download(), ref, f"options {opts}")
        # the launch options may change after the tables are built
        plan.set_option(cm.OPT_STREAM_MAJOR, 0)
        dev.upload(grads)
        plan.allreduce()
        assert_same_bits(dev.download(), ref, f"options {opts}, then no stream-major walk")
        plan.close()
