"""Small jobs cut into slices: the tables on the CPU, the kernels over them on the GPU."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import oracle

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2004_14020_amd", "csrc")
KIB = 1 << 10


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_slice_tables_against_tile_tables(tmp_path):
    exe = str(tmp_path / "slices_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-static-libasan", "-static-libubsan", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(ROOT, "tests", "host", "slices_check.cpp"), os.path.join(CSRC, "plan.cpp"),
                    os.path.join(CSRC, "tiles.cpp"), os.path.join(CSRC, "slices.cpp"), "-o", exe], check=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert res.returncode == 0 and "slices_check ok" in res.stdout, res.stdout[-2000:] + res.stderr[-2000:]


@pytest.mark.gpu
@pytest.mark.parametrize("W", [1, 2, 3, 4, 7, 8, 12, 16, 33, 64])
@pytest.mark.parametrize("dtype", [oracle.F32, oracle.BF16])
def test_ends_of_slices(W, dtype):
    """Every length of a last vector, slices whole and ragged, signed zeros, infinities and NaN; what
    lies between the tensors stays as it is."""
    import torch
    from gpu_util import assert_same_bits, lib_plan, make_inputs, oracle_result
    from paper_2004_14020_amd.device import Replicas
    ve = 4 if dtype == oracle.F32 else 8
    elems = list(range(1, 2 * ve + 1)) + [64 * ve - 1, 64 * ve, 64 * ve + 1, 1000 * ve + 3, W * 512 * ve + 5]
    for pattern in (oracle.PATTERN_RING, oracle.PATTERN_SHUFFLE, oracle.PATTERN_HALVING_DOUBLING):
        if pattern == oracle.PATTERN_HALVING_DOUBLING and W & (W - 1):
            continue
        print(f"case: ends of slices W={W} dtype={dtype} pattern={pattern}", flush=True)
        cfg = oracle.Config(W, dtype, 4096, oracle.SPLIT_NONE, 1, 0, 16, 1, pattern)
        grads = make_inputs(cfg, elems, seed=50 + W)
        bits = [0x80000000, 0x7F800000, 0x7FC00000, 0xFF800000]
        for w in range(W):
            for i, b in enumerate(bits):
                if i == 0 or w == i:
                    g = grads[w][-1][300 * i:300 * i + 300]
                    g[:] = np.uint32(b).view(np.float32) if dtype == oracle.F32 else b >> 16
        ref = oracle_result(cfg, elems, grads)
        for phase, align in ((0, 256), (1280, 16)):
            plan = lib_plan(cfg, elems)
            dev = Replicas(plan, elems, arena_phase=phase, slot_align=align)
            for a in dev.arenas:
                a.fill_(0xA5)
            for w in range(W):
                for t in range(len(elems)):
                    dev.tensor(w, t).copy_(torch.from_numpy(grads[w][t].view(np.float32 if dtype == oracle.F32 else np.int16)))
            plan.allreduce()
            assert_same_bits(dev.download(), ref, f"W {W} phase {phase}")
            for w in range(W):
                for t in range(len(elems)):
                    dev.tensor(w, t).view(torch.uint8).fill_(0xA5)
                assert bool((dev.arenas[w] == 0xA5).all()), f"replica {w}: written outside its tensors"
            plan.close()


@pytest.mark.gpu
@pytest.mark.parametrize("pattern,W,dtype", [("ring", 1, 0), ("ring", 2, 1), ("ring", 3, 0), ("ring", 4, 1), ("ring", 8, 0),
                                             ("ring", 8, 1), ("ring", 12, 0), ("ring", 12, 1), ("ring", 16, 0), ("ring", 24, 1),
                                             ("ring", 32, 0)] + [("hd", W, d) for W in (2, 4, 8, 16, 32, 64) for d in (0, 1)])
def test_every_shape_gives_the_bits_of_the_tiles(pattern, W, dtype):
    """Around the lines between the shapes: the smallest and largest number of vectors per lane, one and
    several rounds, a last workgroup that is nearly empty."""
    import torch
    import paper_2004_14020_amd as cm
    from paper_2004_14020_amd.device import Replicas
    size = 4 if dtype == cm.F32 else 2
    sizes = (1, 2040, 2070, 2570, 3401, 10000, 16381, 16390, 20477, 20490, 24577, 28673, 32767)
    if pattern == "hd":  # every number of vectors per lane
        sizes = (1, 1010, 1030, 2070, 4100, 6150, 8200, 9300, 11000, 13800, 17300, 20400, 20490, 32767)
    for kib in sizes:
        if kib * W > 530000:
            continue
        print(f"case: slices against tiles {pattern} W={W} dtype={dtype} {kib} KiB", flush=True)
        elems = [kib * KIB // size - 300 if kib > 1 else 100, 37, 256, 1]
        plan = cm.Plan(W, elems, dtype=dtype, batch_threshold_bytes=4096, split_mode=cm.SPLIT_FIXED, split_bytes=1000 * KIB,
                       pattern=cm.PATTERN_RING if pattern == "ring" else cm.PATTERN_HALVING_DOUBLING)
        dev = Replicas(plan, elems, with_workspace=False, large_align=256)
        dev.fill_random(kib)
        before = [a.clone() for a in dev.arenas]
        plan.allreduce(torch.cuda.current_stream().cuda_stream)
        got = [a.clone() for a in dev.arenas]
        for a, b in zip(dev.arenas, before):
            a.copy_(b)
        plan.set_option(cm.OPT_SPLIT_TILES, 0)
        plan.allreduce(torch.cuda.current_stream().cuda_stream)
        for w in range(W):
            assert torch.equal(dev.arenas[w], got[w]), f"replica {w}, {kib} KiB"
        plan.close()
