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


def oracle_pattern(pattern):
    return {"ring": oracle.PATTERN_RING, "shuffle": oracle.PATTERN_SHUFFLE, "hd": oracle.PATTERN_HALVING_DOUBLING}[pattern]


@pytest.mark.gpu
@pytest.mark.parametrize("W", [1, 2, 3, 4, 7, 8, 12, 16, 33, 64])
@pytest.mark.parametrize("dtype", [oracle.F32, oracle.BF16])
@pytest.mark.parametrize("many", [False, True])
def test_ends_of_slices(W, dtype, many):
    """Every length of a last vector, slices whole and ragged, signed zeros, infinities and NaN; replicas alike and
    apart; what lies between the tensors stays as it is.  `many`: enough slices for several per wavefront."""
    import torch
    from gpu_util import assert_same_bits, lib_plan, make_inputs, oracle_result
    from paper_2004_14020_amd.device import Replicas
    ve = 4 if dtype == oracle.F32 else 8
    elems = list(range(1, 2 * ve + 1)) + [64 * ve - 1, 64 * ve, 64 * ve + 1, 1000 * ve + 3, W * 512 * ve + 5]
    if many:
        elems += list(range(63 * ve, 65 * ve + 1)) + [2700 * 64 * ve + 7]
    cfg = oracle.Config(W, dtype, 4096, oracle.SPLIT_NONE, 1, 0, 16, 1, oracle.PATTERN_RING)
    inputs = make_inputs(cfg, elems, seed=50 + W)
    bits = [0x80000000, 0x7F800000, 0x7FC00000, 0xFF800000]
    for w in range(W):
        for i, b in enumerate(bits):
            if i == 0 or w == i:
                g = inputs[w][-1][300 * i:300 * i + 300]
                g[:] = np.uint32(b).view(np.float32) if dtype == oracle.F32 else b >> 16
    for pattern in (oracle.PATTERN_RING, oracle.PATTERN_SHUFFLE, oracle.PATTERN_HALVING_DOUBLING):
        if pattern == oracle.PATTERN_HALVING_DOUBLING and W & (W - 1):
            continue
        print(f"case: ends of slices W={W} dtype={dtype} pattern={pattern} many={many}", flush=True)
        cfg = oracle.Config(W, dtype, 4096, oracle.SPLIT_NONE, 1, 0, 16, 1, pattern)
        ref = oracle_result(cfg, elems, inputs)
        apart = [256 * (w * 5 % 7) for w in range(W)]
        for phase, align, phases in ((0, 256, None), (1280, 16, None), (0, 16, apart)):
            plan = lib_plan(cfg, elems)
            dev = Replicas(plan, elems, arena_phase=phase, slot_align=align, arena_phases=phases)
            shape = plan.slices()
            assert shape and (shape[2] > 1) == many, shape
            for a in dev.arenas:
                a.fill_(0xA5)
            for w in range(W):
                for t in range(len(elems)):
                    dev.tensor(w, t).copy_(torch.from_numpy(inputs[w][t].view(np.float32 if dtype == oracle.F32 else np.int16)))
            plan.allreduce()
            assert_same_bits(dev.download(), ref, f"W {W} phase {phase}")
            for w in range(W):
                for t in range(len(elems)):
                    dev.tensor(w, t).view(torch.uint8).fill_(0xA5)
                assert bool((dev.arenas[w] == 0xA5).all()), f"replica {w}: written outside its tensors"
            plan.close()


# KiB per replica: the lines between the shapes, and from 32 MiB on the largest jobs that have slices and ones beyond
CHAIN_SIZES = (1, 2040, 2570, 3401, 5000, 7000, 8300, 10000, 11000, 13000, 14800, 16381, 20400, 20490, 22000, 24577, 26000, 28673,
               30000, 32767)
TREE_SIZES = (1, 1010, 1030, 2070, 4100, 6150, 7700, 8200, 9300, 10800, 12500, 13800, 15500, 17300, 20300, 20490, 32767)
LONG_SIZES = {2: (60000, 111 << 10, 113 << 10), 3: (47 << 10, 49 << 10), 4: (47 << 10, 49 << 10), 6: (47 << 10, 49 << 10),
              7: (35 << 10, 37 << 10), 8: (35 << 10, 37 << 10)}


def rounds(*vecs):
    return {(256, v) for v in (1,) + vecs}


# shapes (lanes, slices per wavefront) that these sizes come to, and the sizes that have tiles
FP32, BF16 = rounds(4, 6, 8, 10, 12, 14, 16, 18, 20), rounds(4, 6, 8, 10, 12, 14, 16)
WIDE_8 = {(1024, 6), (1024, 8), (512, 16), (512, 18)}
WIDE_BF16 = {(1024, 4), (1024, 6)}
ABOVE = {2: (113 << 10,), 3: (49 << 10,), 4: (49 << 10,), 6: (49 << 10,), 7: (37 << 10,), 8: (37 << 10,)}
JOBS = ([("ring", 1, 0, FP32, CHAIN_SIZES[13:]), ("ring", 1, 1, BF16, CHAIN_SIZES[12:])] +
        [("ring", W, d, BF16 if d else FP32, ABOVE[W]) for W in (2, 3, 4, 6, 7) for d in (0, 1)] +
        [("ring", 8, 0, FP32 | WIDE_8, ABOVE[8]), ("ring", 8, 1, BF16, ABOVE[8]),
         ("shuffle", 8, 0, FP32 | WIDE_8 | {(1024, 5)}, (35 << 10, 37 << 10)), ("ring", 9, 0, FP32 | WIDE_8 - {(1024, 6)}, ()),
         ("ring", 12, 0, FP32 | WIDE_8 - {(512, 16)}, ()), ("ring", 12, 1, BF16 | WIDE_BF16, (24577, 26000)),
         ("ring", 16, 0, FP32 | {(512, 14), (512, 16), (512, 18), (512, 20)}, ()), ("ring", 16, 1, BF16 | WIDE_BF16, ()),
         ("ring", 64, 0, rounds(4, 6, 8, 12, 14), ()), ("ring", 64, 1, rounds(4, 6, 8, 12, 14), ()),
         ("hd", 2, 0, rounds(2, 4, 6, 8, 12, 16, 20), (113 << 10,)), ("hd", 2, 1, rounds(2, 4, 6, 8, 12, 16), (113 << 10,)),
         ("hd", 4, 0, rounds(2, 4, 6, 8, 12, 16, 20), (49 << 10,)), ("hd", 4, 1, rounds(2, 4, 6, 8, 12, 16), (49 << 10,)),
         ("hd", 8, 0, rounds(2, 4, 6, 8, 12, 16, 18), (35 << 10, 37 << 10)),
         ("hd", 8, 1, rounds(2, 4, 6, 8, 12, 14), (35 << 10, 37 << 10)),
         ("hd", 16, 0, rounds(2, 4, 6, 8, 12, 14), ()), ("hd", 16, 1, rounds(2, 4, 6, 8, 10), ()),
         ("hd", 32, 0, rounds(2, 4, 6, 8, 12, 14), (15500, 17300, 20300, 20490)),
         ("hd", 32, 1, rounds(2, 4, 6, 8), (8200, 9300, 10800, 12500, 13800, 15500, 17300, 20300, 20490)),
         ("hd", 64, 0, rounds(2, 4, 6, 8, 12), ()), ("hd", 64, 1, rounds(2, 4, 6, 8), (8200, 9300, 10800))])


def same_as_tiles(plan, dev, what):
    """One call as the library cuts the job, one over tiles (an option that asks for them): the same bits."""
    import torch
    import paper_2004_14020_amd as cm
    stream = torch.cuda.current_stream().cuda_stream
    before = [a.clone() for a in dev.arenas]
    plan.allreduce(stream)
    got = [a.clone() for a in dev.arenas]
    for a, b in zip(dev.arenas, before):
        a.copy_(b)
    plan.set_option(cm.OPT_SPLIT_TILES, 0)
    assert plan.slices() is None
    plan.allreduce(stream)
    for w, (a, b) in enumerate(zip(dev.arenas, got)):
        assert torch.equal(a, b), f"replica {w}, {what}"


@pytest.mark.gpu
@pytest.mark.parametrize("pattern,W,dtype,shapes,tiles", JOBS, ids=[f"{j[0]}-{j[1]}-{j[2]}" for j in JOBS])
def test_every_shape_gives_the_bits_of_the_tiles(pattern, W, dtype, shapes, tiles):
    """Around the lines between the shapes: the smallest and largest number of vectors per lane, one and
    several rounds, a last workgroup that is nearly empty."""
    import paper_2004_14020_amd as cm
    from paper_2004_14020_amd.device import Replicas
    size = 4 if dtype == cm.F32 else 2
    met, over_tiles = set(), []
    for kib in (TREE_SIZES if pattern == "hd" else CHAIN_SIZES) + LONG_SIZES.get(W, ()):
        if kib * W > 700000 or (pattern == "hd" and W == 2 and kib == 60000):
            continue
        print(f"case: slices against tiles {pattern} W={W} dtype={dtype} {kib} KiB", flush=True)
        elems = [kib * KIB // size - 300 if kib > 1 else 100, 37, 256, 1]
        plan = cm.Plan(W, elems, dtype=dtype, batch_threshold_bytes=4096, split_mode=cm.SPLIT_FIXED, split_bytes=1000 * KIB,
                       pattern=oracle_pattern(pattern))
        dev = Replicas(plan, elems, with_workspace=False, large_align=256)
        if plan.slices() is None:
            over_tiles.append(kib)
        else:
            met.add(plan.slices()[1:])
            dev.fill_random(kib)
            same_as_tiles(plan, dev, f"{kib} KiB")
        plan.close()
    assert (met, tuple(over_tiles)) == (shapes, tuple(tiles))


@pytest.mark.gpu
@pytest.mark.parametrize("W,dtype,tensors,shape", [(16, 0, 50000, (1024, 7)), (8, 0, 35000, (256, 1)), (16, 1, 50000, (1024, 5)),
                                                   (3, 0, 60000, (256, 1))])
def test_slices_of_half_a_kilobyte(W, dtype, tensors, shape):
    """A great many small tensors: more slices than the bytes come to."""
    import paper_2004_14020_amd as cm
    from paper_2004_14020_amd.device import Replicas
    elems = [512 // (4 if dtype == cm.F32 else 2) - t % 3 for t in range(tensors)]
    plan = cm.Plan(W, elems, dtype=dtype, batch_threshold_bytes=1 << 20, pattern=cm.PATTERN_SHUFFLE)
    dev = Replicas(plan, elems, with_workspace=False, slot_align=1024)
    assert plan.slices()[1:] == shape
    dev.fill_random(W)
    same_as_tiles(plan, dev, f"{tensors} tensors")
    plan.close()


@pytest.mark.gpu
@pytest.mark.parametrize("pattern,W,dtype,kib,shape", [
    ("ring", 16, 0, 26000, (512, 18)), ("ring", 12, 0, 30000, (1024, 8)), ("ring", 12, 1, 21000, (1024, 6)),
    ("ring", 16, 1, 26000, (1024, 4)), ("shuffle", 8, 0, 22000, (1024, 6)), ("ring", 2, 0, 60000, (256, 1)),
    ("ring", 5, 1, 40000, (256, 1)), ("ring", 33, 0, 6000, (256, 8)), ("hd", 8, 0, 13000, (256, 16)),
    ("hd", 16, 1, 20000, (256, 1)), ("hd", 64, 0, 5000, (256, 6))])
def test_larger_jobs_with_replicas_apart(pattern, W, dtype, kib, shape):
    """Many odd tensors whose replicas all lie at other offsets, against the oracle."""
    import paper_2004_14020_amd as cm
    from gpu_util import assert_same_bits, lib_plan
    from paper_2004_14020_amd.device import Replicas
    size = 4 if dtype == cm.F32 else 2
    share = kib * KIB // size // 100
    elems = [share * 40 + 3, 1, share * 7 + 1, 129, share * 53] + [share // 300 + 11 * t for t in range(40)]
    cfg = oracle.Config(W, dtype, 65536, oracle.SPLIT_ADAPTIVE, 8, 1 << 20, 16, 2, oracle_pattern(pattern))
    plan = lib_plan(cfg, elems)
    dev = Replicas(plan, elems, with_workspace=False, slot_align=256, large_align=256,
                   arena_phases=[256 * (w * 5 % 11) for w in range(W)])
    assert plan.slices()[1:] == shape
    dev.fill_random(kib)
    ref = dev.download()
    oracle.allreduce(oracle.build_plan(cfg, elems), ref)
    plan.allreduce()
    assert_same_bits(dev.download(), ref, f"{pattern} W {W}")
    plan.close()
