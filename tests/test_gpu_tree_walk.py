"""Halving-doubling over long tiles (k_tree_walk, and the kernel that takes its tiles where the walk is
switched off or does not exist), bit for bit against the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

SPECIAL = [-0.0, float("inf"), float("-inf"), float("nan"), 1e-40, 3e38]


@pytest.mark.parametrize("W", [2, 4, 8, 16, 32, 64])
@pytest.mark.parametrize("dtype", [oracle.F32, oracle.BF16])
def test_tree_over_long_tiles(W, dtype):
    import paper_2004_14020_amd as cm
    from gpu_util import assert_same_bits, lib_plan, make_inputs, oracle_result
    from paper_2004_14020_amd.device import Replicas
    print(f"case: tree over long tiles W={W} dtype={dtype}", flush=True)
    cfg = oracle.Config(W, dtype, 0, oracle.SPLIT_NONE, 1, 0, 16, 1, oracle.PATTERN_HALVING_DOUBLING)
    ve = 4 if dtype == oracle.F32 else 8
    # vectors of one partial row; one to eight rows of 1024 lanes, whole and ragged, with ends inside a
    # vector; more than one pass of a tile of eight rows
    elems = [1, 5, 255 * ve, 1024 * ve + 1, 2 * 1024 * ve, 3 * 1024 * ve - 7 * ve, 4 * 1024 * ve + 3, 5 * 1024 * ve,
             7 * 1024 * ve + 11 * ve + 2, 8 * 1024 * ve, 17 * 1024 * ve + 1]
    grads = make_inputs(cfg, elems, seed=300 + W)
    # values that are no ordinary numbers: alike at all workers, or at one of them
    for i, v in enumerate(SPECIAL):
        bits = np.array([v], np.float32).view(np.uint32)[0]
        for w in range(W):
            part = grads[w][9][i * 1024:i * 1024 + 512]
            if i == 0 or w == (5 * i) % W:
                part[:] = part.dtype.type(v) if dtype == oracle.F32 else np.uint16(bits >> 16)
    with np.errstate(all="ignore"):
        ref = oracle_result(cfg, elems, grads)
    long_runs = {cm.OPT_LONG_RUN_BYTES: 1, cm.OPT_TAIL_TILES: 0}
    for opts in (long_runs, {**long_runs, cm.OPT_TILE_VECS: 8192}, {**long_runs, cm.OPT_TILE_VECS: 1000},
                 {**long_runs, cm.OPT_STREAM_MAJOR: 2}, {**long_runs, cm.OPT_STREAM_MAJOR: 0},
                 {**long_runs, cm.OPT_TILE_VECS: 4096, cm.OPT_STREAM_MAJOR: 8},
                 {**long_runs, cm.OPT_BLOCK: 256}, {**long_runs, cm.OPT_BLOCK: 512, cm.OPT_TILE_VECS: 8192},
                 {**long_runs, cm.OPT_BLOCK: 256, cm.OPT_TILE_VECS: 1000, cm.OPT_STREAM_MAJOR: 2},
                 {cm.OPT_LONG_RUN_BYTES: 1, cm.OPT_TAIL_TILES: 5}, {**long_runs, cm.OPT_NONTEMPORAL: 0},
                 {**long_runs, cm.OPT_MAX_GRID: 3, cm.OPT_TILE_VECS: 2048}):
        plan = lib_plan(cfg, elems, opts)
        dev = Replicas(plan, elems, arena_phase=1280)
        dev.upload(grads)
        plan.profile(1)
        plan.allreduce()
        assert plan.profile_read()[cm.K_REDUCE]["elements"] == sum(elems)
        assert_same_bits(dev.download(), ref, f"options {opts}")
        plan.close()
