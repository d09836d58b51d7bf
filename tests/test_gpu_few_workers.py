"""World sizes that got kernels of their own: their tiles, whole, ragged and in several passes."""
import pytest

import oracle


@pytest.mark.gpu
@pytest.mark.parametrize("W", [1, 3])
@pytest.mark.parametrize("dtype", [oracle.F32, oracle.BF16])
def test_edges_of_tiles_with_few_workers(W, dtype):
    import paper_2004_14020_amd as cm
    from gpu_util import assert_same_bits, lib_plan, make_inputs, oracle_result
    from paper_2004_14020_amd.device import Replicas
    for pattern in (oracle.PATTERN_RING, oracle.PATTERN_SHUFFLE):
        print(f"case: few workers W={W} dtype={dtype} pattern={pattern}", flush=True)
        cfg = oracle.Config(W, dtype, 0, oracle.SPLIT_NONE, 1, 0, 16, 1, pattern)
        ve = 4 if dtype == oracle.F32 else 8
        # one element, vectors of a partial row, rows of 1024 lanes one to nine deep, ragged ends
        elems = [1, 5, 255 * ve, 1024 * ve + 1, 4095 * ve + 3, W * 4096 * ve, 9 * 1024 * ve + 2, 200001]
        grads = make_inputs(cfg, elems, seed=90 + W)
        grads[0][5][:4] = grads[0][5].dtype.type(0)
        grads[0][5][4:8] = -grads[0][5][:4] if dtype == oracle.F32 else 0x8000
        grads[0][5][8:12] = float("nan") if dtype == oracle.F32 else 0x7FC0
        ref = oracle_result(cfg, elems, grads)
        long_runs = {cm.OPT_LONG_RUN_BYTES: 1, cm.OPT_TAIL_TILES: 0}
        for opts in ({}, {cm.OPT_SMALL_BLOCK: 1024, cm.OPT_SMALL_TILE_VECS: 4096}, long_runs,
                     {**long_runs, cm.OPT_TILE_VECS: 8192}, {**long_runs, cm.OPT_TILE_VECS: 1000, cm.OPT_BLOCK: 256},
                     {cm.OPT_LONG_RUN_BYTES: 1}, {**long_runs, cm.OPT_STREAM_MAJOR: 0}, {**long_runs, cm.OPT_STREAM_MAJOR: 2},
                     {**long_runs, cm.OPT_NONTEMPORAL: 0}, {**long_runs, cm.OPT_SPLIT_TILES: 0}):
            plan = lib_plan(cfg, elems, opts)
            dev = Replicas(plan, elems, arena_phase=1280)
            dev.upload(grads)
            plan.allreduce()
            assert_same_bits(dev.download(), ref, f"W {W} options {opts}")
            plan.close()
