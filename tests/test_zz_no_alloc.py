"""caramel_allreduce_static, the entry point for callers that cannot allocate device memory:
its output against caramel_bind + caramel_allreduce (and the oracle), bit for bit, through the
C ABI -- on two calls in a row, the second with a smaller input, so that the second call finds
the first one's tables in the library's static device array."""
import numpy as np
import pytest
import torch

import oracle
import paper_2004_14020_amd as cm
from paper_2004_14020_amd import binding
from paper_2004_14020_amd.device import Replicas

from gpu_util import assert_same_bits, lib_plan, make_inputs, oracle_result

pytestmark = pytest.mark.gpu

BIG = (300000, 10, 700, 33, 50000, 1, 257, 30011, 64, 129, 3, 4097, 100000, 7, 20000, 70001)
SMALL = (5000, 3, 129, 20000)


def both_ways(cfg, elems, seed, stream, opts=None):
    """(result of the existing entry point, Replicas and unbound plan for the static one, oracle result)."""
    grads = make_inputs(cfg, list(elems), seed)
    ref = oracle_result(cfg, list(elems), grads)
    bound = lib_plan(cfg, list(elems), opts)
    dev = Replicas(bound, list(elems), with_workspace=False)
    dev.upload(grads)
    bound.allreduce(stream)
    want = dev.download()
    assert_same_bits(want, ref, "caramel_allreduce against the oracle")
    dev.upload(grads)                     # fresh inputs in the same memory for the static call
    unbound = lib_plan(cfg, list(elems), opts)
    return want, dev, unbound, bound


@pytest.mark.parametrize("dtype", [oracle.F32, oracle.BF16])
def test_static_entry_point_matches_allreduce_on_two_calls_in_a_row(dtype):
    print(f"case: static entry point dtype={dtype}", flush=True)
    stream = torch.cuda.current_stream().cuda_stream
    cfg_a = oracle.Config(8, dtype, 8192, oracle.SPLIT_FIXED, 8, 1 << 18, 16, 2)
    cfg_b = oracle.Config(4, dtype, 4096, oracle.SPLIT_NONE, 8, 0, 16, 2)
    want_a, dev_a, plan_a, keep_a = both_ways(cfg_a, BIG, 21, stream)
    want_b, dev_b, plan_b, keep_b = both_ways(cfg_b, SMALL, 22, stream)
    # two calls in a row on one stream, no synchronisation in between; the second is smaller
    plan_a.allreduce_static(dev_a.pointers(), stream)
    plan_b.allreduce_static(dev_b.pointers(), stream)
    assert_same_bits(dev_a.download(), want_a, "first static call")
    assert_same_bits(dev_b.download(), want_b, "second (smaller) static call")
    # again with the tables already in place (same plan, pointers and stream), then the larger
    # plan again over what the smaller one left in the array
    dev_b.upload(make_inputs(cfg_b, list(SMALL), 22))
    plan_b.allreduce_static(dev_b.pointers(), stream)
    assert_same_bits(dev_b.download(), want_b, "repeated static call")
    dev_a.upload(make_inputs(cfg_a, list(BIG), 21))
    plan_a.allreduce_static(dev_a.pointers(), stream)
    assert_same_bits(dev_a.download(), want_a, "static call after a smaller one")
    for p in (plan_a, plan_b, keep_a, keep_b):
        p.close()


def test_static_entry_point_rejects_what_does_not_fit():
    """More pointer rows than the static array holds: a clear error, nothing launched."""
    W, n = 64, 9000                                    # 9001 rows x 64 workers x 8 bytes > 4 MiB
    plan = cm.Plan(W, [4] * n, batch_threshold_bytes=0)
    ptrs = [[(1 << 40) + (w * n + t) * 256 for t in range(n)] for w in range(W)]   # never dereferenced
    with pytest.raises(cm.CaramelError) as ei:
        plan.allreduce_static(ptrs)
    assert ei.value.status == binding.EINVAL and "static array" in str(ei.value)
    with pytest.raises(cm.CaramelError):
        plan.allreduce_static([[0] * n for _ in range(W)])
    plan.close()


def test_static_entry_point_takes_longer_tiles_before_it_refuses():
    """Halving-doubling over 32 workers in bf16 has small tiles by default; where the static array cannot
    hold that many, the tables are built with long ones, and the result is the same."""
    W, size = 32, 2
    elems = [16] * 13800 + [(40 << 20) // size]
    print("case: static entry point, tables that fit with long tiles only", flush=True)
    cfg = dict(dtype=cm.BF16, pattern=cm.PATTERN_HALVING_DOUBLING, num_streams=1)
    bound, unbound = cm.Plan(W, elems, **cfg), cm.Plan(W, elems, **cfg)
    dev = Replicas(bound, elems, with_workspace=False, slot_align=32)
    stream = torch.cuda.current_stream().cuda_stream
    dev.fill_random(3)
    bound.profile(1)
    bound.allreduce(stream)
    assert bound.profile_read()[cm.K_REDUCE]["elements"] == 0       # small tiles throughout
    want = [dev.arenas[w].clone() for w in (0, 17, 31)]
    dev.fill_random(3)
    unbound.allreduce_static(dev.pointers(), stream)
    for w, x in zip((0, 17, 31), want):
        assert torch.equal(dev.arenas[w], x), f"replica {w}"
    bound.close()
    unbound.close()
