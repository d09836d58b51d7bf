"""bf16 results: every value with sums on, just below and just above the middle between two of them, the smallest
numbers, overflow, infinities and NaN, against the integer arithmetic of round to nearest, ties to even."""
import numpy as np
import pytest

import paper_2004_14020_amd as cm
from paper_2004_14020_amd.device import Replicas

pytestmark = pytest.mark.gpu


def widen(x):
    return (x.astype(np.uint32) << 16).view(np.float32)


def nearest_even(f):
    b = f.view(np.uint32)
    return ((b + 0x7FFF + (b >> 16 & 1)) >> 16).astype(np.uint16)


def second_values(a):
    """bf16 values to add to each of a: none, quarters of a's last place up to a whole one, either sign, the same a
    little off, the smallest number, the largest, infinities and NaN."""
    exp = (a >> 7 & 0xFF).astype(np.int32)
    for places in (7, 8, 9):
        e = exp - places
        small = np.where(e > 0, e << 7, np.where(e > -7, 1 << np.clip(e + 6, 0, 6), 0)).astype(np.uint16)
        for low in (0, 1, 0x40, 0x7F):  # 1, a little more, 1.5, almost 2
            for sign in (0, 0x8000):
                yield small | low | sign
    for special in (0, 0x8000, 1, 0x8001, 0x7F7F, 0xFF7F, 0x7F80, 0xFF80, 0x7FC0, 0x7F81):
        yield np.full_like(a, special)


@pytest.mark.parametrize("W", [2, 3, 16])
@pytest.mark.parametrize("cut", ["slices", "small tiles", "long tiles"])
def test_rounding_of_every_bf16_value(W, cut):
    a = np.arange(1 << 16, dtype=np.uint32).astype(np.uint16)
    rows = list(second_values(a))
    x = np.tile(a, len(rows))
    y = np.concatenate(rows)
    rng = np.random.Generator(np.random.Philox(key=[W, 7]))
    others = [rng.integers(0, 1 << 16, x.size, dtype=np.uint32).astype(np.uint16) if W == 3 else np.full_like(x, 0x8000)
              for _ in range(W - 2)]
    workers = [x, y] + others
    plan = cm.Plan(W, [x.size], dtype=cm.BF16, pattern=cm.PATTERN_SHUFFLE)  # sums x0 + x1 + ... everywhere
    if cut != "slices":
        plan.set_option(cm.OPT_LONG_RUN_BYTES, 1 if cut == "long tiles" else 1 << 40)
    dev = Replicas(plan, [x.size], with_workspace=False)
    assert (plan.slices() is not None) == (cut == "slices")
    dev.upload([[v] for v in workers])
    plan.allreduce()
    got = dev.download()
    with np.errstate(all="ignore"):
        total = widen(workers[0])
        for v in workers[1:]:
            total = total + widen(v)
        mean = total * np.float32(1.0 / W)
    want = nearest_even(mean)
    nan = np.isnan(mean)
    assert 0.001 < nan.mean() < 0.2 and (np.isinf(mean).sum() > 1000)
    for w in range(W):
        g = got[w][0]
        assert np.array_equal(g[~nan], want[~nan]), f"replica {w}"
        assert bool(((g[nan] & 0x7FC0) == 0x7FC0).all()), f"replica {w}: quiet NaN"
