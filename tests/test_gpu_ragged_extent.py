"""Ragged batches of short sequences among long ones, split by stream-K, where
a short sequence counts for a few steps more than it has: ranges that begin or
end ahead of its first step, sequences of 0, 1 and the limit's steps (8 per
step phase, one less, one more), every phase count, both merges, the merge by
sequence and by split, query tokens and windows -- against the fp64 oracle.

The bar is that of the other attention tests: one bf16 spacing of the fp64
value."""
import numpy as np
import pytest

import oracle
import workloads as W
from _gpu import check, log, q4, run_ext

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib(gpu_lib):
    return gpu_lib


def lengths(b, phases, longest, seed):
    """b lengths: most of 1 to 64 tokens, some at the limit, a few long, some 0."""
    rng = np.random.default_rng(seed)
    lens = rng.integers(1, 65, size=b)
    edge = 8 * phases * 32
    for i, x in enumerate((0, 1, 32, 33, edge - 32, edge - 31, edge, edge + 1, longest)):
        lens[(7 * i + seed) % b] = x
    lens[rng.integers(0, b, size=max(1, b // 10))] = 0
    lens[seed % b] = longest
    return [int(x) for x in lens]


# (batch, Hq, Hkv, D, page, longest, query tokens, window, step phases)
CASES = [
    (9, 8, 1, 128, 16, 4000, 1, 0, 8),
    (40, 8, 1, 128, 16, 9000, 1, 0, 8),
    (300, 8, 1, 128, 16, 2500, 1, 0, 8),
    (64, 32, 2, 128, 16, 5000, 1, 0, 4),
    (300, 32, 2, 128, 64, 1300, 1, 0, 4),
    (64, 24, 4, 128, 1, 3000, 1, 0, 2),
    (50, 24, 3, 64, 4, 3000, 1, 0, 2),
    (33, 32, 8, 128, 16, 4000, 1, 0, 1),
    (33, 12, 4, 256, 16, 3000, 1, 0, 1),
    (150, 8, 1, 256, 32, 1500, 1, 0, 4),
    (40, 8, 2, 64, 16, 5000, 3, 0, 4),
    (40, 8, 1, 128, 16, 6000, 2, 700, 8),
]


@pytest.mark.parametrize("merge", ["kernel", "fused"])
@pytest.mark.parametrize("b,hq,hkv,d,p,longest,tq,window,phases", CASES,
                         ids=[f"B{c[0]}-{c[1]}:{c[2]}-D{c[3]}-P{c[4]}-L{c[5]}-T{c[6]}-W{c[7]}" for c in CASES])
def test_ragged_short_sequences(lib, b, hq, hkv, d, p, longest, tq, window, phases, merge):
    w = W.build(lengths(b, phases, longest, b + d), hq, hkv, d, p, seed=b + d + longest, pool="holes:0.1",
                num_queries=tq, window=window)
    want = oracle.attend_masked(q4(w), w.k_cache, w.v_cache, w.block_table, w.context_lens, w.scale, w.window)[0]
    log(f"ragged extent case B={b} {hq}:{hkv} D={d} P={p} longest={longest} Tq={tq} W={window} merge={merge}")
    lib.set_option(lib.OPT_FIXED_SPLIT, 0)  # stream-K, however small the call
    lib.set_option(lib.OPT_FUSED_MERGE, 2 if merge == "fused" else 0)
    try:
        check(run_ext(lib, w), want, "ragged")
    finally:
        lib.set_option(lib.OPT_FIXED_SPLIT, 1)
        lib.set_option(lib.OPT_FUSED_MERGE, 0)
