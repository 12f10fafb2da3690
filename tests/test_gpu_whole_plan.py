"""Calls whose sequences are all short (by the page table, or by the window):
whole sequences, one workgroup per (sequence, kv-head group), no merge --
against the fp64 oracle on both sides of the lines where that plan begins and
ends, with empty sequences, partial last steps, several kv heads a workgroup,
head sizes 64 to 256, pages of 1 to 64 tokens, query tokens and windows; and
the same call under a captured graph and with the plan's options changed.

The bar is that of the other attention tests: one bf16 spacing of the fp64
value."""
import numpy as np
import pytest

import oracle
import workloads as W
from _gpu import check, log, q4, run_ext, to_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib(gpu_lib):
    return gpu_lib


def ref(w):
    return oracle.attend_masked(q4(w), w.k_cache, w.v_cache, w.block_table, w.context_lens, w.scale, w.window)[0]


def spread(b, cap, seed=0):
    """b lengths from 0 to cap, both among them."""
    lens = np.random.default_rng(seed).integers(0, cap + 1, size=b)
    lens[0], lens[-1] = cap, 0
    if b > 2:
        lens[1] = min(cap, 33)
    return [int(x) for x in lens]


# (batch, Hq, Hkv, D, page, table capacity, query tokens, window): one kv head
# a workgroup up to 256 of them, then 2, 4, 8; capacities at and one page past
# the line
CASES = [
    (2, 8, 2, 64, 16, 64, 1, 0),
    (4, 32, 8, 128, 16, 288, 1, 0),
    (4, 32, 8, 128, 16, 304, 1, 0),
    (32, 32, 8, 128, 16, 160, 1, 0),
    (33, 32, 8, 128, 16, 144, 1, 0),
    (33, 12, 4, 256, 32, 128, 3, 0),
    (64, 32, 8, 128, 1, 150, 1, 0),
    (100, 32, 8, 128, 4, 64, 2, 0),
    (128, 32, 2, 128, 16, 608, 1, 0),
    (256, 32, 2, 128, 64, 256, 1, 0),
    (256, 40, 8, 128, 16, 64, 1, 0),
    (257, 32, 2, 128, 16, 64, 1, 0),
    (5, 16, 16, 64, 16, 320, 1, 0),
    (7, 48, 3, 128, 16, 96, 1, 0),
    # short by the window, whatever the table holds
    (8, 32, 8, 128, 16, 4096, 1, 100),
    (40, 32, 2, 128, 16, 2048, 1, 512),
    (31, 12, 4, 256, 16, 2048, 2, 64),
    (16, 8, 8, 64, 1, 700, 16, 31),
    # a window that leaves a split plan, of fewer steps than the table's
    (8, 32, 8, 128, 16, 8192, 1, 1024),
    (3, 64, 8, 128, 32, 16384, 2, 2000),
    (100, 32, 8, 128, 16, 1024, 1, 512),
]


@pytest.mark.parametrize("b,hq,hkv,d,p,cap,tq,window", CASES,
                         ids=[f"B{c[0]}-{c[1]}:{c[2]}-D{c[3]}-P{c[4]}-cap{c[5]}-T{c[6]}-W{c[7]}" for c in CASES])
def test_short_sequences(lib, b, hq, hkv, d, p, cap, tq, window):
    w = W.build(spread(b, cap, b + cap), hq, hkv, d, p, seed=b + d + cap, pool="holes:0.1", num_queries=tq,
                window=window, max_pages=-(-cap // p))
    log(f"whole plan case B={b} {hq}:{hkv} D={d} P={p} cap={cap} Tq={tq} W={window}")
    check(run_ext(lib, w), ref(w), "short sequences")


def test_options_keep_their_plans(lib):
    """A call that would run whole, under each option that asks for another plan."""
    w = W.build(spread(20, 160), 32, 8, 128, 16, seed=5)
    want = ref(w)
    for opt, val, back in ((lib.OPT_FIXED_SPLIT, 0, 1), (lib.OPT_KV_GROUP, 2, 0), (lib.OPT_MIN_STEPS, 2, 0),
                           (lib.OPT_BLOCKS_PER_CU, 2, 1), (lib.OPT_FUSED_MERGE, 2, 0)):
        lib.set_option(opt, val)
        try:
            check(run_ext(lib, w), want, f"option {opt} = {val}")
        finally:
            lib.set_option(opt, back)


def test_a_captured_call_follows_the_lengths(lib):
    """The plan follows from sizes alone: one capture serves every length, and
    the reservation covers windowed calls of the same table."""
    import torch
    for window in (0, 300):
        cap = 160 if window == 0 else 4096
        w = W.build(spread(12, cap, 3), 32, 8, 128, 16, seed=6, poison=False, window=window, max_pages=cap // 16)
        dev = to_gpu(w)
        q = dev["q"].unsqueeze(1).contiguous()
        out = torch.empty_like(q)
        s = torch.cuda.Stream()
        lib.workspace_reserve(12, 32, 8, 128, 16, cap // 16, stream=s)
        g = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(g, stream=s):
            lib.paged_decode_attention_ext(q, dev["k"], dev["v"], dev["bt"], dev["lens"], out, float(w.scale),
                                           window=window)
        for step in range(3):
            # shorter than the table row's pages: every id stays valid
            lens = np.maximum(w.context_lens - 7 * step, 0).astype(np.int32)
            dev["lens"].copy_(torch.from_numpy(lens))
            out.fill_(float("nan"))
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            want = oracle.attend_masked(q4(w), w.k_cache, w.v_cache, w.block_table, lens, w.scale, window)[0]
            check(out.float().cpu().numpy().astype(np.float64), want, f"window {window} replay {step}")
