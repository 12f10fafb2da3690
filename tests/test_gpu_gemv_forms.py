"""The forms of the projection kernel on the GPU against the fp64 oracle:
every form its planner picks on 256 compute units within the interface's
limits, with every ending it has there (each case names its plan, and the test
asserts it; test_projection_plan.py asserts on the host that the cases leave
none out), with the sizes where a form can go wrong: an odd number of k tiles
(half a 64-k pair at the end), fewer pairs than waves, row tiles that do not
fill the last workgroup, batches one past a column tile, one past a column
group and at the limit.  The prelude runs with its epilogue in the projection
kernel and in a kernel of its own, over the rotations that decide which.

Outputs are fp32 sums rounded once to bf16, so each is held to one bf16
spacing of the fp64 value, as in the other tests of these entry points."""
import numpy as np
import pytest

import oracle
import workloads as W
from _gpu import log, to_gpu
from test_gpu_oproj import check_ulps as check_oproj
from test_gpu_oproj import dev_bf16, host
from test_gpu_oproj import ref as ref_oproj
from test_gpu_oproj import run as run_oproj
from test_gpu_prelude import bits, check_ulps, ref_prelude, run_prelude

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib(gpu_lib):
    return gpu_lib


CUS = 256  # of the GPU these plans are for


def name_of(p, ending):
    """A plan in words: row x column tiles, wide matrix instructions, several
    column groups, and what ends it: the k splits' sum, or unsplit the epilogue
    in the kernel (fused), the residual, or plain sums."""
    return (f"{p.row_tiles}x{p.col_tiles}" + " wide" * p.wide + " groups" * (p.col_groups > 1) + " " +
            ("fused" if p.fused else "split" if p.k_splits > 1 else ending))


def o_proj_name(lib, b, k, h):
    return name_of(lib.o_proj_plan(b, k, h, CUS), "residual")


def prelude_name(lib, b, h, hq, hkv, d, opt):
    rot = opt.get("rotary_dim", d)
    dims = lib.prelude_dims(b, h, hq, hkv, d, rot, opt.get("interleaved", False), 5e5, 1e-6)
    return name_of(lib.prelude_plan(dims, opt.get("qk_norm", False), CUS), "plain")


# (batch, in_features, hidden, plan)
OPROJ = [
    (1, 96, 2560, "1x1 residual"),
    (3, 2080, 128, "1x1 split"),
    (16, 4128, 2576, "2x1 split"),
    (1, 96, 8192, "1x1 residual"),
    (2, 96, 32752, "1x1 residual"),
    (17, 96, 640, "1x2 split"),
    (17, 1056, 2560, "2x2 split"),
    (32, 2080, 4608, "4x2 split"),
    (20, 96, 16400, "3x2 residual"),
    (33, 96, 640, "1x4 residual"),
    (48, 544, 4608, "3x4 residual"),
    (64, 2080, 4608, "4x4 split"),
    (40, 1056, 16384, "4x4 residual"),
    (33, 96, 16400, "8x4 residual"),
    (64, 160, 32752, "8x4 residual"),
    (65, 96, 128, "3x4 groups split"),
    (129, 96, 256, "3x4 groups split"),
    (80, 1056, 2560, "3x4 groups split"),
    (100, 4128, 2560, "4x4 groups split"),
    (96, 1056, 7168, "4x4 groups residual"),
    (65, 96, 7168, "8x4 groups residual"),
    (112, 2080, 4608, "3x4 groups residual"),
    (200, 96, 5120, "8x4 groups residual"),
    (256, 4128, 2560, "4x6 wide groups split"),
    (255, 544, 4608, "6x4 wide groups residual"),
    (129, 4128, 1024, "3x4 groups split"),
    (129, 224, 16384, "8x4 groups residual"),
    (17, 96, 784, "1x2 residual"),
    (33, 96, 16, "1x4 split"),
    (16, 96, 4112, "2x1 residual"),
    (17, 96, 4112, "2x2 residual"),
    (33, 1056, 6656, "2x4 residual"),
    (33, 4128, 1552, "2x4 split"),
    (65, 1056, 3584, "2x4 groups residual"),
    (65, 4128, 128, "2x4 groups split"),
    (16, 96, 8208, "3x1 residual"),
    (9, 1056, 4112, "3x1 split"),
    (17, 1056, 4112, "3x2 split"),
    (33, 544, 4112, "3x4 split"),
    (16, 96, 14336, "4x1 residual"),
    (9, 2080, 4112, "1x1 split"),
    (17, 96, 14336, "4x2 residual"),
    (129, 288, 6656, "4x6 wide groups residual"),
    (33, 288, 16400, "6x4 wide residual"),
    (33, 2592, 6656, "6x4 wide split"),
    (65, 2080, 3584, "6x4 wide groups split"),
    (33, 12320, 6656, "8x4 split"),
    (65, 2080, 4608, "8x4 groups split"),
]


@pytest.mark.parametrize("b,k,h,plan", OPROJ, ids=[f"B{c[0]}-K{c[1]}-H{c[2]}" for c in OPROJ])
def test_oproj_forms(lib, b, k, h, plan):
    assert o_proj_name(lib, b, k, h) == plan
    log(f"o_proj form case B={b} K={k} H={h}: {plan}")
    w = W.build_oproj(b, k, h, seed=b + 3 * k + h)
    z, hn = run_oproj(lib, w)
    rz, rh = ref_oproj(w)
    check_oproj(z, rz, "z")
    check_oproj(hn, rh, "h")


# (batch, hidden, Hq, Hkv, D, options, plan).  The epilogue runs in the projection
# kernel without Q/K norm and with interleaved pairs or a rotated size that is
# a multiple of 32.
PRELUDE = [
    (1, 96, 8, 4, 64, dict(), "2x1 fused"),
    (2, 544, 4, 1, 256, dict(bias=True), "2x1 fused"),
    (16, 1056, 6, 3, 128, dict(rotary_dim=64), "2x1 fused"),
    (9, 96, 64, 8, 128, dict(interleaved=True, bias=True), "4x1 fused"),
    (17, 160, 4, 2, 128, dict(rotary_dim=40), "1x2 split"),
    (17, 160, 5, 5, 64, dict(rotary_dim=40, interleaved=True), "2x2 fused"),
    (20, 96, 64, 8, 128, dict(rotary_dim=0), "4x2 fused"),
    (33, 224, 6, 2, 64, dict(rotary_dim=32), "2x4 fused"),
    (48, 1056, 64, 8, 128, dict(bias=True), "4x4 fused"),
    (64, 544, 12, 4, 256, dict(rotary_dim=128), "2x4 fused"),
    (33, 96, 128, 16, 128, dict(interleaved=True, rotary_dim=64), "8x4 fused"),
    (65, 96, 4, 2, 128, dict(), "2x4 groups fused"),
    (129, 544, 12, 6, 128, dict(bias=True, rotary_dim=96), "4x4 groups fused"),
    (100, 96, 24, 8, 128, dict(interleaved=True, rotary_dim=64, bias=True), "8x4 groups fused"),
    (160, 160, 32, 4, 128, dict(), "4x4 groups fused"),
    (200, 96, 12, 4, 256, dict(), "8x4 groups fused"),
    (256, 160, 40, 8, 128, dict(rotary_dim=64), "8x4 groups fused"),
    (256, 96, 98, 14, 128, dict(interleaved=True), "8x4 groups fused"),
    (1, 2080, 24, 8, 128, dict(qk_norm=True), "1x1 split"),
    (24, 4128, 16, 2, 128, dict(qk_norm=True, bias=True), "2x2 split"),
    (64, 2080, 24, 8, 128, dict(qk_norm=True, rotary_dim=64), "4x4 split"),
    (256, 1056, 8, 4, 128, dict(qk_norm=True, interleaved=True), "2x4 groups plain"),
    (9, 96, 5, 5, 64, dict(qk_norm=True), "1x1 plain"),
    (17, 96, 2, 2, 128, dict(qk_norm=True, bias=True), "1x2 plain"),
    (33, 96, 6, 2, 64, dict(qk_norm=True, interleaved=True), "1x4 plain"),
    (33, 96, 1, 1, 64, dict(qk_norm=True, rotary_dim=32), "1x4 split"),
    (16, 96, 12, 4, 256, dict(qk_norm=True, interleaved=True, bias=True, rotary_dim=128), "2x1 plain"),
    (9, 1312, 24, 8, 64, dict(qk_norm=True), "2x1 split"),
    (17, 96, 12, 4, 256, dict(qk_norm=True, bias=True), "2x2 plain"),
    (33, 1056, 40, 8, 128, dict(qk_norm=True, interleaved=True), "2x4 plain"),
    (33, 4128, 8, 2, 128, dict(rotary_dim=64), "2x4 split"),
    (65, 4128, 2, 1, 64, dict(interleaved=True, bias=True, rotary_dim=32), "2x4 groups split"),
    (16, 96, 64, 8, 128, dict(qk_norm=True), "3x1 plain"),
    (9, 1056, 12, 4, 256, dict(qk_norm=True, bias=True), "3x1 split"),
    (17, 96, 64, 8, 128, dict(qk_norm=True, interleaved=True), "3x2 plain"),
    (17, 1056, 12, 4, 256, dict(qk_norm=True, rotary_dim=128), "3x2 split"),
    (33, 96, 12, 4, 256, dict(qk_norm=True, interleaved=True, bias=True, rotary_dim=128), "3x4 plain"),
    (33, 800, 12, 4, 256, dict(qk_norm=True), "3x4 split"),
    (177, 96, 2, 1, 64, dict(qk_norm=True, bias=True), "3x4 groups plain"),
    (65, 96, 2, 1, 64, dict(qk_norm=True, interleaved=True), "3x4 groups split"),
    (16, 96, 96, 8, 128, dict(qk_norm=True, rotary_dim=64), "4x1 plain"),
    (9, 2080, 12, 4, 256, dict(qk_norm=True, interleaved=True, bias=True, rotary_dim=128), "1x1 split"),
    (17, 96, 96, 8, 128, dict(qk_norm=True), "4x2 plain"),
    (17, 2080, 12, 4, 256, dict(qk_norm=True, bias=True), "4x2 split"),
    (33, 160, 96, 8, 128, dict(qk_norm=True, interleaved=True), "4x4 plain"),
    (65, 160, 40, 8, 128, dict(qk_norm=True, rotary_dim=64), "4x4 groups plain"),
    (65, 2592, 8, 4, 128, dict(interleaved=True, bias=True, rotary_dim=64), "4x4 groups split"),
    (129, 288, 40, 8, 128, dict(), "4x6 wide groups fused"),
    (129, 288, 40, 8, 128, dict(qk_norm=True, bias=True), "4x6 wide groups plain"),
    (129, 2080, 8, 4, 128, dict(qk_norm=True, interleaved=True), "4x6 wide groups split"),
    (33, 288, 128, 16, 128, dict(rotary_dim=64), "6x4 wide fused"),
    (33, 288, 128, 16, 128, dict(qk_norm=True, interleaved=True, bias=True, rotary_dim=64), "6x4 wide plain"),
    (33, 2592, 40, 8, 128, dict(qk_norm=True), "6x4 wide split"),
    (65, 288, 64, 8, 128, dict(bias=True), "6x4 wide groups fused"),
    (65, 288, 64, 8, 128, dict(qk_norm=True, interleaved=True), "6x4 wide groups plain"),
    (80, 2592, 12, 4, 256, dict(qk_norm=True, rotary_dim=128), "6x4 wide groups split"),
    (33, 96, 96, 8, 128, dict(qk_norm=True, interleaved=True, bias=True, rotary_dim=64), "8x4 plain"),
    (33, 4128, 56, 8, 128, dict(), "8x4 split"),
    (65, 96, 40, 8, 128, dict(qk_norm=True, bias=True), "8x4 groups plain"),
    (65, 2080, 12, 4, 256, dict(qk_norm=True, interleaved=True), "8x4 groups split"),
]


@pytest.mark.parametrize("b,h,hq,hkv,d,opt,plan", PRELUDE,
                         ids=[f"B{c[0]}-H{c[1]}-{c[2]}:{c[3]}-D{c[4]}" for c in PRELUDE])
def test_prelude_forms(lib, b, h, hq, hkv, d, opt, plan):
    assert prelude_name(lib, b, h, hq, hkv, d, opt) == plan
    lens = np.random.default_rng(b * 5 + h).integers(0, 200000, size=b)
    lens[-1] = 0                                   # an empty slot: position 0
    w = W.build_prelude(b, h, hq, hkv, d, seed=b * 11 + h, lengths=lens, theta=5.0e5, **opt)
    log(f"prelude form case B={b} H={h} {hq}:{hkv} D={d} {opt}: {plan}")
    got = run_prelude(lib, w)
    for name, g, r in zip("qkv", got, ref_prelude(w)):
        check_ulps(host(g), r, name)


@pytest.mark.parametrize("b,d,page,opt", [(6, 64, 1, dict()), (21, 256, 16, dict(interleaved=True, rotary_dim=64)),
                                          (70, 128, 32, dict(bias=True))], ids=["D64-P1", "D256-P16", "D128-P32"])
def test_append_in_the_projection_kernel_writes_the_same_bits(lib, b, d, page, opt):
    import torch
    lens = [int(x) for x in np.random.default_rng(d).integers(0, 3 * page + 60, size=b)]
    lens[1] = 0
    lens[2] = page  # the last slot of a page
    pw = W.build_prelude(b, 160, 6, 2, d, seed=61, lengths=lens, theta=1e5, **opt)
    aw = W.build(lens, 6, 2, d, page, seed=62, pool="holes:0.3")
    q_sep, k_sep, v_sep = run_prelude(lib, pw)
    dev = to_gpu(aw)
    q = torch.empty_like(q_sep)
    lib.attention_prelude_append(dev_bf16(pw.x), lib.pack_weights(dev_bf16(pw.w_qkv)), dev["lens"], q, dev["k"],
                                 dev["v"], dev["bt"], num_q_heads=6, num_kv_heads=2, head_dim=d,
                                 rope_theta=float(pw.theta), rotary_dim=pw.rotary_dim, interleaved=pw.interleaved,
                                 bias=None if pw.bias is None else dev_bf16(pw.bias), eps=float(pw.eps))
    torch.cuda.synchronize()
    assert np.array_equal(bits(q), bits(q_sep))
    rk, rv = oracle.kv_append(aw.k_cache, aw.v_cache, bits(k_sep), bits(v_sep), aw.block_table, aw.context_lens)
    assert np.array_equal(bits(dev["k"]), rk) and np.array_equal(bits(dev["v"]), rv)


@pytest.mark.parametrize("b", [5, 40, 130])
def test_outputs_over_the_inputs(lib, b):
    """q over x, and the new residual over the attention output: an output
    tile must not be written while another workgroup still reads its input."""
    import torch
    hq, hkv, d = 8, 2, 128
    pw = W.build_prelude(b, hq * d, hq, hkv, d, seed=71, lengths=np.arange(b) * 7 + 1, theta=1e5)
    q, k, v = run_prelude(lib, pw)
    x = dev_bf16(pw.x)
    k2, v2 = torch.empty_like(k), torch.empty_like(v)
    lens = torch.from_numpy(pw.context_lens).cuda()
    lib.attention_prelude(x, lib.pack_weights(dev_bf16(pw.w_qkv)), lens, x.view(b, hq, d), k2, v2, num_q_heads=hq,
                          num_kv_heads=hkv, head_dim=d, rope_theta=float(pw.theta), eps=float(pw.eps))
    torch.cuda.synchronize()
    for got, want, name in ((x.view(b, hq, d), q, "q over x"), (k2, k, "k"), (v2, v, "v")):
        check_ulps(host(got), host(want), name)
    ow = W.build_oproj(b, 1024, 1024, seed=72)
    z, h = run_oproj(lib, ow)
    attn, h2 = dev_bf16(ow.attn), torch.empty((b, 1024), dtype=torch.bfloat16, device="cuda")
    lib.o_proj_residual_norm(attn, lib.pack_weights(dev_bf16(ow.w_o)), dev_bf16(ow.residual), dev_bf16(ow.norm_w),
                             attn, h2, eps=float(ow.eps))
    torch.cuda.synchronize()
    assert np.array_equal(host(attn), z) and np.array_equal(host(h2), h)


@pytest.mark.parametrize("b,k", [(4, 96), (30, 544), (64, 1056), (100, 96), (200, 544)])
def test_a_sequence_of_nan_stays_its_own(lib, b, k):
    """NaN and infinities in one sequence's input reach no other sequence,
    also not through the k range past the end of its row."""
    w = W.build_oproj(b, k, 512, seed=81)
    clean = run_oproj(lib, w)
    w.attn[b // 2, :] = W.BF16_NAN
    w.attn[b // 2, ::2] = 0x7F80  # +inf
    z, h = run_oproj(lib, w)
    keep = np.arange(b) != b // 2
    assert np.array_equal(z[keep], clean[0][keep]) and np.array_equal(h[keep], clean[1][keep])
    assert np.isnan(z[~keep]).all()
