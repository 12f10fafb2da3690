"""The forms of the projection kernel on the GPU against the fp64 oracle:
every (row tiles, column tiles) form its planner picks, whole k ranges and k
splits, with the sizes where a form can go wrong: an odd number of k tiles
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


# (batch, in_features, hidden): row tiles x column tiles of the plan on 256
# compute units, and its k splits
OPROJ = [
    (1, 96, 2560),      # 1 x 1
    (3, 2080, 128),     # 1 x 1, 4 splits
    (16, 4128, 2576),   # several row tiles x 1, splits; the last workgroup has fewer tiles
    (1, 96, 8192),      # 3 x 1
    (2, 96, 32752),     # 4 x 1, hidden above what the splitting kernel sums
    (17, 96, 640),      # 1 x 2
    (17, 1056, 2560),   # 2 x 2, splits
    (32, 2080, 4608),   # 3 x 2, splits
    (20, 96, 16400),    # 4 x 2, 1025 row tiles
    (33, 96, 640),      # 1 x 4
    (48, 544, 4608),    # 2 x 4
    (64, 2080, 4608),   # 3 x 4, splits
    (40, 1056, 16384),  # 4 x 4
    (33, 96, 16400),    # 6 x 4 wide, an odd number of row tiles
    (64, 160, 32752),   # 8 x 4, the last workgroup has fewer tiles
    (65, 96, 128),      # 2 x 4 in two column groups, splits
    (129, 96, 256),     # 2 x 4 in three column groups
    (80, 1056, 2560),   # 3 x 4 in column groups, splits
    (100, 4128, 2560),  # 4 x 4 in column groups, splits
    (96, 1056, 7168),   # 4 x 4 in column groups
    (65, 96, 7168),     # 6 x 4 wide in column groups
    (112, 2080, 4608),  # 6 x 4 wide, splits
    (200, 96, 5120),    # 4 x 6 wide
    (256, 4128, 2560),  # wide forms, splits
    (255, 544, 4608),
    (129, 4128, 1024),
    (129, 224, 16384),  # 8 x 4 in column groups
]


@pytest.mark.parametrize("b,k,h", OPROJ, ids=[f"B{c[0]}-K{c[1]}-H{c[2]}" for c in OPROJ])
def test_oproj_forms(lib, b, k, h):
    log(f"o_proj form case B={b} K={k} H={h}")
    w = W.build_oproj(b, k, h, seed=b + 3 * k + h)
    z, hn = run_oproj(lib, w)
    rz, rh = ref_oproj(w)
    check_oproj(z, rz, "z")
    check_oproj(hn, rh, "h")


# (batch, hidden, Hq, Hkv, D, options).  The epilogue runs in the projection
# kernel without Q/K norm and with interleaved pairs or a rotated size that is
# a multiple of 32.
PRELUDE = [
    (1, 96, 8, 4, 64, dict()),
    (2, 544, 4, 1, 256, dict(bias=True)),
    (16, 1056, 6, 3, 128, dict(rotary_dim=64)),
    (9, 96, 64, 8, 128, dict(interleaved=True, bias=True)),
    (17, 160, 4, 2, 128, dict(rotary_dim=40)),                       # not a multiple of 32
    (17, 160, 5, 5, 64, dict(rotary_dim=40, interleaved=True)),
    (20, 96, 64, 8, 128, dict(rotary_dim=0)),
    (33, 224, 6, 2, 64, dict(rotary_dim=32)),
    (48, 1056, 64, 8, 128, dict(bias=True)),
    (64, 544, 12, 4, 256, dict(rotary_dim=128)),
    (33, 96, 128, 16, 128, dict(interleaved=True, rotary_dim=64)),
    (65, 96, 4, 2, 128, dict()),
    (129, 544, 12, 6, 128, dict(bias=True, rotary_dim=96)),
    (100, 96, 24, 8, 128, dict(interleaved=True, rotary_dim=64, bias=True)),
    (160, 160, 32, 4, 128, dict()),
    (200, 96, 12, 4, 256, dict()),
    (256, 160, 40, 8, 128, dict(rotary_dim=64)),
    (256, 96, 98, 14, 128, dict(interleaved=True)),
    (1, 2080, 24, 8, 128, dict(qk_norm=True)),
    (24, 4128, 16, 2, 128, dict(qk_norm=True, bias=True)),
    (64, 2080, 24, 8, 128, dict(qk_norm=True, rotary_dim=64)),
    (256, 1056, 8, 4, 128, dict(qk_norm=True, interleaved=True)),
]


@pytest.mark.parametrize("b,h,hq,hkv,d,opt", PRELUDE, ids=[f"B{c[0]}-H{c[1]}-{c[2]}:{c[3]}-D{c[4]}" for c in PRELUDE])
def test_prelude_forms(lib, b, h, hq, hkv, d, opt):
    lens = np.random.default_rng(b * 5 + h).integers(0, 200000, size=b)
    lens[-1] = 0                                   # an empty slot: position 0
    w = W.build_prelude(b, h, hq, hkv, d, seed=b * 11 + h, lengths=lens, theta=5.0e5, **opt)
    log(f"prelude form case B={b} H={h} {hq}:{hkv} D={d} {opt}")
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
