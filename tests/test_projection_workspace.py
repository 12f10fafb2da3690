"""The workspace of the projection calls: what one asks for at a batch covers
every smaller batch of the same rows, whatever their plans -- on the planner
for every batch, and on the GPU where a stream reserved (or grown by a call)
for one batch is captured at smaller ones."""
import pytest

from paper_2606_07665_amd import binding as B

CUS = (64, 256, 304)

# (in_features, hidden): model shapes, small ones, and both sides of the
# hidden size up to which o_proj is split along k
OPROJ = [(4096, 4096), (5120, 5120), (8192, 8192), (3072, 3072), (4096, 2560), (96, 128), (2048, 8320), (65536, 16384),
         (32, 32768)]
# (hidden, Hq, Hkv, D)
PRELUDE = [(4096, 32, 8, 128), (8192, 64, 8, 128), (2560, 32, 8, 128), (3072, 12, 4, 256), (4096, 32, 2, 128),
           (2048, 32, 8, 64), (96, 2, 1, 64), (65536, 128, 16, 128)]


def oproj(b, k, h, cus):
    p = B.o_proj_plan(b, k, h, cus)
    need = -(-p.k_splits * b * h * 4 // 256) * 256
    if p.k_splits == 1:
        need += b * (h // 16) * p.ss_parts * 4
    return p, need


def prelude(b, k, hq, hkv, d, norm, cus):
    p = B.prelude_plan(B.prelude_dims(b, k, hq, hkv, d, d, 0, 1e4, 1e-6), norm, cus)
    return p, 0 if p.fused else p.k_splits * b * (hq + 2 * hkv) * d * 4


def _covers(plan_of, what):
    last = 0
    for b in range(1, 257):
        p, need = plan_of(b)
        assert p.workspace_bytes >= need, f"{what}: batch {b} writes {need} bytes of {p.workspace_bytes}"
        assert p.workspace_bytes >= last, f"{what}: batch {b} asks for less than batch {b - 1}"
        last = p.workspace_bytes


@pytest.mark.parametrize("k,h", OPROJ, ids=[f"K{c[0]}-H{c[1]}" for c in OPROJ])
def test_o_proj_workspace_covers_smaller_batches(k, h):
    for cus in CUS:
        _covers(lambda b: oproj(b, k, h, cus), f"{cus} CUs")


@pytest.mark.parametrize("k,hq,hkv,d", PRELUDE, ids=[f"H{c[0]}-{c[1]}:{c[2]}-D{c[3]}" for c in PRELUDE])
def test_prelude_workspace_covers_smaller_batches(k, hq, hkv, d):
    for cus in CUS:
        for norm in (False, True):
            _covers(lambda b: prelude(b, k, hq, hkv, d, norm, cus), f"{cus} CUs, norm {norm}")


def test_plan_arguments():
    assert B.o_proj_plan(0, 96, 128).workgroups == 0
    for bad in ((257, 96, 128, 256), (1, 40, 128, 256), (1, 96, 20, 256), (65, 96, 144, 256), (1, 96, 128, 0)):
        with pytest.raises(B.PdaError):
            B.o_proj_plan(*bad)
    dims = B.prelude_dims(4, 96, 4, 2, 64, 64, 0, 1e4, 1e-6)
    assert B.prelude_plan(dims).fused == 1 and B.prelude_plan(dims, qk_norm=True).fused == 0
    with pytest.raises(B.PdaError):
        B.prelude_plan(dims, num_cus=0)
    dims.batch = 257
    with pytest.raises(B.PdaError):
        B.prelude_plan(dims)


@pytest.mark.gpu
@pytest.mark.parametrize("warm", ["reserved", "called"])
def test_a_workspace_of_one_batch_serves_smaller_captures(gpu_lib, warm):
    """o_proj and both kinds of prelude at the largest batch, then captured at
    smaller ones on that stream; the first graph is replayed after eager calls
    at others, which must not have moved its buffer."""
    import torch
    lib = gpu_lib
    k, h, hq, hkv, d = 4096, 4096, 32, 8, 128
    rows, big = (hq + 2 * hkv) * d, 256
    gen = torch.Generator(device="cuda").manual_seed(3)

    def bf(*shape):
        return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    wo, w = lib.pack_weights(bf(h, k) * 0.02), lib.pack_weights(bf(rows, h) * 0.02)
    x, res, nw, qn = bf(big, k), bf(big, h), bf(h), bf(d)
    z, hn, q = torch.empty_like(res), torch.empty_like(res), torch.empty((big, hq, d), dtype=torch.bfloat16, device="cuda")
    kv = torch.empty((2, big, hkv, d), dtype=torch.bfloat16, device="cuda")
    lens = torch.arange(1, big + 1, dtype=torch.int32, device="cuda")

    def calls(b, norm):
        lib.o_proj_residual_norm(x[:b], wo, res[:b], nw, z[:b], hn[:b])
        lib.attention_prelude(x[:b], w, lens[:b], q[:b], kv[0, :b], kv[1, :b], num_q_heads=hq, num_kv_heads=hkv,
                              head_dim=d, rope_theta=1e4, q_norm=qn if norm else None, k_norm=qn if norm else None)

    def results():
        torch.cuda.synchronize()
        return [t.clone() for t in (z, hn, q, kv)]

    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        if warm == "reserved":
            lib.o_proj_workspace_reserve(big, k, h)
            lib.prelude_workspace_reserve(lib.prelude_dims(big, h, hq, hkv, d, d, 0, 1e4, 1e-6))
        else:
            calls(big, False)
    torch.cuda.synchronize()
    first = None
    for b in (161, 128, 65, 64, 17, 16, 1):
        for norm in (False, True):
            print("capture", warm, b, norm, flush=True)
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=s):
                calls(b, norm)
            first = first or (g, b, norm)
    with torch.cuda.stream(s):
        for b in (200, 129, 100, 33, 8):
            calls(b, True)
        for t in (z, hn, q, kv):
            t.zero_()
        calls(first[1], first[2])
    want = results()
    for t in (z, hn, q, kv):
        t.zero_()
    torch.cuda.synchronize()
    for _ in range(2):
        first[0].replay()
        for a, b in zip(results(), want):
            assert torch.equal(a, b)


@pytest.mark.gpu
def test_a_buffer_that_holds_the_plan_is_captured_and_kept(gpu_lib):
    """One sequence's buffer of o_proj has 87 KB, the plan of four writes 74
    KB: captured with that, whatever a buffer for all smaller batches has; a
    fused prelude is captured with none; and later calls leave the graph the
    buffer that it writes to."""
    import torch
    lib = gpu_lib
    k = h = 4096
    small, b = o_proj_bytes(1), 4
    assert o_proj_bytes(b, plan=True) <= small * 5 // 4 < o_proj_bytes(b)
    gen = torch.Generator(device="cuda").manual_seed(4)

    def bf(*shape):
        return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    wo, w = lib.pack_weights(bf(h, k) * 0.02), lib.pack_weights(bf(6144, h) * 0.02)
    x, res, nw = bf(16, k), bf(16, h), bf(h)
    z, hn, q = torch.empty_like(res), torch.empty_like(res), bf(16, 32, 128)
    kv = torch.empty((2, 16, 8, 128), dtype=torch.bfloat16, device="cuda")
    lens = torch.arange(1, 17, dtype=torch.int32, device="cuda")

    def calls(n, stream=None):
        lib.o_proj_residual_norm(x[:n], wo, res[:n], nw, z[:n], hn[:n], stream=stream)
        lib.attention_prelude(x[:n], w, lens[:n], q[:n], kv[0, :n], kv[1, :n], num_q_heads=32, num_kv_heads=8, head_dim=128,
                              rope_theta=1e4, stream=stream)
    assert lib.prelude_plan(lib.prelude_dims(b, h, 32, 8, 128, 128, 0, 1e4, 1e-6)).fused
    calls(b)
    torch.cuda.synchronize()
    want = [t.clone() for t in (z[:b], hn[:b], q[:b], kv[:, :b])]
    lib.release_workspaces()
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    lib.o_proj_residual_norm(x[:1], wo, res[:1], nw, z[:1], hn[:1], stream=s)
    torch.cuda.synchronize()
    print("capture", flush=True)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        calls(b, s)
    for n in (b, 1, 16):
        calls(n, s)
        torch.cuda.synchronize()
        others = [torch.full((1 << 19,), 7, dtype=torch.int32, device="cuda") for _ in range(32)]
        for t in (z, hn, q, kv):
            t.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for got, t in zip((z[:b], hn[:b], q[:b], kv[:, :b]), want):
            assert torch.equal(got, t)
        assert all(bool((t == 7).all()) for t in others)
        del others
        torch.cuda.empty_cache()
    del g
    lib.release_workspaces()


def o_proj_bytes(batch, plan=False):
    p, need = oproj(batch, 4096, 4096, 256)
    return need if plan else p.workspace_bytes
