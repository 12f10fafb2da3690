"""The workspace of the attention calls: calls of one shape use one workspace
whatever their windows and however they plan.  On the GPU a stream warmed up by
one call is captured with others of that shape (another window, a smaller
batch, a shorter table), and the bound that pda_plan reports never falls as a
size grows."""
import pytest

from paper_2606_07665_amd import binding as B


@pytest.mark.parametrize("hq,hkv,d", [(32, 8, 128), (8, 1, 64), (12, 4, 256), (40, 40, 128), (14, 2, 128)])
def test_the_bound_never_falls(hq, hkv, d):
    for cus in (64, 256):
        rows = {}
        for bi, b in enumerate((1, 2, 3, 16, 31, 64, 129, 256, 1000)):
            for mi, m in enumerate((1, 2, 3, 16, 129, 512, 8192)):
                grid, _, rows[bi, mi] = B.plan(b, hq, hkv, d, 16, m, num_cus=cus)
                # a partial of d + 2 floats a column (16 of them) per workgroup, at the least
                assert rows[bi, mi] >= grid * 16 * (d + 2) * 4
                for prev in ((bi - 1, mi), (bi, mi - 1)):
                    assert rows[bi, mi] >= rows.get(prev, 0)


@pytest.mark.gpu
@pytest.mark.parametrize("b,hq,hkv,d,cap", [(4, 32, 8, 128, 16384), (1, 8, 1, 64, 65536), (40, 32, 2, 128, 4096),
                                            (9, 12, 4, 256, 8192)],
                         ids=["B4-32:8-D128", "B1-8:1-D64", "B40-32:2-D128", "B9-12:4-D256"])
def test_windows_share_a_workspace(gpu_lib, b, hq, hkv, d, cap):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(b)

    def bf(*shape):
        return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    pages = 64
    k, v, q = bf(pages, 16, hkv, d), bf(pages, 16, hkv, d), bf(b, 1, hq, d)
    bt = torch.randint(pages, (b, cap // 16), dtype=torch.int32, device="cuda", generator=gen)
    lens = torch.randint(1, cap + 1, (b,), dtype=torch.int32, device="cuda", generator=gen)
    out = torch.empty_like(q)
    windows = (0, 64, 300, 1024, 3000)
    want = {}
    for w in windows:
        gpu_lib.paged_decode_attention_ext(q, k, v, bt, lens, out, d ** -0.5, window=w)
        torch.cuda.synchronize()
        want[w] = out.clone()
    for warm in windows:
        s = torch.cuda.Stream()
        gpu_lib.release_workspaces()
        torch.cuda.synchronize()
        gpu_lib.paged_decode_attention_ext(q, k, v, bt, lens, out, d ** -0.5, window=warm, stream=s)
        torch.cuda.synchronize()
        for w in windows:
            print(f"warmed at window {warm}, captured at {w}", flush=True)
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=s):
                gpu_lib.paged_decode_attention_ext(q, k, v, bt, lens, out, d ** -0.5, window=w)
            out.fill_(float("nan"))
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, want[w])
            del g


@pytest.mark.gpu
def test_a_buffer_that_holds_the_plan_is_captured_and_kept(gpu_lib):
    """A single request's plan over an 8192-token table writes 534 KB, a
    shorter table's buffer has 688 KB: the call is captured with that, and once
    later calls have grown the stream's workspace the graph still writes to
    its own."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(7)

    def bf(*shape):
        return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    hq, hkv, d = 32, 8, 128
    k, v, q = bf(512, 16, hkv, d), bf(512, 16, hkv, d), bf(4, hq, d)
    bt = torch.randperm(512, dtype=torch.int32, device="cuda", generator=gen).repeat(4, 1)
    lens = torch.tensor([8000, 7000, 100, 5000], dtype=torch.int32, device="cuda")
    out = torch.empty_like(q)

    def attend(b, pages):
        """The arguments of b requests over a table of `pages` pages."""
        return q[:b], k, v, bt[:b, :pages].contiguous(), lens[:b].clamp(max=pages * 16), out[:b], d ** -0.5

    one, short, more = attend(1, 512), attend(1, 64), attend(4, 512)
    gpu_lib.paged_decode_attention(*one)
    torch.cuda.synchronize()
    want = out[:1].clone()
    gpu_lib.release_workspaces()
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    gpu_lib.paged_decode_attention(*short, stream=s)
    torch.cuda.synchronize()
    print("capture", flush=True)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        gpu_lib.paged_decode_attention(*one, stream=s)
    for args in (one, more):  # `one` fits, and grows the workspace early
        gpu_lib.paged_decode_attention(*args, stream=s)
        torch.cuda.synchronize()
        others = [torch.full((1 << 19,), 7, dtype=torch.int32, device="cuda") for _ in range(32)]
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out[:1], want)
        assert all(bool((t == 7).all()) for t in others)
        del others
        torch.cuda.empty_cache()
    del g
    gpu_lib.release_workspaces()


@pytest.mark.gpu
def test_growing_early_beside_a_capture(gpu_lib):
    """While one stream is captured, a call on another whose buffer holds its
    plan, and could be larger, runs and leaves the capture as it is."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(8)

    def bf(*shape):
        return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    hq, hkv, d = 32, 8, 128
    k, v, q = bf(512, 16, hkv, d), bf(512, 16, hkv, d), bf(1, hq, d)
    bt = torch.randperm(512, dtype=torch.int32, device="cuda", generator=gen)[None].contiguous()
    lens, few = (torch.tensor([n], dtype=torch.int32, device="cuda") for n in (8000, 1000))
    short = bt[:, :64].contiguous()
    outs = [torch.empty_like(q) for _ in range(2)]
    gpu_lib.paged_decode_attention(q, k, v, bt, lens, outs[0], d ** -0.5)
    torch.cuda.synchronize()
    want = outs[0].clone()
    gpu_lib.release_workspaces()
    captured, beside = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    for s in (captured, beside):
        gpu_lib.paged_decode_attention(q, k, v, short, few, outs[0], d ** -0.5, stream=s)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    print("capture", flush=True)
    with torch.cuda.graph(g, stream=captured):
        gpu_lib.paged_decode_attention(q, k, v, bt, lens, outs[0], d ** -0.5, stream=captured)
        gpu_lib.paged_decode_attention(q, k, v, bt, lens, outs[1], d ** -0.5, stream=beside)
    torch.cuda.synchronize()
    assert torch.equal(outs[1], want)
    outs[0].zero_()
    torch.cuda.synchronize()
    g.replay()
    torch.cuda.synchronize()
    assert torch.equal(outs[0], want)
    del g
    gpu_lib.release_workspaces()
