"""The binding's native marshalling (pda_native.so): what it declines goes to
the Python checks, and what it accepts gives what those give."""
import numpy as np
import pytest
import torch

import workloads as W
from paper_2606_07665_amd import binding as pda


def _calls(b=3, dev="cpu"):
    """Every natively marshalled call with accepted arguments (name, args, kwargs)."""
    hq, hkv, d, p, n, m, hid, t = 4, 2, 64, 16, 4 * b, 4, 96, 2  # every sequence has pages of its own
    g = torch.Generator().manual_seed(b)

    def bf(*s):
        return torch.randn(*s, generator=g).to(torch.bfloat16).to(dev)

    lens = torch.full((b,), 21, dtype=torch.int32, device=dev)
    bt = (torch.arange(b * m, dtype=torch.int32).view(b, m) % n).to(dev)
    k, v = bf(n, p, hkv, d), bf(n, p, hkv, d)
    rows = (hq + 2 * hkv) * d
    w, wo = bf(rows, hid), bf(hid, hq * d)
    if dev != "cpu":
        w, wo = pda.pack_weights(w), pda.pack_weights(wo)
    shape = dict(num_q_heads=hq, num_kv_heads=hkv, head_dim=d, rope_theta=1e4)
    q = bf(b, hq, d)
    return [
        ("paged_decode_attention", [q, k, v, bt, lens, torch.zeros_like(q), 0.125], {}),
        ("paged_decode_attention_noalloc", [q, k, v, bt, lens, torch.zeros_like(q), 0.125], {}),
        ("paged_decode_attention_ext", [bf(b, t, hq, d), k, v, bt, lens, bf(b, t, hq, d), 0.125], dict(window=7)),
        ("kv_append", [bf(b, hkv, d), bf(b, hkv, d), k, v, bt, lens], {}),
        ("kv_append_n", [bf(b, t, hkv, d), bf(b, t, hkv, d), k, v, bt, lens], {}),
        ("paged_decode_attention_append",
         [q, bf(b, hkv, d), bf(b, hkv, d), k, v, bt, lens, torch.zeros_like(q), 0.125], {}),
        ("attention_prelude", [bf(b, hid), w, lens, torch.zeros_like(q), bf(b, hkv, d), bf(b, hkv, d)],
         dict(shape, bias=bf(rows), rotary_dim=32, interleaved=True)),
        ("attention_prelude_append", [bf(b, hid), w, lens, torch.zeros_like(q), k, v, bt],
         dict(shape, q_norm=bf(d), k_norm=bf(d))),
        ("o_proj_residual_norm", [bf(b, hq * d), wo, bf(b, hid), bf(hid), bf(b, hid), bf(b, hid)], dict(eps=1e-6)),
    ]


NAMES = [c[0] for c in _calls()]


def _variants(args, kwargs):
    """One argument at a time changed to something the call does not take as
    it is: a wrong dtype, rank, extent, layout or kind of object."""
    for i, a in enumerate(args):
        def put(x):
            return args[:i] + [x] + args[i + 1:], kwargs
        if isinstance(a, torch.Tensor):
            yield f"arg {i} dtype", put(a.to(torch.float16 if a.dtype == torch.bfloat16 else torch.int64))
            yield f"arg {i} rank", put(a.unsqueeze(0))
            yield f"arg {i} extent", put(torch.cat([a, a], dim=a.dim() - 1))
            yield f"arg {i} leading extent", put(torch.cat([a, a], dim=0))
            if a.dim() > 1:
                yield f"arg {i} transposed", put(a.transpose(0, a.dim() - 1).contiguous().transpose(0, a.dim() - 1))
            wide = torch.cat([a, a], dim=a.dim() - 1)
            yield f"arg {i} strided", put(wide[..., : a.shape[-1]])
            yield f"arg {i} elsewhere", put(a.cpu() if a.is_cuda else a.to("meta"))
            yield f"arg {i} none", put(None)
        else:
            yield f"arg {i} text", put("x")
    for key, val in kwargs.items():
        if isinstance(val, torch.Tensor):
            yield f"{key} dtype", (args, dict(kwargs, **{key: val.float()}))
            yield f"{key} extent", (args, dict(kwargs, **{key: torch.cat([val, val])}))
        elif isinstance(val, int) and not isinstance(val, bool):
            yield f"{key} none", (args, dict(kwargs, **{key: None}))
            yield f"{key} huge", (args, dict(kwargs, **{key: 1 << 40}))
            yield f"{key} off", (args, dict(kwargs, **{key: val + 1}))


def _outcome(name, args, kwargs):
    try:
        getattr(pda, name)(*args, **kwargs)
        return "accepted"
    except Exception as e:  # noqa: BLE001 - the exception is what is compared
        return f"{type(e).__name__}: {e}"


@pytest.mark.parametrize("i", range(len(NAMES)), ids=NAMES)
def test_cpu_tensors_are_declined_and_refused(i):
    name, args, kwargs = _calls()[i]
    with pytest.raises(ValueError):
        getattr(pda, name)(*args, **kwargs)


def test_wrong_counts_and_kinds_are_declined():
    nat = pda._import_native()
    for f in (nat.attention, nat.kv_append, nat.attention_append, nat.prelude, nat.o_proj):
        for n in (0, 1, 7, 8, 10, 18, 19):
            assert f(*([None] * n)) == pda._DECLINED
            assert f(*([object()] * n)) == pda._DECLINED
            assert f(*([torch.empty(2, 2, dtype=torch.bfloat16, device="meta")] * n)) == pda._DECLINED


@pytest.mark.parametrize("kind", ["missing", "not a library", "other torch"])
def test_without_a_native_module_the_checks_run(monkeypatch, tmp_path, kind):
    """No pda_native.so that fits this process: a warning, and the calls go
    through the Python checks as if it had declined them."""
    path = tmp_path / "pda_native.so"
    if kind == "not a library":
        path.write_bytes(b"\x7fELF nothing")
    if kind == "other torch":
        path = pda.NATIVE_PATH
        monkeypatch.setattr(pda, "_built_for", lambda: "python 3.0.0, torch 0.0.0")
    monkeypatch.setattr(pda, "NATIVE_PATH", str(path))
    monkeypatch.setattr(pda, "_nat", None)
    with pytest.warns(RuntimeWarning, match="marshalled in Python"):
        pda._load_native()
    for name, args, kwargs in _calls():
        with pytest.raises(ValueError, match="must be a GPU tensor"):
            getattr(pda, name)(*args, **kwargs)


class _Recording:
    """The native module, with what it answered."""

    def __init__(self, nat):
        self.nat, self.answers = nat, []

    def __getattr__(self, name):
        def call(*args):
            self.answers.append(getattr(self.nat, name)(*args))
            return self.answers[-1]
        return call


@pytest.mark.gpu
@pytest.mark.parametrize("i", range(len(NAMES)), ids=NAMES)
def test_the_plain_call_is_taken_natively(gpu_lib, monkeypatch, i):
    rec = _Recording(pda._import_native())
    monkeypatch.setattr(pda, "_nat", rec)
    name, args, kwargs = _calls(5, "cuda")[i]
    getattr(pda, name)(*args, **kwargs)
    torch.cuda.synchronize()
    assert rec.answers == [pda.PDA_OK]


@pytest.mark.gpu
@pytest.mark.parametrize("i", range(len(NAMES)), ids=NAMES)
def test_the_stream_is_that_of_the_checks(gpu_lib, monkeypatch, i):
    """Without a stream, the one-query attention calls take the current stream
    of the tensors' device and the others that of the current device: with
    another device current (here only by its answer) the native path leaves
    those to the Python path, unless the caller names the stream."""
    name, args, kwargs = _calls(5, "cuda")[i]
    rec = _Recording(pda._import_native(current_device=lambda: 1))
    monkeypatch.setattr(pda, "_nat", rec)
    of_tensors = name in ("paged_decode_attention", "paged_decode_attention_noalloc")
    getattr(pda, name)(*args, **kwargs)
    getattr(pda, name)(*args, stream=torch.cuda.current_stream(), **kwargs)
    torch.cuda.synchronize()
    assert rec.answers == [pda.PDA_OK if of_tensors else pda._DECLINED, pda.PDA_OK]


@pytest.mark.gpu
@pytest.mark.parametrize("i", range(len(NAMES)), ids=NAMES)
def test_native_and_python_paths_agree(gpu_lib, monkeypatch, i):
    """Accepted calls give the same bits; every changed argument gives the
    same exception, or is accepted by both."""
    got = {}
    for path in ("native", "python"):
        monkeypatch.setattr(pda, "_nat", pda._import_native() if path == "native" else pda._Declining())
        name, args, kwargs = _calls(5, "cuda")[i]
        getattr(pda, name)(*args, **kwargs)
        torch.cuda.synchronize()
        got[path] = [t.view(torch.int16).cpu().numpy() for t in args if t is not None and isinstance(t, torch.Tensor)
                     and t.dtype == torch.bfloat16]
    for a, b in zip(got["native"], got["python"]):
        assert np.array_equal(a, b)
    name, args, kwargs = _calls(5, "cuda")[i]
    for what, (a, k) in _variants(args, kwargs):
        seen = []
        for path in ("native", "python"):
            monkeypatch.setattr(pda, "_nat", pda._import_native() if path == "native" else pda._Declining())
            seen.append(_outcome(name, a, k))
        assert seen[0] == seen[1], f"{name}, {what}: {seen}"
    torch.cuda.synchronize()


@pytest.mark.gpu
def test_an_explicit_stream_is_used(gpu_lib):
    w = W.build([40, 300], 8, 2, 128, 16, seed=3)
    from _gpu import to_gpu
    dev = to_gpu(w)
    s = torch.cuda.Stream()
    outs = []
    for stream in (None, s):
        out = torch.zeros_like(dev["q"])
        torch.cuda.synchronize()
        pda.paged_decode_attention(dev["q"], dev["k"], dev["v"], dev["bt"], dev["lens"], out, float(w.scale),
                                   stream=stream)
        torch.cuda.synchronize()
        outs.append(out.view(torch.int16).cpu().numpy())
    assert np.array_equal(outs[0], outs[1])
