"""The native marshalling of the binding: what is not the plain call is handed back untouched (CPU), and the plain call gives
the results, errors and outputs of the general way (GPU), which an explicit stream takes."""
import math
import sys
import sysconfig
import types

import pytest
import torch

import paper_2601_21444_amd as apbv
import paper_2601_21444_amd.binding as binding


class Sub(torch.Tensor):
    pass


def cpu_args():
    parts, lse, out = torch.zeros(2, 3, 4, 64, dtype=torch.bfloat16), torch.zeros(2, 4, 3), torch.zeros(3, 4, 64, dtype=torch.bfloat16)
    q, k = torch.zeros(5, 2, 64, dtype=torch.bfloat16), torch.zeros(5, 1, 64, dtype=torch.bfloat16)
    return parts, lse, out, q, k


def test_other_than_plain_calls_are_handed_back():
    apbv.load_library()
    nat = binding._native
    parts, lse, out, q, k = cpu_args()
    assert nat.merge_lse(parts, lse, out, None) is None                    # not on a GPU
    assert nat.merge_lse(1, lse, out, None) is None and nat.merge_lse(parts, lse) is None
    assert nat.merge_lse(parts.as_subclass(Sub), lse, out, None) is None
    assert nat.host_attention(q, k, k, k, k, k, k, "scale", out, None) is None
    assert nat.host_attention(q.float(), k, k, k, k, k, k, 1.0, out, None) is None
    assert nat.query_attention(q, k, k, k, k, k, k, 1.0, True, out, None, out) is None
    assert nat.attention_group("xy", 1.0, False) is None and nat.attention_group([], 1.0, False) is None
    assert nat.attention_group([(q,) * 7], 1.0, False) is None             # outputs to be allocated
    for l_p in (True, 2.0, 6, -1):
        assert nat.compress_kv(q, k, k, l_p, 0, 0.0, out, out, out, None, out) is None
    seen = []
    torch.func.vmap(lambda x: (seen.append(nat.merge_lse(x, lse, out, None)), x.sum())[1])(parts[None])
    with torch.overrides.TorchFunctionMode():
        seen.append(nat.merge_lse(parts, lse, out, None))
    assert seen == [None, None]
    with pytest.raises(ValueError):                                        # ... and the general way says what is wrong
        apbv.apbv_merge_lse(parts, lse, out=out)
    with pytest.raises(TypeError):
        apbv.apbv_host_attention(q.float(), k, k, k, k, k, k, 1.0, out=out)


def loaded_again(monkeypatch, module):
    """The binding's native part after loading the library with this module as the extension (None: there is none)."""
    monkeypatch.setitem(sys.modules, "paper_2601_21444_amd._marshal", module)
    monkeypatch.delattr(apbv, "_marshal", raising=False)
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_native", None)
    assert apbv.load_library() is not None and apbv.apbv_version() >= 100
    return binding._native


def test_the_library_loads_without_the_extension(monkeypatch):
    """... and every call goes the general way, whose messages these are."""
    native = loaded_again(monkeypatch, None)
    parts, lse, out, q, k = cpu_args()
    assert native.merge_lse(parts, lse, out, None) is None
    with pytest.raises(ValueError, match="must live on"):
        apbv.apbv_merge_lse(parts, lse, out=out)
    with pytest.raises(ValueError, match="must live on"):
        apbv.apbv_host_attention(q, k, k, k, k, k, k, 1.0, out=out.new_zeros(1, 5, 2, 64))
    assert native.attention_group([], 1.0, False) is None and native.compress_kv() is None and native.query_attention() is None


def test_an_extension_of_another_build_is_not_used(monkeypatch):
    apbv.load_library()
    real = binding._native
    for other in (dict(version=real.version + 1, library=real.library), dict(version=real.version, library=real.library + 8), {}):
        module = types.ModuleType("paper_2601_21444_amd._marshal")
        module.merge_lse = lambda *a: pytest.fail("called")
        for name, value in other.items():
            setattr(module, name, value)
        with pytest.warns(RuntimeWarning, match="marshalling"):
            assert loaded_again(monkeypatch, module).merge_lse(1, 2, 3, 4) is None


def test_the_library_is_built_without_what_the_extension_needs(monkeypatch, tmp_path, capsys):
    from paper_2601_21444_amd import build as b
    ran = []
    monkeypatch.setattr(b, "OBJ", str(tmp_path))
    monkeypatch.setattr(b.subprocess, "run", lambda cmd, **kw: ran.append(cmd))
    b.build(verbose=False)
    assert any(cmd[-1] == b.LIB for cmd in ran) and any(str(cmd[-1]).endswith(sysconfig.get_config_var("EXT_SUFFIX")) for cmd in ran)
    for lacks in ("torch", "CXX"):
        ran.clear()
        with monkeypatch.context() as m:
            if lacks == "torch":
                m.setitem(sys.modules, "torch", None)
            else:
                m.setenv("CXX", str(tmp_path / "no-compiler"))
            b.build(verbose=False)
        assert [cmd[-1] for cmd in ran if "-shared" in cmd] == [b.LIB] and "not built" in capsys.readouterr().out


def bf(*s):
    return torch.randn(s, device="cuda", dtype=torch.bfloat16)


class Recorder:
    """The native marshalling with a note of what each of its functions said."""

    def __init__(self, native):
        self.native, self.said = native, []

    def __getattr__(self, name):
        def call(*args):
            self.said.append(getattr(self.native, name)(*args))
            return self.said[-1]
        return call


@pytest.fixture
def native(monkeypatch):
    apbv.load_library()
    recorder = Recorder(binding._native)
    monkeypatch.setattr(binding, "_native", recorder)
    return recorder


def both(native, call, args, outs, said=0, **kw):
    """The outputs of the native and of the general way, the buffers filled with different values before each; `said`: what the
    native function returns in the call that asks it (None: handed back)."""
    got = []
    for fill, extra in ((1, {}), (3, {"stream": torch.cuda.current_stream()})):
        for t in outs.values():
            t.fill_(fill)
        native.said.clear()
        result = call(*args, **outs, **kw, **extra)
        torch.cuda.synchronize()
        assert native.said == ([] if extra else [said])
        flat = result if isinstance(result, tuple) else (result,)
        got.append(([tuple(t.shape) for t in flat], [t.clone() for t in outs.values() if t.dtype != torch.uint8]))
    assert got[0][0] == got[1][0]
    for a, b in zip(got[0][1], got[1][1]):
        assert torch.equal(a, b)


@pytest.mark.gpu
@pytest.mark.parametrize("batched", [False, True])
@pytest.mark.parametrize("form", ["dense", "strided", "empty segments"])
def test_native_and_general_marshalling_agree(native, batched, form):
    b, L, hq, hkv, d, nv = 2, 150, 4, 2, 64, 40
    lead = (b,) if batched else ()
    n_b = b if batched else 1

    def kv(n, h):
        if form == "strided":                   # a slice of an interleaved cache: every stride differs from the dense one
            return bf(*lead, n + 3, 2 * h, d)[..., 2:n + 2, h:, :] if n else bf(*lead, 0, h, d)
        return bf(*lead, n, h, d)
    nv = 0 if form == "empty segments" else nv
    q, k, v, ka, va, e = kv(L, hq), kv(L, hkv), kv(L, hkv), kv(nv, hkv), kv(nv, hkv), bf(*lead, 0, hkv, d)
    scale = 1 / math.sqrt(d)
    new = lambda *s, dtype=torch.bfloat16: torch.empty((n_b,) + s, device="cuda", dtype=dtype)
    print("marshal", batched, form, flush=True)
    both(native, apbv.apbv_host_attention, (q, ka, va, e, e, k, v, scale), dict(out=new(L, hq, d), lse_out=new(hq, L, dtype=torch.float32)), return_lse=True)
    both(native, apbv.apbv_host_attention, (q, ka, va, e, e, k, v, scale), dict(out=new(L, hq, d)))
    ws = torch.empty(max(256, apbv.apbv_query_attention_workspace_bytes(n_b, hq, d, 9, L + nv, 2)), dtype=torch.uint8, device="cuda")
    both(native, apbv.apbv_query_attention, (q[..., :9, :, :], ka, va, k, v, e, e, scale), dict(out=new(9, hq, d), lse_out=new(hq, 9, dtype=torch.float32), workspace=ws), n_splits=2, return_lse=True)
    for reducer in ("sum", "max", "softmax_sum"):
        ws = torch.empty(apbv.apbv_compress_reduced_workspace_bytes(reducer, n_b, hq, hkv, d, 9, L, 33), dtype=torch.uint8, device="cuda")
        outs = dict(idx_out=new(hkv, 33, dtype=torch.int32), k_c_out=new(33, hkv, d), v_c_out=new(33, hkv, d), scores_out=new(hkv, L, dtype=torch.float64), workspace=ws)
        both(native, apbv.apbv_compress_kv, (q[..., :9, :, :], k, v, 33), outs, reducer=reducer, softmax_scale=scale, return_scores=True)
    del outs["workspace"], outs["scores_out"]
    both(native, apbv.apbv_compress_kv_noalloc, (q[..., :9, :, :], k, v, 33), outs)
    if not batched:
        group = [(q, ka, va, e, e, k, v, new(L, hq, d)[0], new(hq, L, dtype=torch.float32)[0]) for _ in range(2)]
        native.said.clear()
        kept = [(o.clone(), s.clone()) for o, s in apbv.apbv_host_attention_group(group, scale, return_lse=True)]
        assert native.said == [0]
        general = apbv.apbv_host_attention_group([list(g) for g in group], scale, return_lse=True, stream=torch.cuda.current_stream())
        torch.cuda.synchronize()
        for (o, s), (o2, s2) in zip(kept, general):
            assert torch.equal(o, o2) and torch.equal(s, s2)


@pytest.mark.gpu
def test_merge_and_refusals_agree(native):
    parts, lse = bf(3, 7, 4, 64), torch.randn(3, 4, 7, device="cuda")
    outs = dict(out=torch.empty(7, 4, 64, device="cuda", dtype=torch.bfloat16), lse_out=torch.empty(4, 7, device="cuda"))
    both(native, apbv.apbv_merge_lse, (parts, lse), outs, return_lse=True)
    both(native, apbv.apbv_merge_lse, (bf(3, 14, 4, 64)[:, :7], lse), outs, said=None)        # strided parts: handed back
    q, k, e = bf(9, 4, 64), bf(9, 2, 64), bf(0, 2, 64)
    cases = [lambda **s: apbv.apbv_merge_lse(bf(3, 7, 4, 96), lse, out=torch.empty(7 * 4 * 96, device="cuda", dtype=torch.bfloat16), **s),
             lambda **s: apbv.apbv_host_attention(q, e, e, e, e, k, k, -1.0, out=torch.empty_like(q), **s),
             lambda **s: apbv.apbv_host_attention(q, e, e, e, e, k, k, 1.0, out=torch.empty(9 * 4 * 64 + 1, device="cuda", dtype=torch.bfloat16)[1:], **s),
             lambda **s: apbv.apbv_host_attention(q, e, e, e, e, k, k, 1.0, out=torch.empty(3, device="cuda", dtype=torch.bfloat16), **s),
             lambda **s: apbv.apbv_compress_kv(q, k, k, 10, workspace=torch.empty(1 << 20, dtype=torch.uint8, device="cuda"), idx_out=torch.empty(20, dtype=torch.int32, device="cuda"),
                                               k_c_out=torch.empty(2000, dtype=torch.bfloat16, device="cuda"), v_c_out=torch.empty(2000, dtype=torch.bfloat16, device="cuda"), **s)]
    # what the library refuses is refused by it either way; a buffer or a size that the binding refuses is handed back
    for case, status in zip(cases, (-3, -2, -2, None, None)):
        said = []
        for s in ({}, {"stream": torch.cuda.current_stream()}):
            native.said.clear()
            with pytest.raises(Exception) as err:
                case(**s)
            said.append((err.type, str(err.value)))
            assert native.said == ([] if s else [status])
        assert said[0] == said[1]


@pytest.mark.gpu
@pytest.mark.parametrize("asked", [0, 1, 2])
def test_what_is_raised_while_the_stream_is_asked_for_is_not_lost(asked):
    """The functions that name the stream run Python code, where a signal's handler may raise: the call ends with it."""
    binding.load_library()
    parts, lse, out = bf(3, 7, 4, 64), torch.randn(3, 4, 7, device="cuda"), torch.full((7, 4, 64), 5.0, device="cuda", dtype=torch.bfloat16)
    functions = [torch.cuda.is_initialized, binding._current_device, binding._raw_stream]

    def interrupted(*_):
        raise KeyboardInterrupt
    try:
        binding._native.use_stream(*[interrupted if i == asked else f for i, f in enumerate(functions)])
        with pytest.raises(KeyboardInterrupt):
            apbv.apbv_merge_lse(parts, lse, out=out)
    finally:
        binding._native.use_stream(*functions)
    torch.cuda.synchronize()
    assert (out == 5.0).all()
    assert binding._native.merge_lse(parts, lse, out, None) == 0
