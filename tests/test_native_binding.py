"""The native form of the entry points (csrc/binding.cpp): it declines whatever
is not plain, and where it answers, outputs, identities and errors are those of
the Python form."""
import warnings

import pytest
import torch

import paper_2609_33916_amd as pkg
from helpers import gpu_available


@pytest.fixture
def native():
    pkg.lib()
    # the package's build makes both: without the binding calls still work, slower
    assert pkg._native is not None, "the library is built but its native binding is missing or does not load"
    return pkg._native


def test_declines_what_is_not_plain(native):
    x, l = torch.zeros(1, 1, 8, 32), torch.zeros(1, 1, 8)
    c = torch.zeros(1, 8, 32)
    for args in ((x, x, x, None, False, None), (x, None, x, 1.0, False, None), (1, x, x, None, False, None), (x,)):
        assert native.fwd(*args) is NotImplemented
    assert native.fwd_bwd(x, x, x, x, None, False, None, None) is NotImplemented
    assert native.bwd(x, x, x, x, l, x, None, False, None, None) is NotImplemented
    assert native.decode(c, x, x, None, None, None, 8, None, None, None) is NotImplemented


def _both(monkeypatch, call):
    got = call()
    with monkeypatch.context() as m:
        m.setattr(pkg, "_native_lib", None)
        want = call()
    torch.cuda.synchronize()
    return got, want


@pytest.mark.gpu
@pytest.mark.skipif(not gpu_available(), reason="needs a GPU")
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_same_as_the_python_form(native, monkeypatch, dtype):
    q, k, v, g = (torch.randn(2, 3, 100, 64, device="cuda", dtype=dtype) for _ in range(4))
    o, lse = pkg.attn_fwd(q, k, v, causal=True)
    lens = torch.tensor([5, 90], dtype=torch.int32, device="cuda")
    new = torch.randn(2, 3, 64, device="cuda", dtype=torch.bfloat16)
    qd, kc, vc = torch.randn(2, 6, 64, device="cuda", dtype=torch.bfloat16), *(
        torch.randn(2, 3, 100, 64, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    calls = [lambda: pkg.attn_fwd(q, k, v, causal=True), lambda: pkg.attn_fwd(q, k, v, -0.3),
             lambda: pkg.attn_fwd_bwd(q, k, v, g, causal=False),
             lambda: pkg.attn_bwd(q, k, v, o, lse, g, causal=True),
             lambda: pkg.attn_decode(qd, kc, vc, new, new, cache_lens=lens, n=90),
             lambda: pkg.attn_decode(qd, kc, vc, n=100, scale=0.2)]
    for call in calls:
        got, want = _both(monkeypatch, call)
        assert type(got) is tuple and len(got) == len(want)
        for a, b in zip(got, want):
            assert a.dtype == b.dtype and a.shape == b.shape and a.stride() == b.stride() and torch.equal(a, b)


@pytest.mark.gpu
@pytest.mark.skipif(not gpu_available(), reason="needs a GPU")
def test_given_outputs_workspace_stream_and_errors(native, monkeypatch):
    q, k, v, g = (torch.randn(1, 2, 70, 128, device="cuda", dtype=torch.bfloat16) for _ in range(4))
    out = (torch.empty_like(q), torch.empty(1, 2, 70, device="cuda"), *(torch.empty_like(q) for _ in range(3)))
    ws = torch.empty(pkg.attn_workspace_bytes(1, 2, 70, 128), dtype=torch.uint8, device="cuda")
    want = pkg.attn_fwd_bwd(q, k, v, g)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        r = pkg.attn_fwd_bwd(q, k, v, g, out=out, workspace=ws)
    side.synchronize()
    assert all(a is b for a, b in zip(r, out)) and all(torch.equal(a, b) for a, b in zip(r, want))
    odd = torch.zeros(1, 1, 8, 48, device="cuda", dtype=torch.bfloat16)
    half = odd.half()
    for bad in (lambda: pkg.attn_fwd(odd, odd, odd), lambda: pkg.attn_fwd(half, half, half),
                lambda: pkg.attn_fwd(q, k.float(), v), lambda: pkg.attn_fwd(q, k.transpose(1, 2), v),
                lambda: pkg.attn_fwd(q, k, v, scale=float("inf")),
                lambda: pkg.attn_fwd_bwd(q, k, v, g, workspace=ws[1:]), lambda: pkg.attn_fwd(q[0], k[0], v[0])):
        seen = []
        for direct in (True, False):
            with monkeypatch.context() as m:
                if not direct:
                    m.setattr(pkg, "_native_lib", None)
                with pytest.raises((ValueError, TypeError, pkg.AttnError)) as e:
                    bad()
                seen.append((e.type, str(e.value)))
        assert seen[0] == seen[1]


def test_a_binding_that_does_not_load_is_reported(monkeypatch):
    """A missing module is no error; one that fails to import warns, and calls
    go through the Python form in both cases."""
    import importlib
    loaded = pkg.lib()
    for error in (ModuleNotFoundError("no module"), ImportError("undefined symbol: _ZN3c10")):
        def fail(name):
            raise error
        with monkeypatch.context() as m, warnings.catch_warnings(record=True) as seen:
            warnings.simplefilter("always")
            m.setattr(pkg, "_native", None)
            m.setattr(pkg, "_native_lib", None)
            m.setattr(importlib, "import_module", fail)
            pkg._bind_native(loaded)
            assert pkg._native is None and pkg._native_lib is None
        assert [str(w.message) for w in seen if "undefined symbol" in str(w.message)] == \
            ([] if isinstance(error, ModuleNotFoundError) else [str(seen[-1].message)])


def test_a_failed_binding_build_leaves_the_library(monkeypatch, tmp_path):
    """The binding's compile may fail (no torch headers): the library is built,
    the failure is told, and no stale binding stays behind."""
    from paper_2609_33916_amd import build
    lib_path, binding = tmp_path / "libattn_mi355x.so", tmp_path / "_binding.so"
    binding.write_text("stale")
    monkeypatch.setattr(build, "LIB_PATH", str(lib_path))
    monkeypatch.setattr(build, "BINDING_PATH", str(binding))
    monkeypatch.setattr(build, "SOURCES", {"empty.hip": []})
    (tmp_path / "empty.hip").write_text("extern \"C\" int answer() { return 42; }\n")
    monkeypatch.setattr(build, "binding_command", lambda out: ["false"])
    with pytest.warns(RuntimeWarning, match="binding"):
        assert build.build(out=str(lib_path), csrc=str(tmp_path)) == str(lib_path)
    assert lib_path.exists() and not binding.exists()
