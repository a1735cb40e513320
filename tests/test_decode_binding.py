"""The native part of the decode step's binding against the general one in api.py, over what the entry point takes."""
import os
import shutil
import subprocess
import sys
from types import SimpleNamespace

import pytest
import torch

B, H, DK, DV, M = 2, 3, 64, 128, 16


def _args(dtype, device):
    gen = torch.Generator().manual_seed(3)
    t = lambda *s: torch.randn(*s, generator=gen)
    x = dict(q=t(B, H, DK).to(dtype), k=t(B, H, DK).to(dtype), v=t(B, H, DV).to(dtype), g=-t(B, H, M).abs(),
             K_state=t(B, H, M, DK), V_state=t(B, H, M, DV))
    return {n: a.to(device) for n, a in x.items()}


def _both(monkeypatch, x, **kw):
    """(native, general): each a (result, updated memories) or the exception."""
    from paper_2409_07146_amd import api
    out = []
    for native in (True, False):
        if not native:
            monkeypatch.setattr(api, "_native_decode", None)
        y = {n: (a.clone() if isinstance(a, torch.Tensor) and n.endswith("state") else a) for n, a in x.items()}
        own = dict(kw, out=torch.full_like(kw["out"], float("nan"))) if "out" in kw else kw
        try:
            o = api.gsa_decode_step(**y, **own)
            assert "out" not in own or o is own["out"]
            out.append((o, y["K_state"], y["V_state"]))
        except Exception as e:
            out.append(e)
    monkeypatch.undo()
    return out


def test_native_part_is_built_and_leaves_other_cases_alone():
    from paper_2409_07146_amd import _lib
    assert _lib.native is not None
    x = _args(torch.float32, "cpu")
    rest = (1.0, None, None, None, 0, 0.0, 0)
    assert _lib.native.decode_step(1, None, *x.values(), *rest) is None          # not on the GPU
    assert _lib.native.decode_step(1, None, None, *list(x.values())[1:], *rest) is None
    with pytest.raises(TypeError):
        _lib.native.decode_step(1, None)


def test_package_imports_with_a_native_part_that_does_not(tmp_path):
    """A file that is no module, as one built against another torch or Python would be."""
    from paper_2409_07146_amd import _lib
    here = os.path.dirname(_lib.__file__)
    pkg = tmp_path / "paper_2409_07146_amd"
    pkg.mkdir()
    for name in os.listdir(here):
        if name.endswith(".py"):
            shutil.copy(os.path.join(here, name), pkg)
    (pkg / "_binding.so").write_bytes(b"not a shared object")
    code = "import paper_2409_07146_amd as g; from paper_2409_07146_amd import _lib, api; assert _lib.native is None and api._native_decode is None; print(g.__file__)"
    res = subprocess.run([sys.executable, "-c", code], cwd=tmp_path, env=dict(os.environ, PYTHONPATH=str(tmp_path)), capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    assert str(tmp_path) in res.stdout and "native part of the binding is left out" in res.stderr


def test_native_part_of_another_version_is_left_out(monkeypatch):
    import paper_2409_07146_amd
    from paper_2409_07146_amd import _lib
    here = (torch.__version__.split("+")[0], "%d.%d" % sys.version_info[:2])
    assert _lib.native.built_for == here
    for other in (SimpleNamespace(built_for=("1.0.0", here[1])), SimpleNamespace(built_for=(here[0], "2.7")), SimpleNamespace()):
        monkeypatch.setitem(sys.modules, "paper_2409_07146_amd._binding", other)
        monkeypatch.setattr(paper_2409_07146_amd, "_binding", other)
        with pytest.warns(UserWarning, match="left out"):
            assert _lib._load_native() is None


@pytest.mark.parametrize("error", [FileNotFoundError("g++"), RuntimeError("no headers")])
def test_library_is_linked_without_the_native_part(monkeypatch, tmp_path, capsys, error):
    from paper_2409_07146_amd import build

    def fail():
        raise error
    linked = []
    (tmp_path / "_binding.so").write_bytes(b"older")
    monkeypatch.setattr(build, "BINDING", str(tmp_path / "_binding.so"))
    monkeypatch.setattr(build, "OBJ", str(tmp_path))
    monkeypatch.setattr(build, "LIB", str(tmp_path / "libgsa.so"))
    monkeypatch.setattr(build, "_compile", lambda src: src)
    monkeypatch.setattr(build, "_compile_binding", fail)
    monkeypatch.setattr(build.subprocess, "run", lambda cmd, **kw: linked.append(cmd))
    assert build.build() == str(tmp_path / "libgsa.so")
    assert len(linked) == 1 and "-shared" in linked[0] and not (tmp_path / "_binding.so").exists()
    assert "left out" in capsys.readouterr().err


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("opts", [{}, dict(workspace=True), dict(out=True), dict(scale=2, workspace=True, out=True), dict(s=True),
                                  dict(readout="swish"), dict(gate_tau=8.0, feature_map="swish", workspace=True)])
def test_same_results(monkeypatch, dtype, opts):
    import paper_2409_07146_amd as gsa
    x, kw = _args(dtype, "cuda"), dict(opts)
    if kw.pop("workspace", False):
        kw["workspace"] = gsa.alloc_decode_workspace(B, H, DK, DV, M, torch.device("cuda"))
    if kw.pop("out", False):
        kw["out"] = torch.empty_like(x["v"])
    if kw.pop("s", False):
        kw["s"] = torch.rand(B, H, M, device="cuda")
    calls = []
    from paper_2409_07146_amd import api
    native = api._native_decode
    monkeypatch.setattr(api, "_native_decode", lambda *a: calls.append(native(*a)) or calls[-1])
    o = api.gsa_decode_step(**{n: a.clone() for n, a in x.items()}, **kw)
    assert calls == [o]                                       # the native part did it
    if "out" in kw:
        assert o is kw["out"]
    monkeypatch.undo()
    a, b = _both(monkeypatch, x, **kw)
    assert a[0] is not b[0] and not a[0].isnan().any()
    assert all(torch.equal(s, t) for s, t in zip(a, b))


@pytest.mark.gpu
def test_traced_calls_take_the_general_way(monkeypatch):
    from paper_2409_07146_amd import api
    x, taken = _args(torch.float32, "cuda"), []
    native = api._native_decode
    monkeypatch.setattr(api, "_native_decode", lambda *a: taken.append(native(*a)) or taken[-1])
    rest = {n: a for n, a in x.items() if n != "q"}
    traced = torch.jit.trace(lambda q: api.gsa_decode_step(q, **rest), x["q"], check_trace=False)
    assert taken == [None] and "aten::empty_like" in str(traced.graph)


@pytest.mark.gpu
@pytest.mark.parametrize("change", ["strided", "dtype", "shape", "cpu", "readout", "small_ws", "ws_dtype", "mode", "half", "tau"])
def test_same_treatment_of_the_rest(monkeypatch, change):
    from torch.overrides import TorchFunctionMode

    import paper_2409_07146_amd as gsa
    x, kw = _args(torch.float32, "cuda"), {}
    if change == "strided":
        x["q"] = x["q"].transpose(0, 1).contiguous().transpose(0, 1)
    elif change == "dtype":
        x["g"] = x["g"].double()
    elif change == "shape":
        x["K_state"] = x["K_state"][:, :, :8].contiguous()
    elif change == "cpu":
        x["k"] = x["k"].cpu()
    elif change == "readout":
        kw["readout"] = "nothing"
    elif change == "small_ws":
        kw["workspace"] = torch.empty(16, dtype=torch.uint8, device="cuda")
    elif change == "ws_dtype":   # its length counts elements here
        n = gsa.gsa_decode_workspace_bytes(B, H, DK, DV, M)
        kw["workspace"] = torch.empty(n, dtype=torch.int32, device="cuda")
    elif change == "half":
        x["q"], x["k"], x["v"] = (x[n].half() for n in "qkv")
    elif change == "tau":
        kw["gate_tau"] = -1.0
    if change == "mode":
        class Mode(TorchFunctionMode):
            seen = 0

            def __torch_function__(self, func, types, args=(), kwargs=None):
                Mode.seen += func is torch.empty_like
                return func(*args, **(kwargs or {}))
        with Mode():
            a, b = _both(monkeypatch, x, **kw)
        assert Mode.seen == 2   # a mode sees the allocation either way
    else:
        a, b = _both(monkeypatch, x, **kw)
    assert type(a) is type(b)
    if isinstance(a, Exception):
        assert (str(a), getattr(a, "code", None)) == (str(b), getattr(b, "code", None))
    else:
        assert all(torch.equal(s, t) for s, t in zip(a, b))
