"""The native part of the decode step's binding against the general one in api.py, over what the entry point takes."""
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
        try:
            o = api.gsa_decode_step(**y, **kw)
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
    assert all(torch.equal(s, t) for s, t in zip(a, b))


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
        assert (type(a), getattr(a, "code", None)) == (type(b), getattr(b, "code", None))
    else:
        assert all(torch.equal(s, t) for s, t in zip(a, b))
