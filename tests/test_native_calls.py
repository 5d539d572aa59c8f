"""The binding's native calls (csrc/pycall.c) and the ctypes calls that stand in for them where the
module was not built give the same answers; a build without a C compiler goes on without the module."""
import importlib.util
import os
import sys
import types

import numpy as np
import pytest

import paper_2510_03275_amd as P
from paper_2510_03275_amd import binding as Bd

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _ctypes_calls(monkeypatch):
    monkeypatch.setitem(sys.modules, "paper_2510_03275_amd._sdqcall", None)
    monkeypatch.delattr(P, "_sdqcall", raising=False)
    calls = Bd._native_calls()
    assert not any(isinstance(c, types.BuiltinFunctionType) for c in calls)
    return calls


def _use(monkeypatch, calls):
    for name, fn in zip(("_call_linear", "_call_group", "_call_workspace"), calls):
        monkeypatch.setattr(Bd, name, fn)


def _build_module():
    spec = importlib.util.spec_from_file_location("_build", os.path.join(ROOT, "paper_2510_03275_amd", "build.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


def test_ctypes_calls_validate_alike(monkeypatch):
    torch = pytest.importorskip("torch")
    stream = types.SimpleNamespace(cuda_stream=0)
    L = P.sdq_layout_init(130, 512, 2.0, 3)
    x = torch.zeros(3, 512, dtype=torch.bfloat16)
    enc = P.Encoded(L, torch.zeros(16), torch.zeros(16))
    group = P.LinearGroup([enc, enc], [torch.zeros(3, 130)] * 2)
    native = (Bd._call_linear, Bd._call_group, Bd._call_workspace)
    seen = []
    for calls in (native, _ctypes_calls(monkeypatch)):
        _use(monkeypatch, calls)
        got = [calls[2](Bd._addr(L), m) for m in (0, 1, 16, 17, 2048)]
        for fn in (lambda: P.sdq_linear(x, enc.codes, enc.scales, L, x, None, stream),
                   lambda: P.sdq_linear(x, None, enc.scales, L, x, x, stream),
                   lambda: P.sdq_linear(x[0], enc.codes, enc.scales, L, x, x, stream),
                   lambda: P.sdq_linear_group(x, group, x[:, :8].contiguous(), stream, accumulate=True)):
            try:
                fn()
                got.append(0)
            except P.SdqError as e:
                got.append((e.status, str(e)))
        seen.append(got)
    assert seen[0] == seen[1]
    assert seen[0][5][0] == -6 and seen[0][6][0] == -1 and seen[0][7] == 0 and seen[0][8][0] == -6


@pytest.mark.gpu
@pytest.mark.parametrize("m", [1, 5, 40])
def test_ctypes_calls_give_the_same_results(monkeypatch, m):
    from tests.gpu_common import require_gpu
    torch = require_gpu()
    w = torch.from_numpy(np.random.default_rng(1).normal(0, 0.02, (130, 512)).astype(np.float32)).cuda()
    enc = P.quantize(w, 2.0, 3)
    x = torch.randn(m, 512, device="cuda").half()
    out = []
    for calls in ((Bd._call_linear, Bd._call_group, Bd._call_workspace), _ctypes_calls(monkeypatch)):
        _use(monkeypatch, calls)
        ys = [torch.empty(m, 130, device="cuda") for _ in range(2)]
        ws = torch.empty(P.sdq_linear_group_workspace_bytes([enc.layout] * 2, m), dtype=torch.uint8, device="cuda")
        P.sdq_linear_group(x, P.LinearGroup([enc, enc], ys), ws)
        with torch.cuda.stream(torch.cuda.Stream()):
            torch.cuda.current_stream().wait_stream(torch.cuda.default_stream())
            out.append([P.linear(x, enc), *ys])
        torch.cuda.synchronize()
    # one row: the parts of K (a few) are added to y in any order, 2^-24 of the largest per add
    bound = 1e-6 if m == 1 else 0.0
    for a, b in zip(*out):
        assert torch.max(torch.abs(a - b)).item() <= bound * torch.max(torch.abs(a)).item()


def test_module_is_named_for_this_interpreter():
    import sysconfig
    assert os.path.basename(_build_module().PYCALL) == "_sdqcall" + sysconfig.get_config_var("EXT_SUFFIX")
    assert not os.path.exists(os.path.join(ROOT, "paper_2510_03275_amd", "_sdqcall.so"))


def test_build_goes_on_without_a_compiler(monkeypatch, tmp_path):
    mod = _build_module()
    stale = tmp_path / "_sdqcall.so"
    stale.write_bytes(b"")
    monkeypatch.setattr(mod, "PYCALL", str(tmp_path / os.path.basename(mod.PYCALL)))
    monkeypatch.setenv("PATH", str(tmp_path))
    mod._build_pycall()
    assert os.listdir(tmp_path) == []
