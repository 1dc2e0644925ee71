"""The native way from tensors to the C functions: what it takes, what it leaves to ctypes, and that both give the same."""
import subprocess
import sys

import pytest
import torch

from paper_2410_08661_amd import binding as B
from paper_2410_08661_amd import build


class Sub(torch.Tensor):
    pass


def test_anything_but_plain_device_tensors_is_left_alone():
    d = B.make_desc(64, 256, 8, 4, 128)
    w, x = B.Weight(d, "cpu"), torch.zeros((2, 256), dtype=torch.float16)
    N = B._native
    for args in ((d, w, x, x, None), (d, w, None, x, None), (d, None, x, x, None), (None, w, x, x, None), (d, w, x.as_subclass(Sub), x, None),
                 (w, d, x, x, None), (d, w, 3, "y", None), (d, w, x, x), ()):
        assert N.linear_fwd(*args) is None and N.linear_bwd_dx(*args) is None
    for args in ((1, None, None, x, None, None), ("n", b"", b"", x, b"", b""), (1, b"short", b"", x, b"", b""), ()):
        assert N.linear_fwd_group(*args) is None
    assert N.linear_fwd_irregular(d, w, x, x, x, None) is None and N.linear_bwd_dx_irregular(d, w, x, x, x, None) is None
    assert N.weak_grad(d, x, x, x, 1, 0, None) is None and N.linear_bwd(d, w, x, x, x, x, 1, 0, None) is None


def _ways(monkeypatch, call):
    native = call()
    with monkeypatch.context() as m:
        m.setattr(B, "_native", type("None_", (), {n: staticmethod(lambda *a: None) for n in dir(B._native) if not n.startswith("__")}))
        plain = call()
    torch.cuda.synchronize()
    for a, b in zip(native, plain):
        assert torch.equal(a, b) and a.stride() == b.stride()


@pytest.mark.gpu
@pytest.mark.parametrize("oc,ic,k,bits", [(64, 256, 8, 4), (72, 384, 0, 4), (64, 128, 128, 4), (40, 264, 16, 3)])
@pytest.mark.parametrize("m", [0, 1, 3, 40, 100])
def test_native_calls_equal_ctypes(monkeypatch, oc, ic, k, bits, m):
    d = B.make_desc(oc, ic, k, bits, 128)
    w = B.qeft_pack(d, torch.randn((oc, ic), device="cuda").half())
    x, dy = torch.randn((m, ic), device="cuda").half(), torch.randn((m, oc), device="cuda").half()
    perm = torch.randperm(ic, device="cuda").int()
    xw = torch.randn((m, max(k, 8)), device="cuda").half()[:, :k]
    for ws in (None, False):
        _ways(monkeypatch, lambda: [B.qeft_linear_fwd(d, w, x, ws=ws), B.qeft_linear_bwd_dx(d, w, dy, ws=ws)])
    _ways(monkeypatch, lambda: B.qeft_linear_fwd_group([d, d], [w, w], x))
    _ways(monkeypatch, lambda: [B.qeft_linear_fwd_irregular(d, w, perm, x), B.qeft_linear_bwd_dx_irregular(d, w, perm, dy)])
    if k:
        for acc in (False, True):
            _ways(monkeypatch, lambda: [B.qeft_weak_grad(d, dy, xw, accumulate=acc), *B.qeft_linear_bwd(d, w, dy, xw, out_dtype=torch.float16, accumulate=acc)])
    _ways(monkeypatch, lambda: [B.qeft_linear_fwd(d, w, x.as_subclass(Sub))])


@pytest.mark.gpu
def test_native_calls_report_errors_and_keep_to_the_current_stream():
    d = B.make_desc(64, 264, 8, 4, 128)
    w = B.qeft_pack(d, torch.randn((64, 264), device="cuda").half())
    x = torch.randn((4, 264), device="cuda").half()
    for bad, status in ((x[:, 1:], B.QEFT_ERR_SHAPE), (torch.empty((4, 272), device="cuda").half()[:, 4:268], B.QEFT_ERR_ALIGN)):
        with pytest.raises(B.QeftError) as e:
            B.qeft_linear_fwd(d, w, bad, ws=False)
        assert e.value.status in (status, B.QEFT_ERR_ALIGN)
    want, s = B.qeft_linear_fwd(d, w, x, ws=False), torch.cuda.Stream()
    y = torch.zeros((4, 64), dtype=torch.float16, device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):        # (a launch on another stream would not be in it, or break it)
        B.qeft_linear_fwd(d, w, x, y, ws=False)
    torch.cuda.synchronize()
    assert not bool(y.any())
    for _ in range(3):
        y.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want)


def test_the_binding_does_without_the_module():
    code = ("import sys; sys.modules['paper_2410_08661_amd._marshal'] = None\n"
            "from paper_2410_08661_amd import binding as B\n"
            "d = B.make_desc(64, 256, 8, 4, 128)\n"
            "for n in ('linear_fwd', 'linear_fwd_group', 'linear_bwd_dx', 'linear_bwd', 'linear_fwd_irregular', 'linear_bwd_dx_irregular', 'weak_grad'):\n"
            "    assert getattr(B._native, n)(d, None, None) is None\n")
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, cwd=build.ROOT)
    assert r.returncode == 0, r.stderr


def test_a_build_without_a_host_compiler(monkeypatch, tmp_path, capsys):
    old = tmp_path / "_marshal.so"
    old.write_bytes(b"of another torch")
    monkeypatch.setattr(build, "MARSHAL_PATH", str(old))
    monkeypatch.setenv("PATH", str(tmp_path))
    assert build._build_marshal() is False and not old.exists()
    assert "ctypes" in capsys.readouterr().err
