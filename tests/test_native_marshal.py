"""The binding's native part (csrc/marshal.cpp): what it takes gives what the long way gives, and what it declines, or refuses,
is what the long way takes or refuses."""
import ctypes
import os
import shutil
import subprocess
import sys
import warnings

import pytest

torch = pytest.importorskip("torch")          # before the library is loaded: both then use torch's HIP runtime
import paper_2401_10187_amd as km  # noqa: E402
from paper_2401_10187_amd import binding as B  # noqa: E402


def test_mistakes_are_named_without_a_gpu():
    with pytest.raises(ValueError, match="contiguous 2-D CUDA tensor"):
        km.kronmatmul(torch.zeros(2, 4), [torch.zeros(2, 2)] * 2)
    with pytest.raises(ValueError, match="contiguous 2-D CUDA tensor"):
        km.Prepared(torch.zeros(2, 4), [torch.zeros(2, 2)] * 2)
    native = B._start_native()
    assert native.call(torch.zeros(2, 4), [torch.zeros(2, 2)] * 2, None, None, False) is NotImplemented
    assert native.call(None, [], None, None, False) is NotImplemented
    assert native.call(torch.zeros(2, 4), iter(()), None, None, 0) is NotImplemented
    with pytest.raises(TypeError):
        native.call(1, 2)


@pytest.fixture
def no_native(monkeypatch):
    """The binding as it is where the native part cannot be imported."""
    monkeypatch.setattr(B, "_native", None)
    monkeypatch.delattr(km, "_marshal", raising=False)
    monkeypatch.setitem(sys.modules, km.__name__ + "._marshal", None)


def test_without_the_native_part_calls_go_by_ctypes(no_native):
    with pytest.warns(RuntimeWarning, match="native part"), pytest.raises(ValueError, match="contiguous 2-D CUDA tensor"):
        km.kronmatmul(torch.zeros(2, 4), [torch.zeros(2, 2)] * 2)
    with warnings.catch_warnings():                      # said once
        warnings.simplefilter("error")
        with pytest.raises(ValueError, match="contiguous 2-D CUDA tensor"):
            km.kronmatmul(torch.zeros(2, 4), [torch.zeros(2, 2)] * 2)


def test_a_native_part_of_another_torch_is_not_used(monkeypatch):
    native = B._start_native()
    monkeypatch.setattr(B, "_native", None)
    monkeypatch.setattr(native, "built_for", "1.0")
    with pytest.warns(RuntimeWarning, match="built for torch 1.0"):
        assert B._start_native() is not native


def test_the_library_builds_without_the_native_part(monkeypatch, tmp_path, capsys):
    from paper_2401_10187_amd import build
    monkeypatch.setattr(build, "HERE", str(tmp_path))
    monkeypatch.setattr(build, "OBJ", str(tmp_path))
    monkeypatch.setattr(build, "MARSHAL", str(tmp_path / "_marshal.so"))
    (tmp_path / "_marshal.so").write_text("")
    (tmp_path / "marshal.torch").write_text("1.0")
    os.utime(tmp_path / "_marshal.so", (2 ** 32, 2 ** 32))
    assert build._marshal_stale()                        # newer than its source, but of another torch
    (tmp_path / "marshal.torch").write_text(torch.__version__)
    assert not build._marshal_stale()
    monkeypatch.setenv("CXX", str(tmp_path / "no-such-compiler"))
    assert build.build_marshal() is False and "not built" in capsys.readouterr().out
    assert not (tmp_path / "_marshal.so").exists()       # an old one is not left behind


THROWS = """
import ctypes, sys
import torch
import paper_2401_10187_amd as km
from paper_2401_10187_amd import binding as B
entry = ctypes.cast(ctypes.CDLL(sys.argv[1]).entry, ctypes.c_void_p).value
native = B._start_native()
native.start(entry, entry, entry, entry, lambda index: 0, B._raise_status)
try:
    native.bind(1, 1, 0, 0, 0, 0, 0, 0, 0, 0, False, False, 0)(0)
except RuntimeError as e:
    print("raised", e)
"""


def test_an_exception_of_the_library_is_raised(tmp_path):
    """Out of host memory in the planner, for instance: an error like any other, with the interpreter as it was."""
    if not shutil.which("g++"):
        pytest.skip("needs a C++ compiler")
    (tmp_path / "t.cpp").write_text('#include <stdexcept>\nextern "C" int entry(int) { throw std::runtime_error("no memory left"); }\n')
    subprocess.run(["g++", "-shared", "-fPIC", "-o", str(tmp_path / "t.so"), str(tmp_path / "t.cpp")], check=True)
    r = subprocess.run([sys.executable, "-c", THROWS, str(tmp_path / "t.so")], capture_output=True, text=True, timeout=300,
                       cwd=os.path.dirname(B.HERE))
    assert r.returncode == 0 and "raised no memory left" in r.stdout, r.stderr[-2000:]


class Sub(torch.Tensor):
    pass


def _problem(dtype=torch.float32, M=5, shapes=((6, 4), (3, 7))):
    torch.manual_seed(7)
    K = 1
    for p, _ in shapes:
        K *= p
    return torch.randn(M, K, dtype=dtype, device="cuda"), [torch.randn(p, q, dtype=dtype, device="cuda") for p, q in shapes]


def _long_way(X, Fs, **kw):
    """Y of a call that the native part is kept out of: with the stream named."""
    return km.kronmatmul(X, Fs, stream=torch.cuda.current_stream().cuda_stream, **kw)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("transposed", [False, True])
def test_the_same_bits_as_the_long_way(dtype, transposed):
    X, Fs = _problem(dtype)
    given = [F.t().contiguous() for F in Fs] if transposed else Fs
    native = B._native or B._start_native()
    need = km.workspace_size(5, [6, 3], [4, 7], str(dtype), transposed=transposed)
    ws = torch.empty(need + 256, dtype=torch.uint8, device="cuda")
    want = _long_way(X, given, transposed=transposed)
    Y = torch.empty_like(want)
    for args in ((X, given, None, None), (X, tuple(given), None, None), (X, given, Y, None), (X, given, Y, ws), (X, given, None, ws)):
        Y.zero_()
        got = native.call(*args, transposed)
        assert got is not NotImplemented and type(got) is torch.Tensor and not got.requires_grad
        assert (got is Y) == (args[2] is Y) and torch.equal(got, want)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        on_side = km.kronmatmul(X, given, transposed=transposed)
    torch.cuda.current_stream().wait_stream(side)
    assert torch.equal(on_side, want)
    prepared = km.Prepared(X, given, transposed=transposed)
    raw = torch.cuda.current_stream().cuda_stream
    for stream in (None, raw, ctypes.c_void_p(raw)):
        prepared.Y.zero_()
        assert prepared(stream) is prepared.Y and torch.equal(prepared.Y, want)
    leaf = X.clone().requires_grad_()
    assert torch.equal(km.kronmatmul(leaf, given, transposed=transposed), want)


@pytest.mark.gpu
def test_what_is_declined_goes_the_long_way_and_what_is_wrong_is_named():
    X, Fs = _problem()
    native = B._native or B._start_native()
    want = _long_way(X, Fs)
    sub = X.as_subclass(Sub)
    for args in ((sub, Fs), (X, [Fs[0].as_subclass(Sub), Fs[1]]), (X, iter(Fs))):
        if not hasattr(args[1], "__next__"):
            assert native.call(*args, None, None, False) is NotImplemented
        got = km.kronmatmul(*args)
        assert type(got) is torch.Tensor and torch.equal(got, want)
    for bad, match in (((X.t(), Fs), "2-D CUDA"), ((X[:, ::2], Fs), "2-D CUDA"), ((X.half(), [F.half() for F in Fs]), None),
                       ((X, [Fs[0].double(), Fs[1]]), "X's dtype"), ((X, [Fs[0].t(), Fs[1]]), "contiguous"), ((X, Fs[:1]), "columns"),
                       ((X, [Fs[0].cpu(), Fs[1]]), "device"), ((X, Fs, want[:, 1:]), "shape"), ((X, Fs, None, torch.empty(8)), "device")):
        assert native.call(*(bad + (None, None))[:4], False) is NotImplemented
        with pytest.raises((ValueError, TypeError), match=match):
            km.kronmatmul(*bad)
    with pytest.raises(km.KronMatmulError, match="kronmatmul_transposed_ws"):         # too small a workspace
        km.kronmatmul(X, [F.t().contiguous() for F in Fs], workspace=torch.empty(16, dtype=torch.uint8, device="cuda"), transposed=True)
    with pytest.raises(km.KronMatmulError, match="kronmatmul"):
        km.kronmatmul(X, Fs, Y=torch.empty(X.numel() + 200, device="cuda")[1:1 + want.numel()].view(want.shape))
    assert km.kronmatmul(X[:0], Fs).shape == (0, 28)
    with torch.inference_mode():
        assert torch.equal(km.kronmatmul(X, Fs), want)
    with pytest.raises(RuntimeError):                    # a batched tensor of vmap has no memory to point at
        torch.func.vmap(lambda x: km.kronmatmul(x, Fs))(X.view(5, 1, 18))


@pytest.mark.gpu
@pytest.mark.parametrize("transposed", [False, True])
def test_the_same_bits_without_the_native_part(no_native, transposed):
    X, Fs = _problem()
    given = [F.t().contiguous() for F in Fs] if transposed else Fs
    want = _long_way(X, given, transposed=transposed)
    with pytest.warns(RuntimeWarning, match="native part"):
        assert torch.equal(km.kronmatmul(X, given, transposed=transposed), want)
    prepared = km.Prepared(X, given, transposed=transposed)
    for stream in (None, torch.cuda.current_stream().cuda_stream):
        prepared.Y.zero_()
        assert torch.equal(prepared(stream), want)
