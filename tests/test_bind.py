"""The binding's native argument marshalling (_otbind.so): it takes exactly the
arguments that the Python checks take, and leaves every other one to them."""
import os
import shutil
import subprocess
import sys

import pytest
import torch

from paper_2406_18832_amd import build_lib, ot

M, K, N = 5, 48, 33


def _calls(device):
    """(native name, public function, arguments) of each marshalled call."""
    g = torch.Generator().manual_seed(3)
    i8 = lambda *s: torch.randint(-127, 128, s, generator=g, dtype=torch.int8).to(device)
    f32 = lambda *s: (torch.rand(*s, generator=g) * 0.01 + 0.001).to(device)
    f16 = lambda *s: torch.randn(*s, generator=g).half().to(device)
    zW = torch.randint(-9, 9, (N,), generator=g, dtype=torch.int32).to(device)
    q = lambda: torch.empty(M, K, dtype=torch.int8, device=device)
    y = lambda: torch.empty(M, N, dtype=torch.float16, device=device)
    acc = lambda: torch.empty(M, N, dtype=torch.int32, device=device)
    packed = torch.zeros(ot.ot_packed_weights_size(N, K), dtype=torch.int8, device=device)
    ws = torch.empty(64, dtype=torch.uint8, device=device)
    return [
        ("quantize_act", ot.ot_quantize_act, [f16(M, K), 8, f32(K), f32(K), q()]),
        ("quantize_act_per_token", ot.ot_quantize_act_per_token,
         [f16(M, K), 8, q(), torch.empty(M, device=device)]),
        ("ln_quantize_act", ot.ot_ln_quantize_act,
         [f16(M, K), f16(K), f16(K), 1e-5, 8, f32(K), f32(K), q()]),
        ("qlinear", ot.ot_qlinear, [i8(M, K), i8(N, K), f32(N), f32(N), 8, 8, y(), acc(), ws]),
        ("qlinear_noalloc", ot.ot_qlinear_noalloc,
         [i8(M, K), i8(N, K), f32(N), f32(N), 8, 8, y(), acc()]),
        ("qlinear_packed", ot.ot_qlinear_packed,
         [i8(M, K), packed, N, f32(N), f32(N), 8, 8, y(), acc(), ws]),
        ("qlinear_per_token", ot.ot_qlinear_per_token,
         [i8(M, K), i8(N, K), f32(M), f32(N), f32(N), 8, 8, y(), acc(), ws]),
        ("qlinear_asym", ot.ot_qlinear_asym,
         [i8(M, K), i8(N, K), f32(N), zW, f32(N), 8, 8, y(), acc(), ws]),
    ]


NAMES = [n for n in ot._BOUND]


def _entry(name, device):
    return next(c for c in _calls(device) if c[0] == name)


def _wrong_arguments(args):
    """Each argument in turn replaced by ones the call does not take as it is."""
    for i, a in enumerate(args):
        wrong = ["text", None, 3.0 if isinstance(a, int) else 3]
        if isinstance(a, torch.Tensor):
            other = torch.int16 if a.dtype != torch.int16 else torch.int8
            wrong += [a.to(other), a.reshape(-1)[:-1], a.unsqueeze(0)]
            if a.dim() == 2:
                wrong += [a.t(), torch.cat([a, a], 1)[:, ::2], a.new_empty(a.shape[0], a.shape[1] + 16)]
            if a.is_cuda:
                wrong.append(a.cpu())
        for w in wrong:
            yield i, w, args[:i] + [w] + args[i + 1:]


@pytest.mark.parametrize("name", NAMES)
def test_host_tensors_are_left_to_the_python_checks(name):
    ot.lib()
    _, call, args = _entry(name, "cpu")
    assert getattr(ot, "_n_" + name)(*args, None) is None
    with pytest.raises(ValueError, match="must be on the GPU"):
        call(*args)
    for _, _, wrong in _wrong_arguments(args):
        assert getattr(ot, "_n_" + name)(*wrong, None) is None
    assert getattr(ot, "_n_" + name)(*args) is None  # too few arguments
    assert getattr(ot, "_n_" + name)() is None


def _outcome(call, args):
    try:
        call(*args)
    except Exception as e:
        return type(e).__name__, str(e)
    torch.cuda.synchronize()
    return [a.cpu().clone() if isinstance(a, torch.Tensor) else a for a in args]


def _same(a, b):
    if isinstance(a, tuple) or isinstance(b, tuple):
        return a == b
    return all(torch.equal(x, y) if isinstance(x, torch.Tensor) else x == y or x is y
               for x, y in zip(a, b))


@pytest.mark.gpu
@pytest.mark.parametrize("name", NAMES)
def test_native_and_python_marshalling_agree(name, monkeypatch):
    """The same results from the same arguments, and the same error (or
    conversion) for every argument that is not as expected."""
    print(f"[case] binding {name}", flush=True)
    ot.lib()
    _, call, args = _entry(name, "cuda")
    native = getattr(ot, "_n_" + name)
    cases = [args, args[:]]
    if name.startswith("qlinear"):
        cases.append(args[:-1] + [None])
    # wrong arguments that both sides refuse (a call that would read other
    # sizes than its buffers hold is refused by its shape checks)
    refused = [w for i, v, w in _wrong_arguments(args)]
    ran = native(*args, ot._stream(None))
    assert ran == ot.OT_OK
    torch.cuda.synchronize()
    first = [(_outcome(call, c)) for c in cases + refused]
    monkeypatch.setattr(ot, "_n_" + name, ot._unbound)
    second = [(_outcome(call, c)) for c in cases + refused]
    for i, (a, b) in enumerate(zip(first, second)):
        assert _same(a, b), (i, a, b)
    assert not isinstance(first[0], tuple)


@pytest.mark.gpu
def test_streams_and_statuses_pass_through():
    print("[case] binding streams", flush=True)
    ot.lib()
    _, call, args = _entry("qlinear", "cuda")
    want = _outcome(call, args)
    st = torch.cuda.Stream()
    for stream in (st, st.cuda_stream, None):
        args[6].zero_()
        torch.cuda.synchronize()
        call(*args, stream=stream)
        torch.cuda.synchronize()
        assert torch.equal(args[6].cpu(), want[6])
    with torch.cuda.stream(st):
        call(*args)
    torch.cuda.synchronize()
    with pytest.raises(ot.OTError) as e:
        call(*args[:4], 9, *args[5:])
    assert e.value.code == ot.OT_EINVAL
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(*args)
    for _ in range(3):
        args[6].zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(args[6].cpu(), want[6])


class _Wrapper(torch.Tensor):
    """A wrapper subclass that answers for its own layout, with an error."""

    @staticmethod
    def __new__(cls, *shape):
        return torch.Tensor._make_wrapper_subclass(
            cls, shape, dtype=torch.float16, device="cuda", dispatch_sizes_strides_policy="strides")

    @classmethod
    def __torch_dispatch__(cls, func, types, args=(), kwargs=None):
        raise LookupError(f"this tensor has no {func}")


def test_an_error_raised_by_a_tensor_is_the_callers():
    """A tensor that raises from Python while it is looked at: its own error
    reaches the caller, and none is left behind by the native checks."""
    ot.lib()
    x = _Wrapper(M, K)
    with pytest.raises(LookupError, match="this tensor has no"):
        x.is_contiguous()
    _, call, args = _entry("quantize_act", "cpu")
    assert ot._n_quantize_act(x, *args[1:], 0) is None
    with pytest.raises(LookupError, match="this tensor has no"):
        call(x, *args[1:])


_LIAR = """
import sys, types
sys.path.insert(0, {root!r})
import torch
from paper_2406_18832_amd import ot

class Liar:
    __class__ = torch.Tensor      # what unittest.mock's specced objects do

class Own(torch.Tensor):          # answers for itself, as a plain tensor's methods do not
    @classmethod
    def __torch_function__(cls, func, types, args=(), kwargs=None):
        raise LookupError("its own answer")

ot.lib()
args = [8, torch.zeros(48), torch.zeros(48), torch.zeros(5, 48, dtype=torch.int8)]
assert isinstance(Liar(), torch.Tensor)
assert ot._n_quantize_act(Liar(), *args, 0) is None
x = torch.zeros(5, 48, dtype=torch.float16).as_subclass(Own)
assert ot._n_quantize_act(x, *args, 0) is None
try:
    ot.ot_quantize_act(x, *args)
except LookupError as e:
    print("passed", e)
"""


def test_only_plain_tensors_are_taken_natively():
    """An object that only claims to be a tensor has none of a tensor's memory
    to look at, and a subclass may answer for itself: both are left to the
    Python checks (in a process of its own: reading the first is undefined)."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    run = subprocess.run([sys.executable, "-c", _LIAR.format(root=root)], capture_output=True,
                         text=True, timeout=300)
    assert run.returncode == 0 and "passed its own answer" in run.stdout, (run.returncode, run.stdout,
                                                                         run.stderr[-2000:])


_BARE = """
import sys, warnings
sys.path.insert(0, {root!r})
import torch
from paper_2406_18832_amd import ot

with warnings.catch_warnings(record=True) as seen:
    warnings.simplefilter("always")
    assert ot.ot_abi_version() == 1
print([str(w.message) for w in seen])
assert ot.HERE.startswith({root!r}) and ot._n_qlinear is ot._unbound
try:
    ot.ot_quantize_act(torch.zeros(5, 48, dtype=torch.float16), 8, torch.zeros(48), torch.zeros(48),
                       torch.zeros(5, 48, dtype=torch.int8))
except ValueError as e:
    print("passed", e)
"""


def _package_copy(tmp_path):
    """The package's Python files alone in a folder of their own."""
    pkg = tmp_path / "paper_2406_18832_amd"
    shutil.copytree(ot.HERE, pkg, ignore=lambda d, names: [n for n in names if n == "csrc" or
                                                           not n.endswith(".py")])
    return pkg


def _run(code, lib):
    return subprocess.run([sys.executable, "-c", code], env=dict(os.environ, OT_LIBRARY=lib),
                          capture_output=True, text=True, timeout=300)


def test_a_library_without_the_binding_is_enough(tmp_path):
    """libot.so alone serves every call, through the Python checks."""
    _package_copy(tmp_path)
    run = _run(_BARE.format(root=str(tmp_path)), os.path.abspath(ot.LIB_PATH))
    assert run.returncode == 0 and "passed x must be on the GPU" in run.stdout, run.stderr[-2000:]
    assert "arguments are checked in Python" in run.stdout


def test_a_binding_of_another_header_is_not_called(tmp_path):
    """The binding casts the library's addresses to the signatures it was
    compiled with: one of another ot.h stays unbound.  (A copy of the tree's
    binding whose recorded digest is another.)"""
    from paper_2406_18832_amd import _otbind
    assert ot.build_info()["binding_matches_sources"]
    pkg = _package_copy(tmp_path)
    with open(_otbind.__file__, "rb") as f:
        data = f.read()
    digest = build_lib.header_digest().encode()
    assert data.count(digest) == 1 and _otbind.header_sha256.encode() == digest
    (pkg / "_otbind.so").write_bytes(data.replace(digest, b"0" * 64))
    run = _run(_BARE.format(root=str(tmp_path)), os.path.abspath(ot.LIB_PATH))
    assert run.returncode == 0 and "passed x must be on the GPU" in run.stdout, run.stderr[-2000:]
    assert "another include/ot.h" in run.stdout


def test_one_build_makes_library_and_binding(monkeypatch, tmp_path):
    ran = []

    def compiler(cmd, **kw):
        ran.append(cmd)
        return subprocess.CompletedProcess(cmd, 0, "", "")
    monkeypatch.setattr(build_lib.subprocess, "run", compiler)
    monkeypatch.setattr(build_lib.os, "replace", lambda a, b: None)
    build_lib.build()
    assert [c[-1] for c in ran] == [build_lib.LIB + ".tmp", build_lib.BIND + ".tmp"]
    del ran[:]
    build_lib.build(out=str(tmp_path / "libot.so"))  # a build of its own leaves the tree's binding
    assert [c[-1] for c in ran] == [str(tmp_path / "libot.so") + ".tmp"]
