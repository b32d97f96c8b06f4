"""The native half of the Python binding against the general path it stands
for: the same output tensors and bits in every accepted form, the same
exception for every refused one (a form that the native call does not take
comes back and runs through the general path)."""
from __future__ import annotations

import os
import subprocess
import sys

import pytest

torch = pytest.importorskip("torch")

from paper_2606_11357_amd import build as B  # noqa: E402
from paper_2606_11357_amd import tilefuse as T  # noqa: E402

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

K, N = 4096, 1024      # 64 rows or fewer split K through a workspace


def _raised(f, *a, **kw):
    try:
        f(*a, **kw)
    except Exception as e:   # noqa: BLE001
        return type(e), str(e)
    return None


def _cpu(*shape, dtype=torch.float16):
    return torch.zeros(shape, dtype=dtype)


def _refusals(x, packed):
    """(A, packed, K, N, group, out, workspace) the binding refuses."""
    half = x.dtype
    dev = x.device
    return [
        (x.float(), packed, K, N, 128, None, None),
        (x[0], packed, K, N, 128, None, None),
        (x, packed, K - 128, N, 128, None, None),
        (x.t().contiguous().t(), packed, K, N, 128, None, None),
        (x, packed, K, N, 128, torch.empty((1, N), dtype=half, device=dev), None),
        (x, packed, K, N, 128, torch.empty((x.shape[0], N), dtype=torch.float32, device=dev), None),
        (x, packed, K, N, 100, None, None),
        (x, packed, K, N + 4, 128, None, None),
        (x, packed, K, N, 2 ** 40, None, False),
        (x, packed, float(K), N, 128, None, None),
        (x, packed, K, N, 128, None, torch.zeros(16, dtype=torch.uint8)),
        (x, None, K, N, 128, None, False),
        (x[:0], packed, K, N, 128, None, False),
        (_ragged(x), packed, K, N, 128, None, None),
        (x, packed, K, N, 128, _ragged(x), None),
    ]


def _ragged(x):
    """A nested tensor (exactly torch.Tensor, strided) whose rows differ in
    length: asking it for its second size raises."""
    return torch.nested.nested_tensor([torch.zeros(K, dtype=x.dtype), torch.zeros(K // 2, dtype=x.dtype)],
                                      device=x.device)


def test_cpu_tensors_are_refused_alike():
    x, packed = _cpu(4, K), _cpu(1024, dtype=torch.uint8)
    for args in _refusals(x, packed) + [(x, packed, K, N, 128, None, None)]:
        got = _raised(T._matmul, 4, "gemm", *args)
        assert got is not None and got == _raised(T._matmul_general, 4, "gemm", *args)


def test_no_exception_leaves_the_native_call(tmp_path, monkeypatch):
    """The native call's own source, built without its test for the device, on
    CPU tensors whose sizes raise when asked for: they come back as
    NotImplemented (an exception that left the C entry would end the process)."""
    with open(B.BINDING_SRC) as f:
        text = f.read()
    assert text.count("t.is_cuda() && ") == 1
    src = tmp_path / "tf_binding.cpp"
    src.write_text(text.replace("t.is_cuda() && ", ""))
    monkeypatch.setattr(B, "BINDING_SRC", str(src))
    monkeypatch.setattr(B, "BINDING", str(tmp_path / "_tf_binding.so"))
    B.build_binding()
    script = """
import sys; sys.path.insert(0, %r)
import torch, _tf_binding as native
from test_binding_native import _ragged, K, N
native.bind((1,) * 8, 1, None, {}, None)      # addresses that no call below reaches
x, packed = torch.zeros(2, K, dtype=torch.float16), torch.zeros(64, dtype=torch.uint8)
r = _ragged(x)
for args in ((r, packed, K, N, 128, None, False), (x, packed, K, N, 128, r, False)):
    assert native.matmul(4, False, *args) is NotImplemented
print("done")
""" % str(tmp_path)
    env = dict(os.environ, PYTHONPATH=os.pathsep.join([ROOT, os.path.join(ROOT, "tests")]))
    r = subprocess.run([sys.executable, "-c", script], cwd=ROOT, env=env, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "done" in r.stdout, r.stderr[-3000:]


def _without_native(monkeypatch):
    """As if the native module were not built."""
    monkeypatch.setitem(sys.modules, f"{T.__package__}._tf_binding", None)
    monkeypatch.delattr(sys.modules[T.__package__], "_tf_binding", raising=False)
    monkeypatch.setattr(T, "_bound", None)


def test_without_the_native_module_calls_take_the_general_path(monkeypatch):
    _without_native(monkeypatch)
    x, packed = _cpu(4, K), _cpu(1024, dtype=torch.uint8)
    with pytest.warns(RuntimeWarning, match="native binding"):
        got = _raised(T.w4a16_gemm, x, packed, K, N)
    assert got == _raised(T._matmul_general, 4, "gemm", x, packed, K, N, 128, None, None)
    assert got[0] is ValueError


@pytest.mark.gpu
def test_without_the_native_module_results_are_the_same(monkeypatch):
    gen = torch.Generator(device="cuda").manual_seed(2)
    q, z = (torch.randint(0, 256, (rows, N), dtype=torch.uint8, device="cuda", generator=gen) for rows in (K, K // 128))
    s = (0.001 * torch.rand((K // 128, N), device="cuda", generator=gen)).half()
    packed = T.pack_w8(q, z, s, K, N)
    x = torch.randn((3, K), device="cuda", generator=gen).half()
    want = T.w8a16_gemv(x, packed, K, N)
    _without_native(monkeypatch)
    with pytest.warns(RuntimeWarning, match="native binding"):
        got = T.w8a16_gemv(x, packed, K, N)
    assert torch.equal(got, want)


@pytest.mark.gpu
@pytest.mark.parametrize("dt", [torch.float16, torch.bfloat16], ids=["f16", "bf16"])
def test_forms_match_the_general_path(dt):
    gen = torch.Generator(device="cuda").manual_seed(1)
    words = lambda rows: torch.randint(-2 ** 31, 2 ** 31, (rows, N // 8), dtype=torch.int32, device="cuda",  # noqa: E731
                                       generator=gen)
    s = (0.01 * torch.rand((K // 128, N), device="cuda", generator=gen)).to(dt)
    packed = T.pack_w4(words(K), words(K // 128), s, K, N)
    for M, kind in ((1, "gemv"), (8, "gemv"), (16, "gemm"), (40, "gemm"), (300, "gemm")):
        x = torch.randn((M, K), device="cuda", generator=gen).to(dt)
        own = torch.zeros(max(256, T.workspace_bytes(4, M, K, N)), dtype=torch.uint8, device="cuda")
        for ws in (None, False, own):
            want = T._matmul_general(4, kind, x, packed, K, N, 128, None, ws)
            got = T._matmul(4, kind, x, packed, K, N, 128, None, ws)
            out = torch.empty_like(want)
            assert T._matmul(4, kind, x, packed, K, N, 128, out, ws) is out
            side = torch.cuda.Stream()
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):
                there = T._matmul(4, kind, x, packed, K, N, 128, None, own)
            torch.cuda.current_stream().wait_stream(side)
            torch.cuda.synchronize()
            assert got.dtype == dt and got.shape == (M, N) and not got.requires_grad
            assert torch.equal(got, want) and torch.equal(out, want)
            if ws is own:
                assert torch.equal(there, want)
        for args in _refusals(x, packed):
            got = _raised(T._matmul, 4, kind, *args)
            assert got == _raised(T._matmul_general, 4, kind, *args), args[2:5]
    # a workspace smaller than the call needs is refused by the library
    need = T.workspace_bytes(4, 40, K, N)
    small = torch.zeros(need - 16, dtype=torch.uint8, device="cuda")
    x = torch.zeros((40, K), dtype=dt, device="cuda")
    with pytest.raises(T.TileFuseError):
        T._matmul(4, "gemm", x, packed, K, N, 128, None, small)
