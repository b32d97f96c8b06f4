"""Which kernel and form a call takes, read from the plan log (CPU only).

The calls run in a child process that sees no GPU: each passes the argument
checks, logs its plan for 256 compute units and then fails at the launch, so
the operands' addresses are never used."""
from __future__ import annotations

import json
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = r"""
import ctypes, json, sys
hip = ctypes.CDLL("libamdhip64.so")
n = ctypes.c_int(0)
if hip.hipGetDeviceCount(ctypes.byref(n)) == 0 and n.value > 0:
    sys.exit("a GPU is visible: the calls below must not reach one")
from paper_2606_11357_amd import tilefuse as tf
lib = tf.load()
P = ctypes.c_void_p(0x10000)
for kind, bits, bf, M, K, N, G, ws in json.load(sys.stdin):
    need = lib.tf_workspace_bytes(bits, M, K, N, G)
    assert need >= 0
    f = getattr(lib, f"tf_w{bits}a16_{kind}" + ("_bf16" if bf else ""))
    print("call", file=sys.stderr, flush=True)
    assert f(P, P, P, M, K, N, G, P if ws and need else None, need if ws else 0, None) == tf.TF_ERR_HIP
"""


def plans(calls):
    """The plan of each (kind, bits, bf, M, K, N, group, workspace) call."""
    import torch
    env = dict(os.environ, TF_LOG="1", HIP_VISIBLE_DEVICES="-1", ROCR_VISIBLE_DEVICES="-1",
               LD_LIBRARY_PATH=os.pathsep.join([os.path.join(os.path.dirname(torch.__file__), "lib"),
                                                "/opt/rocm/lib", os.environ.get("LD_LIBRARY_PATH", "")]))
    r = subprocess.run([sys.executable, "-c", CHILD], cwd=ROOT, env=env, input=json.dumps(calls), text=True,
                       capture_output=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    got = [part.split("[tilefuse] ")[1].splitlines()[0] for part in r.stderr.split("call\n")[1:]]
    assert len(got) == len(calls)
    return got


def _skip_with_gpu():
    import torch
    if torch.cuda.is_available():
        pytest.skip("runs where no GPU is visible")


def test_one_round_streaming():
    """The streaming matrix-core form requests a whole run at the start only
    where that measured faster: not for few workgroups with small groups."""
    _skip_with_gpu()
    want = [(4, 16, 2048, 2048, 128, True), (4, 16, 2048, 2048, 32, False), (4, 32, 1824, 16384, 32, False),
            (4, 32, 16384, 2048, 32, False), (4, 16, 2048, 264, 256, True), (4, 16, 1856, 1024, 64, False),
            (4, 16, 2048, 11008, 64, True), (8, 16, 2048, 2048, 64, True), (8, 32, 1824, 1024, 32, False),
            (8, 16, 1824, 11008, 32, True), (8, 16, 1024, 2048, 128, False)]
    got = plans([("gemm", bits, False, M, K, N, G, True) for bits, M, K, N, G, _ in want])
    for (bits, M, K, N, G, one), line in zip(want, got):
        assert line.startswith(f"gemv_kernel<{bits},{16 if M <= 16 else 32},8,"), line
        assert ("one-round" in line) == one, line


def _kernel(line):
    return line.split(" M=")[0].split(" rows=")[0]


def test_short_k():
    """Calls whose few steps a pipelined kernel cannot fill run the 128 x 128
    kernel without one (both types: the second of each pair is bf16)."""
    _skip_with_gpu()
    from test_gpu_short_k import ANY_SHAPES
    calls = [("gemm", b, bf, M, K, N, G, ws) for b, M, K, N, G in ANY_SHAPES + [(8, 2322, 576, 15560, 64), (4, 2547, 864, 14776, 96)]
             for bf in (False, True) for ws in (True, False)]
    for c, line in zip(calls, plans(calls)):
        assert _kernel(line) == f"gemm_any_kernel<{c[1]},{'bf16' if c[2] else 'f16'}>", line


def test_short_k_few_rows():
    """33 to 64 rows of 8-bit weights stay on the streaming kernel where it ends
    before the tiled one has started: short K, sooner with more than 48 rows and
    where the rows of A start on cache lines, and only in one round of panels."""
    _skip_with_gpu()
    from test_gpu_short_k import STREAM64_SHAPES
    want = [(c, True) for c in STREAM64_SHAPES + [(8, 48, 1888, 600, 32), (8, 64, 1056, 600, 32), (8, 48, 1024, 600, 64)]]
    want += [(c, False) for c in [(8, 48, 1920, 600, 32), (8, 64, 1120, 600, 32), (8, 48, 768, 600, 128),
                                  (8, 64, 448, 600, 64), (8, 48, 480, 8200, 32), (8, 65, 480, 600, 32),
                                  (4, 48, 480, 600, 32)]]
    calls = [("gemm", b, bf, M, K, N, G, ws) for (b, M, K, N, G), _ in want for bf in (False, True) for ws in (True, False)]
    stays = [stay for _, stay in want for _ in range(4)]
    for c, stay, line in zip(calls, stays, plans(calls)):
        assert line.startswith("gemv_kernel<8,64," if stay else ("gemm_kq_kernel<", "gemm_any_kernel<")), line


def test_tiled_choice():
    """The expected times know the width, the type, what the tiles load and how
    much of the chip works: each of these calls once took a kernel that was 6 to
    39% slower (measured) than the one named."""
    _skip_with_gpu()
    want = [((4, False, 2176, 9984, 944, 128), "gemm_kq_kernel<4,f16,8,8,"),     # 67 us, 64 x 64 tiles 99
            ((8, True, 964, 14336, 4096, 64), "gemm256_kernel<8,2,bf16>"),        # 113, 128 x 128 tiles 124
            ((8, True, 200, 32768, 8192, 128), "gemm_ks_kernel<8,1,bf16,128>"),   # 176, 64 x 64 tiles 187
            ((8, False, 200, 32768, 8192, 128), "gemm_ks_kernel<8,1,f16,128>"),   # 149, 64 x 64 tiles 180
            ((4, False, 512, 8320, 4096, 128), "gemm_ks_kernel<4,1,f16,128>"),    # 38, 128 x 128 tiles 42
            ((4, False, 512, 8192, 4096, 128), "gemm_ks_kernel<4,1,f16,128>")]    # no step between the two
    for (c, name), line in zip(want, plans([("gemm", *c, True) for c, _ in want])):
        assert line.startswith(name), line


def test_kernels_of_the_gpu_tests():
    """The shapes of the GPU tests that are named for a kernel run that kernel:
    the GEMMs of middle sizes, the K-split GEMM's tiles, and each form of the
    256-row GEMM for every width and number of groups in a chunk."""
    _skip_with_gpu()
    import test_gpu_gemm256 as big
    import test_gpu_gemm_kq as kq
    import test_gpu_gemm_ks as ks
    # 64 rows of 8-bit weights with three steps now stream; long K without a
    # workspace takes the tiles that need none
    calls = [("gemm", b, bf, M, K, N, G, ws) for b, M, K, N, G in kq.SHAPES for bf in (False, True) for ws in (True, False)
             if (b, M, K) != (8, 64, 96) and (ws or M != 520)]
    for c, line in zip(calls, plans(calls)):
        assert line.startswith(f"gemm_kq_kernel<{c[1]},"), line
    calls = [("gemm", b, bf, M, K, N, G, ws) for b, M, K, N, G, _ in ks.SHAPES for bf in (False, True) for ws in (True, False)]
    tiles = [t for *_, t in ks.SHAPES for _ in range(4)]
    for c, t, line in zip(calls, tiles, plans(calls)):
        assert line.startswith(f"gemm_ks_kernel<{c[1]},{128 // c[6]},") and t in line, line
    calls = [("gemm", b, bf, M, K, N, G, True) for b, M, K, N, G, _ in big.SHAPES for bf in (False, True)]
    forms = [form for *_, form in big.SHAPES for _ in range(2)]
    seen = set()
    for c, form, line in zip(calls, forms, plans(calls)):
        groups = 128 // min(c[6], 128)
        assert line.startswith(f"gemm256_kernel<{c[1]},{groups},{'bf16' if c[2] else 'f16'}>"), line
        assert form in line, line
        seen.add((c[1], groups, form))
    assert {(b, g, f) for b in (4, 8) for g in (1, 2, 4) for f in (", stream-K,", "whole tiles")} <= seen
