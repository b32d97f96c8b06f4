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
