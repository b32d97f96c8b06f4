"""The 256-row GEMM at ragged sizes, in each of its forms, for every width and
number of groups in a 128-row chunk: stream-K (partial tiles parked and summed
by a second launch), whole tiles, whole-tile rounds followed by stream-K or by
the 64 x 128 tiles; the stream-K forms also under graph replay and sharing one
workspace with split GEMVs.

Tolerances: the rounded-weight bound of the other tiled kernels."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2606_11357_amd.synth import make_inputs

from test_gpu_gemm_kq import _run
from test_gpu_parity import assert_parity, dev, pack, tf  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SK, WHOLE = ", stream-K,", "whole tiles"
HYBRID, REST = "hybrid (whole-tile rounds, then stream-K)", "then the K-split GEMM"
SHAPES = ([(b, 2000, 14336, 2056, g, SK) for b in (4, 8) for g in (128, 64, 32)] +
          [(b, 500, 512, 8200, g, WHOLE) for b in (4, 8) for g in (128, 64, 32)] +
          [(4, 2040, 1024, 12296, 32, HYBRID), (8, 2040, 1024, 12296, 128, HYBRID), (4, 1300, 512, 12296, 64, REST)])


@pytest.mark.parametrize("bf", [False, True], ids=["f16", "bf16"])
@pytest.mark.parametrize("bits,M,K,N,G,form", SHAPES)
def test_against_oracle(tf, bits, M, K, N, G, form, bf):
    got, want = _run(tf, bf, bits, M, K, N, G, None)
    scale = np.abs(want).max()
    bound = (2.0 ** -8 if bf else 2.0 ** -11) * np.abs(want) + (4e-3 if bf else 1e-3) * scale
    assert np.all(np.isfinite(got))
    assert np.all(np.abs(got - want) <= bound), np.abs(got - want).max() / scale


def test_stream_k_shared_workspace_and_graph(tf):
    """Stream-K GEMMs and split GEMVs in turn on one workspace, eager and replayed."""
    cases = [("gemm", 4, 2000, 14336, 2056, 64), ("gemv", 4, 1, 14336, 4096, 128), ("gemm", 8, 2000, 14336, 2056, 32),
             ("gemv", 8, 3, 8192, 520, 128), ("gemm", 8, 2040, 1024, 12296, 128), ("gemm", 4, 2000, 14336, 2056, 64)]
    ws = torch.zeros(max(tf.workspace_bytes(b, m, k, n, g) for _, b, m, k, n, g in cases), dtype=torch.uint8,
                     device="cuda")
    calls, eager = [], []
    for i, (kind, bits, M, K, N, G) in enumerate(cases):
        d = make_inputs(bits, M, K, N, group=G, seed=400 + i)
        fn, x, p = getattr(tf, f"w{bits}a16_{kind}"), dev(d["x"]), pack(tf, d)
        out = torch.empty((M, N), dtype=torch.float16, device="cuda")
        calls.append((fn, x, p, K, N, G, out))
        rows = [0, 1, M // 2, M - 1] if M > 8 else list(range(M))
        fn(x, p, K, N, G, out=out, workspace=ws)
        torch.cuda.synchronize()
        want = oracle.matmul(d["x"][rows], oracle.dequant(d["q"], d["z"], d["s"], G))
        assert_parity(out.cpu().numpy()[rows], want, f"shared workspace, case {i}: {kind} W{bits} {M}x{K}x{N}")
        eager.append(out.clone())

    def run_all():
        for fn, x, p, K, N, G, out in calls:
            fn(x, p, K, N, G, out=out, workspace=ws)

    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        run_all()
    for rep in range(3):
        for *_, out in calls:
            out.zero_()                       # eager work between replays
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for i, (e, (*_, out)) in enumerate(zip(eager, calls)):
            assert torch.equal(out.view(torch.int16), e.view(torch.int16)), f"replay {rep}, case {i}"
