"""The GEMM with 64 x 64 and 128 x 128 tiles (any K and group, K split over the
workgroup's waves and, with a workspace, over workgroups) against the CPU
oracle, at the sizes where its plan changes or its loops end: one 32-row step,
odd step counts (a last half pair), fewer steps than waves, groups that open at
every place of the unrolled loop, ragged tile edges, and each K split.

Tolerances: the output's own rounding (half a unit in the last place, 2^-11 of
the element in fp16, 2^-8 in bf16) plus 1e-3 (bf16: 4e-3) of the largest
output: the kernel rounds each weight once (the rounded-weight bound the other
GEMMs' tests use), one dropped row of K would show as about 1 / sqrt(K)."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2606_11357_amd.synth import make_inputs, make_inputs_bf16

from test_gpu_parity import GUARD, dev, pack, tf  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (bits, M, K, N, group): M >= 33 keeps the streaming kernel out
SHAPES = [
    (4, 33, 32, 8, 32),           # one step: seven of the eight waves idle
    (8, 64, 96, 72, 96),          # three steps, a group that is no power of two
    (8, 65, 96, 72, 96),          # ... on the tiles (64 rows of 8-bit weights with short K stream)
    (4, 65, 160, 136, 32),        # a group a step, two row tiles, ragged columns
    (8, 129, 1376, 264, 32),      # 43 steps: a last half pair, and runs of 4 and 6 steps
    (4, 200, 1344, 520, 192),     # groups of six steps against pairs
    (8, 40, 2080, 520, 160),      # 65 steps, groups of five steps
    (4, 1000, 2080, 4104, 32),    # 128 x 128 tiles (one round), 17-step quarters
    (8, 700, 4000, 4360, 160),    # ... odd steps, groups of five
    (4, 300, 384, 4104, 384),     # 128-row chunks, a group of three chunks, fewer chunks than waves
    (4, 49, 4096, 1032, 128),     # whole chunks, 64 x 64 tiles, K in two slices
    (8, 64, 14336, 264, 256),     # ... and more, groups of two chunks
    (4, 200, 14336, 1032, 128),   # 128-row promise of workspace, K split
    (4, 520, 14336, 2056, 128),   # 128 x 128 tiles, K split (with a workspace)
]


def _run(tf, bf, bits, M, K, N, G, workspace):
    if bf:
        d = make_inputs_bf16(bits, M, K, N, group=G, seed=K + N + M)
        s = dev(d["s_bits"].view(np.int16))
        p = (tf.pack_w4(dev(d["qweight"]), dev(d["qzeros"]), s, K, N, G) if bits == 4
             else tf.pack_w8(dev(d["qweight"]), dev(d["zeros"]), s, K, N, G))
        x, dt = dev(d["x_bits"].view(np.int16)).view(torch.bfloat16), torch.bfloat16
        want = (oracle.w4a16_bf16 if bits == 4 else oracle.w8a16_bf16)(
            d["x_bits"], d["qweight"], d["qzeros"] if bits == 4 else d["zeros"], d["s_bits"], G)
    else:
        d = make_inputs(bits, M, K, N, group=G, seed=K + N + M)
        p, x, dt = pack(tf, d), dev(d["x"]), torch.float16
        want = oracle.matmul(d["x"], oracle.dequant(d["q"], d["z"], d["s"], G))
    buf = torch.full((M * N + 2 * GUARD,), -7.0, dtype=dt, device="cuda")
    out = buf[GUARD:GUARD + M * N].view(M, N)
    fn = getattr(tf, f"w{bits}a16_gemm")
    fn(x, p, K, N, G, out=out, workspace=workspace)
    torch.cuda.synchronize()
    guard = torch.cat([buf[:GUARD], buf[-GUARD:]]).float().cpu().numpy()
    assert np.all(guard == -7.0), "write outside the output"
    first = out.clone()
    fn(x, p, K, N, G, out=out, workspace=workspace)
    torch.cuda.synchronize()
    assert torch.equal(first.view(torch.int16), out.view(torch.int16)), "not reproducible"
    return out.float().cpu().numpy().astype(np.float64), want


@pytest.mark.parametrize("bf", [False, True], ids=["f16", "bf16"])
@pytest.mark.parametrize("ws", [None, False], ids=["workspace", "none"])
@pytest.mark.parametrize("bits,M,K,N,G", SHAPES)
def test_against_oracle(tf, bits, M, K, N, G, ws, bf):
    got, want = _run(tf, bf, bits, M, K, N, G, ws)
    scale = np.abs(want).max()
    bound = (2.0 ** -8 if bf else 2.0 ** -11) * np.abs(want) + (4e-3 if bf else 1e-3) * scale
    assert np.all(np.isfinite(got))
    assert np.all(np.abs(got - want) <= bound), np.abs(got - want).max() / scale


def test_non_finite_rows_stay_apart(tf):
    """An infinity or NaN in one row of A reaches that row only, as the plain
    product has it (no step past a wave's run enters a sum)."""
    bits, M, K, N, G = 4, 65, 1376, 136, 32
    d = make_inputs(bits, M, K, N, group=G, seed=5)
    x = d["x"].copy()
    x[3, K - 1] = np.inf
    x[64, 40] = np.nan
    out = tf.w4a16_gemm(dev(x), pack(tf, d), K, N, G)
    torch.cuda.synchronize()
    got = out.cpu().numpy().astype(np.float64)
    w = oracle.dequant(d["q"], d["z"], d["s"], G)
    last = w[K - 1]
    want3 = np.where(last > 0, np.inf, np.where(last < 0, -np.inf, np.nan))
    np.testing.assert_array_equal(got[3], want3)
    assert np.all(np.isnan(got[64]))
    rest = [r for r in range(M) if r not in (3, 64)]
    assert np.all(np.isfinite(got[rest]))
