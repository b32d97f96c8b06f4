"""The streaming matrix-core form (GEMM entry, 4 to 32 rows) where a wave's run
is one whole round (K just up to 2048: every atom requested at the start) and
just beside it (shorter and longer runs keep the ring), against the oracle:
the last wave's run one atom short, one atom long, and whole.  The factored
form rounds no weight: the bound is the output's rounding (2^-11) and 1e-3 of
the largest output, as for the other kernels."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2606_11357_amd.synth import make_inputs

from test_gpu_parity import dev, pack, tf  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("M,K,N,G", [(4, 2048, 264, 128), (16, 2016, 136, 32), (17, 2048, 520, 128), (32, 2048, 72, 64),
                                     (32, 1824, 264, 32), (9, 2080, 136, 32), (20, 1792, 264, 128)])
def test_one_round(tf, bits, M, K, N, G):
    d = make_inputs(bits, M, K, N, group=G, seed=M + K + N)
    fn = tf.w4a16_gemm if bits == 4 else tf.w8a16_gemm
    p, x = pack(tf, d), dev(d["x"])
    got = fn(x, p, K, N, G).cpu().numpy().astype(np.float64)
    want = oracle.matmul(d["x"], oracle.dequant(d["q"], d["z"], d["s"], G))
    assert np.all(np.abs(got - want) <= 2.0 ** -11 * np.abs(want) + 1e-3 * np.abs(want).max())
    np.testing.assert_array_equal(fn(x, p, K, N, G).cpu().numpy(), got.astype(np.float16))
