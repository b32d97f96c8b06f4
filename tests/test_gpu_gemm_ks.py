"""The GEMM with 64 x 128 and (4-bit) 64 x 256 tiles and K split over the
workgroup's waves, against the CPU oracle for every width and number of groups in
a 128-row chunk: row tiles with one row, columns past N, and chunks (5, 13, 17)
that the four waves share unevenly.

Tolerances: the rounded-weight bound of the other tiled kernels."""
from __future__ import annotations

import numpy as np
import pytest

from test_gpu_gemm_kq import _run
from test_gpu_parity import tf  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

NARROW, WIDE = "tiles of 64x128", "tiles of 64x256"
SHAPES = ([(b, M, K, N, g, NARROW) for b in (4, 8) for g in (128, 64, 32) for M, K, N in ((129, 640, 6152), (257, 1664, 6152))] +
          [(4, 257, 2176, 11000, g, WIDE) for g in (128, 64, 32)])


@pytest.mark.parametrize("bf", [False, True], ids=["f16", "bf16"])
@pytest.mark.parametrize("bits,M,K,N,G,tiles", SHAPES)
def test_against_oracle(tf, bits, M, K, N, G, tiles, bf):
    got, want = _run(tf, bf, bits, M, K, N, G, None)
    scale = np.abs(want).max()
    bound = (2.0 ** -8 if bf else 2.0 ** -11) * np.abs(want) + (4e-3 if bf else 1e-3) * scale
    assert np.all(np.isfinite(got))
    assert np.all(np.abs(got - want) <= bound), np.abs(got - want).max() / scale
