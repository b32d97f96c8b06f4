"""GEMM calls with short K against the CPU oracle: the 128 x 128 kernel without a
pipeline (any K and group, ragged tile edges, a group a step, groups of three
steps and of whole 128-row chunks, one step) and, for 33 to 64 rows of 8-bit
weights, the streaming form with 64 row slots (every block of rows full or
partly used, runs that end inside a round, the last panel partly past N).

Tolerances as for the other tiled kernels, which also round each weight once."""
from __future__ import annotations

import numpy as np
import pytest

from test_gpu_gemm_kq import _run
from test_gpu_parity import tf  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ANY_SHAPES = [(4, 1100, 32, 1032, 32), (4, 700, 96, 2056, 96), (4, 130, 64, 8200, 64), (4, 520, 160, 4360, 32),
              (4, 900, 128, 2056, 128), (8, 1100, 32, 1032, 32), (8, 200, 96, 5000, 96), (8, 385, 224, 5000, 32),
              (8, 1600, 160, 2056, 160), (4, 1478, 480, 5752, 96)]
STREAM64_SHAPES = [(8, 33, 32, 8, 32), (8, 64, 96, 72, 96), (8, 48, 1120, 600, 32), (8, 49, 480, 1456, 96),
                   (8, 64, 672, 264, 32), (8, 33, 640, 8192, 128), (8, 64, 384, 520, 384)]


@pytest.mark.parametrize("bf", [False, True], ids=["f16", "bf16"])
@pytest.mark.parametrize("bits,M,K,N,G", ANY_SHAPES + STREAM64_SHAPES)
def test_against_oracle(tf, bits, M, K, N, G, bf):
    got, want = _run(tf, bf, bits, M, K, N, G, None)
    scale = np.abs(want).max()
    bound = (2.0 ** -8 if bf else 2.0 ** -11) * np.abs(want) + (4e-3 if bf else 1e-3) * scale
    assert np.all(np.isfinite(got))
    assert np.all(np.abs(got - want) <= bound), np.abs(got - want).max() / scale
