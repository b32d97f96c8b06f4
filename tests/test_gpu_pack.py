"""tf_pack_w4 / tf_pack_w8 / tf_pack_w8_sym byte for byte against the packed
layout written out plainly in numpy, at the edges of the blocks the kernel
works on (8 panels by one 32-row atom): one column word, a panel's last
columns, one panel past a block, groups of one atom, of several and of all of
K."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2606_11357_amd.synth import make_inputs, make_inputs_w8sym

from test_gpu_parity import dev, pack, tf  # noqa: F401

pytestmark = pytest.mark.gpu

SHAPES = [(32, 8, 32), (96, 72, 32), (96, 520, 96), (256, 1032, 64), (128, 248, 128), (160, 264, 32)]


def _align(n):
    return -(-n // 256) * 256


def plain_pack(bits, q, z, s_bits, G):
    """Atoms of 32 rows by 64 (32) columns: lane 16 kg + c, dword t holds rows
    8 kg .. of column c + 16 t (8-bit: dwords 2 t, 2 t + 1); metadata entry
    c T + t.  Bytes between the regions are left at zero."""
    K, N = q.shape
    pw = 64 if bits == 4 else 32
    T, panels, atoms, groups = pw // 16, -(-N // pw), K // 32, K // G
    qp, zp, sp = (np.pad(a, ((0, 0), (0, panels * pw - N))) for a in (q, z, s_bits))
    # [atom, kg, row, panel, t, c] -> [panel, atom, kg, c, t, row]
    rows = qp.reshape(atoms, 4, 8, panels, T, 16).transpose(3, 0, 1, 5, 4, 2).astype(np.uint32)
    if bits == 4:
        order = [0, 2, 4, 6, 1, 3, 5, 7]                    # nibble j holds row order[j]
        words = sum(rows[..., r] << np.uint32(4 * j) for j, r in enumerate(order))
    else:
        four = rows.reshape(*rows.shape[:-1], 2, 4)
        words = sum(four[..., b] << np.uint32(8 * b) for b in range(4))
    meta = lambda a: a.reshape(groups, panels, T, 16).transpose(1, 0, 3, 2)  # noqa: E731
    regions = [np.ascontiguousarray(words, dtype=np.uint32), np.ascontiguousarray(meta(sp), dtype=np.uint16),
               np.ascontiguousarray(meta(zp), dtype=np.uint8)]
    out = b"".join(r.tobytes().ljust(_align(r.nbytes), b"\0") for r in regions)
    return np.frombuffer(out, dtype=np.uint8)


@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("K,N,G", SHAPES)
def test_packed_bytes(tf, bits, K, N, G):
    d = make_inputs(bits, 1, K, N, group=G, seed=K + N)
    import torch
    out = torch.zeros(tf.packed_bytes(bits, K, N, G), dtype=torch.uint8, device="cuda")
    if bits == 4:
        tf.pack_w4(dev(d["qweight"]), dev(d["qzeros"]), dev(d["s"]), K, N, G, out=out)
    else:
        tf.pack_w8(dev(d["qweight"]), dev(d["zeros"]), dev(d["s"]), K, N, G, out=out)
    want = plain_pack(bits, d["q"], d["z"], d["s"].view(np.uint16), G)
    np.testing.assert_array_equal(out.cpu().numpy(), want)


@pytest.mark.parametrize("K,N,G", SHAPES)
def test_packed_bytes_sym(tf, K, N, G):
    import torch
    d = make_inputs_w8sym(1, K, N, seed=K + N)
    out = torch.zeros(tf.packed_bytes(8, K, N, G), dtype=torch.uint8, device="cuda")
    tf.pack_w8_sym(dev(d["qweight"]), dev(d["scales"]), K, N, G, out=out)
    codes = (d["q"].astype(np.int16) + 128).astype(np.uint8)
    want = plain_pack(8, codes, np.full((K // G, N), 128, np.uint8),
                      np.tile(d["s"].view(np.uint16), (K // G, 1)), G)
    np.testing.assert_array_equal(out.cpu().numpy(), want)
