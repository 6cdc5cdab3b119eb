"""Balanced attention of fewer rows of 128-token blocks than workgroups that are
resident: every row is split, by the kernel whose pieces fill the GPU better, or
none. Launches on each side of the lines between those.

Rows, pieces and the plain call's bits where nothing is split follow
``test_gpu_balanced.py``, whose helpers read the split back from the workspace's
size; the rows of both calls meet the parity bar against the oracle.
"""

import numpy as np
import pytest

import oracle as orc
import paper_2609_32197_amd as sp
from tests import _parity as P
from tests.test_gpu_balanced import GEOMS, row_sort_bytes, tail_rows
from tests.test_gpu_kernels import _pipeline, _rand_inputs, ctypes_scale

pytestmark = pytest.mark.gpu

# (H, L, d, block, i0, i1, dtype), kept blocks, pieces; all end in a ragged block
SPLIT = [
    ((1, 9000, 128, 128, 66, 71, "bf16"), 4, 4),     # 5 rows: rows kernel
    ((2, 9000, 64, 128, 35, 71, "bf16"), 11, 4),     # 72 rows: rows kernel, its longest list
    ((2, 9000, 128, 128, 35, 71, "bf16"), 12, 3),    # split-key kernel
    ((2, 9000, 128, 128, 35, 71, "bf16"), 28, 3),
    ((2, 9000, 128, 128, 21, 71, "bf16"), 47, 2),    # 100 rows: its longest list
    ((2, 9000, 128, 128, 21, 71, "bf16"), 48, 4),    # rows kernel
    ((2, 9000, 128, 128, 7, 71, "bf16"), 5, 2),      # 128 rows: split-key kernel
    ((3, 9000, 128, 128, 28, 71, "bf16"), 1, 3),     # 129 rows: rows kernel, lists of one
    ((3, 9000, 64, 128, 20, 71, "bf16"), 71, 3),     # 153 rows, every block
    ((2, 10980, 128, 128, 1, 86, "bf16"), 24, 3),    # 170 rows: the last in three
    ((3, 7400, 64, 128, 1, 58, "bf16"), 2, 1),       # 171 rows, left whole: rows kernel
    ((3, 7400, 64, 128, 1, 58, "bf16"), 3, 1),       # split-key kernel
    ((3, 7400, 64, 128, 1, 58, "bf16"), 47, 1),
    ((3, 7400, 64, 128, 1, 58, "bf16"), 48, 2),      # rows kernel, in two
    ((4, 8300, 128, 128, 1, 65, "bf16"), 4, 1),      # 256 rows, whole: rows kernel
    ((4, 8300, 128, 128, 1, 65, "bf16"), 5, 1),      # split-key kernel
    ((4, 8300, 128, 128, 1, 65, "bf16"), 50, 2),     # rows kernel, in two
]


@pytest.mark.parametrize("geo,keep,pieces", SPLIT,
                         ids=lambda x: "H{}L{}d{}b{}_{}-{}_{}".format(*x) if isinstance(x, tuple) else str(x))
def test_every_row_split(gpu, geo, keep, pieces):
    torch = P.torch()
    H, L, d, b, i0, i1, dt = geo
    q, k, v = _rand_inputs(5, H, L, d, dt)
    g = P.geometry(H, L, d, b, i0, i1, dt)
    om, osel, sel, out = _pipeline(q, k, v, g, dt, keep)
    split, kk, nbytes = tail_rows(g, keep, sel)
    nq = i1 - i0
    rows = H * nq
    assert kk == pieces and len(split) == (rows if pieces > 1 else 0)
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    args = (g, P.to_device(q, dt), sel, out["slot_of"], out["K_packed"], out["V_packed"],
            ctypes_scale(d))
    O0, l0 = sp.sparsp_block_sparse_attn(*args)
    O1, l1 = sp.sparsp_block_sparse_attn(*args, workspace=ws)
    if pieces == 1:
        assert torch.equal(O0.view(torch.int16), O1.view(torch.int16))
        assert torch.equal(l0.view(torch.int32), l1.view(torch.int32))
    Qf, Kf, Vf = (orc.decode_input(x, dt) for x in (q, k, v))
    got = [(O.float().cpu().numpy(), l.cpu().numpy()) for O, l in ((O0, l0), (O1, l1))]
    for row in sorted({*range(0, rows, max(1, rows // 20)), rows - 1}):
        h, r = divmod(row, nq)
        o_ref, lse_ref = orc.attend_block(Qf[h], Kf[h], Vf[h], om[h, r], i0 + r, L, b,
                                          ctypes_scale(d))
        fin = np.isfinite(lse_ref)
        for On, ln in got:
            P.check_attention(On[h, r * b:(r + 1) * b], o_ref, True, f"{geo} keep={keep} row={row}")
            lr = ln[h, r * b:(r + 1) * b]
            assert (np.isneginf(lr) == ~fin).all()
            assert np.abs(lr[fin] - lse_ref[fin]).max() <= 1e-4


@pytest.mark.parametrize("geo", GEOMS[:3], ids=lambda g: "H{}L{}d{}b{}_{}-{}_{}".format(*g))
def test_long_lists_without_room(gpu, geo):
    """Two pieces of every row but one float: too small, so the plain call."""
    torch = P.torch()
    H, L, d, b, i0, i1, dt = geo
    q, k, v = _rand_inputs(6, H, L, d, dt)
    g = P.geometry(H, L, d, b, i0, i1, dt)
    _, _, sel, out = _pipeline(q, k, v, g, dt, 29)
    args = (g, P.to_device(q, dt), sel, out["slot_of"], out["K_packed"], out["V_packed"],
            ctypes_scale(d))
    O0, l0 = sp.sparsp_block_sparse_attn(*args)
    rows = H * (i1 - i0)
    for nbytes in (b * (d + 1) * 4, row_sort_bytes(rows) + 2 * rows * b * (d + 1) * 4 - 4):
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        O1, l1 = sp.sparsp_block_sparse_attn(*args, workspace=ws)
        assert torch.equal(O0.view(torch.int16), O1.view(torch.int16))
        assert torch.equal(l0.view(torch.int32), l1.view(torch.int32))
