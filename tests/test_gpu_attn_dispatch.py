"""The bf16 attention kernels on both sides of the rules that pick one by the number
of rows (128-token blocks: split-key up to 256 rows, rows kernel past them; 64-token
blocks: split-key, and at d = 128 in whole top-k launches the rows kernel at 513 to 768
rows of 8 kept blocks or fewer, 769 to 1,024, 1,664 to 2,000 and past 2,560): rows past a round of resident workgroups (tail split by the workspace), ragged
ends, one to several hundred kept blocks, lists with skipped entries, float32 and bf16
output, an explicit row order (the same kernel, so the same bits). Bars: the parity
suite's (bf16 2e-2 / 1e-3, lse 1e-4).
"""

import numpy as np
import pytest

import oracle as orc
import paper_2609_32197_amd as sp
from tests import _parity as P
from tests.test_gpu_kernels import _pipeline, _rand_inputs, ctypes_scale

pytestmark = pytest.mark.gpu

# (H, L, d, block, i0, i1), keep, rows checked per head
CASES = [
    ((16, 2433, 128, 64, 7, 39), 5, 4),      # 512 rows: the split-key kernel's last, ragged end
    ((19, 2433, 128, 64, 12, 39), 1, 27),    # 513 rows, last block one key, diagonal only
    ((60, 1600, 128, 64, 0, 25), 24, 3),     # 1,500 rows: split-key, 476 past a round of 512
    ((5, 16500, 128, 64, 130, 258), 257, 3),  # 640 rows of 257 kept blocks: split-key
    ((12, 4200, 128, 64, 2, 66), 8, 3),      # 768 rows: the rows kernel with its longest list
    ((12, 4200, 128, 64, 2, 66), 9, 3),      # and one block more: split-key
    ((14, 3521, 128, 64, 1, 56), 24, 3),     # 770 rows, last block one key: rows kernel
    ((4, 16500, 128, 64, 50, 258), 257, 3),  # 832 rows of 257 kept blocks, three load rounds
    ((26, 4100, 128, 64, 1, 65), 24, 3),     # 1,664 rows: rows kernel, 640 past its round
    ((50, 4100, 128, 64, 1, 65), 14, 2),     # 3,200 rows: rows kernel, 128 past three rounds
    ((25, 2500, 64, 64, 8, 40), 3, 4),       # 800 rows at d = 64
    ((47, 2500, 64, 64, 2, 40), 24, 3),      # 1,786 rows: 762 past a round of 1,024
    ((48, 2433, 64, 64, 1, 39), 1, 38),      # 1,824 rows, last block one key, diagonal only
    ((90, 1600, 64, 64, 0, 25), 24, 3),      # 2,250 rows: 202 past two rounds
    ((8, 16500, 64, 64, 20, 258), 257, 3),   # 1,904 rows of 257 kept blocks
    ((8, 4097, 128, 128, 1, 33), 6, 4),  # 256 rows, last block one key: split-key
    ((8, 4225, 64, 128, 2, 34), 1, 32),  # the same at d = 64, diagonal only
    ((1, 35000, 128, 128, 17, 274), 8, 9),  # 257 rows: rows kernel
    ((257, 300, 64, 128, 2, 3), 3, 1),   # the same at d = 64, the ragged block alone
    ((2, 33000, 128, 128, 200, 258), 250, 3),  # 116 rows of 250 kept blocks, split in two
]


@pytest.mark.parametrize("geo,keep,check", CASES, ids=lambda x: str(x).replace(" ", ""))
def test_kernels_by_rows(gpu, geo, keep, check):
    torch = P.torch()
    H, L, d, b, i0, i1 = geo
    q, k, v = _rand_inputs(61, H, L, d, "bf16")
    g = P.geometry(H, L, d, b, i0, i1, "bf16")
    om, osel, sel, out = _pipeline(q, k, v, g, "bf16", keep)
    sel = sel.clone()
    rows = np.linspace(0, g.nq - 1, check).astype(int)
    if keep > 4:  # entries to be skipped: out of range, and a block without a slot
        for r in rows:
            sel[:, r, 1] = -1
            sel[:, r, keep // 2] = g.n
        for h in range(H):
            for r in rows:
                om[h, r, osel[h, r, 1]] = False
                om[h, r, osel[h, r, keep // 2]] = False
    args = (g, P.to_device(q, "bf16"), sel, out["slot_of"], out["K_packed"], out["V_packed"],
            ctypes_scale(d))
    ws = torch.empty((sp.sparsp_attn_workspace_bytes(g, keep),), dtype=torch.uint8, device="cuda")
    plain = sp.sparsp_block_sparse_attn(*args, out_dtype=sp.F32)
    low = sp.sparsp_block_sparse_attn(*args, out_dtype=sp.BF16, workspace=ws)
    order = torch.from_numpy(np.random.default_rng(1).permutation(H * g.nq).astype(np.int32)).cuda()
    ordered = sp.sparsp_block_sparse_attn(*args, out_dtype=sp.F32, row_order=order)
    assert torch.equal(plain[0], ordered[0]) and torch.equal(plain[1], ordered[1])
    outs = [(o.float().cpu().numpy(), l.cpu().numpy()) for o, l in (plain, low)]
    for h in sorted({0, H // 2, H - 1}):
        f = [orc.decode_input(x[h], "bf16") for x in (q, k, v)]
        for r in rows:
            o_ref, l_ref = orc.attend_block(*f, om[h, r], i0 + r, L, b, ctypes_scale(d))
            for o, l in outs:
                P.check_attention(o[h, r * b:(r + 1) * b], o_ref, True, f"{geo} h={h} r={r}")
                fin, lg = np.isfinite(l_ref), l[h, r * b:(r + 1) * b]
                assert (np.isneginf(lg) == ~fin).all()
                assert np.abs(lg[fin] - l_ref[fin]).max(initial=0) <= 1e-4
