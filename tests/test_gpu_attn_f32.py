"""The float32 attention kernel at the edges of its tiles and of its launch rule.

Tiles are 16 queries x 16 keys x 16 dims: blocks and head dimensions just below,
at and above multiples of 16, the smallest of each, tiles with a single valid
key, waves without a tile. The launch takes two query groups per wave where
that does not load the fullest CU more, eight key-splitting waves where every
CU has at most one workgroup, and four otherwise; the cases cover all three.
Bars: 1e-5 max-abs on O and lse against the float64 oracle (the float32 bar of
the parity suite; inputs are unit normal, so |O| stays below 5 and a float32
sum of n <= 1,024 products of that size errs by less than n 2^-24 / sqrt(n) ~
2e-6).
"""

import numpy as np
import pytest

import oracle as orc
import paper_2609_32197_amd as sp
from tests import _parity as P
from tests.test_gpu_kernels import _pipeline, _rand_inputs, ctypes_scale

pytestmark = pytest.mark.gpu

# (H, L, d, block, i0, i1), keep
CASES = [
    ((1, 9, 4, 4, 0, 3), 3),             # smallest d and block, last tile one key: eight waves
    ((2, 33, 16, 16, 0, 3), 3),          # exact tiles, last block one key
    ((2, 130, 20, 20, 2, 7), 4),         # d and block just above a tile
    ((1, 177, 60, 44, 0, 5), 5),         # just below
    ((3, 500, 112, 36, 1, 14), 6),       # seven chunks of d
    ((40, 1000, 32, 100, 0, 10), 3),     # four waves, one query group
    ((32, 2049, 24, 64, 0, 33), 2),      # two query groups, ragged last block of one token
    ((16, 2100, 128, 128, 3, 17), 3),    # two query groups, d = 128
]


@pytest.mark.parametrize("geo,keep", CASES, ids=lambda x: str(x).replace(" ", ""))
def test_float32_attention_edges(gpu, geo, keep):
    H, L, d, b, i0, i1 = geo
    torch = P.torch()
    q, k, v = _rand_inputs(31, H, L, d, "f32")
    g = P.geometry(H, L, d, b, i0, i1, "f32")
    om, osel, sel, out = _pipeline(q, k, v, g, "f32", keep)
    np.testing.assert_array_equal(sel.cpu().numpy(), osel)
    # Rows past L of the packed buffers are never attended, whatever they hold.
    last = out["slot_of"][:, g.n - 1].cpu().numpy()
    tail = L - (g.n - 1) * b
    for s in last[last >= 0]:
        out["K_packed"][int(s), tail:] = float("nan")
        out["V_packed"][int(s), :, tail:] = float("nan")
    args = (g, P.to_device(q, "f32"), sel, out["slot_of"], out["K_packed"], out["V_packed"],
            ctypes_scale(d))
    O, lse = sp.sparsp_block_sparse_attn(*args)
    O_ref, lse_ref = orc.sparse_attention(*(x.astype(np.float64) for x in (q, k, v)), om, L, b, i0,
                                          ctypes_scale(d))
    P.check_attention(O.cpu().numpy(), O_ref, False, f"{geo}")
    ln, fin = lse.cpu().numpy(), np.isfinite(lse_ref)
    assert (np.isneginf(ln) == ~fin).all()
    assert np.abs(ln[fin] - lse_ref[fin]).max() <= 1e-5

    # An explicit row order changes the schedule only.
    rows = H * g.nq
    order = torch.from_numpy(np.random.default_rng(3).permutation(rows).astype(np.int32)).cuda()
    O2, lse2 = sp.sparsp_block_sparse_attn(*args, row_order=order)
    assert torch.equal(O, O2) and torch.equal(lse, lse2)

    # Two shards folded together give the whole, and untouched rows stay.
    mid = g.n // 2
    O3, l3 = sp.sparsp_block_sparse_attn_part(*args[:6], (0, mid), (0, H), args[6])
    sp.sparsp_block_sparse_attn_part(*args[:6], (mid, g.n), (0, H), args[6], O=O3, lse=l3,
                                     accumulate=True)
    P.check_attention(O3.cpu().numpy(), O_ref, False, f"{geo} in two parts")
    assert np.abs(l3.cpu().numpy()[fin] - lse_ref[fin]).max() <= 1e-5


@pytest.mark.parametrize("scale", [1.0, 300.0, 1e5, 1e8, 1e20, 1e30])
def test_float32_attention_at_large_scales(gpu, scale):
    """Scales up to the entry point's limit, where softmax picks the best keys. Inputs
    are small whole numbers, so every q.k is exact in float32, best keys that tie tie
    in both, and the next best are at least ``scale`` below. From scale 300 on O is
    the mean of the V rows that tie (at most 32 of them here: below 1e-5 of rounding
    for |V| <= 8); lse is rounded to its own 24 bits, in two steps."""
    H, L, d, b, i0, i1, keep = 3, 1000, 64, 64, 0, 16, 9
    rng = np.random.default_rng(17)
    q, k = (rng.integers(-3, 4, (H, L, d)).astype(np.float32) for _ in range(2))
    v = rng.integers(-8, 9, (H, L, d)).astype(np.float32)
    g = P.geometry(H, L, d, b, i0, i1, "f32")
    om, osel, sel, out = _pipeline(q, k, v, g, "f32", keep)
    O, lse = sp.sparsp_block_sparse_attn(g, P.to_device(q, "f32"), sel, out["slot_of"],
                                         out["K_packed"], out["V_packed"], scale)
    O_ref, lse_ref = orc.sparse_attention(*(x.astype(np.float64) for x in (q, k, v)), om, L, b, i0,
                                          float(np.float32(scale)))
    P.check_attention(O.cpu().numpy(), O_ref, False, f"scale {scale}")
    ln, fin = lse.cpu().numpy(), np.isfinite(lse_ref)
    assert (np.isneginf(ln) == ~fin).all()
    assert (np.abs(ln[fin] - lse_ref[fin]) <= 1e-5 + 4 * 2.0 ** -24 * np.abs(lse_ref[fin])).all()


@pytest.mark.parametrize("d", [32, 20])
def test_float32_attention_of_infinite_scores(gpu, d):
    """Keys of -inf under queries that are positive score -inf and weigh nothing, also
    where they fill a wave's first tiles, or a row's whole list; the keys beside them in
    memory count as ever (d = 20 leaves part of a 16-wide step of the product to
    padding). Bars as above; q.k of 32 uniform products is below 32."""
    H, L, b, i0, i1, keep = 2, 1100, 64, 0, 18, 6
    rng = np.random.default_rng(23)
    q = rng.uniform(0.1, 1.0, (H, L, d)).astype(np.float32)
    k, v = (rng.standard_normal((H, L, d)).astype(np.float32) for _ in range(2))
    g = P.geometry(H, L, d, b, i0, i1, "f32")
    om, osel, sel, _ = _pipeline(q, k, v, g, "f32", keep)
    gone = rng.random((H, L)) < 0.3                # single keys,
    for h in range(H):
        gone[h, osel[h, 2, 0] * b:(osel[h, 2, 0] + 1) * b] = True  # a first block,
        for j in osel[h, 7]:                       # and all that one row keeps
            gone[h, j * b:(j + 1) * b] = True
    k[gone] = -np.inf
    mask = P.torch().from_numpy(P.words_as_int64(om)).cuda()
    out = sp.sparsp_demand_union_gather(g, mask, P.to_device(k, "f32"), P.to_device(v, "f32"))
    O, lse = sp.sparsp_block_sparse_attn(g, P.to_device(q, "f32"), sel, out["slot_of"],
                                         out["K_packed"], out["V_packed"], ctypes_scale(d))
    ln = lse.cpu().numpy()
    assert not np.isfinite(ln[:, 7 * b:8 * b]).any()
    x = np.einsum("hqd,hkd->hqk", q.astype(np.float64), k.astype(np.float64)) * ctypes_scale(d)
    kept = np.repeat(np.repeat(om, b, 1), b, 2)[:, :L, :L]
    x[~kept] = -np.inf
    m = x.max(2, keepdims=True)
    p = np.exp(x - np.where(np.isfinite(m), m, 0.0))
    l = p.sum(2, keepdims=True)
    O_ref = np.divide(p @ v.astype(np.float64), l, out=np.zeros((H, L, d)), where=l > 0)
    assert np.abs(O.cpu().numpy()[:, :L] - O_ref).max() <= 1e-5
    fin = l[..., 0] > 0
    lse_ref = (m + np.log(np.where(l > 0, l, 1.0)))[..., 0]
    assert (np.isneginf(ln[:, :L]) == ~fin).all()
    assert np.abs(ln[:, :L][fin] - lse_ref[fin]).max() <= 1e-5
