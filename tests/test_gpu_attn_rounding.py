"""Rounding of the bf16 attention of 64-token blocks in large launches, against the
split-key kernel on the same rows.

At d = 128 such launches take the rows kernel. Both hold the same operands and round
the probabilities to bf16 once. They differ in how many of the top probabilities enter
as exactly 1, so the 2-norm of the error against float64 must not be larger than the
split-key kernel's (1% for the sampling of a few million elements). The split-key
kernel is reached by attending two runs of heads as parts, which always take it.
Inputs: unit normal, and peaked with a query's mass on a few keys of one or two blocks.
"""

import math

import numpy as np
import pytest

import paper_2609_32197_amd as sp
from tests import _parity as P

pytestmark = pytest.mark.gpu

# (H, n, d, nq), keep
CASES = [
    ((10, 100, 64, 82), 12),    # d = 64: 820 rows
    ((20, 96, 64, 96), 14),     # 1,920 rows
    ((20, 96, 64, 96), 50),
    ((10, 100, 128, 82), 2),    # d = 128: 820 rows
    ((10, 100, 128, 82), 14),
    ((10, 100, 128, 82), 60),
    ((25, 100, 128, 100), 30),  # 2,500 rows
]


def _inputs(torch, H, L, d, peaked):
    gen = torch.Generator(device="cuda").manual_seed(9)
    q, k, v = (torch.randn((H, L, d), generator=gen, device="cuda") for _ in range(3))
    if peaked:  # a low-frequency pattern shared by Q and K: each query's mass is on a few keys
        t = torch.arange(L, device="cuda")[None, :, None] / L
        nu = 20 * torch.rand((H, 1, d), generator=gen, device="cuda")
        f = 2 * math.sqrt(2) * torch.cos(2 * math.pi * (nu * t + torch.rand((H, 1, d), generator=gen,
                                                                        device="cuda")))
        q, k = q + f, k + f
    return [x.to(torch.bfloat16) for x in (q, k, v)]


@pytest.mark.parametrize("geo,keep", CASES, ids=lambda x: str(x).replace(" ", ""))
@pytest.mark.parametrize("peaked", [False, True], ids=["iid", "peaked"])
def test_rounds_no_more_than_the_split_key_kernel(gpu, geo, keep, peaked):
    torch = P.torch()
    H, n, d, nq = geo
    b, L, scale = 64, n * 64, 1 / math.sqrt(d)
    Q, K, V = _inputs(torch, H, L, d, peaked)
    g = P.geometry(H, L, d, b, 0, nq, "bf16")
    _, _, scores = sp.sparsp_block_scores(g, Q, K)
    mask, sel = sp.sparsp_topk_mask(g, scores, keep)
    out = sp.sparsp_demand_union_gather(g, mask, K, V)
    args = (g, Q, sel, out["slot_of"], out["K_packed"], out["V_packed"])
    O, lse = sp.sparsp_block_sparse_attn(*args, scale, out_dtype=sp.F32)
    R = torch.empty_like(O)
    rl = torch.empty_like(lse)
    for heads in ((0, H - 1), (H - 1, H)):
        sp.sparsp_block_sparse_attn_part(*args, (0, n), heads, scale, O=R, lse=rl)
    e_new = e_old = 0.0
    worst = torch.zeros((), dtype=torch.float64, device="cuda")
    for h in range(H):
        rows = sel[h].long()
        k = K[h].view(n, b, d).double()[rows].reshape(nq, keep * b, d)
        v = V[h].view(n, b, d).double()[rows].reshape(nq, keep * b, d)
        s = torch.bmm(Q[h, :nq * b].view(nq, b, d).double(), k.transpose(1, 2).contiguous()) * scale
        ref = torch.bmm(torch.softmax(s, 2), v).reshape(nq * b, d)
        e_new += float((O[h].double() - ref).square().sum())
        e_old += float((R[h].double() - ref).square().sum())
        worst = torch.maximum(worst, (lse[h].double() - torch.logsumexp(s, 2).reshape(-1)).abs().max())
    assert np.isfinite(e_new) and math.sqrt(e_new) <= 1.01 * math.sqrt(e_old), (e_new, e_old)
    assert float(worst) <= 1e-4
