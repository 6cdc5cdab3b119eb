"""Where the running max of the 128-token rows kernel moves: the rule of its 32x32x16
form, replayed here step by step.

A wave of 32 queries moves its queries' maxima to a block's when some query's block max
passes its limit: the max plus clamp(log2(l) - 2, 0, 8), l being the probability mass
since the start (in units of the max) of the keys 0-7 mod 16 or of the keys 8-15 mod 16.
Which probabilities enter bf16 as exactly 1 follows from that, so a kernel that moves
elsewhere differs by their rounding, 2^-9 each: 2e-3 of O and more on unit normal
inputs. The replay rounds the probabilities at the same places; what remains are float32
sums and the share of probabilities near a rounding's tie (2^-24 / 2^-9 of them, by 2^-8
each), below 1e-5 of O.
"""

import math

import pytest

import paper_2609_32197_amd as sp
from tests import _parity as P

pytestmark = pytest.mark.gpu


def _replay(torch, q, kb, vb, scale):
    """O of one query block: q [128, d], kb and vb [keep, 128, d], all float64."""
    c2 = torch.tensor(scale, dtype=torch.float32) * torch.tensor(1.4426950408889634)
    half = (torch.arange(128, device=q.device) // 8) % 2 == 0   # keys 0-7 mod 16
    m = torch.full((128,), -math.inf, device=q.device, dtype=torch.float64)
    lim = m[:, None].expand(128, 2).clone()
    l = torch.zeros((128, 2), device=q.device, dtype=torch.float64)
    o = torch.zeros_like(q)
    for k, v in zip(kb, vb):
        s = (q @ k.T) * float(c2)                               # log2 units
        mx = s.max(1).values
        passed = (mx[:, None] > lim).any(1).view(4, 32).any(1)  # per wave
        moved = passed.repeat_interleave(32)
        m_new = torch.where(moved, torch.maximum(m, mx), m)
        alpha = torch.where(moved, torch.exp2(m - m_new), torch.ones_like(m))
        m = m_new
        l = l * alpha[:, None]
        o = o * alpha[:, None]
        lim = torch.where(moved[:, None], m[:, None] + (torch.log2(l) - 2).clamp(0, 8), lim)
        p = torch.exp2(s - m[:, None])
        l = l + torch.stack([p[:, half].sum(1), p[:, ~half].sum(1)], 1)
        o = o + p.to(torch.float32).to(torch.bfloat16).double() @ v
    return o / l.sum(1, keepdim=True)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("keep", [2, 12, 40])
def test_max_moves_by_the_lane_pair_rule(gpu, d, keep):
    torch = P.torch()
    H, n, b = 10, 50, 128                        # 500 rows: the rows kernel
    gen = torch.Generator(device="cuda").manual_seed(7 + keep)
    Q, K, V = (torch.randn((H, n * b, d), generator=gen, device="cuda").to(torch.bfloat16)
               for _ in range(3))
    g = P.geometry(H, n * b, d, b, 0, n, "bf16")
    scale = 1 / math.sqrt(d)
    _, _, scores = sp.sparsp_block_scores(g, Q, K)
    mask, sel = sp.sparsp_topk_mask(g, scores, keep)
    out = sp.sparsp_demand_union_gather(g, mask, K, V)
    O, _ = sp.sparsp_block_sparse_attn(g, Q, sel, out["slot_of"], out["K_packed"],
                                       out["V_packed"], scale, out_dtype=sp.F32)
    err = ref2 = 0.0
    for h, r in ((0, 0), (1, 7), (3, 20), (5, 33), (7, 41), (9, 49)):
        at = sel[h, r].long()
        ref = _replay(torch, Q[h, r * b:(r + 1) * b].double(), K[h].view(n, b, d)[at].double(),
                      V[h].view(n, b, d)[at].double(), scale)
        err += float((O[h, r * b:(r + 1) * b].double() - ref).square().sum())
        ref2 += float(ref.square().sum())
    assert math.sqrt(err / ref2) <= 1e-4, math.sqrt(err / ref2)
