"""sparsp_chunked_attn over plans that no schedule makes: ranges that overlap (a
block counts once per chunk that holds it), gaps, empty ranges, heads in no chunk.

The reference is the calls the plan stands for: sparsp_block_sparse_attn_part
per chunk in plan order, from the empty result. The kernel depends on a launch's
number of rows, so chunks that share a launch may round elsewhere: held to the bars
of the parity suite (1e-5; 2e-2 max-abs and 1e-3 mean-abs; lse 1e-5 and 1e-4). A
schedule takes each shard over all heads, and equals those calls bit for bit.
"""

import math

import numpy as np
import pytest

import paper_2609_32197_amd as sp
from tests import _parity as P
from tests.test_gpu_chunked import _setup

pytestmark = pytest.mark.gpu

GEOMS = [(5, 700, 64, 64, 2, 11, "f32"), (5, 1500, 128, 128, 1, 12, "bf16"),
         (5, 900, 64, 64, 0, 14, "bf16")]
# (kv_lo, kv_hi, head_begin, head_end) with kv in fractions of n
PLANS = {
    "overlap": [(0, .5, 0, 5), (.25, .75, 1, 3), (.5, 1, 0, 4)],
    "twice": [(0, 1, 0, 2), (0, 1, 1, 2)],
    "gaps": [(.6, .8, 0, 3), (0, .3, 1, 5), (.8, 1, 2, 3)],
    "empty": [(.5, .5, 0, 5), (.2, .4, 3, 4)],
    "none": [],
}


@pytest.mark.parametrize("geo", GEOMS, ids=lambda g: "d{2}b{3}_{6}".format(*g))
@pytest.mark.parametrize("name", PLANS)
def test_plan_equals_its_parts(gpu, geo, name):
    import torch
    g, _, sel, out, Qd, _, scale = _setup(geo, 12)
    plan = [sp.Chunk(0, int(a * g.n), int(b * g.n), h0, h1, 0) for a, b, h0, h1 in PLANS[name]]
    args = (g, Qd, sel, out["slot_of"], out["K_packed"], out["V_packed"])
    O = torch.full((g.H, g.nq * g.block, g.d), float("nan"), device="cuda")
    lse = torch.full((g.H, g.nq * g.block), float("nan"), device="cuda")
    sp.sparsp_chunked_attn(*args, plan, scale, O=O, lse=lse)
    R, rl = torch.zeros_like(O), torch.full_like(lse, -math.inf)
    for c in plan:
        sp.sparsp_block_sparse_attn_part(*args, (c.kv_blk_begin, c.kv_blk_end),
                                         (c.head_begin, c.head_end), scale, O=R, lse=rl,
                                         accumulate=True)
    got, ref = O.cpu().numpy(), R.cpu().numpy().astype(np.float64)
    P.check_attention(got, ref, g.dtype == sp.BF16, f"{geo} {name}")
    ln, rn = lse.cpu().numpy(), rl.cpu().numpy()
    fin = np.isfinite(rn)
    assert (np.isneginf(ln) == ~fin).all()
    assert np.abs(ln[fin] - rn[fin]).max(initial=0) <= (1e-4 if g.dtype == sp.BF16 else 1e-5)


MANY = [(12, 9000, 128, 128, 10, 60, "bf16"), (3, 3000, 64, 128, 0, 24, "bf16"),
        (12, 3000, 64, 128, 0, 24, "bf16"), (12, 5000, 128, 64, 0, 60, "bf16")]


# (a launch takes up to 16 shards one after another)
@pytest.mark.parametrize("geo, ranks", [(g, r) for g in GEOMS + MANY for r in (1, 4)]
                         + [(g, r) for g in MANY for r in (16, 17, 23)],
                         ids=lambda v: v if isinstance(v, int) else
                         "h{0}d{2}b{3}_{6}".format(*v))
def test_schedule_folds_one_shard_after_another(gpu, geo, ranks):
    """Each shard has a softmax of its own, as when shards arrive one by one: attending
    them together would round more (bf16: fewer top probabilities are exact)."""
    g, _, sel, out, Qd, _, scale = _setup(geo, 9)
    rank = ranks // 2
    plan = sp.sparsp_chunk_plan(g, out["demand"], ranks, rank, 2, 1)
    args = (g, Qd, sel, out["slot_of"], out["K_packed"], out["V_packed"])
    O, lse = sp.sparsp_chunked_attn(*args, plan, scale)
    R, rl = None, None
    for k in range(ranks):
        p = (rank + k) % ranks
        shard = (p * g.n // ranks, (p + 1) * g.n // ranks)
        R, rl = sp.sparsp_block_sparse_attn_part(*args, shard, (0, g.H), scale, O=R, lse=rl,
                                                 accumulate=k > 0)
    assert (O == R).all() and (lse == rl).all()
