"""The score, top-k and row-order kernels at the edges of their tiles and instances.

* Scores: output tiles of 64 x 64, slices of 32 of d, pooled tiles that are not
  16-byte aligned (read word by word). Held to the parity suite's bound, which is
  derived from the order-free error of a float32 sum.
* Top-k: every number of mask words has an instance up to 16, then 24, 32, 48 and
  64; rows one block before, at and after a word and an instance boundary, scores
  of one scale (the search stops early), of widely different scales and with ties
  across the cut. Bit-exact.
* Row order: the documented queue assignment is checked where heads do not divide
  by eight, a queue stays empty, and rows do not fit the LDS cache.
"""

import numpy as np
import pytest

import oracle as orc
import paper_2609_32197_amd as sp
from tests import _parity as P
from tests.test_gpu_kernels import _rand_inputs

pytestmark = pytest.mark.gpu

SCORES = [  # (H, L, d, block, i0, i1, dtype)
    (1, 63, 8, 1, 0, 1, "bf16"), (2, 65, 24, 1, 0, 65, "bf16"), (1, 130, 256, 2, 1, 64, "bf16"),
    (3, 127, 4, 1, 60, 127, "f32"), (2, 700, 36, 11, 0, 64, "f32"), (1, 520, 100, 8, 0, 65, "f32"),
]


@pytest.mark.parametrize("shift", [0, 1], ids=["aligned", "unaligned"])
@pytest.mark.parametrize("geo", SCORES, ids=lambda g: "L{1}d{2}b{3}_{6}".format(*g))
def test_score_edges(gpu, geo, shift):
    torch = P.torch()
    H, L, d, b, i0, i1, dt = geo
    q, k, _ = _rand_inputs(41, H, L, d, dt)
    g = P.geometry(H, L, d, b, i0, i1, dt)
    out = []
    for shape in ((H, g.nq, d), (H, g.n, d), (H, g.nq, g.n)):
        flat = torch.empty((int(np.prod(shape)) + 1,), device="cuda")
        out.append(flat[shift:shift + int(np.prod(shape))].view(shape))
    pq, pk, sc = sp.sparsp_block_scores(g, P.to_device(q, dt), P.to_device(k, dt), *out)
    opq, opk, osc, aq, ak = P.oracle_pooled_scores(q, k, dt, L, b, i0, i1, d, with_abs=True)
    err = np.abs(sc.cpu().numpy().astype(np.float64) - osc.astype(np.float64))
    tol = P.score_tolerance(opq, opk, aq, ak, osc, d, b, dt)
    assert (err <= tol).all(), f"max excess {(err - tol).max():.3g}"


@pytest.mark.parametrize("n", [63, 64, 65, 576, 577, 640, 1024, 1025, 1536, 1537, 2048, 2049, 3072,
                               3073])
@pytest.mark.parametrize("kind", ["normal", "scales", "ties"])
def test_topk_instances(gpu, n, kind):
    rng = np.random.default_rng(n)
    H, nq, i0 = 2, 5, n // 2
    s = rng.standard_normal((H, nq, n)).astype(np.float32)
    if kind == "scales":
        s *= np.float32(10.0) ** rng.integers(-30, 30, size=s.shape).astype(np.float32)
        s[:, :, ::7] = -np.inf
    elif kind == "ties":
        s = np.round(s * 4) / 4
    G = (0, n - 1)
    g = sp.Geometry(H, n, 8, 1, i0, i0 + nq, sp.BF16)
    for keep in (3, 1 + n // 7, n - 1, n):
        m, sel = sp.sparsp_topk_mask(g, P.to_device(s, "f32"), keep, G)
        om, osel = orc.select_topk(s, keep, i0, G)
        np.testing.assert_array_equal(m.cpu().numpy(), P.words_as_int64(om))
        np.testing.assert_array_equal(sel.cpu().numpy(), osel)


@pytest.mark.parametrize("H,nq,n", [(1, 3, 5), (5, 40, 70), (11, 130, 140), (16, 1000, 1000)])
def test_row_order_queues(gpu, H, nq, n):
    torch = P.torch()
    rng = np.random.default_rng(H)
    counts = rng.integers(0, n + 1, size=(H, nq)).astype(np.int32)
    counts[H // 2] = counts[0]  # heads of equal total
    g = sp.Geometry(H, n, 8, 1, 0, nq, sp.BF16)
    order = sp.sparsp_row_order(g, torch.from_numpy(counts).cuda()).cpu().numpy()
    assert (np.sort(order) == np.arange(H * nq)).all()
    tot = counts.sum(1).astype(np.int64)
    room = [H // 8 + (x < H % 8) for x in range(8)]
    load, heads = [0] * 8, [[] for _ in range(8)]
    for h in sorted(range(H), key=lambda h: (-tot[h], h)):
        x = min((x for x in range(8) if room[x]), key=lambda x: (load[x], x))
        heads[x].append(h)
        load[x] += int(tot[h])
        room[x] -= 1
    lens = [len(x) * nq for x in heads]
    at = 0
    queues = [[] for _ in range(8)]
    for k in range(max(lens)):
        for x in range(8):
            if k < lens[x]:
                queues[x].append(int(order[at]))
                at += 1
    flat = counts.reshape(-1)
    for x in range(8):
        assert sorted({r // nq for r in queues[x]}) == sorted(heads[x])
        c = flat[queues[x]]
        assert (np.diff(c) <= 0).all()
