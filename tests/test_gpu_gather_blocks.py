"""The gather by slots at the edges of its workgroups (one slot or several each, slots
past the end of the last one, heads whose blocks are all or none demanded, more heads
than a workgroup has threads, ragged last blocks) and the flat walk of blocks that are
no whole 16 KB steps; for the demand gather and for the per-consumer packing (a shard
that starts and ends inside a workgroup). Bit-exact."""

import numpy as np
import pytest

import oracle as orc
import paper_2609_32197_amd as sp
from tests import _parity as P
from tests.test_gpu_kernels import _rand_inputs

pytestmark = pytest.mark.gpu

# (H, n, tail, d, block, dtype): K blocks of 256, 512, 1,536 (bf16: flat walk), 2,304, 768,
# 512, 3,840, 5,376 (flat walk), 30,720 (flat walk) and, in 300 heads, 256 16-byte chunks
CASES = [(3, 9, 5, 32, 32, "f32"), (2, 21, 64, 64, 64, "bf16"), (3, 13, 1, 192, 64, "bf16"),
         (2, 4, 50, 96, 96, "f32"), (2, 1, 7, 96, 32, "f32"),
         (5, 1, 3, 64, 64, "bf16"), (2, 9, 159, 96, 160, "f32"), (2, 5, 200, 96, 224, "f32"),
         (1, 4, 900, 64, 3840, "bf16"), (300, 5, 31, 32, 32, "f32")]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "n{1}d{3}b{4}_{5}".format(*c))
def test_blocked_gather(gpu, case):
    torch = P.torch()
    H, n, tail, d, b, dt = case
    L = (n - 1) * b + tail
    _, k, v = _rand_inputs(51, H, L, d, dt)
    Kd, Vd = P.to_device(k, dt), P.to_device(v, dt)
    rng = np.random.default_rng(n)
    mask = rng.random((H, 2 if n > 1 else 1, n)) < 0.4
    mask[0, :, :] = True
    mask[-1, :, :] = False
    mask[-1, 0, n - 1] = True
    g = P.geometry(H, L, d, b, 0, mask.shape[1], dt)
    out = sp.sparsp_demand_union_gather(g, torch.from_numpy(P.words_as_int64(mask)).cuda(), Kd, Vd)
    head_off, gather_blk, slot_of = orc.packing_plan(orc.demand_union(mask))
    S = int(head_off[-1])
    np.testing.assert_array_equal(out["slot_of"].cpu().numpy(), slot_of)
    Kp, Vp = orc.pack_kv(k, v, head_off, gather_blk, L, b)
    np.testing.assert_array_equal(P.from_device_bits(out["K_packed"], dt)[:S], Kp)
    np.testing.assert_array_equal(P.from_device_bits(out["V_packed"], dt)[:S], Vp)
    if n < 4:
        return
    R = 3
    demands = [rng.random((H, n)) < 0.5 for _ in range(R)]
    words = torch.from_numpy(np.stack([orc.mask_to_words(x) for x in demands]).view(np.int64)).cuda()
    for p in range(R):
        got = sp.sparsp_pack_for_consumers(g, words, R, p, Kd, Vd)
        want = orc.pack_by_consumer(orc.provide_masks(demands, R, p), k, v, L, b)
        S = int(want["head_off"][-1])
        np.testing.assert_array_equal(P.from_device_bits(got["K_packed"][:S], dt), want["K_packed"])
        np.testing.assert_array_equal(P.from_device_bits(got["V_packed"][:S], dt), want["V_packed"])
