"""The work queue of the persistent kernels at the counts where it can go wrong: a launch's first items are dealt by
workgroup index, the others claimed from eight lists (head count a multiple of 8) or from one, so every item has to be
done exactly once around one, two and more items per workgroup.  All heads hold the same data: outputs start as NaN, every
head has to show the bits of the first, and the first is checked against the oracle."""
import numpy as np
import pytest
from oracle import attention as ora

from parity_util import compare_all, randn_bf16, to64

pytestmark = pytest.mark.gpu


# (256 CUs: one 256-row forward / dQ item and one dK/dV item per CU, two or three at head dimension 64)
@pytest.mark.parametrize("S,H,D,lens", [
    (40, 1, 128, None), (40, 7, 128, None), (40, 8, 128, None),
    (40, 255, 128, None), (40, 256, 128, None), (40, 257, 128, None), (40, 264, 128, None),
    (300, 256, 128, None),       # two 256-row items and three 128-row items per workgroup
    (300, 261, 128, None),       # the same with one list
    (130, 264, 64, None), (130, 513, 64, None), (300, 512, 64, None),
    (200, 176, 128, [70, 0, 1, 129]),   # packed: list entries without an item
    (200, 171, 128, [70, 0, 1, 129]),
])
def test_every_item_is_done_once(S, H, D, lens):
    import torch
    from paper_2401_09149_amd import binding
    print(f"case S{S} H{H} D{D} {lens}", flush=True)
    dev, scale = "cuda:0", D ** -0.5
    one = [randn_bf16((1, S, 1, D), 700 + j) for j in range(4)]
    q, k, v, do = (t.to(dev).expand(1, S, H, D).contiguous() for t in one)
    cu = None if lens is None else torch.tensor([0] + lens, dtype=torch.int32).cumsum(0).to(torch.int32).to(dev)
    o = torch.full_like(q, float("nan"))
    lse = torch.full((1, H, S), float("nan"), device=dev)
    grads = [torch.full_like(t, float("nan")) for t in (q, k, v)]
    ws = binding.alloc_bwd_workspace(q, k, cu)
    before = binding.ie_attn_set_tile_rows(256 if D == 128 else 0)   # the forward with a queue
    try:
        for _ in range(2):   # (the forward's counters are left clear by the launch before)
            binding.ie_attn_fwd(q, k, v, o, lse, cu, scale, True)
        for phase in (binding.BWD_DELTA, binding.BWD_DQ, binding.BWD_DKDV):   # (a launch with a queue each)
            binding.ie_attn_bwd_phases(q, k, v, o, do, lse, *grads, cu, scale, True, ws, phase)
        torch.cuda.synchronize()
    finally:
        binding.ie_attn_set_tile_rows(before)
    for t in (o, *grads):
        assert torch.equal(t, t[:, :, :1].expand_as(t))
    assert torch.equal(lse, lse[:, :1].expand_as(lse))
    got = (o[:, :, :1], lse[:, :1], *(t[:, :, :1] for t in grads))
    ref = ora.attn_fwd_bwd(*(to64(t) for t in one), scale, True, None if cu is None else np.asarray(cu.cpu()))
    compare_all(got, ref, f"S{S} H{H} D{D}")
