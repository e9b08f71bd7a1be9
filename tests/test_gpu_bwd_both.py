"""dK/dV and dQ in one launch (attn_bwd_both_kernel) against the same pass in two.  At head dimension 64 the item bodies
are the same; at head dimension 128 the shared launch's dQ items (dq_item_seq) are others, which add the same products in
the same order as dq_item: the same bits either way.  The one-launch form is taken where all items of both kinds are
resident at once, and also where bwd64_route or bwd128_in_one_launch (csrc/dispatch.hpp) says so
(tests/test_dispatch_rules.py holds the cases to it); a call that names the phases one by one takes the kernels of their
own."""
import numpy as np
import pytest
from oracle import attention as ora

from parity_util import compare_all, randn_bf16, to64

pytestmark = pytest.mark.gpu


DEALT = [
    (1, 512, 2, 2, 64, True, None),       # 16 items, one per workgroup
    (1, 4096, 8, 8, 64, True, None),      # 512 items: the last size where all are resident
    (1, 4097, 8, 8, 64, True, None),      # one tile more per head: a second round, one-row tiles
    (4, 2000, 12, 12, 64, False, None),   # three rounds
    (1, 700, 48, 48, 64, True, None),     # 576 short items
    (1, 8192, 4, 1, 64, False, None),     # fewer dK/dV items than CUs
    (1, 1, 3, 1, 64, True, None),
    (1, 1000, 4, 2, 64, True, [300, 0, 1, 699]),
    (1, 2047, 8, 8, 128, True, None),     # 256 items
    (2, 300, 6, 2, 128, False, None),
    (1, 1000, 4, 1, 128, True, [300, 0, 1, 699]),
]
MORE = [
    (1, 300, 128, 128, 128, True, None),   # 384 items of each kind
    (2, 200, 160, 40, 128, False, None),   # 160 dK/dV items of four heads each, 640 of dQ
    (1, 260, 150, 150, 128, True, [1, 259]),
    (1, 1000, 80, 80, 64, True, None),     # 640 items of each kind
    (1, 1300, 80, 20, 64, False, None),
    (1, 500, 150, 150, 64, True, [1, 499]),
]
QUEUED = (1, 6400, 56, 14, 64, False, None)   # long bidirectional items of grouped heads


@pytest.mark.parametrize("B,S,Hq,Hkv,D,causal,lens", DEALT + [
    (4, 2000, 16, 16, 64, False, None),   # (several rounds, of which the call makes two launches as well)
])
def test_one_launch_gives_the_bits_of_two(B, S, Hq, Hkv, D, causal, lens):
    import torch
    from paper_2401_09149_amd import binding
    print(f"case B{B} S{S} Hq{Hq} Hkv{Hkv} D{D} {causal} {lens}", flush=True)
    dev, scale = "cuda:0", D ** -0.5
    q, do = (randn_bf16((B, S, Hq, D), 300 + j).to(dev) for j in range(2))
    k, v = (randn_bf16((B, S, Hkv, D), 302 + j).to(dev) for j in range(2))
    cu = None
    if lens:
        cu = torch.tensor([0] + lens, dtype=torch.int32).cumsum(0).to(torch.int32).to(dev)
    o, lse = binding.attn_fwd(q, k, v, scale, causal, cu)
    ws = binding.alloc_bwd_workspace(q, k, cu)
    want = [torch.full_like(t, float("nan")) for t in (q, k, v)]
    for phase in (binding.BWD_DELTA, binding.BWD_DQ, binding.BWD_DKDV):
        binding.ie_attn_bwd_phases(q, k, v, o, do, lse, *want, cu, scale, causal, ws, phase)
    for _ in range(2):
        got = [torch.full_like(t, float("nan")) for t in (q, k, v)]
        binding.ie_attn_bwd(q, k, v, o, do, lse, *got, cu, scale, causal, ws)
        torch.cuda.synchronize()
        for a, b in zip(got, want):
            assert torch.equal(a, b)


@pytest.mark.parametrize("B,S,Hq,Hkv,D,causal,lens", MORE)
def test_more_items_than_cus_in_one_launch(B, S, Hq, Hkv, D, causal, lens):
    """Dealt out by the hardware: all kv heads hold the same data, so every group of heads has to show the bits of the
    first, which is checked against the oracle."""
    import torch
    from paper_2401_09149_amd import binding
    print(f"case B{B} S{S} Hq{Hq} Hkv{Hkv} D{D} {causal} {lens}", flush=True)
    dev, g = "cuda:0", Hq // Hkv
    scale = D ** -0.5
    q1, do1 = (randn_bf16((B, S, g, D), 800 + j) for j in range(2))
    k1, v1 = (randn_bf16((B, S, 1, D), 802 + j) for j in range(2))
    q, k, v, do = (t.to(dev).repeat(1, 1, Hkv, 1) for t in (q1, k1, v1, do1))
    cu = None if lens is None else torch.tensor([0] + lens, dtype=torch.int32).cumsum(0).to(torch.int32).to(dev)
    o, lse = binding.attn_fwd(q, k, v, scale, causal, cu)
    got = [torch.full_like(t, float("nan")) for t in (q, k, v)]
    binding.ie_attn_bwd(q, k, v, o, do, lse, *got, cu, scale, causal, binding.alloc_bwd_workspace(q, k, cu))
    torch.cuda.synchronize()
    first = [t[:, :, :n] for t, n in zip((o, *got), (g, g, 1, 1))]
    for t, f in zip((o, *got), first):
        assert torch.equal(t, f.repeat(1, 1, Hkv, 1))
    ref = ora.attn_fwd_bwd(*(to64(t) for t in (q1, k1, v1, do1)), scale, causal, None if cu is None else np.asarray(cu.cpu()))
    compare_all((first[0], lse[:, :g], *first[1:]), ref, f"S{S} Hq{Hq}")


def test_queued_launch_gives_the_bits_of_two():
    import torch
    from paper_2401_09149_amd import binding
    B, S, Hq, Hkv, D, causal, _ = QUEUED
    dev, scale = "cuda:0", D ** -0.5
    q, do = (randn_bf16((B, S, Hq, D), 900 + j).to(dev) for j in range(2))
    k, v = (randn_bf16((B, S, Hkv, D), 902 + j).to(dev) for j in range(2))
    o, lse = binding.attn_fwd(q, k, v, scale, causal)
    ws = binding.alloc_bwd_workspace(q, k)
    want, got = ([torch.full_like(t, float("nan")) for t in (q, k, v)] for _ in range(2))
    for phase in (binding.BWD_DELTA, binding.BWD_DQ, binding.BWD_DKDV):
        binding.ie_attn_bwd_phases(q, k, v, o, do, lse, *want, None, scale, causal, ws, phase)
    binding.ie_attn_bwd(q, k, v, o, do, lse, *got, None, scale, causal, ws)
    torch.cuda.synchronize()
    for a, b in zip(got, want):
        assert torch.equal(a, b)
