"""The forward kernel of one hand-sequenced wave per SIMD (attn_fwd_seq_kernel) at its edges: lengths around its 32-key
blocks, 64-key tiles, the four stages of its ring and its 128-row items, against the oracle.  Calls of these sizes take it
by fwd128_route (csrc/dispatch.hpp), which tests/test_dispatch_rules.py checks.  And scores far below and far above the
others of their row, in all forward kernels."""
import numpy as np
import pytest
from oracle import attention as ora

from parity_util import TOL_LSE, TOL_O, compare_all, randn_bf16, to64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,S,Hq,Hkv,causal,lens", [
    *((1, s, 2, 1, c, None) for s in (385, 415, 416, 447, 449, 480, 511, 512, 513, 577, 639, 641) for c in (True,)),
    *((1, s, 2, 1, False, None) for s in (897, 929, 960, 991, 1023, 1024, 1025)),
    (2, 700, 3, 3, True, None),
    (1, 1100, 4, 2, False, None),
    (1, 2500, 2, 2, True, [1, 33, 66, 2400]),
    (1, 2300, 2, 1, False, [64, 2200, 0, 36]),
])
def test_against_the_oracle(B, S, Hq, Hkv, causal, lens):
    import torch
    from paper_2401_09149_amd import binding
    print(f"case B{B} S{S} Hq{Hq} Hkv{Hkv} {causal} {lens}", flush=True)
    dev, D = "cuda:0", 128
    # scores from small to far beyond the first block's: blocks that are done again are among them
    q, k, v = (randn_bf16((B, S, h, D), 950 + j) for j, h in enumerate((Hq, Hkv, Hkv)))
    k = (k.float() * torch.linspace(0.2, 6.0, S).view(1, S, 1, 1)).to(torch.bfloat16)
    cu = None if lens is None else torch.tensor([0] + lens, dtype=torch.int32).cumsum(0).to(torch.int32)
    o, lse = binding.attn_fwd(q.to(dev), k.to(dev), v.to(dev), D ** -0.5, causal, None if cu is None else cu.to(dev))
    torch.cuda.synchronize()
    ro, rlse = ora.attn_fwd(to64(q), to64(k), to64(v), D ** -0.5, causal, None if cu is None else np.asarray(cu))
    # With scores as large as these a row is nearly one key's, and o nearly a value vector (up to 4.6 here).  bf16 rounds to
    # within 2^-8 of a number: the probabilities cost 2^-8 max|v|, the result 2^-8 |o|; 1e-3 for the sums.
    assert (np.abs(to64(o) - ro) <= 2.0 ** -8 * (np.abs(to64(v)).max() + np.abs(ro)) + 1e-3).all()
    assert np.abs(to64(lse) - rlse).max() <= TOL_LSE * max(1.0, np.abs(rlse).max() / 8)   # (fp32: relative for large sums)


@pytest.mark.parametrize("rows", [0, 128, 256])
@pytest.mark.parametrize("S,causal", [(640, True), (1024, False)])
def test_scores_that_overflow_downwards(S, causal, rows):
    """Keys whose fp32 scores are -inf, among finite ones of every row's first block and in both halves of the wave that holds
    them: probability 0, and nothing else changes.  rows 0 takes the hand-sequenced kernel (tests/test_dispatch_rules.py), 128
    and 256 the others."""
    import torch
    from paper_2401_09149_amd import binding
    print(f"case S{S} {causal} rows {rows}", flush=True)
    dev, D, H = "cuda:0", 128, 2
    q, k, v = (randn_bf16((1, S, H, D), 970 + j) for j in range(3))
    q[..., 0], k[..., 0] = 2.0 ** 100, 0.0
    for key in (2, 5, 40, 300):   # (keys 0 to 3 and 4 to 7 lie in different halves)
        k[:, key, :, 0] = -(2.0 ** 100)
    before = binding.ie_attn_set_tile_rows(rows)
    try:
        o, lse = binding.attn_fwd(q.to(dev), k.to(dev), v.to(dev), D ** -0.5, causal)
        torch.cuda.synchronize()
    finally:
        binding.ie_attn_set_tile_rows(before)
    ro, rlse = ora.attn_fwd(to64(q), to64(k), to64(v), D ** -0.5, causal)
    assert np.abs(to64(o) - ro).max() <= TOL_O
    assert np.abs(to64(lse) - rlse).max() <= TOL_LSE


LAZY_64 = [(513, 160, True, None), (641, 60, False, None), (1500, 66, True, None),   # (1500 x 66 also in flipped order)
           (1500, 64, True, [1, 65, 330, 1104]), (1500, 52, False, [64, 1400, 0, 36])]
SEARCHING_64 = [(513, 2, True, None), (641, 3, False, None), (1500, 2, True, [1, 65, 330, 1104])]


@pytest.mark.parametrize("S,H,causal,lens", LAZY_64 + SEARCHING_64)
def test_blocks_beyond_the_reference_at_head_dimension_64(S, H, causal, lens):
    """Scores far above those of their row's first block at head dimension 64, where launches of many items (LAZY_64) take
    unmasked blocks against the maximum that is there, and again where a lane's sum passes 2^24: keys grow along the
    sequence, so that it does.  All heads hold the same data and have to show the bits of the first."""
    import torch
    from paper_2401_09149_amd import binding
    print(f"case S{S} H{H} {causal} {lens}", flush=True)
    dev, D = "cuda:0", 64
    q, k, v = (randn_bf16((1, S, 1, D), 980 + j) for j in range(3))
    k = (k.float() * torch.linspace(0.2, 14.0, S).view(1, S, 1, 1)).to(torch.bfloat16)
    cu = None if lens is None else torch.tensor([0] + lens, dtype=torch.int32).cumsum(0).to(torch.int32)
    # scores of the last query (of the longest document, without the last 128 keys, where masks are) against its first block's
    end, n = (S, S) if lens is None else (int(cu[lens.index(max(lens)) + 1]), max(lens))
    s = to64(k)[0, end - n:end - 128, 0] @ to64(q)[0, end - 1, 0] * D ** -0.5 / np.log(2.0)
    assert s.max() > s[:32].max() + 24
    o, lse = binding.attn_fwd(*(t.to(dev).repeat(1, 1, H, 1) for t in (q, k, v)), D ** -0.5, causal, None if cu is None else cu.to(dev))
    torch.cuda.synchronize()
    assert torch.equal(o, o[:, :, :1].expand_as(o)) and torch.equal(lse, lse[:, :1].expand_as(lse))
    ro, rlse = ora.attn_fwd(to64(q), to64(k), to64(v), D ** -0.5, causal, None if cu is None else np.asarray(cu))
    # (the bounds of test_against_the_oracle, for the same reason)
    assert (np.abs(to64(o[:, :, :1]) - ro) <= 2.0 ** -8 * (np.abs(to64(v)).max() + np.abs(ro)) + 1e-3).all()
    assert np.abs(to64(lse[:, :1]) - rlse).max() <= TOL_LSE * max(1.0, np.abs(rlse).max() / 8)


@pytest.mark.parametrize("D", [64, 128])
def test_items_in_the_opposite_order(D):
    """Launches that run the second item on each CU in the opposite order (fwd_flips in csrc/dispatch.hpp) do the same items
    as launches of fewer heads, which do not."""
    import torch
    from paper_2401_09149_amd import binding
    dev, S, H = "cuda:0", 1100, 60
    q, k, v = (randn_bf16((1, S, H, D), 990 + j).to(dev) for j in range(3))
    before = binding.ie_attn_set_tile_rows(128)
    try:
        o, lse = binding.attn_fwd(q, k, v, D ** -0.5, True)
        parts = [binding.attn_fwd(*(t[:, :, h:h + 20].contiguous() for t in (q, k, v)), D ** -0.5, True) for h in (0, 20, 40)]
        torch.cuda.synchronize()
    finally:
        binding.ie_attn_set_tile_rows(before)
    assert torch.equal(o, torch.cat([a for a, _ in parts], 2)) and torch.equal(lse, torch.cat([b for _, b in parts], 1))


MANY_HEADS = [   # S, heads of all batch entries, D, causal, backward, heads, heads per kv head, tiles per head that go head by head
    (129, 520, 64, False, False, 8, 1, 2), (200, 264, 128, False, True, 8, 1, 2), (384, 400, 128, False, True, 8, 1, 3),   # lists, all tiles
    (300, 688, 128, True, False, 8, 1, 3), (641, 352, 128, True, False, 8, 1, 5), (513, 624, 64, True, False, 8, 1, 5),    # odd shares
    (129, 521, 64, False, False, 1, 1, 0), (200, 265, 128, False, True, 5, 1, 0),   # one list of heads, tile by tile
    (641, 351, 128, True, False, 3, 1, 5), (1152, 86, 64, False, False, 2, 1, 9), (513, 309, 128, False, True, 3, 1, 5),   # one list, head by head
    (256, 1537, 128, False, False, 1, 1, 2),
    (129, 520, 64, False, False, 8, 4, 2), (384, 400, 128, False, True, 8, 2, 3), (641, 352, 128, True, False, 8, 4, 5),   # grouped heads
    (641, 354, 128, True, False, 6, 3, 5), (1152, 86, 64, False, False, 2, 2, 9),
    (400, 196, 128, False, False, 4, 4, 4), (140, 2816, 128, False, False, 8, 1, 2),   # grouped in one list; more K and V than caches hold
]


@pytest.mark.parametrize("S,heads,D,causal,backward,H,group,share", MANY_HEADS)
def test_many_heads_in_head_by_head_order(S, heads, D, causal, backward, H, group, share):
    """Launches of many heads (fwd_head_by_head in csrc/dispatch.hpp; bidirectional at head dimension 128 the shared backward
    launch too): the batch repeats two entries, of which the first two are compared with the oracle and the others, bit for
    bit, with those two: every item has run, for its own rows."""
    import torch
    from paper_2401_09149_amd import binding
    print(f"case S{S} heads {heads} D{D} {causal} H{H} group {group}", flush=True)
    dev, U = "cuda:0", 2
    B = heads // H
    small = [randn_bf16((U, S, H if j in (0, 3) else H // group, D), 990 + j) for j in range(4)]
    q, k, v, do = (x.to(dev).repeat((B + 1) // U, 1, 1, 1)[:B].contiguous() for x in small)
    o, lse = binding.attn_fwd(q, k, v, D ** -0.5, causal)
    got = (o, lse) + (binding.attn_bwd(q, k, v, o, do, lse, D ** -0.5, causal) if backward else ())
    torch.cuda.synchronize()
    for t in got:
        for u in range(U):
            assert torch.equal(t[u::U], t[u:u + 1].expand_as(t[u::U]))
    if backward:
        compare_all([t[:U] for t in got], ora.attn_fwd_bwd(*(to64(x) for x in small), D ** -0.5, causal))
    else:
        ro, rlse = ora.attn_fwd(*(to64(x) for x in small[:3]), D ** -0.5, causal)
        assert np.abs(to64(o[:U]) - ro).max() <= TOL_O and np.abs(to64(lse[:U]) - rlse).max() <= TOL_LSE
