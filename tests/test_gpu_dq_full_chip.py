"""Head dimension 128 with items for every CU: the launches whose dQ runs on 16x16x32 products and whose dK/dV has a kernel
of its own, at the edges that the small parity cases (one launch for both, 32x32x16 products) reach only there: one-row
tails, ragged causal and bidirectional lengths, grouped heads, empty and one-token documents, large scores, outlier keys.
All heads run; the first and the last kv head are compared with the fp64 oracle element by element.  Tolerances are
parity_util's; the two wider ones are those of the same cases in test_gpu_parity_small, with their reasons there: dq and dk
carry the factor `scale` or the outliers' magnitude."""
import numpy as np
import pytest

from parity_util import TOL_GRAD_ABS, compare_all, randn_bf16, run_gpu, to64

pytestmark = pytest.mark.gpu

CASES = {   # B, S, Hq, Hkv, causal, document lengths
    "one_row_tail": (1, 1025, 64, 64, True, None),
    "ragged_causal_grouped": (2, 1029, 32, 16, True, None),
    "ragged_bidirectional_grouped": (2, 1029, 24, 8, False, None),
    "short_bidirectional": (4, 130, 64, 16, False, None),
    "whole_tiles_bidirectional": (1, 1280, 48, 48, False, None),
    "large_scores": (1, 1153, 64, 64, True, None),
    "outlier_keys": (1, 1300, 64, 64, True, None),
    "packed": (1, 8300, 16, 8, True, [300, 0, 1, 699, 2048, 129, 0, 127, 256, 1, 2500, 2239]),
}


@pytest.mark.parametrize("name", CASES)
def test_dq_full_chip(oracle, name):
    from paper_2401_09149_amd import binding
    B, S, Hq, Hkv, causal, lens = CASES[name]
    print("case", name, CASES[name], flush=True)
    seed = 900 + sorted(CASES).index(name) * 4
    q, do = randn_bf16((B, S, Hq, 128), seed), randn_bf16((B, S, Hq, 128), seed + 1)
    k, v = randn_bf16((B, S, Hkv, 128), seed + 2), randn_bf16((B, S, Hkv, 128), seed + 3)
    scale, widen = 128 ** -0.5, 1
    if name == "large_scores":
        scale, widen = 4 * scale, 4
    if name == "outlier_keys":
        k = k.float()
        k[:, 700] *= 12.0
        k[:, 1000] *= 30.0
        k, widen = k.to(q.dtype), 30
    cu = None if lens is None else np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    group = Hq // Hkv
    refs = {}
    for g in (0, Hkv - 1):
        hs = slice(g * group, (g + 1) * group)
        refs[g] = oracle.attn_fwd_bwd(to64(q[:, :, hs]), to64(k[:, :, g:g + 1]), to64(v[:, :, g:g + 1]), to64(do[:, :, hs]),
                                      scale, causal, cu)
    try:
        for rows in (0, 256, 128):   # the sizes' own choice, and both sizes of a work item
            binding.ie_attn_set_tile_rows(rows)
            o, lse, dq, dk, dv = run_gpu(q, k, v, do, scale, causal, cu)
            for g, ref in refs.items():
                hs = slice(g * group, (g + 1) * group)
                compare_all((o[:, :, hs], lse[:, hs], dq[:, :, hs], dk[:, :, g:g + 1], dv[:, :, g:g + 1]), ref,
                            f"{name} kv head {g} rows{rows}", grad_abs_tol=widen * TOL_GRAD_ABS)
    finally:
        binding.ie_attn_set_tile_rows(0)
