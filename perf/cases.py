"""The work that a training or evaluation program has this package do, as cases that can be timed and compared.

Three kinds, each through the package's public calls:
  attn    autograd.attention forward and backward (`train`), or binding.attn_fwd alone (evaluation, prefill,
          activation recomputation);
  linear  the four linear modules of a Transformer layer (QKV, output, gate/up, down) on M tokens through
          autograd.linear: forward and both gradients (`train`), or the forward products alone;
  sp      the eight local re-layouts either side of the sequence-parallel all-to-alls of one layer.

listed() is a fixed selection, draw(rng) gives more of the same ranges.  bf16 throughout, as the package takes it."""
import math
import random

import torch

from paper_2401_09149_amd import autograd, binding

DEV = "cuda:0"


def _attn(name, B, S, Hq, Hkv, D, causal=True, train=True, stored_ds=False, doc_min=0, doc_max=0, doc_seed=0):
    """doc_max > 0: S tokens of packed documents of log-uniform lengths doc_min .. doc_max (B = 1)."""
    return {"name": name, "kind": "attn", "B": B, "S": S, "Hq": Hq, "Hkv": Hkv, "D": D, "causal": causal, "train": train,
            "stored_ds": stored_ds, "doc_min": doc_min, "doc_max": doc_max, "doc_seed": doc_seed}


def _linear(name, M, hidden, mlp, train):
    return {"name": name, "kind": "linear", "M": M, "hidden": hidden, "mlp": mlp, "train": train}


def _sp(name, B, Sl, Hq, Hkv, D, P):
    return {"name": name, "kind": "sp", "B": B, "Sl": Sl, "Hq": Hq, "Hkv": Hkv, "D": D, "P": P}


def listed():
    return [
        # The smallest configuration: a few workgroups per kernel, so launches, host work and latency are what counts.
        _attn("attn_train_s512_h2_d64", 1, 512, 2, 2, 64),
        # Evaluation or prefill of one prompt of ordinary, odd length; grouped kv heads; forward only.
        _attn("attn_fwd_s3001_q32kv8_d128", 1, 3001, 32, 8, 128, train=False),
        # The short-sequence plan of 7B: 4096 tokens, two sequences, all heads on one GPU.
        _attn("attn_train_b2_s4096_h32_d128", 2, 4096, 32, 32, 128),
        # 8192 tokens with sequence parallelism of degree 8: few heads per GPU, fewer work items than a full chip wants.
        _attn("attn_train_s8192_h8_d128", 1, 8192, 8, 8, 128),
        # The headline configuration: 7B at 32K tokens, all heads.
        _attn("attn_train_s32768_h32_d128", 1, 32768, 32, 32, 128),
        # Grouped-query attention of a long sequence, one kv head per GPU.
        _attn("attn_train_s65536_q8kv1_d128", 1, 65536, 8, 1, 128),
        # Documents of very different lengths packed into one sequence.
        _attn("attn_train_packed_s65536_h8_d128", 1, 65536, 8, 8, 128, doc_min=256, doc_max=16384, doc_seed=1),
        # Bidirectional attention with small heads over a batch of ragged length.
        _attn("attn_train_b4_s2000_h16_d64_full", 4, 2000, 16, 16, 64, causal=False),
        # The backward option that trades workspace for matrix work.
        _attn("attn_train_s16384_h16_d128_stored_ds", 1, 16384, 16, 16, 128, stored_ds=True),
        # One layer's linear modules of 7B on one GPU's share of the tokens: forward and both gradients.
        _linear("linear_train_m8192_h4096", 8192, 4096, 11008, True),
        # The same modules on a short prompt of odd length (evaluation): the weights are most of the bytes.
        _linear("linear_fwd_m200_h4096", 200, 4096, 11008, False),
        # All re-layouts of one layer: 7B at 32K tokens over four GPUs.
        _sp("sp_b1_sl8192_h32_d128_p4", 1, 8192, 32, 32, 128, 4),
    ]


def _size(rng, lo, hi, step=1):
    """A multiple of `step`, spread over the logarithm of lo .. hi."""
    x = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(x / step)) * step))


def _draw_attn(rng):
    variant = rng.choices(["dense", "packed", "d64", "stored_ds"], [5, 2, 2, 1])[0]
    if variant == "dense":
        S = _size(rng, 256, 65536)
        group = rng.choice([1, 1, 1, 2, 4, 8])
        room = max(1, int(16 * 32768 ** 2 / S ** 2))   # (batch entries x heads: half the headline configuration's work at most)
        Hkv = max(1, min(rng.randint(1, 40), 64, room) // group)
        B = rng.choice([1, 1, 2, 4])
        B = B if B * Hkv * group <= room else 1
        c = _attn("", B, S, Hkv * group, Hkv, 128, causal=rng.random() < 0.85, train=rng.random() < 0.7)
    elif variant == "packed":
        S = _size(rng, 2048, 65536)
        heads, group = rng.randint(1, 8), rng.choice([1, 1, 4])
        lo = _size(rng, 64, 512)
        c = _attn("", 1, S, heads * group if S <= 16384 else heads, heads, 128, train=rng.random() < 0.8, doc_min=lo,
                  doc_max=_size(rng, 2 * lo, max(4 * lo, min(S, 16384))), doc_seed=rng.randint(0, 1 << 20))
    elif variant == "d64":
        group = rng.choice([1, 1, 2])
        S = _size(rng, 128, 8192)
        Hkv = rng.randint(1, 16)
        B = max(1, min(4, 4096 * 8 // S))
        c = _attn("", B, S, Hkv * group, Hkv, 64, causal=rng.random() < 0.5, train=rng.random() < 0.8)
    else:
        S = _size(rng, 1024, 16384, 128)
        c = _attn("", 1, S, 0, 0, 128, stored_ds=True)
        c["Hq"] = c["Hkv"] = rng.randint(1, 16 if S > 8192 else 32)
    return c


def _draw_linear(rng):
    hidden = _size(rng, 512, 8192, 64)
    mlp = 64 * int(hidden * rng.uniform(2.0, 4.0) / 64)
    if rng.random() < 0.5:
        return _linear("", _size(rng, 64, 16384 if hidden <= 4096 else 8192, 64), hidden, mlp, True)
    return _linear("", _size(rng, 1, 8192), hidden, mlp, False)


def _draw_sp(rng):
    P = rng.choice([2, 4, 8, 16, 32])
    group = rng.choice([1, 1, 2, 4])
    Hkv = P * rng.randint(1, max(1, 64 // (P * group)))
    D = rng.choice([64, 128, 128])
    B = rng.choice([1, 1, 2])
    Sl = _size(rng, 64, max(128, 8192 * 32 * 128 // (B * Hkv * group * D)))
    return _sp("", B, Sl, Hkv * group, Hkv, D, P)


def draw(rng):
    c = rng.choices([_draw_attn, _draw_linear, _draw_sp], [5, 3, 1])[0](rng)
    del c["name"]
    return c


def _doc_lengths(case):
    """Document lengths of a packed case: log-uniform, the last one cut to fill S tokens exactly."""
    rng, out, left = random.Random(case["doc_seed"]), [], case["S"]
    while left > 0:
        n = min(left, int(round(math.exp(rng.uniform(math.log(case["doc_min"]), math.log(case["doc_max"]))))))
        out.append(n)
        left -= n
    return out


def _modules(case):
    """(outputs, inputs) of the layer's linear modules."""
    h, m = case["hidden"], case["mlp"]
    return [(3 * h, h), (h, h), (2 * m, h), (h, m)]


def _randn(gen, shape, std=1.0):
    return torch.randn(shape, generator=gen, device=DEV, dtype=torch.float32).mul_(std).to(torch.bfloat16)


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    s = {"case": case}
    if case["kind"] == "attn":
        B, S, Hq, Hkv, D = (case[k] for k in ("B", "S", "Hq", "Hkv", "D"))
        s["q"] = _randn(gen, (B, S, Hq, D))
        s["k"], s["v"] = _randn(gen, (B, S, Hkv, D)), _randn(gen, (B, S, Hkv, D))
        s["cu"] = None
        if case["doc_max"]:
            lengths = _doc_lengths(case)
            random.Random(seed).shuffle(lengths)   # other inputs: the same documents in another order
            offsets = [0]
            for n in lengths:
                offsets.append(offsets[-1] + n)
            s["cu"] = torch.tensor(offsets, dtype=torch.int32, device=DEV)
        if case["train"]:
            for k in ("q", "k", "v"):
                s[k].requires_grad_(True)
            s["dout"] = _randn(gen, (B, S, Hq, D))
            # one workspace for all layers, as a training program keeps it
            s["workspace"] = binding.alloc_bwd_workspace(s["q"], s["k"], s["cu"], fast=case["stored_ds"], causal=case["causal"])
    elif case["kind"] == "linear":
        M = case["M"]
        s["x"] = [_randn(gen, (M, k)) for _, k in _modules(case)]
        s["w"] = [_randn(gen, (n, k), k ** -0.5) for n, k in _modules(case)]
        if case["train"]:
            for t in s["x"] + s["w"]:
                t.requires_grad_(True)
            s["dy"] = [_randn(gen, (M, n)) for n, _ in _modules(case)]
    else:
        B, Sl, Hq, Hkv, D, P = (case[k] for k in ("B", "Sl", "Hq", "Hkv", "D", "P"))
        nq, nk = B * Sl * Hq * D, B * Sl * Hkv * D
        new = lambda n: torch.empty(n, dtype=torch.bfloat16, device=DEV)  # noqa: E731
        # what the projections, the attention calls and the exchanges hand over, and the buffers that receive the result
        s["qkv_local"], s["recv_qkv"], s["recv_dqkv"] = (_randn(gen, nq + 2 * nk) for _ in range(3))
        s["o"], s["recv_o"], s["dout_local"], s["recv_do"], s["dq"] = (_randn(gen, nq) for _ in range(5))
        s["dk"], s["dv"] = (_randn(gen, nk) for _ in range(2))
        s["send_qkv"], s["send_dqkv"], s["dqkv_local"] = (new(nq + 2 * nk) for _ in range(3))
        s["q"], s["send_o"], s["o_local"], s["send_do"], s["dout"] = (new(nq) for _ in range(5))
        s["k"], s["v"] = new(nk), new(nk)
    return s


def run(s):
    case = s["case"]
    if case["kind"] == "attn":
        scale = case["D"] ** -0.5
        if not case["train"]:
            return binding.attn_fwd(s["q"], s["k"], s["v"], scale, case["causal"], s["cu"])
        o = autograd.attention(s["q"], s["k"], s["v"], scale, case["causal"], s["cu"], workspace=s["workspace"], stored_ds=case["stored_ds"])
        return (o,) + torch.autograd.grad(o, (s["q"], s["k"], s["v"]), s["dout"])
    if case["kind"] == "linear":
        out = []
        if not case["train"]:
            with torch.no_grad():
                return [autograd.linear(x, w) for x, w in zip(s["x"], s["w"])]
        for x, w, dy in zip(s["x"], s["w"], s["dy"]):
            y = autograd.linear(x, w)
            out.append((y,) + torch.autograd.grad(y, (x, w), dy))
        return out
    shape_qkv = tuple(case[k] for k in ("B", "Sl", "Hq", "Hkv", "D", "P"))
    shape_o = tuple(case[k] for k in ("B", "Sl", "Hq", "D", "P"))
    binding.ie_sp_pack_qkv(s["qkv_local"], s["send_qkv"], *shape_qkv)
    binding.ie_sp_unpack_qkv(s["recv_qkv"], s["q"], s["k"], s["v"], *shape_qkv)
    binding.ie_sp_pack_o(s["o"], s["send_o"], *shape_o)
    binding.ie_sp_unpack_o(s["recv_o"], s["o_local"], *shape_o)
    binding.ie_sp_pack_do(s["dout_local"], s["send_do"], *shape_o)
    binding.ie_sp_unpack_do(s["recv_do"], s["dout"], *shape_o)
    binding.ie_sp_pack_dqkv(s["dq"], s["dk"], s["dv"], s["send_dqkv"], *shape_qkv)
    binding.ie_sp_unpack_dqkv(s["recv_dqkv"], s["dqkv_local"], *shape_qkv)
    return {k: s[k] for k in ("send_qkv", "q", "k", "v", "send_o", "o_local", "send_do", "dout", "send_dqkv", "dqkv_local")}


def work(case):
    if case["kind"] == "attn":
        B, S, Hq, Hkv, D = (case[k] for k in ("B", "S", "Hq", "Hkv", "D"))
        lengths = _doc_lengths(case) if case["doc_max"] else [S] * B
        pairs = sum(n * (n + 1) // 2 if case["causal"] else n * n for n in lengths)   # visible (query, key) pairs of one head
        nq, nk = B * S * Hq * D, B * S * Hkv * D
        if not case["train"]:
            return {"bytes": 2 * (2 * nq + 2 * nk) + 4 * B * S * Hq, "flops": 4.0 * D * Hq * pairs}
        # forward: two products, backward: five; q, dout, k, v in, o, dq, dk, dv out
        return {"bytes": 2 * (4 * nq + 4 * nk), "flops": 14.0 * D * Hq * pairs}
    if case["kind"] == "linear":
        M, nbytes, flops = case["M"], 0, 0.0
        for n, k in _modules(case):
            once = 2 * (M * k + n * k + M * n)
            nbytes += 2 * once if case["train"] else once   # x, w, dy in; y, dx, dw out
            flops += (6.0 if case["train"] else 2.0) * M * n * k
        return {"bytes": nbytes, "flops": flops}
    nq, nk = (case["B"] * case["Sl"] * case[h] * case["D"] for h in ("Hq", "Hkv"))
    return {"bytes": 2 * 2 * (4 * (nq + 2 * nk) + 4 * nq), "flops": 0}


def tolerance(case):
    if case["kind"] == "sp":
        return "exact"   # copies
    if case["kind"] == "linear":
        # fp32 accumulation and one rounding to bf16: results of another summation order differ where the rounding flips.
        # Against float64 results rounded once: up to 6.3e-5 and one last place, 7.8e-3.
        return {"rel": 3e-4, "max": 3.2e-2}
    # bf16 probabilities and score gradients between the products, bf16 results: 2.0e-3 to 2.5e-3 and up to 0.1 against
    # float64 (512 to 8192 tokens, both head dimensions, packed, grouped and bidirectional).
    return {"rel": 1e-2, "max": 0.4}
