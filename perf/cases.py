"""The work that users of this library have it do, as timed cases.

A case is a dict of plain values; `kind` says which entry points a pass goes through:

  train    one attention layer of a training step: forward, then the recompute backward (with
           `bias_grad` the backward that also returns the gradient of a learnable bias)
  forward  the forward pass alone (evaluation, long-context scoring)
  packed   a training step over sequences of different lengths packed along the token axis, each
           with the bias -ln(its own length)
  shared   a training step with fewer key/value heads than query heads
  append   new tokens at the end of a key/value sequence that is already there: one token
           (generation) or a chunk of them (chunked prompt processing)
  norm     the norm over the concatenated heads that follows attention in hybrid-norm blocks,
           forward and backward
"""
import math
import random

import torch

import paper_2409_04431_amd as sa

_DTYPES = {"bf16": torch.bfloat16, "fp32": torch.float32}


def _case(name, kind, dtype, B, H, N, d, **more):
    c = {"name": name, "kind": kind, "dtype": dtype, "B": B, "H": H, "N": N, "d": d}
    c.update(more)
    return c


def listed():
    return [
        # The precision path at its smallest, a numerical check of a model's layer: three launches
        # of a handful of workgroups, so latency is all there is.
        _case("fp32_small_train", "train", "fp32", 1, 2, 256, 64),
        # The precision path at an ordinary size with a ragged length.
        _case("fp32_causal_train", "train", "fp32", 2, 8, 1000, 128, causal=True),
        # Short ragged sequences in the [B, N, H, d] layout that projections produce: many small
        # heads, fixed costs per workgroup.
        _case("short_train", "train", "bf16", 32, 12, 250, 64, layout="bnhd"),
        # An image model's layer: B 4, H 12, 1024 tokens, d 64, values scaled by d^-1/2.
        _case("image_train", "train", "bf16", 4, 12, 1024, 64, scale=0.125),
        # The paper's kernel-benchmark shape (B 32, H 12, d 64) at 4096 causal tokens.
        _case("batch_causal_train", "train", "bf16", 32, 12, 4096, 64, causal=True),
        # The library's main workload: B 8, H 16, 4096 causal tokens, d 128.
        _case("causal_train", "train", "bf16", 8, 16, 4096, 128, causal=True),
        # Long sequences with ALiBi: H 32, 16384 causal tokens, d 128.
        _case("long_alibi_train", "train", "bf16", 1, 32, 16384, 128, causal=True, alibi=True),
        # Long-context scoring, forward only, the largest case: 65536 tokens, d 64.
        _case("long_forward", "forward", "bf16", 2, 8, 65536, 64, v_uniform=True),
        # A speech minibatch with dynamic batching: 24 sequences of 150 to 1600 frames, a bias per
        # sequence and its gradient.
        _case("packed_train", "packed", "bf16", 24, 8, 1600, 64, shortest=150, lengths_seed=3, bias_grad=True),
        # One key/value head for all query heads.
        _case("shared_kv_train", "shared", "bf16", 4, 16, 2048, 128, kv_heads=1, causal=True),
        # Generation: one new token per sequence against 4001 keys, ALiBi.
        _case("one_token", "append", "bf16", 8, 16, 1, 128, keys=4001, alibi=True),
        # The norm after the main workload's attention.
        _case("norm_train", "norm", "bf16", 8, 16, 4096, 128, norm="layer"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _batch(rng, heads, per_head, budget, most=64):
    """A batch size whose work stays within `budget`, at random between one and the largest such."""
    return _log_int(rng, 1, max(1, min(most, int(budget / (heads * per_head)))))


def draw(rng):
    """One more case of the ranges the listed ones stand for."""
    kind = rng.choice(["train", "train", "train", "train", "forward", "packed", "shared", "append", "append", "norm"])
    d = rng.choice([64, 128])
    H = rng.choice([2, 4, 8, 12, 16, 24, 32])
    c = {"kind": kind, "dtype": "bf16", "H": H, "d": d}
    elements = 1 << 26  # of one tensor
    if kind == "train":
        c["causal"], c["alibi"] = rng.random() < 0.6, rng.random() < 0.25
        c["bias_grad"] = rng.random() < 0.2
        c["layout"] = rng.choice(["bhnd", "bnhd"])
        if rng.random() < 0.25:
            c["dtype"] = "fp32"
            c["N"] = _log_int(rng, 64, 2048)
            c["B"] = _batch(rng, H, max(14.0 * c["N"] ** 2 * d / 6e10, c["N"] * d / elements), 1.0, 8)
        else:
            c["N"] = _log_int(rng, 64, 16384)
            if rng.random() < 0.4:
                c["N"] = max(64, c["N"] // 64 * 64)
            c["B"] = _batch(rng, H, max(14.0 * c["N"] ** 2 * d / 4e12, c["N"] * d / elements), 1.0)
        if c["alibi"]:
            c["bias_grad"] = False
    elif kind == "forward":
        c["causal"], c["alibi"] = rng.random() < 0.5, False
        c["N"] = _log_int(rng, 1024, 65536)
        c["B"] = _batch(rng, H, max(4.0 * c["N"] ** 2 * d / 8e12, c["N"] * d / elements), 1.0)
        c["H"] = H if c["N"] < 32768 else min(H, 8)
    elif kind == "packed":
        c["causal"] = rng.random() < 0.3
        c["N"] = _log_int(rng, 200, 4000)
        c["shortest"] = max(16, c["N"] // rng.choice([2, 4, 10]))
        c["B"] = rng.randint(4, max(4, min(48, 2 * elements // (H * d * c["N"]))))
        c["lengths_seed"] = rng.randrange(1000)
        c["bias_grad"] = rng.random() < 0.5
    elif kind == "shared":
        c["H"] = rng.choice([8, 16, 32])
        c["kv_heads"] = rng.choice([1, 1, 2, 4, 8])
        if c["kv_heads"] == c["H"]:
            c["kv_heads"] = 1
        c["causal"] = rng.random() < 0.8
        c["N"] = _log_int(rng, 256, 8192)
        c["B"] = _batch(rng, c["H"], max(14.0 * c["N"] ** 2 * d / 3e12, c["N"] * d / elements), 1.0, 16)
    elif kind == "append":
        c["alibi"] = rng.random() < 0.4
        if rng.random() < 0.6:  # generation
            c["N"], c["causal"] = 1, False
            c["keys"] = _log_int(rng, 200, 32768)
            c["B"] = _log_int(rng, 1, max(1, min(64, elements // (H * d * c["keys"]))))
        else:  # a chunk of a prompt behind a prefix
            c["N"], c["causal"] = _log_int(rng, 16, 1024), True
            c["keys"] = c["N"] + 32 * _log_int(rng, 4, 512)
            c["B"] = _log_int(rng, 1, max(1, min(8, elements // (H * d * c["keys"]))))
    else:
        c["norm"] = rng.choice(["layer", "rms"])
        c["layout"] = rng.choice(["bhnd", "bnhd"])
        c["N"] = _log_int(rng, 128, 16384)
        c["B"] = _batch(rng, H, c["N"] * d / elements, 1.0)
    return c


def _lengths(case):
    r = random.Random(case["lengths_seed"])
    n = [r.randint(case["shortest"], case["N"]) for _ in range(case["B"])]
    n[0] = case["N"]
    return n


def prepare(case, seed):
    """Inputs, biases and output buffers, as a training or serving program holds them."""
    kind, dt, dev = case["kind"], _DTYPES[case["dtype"]], "cuda"
    B, H, N, d = case["B"], case["H"], case["N"], case["d"]
    g = torch.Generator(device=dev).manual_seed(seed)
    scale = case.get("scale", 1.0)

    def rand(*shape, by=1.0):
        x = torch.randn(*shape, generator=g, device=dev)
        return (x * by if by != 1.0 else x).to(dt)

    def heads(n_heads, n, by=1.0):
        """[B, heads, n, d], or that view of a [B, n, heads, d] tensor."""
        if case.get("layout") == "bnhd":
            return rand(B, n, n_heads, d, by=by).transpose(1, 2)
        return rand(B, n_heads, n, d, by=by)

    s = {"case": case}
    if kind == "norm":
        s["x"], s["dy"] = heads(H, N, by=0.3), heads(H, N)
        s["y"], s["dx"] = torch.empty_like(s["x"]), torch.empty_like(s["x"])
        s["stats"] = torch.empty(B, N, 2, dtype=torch.float32, device=dev)
        return s
    if case.get("alibi"):
        s["slopes"] = torch.tensor([2.0 ** (-8.0 * (h + 1) / H) for h in range(H)], dtype=torch.float32, device=dev)
    if kind == "packed":
        n = _lengths(case)
        total = sum(n)
        s["q"], s["k"], s["v"], s["dout"] = (rand(total, H, d) for _ in range(4))
        s["cu"] = torch.tensor([sum(n[:i]) for i in range(B + 1)], dtype=torch.int32, device=dev)
        s["bias"] = torch.tensor([-math.log(x) for x in n], dtype=torch.float32, device=dev)
        rows, groups = (H, total), (B, H)
    else:
        n_keys, kv_heads = case.get("keys", N), case.get("kv_heads", H)
        s["q"] = heads(H, N, by=scale)
        s["k"] = heads(kv_heads, n_keys, by=scale)
        if case.get("v_uniform"):
            s["v"] = (torch.rand(B, kv_heads, n_keys, d, generator=g, device=dev) * 2.0 - 1.0).to(dt)
        else:
            s["v"] = heads(kv_heads, n_keys, by=scale)
        if kind in ("train", "shared"):
            s["dout"] = heads(H, N)
        s["bias"] = -math.log(n_keys)
        rows, groups = (B, H, N), (B, H)
    s["o"] = torch.empty_like(s["q"])
    if "dout" in s:
        s["dq"], s["dk"], s["dv"] = torch.empty_like(s["q"]), torch.empty_like(s["k"]), torch.empty_like(s["v"])
    if case.get("bias_grad"):
        s["db_rows"] = torch.empty(*rows, dtype=torch.float32, device=dev)
        s["db"] = torch.empty(*groups, dtype=torch.float32, device=dev)
    if kind == "shared":  # the workspace a training program allocates once
        need = sa.sigmoid_attn_mqa_bwd_workspace_bytes(B, H, case["kv_heads"], N, d, dt, case.get("causal", False))
        s["workspace"] = torch.empty(need, dtype=torch.uint8, device=dev) if need else None
    return s


def run(s):
    """One pass through the entry points; returns every output."""
    case = s["case"]
    kind, causal = case["kind"], case.get("causal", False)
    if kind == "norm":
        sa.sattn_headconcat_norm_fwd(s["x"], s["y"], s["stats"], kind=case["norm"])
        sa.sattn_headconcat_norm_bwd(s["x"], s["dy"], s["stats"], s["dx"], kind=case["norm"])
        return s["y"], s["stats"], s["dx"]
    q, k, v, o, bias, slopes = s["q"], s["k"], s["v"], s["o"], s["bias"], s.get("slopes")
    if kind == "forward":
        sa.sigmoid_attn_fwd(q, k, v, o, bias, causal, slopes)
        return o
    if kind == "append":
        sa.sigmoid_attn_cross_aligned_fwd(q, k, v, o, bias, causal, slopes)
        return o
    dout, dq, dk, dv = s["dout"], s["dq"], s["dk"], s["dv"]
    if kind == "packed":
        cu, n = s["cu"], case["N"]
        sa.sigmoid_attn_varlen_fwd(q, k, v, o, cu, n, 0.0, causal, slopes, bias_per_seq=bias)
        if case.get("bias_grad"):
            sa.sigmoid_attn_varlen_bwd_bias_grad(q, k, v, dout, dq, dk, dv, s["db_rows"], cu, n, 0.0, causal, slopes,
                                                 bias_per_seq=bias, db=s["db"])
            return o, dq, dk, dv, s["db_rows"], s["db"]
        sa.sigmoid_attn_varlen_bwd(q, k, v, dout, dq, dk, dv, cu, n, 0.0, causal, slopes, bias_per_seq=bias)
        return o, dq, dk, dv
    if kind == "shared":
        sa.sigmoid_attn_mqa_fwd(q, k, v, o, bias, causal, slopes)
        sa.sigmoid_attn_mqa_bwd_split(q, k, v, dout, dq, dk, dv, bias, causal, slopes, workspace=s["workspace"])
        return o, dq, dk, dv
    sa.sigmoid_attn_fwd(q, k, v, o, bias, causal, slopes)
    if case.get("bias_grad"):
        sa.sigmoid_attn_bwd_bias_grad(q, k, v, dout, dq, dk, dv, s["db_rows"], bias, causal, slopes, db=s["db"])
        return o, dq, dk, dv, s["db_rows"], s["db"]
    sa.sigmoid_attn_bwd(q, k, v, dout, dq, dk, dv, bias, causal, slopes)
    return o, dq, dk, dv


def work(case):
    """Two (forward) and five (backward) products of 2 d flops per unmasked pair; every input read
    once, every output written once."""
    kind, B, H, N, d = case["kind"], case["B"], case["H"], case["N"], case["d"]
    size = 2 if case["dtype"] == "bf16" else 4
    if kind == "norm":
        return {"bytes": B * N * (4.0 * H * d * size + 8), "flops": 20.0 * B * N * H * d}
    causal = case.get("causal", False)
    if kind == "packed":
        lengths = _lengths(case)
        pairs = H * sum(n * (n + 1) / 2 if causal else n * n for n in lengths)
        q_el = kv_el = H * d * sum(lengths)
    else:
        n_keys = case.get("keys", N)
        pairs = B * H * (N * (n_keys - N) + N * (N + 1) / 2 if causal else N * n_keys)
        q_el, kv_el = B * H * N * d, B * case.get("kv_heads", H) * n_keys * d
    forward_only = kind in ("forward", "append")
    tensors = 2 * q_el + 2 * kv_el if forward_only else 4 * q_el + 4 * kv_el
    more = 4.0 * q_el / d if case.get("bias_grad") else 0.0
    return {"bytes": float(tensors * size) + more, "flops": (4.0 if forward_only else 14.0) * pairs * d}


def tolerance(case):
    """Four times what the results differ by from the same sums in 64 bits (relative 2-norm, largest
    difference over the root mean square): 2.4e-3 and 2e-2 in bf16, where P, dS and the results are
    rounded to bf16; 6.7e-7 and 9e-6 in fp32 at 1000 tokens, a little more at 2048."""
    if case["dtype"] == "fp32":
        return {"rel": 4e-6, "max": 5e-5}
    return {"rel": 1e-2, "max": 8e-2}
