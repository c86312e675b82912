"""Performance cases of the library: the calls that a MosaicBERT-style training or serving program makes, one layer
step each, through `paper_2312_17482_amd.binding`.

Kinds of cases ("kind"):
  step    one attention layer the explicit way: index maps -> gather QKV -> forward -> gather dO -> backward -> scatter
          of O and of dQKV, on a padded batch; every buffer is the program's own and lives as long as it does
  rows    the same layer with the gather and scatter done by the attention calls themselves (token_rows)
  packed  attention forward + backward on packed sequences, the work plan built once per batch as for a whole encoder
  masked  attention forward + backward over the padded batch with a key-padding mask, no unpadding
  generic packed attention forward + backward in the combinations without a matrix-core kernel (fp32, other head sizes)
  norm    residual add + LayerNorm, forward + backward
  geglu   the GeGLU feed-forward, forward + backward (projections computed again in the backward)
  linear  a bias-free projection of selected token rows: gather of the rows + projection (the masked-token head, or
          with every row selected the QKV / output projections)

Sequence lengths belong to the case (recipe "lengths", drawn with "lengths_seed"); the run's seed shuffles their order
and draws every value.
"""
import math
import random

import numpy as np
import torch

BF16, F32 = torch.bfloat16, torch.float32


def listed():
    return [
        # a small fine-tuning or serving batch: eight sequences; launches and latency are the whole of it
        {"name": "step_small", "kind": "step", "B": 8, "L": 128, "H": 12, "lengths": "mix60", "lengths_seed": 1},
        # the pretraining microbatch of the base model, the workload bench.py reports
        {"name": "step_base", "kind": "step", "B": 256, "L": 128, "H": 12, "lengths": "mix60", "lengths_seed": 2},
        # the large model's microbatch, reading and writing the padded batch directly
        {"name": "rows_large", "kind": "rows", "B": 256, "L": 128, "H": 16, "lengths": "mix60", "lengths_seed": 3},
        # medium sequences, uniformly ragged
        {"name": "packed_512", "kind": "packed", "B": 64, "L": 512, "H": 12, "lengths": "uniform64",
         "lengths_seed": 4},
        # documents of very different length, a few long ones
        {"name": "packed_ragged", "kind": "packed", "B": 16, "L": 2048, "H": 16, "lengths": "lognormal",
         "lengths_seed": 5},
        # long-context training with every position used
        {"name": "packed_full", "kind": "packed", "B": 16, "L": 2048, "H": 16, "lengths": "full", "lengths_seed": 6},
        # a program that keeps its padded batch and passes the padding mask
        {"name": "masked_512", "kind": "masked", "B": 64, "L": 512, "H": 12, "lengths": "mix60", "lengths_seed": 7},
        # fp32 fine-tuning or validation of a small batch
        {"name": "fp32_256", "kind": "generic", "B": 16, "L": 256, "H": 12, "D": 64, "dtype": "f32",
         "lengths": "mix60", "lengths_seed": 8},
        # Add & Norm of the pretraining microbatch's real tokens
        {"name": "norm_base", "kind": "norm", "T": 26963, "W": 768, "dtype": "bf16"},
        # feed-forward of a small batch: few row tiles
        {"name": "geglu_small", "kind": "geglu", "T": 945, "hidden": 768, "inter": 3072},
        # feed-forward of the pretraining microbatch
        {"name": "geglu_base", "kind": "geglu", "T": 26963, "hidden": 768, "inter": 3072},
        # masked-token head: 30 % of the microbatch's tokens onto the vocabulary
        {"name": "linear_vocab", "kind": "linear", "T": 26963, "rows": 8089, "n_in": 768, "n_out": 30528},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "rows", "packed", "packed", "masked", "generic", "norm", "geglu", "linear"])
    ls = rng.randrange(1 << 20)
    if kind in ("step", "rows"):
        # up to the single-tile length and past it, 32768 positions at most
        L = rng.choice([64, 97, 120, 128, 128, 128, 200, 256])
        B = _log_int(rng, 4, 32768 // L)
        return {"kind": kind, "B": B, "L": L, "H": rng.choice([4, 8, 12, 12, 16]), "lengths": "mix60",
                "lengths_seed": ls}
    if kind in ("packed", "masked"):
        L = _log_int(rng, 130, 2048)
        B = _log_int(rng, 1, max(1, 32768 // L))
        return {"kind": kind, "B": B, "L": L, "H": rng.choice([4, 8, 12, 12, 16]),
                "lengths": rng.choice(["uniform64", "lognormal", "full"] if kind == "packed" else ["mix60", "uniform64"]),
                "lengths_seed": ls}
    if kind == "generic":
        dtype = rng.choice(["f32", "f32", "bf16"])
        L = _log_int(rng, 24, 256)
        return {"kind": kind, "B": _log_int(rng, 1, 4096 // L), "L": L, "H": rng.choice([2, 4, 12]),
                "D": rng.choice([16, 32, 64] if dtype == "f32" else [32, 48]), "dtype": dtype,
                "lengths": "mix60", "lengths_seed": ls}
    if kind == "norm":
        return {"kind": kind, "T": _log_int(rng, 30, 32768), "W": rng.choice([256, 512, 768, 768, 1024]),
                "dtype": rng.choice(["bf16", "bf16", "bf16", "f32"])}
    hidden = rng.choice([256, 512, 768, 768, 1024])
    if kind == "geglu":
        inter = rng.choice([2, 4, 4]) * hidden
        top = int(26963 * 768 * 3072 / (hidden * inter))
        return {"kind": kind, "T": _log_int(rng, 60, min(32768, top)), "hidden": hidden, "inter": inter}
    T = _log_int(rng, 100, 26963)
    n_out = rng.choice([30528, hidden, 3 * hidden])
    return {"kind": kind, "T": T, "rows": T if n_out != 30528 else max(1, int(0.3 * T)), "n_in": hidden, "n_out": n_out}


# ---------------------------------------------------------------------------------------------------- inputs
def _case_lengths(case):
    """The case's sequence lengths, ascending."""
    B, L = case["B"], case["L"]
    rng = np.random.default_rng(case["lengths_seed"])
    kind = case["lengths"]
    if kind == "full":
        n = np.full(B, L)
    elif kind == "mix60":       # most sequences fill the position range, the others anything down to an eighth
        n = np.where(rng.random(B) < 0.6, L, rng.integers(L // 8, L, size=B))
    elif kind == "uniform64":
        n = rng.integers(64, L + 1, size=B)
    else:                       # lognormal
        n = np.clip(np.rint(rng.lognormal(6.0, 0.8, size=B)), 8, L)
    return sorted(int(x) for x in n)


def _lengths(case, seed):
    n = _case_lengths(case)
    random.Random(seed).shuffle(n)
    return n


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _normal(gen, shape, std=1.0, dtype=BF16):
    return (torch.randn(shape, generator=gen, device="cuda", dtype=F32) * std).to(dtype)


def _attention_inputs(case, seed):
    """Lengths, and QKV [rows, 3, H, D] and dO [rows, H, D]: rows of the padded batch (step, rows, masked) or packed
    tokens (packed, generic).  Q, K, V ~ N(0, 1/64) as the benchmark draws them, dO ~ N(0, 1)."""
    n, gen = _lengths(case, seed), _gen(seed)
    H, D = case["H"], case.get("D", 64)
    dtype = F32 if case.get("dtype") == "f32" else BF16
    rows = sum(n) if case["kind"] in ("packed", "generic") else case["B"] * case["L"]
    qkv = _normal(gen, (rows, 3, H, D), 0.125, dtype)
    do = _normal(gen, (rows, H, D), 1.0, dtype)
    if case["kind"] == "masked":   # the loss of a padded model takes no gradient from padding
        do = do * _mask(n, case["L"]).view(-1, 1, 1).to(dtype)
    return n, qkv, do


def _mask(n, L):
    return (torch.arange(L, device="cuda")[None, :] < torch.tensor(n, device="cuda")[:, None]).to(torch.int32)


def _cu(n):
    return torch.tensor([0] + list(np.cumsum(n)), dtype=torch.int32, device="cuda")


def _norm_inputs(case, seed):
    gen, T, W = _gen(seed), case["T"], case["W"]
    dtype = F32 if case["dtype"] == "f32" else BF16
    x, r, dy = (_normal(gen, (T, W), 1.0, dtype) for _ in range(3))
    gamma = (1.0 + 0.1 * torch.randn(W, generator=gen, device="cuda")).to(dtype)
    beta = (0.1 * torch.randn(W, generator=gen, device="cuda")).to(dtype)
    return x, r, dy, gamma, beta


def _geglu_inputs(case, seed):
    gen, T, hidden, inter = _gen(seed), case["T"], case["hidden"], case["inter"]
    return (_normal(gen, (T, hidden)), _normal(gen, (2 * inter, hidden), 0.02), _normal(gen, (hidden, inter), 0.02),
            _normal(gen, (T, hidden)))


def _linear_inputs(case, seed):
    gen = _gen(seed)
    x = _normal(gen, (case["T"], case["n_in"]))
    wt = _normal(gen, (case["n_out"], case["n_in"]), 0.02)
    if case["rows"] == case["T"]:
        return x, wt, None
    rows = torch.randperm(case["T"], generator=gen, device="cuda")[:case["rows"]].sort().values.to(torch.int32)
    return x, wt, rows


def prepare(case, seed):
    from paper_2312_17482_amd import binding as mb
    s = {"kind": case["kind"], "mb": mb}
    if case["kind"] in ("step", "rows", "packed", "masked", "generic"):
        n, qkv, do = _attention_inputs(case, seed)
        B, L, H, D = case["B"], case["L"], case["H"], case.get("D", 64)
        s.update(B=B, L=L, H=H, D=D, scale=1.0 / math.sqrt(D), slopes=mb.mb_alibi_slopes(H).cuda(), do=do, qkv=qkv)
        if case["kind"] in ("step", "rows"):
            cap = B * L
            need = mb.mb_alibi_attn_bwd_workspace_bytes(B, cap, L, H, D, mb.MB_BF16)
            s.update(mask=_mask(n, L), lse=torch.zeros((H, cap), dtype=F32, device="cuda"),
                     workspace=torch.empty(max(need, 16), dtype=torch.uint8, device="cuda"),
                     o_padded=torch.empty_like(do), dqkv_padded=torch.empty_like(qkv))
            if case["kind"] == "step":
                s.update(qkv_packed=torch.empty_like(qkv), do_packed=torch.empty_like(do), o=torch.empty_like(do),
                         dqkv=torch.empty_like(qkv))
        elif case["kind"] == "packed":
            s.update(cu=_cu(n), dqkv=torch.empty_like(qkv))
            s["plan"] = mb.mb_attn_plan(s["cu"], L, H) if L > 128 else None
        elif case["kind"] == "masked":
            s.update(cu=_cu([L] * B), key_lens=torch.tensor(n, dtype=torch.int32, device="cuda"),
                     dqkv=torch.empty_like(qkv))
        else:
            s.update(cu=_cu(n), dqkv=torch.empty_like(qkv))
    elif case["kind"] == "norm":
        s["x"], s["r"], s["dy"], s["gamma"], s["beta"] = _norm_inputs(case, seed)
    elif case["kind"] == "geglu":
        s["x"], s["w1v"], s["w2"], s["dy"] = _geglu_inputs(case, seed)
    else:
        s["x"], s["wt"], s["rows"] = _linear_inputs(case, seed)
    return s


# ---------------------------------------------------------------------------------------------------- one pass
def run(s):
    return _RUN[s["kind"]](s)


def _run_step(s):
    mb, B, L, H, D = s["mb"], s["B"], s["L"], s["H"], s["D"]
    W, cap = H * D, s["B"] * s["L"]
    seqlens, cu, indices, meta = mb.mb_unpad_index(s["mask"])
    qkv = mb.mb_unpad(s["qkv"].view(cap, 3 * W), indices, cap, meta, out=s["qkv_packed"].view(cap, 3 * W))
    q, k, v = (qkv.view(cap, 3, H, D)[:, i] for i in range(3))
    o, lse = mb.mb_alibi_attn_fwd(q, k, v, cu, L, s["slopes"], s["scale"], out=s["o"], lse=s["lse"])
    do = mb.mb_unpad(s["do"].view(cap, W), indices, cap, meta, out=s["do_packed"].view(cap, W)).view(cap, H, D)
    mb.mb_alibi_attn_bwd(do, q, k, v, o, lse, cu, L, s["slopes"], s["scale"], dq=s["dqkv"][:, 0], dk=s["dqkv"][:, 1],
                         dv=s["dqkv"][:, 2], workspace=s["workspace"])
    mb.mb_pad(o.view(cap, W), indices, cap, meta, B, L, out=s["o_padded"].view(cap, W))
    mb.mb_pad(s["dqkv"].view(cap, 3 * W), indices, cap, meta, B, L, out=s["dqkv_padded"].view(cap, 3 * W))
    return {"seqlens": seqlens, "cu": cu, "meta": meta, "o": s["o_padded"], "lse": lse, "dqkv": s["dqkv_padded"]}


def _run_rows(s):
    mb, B, L, H, D = s["mb"], s["B"], s["L"], s["H"], s["D"]
    W, cap = H * D, s["B"] * s["L"]
    seqlens, cu, indices, meta = mb.mb_unpad_index(s["mask"])
    q, k, v = (s["qkv"][:, i] for i in range(3))
    o, lse = mb.mb_alibi_attn_fwd(q, k, v, cu, L, s["slopes"], s["scale"], out=s["o_padded"], lse=s["lse"],
                                  token_rows=indices, T=cap)
    mb.mb_zero_padding(o.view(cap, W), indices, cap, meta, B, L)
    d = s["dqkv_padded"]
    mb.mb_alibi_attn_bwd(s["do"], q, k, v, o, lse, cu, L, s["slopes"], s["scale"], dq=d[:, 0], dk=d[:, 1], dv=d[:, 2],
                         workspace=s["workspace"], token_rows=indices, T=cap)
    mb.mb_zero_padding(d.view(cap, 3 * W), indices, cap, meta, B, L)
    return {"seqlens": seqlens, "cu": cu, "meta": meta, "o": o, "lse": lse, "dqkv": d}


def _run_attention(s):
    mb, d = s["mb"], s["dqkv"]
    q, k, v = (s["qkv"][:, i] for i in range(3))
    opt = {name: s[name] for name in ("plan", "key_lens") if name in s}
    o, lse = mb.mb_alibi_attn_fwd(q, k, v, s["cu"], s["L"], s["slopes"], s["scale"], **opt)
    mb.mb_alibi_attn_bwd(s["do"], q, k, v, o, lse, s["cu"], s["L"], s["slopes"], s["scale"], dq=d[:, 0], dk=d[:, 1],
                         dv=d[:, 2], **opt)
    return {"o": o, "lse": lse, "dqkv": d}


def _run_norm(s):
    mb = s["mb"]
    y, total, mean, rstd = mb.mb_add_layernorm_fwd(s["x"], s["r"], s["gamma"], s["beta"], 1e-12)
    ds, dgamma, dbeta = mb.mb_add_layernorm_bwd(s["dy"], total, s["gamma"], mean, rstd)
    return {"y": y, "s": total, "mean": mean, "rstd": rstd, "ds": ds, "dgamma": dgamma, "dbeta": dbeta}


def _run_geglu(s):
    mb = s["mb"]
    y, act = mb.mb_geglu_fwd(s["x"], s["w1v"], s["w2"])
    dx, dw1v, dw2 = mb.mb_geglu_bwd(s["dy"], s["x"], s["w1v"], s["w2"], act)
    return {"y": y, "act": act, "dx": dx, "dw1v": dw1v, "dw2": dw2}


def _run_linear(s):
    mb, x = s["mb"], s["x"]
    if s["rows"] is not None:
        x = mb.mb_unpad(x, s["rows"], s["rows"].numel(), None)
    return mb.mb_linear_fwd(x, s["wt"])


_RUN = {"step": _run_step, "rows": _run_rows, "packed": _run_attention, "masked": _run_attention,
        "generic": _run_attention, "norm": _run_norm, "geglu": _run_geglu, "linear": _run_linear}


# ---------------------------------------------------------------------------------------------------- work
def work(case):
    """Each input read once and each output written once (a padded output in full); matrix products on real tokens:
    4 H D n^2 forward and 10 H D n^2 backward per sequence."""
    kind = case["kind"]
    if kind in ("step", "rows", "packed", "masked", "generic"):
        n, H, D, B, L = _case_lengths(case), case["H"], case.get("D", 64), case["B"], case["L"]
        e = 4 if case.get("dtype") == "f32" else 2
        T, W = sum(n), H * D
        if kind == "masked":   # every position is a query of the forward, the real ones are keys; dO is zero on padding
            return {"bytes": 4 * W * e * (B * L + T) + 4 * H * B * L, "flops": 14 * W * L * T}
        flops = 14 * W * sum(x * x for x in n)
        out = B * L if kind in ("step", "rows") else T
        return {"bytes": 4 * W * e * (T + out) + 4 * H * T + (4 * B * L if kind in ("step", "rows") else 0),
                "flops": flops}
    if kind == "norm":
        e = 4 if case["dtype"] == "f32" else 2
        return {"bytes": 6 * case["T"] * case["W"] * e + 8 * case["T"], "flops": 20 * case["T"] * case["W"]}
    if kind == "geglu":        # forward 6, backward 12 T hidden inter; the projections are not counted twice
        T, hidden, inter = case["T"], case["hidden"], case["inter"]
        return {"bytes": 2 * T * (4 * hidden + inter) + 18 * hidden * inter, "flops": 18 * T * hidden * inter}
    rows, n_in, n_out = case["rows"], case["n_in"], case["n_out"]
    return {"bytes": 2 * (rows * n_in + n_in * n_out + rows * n_out), "flops": 2 * rows * n_in * n_out}


def tolerance(case):
    """About four times what the start shows against 64 bits: half a unit in the last place of bf16 is 2^-9 of a value,
    and P, dS and the feed-forward's intermediate tensors are rounded once more on their way."""
    if case.get("dtype") == "f32":
        return {"rel": 4e-6}
    return {"rel": 1.2e-2}


# ---------------------------------------------------------------------------------------------------- 64 bits
def exact(case, seed):
    kind = case["kind"]
    if kind in ("step", "rows", "packed", "masked", "generic"):
        return _exact_attention(case, seed)
    if kind == "norm":
        return _exact_norm(case, seed)
    if kind == "geglu":
        return _exact_geglu(case, seed)
    x, wt, rows = _linear_inputs(case, seed)
    x = x if rows is None else x[rows.long()]
    return x.double() @ wt.double().T


def _exact_attention(case, seed):
    n, qkv, do = _attention_inputs(case, seed)
    B, L, H, D = case["B"], case["L"], case["H"], case.get("D", 64)
    padded = case["kind"] in ("step", "rows", "masked")
    scale = 1.0 / math.sqrt(D)
    slopes = 2.0 ** (-8.0 * torch.arange(1, H + 1, device="cuda", dtype=torch.float64) / H)
    o, dqkv = (torch.zeros(x.shape, dtype=torch.float64, device="cuda") for x in (do, qkv))
    lse = torch.zeros((H, B * L if padded else sum(n)), dtype=torch.float64, device="cuda")
    at = 0                                            # first token of the sequence in lse's own (packed) numbering
    for b, keys in enumerate(n):
        queries = L if case["kind"] == "masked" else keys
        r0 = b * L if padded else at
        q, k, v = (qkv[r0:r0 + queries, i].double().permute(1, 0, 2).contiguous() for i in range(3))
        k, v = k[:, :keys].contiguous(), v[:, :keys].contiguous()
        g = do[r0:r0 + queries].double().permute(1, 0, 2).contiguous()
        i = torch.arange(queries, device="cuda", dtype=torch.float64)
        dist = (i[:, None] - i[None, :keys]).abs()
        S = scale * torch.bmm(q, k.transpose(1, 2)) - slopes[:, None, None] * dist
        ls = torch.logsumexp(S, dim=2)
        P = torch.exp(S - ls[:, :, None])
        ob = torch.bmm(P, v)
        dP = torch.bmm(g, v.transpose(1, 2))
        dS = P * (dP - (g * ob).sum(2, keepdim=True)) * scale
        o[r0:r0 + queries] = ob.permute(1, 0, 2)
        lse[:, at:at + queries] = ls
        dqkv[r0:r0 + queries, 0] = torch.bmm(dS, k).permute(1, 0, 2)
        dqkv[r0:r0 + keys, 1] = torch.bmm(dS.transpose(1, 2), q).permute(1, 0, 2)
        dqkv[r0:r0 + keys, 2] = torch.bmm(P.transpose(1, 2), g).permute(1, 0, 2)
        at += queries
    out = {"o": o, "lse": lse, "dqkv": dqkv}
    if case["kind"] in ("step", "rows"):
        out.update(seqlens=None, cu=None, meta=None)
    return out


def _exact_norm(case, seed):
    x, r, dy, gamma, beta = (t.double() for t in _norm_inputs(case, seed))
    s = x + r
    if case["dtype"] == "bf16":    # the stored sum is part of the definition: it is what is normalised
        s = s.to(F32).to(BF16).double()
    mean = s.mean(1)
    rstd = 1.0 / torch.sqrt(((s - mean[:, None]) ** 2).mean(1) + 1e-12)
    xh = (s - mean[:, None]) * rstd[:, None]
    g = dy * gamma
    ds = rstd[:, None] * (g - g.mean(1, keepdim=True) - xh * (g * xh).mean(1, keepdim=True))
    return {"y": xh * gamma + beta, "s": s, "mean": mean, "rstd": rstd, "ds": ds, "dgamma": (dy * xh).sum(0),
            "dbeta": dy.sum(0)}


def _exact_geglu(case, seed):
    x, w1v, w2, dy = (t.double() for t in _geglu_inputs(case, seed))
    inter = case["inter"]
    h, g = x @ w1v[:inter].T, x @ w1v[inter:].T
    phi = 0.5 * torch.erfc(-h * math.sqrt(0.5))
    gelu = h * phi
    act = gelu * g
    y = act @ w2.T
    da = dy @ w2
    dw2 = dy.T @ act
    dh = da * g * (phi + h * torch.exp(-0.5 * h * h) / math.sqrt(2.0 * math.pi))
    dg = da * gelu
    del h, g, phi, gelu, da
    dhg = torch.cat((dh, dg), 1)
    return {"y": y, "act": act, "dx": dhg @ w1v, "dw1v": dhg.T @ x, "dw2": dw2}
