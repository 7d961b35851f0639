"""The performance cases: the attention calls a user of this framework makes, from the
smallest to the largest, each through the public binding (paper_2606_28560_amd.fibattn).

A case is one layer's work: rotary embeddings, the forward, and for training the
backward with respect to the unrotated q and k.  Kinds:
  step     training step of a layer with a host alpha: fibattn_rope of k, the forward
           that rotates q where it loads it, the backward with R^T;
  plain    forward and backward of q, k that are rotated already (no RoPE call);
  forward  evaluation: fibattn_rope of k and the forward, no rotated q kept;
  serve    the same with every output buffer kept by the caller;
  learned  training step with alpha = 0.5 + sigmoid(theta), theta on the device;
  fused    training step that reads q and v as slices of a [B,T,3,H,D] projection output
           and writes dq, dk, dv into the matching gradient buffer.
"""
import math

import numpy as np
import torch

from paper_2606_28560_amd import fibattn as F
from paper_2606_28560_amd import schedules

ROPE_BASE = 10000.0
BASES = {"fib15": schedules.FIB15, "pow2_11": schedules.POW2_11}
DTYPES = {"bf16": torch.bfloat16, "fp32": torch.float32}


def _case(name, kind, dtype, B, H, H_kv, T, D, W, base, alpha):
    return {"name": name, "kind": kind, "dtype": dtype, "B": B, "H": H, "H_kv": H_kv, "T": T, "D": D, "W": W,
            "base": base, "alpha": alpha}


def listed():
    return [
        # a layer of a small float32 model, gradients checked in a notebook or a unit test:
        # latency of a handful of launches
        _case("fp32_T128_d32", "plain", "fp32", 1, 2, 2, 128, 32, 8, "fib15", 1.0),
        # evaluation of one short text, buffers kept: the latency of a serving call
        _case("serve_T777", "serve", "bf16", 1, 8, 2, 777, 64, 8, "fib15", 1.0),
        # one layer of the 60M model in training, fixed alpha (integer offsets)
        _case("layer60m_T1024", "step", "bf16", 8, 8, 8, 1024, 64, 8, "fib15", 1.0),
        # the same model with its 8 query heads on 2 key/value heads
        _case("gqa_T1024", "step", "bf16", 8, 8, 2, 1024, 64, 8, "fib15", 1.0),
        # a layer of the linear stagger (interpolated offsets), q and v left where a fused
        # projection wrote them, an odd length
        _case("fused_T1000", "fused", "bf16", 16, 8, 8, 1000, 64, 10, "fib15", 0.8333333),
        # evaluation at four times the training length (a layer of the coprime stagger)
        _case("extrap_T4096", "forward", "bf16", 4, 8, 8, 4096, 64, 8, "fib15", 0.9666666),
        # training of alpha itself, the largest batch, both bases in use: the power-of-2 one
        _case("learned_T1024", "learned", "bf16", 32, 8, 8, 1024, 64, 10, "pow2_11", 0.0),
        # the head size of larger models, grouped heads, an odd length
        _case("d128_T2000", "step", "bf16", 2, 16, 4, 2000, 128, 8, "fib15", 0.9),
        # small heads with the power-of-2 control base
        _case("d32_T1024", "step", "bf16", 8, 8, 8, 1024, 32, 10, "pow2_11", 0.8),
        # a wide local window, as models with sliding windows use
        _case("w64_T2048", "step", "bf16", 4, 8, 8, 2048, 64, 64, "fib15", 1.3),
        # the widest window in evaluation
        _case("w128_T1500", "forward", "bf16", 4, 8, 8, 1500, 64, 128, "fib15", 1.0),
        # float32 training of the 60M layer (no autocast)
        _case("fp32_T1024", "step", "fp32", 4, 8, 8, 1024, 64, 12, "fib15", 0.9),
    ]


def draw(rng):
    most = [work(c) for c in listed()]
    most = {k: max(w[k] for w in most) for k in ("bytes", "flops")}
    while True:
        kind = rng.choice(["step", "step", "step", "forward", "forward", "learned", "plain", "fused"])
        dtype = rng.choice(["bf16", "bf16", "bf16", "fp32"])
        D = rng.choice([64, 64, 64, 128, 32])
        H_kv = rng.choice([1, 2, 4, 8])
        H = H_kv * rng.choice([1, 1, 1, 2, 4])
        if kind == "fused":
            H = H_kv  # one projection output holds as many key/value heads as query heads
        T = int(round(math.exp(rng.uniform(math.log(48), math.log(6000)))))
        W = rng.choice([6, 8, 10, 12, 16, int(round(math.exp(rng.uniform(0.0, math.log(128)))))])
        B = int(round(math.exp(rng.uniform(0.0, math.log(40)))))
        base = rng.choice(["fib15", "fib15", "pow2_11"])
        alpha = rng.choice([1.0, round(rng.uniform(0.5, 1.5), 4), round(rng.uniform(0.5, 1.5), 4)])
        c = _case("", kind, dtype, B, H, H_kv, T, D, W, base, alpha)
        del c["name"]
        w = work(c)
        if all(w[k] <= most[k] for k in most):
            return c


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    B, H, Hkv, T, D = (case[x] for x in ("B", "H", "H_kv", "T", "D"))
    dt = DTYPES[case["dtype"]]

    def normal(*shape):
        return torch.randn(shape, generator=g, device="cuda").to(dt)

    s = {"case": case, "W": case["W"], "base": BASES[case["base"]], "alpha": float(np.float32(case["alpha"]))}
    if case["kind"] == "fused":
        qkv = normal(B, T, 3, H, D)  # the projection's output
        s["q"], s["k"], s["v"] = (qkv[:, :, n].transpose(1, 2) for n in range(3))
        s["grad"] = torch.empty_like(qkv)  # its gradient
    else:
        s["q"], s["k"], s["v"] = normal(B, H, T, D), normal(B, Hkv, T, D), normal(B, Hkv, T, D)
    if case["kind"] in ("step", "plain", "learned", "fused"):
        s["dO"] = normal(B, H, T, D)
    if case["kind"] == "learned":
        s["theta"] = torch.randn(1, generator=g, device="cuda")
        s["dtheta"] = torch.empty(1, device="cuda")
    if case["kind"] == "serve":
        s["k_out"], s["o"] = torch.empty_like(s["k"]), torch.empty_like(s["q"])
        s["lse"] = torch.empty((B, H, T), device="cuda")
    return s


def run(s):
    kind, W, base, alpha = s["case"]["kind"], s["W"], s["base"], s["alpha"]
    q, k, v = s["q"], s["k"], s["v"]
    if kind == "serve":
        K = F.fibattn_rope(k, ROPE_BASE, out=s["k_out"])
        o, lse, _ = F.fibattn_forward_rope_q(q, K, v, W, base, alpha, ROPE_BASE, o=s["o"], lse=s["lse"], keep_q=False)
        return {"o": o, "lse": lse}
    if kind == "forward":
        # only the matrix-core shapes rotate q without a buffer for the rotated rows
        keep = not (s["case"]["dtype"] == "bf16" and s["case"]["D"] == 64 and W <= 16)
        K = F.fibattn_rope(k, ROPE_BASE)
        o, lse, _ = F.fibattn_forward_rope_q(q, K, v, W, base, alpha, ROPE_BASE, keep_q=keep)
        return {"o": o, "lse": lse}
    if kind == "plain":
        o, lse = F.fibattn_forward(q, k, v, W, base, alpha)
        dq, dk, dv, da = F.fibattn_backward(q, k, v, o, lse, s["dO"], W, base, alpha)
    elif kind == "step":
        K = F.fibattn_rope(k, ROPE_BASE)
        o, lse, Q = F.fibattn_forward_rope_q(q, K, v, W, base, alpha, ROPE_BASE)
        dq, dk, dv, da = F.fibattn_backward(Q, K, v, o, lse, s["dO"], W, base, alpha, rope_base=ROPE_BASE)
    elif kind == "fused":
        grad = s["grad"]
        K = F.fibattn_rope(k.contiguous(), ROPE_BASE)  # RoPE takes packed rows
        o, lse, Q = F.fibattn_forward_rope_q(q, K, v, W, base, alpha, ROPE_BASE)
        dq, dk, dv = (grad[:, :, n].transpose(1, 2) for n in range(3))
        da = F.fibattn_backward(Q, K, v, o, lse, s["dO"], W, base, alpha, dq=dq, dk=dk, dv=dv,
                                rope_base=ROPE_BASE)[3]
        return {"o": o, "lse": lse, "grad": grad, "dalpha": da}
    else:
        _, K, table = F.fibattn_rope_qk_table(None, k, ROPE_BASE, theta=s["theta"], base=base, W=W)
        o, lse, Q = F.fibattn_forward_rope_q_dt(q, K, v, W, table, ROPE_BASE)
        dq, dk, dv, da = F.fibattn_backward_dt(Q, K, v, o, lse, s["dO"], W, table, dtheta=s["dtheta"],
                                               rope_base=ROPE_BASE)
        return {"o": o, "lse": lse, "dq": dq, "dk": dk, "dv": dv, "dalpha": da, "dtheta": s["dtheta"]}
    return {"o": o, "lse": lse, "dq": dq, "dk": dk, "dv": dv, "dalpha": da}


def _rungs(alpha, base, W):
    """(floor of the distance, weight of the next row, base value) of the rungs past the
    window: distances fl32(alpha f), equal ones once."""
    out, last = [], -1.0
    for f in base:
        d = float(np.float32(alpha) * np.float32(f))
        if d > W and d != last:
            out.append((int(math.floor(d)), d - math.floor(d), f))
            last = d
    return out


def work(case):
    B, H, Hkv, T, D, W = (case[x] for x in ("B", "H", "H_kv", "T", "D", "W"))
    es = 2 if case["dtype"] == "bf16" else 4
    rows_q, rows_k = B * H * T, B * Hkv * T
    # a learned alpha lies between 0.5 and 1.5: counted at 1, interpolating
    alpha = 1.0 if case["kind"] == "learned" else case["alpha"]
    entries = sum(max(0, T - d) for d in range(W + 1))
    for d0, w, _ in _rungs(alpha, BASES[case["base"]], W):
        entries += max(0, T - d0) * (2 if w or case["kind"] == "learned" else 1)
    entries *= B * H
    nbytes = es * D * (2 * rows_q + 2 * rows_k) + 4 * rows_q  # q, k, v; o, lse
    flops = 4 * D * entries  # q.k and p.v
    if case["kind"] in ("step", "plain", "learned", "fused"):
        nbytes += es * D * (2 * rows_q + 2 * rows_k)  # dO; dq, dk, dv
        flops += 10 * D * entries  # q.k again, dO.v, dq, dk, dv
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # against 64 bits, relative 2-norm: up to 2.5e-7 in float32; in bfloat16 2.5e-3 to
    # 3.7e-3 (the rounding of the stored outputs and of the entries' weights)
    if case["dtype"] == "fp32":
        return {"rel": 4e-6, "max": 2e-4}
    return {"rel": 1e-2, "max": 0.1}


def _rope64(x, transpose=False):
    T, D = x.shape[-2:]
    inv = ROPE_BASE ** (-2.0 * torch.arange(D // 2, dtype=torch.float64, device=x.device) / D)
    ang = torch.arange(T, dtype=torch.float64, device=x.device)[:, None] * inv
    c, s = ang.cos(), -ang.sin() if transpose else ang.sin()
    u, w = x[..., : D // 2], x[..., D // 2 :]
    return torch.cat([u * c - w * s, w * c + u * s], dim=-1)


def _down(x, d):
    """Row i of the result is row i - d of x; zero rows before the start."""
    return torch.nn.functional.pad(x, (0, 0, d, 0))[:, :, : x.shape[2]]


def _up(x, d):
    """Row j of the result is row j + d of x; zero rows past the end."""
    return torch.nn.functional.pad(x, (0, 0, 0, d))[:, :, d:]


def exact(case, seed):
    s = prepare(case, seed)
    kind, W, base = case["kind"], s["W"], s["base"]
    B, H, Hkv, T, D = (case[x] for x in ("B", "H", "H_kv", "T", "D"))
    G, tau = H // Hkv, 1.0 / math.sqrt(D)
    sg = 0.0
    alpha = s["alpha"]
    if kind == "learned":
        sg = 1.0 / (1.0 + math.exp(-float(s["theta"].double().item())))
        alpha = float(np.float32(0.5 + sg))
    q, k, v = (s[n].double() for n in ("q", "k", "v"))
    rope = kind != "plain"
    if rope:
        q, k = _rope64(q), _rope64(k)
    k, v = (x.repeat_interleave(G, dim=1) for x in (k, v))
    entries = [(d, 0.0, 0) for d in range(min(W, T - 1) + 1)]
    entries += [r for r in _rungs(alpha, base, W) if r[0] + (r[1] > 0) < T]
    row = torch.arange(T, device=q.device)

    def blend(x, d0, w):
        return _down(x, d0) if w == 0.0 else (1.0 - w) * _down(x, d0) + w * _down(x, d0 + 1)

    logits = torch.full((len(entries), B, H, T), -math.inf, dtype=torch.float64, device=q.device)
    for n, (d0, w, _) in enumerate(entries):
        seen = row >= d0 + (1 if w else 0)
        logits[n] = torch.where(seen, (q * blend(k, d0, w)).sum(-1) * tau, logits[n])
    lse = torch.logsumexp(logits, dim=0)
    p = torch.exp(logits - lse)
    o = torch.zeros_like(q)
    for n, (d0, w, _) in enumerate(entries):
        o += p[n][..., None] * blend(v, d0, w)
    if "dO" not in s:
        return {"o": o, "lse": lse}
    dO = s["dO"].double()
    delta = (dO * o).sum(-1)
    dq, dk, dv = torch.zeros_like(q), torch.zeros_like(q), torch.zeros_like(q)
    dalpha = torch.zeros((), dtype=torch.float64, device=q.device)
    for n, (d0, w, f) in enumerate(entries):
        pn = p[n]
        dS = pn * ((dO * blend(v, d0, w)).sum(-1) - delta) * tau
        dq += dS[..., None] * blend(k, d0, w)
        gk, gv = dS[..., None] * q, pn[..., None] * dO
        if w == 0.0:
            dk += _up(gk, d0)
            dv += _up(gv, d0)
        else:
            dk += (1.0 - w) * _up(gk, d0) + w * _up(gk, d0 + 1)
            dv += (1.0 - w) * _up(gv, d0) + w * _up(gv, d0 + 1)
        if f:
            dalpha += f * (dS * (q * (_down(k, d0 + 1) - _down(k, d0))).sum(-1)
                           + pn * (dO * (_down(v, d0 + 1) - _down(v, d0))).sum(-1)).sum()
    dk, dv = (x.view(B, Hkv, G, T, D).sum(2) for x in (dk, dv))
    if rope:
        dq, dk = _rope64(dq, transpose=True), _rope64(dk, transpose=True)
    dalpha = dalpha.reshape(1)
    if kind == "fused":
        grad = torch.stack([x.transpose(1, 2) for x in (dq, dk, dv)], dim=2)
        return {"o": o, "lse": lse, "grad": grad, "dalpha": dalpha}
    out = {"o": o, "lse": lse, "dq": dq, "dk": dk, "dv": dv, "dalpha": dalpha}
    if kind == "learned":
        out["dtheta"] = dalpha * sg * (1.0 - sg)
    return out
