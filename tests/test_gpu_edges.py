"""The kernels outside the bfloat16, d_head 64, W <= 16 path at the edges of what their
arguments may hold: an lse that is not the forward's own, infinities, probabilities below the
normal range, sums that cancel, angles near a half turn.  The reference (rows below) takes the
entries of every query one by one in float64; an entry that a query does not have is not read."""
import math

import numpy as np
import pytest
import torch

from paper_2606_28560_amd import fibattn as F
from paper_2606_28560_amd import inputs, schedules

pytestmark = pytest.mark.gpu

FIB, POW2 = schedules.FIB15, schedules.POW2_11
DT = {"bf16": torch.bfloat16, "fp32": torch.float32}
INF = float("inf")


def make(B, H, Hkv, T, D, dtype, seed):
    x = inputs.attention_inputs(B, H, T, D, dtype, seed, 0, names=("q", "dO"))
    x.update(inputs.attention_inputs(B, Hkv, T, D, dtype, seed, 0, names=("k", "v")))
    return x


def entries(W, base, alpha, T):
    """(distance of row r0, weight of row r1, base value; 0 in the window), as the table has them."""
    return [(d, 0.0, 0) for d in range(min(W, T - 1) + 1)] + [
        (d, float(w), f) for d, w, f in F.fibattn_rung_table(alpha, base, W) if d < T]


def rows(x, W, base, alpha, o=None, lse=None):
    """Forward and (with x["dO"]) backward in float64, on the given o and lse where passed."""
    q, k, v = (x[n].double() for n in ("q", "k", "v"))
    B, H, T, D = q.shape
    G, tau = H // k.shape[1], 1.0 / math.sqrt(D)
    k, v = k.repeat_interleave(G, 1), v.repeat_interleave(G, 1)
    pos = torch.arange(T)
    ent = entries(W, base, alpha, T)

    def shifted(t, d):  # row i of the result is row i - d; zero rows before the start
        return torch.cat([torch.zeros_like(t[:, :, :min(d, T)]), t[:, :, :T - min(d, T)]], 2)

    def blend(t, d, w):
        return shifted(t, d) if w == 0 else (1 - w) * shifted(t, d) + w * shifted(t, d + 1)

    s = torch.full((len(ent), B, H, T), -INF, dtype=torch.float64)
    for n, (d, w, _) in enumerate(ent):
        dot = (q * shifted(k, d)).sum(-1)
        if w:
            dot = (1 - w) * dot + w * (q * shifted(k, d + 1)).sum(-1)
        s[n] = torch.where(pos >= d + (w > 0), dot * tau, s[n])
    has = [(pos >= d + (w > 0)) for d, w, _ in ent]
    m = torch.where(s.isnan(), -INF, s).max(0).values
    e = torch.exp(s - m)
    e = torch.stack([torch.where(h, a, 0.0) for h, a in zip(has, e)])
    l = e.sum(0)
    out = {"lse": m + torch.log(l)}
    acc = torch.zeros_like(q)
    for n, (d, w, _) in enumerate(ent):
        t = e[n][..., None] * blend(v, d, w)
        acc = acc + torch.where(has[n][:, None], t, 0.0)
    out["o"] = acc / l[..., None]
    if "dO" not in x:
        return out
    dO = x["dO"].double()
    o, lse = (out["o"] if o is None else o.double()), (out["lse"] if lse is None else lse.double())
    delta = (dO * o).sum(-1)
    dq, dk, dv = torch.zeros_like(q), torch.zeros_like(q), torch.zeros_like(q)
    xa, xb, y, dsum = (torch.zeros_like(lse) for _ in range(4))
    l1 = torch.zeros_like(lse)

    def back(t, d, keep):  # row i goes to row i - d
        t = torch.where(keep[:, None], t, 0.0)
        return torch.cat([t[:, :, d:], torch.zeros_like(t[:, :, :min(d, T)])], 2)

    for n, (d, w, f) in enumerate(ent):
        h = has[n]
        p = torch.exp(s[n] - lse)
        dP = (dO * shifted(v, d)).sum(-1)
        if w:
            dP = (1 - w) * dP + w * (dO * shifted(v, d + 1)).sum(-1)
        c = tau * p * (dP - delta)
        dq = dq + torch.where(h[:, None], c[..., None] * blend(k, d, w), 0.0)
        dsum = dsum + torch.where(h, p * dP, 0.0)
        gk, gv = c[..., None] * q, p[..., None] * dO
        dk, dv = dk + back((1 - w) * gk if w else gk, d, h), dv + back((1 - w) * gv if w else gv, d, h)
        if w:
            dk, dv = dk + back(w * gk, d + 1, h), dv + back(w * gv, d + 1, h)
        if f:
            ds = (q * (shifted(k, d + 1) - shifted(k, d))).sum(-1)
            db = (dO * (shifted(v, d + 1) - shifted(v, d))).sum(-1)
            xa, xb = xa + torch.where(h, f * p * dP * ds, 0.0), xb + torch.where(h, f * p * db, 0.0)
            y = y + torch.where(h, f * p * ds, 0.0)
            l1 = l1 + torch.where(h, (f * (c * ds + p * db)).abs(), 0.0)
    out["dalpha"] = float((tau * (xa - dsum * y) + xb).sum().detach())
    out["l1"] = float(l1.sum().detach())
    out["dq"] = dq
    out["dk"], out["dv"] = (t.view(B, H // G, G, T, D).sum(2) for t in (dk, dv))
    return out


def run(x, W, base, alpha, o=None, lse=None, rope_base=0.0):
    """o, lse, dq, dk, dv, dalpha of the library on CPU inputs, on the CPU."""
    g = {n: t.cuda() for n, t in x.items()}
    fo, fl = F.fibattn_forward(g["q"], g["k"], g["v"], W, base, alpha)
    res = {"o": fo, "lse": fl}
    if "dO" in g:
        o, lse = (fo if o is None else o.cuda()), (fl if lse is None else lse.cuda())
        res["dq"], res["dk"], res["dv"], da = F.fibattn_backward(
            g["q"], g["k"], g["v"], o, lse, g["dO"], W, base, alpha, rope_base=rope_base)
        res["dalpha"] = da
    torch.cuda.synchronize()
    res = {n: t.cpu() for n, t in res.items()}
    if "dalpha" in res:
        res["dalpha"] = float(res["dalpha"])
    return res


def close(got, want, dtype, names=("o", "lse", "dq", "dk", "dv")):
    """Finite elements near the reference's (1e-5, bfloat16 2e-2, of the largest; lse 1e-5 and
    1e-3), the others NaN, inf or -inf as the reference's are."""
    for n in names:
        if n not in got:
            continue
        a, b = got[n].double(), want[n]
        for what, f in (("nan", torch.isnan), ("inf", torch.isposinf), ("-inf", torch.isneginf)):
            bad = f(a) != f(b)
            assert not bad.any(), (n, what, bad.nonzero()[:4].tolist(), a[bad][:4].tolist(), b[bad][:4].tolist())
        fin = torch.isfinite(b)
        if fin.any():
            tol = 1e-5 if dtype == "fp32" else 1e-3 if n == "lse" else 2e-2
            err = (a - b)[fin].abs().max()
            assert err <= tol * max(1.0, float(b[fin].abs().max())), (n, float(err))


SHAPES = [
    # (H, H_kv, T, D, dtype, W, base, alpha): every head size and storage type, windows of one
    # chunk and of several, integer and interpolated offsets, grouped heads, the kernel of
    # small float32 launches (few rows) and the one of large ones
    (2, 2, 150, 64, "bf16", 20, FIB, 0.9),
    (4, 1, 150, 64, "bf16", 40, FIB, 1.0),
    (2, 2, 130, 128, "bf16", 8, FIB, 1.0),
    (2, 1, 130, 128, "bf16", 17, POW2, 0.9),
    (2, 2, 130, 32, "bf16", 10, POW2, 1.3),
    (2, 2, 130, 32, "bf16", 3, FIB, 1.0),
    (2, 1, 130, 64, "fp32", 9, FIB, 0.9),
    (1, 1, 130, 128, "fp32", 40, FIB, 1.0),
    (100, 100, 130, 32, "fp32", 8, FIB, 1.2),
    (100, 100, 130, 64, "fp32", 40, FIB, 1.0),
]


@pytest.mark.parametrize("H,Hkv,T,D,dtype,W,base,alpha", SHAPES)
def test_backward_on_another_lse(H, Hkv, T, D, dtype, W, base, alpha):
    # an lse over more keys than these (0.75 to 1.5 larger), and +inf, which drops a query:
    # dq, dk, dv and dalpha are those of p = exp(s - lse)
    x = make(1, H, Hkv, T, D, dtype, 900)
    lse = rows({n: x[n] for n in ("q", "k", "v")}, W, base, alpha)["lse"]
    o = rows({n: x[n] for n in ("q", "k", "v")}, W, base, alpha)["o"].to(DT[dtype])
    lse = (lse + 0.75 + 0.75 * (torch.arange(T) % 2)).float()
    lse[:, :, 5::17] = INF
    got, want = run(x, W, base, alpha, o, lse), rows(x, W, base, alpha, o, lse)
    close(got, want, dtype, ("dq", "dk", "dv"))
    assert (got["dq"][:, :, 5::17] == 0).all()
    assert abs(got["dalpha"] - want["dalpha"]) <= (1e-5 if dtype == "fp32" else 1e-3) * max(1.0, want["l1"])


@pytest.mark.parametrize("H,Hkv,T,D,dtype,W,base,alpha", SHAPES)
def test_infinite_values(H, Hkv, T, D, dtype, W, base, alpha):
    # some elements of two value rows are +inf and -inf: they reach exactly the outputs of the
    # queries that attend those rows, with their sign
    x = make(1, H, Hkv, T, D, dtype, 910)
    j = T // 2
    x["v"][:, :, j, ::3] = INF
    x["v"][:, :, j, 1::3] = -INF
    x["v"][:, :, T // 3, 5] = -INF
    del x["dO"]
    close(run(x, W, base, alpha), rows(x, W, base, alpha), dtype)


@pytest.mark.parametrize("H,Hkv,T,D,dtype,W,base,alpha", SHAPES + [
    (2, 2, 130, 128, "bf16", 0, FIB, 0.9), (2, 2, 130, 32, "bf16", 0, FIB, 1.0), (2, 2, 130, 64, "fp32", 0, FIB, 1.0)])
def test_logits_of_minus_infinity(H, Hkv, T, D, dtype, W, base, alpha):
    # keys of -inf under queries that are positive have no weight: alone in the window, the whole
    # window, or a rung's row; with no key left the query is NaN
    x = make(1, H, Hkv, T, D, dtype, 920)
    x["q"] = x["q"].abs() + 0.125
    j = T // 2
    x["k"][:, :, j] = -INF
    x["k"][:, :, j + 10: j + 12 + W] = -INF
    del x["dO"]
    close(run(x, W, base, alpha), rows(x, W, base, alpha), dtype)


@pytest.mark.parametrize("what", ["v", "dO", "k"])
@pytest.mark.parametrize("H,Hkv,T,D,dtype,W,base,alpha", SHAPES)
def test_gradients_of_infinities(H, Hkv, T, D, dtype, W, base, alpha, what):
    # one element of one row is inf (for k: a whole row -inf under positive queries)
    x = make(1, H, Hkv, T, D, dtype, 930)
    j = T // 2
    if what == "k":
        x["q"] = x["q"].abs() + 0.125
        x["k"][:, :, j] = -INF
    else:
        x[what][:, :, j, 3] = INF
    ref = rows({n: x[n] for n in ("q", "k", "v")}, W, base, alpha)
    o, lse = ref["o"].to(DT[dtype]), ref["lse"].float()
    got, want = run(x, W, base, alpha, o, lse), rows(x, W, base, alpha, o, lse)
    close(got, want, dtype, ("dk", "dv"))
    # dq may read row r1 of a rung with w = 0 too (dalpha needs it): 0 times its values
    skip = torch.zeros(T, dtype=torch.bool)
    for d, w, f in entries(W, base, alpha, T):
        if f and w == 0:
            skip[j + d + 1: j + d + 2] = True
            if what == "dO":
                skip[j] = True
    close({"dq": got["dq"][:, :, ~skip]}, {"dq": want["dq"][:, :, ~skip]}, dtype)


@pytest.mark.parametrize("what", ["o", "dq", "dk", "dv"])
@pytest.mark.parametrize("D,dtype,W", [(128, "bf16", 8), (64, "bf16", 20), (32, "bf16", 8), (64, "fp32", 8), (64, "fp32", 40)])
@pytest.mark.parametrize("rung", [False, True])
def test_probability_below_the_normal_range(D, dtype, W, rung, what):
    # p = 2^-130 (a subnormal float32, which bfloat16 parts cannot hold) times a value or a dO
    # of 2^127, or a dP of 2^110: results of ordinary size
    T, d = 128, 55 if rung else 2
    x = {n: torch.zeros(1, 1, T, D, dtype=DT[dtype]) for n in ("q", "k", "v", "dO")}
    i = T - 5
    x["q"][:, :, i, 0] = 1.0
    x["k"][:, :, i - d, 0] = float(torch.tensor(-130.0 * math.log(2.0) * math.sqrt(D)).to(DT[dtype]))
    if what == "o":
        x["v"][:, :, i - d, 1] = 2.0 ** 127
        del x["dO"]
    elif what == "dv":
        x["dO"][:, :, i, 1] = 2.0 ** 127
    else:
        x["v"][:, :, i - d, 1], x["dO"][:, :, i, 1] = 2.0 ** 55, 2.0 ** 55
    o, lse = torch.zeros(1, 1, T, D, dtype=DT[dtype]), torch.zeros(1, 1, T)
    row, dim = (i, 1 if what == "o" else 0) if what in ("o", "dq") else (i - d, 0 if what == "dk" else 1)
    a, b = (float(r[what][0, 0, row, dim]) for r in (run(x, W, FIB, 1.0, o, lse), rows(x, W, FIB, 1.0, o, lse)))
    assert abs(b) > 1e-8 and abs(a - b) <= 1e-2 * abs(b), (a, b)


@pytest.mark.parametrize("what", ["o", "dq", "dk", "dv"])
@pytest.mark.parametrize("D,W,alpha", [(64, 40, 1.0), (64, 20, 0.9), (128, 8, 1.0), (128, 8, 0.9), (32, 12, 0.9), (32, 5, 1.0)])
def test_weights_of_24_bits(D, W, alpha, what):
    # bfloat16 rows times float32 weights, two of the rows chosen so that the sum cancels to
    # 2^-12 or less of its terms: what is left shows the error of the weights.  Rounded to 24
    # bits they have 6e-8, and 1e-7 to 2e-7 from the logits and from lse log2 e; two bfloat16
    # parts have up to 7.6e-6.  Bound: 4e-7 of the terms' sum.
    H, T = 16, 160
    x = {n: t.double() for n, t in make(1, H, H, T, D, "bf16", 940).items()}
    if what in ("dq", "dk"):  # logits of 0: tau dS does not move with the rows that are chosen
        x["k" if what == "dk" else "q"].zero_()
    fwd = rows({n: x[n] for n in ("q", "k", "v")}, W, FIB, alpha)
    o, lse = fwd["o"].bfloat16(), fwd["lse"].float()
    var, at = {"o": "v", "dq": "k", "dk": "q", "dv": "dO"}[what], T - 1 if what in ("o", "dq") else 4
    if what == "o":
        del x["dO"]
    # the weight of every row, as the derivative
    x[var].requires_grad_()
    rows(x, W, FIB, alpha, o, lse)[what][0, :, at, 0].sum().backward()
    w = x[var].grad[0, :, :, 0]
    x[var] = x[var].detach()
    for h in range(H):
        a, b = (int(n) for n in w[h].abs().argsort(descending=True)[:2])
        y = x[var][0, h]
        y[b] = 0.0
        for n in (a, b):
            y[n] = 0.0
            y[n] = (-(w[h, :, None] * y).sum(0) / w[h, n]).bfloat16().double()
    mass = (w[:, :, None] * x[var][0]).abs().sum(1)
    g = {n: t.bfloat16() for n, t in x.items()}
    want, got = rows(g, W, FIB, alpha, o, lse)[what][0, :, at], run(g, W, FIB, alpha, o, lse)[what][0, :, at].double()
    assert (want.abs() <= 2.0 ** -12 * mass).all()
    err = ((got - want).abs() - 2.0 ** -8 * want.abs()).clamp_min(0.0) / mass
    print(f"{what} D{D} W{W} alpha {alpha}: error over the terms' sum {float(err.max()):.1e}", flush=True)
    assert err.max() <= 4e-7


def test_dalpha_adds_float64_products():
    # bfloat16, logits of 0, lse 0 (p = 1): dP = +-(2^23 + 1) in the window, three of each sign,
    # and two rungs whose f p dP need 31 bits, all of which cancel to a small exact number
    T, D, W, base, alpha = 192, 64, 40, [101, 203], 0.5  # distances 50.5 and 101.5
    x = {n: torch.zeros(1, 1, T, D, dtype=torch.bfloat16) for n in ("q", "k", "v", "dO")}
    i = T - 1
    x["q"][:, :, i, 0] = 1.0
    x["dO"][:, :, i, 1], x["dO"][:, :, i, 2] = 4096.0, 1.0

    def value(j, hi, lo):  # dP = 4096 hi + lo
        x["v"][:, :, j, 1], x["v"][:, :, j, 2] = hi, lo

    for j, sign in ((T - 32, 1), (T - 31, 1), (T - 30, 1), (T - 16, -1), (T - 15, -1), (T - 14, -1)):
        value(j, sign * 2048.0, sign * 1.0)
    value(i, 0.0, 5.0)
    for d, hi, lo in ((50, 2048.0, 1.0), (101, -1016.0, 3.0)):
        for y in (0, 1):
            value(i - d - y, hi, lo)
        x["k"][:, :, i - d, 0], x["k"][:, :, i - d - 1, 0] = 1.0, -1.0  # logit 0, <q, k1 - k0> = -2
    lse, o = torch.zeros(1, 1, T), torch.zeros(1, 1, T, D, dtype=torch.bfloat16)
    want = rows(x, W, base, alpha, o, lse)["dalpha"]
    got = run(x, W, base, alpha, o, lse)["dalpha"]
    assert abs(got - want) <= 2.0 ** -23 * abs(want), (got, want)


ROTATED = [(32, "bf16", 8), (64, "bf16", 20), (128, "bf16", 8), (32, "fp32", 8), (64, "fp32", 8), (128, "fp32", 8),
           (64, "fp32", 40)]


@pytest.mark.parametrize("H", [2, 64])
@pytest.mark.parametrize("D,dtype,W", ROTATED)
def test_gradients_rotated_back(D, dtype, W, H):
    # float32: the bits of the RoPE launch on the gradients that are not rotated.  bfloat16:
    # one rounding (2^-8 of the value at most), also at 355 and 710 radians, near a half turn,
    # where the other element of the pair is 0 and the small sine counts to its last bits (the
    # float32 sums before: 2e-6 of the largest).
    T = 720
    x = make(1, H, H, T, D, dtype, 960)
    x["k"][..., 0] = 0.0
    x["q"][..., 0] = 0.0
    got = run(x, W, FIB, 0.9, rope_base=10000.0)
    plain = run(x, W, FIB, 0.9) if dtype == "fp32" else rows(x, W, FIB, 0.9, got["o"], got["lse"])
    t = torch.tensor([355, 710])
    ang = t.double()[:, None] * 10000.0 ** (-2.0 * torch.arange(D // 2, dtype=torch.float64) / D)
    c, s = ang.cos(), ang.sin()
    for n in ("dq", "dk"):
        if dtype == "fp32":
            assert torch.equal(got[n], F.fibattn_rope(plain[n].cuda(), transpose=True).cpu()), n
            continue
        u, w = plain[n][0, :, t, :D // 2], plain[n][0, :, t, D // 2:]
        want = torch.cat([u * c + w * s, w * c - u * s], -1)
        err = (got[n][0, :, t].double() - want).abs() - 2.0 ** -8 * want.abs()
        # element 0 is w s: what is uncertain in w counts s times
        slack = 2e-6 * plain[n].abs().max() * torch.cat([torch.where(torch.arange(D // 2) == 0, s.abs(), 1.0)] + [torch.ones_like(s)], -1)
        print(f"{n}: error past the rounding, of what the sums leave open {float((err / slack).max()):.2f}", flush=True)
        assert (err <= slack).all(), n
    if dtype == "fp32":
        assert torch.equal(got["dv"], plain["dv"]) and got["dalpha"] == plain["dalpha"]


@pytest.mark.parametrize("H,T", [(2, 150), (64, 1500)])
@pytest.mark.parametrize("D,dtype,W", ROTATED)
def test_rotated_q_has_the_bits_of_the_rope_launch(D, dtype, W, H, T):
    # also where the rotated rows take the place of q, for which they are written by the wave
    # that has read them, and with a device table; o and lse are those of the rotated q
    x = {n: t.cuda() for n, t in make(1, H, H, T, D, dtype, 950).items()}
    K, Q = F.fibattn_rope(x["k"]), F.fibattn_rope(x["q"])
    o, lse, got = F.fibattn_forward_rope_q(x["q"], K, x["v"], W, FIB, 0.9)
    want_o, want_lse = F.fibattn_forward(Q, K, x["v"], W, FIB, 0.9)
    place = x["q"].clone()
    o2, lse2, _ = F.fibattn_forward_rope_q(place, K, x["v"], W, FIB, 0.9, q_out=place)
    table = F.fibattn_device_table(torch.tensor([0.9], device="cuda"), FIB, W)
    od, ld, Qd = F.fibattn_forward_rope_q_dt(x["q"], K, x["v"], W, table)
    torch.cuda.synchronize()
    assert torch.equal(Qd, Q) and torch.equal(od, o) and torch.equal(ld, lse)
    assert torch.equal(got, Q) and torch.equal(o, want_o) and torch.equal(lse, want_lse)
    assert torch.equal(place, Q) and torch.equal(o2, o) and torch.equal(lse2, lse)


@pytest.mark.parametrize("H,Hkv,T,D,dtype,W,base,alpha", [c for c in SHAPES if c[4] == "bf16"])
def test_logits_far_apart(H, Hkv, T, D, dtype, W, base, alpha):
    # logits of +-60: most weights are below what the matrix cores take in full, with rows of
    # ordinary size beside them
    x = make(1, H, Hkv, T, D, dtype, 970)
    x["q"] = (20.0 * x["q"].float()).bfloat16()
    ref = rows({n: x[n] for n in ("q", "k", "v")}, W, base, alpha)
    got = run(x, W, base, alpha, ref["o"].bfloat16(), ref["lse"].float())
    close(got, rows(x, W, base, alpha, ref["o"].bfloat16(), ref["lse"].float()), dtype)
