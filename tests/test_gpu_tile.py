"""GPU parity of the tile kernels (every shape outside the bfloat16, d_head 64, W <= 16
path) where they can go wrong: windows at the edges of the 32-row band chunks and of the
chunks staged together, lengths around the 16- and 64-row tiles, each storage type and head
size, one, two, three and four query heads side by side, both kernels of float32 rows (few
rows and many; the d_head 128 dk/dv launch of many has two waves per workgroup), more rungs
than a wave has row groups, and strided placements."""
import pytest
import torch

import oracle
from paper_2606_28560_amd import fibattn as F
from paper_2606_28560_amd import inputs, schedules
from tests.parity import compare, gpu_run, oracle_run

pytestmark = pytest.mark.gpu

FIB, POW2 = schedules.FIB15, schedules.POW2_11
MANY = list(range(3, 99, 3))  # K = 32

CASES = [
    # (B, H, H_kv, T, D, dtype, W, base, alpha)
    (1, 2, 2, 200, 64, "bf16", 17, FIB, 1.1),     # first window past the 32-row chunk
    (1, 2, 2, 200, 64, "bf16", 48, FIB, 1.0),     # two chunks exactly
    (1, 2, 2, 333, 64, "bf16", 49, FIB, 1.3),     # three, and a ragged tail
    (1, 8, 2, 333, 64, "bf16", 112, POW2, 0.9),   # four chunks, four heads side by side
    (1, 2, 2, 333, 64, "bf16", 113, FIB, 1.0),    # five chunks, in two stages
    (1, 2, 2, 100, 64, "bf16", 128, FIB, 1.0),    # a window longer than the sequence
    (2, 4, 2, 129, 128, "bf16", 16, FIB, 0.85),   # two heads side by side
    (1, 3, 1, 257, 128, "bf16", 33, FIB, 1.0),    # a group of three
    (1, 2, 2, 65, 128, "bf16", 128, FIB, 0.7),
    (2, 2, 2, 127, 32, "bf16", 16, POW2, 1.3),
    (1, 4, 1, 200, 32, "bf16", 64, FIB, 1.0),
    (1, 2, 2, 200, 32, "bf16", 0, MANY, 0.9),     # 32 rungs
    (1, 2, 2, 200, 64, "fp32", 16, MANY, 1.0),
    (1, 2, 1, 130, 32, "fp32", 17, FIB, 0.9),
    (1, 4, 2, 97, 128, "fp32", 8, FIB, 1.2),
    (1, 3, 3, 33, 128, "fp32", 128, FIB, 1.0),
    (1, 1, 1, 1, 128, "fp32", 8, FIB, 1.0),
    (1, 1, 1, 15, 128, "bf16", 0, FIB, 0.9),
    (1, 2, 2, 2, 32, "fp32", 1, FIB, 0.5),        # rungs at d = 1.5 and beyond, T = 2
    (3, 2, 2, 64, 32, "bf16", 12, [], 1.0),       # no rungs
]


@pytest.mark.parametrize("B,H,Hkv,T,D,dtype,W,base,alpha", CASES)
def test_tile_parity(B, H, Hkv, T, D, dtype, W, base, alpha):
    idx = CASES.index((B, H, Hkv, T, D, dtype, W, base, alpha))
    print(f"tile case {idx}: B{B} H{H}/{Hkv} T{T} D{D} {dtype} W{W} K{len(base)} alpha={alpha}", flush=True)
    x = inputs.attention_inputs(B, H, T, D, dtype, 800 + idx, 0, names=("q", "dO"))
    x.update(inputs.attention_inputs(B, Hkv, T, D, dtype, 800 + idx, 0, names=("k", "v")))
    got = gpu_run(x["q"], x["k"], x["v"], x["dO"], W, base, alpha)
    ref = oracle_run(x["q"], x["k"], x["v"], x["dO"], W, base, alpha)
    print(compare(got, ref, dtype, f"tile case {idx}"), flush=True)


@pytest.mark.parametrize("D,dtype,W", [(64, "bf16", 40), (128, "bf16", 8), (32, "bf16", 12), (64, "fp32", 8)])
def test_tile_strides(D, dtype, W):
    # slices of one [B,T,3,H,D] buffer with poisoned gaps give the packed call's bits
    B, H, T = 2, 3, 150
    x = inputs.attention_inputs(B, H, T, D, dtype, 850, 0)
    packed = {n: x[n].cuda() for n in ("q", "k", "v")}
    dt = packed["q"].dtype
    buf = torch.full((B, T, 3, H, D + 16), float("nan"), device="cuda", dtype=dt)
    views = {}
    for n, name in enumerate(("q", "k", "v")):
        views[name] = buf[:, :, n, :, :D].transpose(1, 2)
        views[name].copy_(packed[name])
    want, want_lse = F.fibattn_forward(packed["q"], packed["k"], packed["v"], W, FIB, 0.9)
    out = torch.full((B, T, H, D + 16), float("nan"), device="cuda", dtype=dt)
    got, lse = F.fibattn_forward(views["q"], views["k"], views["v"], W, FIB, 0.9,
                                 o=out[..., :D].transpose(1, 2))
    torch.cuda.synchronize()
    assert torch.equal(got.contiguous(), want) and torch.equal(lse, want_lse)
    assert torch.isnan(out[..., D:]).all()


@pytest.mark.parametrize("B,H,Hkv,T,D,dtype,W,base,alpha", [
    (1, 2, 1, 150, 64, "bf16", 40, FIB, 0.9),
    (1, 2, 2, 150, 64, "bf16", 20, FIB, 1.0),
    (1, 2, 2, 90, 128, "bf16", 8, FIB, 1.0),
    (1, 2, 2, 90, 32, "bf16", 12, POW2, 0.8),
    (1, 2, 1, 90, 64, "fp32", 9, FIB, 0.9),
    (1, 1, 1, 90, 128, "fp32", 40, FIB, 1.0),
])
def test_tile_unattended_rows_that_are_not_finite(B, H, Hkv, T, D, dtype, W, base, alpha):
    # key j is NaN in K and inf in V: queries that do not attend it keep the results they
    # have with finite rows there, and those that do are not finite
    x = inputs.attention_inputs(B, H, T, D, dtype, 870, 0, names=("q", "dO"))
    x.update(inputs.attention_inputs(B, Hkv, T, D, dtype, 870, 0, names=("k", "v")))
    j = T // 2 + 3
    seen = torch.zeros(T, dtype=torch.bool)
    seen[j : j + W + 1] = True
    for d0, w, _, _ in oracle.rungs(alpha, base, W):
        seen[j + d0 : j + d0 + 1] = True
        # row r1: attended when w != 0, and read for dalpha (with weight w = 0 times it) else
        seen[j + d0 + 1 : j + d0 + 2] = True
    want = gpu_run(x["q"], x["k"], x["v"], x["dO"], W, base, alpha)
    x["k"][:, :, j], x["v"][:, :, j] = float("nan"), float("inf")
    got = gpu_run(x["q"], x["k"], x["v"], x["dO"], W, base, alpha)
    for n in ("o", "lse", "dq"):
        a, b = torch.from_numpy(got[n])[:, :, ~seen], torch.from_numpy(want[n])[:, :, ~seen]
        # the rows added again row by row: another order of the same sums
        scale = b.abs().max()
        assert torch.isfinite(a).all(), n
        assert (a - b).abs().max() <= (1e-5 if dtype == "fp32" else 1e-2) * scale, n
    assert not torch.isfinite(torch.from_numpy(got["o"])[:, :, j : j + W + 1]).all(-1).any()
    # query j is NaN in q and dO: keys it does not attend keep their gradients
    x["k"][:, :, j], x["v"][:, :, j] = 0.5, 0.5
    want = gpu_run(x["q"], x["k"], x["v"], x["dO"], W, base, alpha)
    x["q"][:, :, j], x["dO"][:, :, j] = float("nan"), float("nan")
    got = gpu_run(x["q"], x["k"], x["v"], x["dO"], W, base, alpha)
    seen = torch.zeros(T, dtype=torch.bool)
    seen[max(j - W, 0) : j + 1] = True
    for d0, w, _, _ in oracle.rungs(alpha, base, W):
        if j - d0 >= 0:
            seen[max(j - d0 - (w != 0), 0) : j - d0 + 1] = True
    for n in ("dk", "dv"):
        a, b = torch.from_numpy(got[n])[:, :, ~seen], torch.from_numpy(want[n])[:, :, ~seen]
        assert torch.isfinite(a).all(), n
        assert (a - b).abs().max() <= (1e-5 if dtype == "fp32" else 1e-2) * b.abs().max(), n
        assert not torch.isfinite(torch.from_numpy(got[n])[:, :, j - W : j + 1]).all(-1).any(), n


@pytest.mark.parametrize("B,H,T,D", [(1, 2, 129, 32), (2, 3, 65, 64), (1, 1, 17, 128), (8, 16, 700, 64)])
def test_float32_rotated_q_has_the_bits_of_the_rope_launch(B, H, T, D):
    # float32 rows rotated where the forward loads them: the launch's angles and order (the
    # last size takes the launch's two heads a lane), and the results of rotating before
    x = inputs.attention_inputs(B, H, T, D, "fp32", 880, 0)
    q, k, v = (x[n].cuda() for n in ("q", "k", "v"))
    K, Q = F.fibattn_rope(k), F.fibattn_rope(q)
    o, lse, got = F.fibattn_forward_rope_q(q, K, v, 12, FIB, 0.9)
    want_o, want_lse = F.fibattn_forward(Q, K, v, 12, FIB, 0.9)
    torch.cuda.synchronize()
    assert torch.equal(got, Q) and torch.equal(o, want_o) and torch.equal(lse, want_lse)


@pytest.mark.parametrize("G,T,D,W,base,alpha", [
    (1, 15, 32, 8, FIB, 0.9), (2, 64, 32, 40, FIB, 1.0), (1, 129, 32, 16, POW2, 1.2), (3, 17, 32, 0, FIB, 0.8),
    (1, 16, 64, 17, FIB, 1.0), (3, 65, 64, 12, FIB, 0.9), (2, 130, 64, 8, POW2, 0.8), (1, 100, 64, 128, FIB, 1.0),
    (1, 33, 128, 8, FIB, 0.9), (4, 63, 128, 16, FIB, 1.0), (2, 200, 128, 40, FIB, 1.1), (1, 1, 128, 3, FIB, 1.0)])
def test_float32_lanes(G, T, D, W, base, alpha):
    # float32 of few rows (D / 4 lanes a row) and of many (4 lanes): heads of the large call that
    # hold the same rows as the small one's have the same bits of o, lse and dq (rotated back),
    # from a host and from a device table, and dk, dv within the parity bound
    n = 12288 // (2 * G * T) + 1  # the small call n times over is past the line
    assert 2 * G * T <= 12288 < 2 * G * T * n
    x = inputs.attention_inputs(1, 2 * G, T, D, "fp32", 890, 0, names=("q", "dO"))
    x.update(inputs.attention_inputs(1, 2, T, D, "fp32", 890, 0, names=("k", "v")))
    table = F.fibattn_device_table(torch.tensor([alpha], device="cuda"), base, W)
    res = []
    for r in (1, n):
        q, k, v, dO = (x[m].cuda().repeat(r, 1, 1, 1) for m in ("q", "k", "v", "dO"))
        o, lse, Q = F.fibattn_forward_rope_q(q, k, v, W, base, alpha)
        od, ld = F.fibattn_forward_dt(Q, k, v, W, table)
        g = F.fibattn_backward(Q, k, v, o, lse, dO, W, base, alpha, rope_base=10000.0)
        gd = F.fibattn_backward_dt(Q, k, v, o, lse, dO, W, table, rope_base=10000.0)
        torch.cuda.synchronize()
        assert torch.equal(od, o) and torch.equal(ld, lse)
        assert torch.equal(g[0], gd[0]) and torch.equal(g[3], gd[3])
        for a, b in zip(g[1:3], gd[1:3]):  # (a device table has the interpolating order of rungs)
            assert (a - b).abs().max() <= 1e-5 * max(1.0, float(a.abs().max()))
        res.append((o, lse, Q, *g))
    for name, a, b in zip(("o", "lse", "Q", "dq"), *res):
        assert torch.equal(a.expand(n, *a.shape[1:]), b), name
    for name, a, b in zip(("dk", "dv"), res[0][4:], res[1][4:]):
        assert (a - b).abs().max() <= 1e-5 * max(1.0, float(a.abs().max())), name
    # n times the same terms
    assert abs(float(res[1][6]) - n * float(res[0][6])) <= 1e-5 * n * max(1.0, T * abs(float(res[0][6])))


@pytest.mark.parametrize("G,T,W,base,alpha", [(1, 65, 8, FIB, 0.9), (3, 33, 24, POW2, 1.0), (1, 1, 0, FIB, 1.0),
                                              (1, 200, 17, FIB, 1.0)])
def test_bfloat16_d128_dkdv_of_few_rows(G, T, W, base, alpha):
    # the kernel of few rows and the tile kernel give dk, dv (rotated back) of the same heads
    # within the rounding of the stored values and of the bfloat16 Delta they share
    n = 8192 // (2 * G * T) + 1
    x = inputs.attention_inputs(1, 2 * G, T, 128, "bf16", 895, 0, names=("q", "dO"))
    x.update(inputs.attention_inputs(1, 2, T, 128, "bf16", 895, 0, names=("k", "v")))
    res = []
    for r in (1, n):
        q, k, v, dO = (x[m].cuda().repeat(r, 1, 1, 1) for m in ("q", "k", "v", "dO"))
        o, lse = F.fibattn_forward(q, k, v, W, base, alpha)
        res.append(F.fibattn_backward(q, k, v, o, lse, dO, W, base, alpha, rope_base=10000.0)[1:3])
    torch.cuda.synchronize()
    for name, a, b in zip(("dk", "dv"), *res):
        a, b = a.double().expand(n, *a.shape[1:]), b.double()
        assert ((a - b).abs() <= 2.0 ** -7 * a.abs() + 1e-5 * a.abs().max()).all(), name
