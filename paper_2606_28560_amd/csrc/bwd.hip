// Backward kernels: dq + dalpha (query-stationary), dk/dv (key-stationary, no
// atomics), and the fixed-order dalpha reduction.
//
// The gradient is that of the forward in fwd.hip with the inclusion masks held
// constant (Section 2 "Implementation note": a hard mask carries no gradient to
// alpha, so alpha acts only through the blend weights, dw_k/dalpha = f_k).
// With p_e = exp(s_e - lse_i), Delta_i = <dO_i, o_i>, dP_e = <dO_i, vhat_e> and
// dS_e = p_e (dP_e - Delta_i):
//   dq_i   = tau sum_e dS_e khat_e
//   dk_j   = sum over entries e that read row j of  weight_e(j) tau dS_e q_i
//   dv_j   = sum over entries e that read row j of  weight_e(j) p_e dO_i
//   dL/dw  = tau dS_e <q_i, k[r1] - k[r0]> + p_e <dO_i, v[r1] - v[r0]>  (rung entries)
//   dalpha = sum_{b,h,i,rungs} f_k dL/dw
// The row -1 (reached only when w == 0) is a zero vector.
// dalpha is a sum with heavy cancellation (its magnitude is a small fraction of the
// sum of its terms' magnitudes), so it does not take Delta from the stored o (rounded
// to the storage type) but from the entries themselves, Delta_i = sum_e p_e dP_e (the
// same quantity, since o_i = sum_e p_e vhat_e): per query it accumulates
// Xa = sum f p dP <q, k[r1]-k[r0]>, Xb = sum f p <dO, v[r1]-v[r0]>, Y = sum f p <q, k[r1]-k[r0]>
// and the entries' sum of p dP, and adds tau (Xa - Delta Y) + Xb.
//
// Because every rung offset is shared, the queries that read key row j are again a
// fixed set of shifted positions: j .. j+W through the window, and j + floor(d_k)
// (as the row r0, weight 1-w) and j + floor(d_k) + 1 (as r1, weight w) through rung k.
// The dk/dv kernel therefore keeps its key rows and gathers their contributions, so
// every dk/dv row is written once, without atomics.
#include <algorithm>

#include "launch.h"
#include "tile.h"

namespace fibattn {

// ---------------------------------------------------------------------------
// dq, Delta and per-workgroup dalpha partials in bfloat16.
// ---------------------------------------------------------------------------
// A wave owns 16 consecutive queries (lane layouts in tile.h), as in the forward: the band
// chunks' K and V rows are staged in LDS, S = K.Q^T and dP = V.dO^T taken on the matrix
// cores, dq += K^T (tau dS) there; rungs are dot products of the rows r0 and r1 (r1 is
// needed for dalpha even when w = 0) on the VALU, four lanes per row.  The dalpha parts are
// multiplied and added up in float64.
//
// What bounds it: as the forward, the latency of the rung gathers and their VALU work.
// Against a kernel with one lane group per query, every row read from global memory by
// every query (us a launch, interpolating): bf16 d 64 B4 H8 T2048 W64 137 -> 21.7; bf16
// d 128 B2 H16 on 4 T2000 W8 79 -> 36.5; bf16 d 32 B8 H8 T1024 W10 23.3 -> 14.8 (the R^T of
// dq, then a launch of its own, not included in the first figure).

// dq and the dalpha parts of query ic, its entries one by one and only those it has, in the
// order of the float32 kernel (quad layout; nact rungs, the wave's).  The parts are the whole
// quad's, on its lane 0.
template <typename TL>
__device__ __forceinline__ void dq_by_entry(const typename TL::Slice &qq, const typename TL::Slice &gg, const void *K,
                                            const void *V, uint32_t sk, uint32_t sv, int ic, int gq, int W,
                                            const RungTable &rt, int nact, float tau, float sl2, float lse2, float delta,
                                            typename TL::Acc &acc, double &xa, double &xb, double &y, double &dsum) {
    TL::zero(acc);
    xa = xb = y = dsum = 0.0;
    for (int e = 0; e <= W + nact; ++e) {
        const int r = e - W - 1, d = r < 0 ? e : rt.d0[r];
        const float w = r < 0 ? 0.f : rt.w[r];
        const bool in = ic >= d + (w != 0.f), has1 = r >= 0 && ic > d;  // row -1 is the zero row
        const int r0 = in ? ic - d : ic, r1 = has1 ? ic - d - 1 : ic;
        const typename TL::Slice k0 = TL::load(K, r0, gq, sk), k1 = TL::load(K, r1, gq, sk);
        const float s0 = TL::row_dot(qq, k0), sn = TL::row_dot(qq, k1), s1 = has1 ? sn : 0.f;
        const float dP0 = TL::row_dot(gg, TL::load(V, r0, gq, sv));
        const float dPn = TL::row_dot(gg, TL::load(V, r1, gq, sv)), dP1 = has1 ? dPn : 0.f;
        const float s = w != 0.f ? (1.f - w) * s0 + w * s1 : s0;
        const float dP = w != 0.f ? (1.f - w) * dP0 + w * dP1 : dP0;
        const float p = exp2f(s * sl2 - lse2);
        const float c = r < 0 ? tau * p * (dP - delta) : tau * (p * (dP - delta));
        if (!in) continue;
        if (w != 0.f)
            TL::axpy2(acc, c * (1.f - w), k0, c * w, k1);
        else
            TL::axpy(acc, c, k0);
        dsum += (double)p * (double)dP;
        if (r < 0 || gq) continue;
        const double fp = (double)rt.f[r] * (double)p;
        xa += fp * (double)dP * (double)(s1 - s0);
        xb += fp * (double)(dP1 - dP0);
        y += fp * (double)(s1 - s0);
    }
}

template <int D>
constexpr int dq_waves = D <= 64 ? 4 : 3;

// DEV: the rung table is the one at rtp, built on the device (rt_arg unused).
template <int D, bool INTERP, bool DEV>
__global__ __launch_bounds__(256, (dq_waves<D>)) void bwd_dq_tile_kernel(
    const uint16_t *__restrict__ q, const uint16_t *__restrict__ k, const uint16_t *__restrict__ v,
    const uint16_t *__restrict__ o, const float *__restrict__ lse, const uint16_t *__restrict__ dO,
    uint16_t *__restrict__ dq, float *__restrict__ delta_out, double *__restrict__ partials, int T,
    int W, RungTable rt_arg, const RungTable *__restrict__ rtp, RopeFreq rf, float tau, float sl2, TileShape ts, Heads hd,
    Layouts lay) {
    using S = uint16_t;
    using TL = Tile<S, D>;
    using Slice = typename TL::Slice;
    const RungTable &rt = DEV ? *rtp : rt_arg;
    const bool bad = DEV && table_unusable(rt, W);  // bad device alpha, or another W
    constexpr int NBUF = TL::NC <= 1 ? 2 : 1;       // rungs in flight
    extern __shared__ __align__(16) char smem[];
    __shared__ double sfreq[D / 2], red[4];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nw = blockDim.x >> 6;
    const int nm = lane & 15, gm = lane >> 4;  // MFMA layout
    const int nq = lane >> 2, gq = lane & 3;   // quad layout
    if (block_number() >= ts.blocks) return;
    const int blk = xcd_remap(block_number(), ts.blocks);
    const int runs = nw / ts.hs, wv = wave / ts.hs;
    const int bh = (blk / ts.tiles) * ts.hs + wave % ts.hs;  // this wave's query head
    const int T0 = (blk % ts.tiles) * 16 * runs;
    const int bk = hd.kv_of(bh);
    const S *K = k + lay.k.head(bk, hd.kv_heads());
    const S *V = v + lay.v.head(bk, hd.kv_heads());
    constexpr int es = (int)sizeof(S);
    const uint32_t sk = (uint32_t)(lay.k.st * es), sv = (uint32_t)(lay.v.st * es);

    const int t0 = T0 + 16 * wv;
    const int im = t0 + nm;                     // MFMA layout query
    const int i = t0 + nq, ic = min(i, T - 1);  // quad layout query
    const S *Q = q + lay.q.head(bh, hd.H), *G = dO + lay.g.head(bh, hd.H);
    Slice qq = TL::load(Q, ic, gq, (uint32_t)(lay.q.st * es));
    Slice gg = TL::load(G, ic, gq, (uint32_t)(lay.g.st * es));
    const float lse2 = lse[(size_t)bh * T + ic] * kLog2e;
    float delta;
    {
        const Slice oo = TL::load(o + lay.o.head(bh, hd.H), ic, gq, (uint32_t)(lay.o.st * es));
        delta = quad_sum(TL::dot(gg, oo));
    }
    if (rf.on && threadIdx.x < D / 2) sfreq[threadIdx.x] = rf.inv[threadIdx.x] * 0.15915494309189533576888376337251;

    int nact = 0;  // rungs some query of this wave includes: a prefix of the table
#pragma unroll
    for (int r = 0; r < kMaxRungs; ++r) nact += ((r < rt.n) & (rt.d0[r] <= min(t0 + 15, T - 1))) ? 1 : 0;
    nact = t0 < T ? __builtin_amdgcn_readfirstlane(nact) : 0;
    // rows r0 and r1 of rung r (an entry the query does not have reads the query's own row,
    // as in the forward)
    auto load_rung = [&](int r, const void *X, uint32_t st, Slice *x) {
        const int d = rt.d0[r], lim = INTERP && rt.w[r] != 0.f ? d + 1 : d;
        x[0] = TL::load(X, ic >= lim ? ic - d : ic, gq, st);
        x[1] = TL::load(X, ic > d ? ic - d - 1 : ic, gq, st);
    };
    Slice kx[NBUF][2], vx[NBUF][2];
    // in flight during the band phase, as far as the registers go
    if (TL::NC <= 2 && nact > 0) load_rung(0, V, sv, vx[0]);
    if (TL::NC <= 1 && nact > 0) load_rung(0, K, sk, kx[0]);

    // ---- window band (MFMA layout) ----
    typename TL::Acc acc;
    TL::zero(acc);
    double dsum = 0.0;  // the entries' sum of p dP (this lane's part)
    bool weak = false, tiny = false;  // weights that tiny_weight names, and large rows beside them
    {
        const Slice qm = TL::from_quad(qq, lane), gmm = TL::from_quad(gg, lane);
        const float lse2_m = __shfl(lse2, 4 * nm, 64), delta_m = __shfl(delta, 4 * nm, 64);
        const unsigned reach = (unsigned)min(W, im);  // 0 <= im - key <= W and key >= 0
        const int nc = min(ts.nc, (T0 + 16 * runs + 31) >> 5);
        for (int c0 = 0; c0 < nc; c0 += ts.cps) {
            // chunks as in the forward
            const int n = min(ts.cps, nc - c0);
            const int rbeg = T0 + 16 - 32 * (c0 + n), rows = 16 * (runs - 1) + 32 * n;
            char *kr = smem, *vr = smem + rows * TL::kRow;
            if (c0 > 0) __syncthreads();  // every wave is done with the rows staged before
            TL::stage(kr, K, rbeg, rows, T, lay.k.st, wave, nw);
            TL::stage(vr, V, rbeg, rows, T, lay.v.st, wave, nw);
            wait_vmem();
            __syncthreads();
            float least = INFINITY;
            for (int c = 0; c < n; ++c) {
                if (t0 + 16 - 32 * (c0 + c) <= 0) break;
                const int base = 16 * wv + 32 * (n - 1 - c);
                float ds[8];
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    const f32x4 s = TL::scores(TL::staged(kr, base + 16 * b + nm, gm), qm);
                    const f32x4 dp = TL::scores(TL::staged(vr, base + 16 * b + nm, gm), gmm);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int key = rbeg + base + 16 * b + 4 * gm + e;
                        const bool in = (unsigned)(im - key) <= reach;
                        const float xe = fmaf(s[e], sl2, -lse2_m);
                        least = fminf(least, xe);
                        const float p = in ? fast_exp2(xe) : 0.f, dP = in ? dp[e] : 0.f;
                        ds[4 * b + e] = tau * p * (dP - delta_m);
                        dsum = fma((double)p, (double)dP, dsum);
                    }
                }
                TL::accumulate(acc, kr, base, TL::weights(ds), gm);
            }
            if (tiny_weight(least))
                tiny |= TL::large_rows(kr, 16 * wv, 32 * n) || TL::large_rows(vr, 16 * wv, 32 * n), weak = true;
        }
    }
    if constexpr (TL::NC > 2) {
        // wide rows: read again rather than held through the band phase (which would spill)
        int row = ic;
        asm volatile("" : "+v"(row));
        qq = TL::load(Q, row, gq, (uint32_t)(lay.q.st * es));
        gg = TL::load(G, row, gq, (uint32_t)(lay.g.st * es));
    }
    if (nact > 0) {
        if (TL::NC > 2) load_rung(0, V, sv, vx[0]);
        if (TL::NC > 1) load_rung(0, K, sk, kx[0]);
    }
    if (weak) tiny |= TL::large_rows(gg);
    TL::to_quad_acc(acc, lane);
    // the query's band sum, on each of its four quad lanes
    dsum += __shfl_xor(dsum, 16, 64);
    dsum += __shfl_xor(dsum, 32, 64);
    dsum = __shfl(dsum, nq, 64);

    // ---- rungs (quad layout); row r1 = -1 is the zero row ----
    // xa, xb, y: this lane's parts of the sums over <q, k[r1]-k[r0]> and <dO, v[r1]-v[r0]>
    double xa = 0.0, xb = 0.0, y = 0.0;
    float dP = 0.f, dv = 0.f;
    auto value_dots = [&](int r, const Slice *x) {
        const bool has1 = i - rt.d0[r] - 1 >= 0;
        const float w = rt.w[r];
        const float a = TL::dot(gg, x[0]), t = TL::dot(gg, x[1]), b = has1 ? t : 0.f;
        dv = b - a;
        dP = quad_sum(INTERP ? (1.f - w) * a + w * b : a);
    };
    auto key_terms = [&](int r, const Slice *x) {
        const int d0 = rt.d0[r];
        const float w = rt.w[r];
        const bool in = i < T && (INTERP ? d0 < i || (d0 == i && w == 0.f) : d0 <= i);
        const float a = TL::dot(qq, x[0]), t = TL::dot(qq, x[1]), b = i - d0 - 1 >= 0 ? t : 0.f;
        const float s = quad_sum(INTERP ? (1.f - w) * a + w * b : a);
        const float p = in ? exp2f(fmaf(s, sl2, -lse2)) : 0.f;
        const float c = tau * p * (dP - delta);
        if constexpr (INTERP)
            TL::axpy2(acc, c * (1.f - w), x[0], c * w, x[1]);
        else
            TL::axpy(acc, c, x[0]);
        const double fp = (double)rt.f[r] * (double)p, ds = (double)(b - a);
        xa = fma(fp * (double)dP, ds, xa);
        xb = fma(fp, (double)dv, xb);
        y = fma(fp, ds, y);
        dsum = fma((double)p, (double)dP, dsum);
    };
    if constexpr (NBUF == 2) {
        for (int r = 0; r < nact; r += 2) {
            if (r + 1 < nact) {
                load_rung(r + 1, V, sv, vx[1]);
                load_rung(r + 1, K, sk, kx[1]);
            }
            value_dots(r, vx[0]);
            key_terms(r, kx[0]);
            if (r + 1 < nact) {
                if (r + 2 < nact) {
                    load_rung(r + 2, V, sv, vx[0]);
                    load_rung(r + 2, K, sk, kx[0]);
                }
                value_dots(r + 1, vx[1]);
                key_terms(r + 1, kx[1]);
            }
        }
    } else {
        // one buffer each: the next rung's values load while this one's keys are used (held
        // there: loads moved across spill 2 to 24 registers at d 128)
        for (int r = 0; r < nact; ++r) {
            const int nx = min(r + 1, nact - 1);
            value_dots(r, vx[0]);
            load_rung(nx, V, sv, vx[0]);
            __builtin_amdgcn_sched_barrier(0);
            key_terms(r, kx[0]);
            load_rung(nx, K, sk, kx[0]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // as in the forward: entries the query does not have took part with weights of 0
    if (tiny || __builtin_amdgcn_ballot_w64(!(TL::finite(acc) && (xa + xb + y + dsum) * 0.0 == 0.0)))
        dq_by_entry<TL>(qq, gg, K, V, sk, sv, ic, gq, W, rt, nact, tau, sl2, lse2, delta, acc, xa, xb, y, dsum);

    if (rf.on) TL::rope_t(acc, i, sfreq, gq);  // gradient w.r.t. the unrotated q
    if (i < T) {
        TL::store(dq + lay.dq.head(bh, hd.H) + i * lay.dq.st, gq, acc, bad ? NAN : 1.f);
        if (gq == 0) delta_out[(size_t)bh * T + i] = bad ? NAN : delta;
    }
    // this lane's part of the query's dalpha; wave sums, then the waves in order
    double dal = i < T ? (double)tau * (xa - dsum * y) + xb : 0.0;
    if (bad) dal = NAN;
#pragma unroll
    for (int st = 32; st >= 1; st >>= 1) dal += __shfl_xor(dal, st, 64);
    if (lane == 0) red[wave] = dal;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = red[0];
        for (int u = 1; u < nw; ++u) s += red[u];
        partials[block_number()] = s;
    }
}

// ---------------------------------------------------------------------------
// dq, Delta and dalpha partials in float32: as the forward's float32 kernel, L lanes per
// query on the VALU, every sum in the order that tile.h states.  The window's K and V rows
// are shared by the queries of a tile; staged in LDS they take the launch
// of B4 H8 T1024 d 64 W 12 from 26.1 to 22.3 us (the forward, which reads each tensor's
// window once, gained nothing from it).
// ---------------------------------------------------------------------------
template <int D, int L, bool DEV>
__global__ __launch_bounds__(256, 2) void bwd_dq_f32_kernel(
    const float *__restrict__ q, const float *__restrict__ k, const float *__restrict__ v,
    const float *__restrict__ o, const float *__restrict__ lse, const float *__restrict__ dO,
    float *__restrict__ dq, float *__restrict__ delta_out, double *__restrict__ partials, int T, int W,
    RungTable rt_arg, const RungTable *__restrict__ rtp, RopeFreq rf, float tau, int tiles, int blocks, int rows,
    Heads hd, Layouts lay) {
    using TL = Tile<float, D, L>;
    using Slice = typename TL::Slice;
    const RungTable &rt = DEV ? *rtp : rt_arg;
    const bool bad = DEV && table_unusable(rt, W);  // bad device alpha, or another W
    extern __shared__ __align__(16) char smem[];
    __shared__ double sfreq[D / 2], red[4];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    constexpr int RW = 64 / L, QPB = 4 * RW;  // queries per wave and workgroup
    const int nq = lane / L, gq = lane % L;
    if (block_number() >= blocks) return;
    const int blk = xcd_remap(block_number(), blocks);
    const int bh = blk / tiles, T0 = (blk % tiles) * QPB, t0 = T0 + RW * wave;
    const int bk = hd.kv_of(bh);
    const float *K = k + lay.k.head(bk, hd.kv_heads());
    const float *V = v + lay.v.head(bk, hd.kv_heads());
    const uint32_t sk = (uint32_t)(4 * lay.k.st), sv = (uint32_t)(4 * lay.v.st);
    const int i = t0 + nq, ic = min(i, T - 1), last = min(t0 + RW - 1, T - 1);
    const float sl2 = tau * kLog2e;
    const Slice qq = TL::load(q + lay.q.head(bh, hd.H), ic, gq, (uint32_t)(4 * lay.q.st));
    const Slice gg = TL::load(dO + lay.g.head(bh, hd.H), ic, gq, (uint32_t)(4 * lay.g.st));
    const float delta = TL::row_dot(gg, TL::load(o + lay.o.head(bh, hd.H), ic, gq, (uint32_t)(4 * lay.o.st)));
    const float lse2 = lse[(size_t)bh * T + ic] * kLog2e;
    // the window's rows of the workgroup, [T0 + 64 - rows, T0 + 64), where they are staged
    // (four lanes per query only)
    if constexpr (L != 4) rows = 0;
    const int rbeg = T0 + 64 - rows;
    char *kr = smem, *vr = smem + rows * TL::kRow;
    if (rows > 0) {
        TL::stage(kr, K, rbeg, rows, T, lay.k.st, wave, 4, true);
        TL::stage(vr, V, rbeg, rows, T, lay.v.st, wave, 4, true);
    }
    if (rf.on && threadIdx.x < D / 2) sfreq[threadIdx.x] = rf.inv[threadIdx.x] * 0.15915494309189533576888376337251;
    int nact = 0;  // rungs some query of this wave includes: a prefix of the table
#pragma unroll
    for (int r = 0; r < kMaxRungs; ++r) nact += ((r < rt.n) & (rt.d0[r] <= last)) ? 1 : 0;
    nact = t0 < T ? __builtin_amdgcn_readfirstlane(nact) : 0;
    const int reach = min(W, ic), nwin = t0 < T ? min(W, last) + 1 : 0;

    typename TL::Acc acc;
    TL::zero(acc);
    double xa = 0.0, xb = 0.0, y = 0.0, dsum = 0.0;  // dalpha parts, Delta from the entries
    wait_vmem();
    __syncthreads();
    // an entry the query does not have reads the query's own row
    for (int d = 0; d < nwin; d += 2) {
        Slice kk[2], vv[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int row = d + u <= reach ? ic - d - u : ic;
            kk[u] = rows > 0 ? TL::staged_quad(kr, row - rbeg, gq) : TL::load(K, row, gq, sk);
            vv[u] = rows > 0 ? TL::staged_quad(vr, row - rbeg, gq) : TL::load(V, row, gq, sv);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const float s = TL::row_dot(qq, kk[u]);
            const float dP = TL::row_dot(gg, vv[u]);
            const float p = d + u <= reach ? exp2f(s * sl2 - lse2) : 0.f;
            const float c = tau * p * (dP - delta);
            dsum += (double)p * (double)dP;
            TL::axpy(acc, c, kk[u]);
        }
    }
    // rows r0 and r1 of rung r
    auto load_rung = [&](int r, const void *X, uint32_t st, Slice *x) {
        const int d = rt.d0[r], lim = rt.w[r] != 0.f ? d + 1 : d;
        x[0] = TL::load(X, ic >= lim ? ic - d : ic, gq, st);
        x[1] = TL::load(X, ic > d ? ic - d - 1 : ic, gq, st);
    };
    Slice kx[2], vx[2];
    if (nact > 0) {
        load_rung(0, V, sv, vx);
        load_rung(0, K, sk, kx);
    }
    // the next rung's values load while this one's keys are used
    for (int r = 0; r < nact; ++r) {
        const int d0 = rt.d0[r], nx = min(r + 1, nact - 1);
        const float w = rt.w[r];
        const bool in = ic >= d0 + (w != 0.f), has1 = ic > d0;  // row -1 is the zero row
        const float dP0 = TL::row_dot(gg, vx[0]), dPn = TL::row_dot(gg, vx[1]), dP1 = has1 ? dPn : 0.f;
        load_rung(nx, V, sv, vx);
        const float s0 = TL::row_dot(qq, kx[0]), sn = TL::row_dot(qq, kx[1]), s1 = has1 ? sn : 0.f;
        const float s = (1.f - w) * s0 + w * s1;
        const float dP = (1.f - w) * dP0 + w * dP1;
        const float p = in ? exp2f(s * sl2 - lse2) : 0.f;
        const float dS = p * (dP - delta);
        const float c = tau * dS;
        TL::axpy2(acc, c * (1.f - w), kx[0], c * w, kx[1]);
        load_rung(nx, K, sk, kx);
        const double fp = (double)rt.f[r] * (double)p;
        xa += fp * (double)dP * (double)(s1 - s0);
        xb += fp * (double)(dP1 - dP0);
        y += fp * (double)(s1 - s0);
        dsum += (double)p * (double)dP;
    }
    if (__builtin_amdgcn_ballot_w64(!(TL::finite(acc) && (xa + xb + y + dsum) * 0.0 == 0.0)))
        dq_by_entry<TL>(qq, gg, K, V, sk, sv, ic, gq, W, rt, nact, tau, sl2, lse2, delta, acc, xa, xb, y, dsum);
    double dal = gq == 0 && i < T ? (double)tau * (xa - dsum * y) + xb : 0.0;
    if (bad) dal = NAN;
    if (rf.on) TL::rope_t(acc, i, sfreq, gq);  // gradient w.r.t. the unrotated q
    if (i < T) {
        TL::store(dq + lay.dq.head(bh, hd.H) + i * lay.dq.st, gq, acc, bad ? NAN : 1.f);
        if (gq == 0) delta_out[(size_t)bh * T + i] = bad ? NAN : delta;
    }
#pragma unroll
    for (int st = 32; st >= 1; st >>= 1) dal += __shfl_xor(dal, st, 64);
    if (lane == 0) red[wave] = dal;
    __syncthreads();
    if (threadIdx.x == 0) partials[block_number()] = ((red[0] + red[1]) + red[2]) + red[3];
}

// ---------------------------------------------------------------------------
// dk, dv: key-stationary, no atomics.
// ---------------------------------------------------------------------------
// A wave owns 16 consecutive keys of one key/value head and the terms of one query head at
// a time; the waves of a workgroup are ts.hs query heads of the group side by side times
// runs of 16 keys, a group of G heads takes G / hs passes, and the heads' sums meet in LDS
// at the end.
//   - window band: the queries j .. j + W lie in 32-row chunks from the wave's first key on.
//     Their q and dO rows are staged in LDS; S = Q.K^T and dP = dO.V^T on the matrix cores,
//     dk += Q^T (tau dS) and dv += dO^T P there (weights as in tile.h);
//   - rungs, four lanes per key: query i0 = j + floor(d) reads key j as r0 (weight 1 - w)
//     and j - 1 as r1, query i0 + 1 reads j + 1 as r0 and j as r1 (weight w).  A key takes
//     the products of its own row with both queries; the two with its neighbours' rows
//     are those of the keys four lanes before and on.  For the wave's first and last key
//     (the edges) they are taken before the loop, 16 rungs at a time.
//
// What bounds it: as dq, the latency of the rung gathers and their VALU work (47 to 54 % of
// the issue slots in bfloat16); two (NC 4) or four (NC 2) waves per SIMD, as the registers of
// two query and two dO rows in flight allow.  Us a launch, against one lane group per key,
// every query row read from global memory by every key it attends (R^T of dk and the dalpha
// sum then launches of their own, not included): bf16 d 64 B4 H8 T2048 W64 103 -> 28.3; bf16
// d 128 B2 H16 on 4 T2000 W8 104 -> 53.6; bf16 d 32 B8 H8 T1024 W10 25.6 -> 18.5; fp32 d 64
// B4 H8 T1024 W12 52 -> 25.6.

// The terms of one query head in dk, dv of key j, its queries one by one and only those that
// read it (quad layout; nact rungs, the wave's).
template <typename TL>
__device__ __forceinline__ void dkdv_by_entry(const void *Q, const void *G, const void *K, const void *V, const float *L,
                                              const float *Dl, uint32_t sq, uint32_t sg, uint32_t sk, uint32_t sv,
                                              int j, int gq, int T, int W, const RungTable &rt, int nact, float tau,
                                              float sl2, typename TL::Acc &adk, typename TL::Acc &adv) {
    const typename TL::Slice kj = TL::load(K, j, gq, sk), vj = TL::load(V, j, gq, sv);
    // a window entry, or one of the two of a rung: y = 0 with key j as row r0, 1 as row r1
    for (int e = 0; e <= W + 2 * nact; ++e) {
        const int r = e <= W ? -1 : (e - W - 1) >> 1, y = e <= W ? 0 : (e - W - 1) & 1;
        const float w = r < 0 ? 0.f : rt.w[r], wt = y ? w : 1.f - w;
        const int i = j + (r < 0 ? e : rt.d0[r] + y);
        const bool in = i < T && (w == 0.f ? y == 0 : y || j >= 1);
        const int row = in ? i : j, nb = y ? min(j + 1, T - 1) : max(j - 1, 0);  // the entry's other row
        const typename TL::Slice x = TL::load(Q, row, gq, sq), g = TL::load(G, row, gq, sg);
        float s = TL::row_dot(x, kj), dP = TL::row_dot(g, vj);
        if (w != 0.f) {
            s = fmaf(1.f - wt, TL::row_dot(x, TL::load(K, nb, gq, sk)), wt * s);
            dP = fmaf(1.f - wt, TL::row_dot(g, TL::load(V, nb, gq, sv)), wt * dP);
        }
        const float p = prob(s, sl2, L[row] * kLog2e);
        if (!in) continue;
        TL::axpy(adk, tau * p * (dP - Dl[row]) * wt, x);
        TL::axpy(adv, p * wt, g);
    }
}

// dalpha: the partials of the dq kernel, which has completed, in a fixed order (by the whole
// workgroup; red: a value per thread).
template <bool DEV>
__device__ __forceinline__ void sum_partials(double *red, const double *partials, int n, float *dalpha, float *dtheta,
                                             const RungTable &rt) {
    double s = 0.0;
    for (int t = threadIdx.x; t < n; t += blockDim.x) s += partials[t];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int st = blockDim.x >> 1; st >= 1; st >>= 1) {
        if ((int)threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const float da = (float)red[0];
        *dalpha = da;
        // a table built from theta: d L / d theta = dalpha * d alpha / d theta
        if (DEV && dtheta) *dtheta = (float)((double)da * rt.dadtheta);
    }
    __syncthreads();
}

template <typename S, int D>
constexpr int dkdv_waves = Tile<S, D>::kF32 ? (D == 32 ? 3 : D == 64 ? 2 : 1) : Tile<S, D>::NC <= 2 ? 4 : 2;

template <typename S, int D, bool INTERP, bool DEV>
__global__ __launch_bounds__(256, (dkdv_waves<S, D>)) void bwd_dkdv_tile_kernel(
    const S *__restrict__ q, const S *__restrict__ k, const S *__restrict__ v,
    const float *__restrict__ lse, const S *__restrict__ dO, const float *__restrict__ delta_in,
    S *__restrict__ dk, S *__restrict__ dv, const double *__restrict__ partials, int n_partials,
    float *__restrict__ dalpha, float *__restrict__ dtheta, int T, int W, RungTable rt_arg,
    const RungTable *__restrict__ rtp, RopeFreq rf, float tau, float sl2, TileShape ts, Heads hd, Layouts lay) {
    using TL = Tile<S, D>;
    using Slice = typename TL::Slice;
    const RungTable &rt = DEV ? *rtp : rt_arg;
    extern __shared__ __align__(16) char smem[];
    __shared__ double sfreq[D / 2];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nw = blockDim.x >> 6;
    const int nm = lane & 15, gm = lane >> 4;  // MFMA layout
    const int nq = lane >> 2, gq = lane & 3;   // quad layout
    if (block_number() >= ts.blocks) return;
    const int blk = xcd_remap(block_number(), ts.blocks);
    const int runs = nw / ts.hs, wv = wave / ts.hs, hs = wave % ts.hs;  // run of keys, head slot
    const int bk = blk / ts.tiles;  // batch * key/value heads + key/value head
    const int T0 = (blk % ts.tiles) * 16 * runs;
    const S *K = k + lay.k.head(bk, hd.kv_heads());
    const S *V = v + lay.v.head(bk, hd.kv_heads());
    constexpr int es = (int)sizeof(S);
    const uint32_t sq = (uint32_t)(lay.q.st * es), sg = (uint32_t)(lay.g.st * es);
    const uint32_t sk = (uint32_t)(lay.k.st * es), sv = (uint32_t)(lay.v.st * es);
    if (rf.on && threadIdx.x < D / 2) sfreq[threadIdx.x] = rf.inv[threadIdx.x] * 0.15915494309189533576888376337251;

    if (block_number() == 0)
        sum_partials<DEV>(reinterpret_cast<double *>(smem), partials, n_partials, dalpha, dtheta, rt);

    const int t0 = T0 + 16 * wv;
    const int jm = t0 + nm;                     // MFMA layout key
    const int j = t0 + nq, jc = min(j, T - 1);  // quad layout key
    Slice kj = TL::load(K, jc, gq, sk), vj = TL::load(V, jc, gq, sv);
    int nact = 0;  // rungs through which a query reads some key of this wave: a prefix
#pragma unroll
    for (int r = 0; r < kMaxRungs; ++r) nact += ((r < rt.n) & (rt.d0[r] < T - t0)) ? 1 : 0;
    nact = __builtin_amdgcn_readfirstlane(nact);
    const int passes = hd.G / ts.hs;

    // ---- window band (MFMA layout) ----
    // float32 with a window of one chunk: on the VALU, every product in the forward's order.
    // The rounding of a logit is then the one that lse holds too, and cancels in the
    // probability; logits from the matrix cores have errors of their own (dk, dv 5 to 25 %
    // further from 64 bits than the VALU's at W <= 16, nearer at W >= 24; B4 H8 T1024 d 64
    // W 12: 25.1 us with them, 25.6 here).
    const bool valu = TL::kF32 && W <= 16;
    bool tiny = false;
    typename TL::Acc adk, adv;
    TL::zero(adk);
    TL::zero(adv);
    {
        const Slice km = TL::from_quad(kj, lane), vm = TL::from_quad(vj, lane);
        const unsigned reach = (unsigned)min(W, T - 1 - jm);  // 0 <= query - jm <= W and query < T
        bool first = true;
        const int nc = min(ts.nc, (T - T0 + 31) >> 5);  // chunks with rows below T
        for (int pass = 0; pass < passes; ++pass)
            for (int c0 = 0; c0 < nc; c0 += ts.cps) {
                // chunks c0 .. c0 + n - 1 of every run: chunk c of run wv is the queries
                // [T0 + 16 wv + 32 c, T0 + 16 wv + 32 (c + 1))
                const int n = min(ts.cps, nc - c0);
                const int rbeg = T0 + 32 * c0, rows = 16 * (runs - 1) + 32 * n;
                char *qr = smem, *gr = smem + ts.hs * rows * TL::kRow;
                float *sl = reinterpret_cast<float *>(gr + ts.hs * rows * TL::kRow), *sd = sl + ts.hs * rows;
                if (!first) __syncthreads();  // every wave is done with the rows staged before
                first = false;
                for (int u = 0; u < ts.hs; ++u) {
                    const int bh = hd.q_of(bk, pass * ts.hs + u);
                    TL::stage(qr + u * rows * TL::kRow, q + lay.q.head(bh, hd.H), rbeg, rows, T, lay.q.st, wave, nw);
                    TL::stage(gr + u * rows * TL::kRow, dO + lay.g.head(bh, hd.H), rbeg, rows, T, lay.g.st, wave, nw);
                }
                for (int x = threadIdx.x; x < ts.hs * rows; x += blockDim.x) {
                    const size_t at = (size_t)hd.q_of(bk, pass * ts.hs + x / rows) * T + min(rbeg + x % rows, T - 1);
                    sl[x] = TL::kF32 && !valu ? lse[at] : lse[at] * kLog2e;  // as prob and prob_low take it
                    sd[x] = delta_in[at];
                }
                wait_vmem();
                __syncthreads();
                const char *qb = qr + hs * rows * TL::kRow, *gb = gr + hs * rows * TL::kRow;
                if (valu) {  // one chunk: query j + d in staged row 16 wv + nq + d
                    int row = jc;
                    asm volatile("" : "+v"(row));  // read here, not held beside the other path's
                    const Slice ka = TL::load(K, row, gq, sk), va = TL::load(V, row, gq, sv);
                    for (int d = 0; d <= W; ++d) {
                        const int r = 16 * wv + nq + d;
                        const bool in = j + d < T;
                        Slice x = TL::staged(qb, r, gq), y = TL::staged(gb, r, gq);
                        const float s = TL::row_dot(x, ka), dP = TL::row_dot(y, va);
                        const float pr = prob(s, sl2, sl[hs * rows + r]);
                        const float c = in ? tau * pr * (dP - sd[hs * rows + r]) : 0.f;
                        if (__builtin_amdgcn_ballot_w64(!in)) {  // clamped rows: 0 times them must be 0
#pragma unroll
                            for (int e = 0; e < TL::NC; ++e) {
                                x.c[e] = in ? x.c[e] : u32x4{0u, 0u, 0u, 0u};
                                y.c[e] = in ? y.c[e] : u32x4{0u, 0u, 0u, 0u};
                            }
                        }
                        TL::axpy(adk, c, x);
                        TL::axpy(adv, in ? pr : 0.f, y);
                    }
                    continue;
                }
                float least = INFINITY;
                for (int c = 0; c < n; ++c) {
                    if (t0 + 32 * (c0 + c) >= T) break;
                    const int base = 16 * wv + 32 * c;  // the chunk's first staged row
                    float ds[8], p[8];
#pragma unroll
                    for (int b = 0; b < 2; ++b) {
                        constexpr int CH = TL::NC == 2 ? 4 : 8;
                        const f32x4 s = TL::template scores<CH>(TL::staged(qb, base + 16 * b + nm, gm), km);
                        const f32x4 dp = TL::template scores<CH>(TL::staged(gb, base + 16 * b + nm, gm), vm);
                        const int si = base + 16 * b + 4 * gm;
                        const f32x4 l2 = *reinterpret_cast<const f32x4 *>(sl + hs * rows + si);
                        const f32x4 de = *reinterpret_cast<const f32x4 *>(sd + hs * rows + si);
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const bool in = jm < T && (unsigned)(rbeg + si + e - jm) <= reach;
                            float x;
                            if constexpr (TL::kF32) {
                                x = prob_low(s[e], sl2, l2[e]);
                            } else {
                                const float xe = fmaf(s[e], sl2, -l2[e]);
                                least = fminf(least, xe);
                                x = fast_exp2(xe);
                            }
                            p[4 * b + e] = in ? x : 0.f;
                            ds[4 * b + e] = in ? tau * x * (dp[e] - de[e]) : 0.f;
                        }
                    }
                    TL::accumulate(adk, qb, base, TL::weights(ds), gm);
                    TL::accumulate(adv, gb, base, TL::weights(p), gm);
                }
                if constexpr (!TL::kF32)
                    if (tiny_weight(least)) {
                        tiny |= TL::large_rows(qb, 16 * wv, 32 * n) || TL::large_rows(gb, 16 * wv, 32 * n) ||
                                TL::large_rows(vm);
                        for (int x = lane; x < 32 * n; x += 64)  // Delta, which is as large as o
                            tiny |= fabsf(sd[hs * rows + 16 * wv + x]) >= 0x1p40f;
                        tiny = __builtin_amdgcn_ballot_w64(tiny);
                    }
            }
    }
    if (!valu) {
        TL::to_quad_acc(adk, lane);
        TL::to_quad_acc(adv, lane);
    }
    if constexpr (TL::NC > 1) {
        // read again rather than held through the band phase
        int row = jc;
        asm volatile("" : "+v"(row));
        kj = TL::load(K, row, gq, sk);
        vj = TL::load(V, row, gq, sv);
    }

    // ---- rungs (quad layout) ----
    for (int pass = 0; pass < (nact > 0 ? passes : 0); ++pass) {
        // opaque copies keep the index arithmetic inside the pass loop (hoisted for all
        // rungs at once it would not fit the registers)
        int jp = j, tp = t0;
        asm volatile("" : "+v"(jp), "+s"(tp));
        const int bh = hd.q_of(bk, pass * ts.hs + hs);
        const S *Q = q + lay.q.head(bh, hd.H), *G = dO + lay.g.head(bh, hd.H);
        const float *L = lse + (size_t)bh * T, *Dl = delta_in + (size_t)bh * T;
        // Query rows of a rung: those of i0 and i0 + 1, or those of two rungs.  A query that
        // does not read the key is replaced by the one at the key's own position, which does.
        Slice xq[2], xg[2];
        float xl[2], xd[2];
        auto has = [&](int r, int y) {
            if constexpr (INTERP) {
                const bool two = rt.w[r] != 0.f;  // row r1 exists
                return jp + rt.d0[r] + y < T && (y ? two : !two || jp >= 1);
            } else {
                return r + y < nact && jp + rt.d0[min(r + y, nact - 1)] < T;
            }
        };
        auto row_of = [&](int r, int y) {
            return has(r, y) ? jp + (INTERP ? rt.d0[r] + y : rt.d0[min(r + y, nact - 1)]) : min(jp, T - 1);
        };
        auto load_q = [&](int r) {
#pragma unroll
            for (int y = 0; y < 2; ++y) {
                const int row = row_of(r, y);
                xq[y] = TL::load(Q, row, gq, sq);
                xl[y] = L[row];
                xd[y] = Dl[row];
            }
        };
        auto load_g = [&](int r) {
#pragma unroll
            for (int y = 0; y < 2; ++y) xg[y] = TL::load(G, row_of(r, y), gq, sg);
        };

        // <q, k> and <dO, v> of the wave's edges, rung nq (and nq + 16) on this quad: query
        // t0 + d with key t0 - 1, query t0 + 16 + d with key t0 + 16
        float es_[2][2], ep_[2][2];
        if constexpr (INTERP) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    es_[h][u] = ep_[h][u] = 0.f;
                    if (16 * h < nact) {
                        const int i = tp + 16 * u + rt.d0[min(nq + 16 * h, nact - 1)];
                        const int key = u ? min(tp + 16, T - 1) : max(tp - 1, 0), row = i < T ? i : key;
                        es_[h][u] = TL::row_dot(TL::load(Q, row, gq, sq), TL::load(K, key, gq, sk));
                        ep_[h][u] = TL::row_dot(TL::load(G, row, gq, sg), TL::load(V, key, gq, sv));
                    }
                }
        }
        load_q(0);
        load_g(0);
        constexpr int RB = INTERP ? 1 : 2;
        for (int r = 0; r < nact; r += RB) {
            const int nx = min(r + RB, nact - 1);
            // logits and dP of the two entries
            float s[2], dP[2], c[2], p[2];
#pragma unroll
            for (int y = 0; y < 2; ++y) {
                s[y] = TL::row_dot(xq[y], kj);
                dP[y] = TL::row_dot(xg[y], vj);
            }
            if constexpr (INTERP) {
                // query i0 with key j - 1 is query i0 + 1 of the key four lanes before,
                // query i0 + 1 with key j + 1 is query i0 of the key four lanes on
                const float w = rt.w[r];
                auto shift = [&](float x, int by, bool edge, const float *e0, const float *e1, int u) {
                    const float y = __shfl(x, lane + by, 64);
                    const float e = r < 16 ? e0[u] : e1[u];
                    const float z = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(e), 4 * (r & 15)));
                    return edge ? z : y;
                };
                const float sb = shift(s[1], -4, lane < 4, es_[0], es_[1], 0);
                const float pb = shift(dP[1], -4, lane < 4, ep_[0], ep_[1], 0);
                const float sn = shift(s[0], 4, lane >= 60, es_[0], es_[1], 1);
                const float pn = shift(dP[0], 4, lane >= 60, ep_[0], ep_[1], 1);
                if (w != 0.f) {
                    s[0] = fmaf(w, sb, (1.f - w) * s[0]);
                    dP[0] = fmaf(w, pb, (1.f - w) * dP[0]);
                    s[1] = fmaf(w, s[1], (1.f - w) * sn);
                    dP[1] = fmaf(w, dP[1], (1.f - w) * pn);
                }
            }
#pragma unroll
            for (int y = 0; y < 2; ++y) {
                const bool in = has(r, y);
                const float x = TL::kF32 && !valu ? prob_low(s[y], sl2, xl[y]) : prob(s[y], sl2, xl[y] * kLog2e);
                const float wt = INTERP ? (y ? rt.w[r] : 1.f - rt.w[r]) : 1.f;
                p[y] = in ? x * wt : 0.f;
                c[y] = in ? tau * x * (dP[y] - xd[y]) * wt : 0.f;
            }
            // the next rung's rows load as soon as this one's are used
            TL::axpy2(adk, c[0], xq[0], c[1], xq[1]);
            load_q(nx);
            __builtin_amdgcn_sched_barrier(0);
            TL::axpy2(adv, p[0], xg[0], p[1], xg[1]);
            load_g(nx);
        }
    }

    // as in the forward: queries that do not read the key took part with weights of 0
    if (tiny || __builtin_amdgcn_ballot_w64(!(TL::finite(adk) && TL::finite(adv)))) {
        TL::zero(adk);
        TL::zero(adv);
        for (int pass = 0; pass < passes; ++pass) {
            const int bh = hd.q_of(bk, pass * ts.hs + hs);
            dkdv_by_entry<TL>(q + lay.q.head(bh, hd.H), dO + lay.g.head(bh, hd.H), K, V, lse + (size_t)bh * T,
                                delta_in + (size_t)bh * T, sq, sg, sk, sv, jc, gq, T, W, rt, nact, tau, sl2, adk, adv);
        }
    }

    if (ts.hs > 1) {
        // head slots 1 .. hand their sums to slot 0 of the same keys, vector by vector,
        // lane-minor (a wave's accesses cover consecutive banks)
        f32x4 *xfer = reinterpret_cast<f32x4 *>(smem);
        __syncthreads();  // every wave is done with the staged rows
        if (hs > 0) {
            f32x4 *dst = xfer + (size_t)(wv * (ts.hs - 1) + hs - 1) * 2 * TL::NB * 64 + lane;
#pragma unroll
            for (int b = 0; b < TL::NB; ++b) {
                dst[b * 64] = adk.c[b];
                dst[(TL::NB + b) * 64] = adv.c[b];
            }
        }
        __syncthreads();
        if (hs > 0) return;  // no barrier below
        for (int u = 1; u < ts.hs; ++u) {
            const f32x4 *src = xfer + (size_t)(wv * (ts.hs - 1) + u - 1) * 2 * TL::NB * 64 + lane;
#pragma unroll
            for (int b = 0; b < TL::NB; ++b) {
                adk.c[b] += src[b * 64];
                adv.c[b] += src[(TL::NB + b) * 64];
            }
        }
    }
    if (rf.on) TL::rope_t(adk, j, sfreq, gq);  // gradient w.r.t. the unrotated k
    if (j < T) {
        const float sc = DEV && table_unusable(rt, W) ? NAN : 1.f;  // bad device alpha, or another W
        TL::store(dk + lay.dk.head(bk, hd.kv_heads()) + j * lay.dk.st, gq, adk, sc);
        TL::store(dv + lay.dv.head(bk, hd.kv_heads()) + j * lay.dv.st, gq, adv, sc);
    }
}

// ---------------------------------------------------------------------------
// dk, dv where 16 keys a wave would leave the chip idle: one key per lanes of one 16-byte
// chunk each, the query heads of its group one after another.
// ---------------------------------------------------------------------------
template <typename S, int D, bool DEV>
__global__ __launch_bounds__(256) void bwd_dkdv_rows_kernel(
    const S *__restrict__ q, const S *__restrict__ k, const S *__restrict__ v,
    const float *__restrict__ lse, const S *__restrict__ dO, const float *__restrict__ delta_in,
    S *__restrict__ dk, S *__restrict__ dv, const double *__restrict__ partials, int n_partials,
    float *__restrict__ dalpha, float *__restrict__ dtheta, int T, int W, RungTable rt_arg,
    const RungTable *__restrict__ rtp, RopeFreq rf, float tau, float sl2, int tiles, int blocks, Heads hd, Layouts lay) {
    constexpr int es = (int)sizeof(S), L = D * es / 16, RW = 64 / L;
    using TL = Tile<S, D, L>;
    using Slice = typename TL::Slice;
    const RungTable &rt = DEV ? *rtp : rt_arg;
    __shared__ double sfreq[D / 2], red[256];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nk = lane / L, g = lane % L;
    if (block_number() >= blocks) return;
    const int blk = xcd_remap(block_number(), blocks);
    const int bk = blk / tiles, t0 = ((blk % tiles) * 4 + wave) * RW;
    if (rf.on && threadIdx.x < D / 2) sfreq[threadIdx.x] = rf.inv[threadIdx.x] * 0.15915494309189533576888376337251;
    if (block_number() == 0)
        sum_partials<DEV>(red, partials, n_partials, dalpha, dtheta, rt);
    else if (rf.on)
        __syncthreads();
    if (t0 >= T) return;  // no barrier below
    const S *K = k + lay.k.head(bk, hd.kv_heads()), *V = v + lay.v.head(bk, hd.kv_heads());
    const uint32_t sq = (uint32_t)(es * lay.q.st), sg = (uint32_t)(es * lay.g.st);
    const uint32_t sk = (uint32_t)(es * lay.k.st), sv = (uint32_t)(es * lay.v.st);
    const int j = t0 + nk, jc = min(j, T - 1);
    const int before = max(jc - 1, 0), after = min(jc + 1, T - 1);
    const Slice kj = TL::load(K, jc, g, sk), vj = TL::load(V, jc, g, sv);
    // the rows beside the key's: the other row of a rung entry
    const Slice kb = TL::load(K, before, g, sk), vb = TL::load(V, before, g, sv);
    const Slice ka = TL::load(K, after, g, sk), va = TL::load(V, after, g, sv);
    int nact = 0;  // rungs through which a query reads some key of this wave: a prefix
#pragma unroll
    for (int r = 0; r < kMaxRungs; ++r) nact += ((r < rt.n) & (rt.d0[r] < T - t0)) ? 1 : 0;
    nact = __builtin_amdgcn_readfirstlane(nact);
    const int wmax = min(W, T - 1 - t0);

    typename TL::Acc adk, adv;
    TL::zero(adk);
    TL::zero(adv);
    // per-lane products of a logit or a dP, blended before the sum over the lanes
    auto dots = [&](const Slice &x, const Slice &y) {
        if constexpr (TL::kF32)
            return chunk_dot(x.c[0], y.c[0]);
        else
            return TL::dot(x, y);
    };
    auto sum = [&](float t) { return chunk_sum<1, L>(&t); };
    for (int hg = 0; hg < hd.G; ++hg) {
        const int bh = hd.q_of(bk, hg);
        const S *Q = q + lay.q.head(bh, hd.H), *G = dO + lay.g.head(bh, hd.H);
        const float *Le = lse + (size_t)bh * T, *De = delta_in + (size_t)bh * T;
        // a query that does not read the key is replaced by the key's own, with weight 0
        for (int d = 0; d <= wmax; d += 2) {
            Slice x[2], y[2];
            float l[2], dl[2], p[2], c[2];
            bool in[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                in[u] = j + d + u < T && d + u <= W;
                const int row = in[u] ? j + d + u : jc;
                x[u] = TL::load(Q, row, g, sq);
                y[u] = TL::load(G, row, g, sg);
                l[u] = Le[row] * kLog2e;
                dl[u] = De[row];
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const float s = sum(dots(x[u], kj)), dP = sum(dots(y[u], vj));
                p[u] = in[u] ? prob(s, sl2, l[u]) : 0.f;
                c[u] = in[u] ? tau * p[u] * (dP - dl[u]) : 0.f;
            }
            TL::add2(adk, c[0], x[0], c[1], x[1]);
            TL::add2(adv, p[0], y[0], p[1], y[1]);
        }
        // a rung's two queries: i0 has the key as row r0, i0 + 1 as row r1
        for (int r = 0; r < nact; ++r) {
            const int d0 = rt.d0[r];
            const float w = rt.w[r];
            Slice x[2], y[2];
            float l[2], dl[2], p[2], c[2];
            bool in[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                in[u] = j + d0 + u < T && (w == 0.f ? u == 0 : u || j >= 1);
                if (u && w == 0.f) break;
                const int row = in[u] ? j + d0 + u : jc;
                x[u] = TL::load(Q, row, g, sq);
                y[u] = TL::load(G, row, g, sg);
                l[u] = Le[row] * kLog2e;
                dl[u] = De[row];
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                if (u && w == 0.f) break;
                const float wt = u ? w : 1.f - w;
                float s = wt * dots(x[u], kj), dP = wt * dots(y[u], vj);
                if (w != 0.f) {
                    s = fmaf(1.f - wt, dots(x[u], u ? ka : kb), s);
                    dP = fmaf(1.f - wt, dots(y[u], u ? va : vb), dP);
                }
                const float x0 = prob(sum(s), sl2, l[u]);
                p[u] = in[u] ? x0 * wt : 0.f;
                c[u] = in[u] ? tau * x0 * (sum(dP) - dl[u]) * wt : 0.f;
            }
            if (w != 0.f) {
                TL::add2(adk, c[0], x[0], c[1], x[1]);
                TL::add2(adv, p[0], y[0], p[1], y[1]);
            } else {
                TL::axpy(adk, c[0], x[0]);
                TL::axpy(adv, p[0], y[0]);
            }
        }
    }
    // as in the forward: queries that do not read the key took part with weights of 0
    if (__builtin_amdgcn_ballot_w64(!(TL::finite(adk) && TL::finite(adv)))) {
        TL::zero(adk);
        TL::zero(adv);
        for (int hg = 0; hg < hd.G; ++hg) {
            const int bh = hd.q_of(bk, hg);
            dkdv_by_entry<TL>(q + lay.q.head(bh, hd.H), dO + lay.g.head(bh, hd.H), K, V, lse + (size_t)bh * T,
                              delta_in + (size_t)bh * T, sq, sg, sk, sv, jc, g, T, W, rt, nact, tau, sl2, adk, adv);
        }
    }
    if (rf.on) TL::rope_t(adk, j, sfreq, g);  // gradient w.r.t. the unrotated k
    if (j < T) {
        const float sc = DEV && table_unusable(rt, W) ? NAN : 1.f;  // bad device alpha, or another W
        TL::store(dk + lay.dk.head(bk, hd.kv_heads()) + j * lay.dk.st, g, adk, sc);
        TL::store(dv + lay.dv.head(bk, hd.kv_heads()) + j * lay.dv.st, g, adv, sc);
    }
}

template <typename S, int D>
static size_t num_partials_t(int BH, int T) {
    constexpr int QPB = 256 / (D / Vec<S>::N);
    return (size_t)((T + QPB - 1) / QPB) * (size_t)BH;
}

size_t bwd_num_partials(int dtype, int D, int BH, int T) {
    if (dtype == 0 && D == 32) return num_partials_t<float, 32>(BH, T);
    if (dtype == 0 && D == 64) return num_partials_t<float, 64>(BH, T);
    if (dtype == 1 && D == 32) return num_partials_t<uint16_t, 32>(BH, T);
    if (dtype == 1 && D == 64) return num_partials_t<uint16_t, 64>(BH, T);
    if (dtype == 0 && D == 128) return num_partials_t<float, 128>(BH, T);
    if (dtype == 1 && D == 128) return num_partials_t<uint16_t, 128>(BH, T);
    return 0;
}

template <typename S, int D>
static hipError_t launch_bwd_t(const void *q, const void *k, const void *v, const void *o,
                               const float *lse, const void *dO, void *dq, void *dk, void *dv,
                               float *dalpha, float *dtheta, float *delta_ws, double *partials, int BH,
                               const Heads &hd, int T, int W, const RungTable &rt,
                               const RungTable *rtp, const RopeFreq &rf, const Layouts &lay, hipStream_t s) {
    using TL = Tile<S, D>;
    constexpr int nw = TL::kRow == 512 ? 2 : 4;  // waves per workgroup (float32 d 128: its rows' LDS)
    const float tau = 1.f / sqrtf((float)D);
    TileShape ts;
    ts.hs = tile_heads(hd.G, nw);
    const int runs = nw / ts.hs;
    ts.tiles = (T + 16 * runs - 1) / (16 * runs);
    ts.blocks = ts.tiles * (BH / ts.hs);
    ts.nc = band_chunks(W);
    const size_t fixed = 2 * (size_t)16 * (runs - 1) * TL::kRow, per = 2 * (size_t)32 * TL::kRow;
    ts.cps = tile_chunks(ts.nc, fixed, per, TL::NC);
    int nb = ts.blocks;  // dq workgroups = dalpha partials
    bool interp = false;
    for (int r = 0; r < rt.n && !interp; ++r) interp = rt.w[r] != 0.f;
    hipError_t e;
    if constexpr (TL::kF32) {
        const bool wide = f32_wide(BH, T);
        const int per = wide ? 1024 / D : 64, tiles = T / per + (T % per != 0);
        // the window's rows are staged where two workgroups still share a CU's LDS
        int rows = 64 + ((W + 15) & ~15);
        if (wide || 2 * (size_t)rows * TL::kRow > 78 * 1024) rows = 0;
        nb = tiles * BH;
        auto dqk = wide ? (rtp ? bwd_dq_f32_kernel<D, D / 4, true> : bwd_dq_f32_kernel<D, D / 4, false>)
                        : (rtp ? bwd_dq_f32_kernel<D, 4, true> : bwd_dq_f32_kernel<D, 4, false>);
        e = launch(kBwdDq, dqk, grid_of(nb), dim3(256), (unsigned)(2 * rows * TL::kRow), s, (const S *)q,
                   (const S *)k, (const S *)v, (const S *)o, lse, (const S *)dO, (S *)dq, delta_ws, partials, T, W, rt,
                   rtp, rf, tau, tiles, nb, rows, hd, lay);
    } else {
        auto dqk = rtp ? bwd_dq_tile_kernel<D, true, true>
                       : interp ? bwd_dq_tile_kernel<D, true, false> : bwd_dq_tile_kernel<D, false, false>;
        e = launch(kBwdDq, dqk, grid_of(nb), dim3(64 * nw), (unsigned)(fixed + per * ts.cps), s, (const S *)q,
                   (const S *)k, (const S *)v, (const S *)o, lse, (const S *)dO, (S *)dq, delta_ws, partials, T, W,
                   rt, rtp, rf, tau, kLog2e / sqrtf((float)D), ts, hd, lay);
    }
    if (e != hipSuccess) return e;
    // dk, dv of few rows: one key per lanes of one 16-byte chunk, unless the tile kernel has
    // the heads of a group side by side or a long window on the matrix cores.  Against the
    // tile kernel, W 3 to 17: float32 d 32 / 64 / 128 at 4096 queries and groups of one 0.80
    // to 0.94 / 0.71 to 0.79 / 0.48 to 0.55 times, of three 0.75 / 0.61 / 0.37, of two 1.2 /
    // 1.0 / 0.65 to 0.86, of four 1.8 / 1.5 / 0.62 to 0.75; d 32 and W 64 1.1 to 1.2; at
    // 16000 queries and W 64 1.1 to 1.3.  bfloat16 d 128, groups of one, up to 8192 queries
    // 0.71 to 1.02, at 16000 1.15 to 1.34, W 64 1.2 to 1.7, groups of two 1.05 to 1.27;
    // d 32 and 64 0.91 to 1.3.
    if constexpr (TL::kF32 || D == 128) {
        const bool few = TL::kF32 ? f32_wide(BH, T) && (D == 128 || (ts.hs == 1 && (D == 64 || W <= 32)))
                                  : (long long)BH * T <= 8192 && ts.hs == 1 && W <= 24;
        if (few) {
            constexpr int kper = 4096 / TL::kRow;  // keys per workgroup
            const int ktiles = T / kper + (T % kper != 0), kb = ktiles * (BH / hd.G);
            return launch(kBwdDkDv, rtp ? bwd_dkdv_rows_kernel<S, D, true> : bwd_dkdv_rows_kernel<S, D, false>,
                          grid_of(kb), dim3(256), 0, s, (const S *)q, (const S *)k, (const S *)v, lse, (const S *)dO,
                          delta_ws, (S *)dk, (S *)dv, partials, nb, dalpha, dtheta, T, W, rt, rtp, rf, tau,
                          kLog2e / sqrtf((float)D), ktiles, kb, hd, lay);
        }
    }
    // dk, dv: a head slot's q and dO rows of the staged chunks, their lse and Delta; the
    // sums of the slots past the first take their place at the end
    TileShape tk = ts;
    const size_t row = 2 * TL::kRow + 2 * sizeof(float);
    const size_t kfixed = row * ts.hs * 16 * (runs - 1), kper = row * ts.hs * 32;
    tk.blocks = ts.tiles * (BH / hd.G);
    tk.cps = tile_chunks(ts.nc, kfixed, kper, TL::NC);
    const size_t sums = (size_t)(nw - runs) * 64 * 2 * sizeof(typename TL::Acc);
    const size_t lds = std::max({kfixed + kper * tk.cps, sums, 64 * nw * sizeof(double)});
    auto dkk = rtp ? bwd_dkdv_tile_kernel<S, D, true, true>
                   : interp ? bwd_dkdv_tile_kernel<S, D, true, false> : bwd_dkdv_tile_kernel<S, D, false, false>;
    return launch(kBwdDkDv, dkk, grid_of(tk.blocks), dim3(64 * nw), (unsigned)lds, s, (const S *)q,
                  (const S *)k, (const S *)v, lse, (const S *)dO, delta_ws, (S *)dk, (S *)dv, partials, nb, dalpha,
                  dtheta, T, W, rt, rtp, rf, tau, kLog2e / sqrtf((float)D), tk, hd, lay);
}

static hipError_t launch_backward_rows(int dtype, int D, const void *q, const void *k, const void *v,
                                          const void *o, const float *lse, const void *dO, void *dq,
                                          void *dk, void *dv, float *dalpha, float *dtheta, float *delta_ws,
                                          double *partials, int BH, const Heads &hd, int T, int W,
                                          const RungTable &rt, const RungTable *rtp, const RopeFreq &rf,
                                          const Layouts &lay, hipStream_t s) {
#define FIBATTN_BWD(S_, D_)                                                                  \
    return launch_bwd_t<S_, D_>(q, k, v, o, lse, dO, dq, dk, dv, dalpha, dtheta, delta_ws, partials, \
                                BH, hd, T, W, rt, rtp, rf, lay, s)
    if (dtype == 0 && D == 32) FIBATTN_BWD(float, 32);
    if (dtype == 0 && D == 64) FIBATTN_BWD(float, 64);
    if (dtype == 1 && D == 32) FIBATTN_BWD(uint16_t, 32);
    if (dtype == 1 && D == 64) FIBATTN_BWD(uint16_t, 64);
    if (dtype == 0 && D == 128) FIBATTN_BWD(float, 128);
    if (dtype == 1 && D == 128) FIBATTN_BWD(uint16_t, 128);
#undef FIBATTN_BWD
    return hipErrorInvalidValue;
}

hipError_t launch_backward(int dtype, int D, const void *q, const void *k, const void *v,
                           const void *o, const float *lse, const void *dO, void *dq, void *dk,
                           void *dv, float *dalpha, float *dtheta, float *delta_ws, double *partials,
                           const RungTerms &terms, int BH, const Heads &hd, int T, int W,
                           const RungTable &rt, const RungTable *rtp, const RopeFreq &rf,
                           const Layouts &lay, hipStream_t s) {
    if (backward_mfma_supported(dtype, D, W))
        return launch_backward_mfma(q, k, v, o, lse, dO, dq, dk, dv, dalpha, dtheta, delta_ws, partials,
                                    terms, BH, hd, T, W, rt, rtp, rf, lay, s);
    return launch_backward_rows(dtype, D, q, k, v, o, lse, dO, dq, dk, dv, dalpha, dtheta, delta_ws,
                                   partials, BH, hd, T, W, rt, rtp, rf, lay, s);
}

}  // namespace fibattn
