// Forward kernels for every storage type, head size and window outside the bfloat16,
// d_head 64, W <= 16 path (fwd_mfma.hip): a tile kernel on the matrix cores for bfloat16,
// one on the VALU for float32 (below).  Both: window band + shared rung offsets, softmax,
// weighted values, lse.
//
// Section 2 "Attended set": every query i of a (b, h) attends to distances 0..W and to
// the rung distances d_k = alpha f_k, each rung read as the blend of rows
// i - floor(d_k) (weight 1 - w_k) and i - floor(d_k) - 1 (weight w_k).  Because the
// offsets are shared, a block of consecutive queries reads, for each rung, one
// contiguous shifted block of key/value rows.
//
// A wave owns 16 consecutive queries (lane layouts in tile.h).  The tile kernel:
//   - window band: the keys i - W .. i lie in 32-row chunks that end at the wave's last
//     query (one for W <= 16, five for W = 128).  The workgroup's chunks are copied to LDS
//     a few at a time; per chunk, S = K.Q^T on the matrix cores, masked to 0 <= i - j <= W,
//     and V^T.P^T accumulated there, with the running maximum of an online softmax;
//   - rungs: per-row dot products on the VALU (four lanes per row), blended in score
//     space, their probabilities' weighted values added in the same registers.
// The whole softmax runs in base 2.
//
// What bounds it: the latency of the rung gathers (L2) and the VALU work (37 to 50 % of the
// issue slots); the band, on the matrix cores, is a fraction of it at any window.  Us a
// launch, without and with q rotated on load, against a kernel with one lane group per query,
// every row read from global memory by every query and no matrix cores: bf16 d 64 B4 H8 T1500
// W128, integer offsets, 115 -> 15.7 (17.6); bf16 d 64 B4 H8 T2048 W64 75 -> 16.1 (18.5); bf16
// d 128 B2 H16 on 4 T2000 W8 58 -> 27.7 (32.1); bf16 d 32 B8 H8 T1024 W10 24 -> 10.9 (14.2).
#include "launch.h"
#include "tile.h"

namespace fibattn {

constexpr float kFwdSlack = 8.f;  // log2 units a rung's logit may exceed the running reference

// Waves per SIMD the registers are budgeted for: a slice is NC 16-byte pieces, and a rung
// holds four of them in flight (rows r0, r1 of K and V) next to q's slice and D / 4 sums.
template <int D>
constexpr int fwd_waves = D <= 64 ? 4 : 3;

// The softmax and the weighted values of query ic, its entries one by one and only those it
// has, the maximum first (quad layout; nact rungs, the wave's).
template <typename TL>
__device__ __forceinline__ void forward_by_entry(const typename TL::Slice &qq, const void *K, const void *V, uint32_t sk,
                                                 uint32_t sv, int ic, int gq, int W, const RungTable &rt, int nact,
                                                 float sl2, typename TL::Acc &acc, float &m, float &l) {
    float mx = -INFINITY;
    for (int pass = 0; pass < 2; ++pass) {
        if (pass) {
            TL::zero(acc);
            l = 0.f;
            m = mx;
        }
        for (int e = 0; e <= W + nact; ++e) {
            const int d = e <= W ? e : rt.d0[e - W - 1];
            const float w = e <= W ? 0.f : rt.w[e - W - 1];
            const bool in = ic >= d + (w != 0.f);
            const int r0 = in ? ic - d : ic, r1 = in ? r0 - 1 : ic;
            float s = quad_sum(TL::dot(qq, TL::load(K, r0, gq, sk)));
            if (w != 0.f) s = (1.f - w) * s + w * quad_sum(TL::dot(qq, TL::load(K, r1, gq, sk)));
            s *= sl2;
            if (!pass) {
                mx = in ? fmaxf(mx, s) : mx;
            } else if (in) {
                const float p = exp2f(s - mx);
                l += p;
                TL::axpy(acc, p * (1.f - w), TL::load(V, r0, gq, sv));
                if (w != 0.f) TL::axpy(acc, p * w, TL::load(V, r1, gq, sv));
            }
        }
    }
}

// INTERP: some rung has w != 0, so the second row r1 is read; otherwise two rungs are
// taken together.  DEV: the rung table is the one at rtp, built on the device (rt_arg
// unused).  rf.on: q holds unrotated rows; each is rotated where it is loaded (a query row
// is used by one query only, so qrot may be q itself: no restrict on q) and written to qrot,
// placed by lay.dq, for the backward: d 128 B4 H8 T1024 3.7 us more here against 5.5 us for a
// launch of its own, T4096 7.4 against 14.8; d 64 W24 T4096 3.7 against 7.1; d 32 B16 H8
// T4096, where the chip is full of angles, 16 against 13.
template <int D, bool INTERP, bool DEV>
__global__ __launch_bounds__(256, (fwd_waves<D>)) void fwd_tile_kernel(
    const uint16_t *q, const uint16_t *__restrict__ k, const uint16_t *__restrict__ v, uint16_t *__restrict__ o,
    float *__restrict__ lse, int T, int W, RungTable rt_arg, const RungTable *__restrict__ rtp, float sl2,
    TileShape ts, Heads hd, Layouts lay, uint16_t *qrot, RopeFreq rf) {
    using S = uint16_t;
    using TL = Tile<S, D>;
    using Slice = typename TL::Slice;
    const RungTable &rt = DEV ? *rtp : rt_arg;
    __shared__ double sfreq[D / 2];
    constexpr int RB = INTERP ? 1 : 2;          // rungs per batch: two rows of K and of V
    constexpr int NBUF = TL::NC <= 2 ? 2 : 1;   // batches in flight
    extern __shared__ __align__(16) char smem[];

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
    const S *Q = q + lay.q.head(bh, hd.H);
    const S *K = k + lay.k.head(bk, hd.kv_heads());
    const S *V = v + lay.v.head(bk, hd.kv_heads());
    const uint32_t sk = (uint32_t)(lay.k.st * (int)sizeof(S)), sv = (uint32_t)(lay.v.st * (int)sizeof(S));

    const int t0 = T0 + 16 * wv;
    const int im = t0 + nm;                        // MFMA layout query
    const int i = t0 + nq, ic = min(i, T - 1);     // quad layout query
    Slice qq = TL::load(Q, ic, gq, (uint32_t)(lay.q.st * (int)sizeof(S)));
    if (rf.on) {
        if (threadIdx.x < D / 2) sfreq[threadIdx.x] = rf.inv[threadIdx.x] * TL::kRopeUnit;
        __syncthreads();
    }

    // rungs some query of this wave includes: a prefix of the table (sorted by d)
    int nact = 0;
#pragma unroll
    for (int r = 0; r < kMaxRungs; ++r) nact += ((r < rt.n) & (rt.d0[r] <= min(t0 + 15, T - 1))) ? 1 : 0;
    nact = t0 < T ? __builtin_amdgcn_readfirstlane(nact) : 0;

    // the two rows of a batch: r0 and r1 of a rung, or r0 of two rungs (the second clamped
    // to an active one and masked).  An entry the query does not have (weight 0) reads the
    // query's own row: 0 times a row it does not attend could be NaN.
    auto load_batch = [&](int rb, const void *X, uint32_t st, Slice *x) {
        if constexpr (INTERP) {
            const int d = rt.d0[rb], two = rt.w[rb] != 0.f;
            const bool in = ic >= d + two;
            const int r0 = in ? ic - d : ic;
            x[0] = TL::load(X, r0, gq, st);
            x[1] = TL::load(X, in ? r0 - two : r0, gq, st);
        } else {
#pragma unroll
            for (int y = 0; y < 2; ++y) {
                const int d = rt.d0[min(rb + y, nact - 1)];
                x[y] = TL::load(X, ic >= d ? ic - d : ic, gq, st);
            }
        }
    };
    Slice kx[NBUF][2], vx[NBUF][2];
    // in flight during the band phase, as far as the registers go
    if (nact > 0) load_batch(0, K, sk, kx[0]);
    if (TL::NC <= 2 && nact > 0) load_batch(0, V, sv, vx[0]);

    // ---- window band (MFMA layout) ----
    Slice qm;
    float m = 0.f, l = 0.f;
    bool tiny = false;
    typename TL::Acc acc;
    TL::zero(acc);
    const unsigned reach = (unsigned)min(W, im);  // 0 <= im - key <= W and key >= 0
    const int nc = min(ts.nc, (T0 + 16 * runs + 31) >> 5);  // chunks with rows >= 0
    for (int c0 = 0; c0 < nc; c0 += ts.cps) {
        // chunks c0 .. c0 + n - 1 of every run: chunk c of run wv is the rows
        // [T0 + 16 wv + 16 - 32 (c + 1), T0 + 16 wv + 16 - 32 c)
        const int n = min(ts.cps, nc - c0);
        const int rbeg = T0 + 16 - 32 * (c0 + n), rows = 16 * (runs - 1) + 32 * n;
        char *kr = smem, *vr = smem + rows * TL::kRow;
        if (c0 > 0) __syncthreads();  // every wave is done with the rows staged before
        TL::stage(kr, K, rbeg, rows, T, lay.k.st, wave, nw);
        TL::stage(vr, V, rbeg, rows, T, lay.v.st, wave, nw);
        if (c0 == 0) {
            if (rf.on) {  // rotated while the copies are in flight
                TL::rope(qq, i, sfreq, gq);
                if (i < T) TL::put(qrot + lay.dq.head(bh, hd.H) + i * lay.dq.st, gq, qq);
            }
            qm = TL::from_quad(qq, lane);
        }
        wait_vmem();
        __syncthreads();
        float least = INFINITY;
        for (int c = 0; c < n; ++c) {
            if (t0 + 16 - 32 * (c0 + c) <= 0) break;  // rows before the start
            const int base = 16 * wv + 32 * (n - 1 - c);  // the chunk's first staged row
            float p[8], mx = -INFINITY, low = INFINITY;
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const f32x4 s = TL::scores(TL::staged(kr, base + 16 * b + nm, gm), qm);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int key = rbeg + base + 16 * b + 4 * gm + e;
                    p[4 * b + e] = (unsigned)(im - key) <= reach ? s[e] : -INFINITY;
                    mx = fmaxf(mx, p[4 * b + e]);
                    low = fminf(low, s[e]);
                }
            }
            mx = max4(mx) * sl2;
            if (c0 + c == 0) {
                m = mx;  // -inf only where key im itself has a logit of -inf
            } else if (__builtin_amdgcn_ballot_w64(mx > m)) {
                const float mn = fmaxf(m, mx), f = exp2f(m - mn);
                m = mn;
                l *= f;
                TL::scale(acc, f);
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) p[e] = fmaf(p[e], sl2, -m);
            least = fminf(least, fmaf(low, sl2, -m));
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                p[e] = fast_exp2(p[e]);
                l += p[e];
            }
            TL::accumulate(acc, vr, base, TL::weights(p), gm);
        }
        if (tiny_weight(least)) tiny |= TL::large_rows(vr, 16 * wv, 32 * n);
    }
    if (TL::NC > 2 && nact > 0) load_batch(0, V, sv, vx[0]);
    l = sum4(l);
    // hand the band results to the quad layout
    TL::to_quad_acc(acc, lane);
    m = to_quad(m, lane);
    l = to_quad(l, lane);

    // ---- rungs (quad layout) ----
    float p[RB];
    auto logits = [&](int rb, const Slice *x) {
        float s[RB], mb = m;
        if constexpr (INTERP) {
            const int d0 = rt.d0[rb];
            const float w = rt.w[rb];
            const bool in = d0 < i || (d0 == i && w == 0.f);
            const float part = quad_sum((1.f - w) * TL::dot(qq, x[0]) + w * TL::dot(qq, x[1]));
            s[0] = in ? part : -INFINITY;
            mb = fmaxf(mb, s[0] * sl2);
        } else {
#pragma unroll
            for (int y = 0; y < 2; ++y) {
                const float part = quad_sum(TL::dot(qq, x[y]));
                const bool in = rb + y < nact && rt.d0[rb + y < nact ? rb + y : nact - 1] <= i;
                s[y] = in ? part : -INFINITY;
                mb = fmaxf(mb, s[y] * sl2);
            }
        }
        // The running reference moves only when a logit exceeds it by more than kFwdSlack
        // log2 units (exp2(s - m) <= 2^kFwdSlack; o = acc / l and lse = m + log2(l) hold
        // for any reference).
        const bool grow = mb > m + kFwdSlack;
        if (__builtin_amdgcn_ballot_w64(grow)) {
            const float mn = grow ? mb : m, f = exp2f(m - mn);
            m = mn;
            l *= f;
            TL::scale(acc, f);
        }
#pragma unroll
        for (int y = 0; y < RB; ++y) {
            p[y] = exp2f(fmaf(s[y], sl2, -m));
            l += p[y];
        }
    };
    auto values = [&](int rb, const Slice *x) {
        if constexpr (INTERP) {
            const float w = rt.w[rb];
            TL::axpy2(acc, p[0] * (1.f - w), x[0], p[0] * w, x[1]);
        } else {
            TL::axpy2(acc, p[0], x[0], p[1], x[1]);
        }
    };
    if constexpr (NBUF == 2) {
        for (int rb = 0; rb < nact; rb += 2 * RB) {
            if (rb + RB < nact) {
                load_batch(rb + RB, K, sk, kx[1]);
                load_batch(rb + RB, V, sv, vx[1]);
            }
            logits(rb, kx[0]);
            values(rb, vx[0]);
            if (rb + RB < nact) {
                if (rb + 2 * RB < nact) {
                    load_batch(rb + 2 * RB, K, sk, kx[0]);
                    load_batch(rb + 2 * RB, V, sv, vx[0]);
                }
                logits(rb + RB, kx[1]);
                values(rb + RB, vx[1]);
            }
        }
    } else {
        // one buffer each for K and V: the next batch's keys load while this one's values
        // are added, its values while the next logits are taken
        for (int rb = 0; rb < nact; rb += RB) {
            const int nx = min(rb + RB, nact - 1);
            logits(rb, kx[0]);
            load_batch(nx, K, sk, kx[0]);
            values(rb, vx[0]);
            load_batch(nx, V, sv, vx[0]);
        }
    }
    // Entries a query does not have took part with weights of 0: rows of the chunks outside
    // its window, and its own row in the place of a rung's.  If that, or what the query does
    // attend, left anything that is not finite, the entries are taken one by one instead;
    // so are weights too small for the matrix cores, where they count.
    if (tiny || __builtin_amdgcn_ballot_w64(!(TL::finite(acc) && l * 0.f == 0.f)))
        forward_by_entry<TL>(qq, K, V, sk, sv, ic, gq, W, rt, nact, sl2, acc, m, l);

    if (i < T) {
        const bool bad = DEV && table_unusable(rt, W);  // bad device alpha, or another W
        TL::store(o + lay.o.head(bh, hd.H) + i * lay.o.st, gq, acc, bad ? NAN : 1.f / l);
        if (gq == 0) __builtin_nontemporal_store(bad ? NAN : (m + log2f(l)) * kLn2, lse + (size_t)bh * T + i);
    }
}

// ---------------------------------------------------------------------------
// float32: the same set on the VALU, L lanes per query, every sum in the order that tile.h
// states, whatever L is.  Four lanes, or D / 4 of one 16-byte chunk each where 16 queries a
// wave would leave the chip idle (f32_wide).
// ---------------------------------------------------------------------------
template <int D, int L, bool DEV>
__global__ __launch_bounds__(256, 2) void fwd_f32_kernel(
    const float *q, const float *__restrict__ k, const float *__restrict__ v, float *__restrict__ o,
    float *__restrict__ lse, int T, int W, RungTable rt_arg, const RungTable *__restrict__ rtp, float sl2, int tiles,
    int blocks, Heads hd, Layouts lay, float *qrot, RopeFreq rf) {
    using TL = Tile<float, D, L>;
    using Slice = typename TL::Slice;
    constexpr int NC = TL::NC, RW = 64 / L, QPB = 4 * RW;  // queries per wave and workgroup
    const RungTable &rt = DEV ? *rtp : rt_arg;
    extern __shared__ __align__(16) char smem[];
    __shared__ double sfreq[D / 2];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nq = lane / L, gq = lane % L;
    if (block_number() >= blocks) return;
    const int blk = xcd_remap(block_number(), blocks);
    const int bh = blk / tiles, t0 = (blk % tiles) * QPB + RW * wave;
    if (rf.on) {
        if (threadIdx.x < D / 2) sfreq[threadIdx.x] = rf.inv[threadIdx.x] * TL::kRopeUnit;
        __syncthreads();
    }
    if (t0 >= T) return;  // no barrier below
    const int bk = hd.kv_of(bh);
    const float *K = k + lay.k.head(bk, hd.kv_heads());
    const float *V = v + lay.v.head(bk, hd.kv_heads());
    const uint32_t sk = (uint32_t)(4 * lay.k.st), sv = (uint32_t)(4 * lay.v.st);
    const int i = t0 + nq, ic = min(i, T - 1), last = min(t0 + RW - 1, T - 1);
    Slice qq = TL::load(q + lay.q.head(bh, hd.H), ic, gq, (uint32_t)(4 * lay.q.st));
    if (rf.on) {  // as in the tile kernel
        TL::rope(qq, i, sfreq, gq);
        if (i < T) TL::put(qrot + lay.dq.head(bh, hd.H) + i * lay.dq.st, gq, qq);
    }
    int nact = 0;  // rungs some query of this wave includes: a prefix of the table
#pragma unroll
    for (int r = 0; r < kMaxRungs; ++r) nact += ((r < rt.n) & (rt.d0[r] <= last)) ? 1 : 0;
    nact = __builtin_amdgcn_readfirstlane(nact);
    const int nwin = (min(W, last) + 4) & ~3;  // window entries, in fours
    // the wave's logits, entry by entry (LDS accesses of one wave keep their order)
    float *sc = reinterpret_cast<float *>(smem) + RW * wave + nq;

    // logits and their maximum; an entry the query does not have reads its own row
    float m = -INFINITY;
    auto keep = [&](int e, bool in, float s) {
        s = in ? s * sl2 : -INFINITY;
        if (gq == 0) sc[QPB * e] = s;
        m = fmaxf(m, s);
    };
    const int reach = min(W, ic);
    for (int d = 0; d < nwin; d += 4) {
        Slice x[4];
#pragma unroll
        for (int y = 0; y < 4; ++y) x[y] = TL::load(K, d + y <= reach ? ic - d - y : ic, gq, sk);
#pragma unroll
        for (int y = 0; y < 4; ++y) keep(d + y, d + y <= reach, TL::row_dot(qq, x[y]));
    }
    // two rungs together (the second clamped to an active one and masked)
    for (int r = 0; r < nact; r += 2) {
        Slice x[2], x1[2];
        float w[2];
        bool in[2];
#pragma unroll
        for (int y = 0; y < 2; ++y) {
            const int a = min(r + y, nact - 1), d0 = rt.d0[a];
            w[y] = rt.w[a];
            in[y] = r + y < nact && ic >= d0 + (w[y] != 0.f);
            const int r0 = in[y] ? ic - d0 : ic;
            x[y] = TL::load(K, r0, gq, sk);
            if (w[y] != 0.f) x1[y] = TL::load(K, in[y] ? r0 - 1 : r0, gq, sk);
        }
#pragma unroll
        for (int y = 0; y < 2; ++y) {
            float t[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) t[c] = (1.f - w[y]) * chunk_dot(qq.c[c], x[y].c[c]);
            if (w[y] != 0.f) {
#pragma unroll
                for (int c = 0; c < NC; ++c) t[c] = fmaf(w[y], chunk_dot(qq.c[c], x1[y].c[c]), t[c]);
            }
            keep(nwin + r + y, in[y], chunk_sum<NC, L>(t));
        }
    }
    __builtin_amdgcn_wave_barrier();

    // probabilities and weighted values
    typename TL::Acc acc;
    TL::zero(acc);
    float l = 0.f;
#pragma unroll 4
    for (int d = 0; d < nwin; ++d) {
        const Slice x = TL::load(V, d <= reach ? ic - d : ic, gq, sv);
        const float p = exp2f(sc[QPB * d] - m);
        l += p;
        TL::axpy(acc, p, x);
    }
#pragma unroll 2
    for (int r = 0; r < nact; ++r) {
        const int d0 = rt.d0[r];
        const float w = rt.w[r];
        const bool in = ic >= d0 + (w != 0.f);
        const int r0 = in ? ic - d0 : ic;
        const Slice x = TL::load(V, r0, gq, sv);
        const float p = exp2f(sc[QPB * (nwin + r)] - m);
        l += p;
        TL::axpy(acc, p * (1.f - w), x);
        if (w != 0.f) TL::axpy(acc, p * w, TL::load(V, in ? r0 - 1 : r0, gq, sv));
    }
    if (__builtin_amdgcn_ballot_w64(!TL::finite(acc))) {  // as in the tile kernel: 0 times its own row
        TL::zero(acc);
        for (int d = 0; d < nwin; ++d)
            if (d <= reach) TL::axpy(acc, exp2f(sc[QPB * d] - m), TL::load(V, ic - d, gq, sv));
        for (int r = 0; r < nact; ++r) {
            const int d0 = rt.d0[r];
            const float w = rt.w[r], p = exp2f(sc[QPB * (nwin + r)] - m);
            if (ic >= d0 + (w != 0.f)) {
                TL::axpy(acc, p * (1.f - w), TL::load(V, ic - d0, gq, sv));
                if (w != 0.f) TL::axpy(acc, p * w, TL::load(V, ic - d0 - 1, gq, sv));
            }
        }
    }
    if (i < T) {
        const bool bad = DEV && table_unusable(rt, W);  // bad device alpha, or another W
        TL::store(o + lay.o.head(bh, hd.H) + i * lay.o.st, gq, acc, bad ? NAN : 1.f / l);
        if (gq == 0) __builtin_nontemporal_store(bad ? NAN : (m + log2f(l)) * kLn2, lse + (size_t)bh * T + i);
    }
}

template <int D, int L>
static hipError_t launch_fwd_f32_lanes(const void *q, const void *k, const void *v, void *o, float *lse, int BH,
                                 const Heads &hd, int T, int W, const RungTable &rt, const RungTable *rtp,
                                 const Layouts &lay, hipStream_t s, const RopeFreq &rf, void *q_rot) {
    constexpr int QPB = 256 / L;
    const int tiles = T / QPB + (T % QPB != 0);
    const size_t lds = QPB * sizeof(float) * (size_t)(W + 4 + (rtp ? kMaxRungs : rt.n + 1));
    return launch(kForward, rtp ? fwd_f32_kernel<D, L, true> : fwd_f32_kernel<D, L, false>,
                  grid_of((long long)tiles * BH), dim3(256), (unsigned)lds, s, (const float *)q, (const float *)k,
                  (const float *)v, (float *)o, lse, T, W, rt, rtp, kLog2e / sqrtf((float)D), tiles, tiles * BH, hd,
                  lay, (float *)q_rot, rf);
}

template <int D, typename... A>
static hipError_t launch_fwd_f32(const void *q, const void *k, const void *v, void *o, float *lse, int BH,
                                 const Heads &hd, int T, A... a) {
    return f32_wide(BH, T) ? launch_fwd_f32_lanes<D, D / 4>(q, k, v, o, lse, BH, hd, T, a...)
                                        : launch_fwd_f32_lanes<D, 4>(q, k, v, o, lse, BH, hd, T, a...);
}

// Query heads side by side in a workgroup of nw waves, for G heads per key/value head:
// they read the same key/value rows, so the staged rows serve all of them.
int tile_heads(int G, int nw) {
    for (int h = nw; h > 1; h >>= 1)
        if (G % h == 0) return h;
    return 1;
}

// Chunks staged at a time: as many as keep `fixed` + `per` bytes a chunk, next to a kernel's
// static LDS (frequencies and sums, under 1 KB), within the LDS of a workgroup when four
// (slices of up to 32 bytes) or three workgroups share a CU.
int tile_chunks(int nc, size_t fixed, size_t per, int slice_pieces) {
    const size_t budget = slice_pieces <= 2 ? 39 * 1024 : 52 * 1024;
    int c = 1;
    while (c < nc && fixed + (size_t)(c + 1) * per <= budget) ++c;
    return c;
}

template <int D>
static hipError_t launch_fwd_tile(const void *q, const void *k, const void *v, void *o, float *lse,
                               int BH, const Heads &hd, int T, int W, const RungTable &rt,
                               const RungTable *rtp, const Layouts &lay, hipStream_t s, const RopeFreq &rf,
                               void *q_rot) {
    using S = uint16_t;
    using TL = Tile<S, D>;
    constexpr int nw = 4;
    TileShape ts;
    ts.hs = tile_heads(hd.G, nw);
    const int runs = nw / ts.hs;
    ts.tiles = (T + 16 * runs - 1) / (16 * runs);
    ts.blocks = ts.tiles * (BH / ts.hs);
    ts.nc = band_chunks(W);
    const size_t fixed = 2 * (size_t)16 * (runs - 1) * TL::kRow, per = 2 * (size_t)32 * TL::kRow;
    ts.cps = tile_chunks(ts.nc, fixed, per, TL::NC);
    bool interp = false;
    for (int r = 0; r < rt.n && !interp; ++r) interp = rt.w[r] != 0.f;
    const float sl2 = kLog2e / sqrtf((float)D);
    auto kern = rtp ? fwd_tile_kernel<D, true, true>
                    : interp ? fwd_tile_kernel<D, true, false> : fwd_tile_kernel<D, false, false>;
    return launch(kForward, kern, grid_of(ts.blocks), dim3(64 * nw), (unsigned)(fixed + per * ts.cps), s,
                  (const S *)q, (const S *)k, (const S *)v, (S *)o, lse, T, W, rt, rtp, sl2, ts, hd, lay,
                  (S *)q_rot, rf);
}

hipError_t launch_forward(int dtype, int D, const void *q, const void *k, const void *v, void *o,
                          float *lse, int BH, const Heads &hd, int T, int W, const RungTable &rt,
                          const RungTable *rtp, const Layouts &lay, hipStream_t s,
                          const RopeFreq *rq, void *q_rot) {
    if (forward_mfma_supported(dtype, D, W))
        return launch_forward_mfma(q, k, v, o, lse, BH, hd, T, W, rt, rtp, lay, s, rq, q_rot);
    const RopeFreq rf = rq ? *rq : RopeFreq{};
    if (dtype == 0 && D == 32) return launch_fwd_f32<32>(q, k, v, o, lse, BH, hd, T, W, rt, rtp, lay, s, rf, q_rot);
    if (dtype == 0 && D == 64) return launch_fwd_f32<64>(q, k, v, o, lse, BH, hd, T, W, rt, rtp, lay, s, rf, q_rot);
    if (dtype == 1 && D == 32) return launch_fwd_tile<32>(q, k, v, o, lse, BH, hd, T, W, rt, rtp, lay, s, rf, q_rot);
    if (dtype == 1 && D == 64) return launch_fwd_tile<64>(q, k, v, o, lse, BH, hd, T, W, rt, rtp, lay, s, rf, q_rot);
    if (dtype == 0 && D == 128) return launch_fwd_f32<128>(q, k, v, o, lse, BH, hd, T, W, rt, rtp, lay, s, rf, q_rot);
    if (dtype == 1 && D == 128) return launch_fwd_tile<128>(q, k, v, o, lse, BH, hd, T, W, rt, rtp, lay, s, rf, q_rot);
    return hipErrorInvalidValue;
}

}  // namespace fibattn
