// Helpers of the tile kernels (fwd.hip, bwd.hip): every storage type and head size, any
// window, on gfx950 matrix cores.
//
// Lane layout: a wave owns 16 consecutive rows (queries in the forward and dq kernels,
// keys in the dk/dv kernel).  A row of D values is spread over four lanes; piece s of lane
// g is the row's 16-byte chunk 4s + g, so each 16-byte load instruction reads 64
// contiguous bytes of each of 16 rows.  The lane's values are its "slice", slice position
// 4b + i being element i of accumulator block b:
//   bfloat16: chunk 4s + g holds dims 32s + 8g + j: position 8s + j;
//   float32:  chunk 4s + g holds dims 16s + 4g + e: position 4s + e.
// In the MFMA layout row n is on lanes n + 16g, in the quad layout on lanes 4n + g (where
// rows are read from global memory: neighbouring lanes read neighbouring chunks).
// Products over the head dims take the slices as they are: v_mfma_f32_16x16x32_bf16 has
// k index 8g + j on lane group g, v_mfma_f32_16x16x4_f32 k index g.  Products over rows
// (P.V and the gradients) leave lane (n, g) with exactly its own slice of the output row.
//
// Precision: float32 rows are multiplied in float32.  bfloat16 rows are multiplied
// exactly (bf16 products in float32 accumulators); the float32 weights they are scaled by
// (probabilities, tau dS) keep their 24 bits: on the VALU they multiply the unpacked rows,
// on the matrix cores they are three bfloat16 parts of 8 bits, each with its own product.
#pragma once

#include "mfma.h"

namespace fibattn {

// ---- float32 rows on the VALU, every sum in one fixed order (fwd.hip, bwd.hip) -------
// The order is that of one lane per 16-byte chunk: a chain over the chunk's four products,
// then pairs of chunks, the farthest first.  dalpha is a sum of terms that cancel, which
// carries the rounding of lse and of the probabilities up by one to two decimal digits:
// another order of the same sums moves it by more than a float32 result may move.
__device__ __forceinline__ float chunk_dot(const u32x4 &x, const u32x4 &y) {
    float s = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) s = fmaf(__uint_as_float(x[e]), __uint_as_float(y[e]), s);
    return s;
}
// A value of lane l ^ M (M < 64, a power of two).
template <int M>
__device__ __forceinline__ float lane_xor(float x) {
    const int i = __float_as_int(x);
    if constexpr (M == 1) return __int_as_float(__builtin_amdgcn_update_dpp(0, i, 0xB1, 0xF, 0xF, true));
    if constexpr (M == 2) return __int_as_float(__builtin_amdgcn_update_dpp(0, i, 0x4E, 0xF, 0xF, true));
    if constexpr (M == 8) return __int_as_float(__builtin_amdgcn_update_dpp(0, i, 0x128, 0xF, 0xF, true));  // row_ror:8
    return __shfl_xor(x, M, 64);
}
// Sum of a row's chunk values, this lane's at positions L x + g of the row's L lanes.
template <int NC, int L = 4>
__device__ __forceinline__ float chunk_sum(float *t) {
#pragma unroll
    for (int h = NC / 2; h >= 1; h >>= 1)
#pragma unroll
        for (int x = 0; x < h; ++x) t[x] += t[x + h];
    float s = t[0];
    if constexpr (L > 16) s += lane_xor<16>(s);
    if constexpr (L > 8) s += lane_xor<8>(s);
    if constexpr (L > 4) s += lane_xor<4>(s);
    s += lane_xor<2>(s);
    s += lane_xor<1>(s);
    return s;
}
// Either bfloat16 of a word at least 2^16, or not finite.
constexpr uint32_t kLargeRow = 0x4780;
__device__ __forceinline__ bool large_pair(uint32_t w) {
    return (w & 0x7fff0000u) >= kLargeRow << 16 || (w & 0x7fffu) >= kLargeRow;
}
// L: lanes per row in the quad layout, 4 (neighbouring lanes L n + g), or one per 16-byte
// chunk of the row, which take the VALU functions alone.
template <typename S, int D, int L = 4>
struct Tile {
    static constexpr int kRow = D * (int)sizeof(S);  // bytes of a row
    static constexpr int NC = kRow / (16 * L);       // 16-byte pieces of a slice
    static constexpr int NB = D / (4 * L);           // accumulator blocks of a slice
    static constexpr bool kF32 = sizeof(S) == 4;

    struct Slice {
        u32x4 c[NC];
    };
    struct Acc {
        f32x4 c[NB];
    };

    __device__ static __forceinline__ void zero(Acc &a) {
#pragma unroll
        for (int b = 0; b < NB; ++b) a.c[b] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    __device__ static __forceinline__ void scale(Acc &a, float s) {
#pragma unroll
        for (int b = 0; b < NB; ++b) a.c[b] *= s;
    }

    __device__ static __forceinline__ bool finite(const Acc &a) {
        float x = 0.f;  // NaN if any element is not finite
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int e = 0; e < 4; ++e) x = fmaf(a.c[b][e], 0.f, x);
        return x == 0.f;
    }

    // Slice g of row `row`, rows `st` bytes apart from a uniform base (the host keeps
    // every row offset below 2^31 bytes).
    __device__ static __forceinline__ Slice load(const void *base, int row, int g, uint32_t st) {
        const char *p = reinterpret_cast<const char *>(base);
        const uint32_t off = (uint32_t)row * st + (uint32_t)g * 16u;
        Slice s;
#pragma unroll
        for (int x = 0; x < NC; ++x) s.c[x] = *reinterpret_cast<const u32x4 *>(p + off + 16 * L * x);
        return s;
    }
    // The lane's slice of an output row: a.c times `scale`, rounded to S.
    __device__ static __forceinline__ void store(void *row, int g, const Acc &a, float scale) {
        char *p = reinterpret_cast<char *>(row) + 16 * g;
#pragma unroll
        for (int x = 0; x < NC; ++x) {
            u32x4 v;
            if constexpr (kF32) {
                v = __builtin_bit_cast(u32x4, a.c[x] * scale);
            } else {
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const f32x4 &h = a.c[2 * x + (w >> 1)];
                    v[w] = pack_bf16(h[2 * (w & 1)] * scale, h[2 * (w & 1) + 1] * scale);
                }
            }
            __builtin_nontemporal_store(v, reinterpret_cast<u32x4 *>(p + 16 * L * x));
        }
    }

    // <x, y> over the slice, in four chains.
    __device__ static __forceinline__ float dot(const Slice &x, const Slice &y) {
        float s[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float &t = s[e];
                if constexpr (kF32)
                    t = fmaf(__uint_as_float(x.c[c][e]), __uint_as_float(y.c[c][e]), t);
                else
                    t = __builtin_amdgcn_fdot2_f32_bf16(as_bf2(x.c[c][e]), as_bf2(y.c[c][e]), t, false);
            }
        return (s[0] + s[1]) + (s[2] + s[3]);
    }

    // The same over the row's lanes; float32 rows in the fixed order above.
    __device__ static __forceinline__ float row_dot(const Slice &x, const Slice &y) {
        if constexpr (kF32) {
            float t[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) t[c] = chunk_dot(x.c[c], y.c[c]);
            return chunk_sum<NC, L>(t);
        } else {
            float t = dot(x, y);
            return chunk_sum<1, L>(&t);
        }
    }

    // acc += a x + b y with float32 weights.
    __device__ static __forceinline__ void axpy2(Acc &acc, float a, const Slice &x, float b, const Slice &y) {
        if constexpr (kF32) {
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    acc.c[c][e] = fmaf(a, __uint_as_float(x.c[c][e]),
                                       fmaf(b, __uint_as_float(y.c[c][e]), acc.c[c][e]));
        } else {
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    f32x4 &d = acc.c[2 * c + (w >> 1)];
                    const int e = 2 * (w & 1);
                    d[e] = fmaf(a, bf16_lo(x.c[c][w]), fmaf(b, bf16_lo(y.c[c][w]), d[e]));
                    d[e + 1] = fmaf(a, bf16_hi(x.c[c][w]), fmaf(b, bf16_hi(y.c[c][w]), d[e + 1]));
                }
        }
    }
    // The same with the two products added to each other first: a chain of half as many
    // roundings (float32 dk and dv of W 64: 0.97 -> 0.90 times as far from 64 bits).
    __device__ static __forceinline__ void add2(Acc &acc, float a, const Slice &x, float b, const Slice &y) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                if constexpr (kF32) {
                    acc.c[c][w] += fmaf(a, __uint_as_float(x.c[c][w]), b * __uint_as_float(y.c[c][w]));
                } else {
                    f32x4 &d = acc.c[2 * c + (w >> 1)];
                    const int e = 2 * (w & 1);
                    d[e] += fmaf(a, bf16_lo(x.c[c][w]), b * bf16_lo(y.c[c][w]));
                    d[e + 1] += fmaf(a, bf16_hi(x.c[c][w]), b * bf16_hi(y.c[c][w]));
                }
            }
    }
    // acc += a x.
    __device__ static __forceinline__ void axpy(Acc &acc, float a, const Slice &x) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                if constexpr (kF32) {
                    acc.c[c][w] = fmaf(a, __uint_as_float(x.c[c][w]), acc.c[c][w]);
                } else {
                    f32x4 &d = acc.c[2 * c + (w >> 1)];
                    const int e = 2 * (w & 1);
                    d[e] = fmaf(a, bf16_lo(x.c[c][w]), d[e]);
                    d[e + 1] = fmaf(a, bf16_hi(x.c[c][w]), d[e + 1]);
                }
            }
    }

    // A quad-layout slice moved to the MFMA layout, and an accumulator or a value moved
    // from the MFMA to the quad layout.
    __device__ static __forceinline__ Slice from_quad(const Slice &x, int lane) {
        const int src = 4 * (lane & 15) + (lane >> 4);
        Slice y;
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) y.c[c][e] = __shfl(x.c[c][e], src, 64);
        return y;
    }
    __device__ static __forceinline__ void to_quad_acc(Acc &a, int lane) {
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int e = 0; e < 4; ++e) a.c[b][e] = to_quad(a.c[b][e], lane);
    }

    // ---- rows staged in LDS -----------------------------------------------------------
    // Row-major, 16-byte chunk c of staged row r in slot c ^ swz(r), so that eight lanes
    // reading one chunk of consecutive rows cover the banks.
    __device__ static __forceinline__ int swz(int r) { return kRow == 64 ? (r >> 1) & 3 : r & 7; }
    __device__ static __forceinline__ const char *chunk(const char *buf, int r, int c) {
        return buf + r * kRow + 16 * (c ^ swz(r));
    }
    __device__ static __forceinline__ Slice staged(const char *buf, int r, int g) {
        Slice s;
#pragma unroll
        for (int x = 0; x < NC; ++x) s.c[x] = *reinterpret_cast<const u32x4 *>(chunk(buf, r, 4 * x + g));
        return s;
    }
    // A buffer laid out for the quad layout (stage with quad), whose eight neighbouring lanes
    // read four chunks each of two consecutive rows: slot c ^ 4 (r & 1).
    __device__ static __forceinline__ Slice staged_quad(const char *buf, int r, int g) {
        Slice s;
#pragma unroll
        for (int x = 0; x < NC; ++x)
            s.c[x] = *reinterpret_cast<const u32x4 *>(buf + r * kRow + 16 * ((4 * x + g) ^ (4 * (r & 1))));
        return s;
    }
    // Rows [r_begin, r_begin + nrows) of rows `st` elements apart, copied by direct-to-LDS
    // loads (1 KB per wave and instruction; nrows is a multiple of 16).  Rows outside [0, T)
    // are clamped copies of real rows: callers mask them.
    __device__ static __forceinline__ void stage(char *buf, const S *X, int r_begin, int nrows, int T, long long st,
                                                 int wave, int nwaves, bool quad = false) {
        const int lane = threadIdx.x & 63;
        constexpr int per = kRow / 16;  // chunks per row
        const int nblk = nrows * kRow / 1024;
        for (int blk = wave; blk < nblk; blk += nwaves) {
            const int u = blk * 64 + lane;
            const int rr = u / per, ch = (u % per) ^ (quad ? 4 * (rr & 1) : swz(rr));
            const int row = min(max(r_begin + rr, 0), T - 1);
            __builtin_amdgcn_global_load_lds(X + row * st + ch * (16 / (int)sizeof(S)),
                                             (__attribute__((address_space(3))) void *)(buf + 1024 * blk), 16, 0, 0);
        }
    }

    // ---- matrix products --------------------------------------------------------------
    // <rows a, columns b> over the head dims, 16 x 16.  float32: CH chains, which the
    // matrix pipeline overlaps and whose partial sums round less than one long chain.
    template <int CH = 4>
    __device__ static __forceinline__ f32x4 scores(const Slice &a, const Slice &b) {
        const f32x4 z{0.f, 0.f, 0.f, 0.f};
        if constexpr (kF32) {
            f32x4 r[CH];
#pragma unroll
            for (int x = 0; x < CH; ++x) r[x] = z;
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    r[(4 * c + e) % CH] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                        __uint_as_float(a.c[c][e]), __uint_as_float(b.c[c][e]), r[(4 * c + e) % CH], 0, 0, 0);
#pragma unroll
            for (int h = CH / 2; h >= 1; h >>= 1)
#pragma unroll
                for (int x = 0; x < h; ++x) r[x] += r[x + h];
            return r[0];
        } else {
            f32x4 r = z;
#pragma unroll
            for (int c = 0; c < NC; ++c)
                r = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a.c[c]),
                                                            __builtin_bit_cast(bf16x8, b.c[c]), r, 0, 0, 0);
            return r;
        }
    }
    // Weights of a 32-row chunk (two 16-row blocks of C-layout weights, p[4b + e] for row
    // 16b + 4g + e and the lane's column), as matrix operands.
    struct Weights {
        u32x4 h, m, l;  // bfloat16: the leading 8 bits, the next and the last
        float f[8];     // float32
    };
    __device__ static __forceinline__ Weights weights(const float *p) {
        Weights w;
        if constexpr (kF32) {
#pragma unroll
            for (int e = 0; e < 8; ++e) w.f[e] = p[e];
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                w.h[e] = pack_bf16(p[2 * e], p[2 * e + 1]);
                const float a = p[2 * e] - bf16_lo(w.h[e]), b = p[2 * e + 1] - bf16_hi(w.h[e]);
                w.m[e] = pack_bf16(a, b);
                w.l[e] = pack_bf16(a - bf16_lo(w.m[e]), b - bf16_hi(w.m[e]));
            }
        }
        return w;
    }
    // acc += rows^T . w over the staged rows [base, base + 32) (MFMA layout).
    __device__ static __forceinline__ void accumulate(Acc &acc, const char *buf, int base, const Weights &w, int g) {
        const int m = threadIdx.x & 15;
        if constexpr (kF32) {
            // A operand of step (block h, e): dim 16b + m of row base + 16h + 4g + e
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int r = base + 16 * h + 4 * g + e;
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
                        const float a = *reinterpret_cast<const float *>(chunk(buf, r, 4 * b + (m >> 2)) + 4 * (m & 3));
                        acc.c[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, w.f[4 * h + e], acc.c[b], 0, 0, 0);
                    }
                }
        } else {
            // A operand by LDS transpose reads (lane addressing as dma_operand_t)
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                v4i16 t[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int r = base + 16 * h + 4 * g + (m >> 2);
                    t[h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                        (__attribute__((address_space(3))) v4i16 *)(chunk(buf, r, 4 * (b >> 1) + (m & 3)) + 8 * (b & 1)));
                }
                const bf16x8 A = __builtin_bit_cast(bf16x8, t);
                acc.c[b] = mfma(A, __builtin_bit_cast(bf16x8, w.l), acc.c[b]);
                acc.c[b] = mfma(A, __builtin_bit_cast(bf16x8, w.m), acc.c[b]);
                acc.c[b] = mfma(A, __builtin_bit_cast(bf16x8, w.h), acc.c[b]);
            }
        }
    }

    // Whether `rows` staged bfloat16 rows from `base` on, or the wave's rows x, hold a large
    // element.
    __device__ static __forceinline__ bool large_rows(const char *buf, int base, int rows) {
        bool t = false;
#pragma unroll 1
        for (int i = threadIdx.x & 63; i < rows * (kRow / 16); i += 64) {
            const u32x4 w = *reinterpret_cast<const u32x4 *>(buf + base * kRow + 16 * i);
#pragma unroll
            for (int e = 0; e < 4; ++e) t |= large_pair(w[e]);
        }
        return __builtin_amdgcn_ballot_w64(t);
    }
    __device__ static __forceinline__ bool large_rows(const Slice &x) {
        bool t = false;
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) t |= large_pair(x.c[c][e]);
        return __builtin_amdgcn_ballot_w64(t);
    }

    // What a frequency (radians per position) is multiplied with for rope: the RoPE launch of
    // bfloat16 rows of 64 reduces the angle in radians, the others' in revolutions.
    static constexpr double kRopeUnit = !kF32 && D == 64 ? 1.0 : 0.15915494309189533576888376337251;
    // RoPE of the lane's slice of a row at position t, with the angles, the order of the
    // products and the rounding of the RoPE launch: its bits.  Partners as in rope_t.
    __device__ static __forceinline__ void rope(Slice &x, int t, const double *sf, int g) {
        if constexpr (NC == 1 && kF32) {
            const bool hi = g >= L / 2;  // this lane holds the second halves of its pairs
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float c, s;
                rope_cs_f64(t, sf[4 * (g & (L / 2 - 1)) + e], c, s);
                const float u = __uint_as_float(x.c[0][e]), o = lane_xor<L / 2>(u);
                x.c[0][e] = __float_as_uint(hi ? fmaf(s, o, c * u) : fmaf(c, u, -(s * o)));
            }
        } else if constexpr (kF32) {
#pragma unroll
            for (int a = 0; a < NC / 2; ++a)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float c, s, u, w;
                    rope_cs_f64(t, sf[4 * (L * a + g) + e], c, s);
                    u = __uint_as_float(x.c[a][e]);
                    w = __uint_as_float(x.c[a + NC / 2][e]);
                    x.c[a][e] = __float_as_uint(fmaf(c, u, -(s * w)));
                    x.c[a + NC / 2][e] = __float_as_uint(fmaf(s, u, c * w));
                }
        } else if constexpr (D == 32) {
            const bool hi = g & 2;  // this lane holds the second halves of its pairs
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t own = x.c[0][e];
                const uint32_t oth = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)own, 0x4E, 0xF, 0xF, true);
                float r[2];
#pragma unroll
                for (int z = 0; z < 2; ++z) {
                    float c, s;
                    rope_cs_f64(t, sf[8 * (g & 1) + 2 * e + z], c, s);
                    const float a = z ? bf16_hi(own) : bf16_lo(own), b = z ? bf16_hi(oth) : bf16_lo(oth);
                    r[z] = hi ? fmaf(s, b, c * a) : fmaf(c, a, -(s * b));
                }
                x.c[0][e] = pack_bf16(r[0], r[1]);
            }
        } else {
#pragma unroll
            for (int a = 0; a < NC / 2; ++a)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint32_t uw = x.c[a][e], ww = x.c[a + NC / 2][e];
                    float ox[2], oy[2];
#pragma unroll
                    for (int z = 0; z < 2; ++z) {
                        float c, s;
                        const float u = z ? bf16_hi(uw) : bf16_lo(uw), w = z ? bf16_hi(ww) : bf16_lo(ww);
                        if constexpr (D == 64) {
                            rope_cs(t, sf[32 * a + 8 * g + 2 * e + z], c, s);
                            rope_rotate(u, w, c, s, ox[z], oy[z]);
                        } else {
                            rope_cs_f64(t, sf[32 * a + 8 * g + 2 * e + z], c, s);
                            ox[z] = fmaf(c, u, -(s * w));
                            oy[z] = fmaf(s, u, c * w);
                        }
                    }
                    x.c[a][e] = pack_bf16(ox[0], ox[1]);
                    x.c[a + NC / 2][e] = pack_bf16(oy[0], oy[1]);
                }
        }
    }
    // The lane's slice written to a row (read again by the backward: ordinary stores).
    __device__ static __forceinline__ void put(void *row, int g, const Slice &x) {
#pragma unroll
        for (int c = 0; c < NC; ++c) *reinterpret_cast<u32x4 *>(reinterpret_cast<char *>(row) + 16 * g + 16 * L * c) = x.c[c];
    }

    // R^T (the inverse RoPE rotation) of the lane's slice at position t.  float32: the RoPE
    // launch's angles and order, its bits.  bfloat16: float32 sums rotated with cos and sin of
    // the hardware units (2.3e-7) and rounded once, where a launch on the stored gradients
    // rounds twice: dq and dk are 0.91 times as far from 64 bits as with it (float64 angles
    // here: B4 H8 T2048 d 64 W 64 step 74.1 -> 79.4 us).  sf: revolutions per position of
    // every frequency.  The partner of dim d < D/2 is d + D/2: D/8 slice
    // positions on, except for bfloat16 rows of 32, whose partner lanes are g and g + 2.
    __device__ static __forceinline__ void rope_t(Acc &a, int t, const double *sf, int g) {
        if constexpr (NC == 1) {
            constexpr int PV = 16 / (int)sizeof(S);
            const bool hi = g >= L / 2;  // this lane holds the second halves of its pairs
#pragma unroll
            for (int p = 0; p < PV; ++p) {
                float c, s;
                const double f = sf[PV * (g & (L / 2 - 1)) + p];
                const float x = a.c[p >> 2][p & 3], o = lane_xor<L / 2>(x);
                if constexpr (kF32) {
                    rope_cs_f64(t, f, c, s);
                    a.c[p >> 2][p & 3] = hi ? fmaf(-s, o, c * x) : fmaf(c, x, s * o);
                } else {
                    rope_cs_rev(t, f, c, s);
                    a.c[p >> 2][p & 3] = hi ? x * c - o * s : x * c + o * s;
                }
            }
        } else {
            constexpr int HB = NB / 2;
#pragma unroll
            for (int b = 0; b < HB; ++b)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int p = 4 * b + e;
                    const int dim = kF32 ? 4 * (L * b + g) + e : 32 * (p >> 3) + 8 * g + (p & 7);
                    float c, s;
                    const float x = a.c[b][e], y = a.c[HB + b][e];
                    if constexpr (kF32) {
                        rope_cs_f64(t, sf[dim], c, s);
                        a.c[b][e] = fmaf(c, x, s * y);
                        a.c[HB + b][e] = fmaf(-s, x, c * y);
                    } else {
                        rope_cs_rev(t, sf[dim], c, s);
                        a.c[b][e] = x * c + y * s;
                        a.c[HB + b][e] = y * c - x * s;
                    }
                }
        }
    }
};

// Probability exp(tau s - lse) of a backward entry, with the forward's sl2 = fl(tau log2e),
// whose rounding the saved lse shares, and lse2 = fl(lse log2e), which mostly gives back the
// base-2 value that the forward rounded to lse.
__device__ __forceinline__ float prob(float s, float sl2, float lse2) { return exp2f(fmaf(s, sl2, -lse2)); }
// The same with what the rounding of lse log2e loses multiplied back in (lse itself given):
// for float32 logits from the matrix cores, which are not rounded as the forward's and gain
// nothing from its rounding of lse.  dk and dv against 64 bits, as a multiple of one lane
// group per key: matrix cores (W 24 to 128) 0.82 to 0.90 with it, 0.88 to 0.94 without;
// logits in the forward's order (W 4 to 16) 0.91 to 0.95 with it, 0.89 to 0.92 without.
__device__ __forceinline__ float prob_low(float s, float sl2, float l) {
    const float v = l * kLog2e;
    // kLog2e + 1.925963e-8 = log2(e); an infinite lse (a dropped query) loses nothing
    float low = fmaf(l, 1.925963033500e-8f, fmaf(l, kLog2e, -v)) * kLn2;
    low = __builtin_isfinite(v) ? low : 0.f;
    const float p = prob(s, sl2, v);
    return fmaf(p, -low, p);
}

// Weights 2^x of a bfloat16 band that the matrix cores cannot take in full: three bfloat16
// parts hold 24 bits from 2^-109 on (their last one is a multiple of 2^-133), and the exp2
// instruction gives 0 below 2^-126.  They count only next to large rows: where every element
// is below 2^16 what is lost of a sum is below 2^-70 (rows of weights times dP: 2^-126 2^39
// 2^16).  Heads whose logits spread by more than 69 in a window are ordinary: their waves look
// at the staged rows (least: the least x of the lane's rows, in the window or not) and go on.
constexpr float kLeastWeight = -100.f;
__device__ __forceinline__ bool tiny_weight(float least) { return __builtin_amdgcn_ballot_w64(least < kLeastWeight); }

// Weight and lane bookkeeping of a launch: `nw` waves per workgroup are `hs` query heads
// of one group (all reading the same rows) times nw / hs runs of 16 rows.
struct TileShape {
    int blocks; // workgroups
    int tiles;  // workgroups along the sequence
    int hs;     // query heads side by side
    int nc;     // 32-row band chunks: they cover W + 16 rows
    int cps;    // chunks staged at a time
};

// This workgroup's number in a grid_of grid (>= the workgroup count: nothing to do).
__device__ __forceinline__ int block_number() { return (int)(blockIdx.y * gridDim.x + blockIdx.x); }

inline int band_chunks(int W) { return (W + 16 + 31) / 32; }

}  // namespace fibattn
