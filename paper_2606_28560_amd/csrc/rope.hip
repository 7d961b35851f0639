// RoPE at true positions (Section 2 "Attended set": rotary embeddings are applied
// at the true positions before gathering; Section 3: base 1e4).
//
// Rotate-half pairing: for j < D/2 the pair (x_j, x_{j+D/2}) of the row at position t
// rotates by theta = t * base^(-2j/D).  A workgroup owns a few consecutive positions
// and a group of (b, h) rows at those positions; it evaluates cos/sin of its angles
// once, rounds them to float32 in LDS, and rotates every row with them.
#include <algorithm>

#include "launch.h"

namespace fibattn {

// blockIdx.z selects the tensor: (x0 -> y0) of BH0 rows (batch * heads) or (x1 -> y1) of BH1
// (k may have fewer heads than q), each packed [BH, T, D].

// Any storage type and head size (bfloat16 with d_head 64 has the kernel below): a lane
// rotates the pairs of a 16-byte piece of the row's first half and the matching piece of
// its second half, NP heads apart by blockDim / lanes; a workgroup owns 512 / D positions,
// one angle per thread.  The loads are issued before the angles are evaluated.
// What bounds it: the latency of one load, one angle and one store per workgroup, and memory
// for large tensors.  NP = 2 from 1024 workgroups on (four a CU), where fewer angles per row
// pay; NP = 1 below, where workgroups are short.
// Us a launch, against one element pair per thread with float64 pow and sincos: bf16 d 128
// B2 H16 T2000 20.2 -> 5.0; bf16 d 32 B8 H8 T1024 8.0 -> 4.9; fp32 d 64 B4 H8 T1024 11.4 -> 5.8.
template <typename S, int D, int NP>
__global__ __launch_bounds__(256) void rope_kernel(const S *x0, S *y0, const S *x1, S *y1, int T, RopeFreq rf,
                                                   int transpose, int BH0, int BH1, TableJob job) {
    constexpr int HALF = D / 2, TP = 256 / HALF, VN = Vec<S>::N;
    constexpr int LPR = HALF / VN;              // lanes per row
    constexpr int HR = 256 / (LPR * TP);        // heads per pass
    __shared__ float cs[256], sn[256];
    if (job.out && blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0 && threadIdx.x == 0)
        table_from_theta(job.theta, job.alpha, job.b, job.W, job.out);
    const S *x = blockIdx.z ? x1 : x0;
    S *y = blockIdx.z ? y1 : y0;
    const int BH = blockIdx.z ? BH1 : BH0;
    const int col = VN * (threadIdx.x % LPR), tt = threadIdx.x / LPR % TP, hh = threadIdx.x / (LPR * TP);
    // one pass each unless the grid had to be cut to its limits
    for (long long t0 = (long long)blockIdx.x * TP; t0 < T; t0 += (long long)gridDim.x * TP)
        for (int b = blockIdx.y; b * HR * NP < BH; b += gridDim.y) {
            const int t = (int)min(t0 + tt, (long long)T - 1), bh0 = b * HR * NP + hh;
            float u[NP][VN], w[NP][VN];
#pragma unroll
            for (int n = 0; n < NP; ++n) {
                const S *p = x + ((size_t)min(bh0 + n * HR, BH - 1) * T + t) * D + col;
                Vec<S>::load(p, u[n]);
                Vec<S>::load(p + HALF, w[n]);
            }
            if (b == (int)blockIdx.y) {
                float c, s;
                rope_cs_f64((int)t0 + (int)threadIdx.x / HALF,
                            rf.inv[threadIdx.x % HALF] * 0.15915494309189533576888376337251, c, s);
                __syncthreads();  // the angles of the positions before are done with
                cs[threadIdx.x] = c;
                sn[threadIdx.x] = transpose ? -s : s;
                __syncthreads();
            }
            if (t0 + tt >= T) continue;
#pragma unroll
            for (int n = 0; n < NP; ++n) {
                if (bh0 + n * HR >= BH) continue;
                float ox[VN], oy[VN];
#pragma unroll
                for (int e = 0; e < VN; ++e) {
                    const float c = cs[tt * HALF + col + e], s = sn[tt * HALF + col + e];
                    ox[e] = fmaf(c, u[n][e], -(s * w[n][e]));
                    oy[e] = fmaf(s, u[n][e], c * w[n][e]);
                }
                S *p = y + ((size_t)(bh0 + n * HR) * T + t) * D + col;
                Vec<S>::store(p, ox);
                Vec<S>::store(p + HALF, oy);
            }
        }
}

// bfloat16, d_head 64: a workgroup owns 4 NP positions of 16 (b, h) rows; each lane group
// of four handles NP positions (t, t + 4) of one head.  NP = 2 (two rows' loads in flight
// per lane) for two tensors (10.7 -> 10.2 us for q and k of the 60M layer) and for one
// tensor of at least 2^17 rows (k of the T = 4096 layer: 11.4 -> 10.1 us); NP = 1 for a
// smaller single tensor, which doubles its workgroup count (k of the T = 1024 layer keeps
// 1024 workgroups).
// Lane group g of a row's four lanes holds dims [8g, 8g+8) and [32+8g, 32+8g+8),
// i.e. the eight rotate-half pairs (j, j+32), j in [8g, 8g+8): two 16-byte loads
// and stores per lane and row, reading 64 contiguous bytes per row per instruction.
// The loads are issued before the angles are evaluated.
constexpr int kRope64RB = 16;

// two float32 -> bfloat16 (round to nearest even) in one conversion instruction
typedef __bf16 rope_bf16x2 __attribute__((ext_vector_type(2)));
typedef float rope_f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack2_bf16(float lo, float hi) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((rope_f32x2){lo, hi}, rope_bf16x2));
}

template <int NP>
__global__ __launch_bounds__(256) void rope_bf16_d64_kernel(const uint16_t *x0, uint16_t *y0,
                                                            const uint16_t *x1, uint16_t *y1,
                                                            int T, RopeFreq rf, int transpose,
                                                            int BH0, int BH1, TableJob job) {
    constexpr int kRope64TP = 4 * NP;  // positions per workgroup
    __shared__ float cs[kRope64TP * 32], sn[kRope64TP * 32];
    const uint16_t *x = blockIdx.z ? x1 : x0;
    uint16_t *y = blockIdx.z ? y1 : y0;
    const int BH = blockIdx.z ? BH1 : BH0;
    if (job.out && blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0 && threadIdx.x == 0)
        table_from_theta(job.theta, job.alpha, job.b, job.W, job.out);
    if (blockIdx.y * kRope64RB >= BH) return;  // the tensor with fewer heads
    const int t0 = blockIdx.x * kRope64TP;
    const int g = threadIdx.x & 3;
    const int rr = threadIdx.x >> 2;  // 0..63
    const int bh = blockIdx.y * kRope64RB + (rr >> 2);
    const int bhc = min(bh, BH - 1);
    uint4 a[NP], b[NP];
    const uint16_t *xr[NP];
    uint16_t *yr[NP];
#pragma unroll
    for (int h = 0; h < NP; ++h) {  // positions t0 + (rr & 3) (and t0 + (rr & 3) + 4)
        const int tc = min(t0 + (rr & 3) + 4 * h, T - 1);
        const size_t row = ((size_t)bhc * T + tc) * 64;
        xr[h] = x + row;
        yr[h] = y + row;
        a[h] = *reinterpret_cast<const uint4 *>(xr[h] + 8 * g);
        b[h] = *reinterpret_cast<const uint4 *>(xr[h] + 32 + 8 * g);
    }
    if (threadIdx.x < kRope64TP * 32) {
        float c, sv;
        rope_cs(t0 + (threadIdx.x >> 5), rf.inv[threadIdx.x & 31], c, sv);
        cs[threadIdx.x] = c;
        sn[threadIdx.x] = transpose ? -sv : sv;
    }
    __syncthreads();
    if (bh >= BH) return;
#pragma unroll
    for (int h = 0; h < NP; ++h) {
        const int tt = (rr & 3) + 4 * h;
        if (t0 + tt >= T) continue;
        const uint32_t aw[4] = {a[h].x, a[h].y, a[h].z, a[h].w}, bw[4] = {b[h].x, b[h].y, b[h].z, b[h].w};
        uint32_t ow[4], pw[4];
        const float *C = cs + tt * 32 + 8 * g;
        const float *Sn = sn + tt * 32 + 8 * g;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float u0 = bf16_lo(aw[w]), u1 = bf16_hi(aw[w]);
            const float v0 = bf16_lo(bw[w]), v1 = bf16_hi(bw[w]);
            const float c0 = C[2 * w], c1 = C[2 * w + 1], s0 = Sn[2 * w], s1 = Sn[2 * w + 1];
            ow[w] = pack2_bf16(u0 * c0 - v0 * s0, u1 * c1 - v1 * s1);
            pw[w] = pack2_bf16(v0 * c0 + u0 * s0, v1 * c1 + u1 * s1);
        }
        *reinterpret_cast<uint4 *>(yr[h] + 8 * g) = make_uint4(ow[0], ow[1], ow[2], ow[3]);
        *reinterpret_cast<uint4 *>(yr[h] + 32 + 8 * g) = make_uint4(pw[0], pw[1], pw[2], pw[3]);
    }
}

RopeFreq make_rope_freq(double rope_base, int D) {
    RopeFreq rf;
    rf.on = rope_base > 0.0;
    for (int j = 0; j < 64; ++j) rf.inv[j] = (j < D / 2 && rf.on) ? pow(rope_base, -2.0 * (double)j / (double)D) : 0.0;
    return rf;
}

template <typename S, int D>
static hipError_t launch_rope_t(const void *x0, void *y0, const void *x1, void *y1, int T, const RopeFreq &rf,
                                int transpose, int BH0, int BH1, const TableJob &job,
                                hipStream_t s) {
    constexpr int TP = 512 / D, HR = 256 * Vec<S>::N / (D / 2 * TP);
    const int rows = x1 ? std::max(BH0, BH1) : BH0, nt = T / TP + (T % TP != 0), z = x1 ? 2 : 1;
    const int np = (long long)nt * ((rows + 2 * HR - 1) / (2 * HR)) * z >= 1024 ? 2 : 1;
    return launch(kRope, np == 2 ? rope_kernel<S, D, 2> : rope_kernel<S, D, 1>,
                  dim3(std::min(nt, 1 << 22), std::min((rows + np * HR - 1) / (np * HR), 65535), z), dim3(256), 0, s, (const S *)x0, (S *)y0,
                  (const S *)x1, (S *)y1, T, rf, transpose, BH0, BH1, job);
}

// One launch for one tensor (x1 == nullptr) or two tensors of BH0 and BH1 rows (batch *
// heads), packed.  The table job (job.out set) rides on it.
hipError_t launch_rope(int dtype, int D, const void *x0, void *y0, const void *x1, void *y1, int BH0, int BH1, int T,
                       float rope_base, int transpose, hipStream_t s, const TableJob *job) {
    const RopeFreq rf = make_rope_freq((double)rope_base, D);
    TableJob nojob{};
    const TableJob &tj = job ? *job : nojob;
    if (dtype == 1 && D == 64) {
        const int rows = x1 ? std::max(BH0, BH1) : BH0;
        const bool np2 = x1 || (long long)BH0 * T >= (1ll << 17);
        const int tp = np2 ? 8 : 4;  // positions per workgroup
        return launch(kRope, np2 ? rope_bf16_d64_kernel<2> : rope_bf16_d64_kernel<1>,
                      dim3((T + tp - 1) / tp, (rows + kRope64RB - 1) / kRope64RB, x1 ? 2 : 1), dim3(256), 0, s, x0,
                      y0, x1, y1, T, rf, transpose, BH0, BH1, tj);
    }
#define FIBATTN_ROPE(S, DD)                                                    \
    if ((dtype == 0) == (sizeof(S) == 4) && D == DD)                           \
        return launch_rope_t<S, DD>(x0, y0, x1, y1, T, rf, transpose, BH0, BH1, tj, s);
    FIBATTN_ROPE(float, 32)
    FIBATTN_ROPE(float, 64)
    FIBATTN_ROPE(float, 128)
    FIBATTN_ROPE(uint16_t, 32)
    FIBATTN_ROPE(uint16_t, 128)
#undef FIBATTN_ROPE
    return hipErrorInvalidValue;
}

}  // namespace fibattn
