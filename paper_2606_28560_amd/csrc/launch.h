// Host-side launchers of the fibattn kernels (internal to libfibattn.so).
#pragma once

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.h"

namespace fibattn {

// 4: the dalpha sum, which the dk/dv launch carries
enum KernelId { kRope = 0, kForward = 1, kBwdDq = 2, kBwdDkDv = 3, kAlpha = 5, kNumKernels = 6 };

// The start/stop event pair for the next launch of kernel `id` while kernel timing is
// active for it; false otherwise.
bool timing_events(int id, hipEvent_t *start, hipEvent_t *stop);

// Launches `kernel`; while timing is active for `id` the launch carries an event pair that
// takes the dispatch's own start and end timestamps (hipExtLaunchKernel), so the pair
// measures this kernel alone, free of marker packets and launch gaps.
template <typename... P, typename... A>
hipError_t launch(int id, void (*kernel)(P...), dim3 grid, dim3 block, unsigned lds, hipStream_t s,
                  A... args) {
    hipEvent_t e0, e1;
    if (timing_events(id, &e0, &e1))
        hipExtLaunchKernelGGL(kernel, grid, block, lds, s, e0, e1, 0u, static_cast<P>(args)...);
    else
        hipLaunchKernelGGL(kernel, grid, block, lds, s, static_cast<P>(args)...);
    return hipGetLastError();
}

// Grid of `blocks` workgroups of up to 256 threads: one row, or rows of 2^23 (a dimension
// times the workgroup's threads stays below 2^32); kernels drop the last row's excess.
inline dim3 grid_of(long long blocks) {
    const long long x = blocks < (1ll << 23) ? blocks : 1ll << 23;
    return dim3((unsigned)x, (unsigned)((blocks + x - 1) / x));
}

// dtype: 0 float32, 1 bfloat16.  All launchers return hipGetLastError() of their launches.
// BH = batch * query heads; k, v (and dk, dv) hold BH / hd.G heads.  rtp != nullptr:
// the rung table is the device-resident one at rtp (rt unused).  rq: q is unrotated and
// each query row is rotated with these frequencies where the forward loads it; the rotated
// rows go to q_rot, placed by lay.dq (null: only where forward_mfma_supported).
hipError_t launch_forward(int dtype, int D, const void *q, const void *k, const void *v, void *o,
                          float *lse, int BH, const Heads &hd, int T, int W, const RungTable &rt,
                          const RungTable *rtp, const Layouts &lay, hipStream_t s,
                          const RopeFreq *rq = nullptr, void *q_rot = nullptr);

// Tile kernels (fwd.hip, bwd.hip): query heads side by side in a workgroup of nw waves, and
// band chunks staged at a time (tile.h).
int tile_heads(int G, int nw);
int tile_chunks(int nc, size_t fixed, size_t per, int slice_pieces);

// float32 forward and dq: D / 4 lanes per query in the place of 4 up to 12288 queries, where
// 4 lanes make at most 768 waves for the 1024 SIMDs and a launch is the latency of one
// wave's chain of rows.  Measured against 4 lanes over batches of 128 to 65536 queries, d 32
// / 64 / 128, W 3 to 64: forward at 4096 queries 0.92 to 0.99 / 0.73 to 0.87 / 0.47 to 0.72
// times, at 12000 0.97 to 1.02 / 0.94 to 0.98 / 0.84 to 1.03, at 16000 0.97 to 1.02 / 1.05 to
// 1.11 / 1.03 to 1.20; dq the same within 0.1.
inline bool f32_wide(int BH, int T) { return (long long)BH * T <= 12288; }

// dalpha partials the workspace holds: at least one per workgroup of the dq kernel.
size_t bwd_num_partials(int dtype, int D, int BH, int T);

// dtheta (nullable, device tables only): also writes dalpha * rtp->dadtheta there.
hipError_t launch_backward(int dtype, int D, const void *q, const void *k, const void *v,
                           const void *o, const float *lse, const void *dO, void *dq, void *dk,
                           void *dv, float *dalpha, float *dtheta, float *delta_ws, double *partials,
                           const RungTerms &terms, int BH, const Heads &hd, int T, int W,
                           const RungTable &rt, const RungTable *rtp, const RopeFreq &rf,
                           const Layouts &lay, hipStream_t s);

// bfloat16, d_head = 64, W <= 16: matrix-core band + VALU rungs (fwd_mfma.hip, bwd_mfma.hip).
bool forward_mfma_supported(int dtype, int D, int W);
// rq, q_rot: as launch_forward.
hipError_t launch_forward_mfma(const void *q, const void *k, const void *v, void *o, float *lse,
                               int BH, const Heads &hd, int T, int W, const RungTable &rt,
                               const RungTable *rtp, const Layouts &lay, hipStream_t s,
                               const RopeFreq *rq = nullptr, void *q_rot = nullptr);
bool backward_mfma_supported(int dtype, int D, int W);
size_t bwd_mfma_num_partials(int BH, int T);
hipError_t launch_backward_mfma(const void *q, const void *k, const void *v, const void *o,
                                const float *lse, const void *dO, void *dq, void *dk, void *dv,
                                float *dalpha, float *dtheta, float *delta_ws, double *partials,
                                const RungTerms &terms, int BH, const Heads &hd, int T, int W,
                                const RungTable &rt, const RungTable *rtp, const RopeFreq &rf,
                                const Layouts &lay, hipStream_t s);

RopeFreq make_rope_freq(double rope_base, int D);  // on = 0 when rope_base <= 0

// Device-resident alpha: builds the rung table from *alpha (one thread) into *out.
hipError_t launch_rung_table(const float *alpha, const BaseTable &b, int W, RungTable *out,
                             hipStream_t s);
// The same from *theta: alpha = 0.5 + sigmoid(theta) (written to *alpha_out when not null)
// and the table, which also records d alpha / d theta, in one launch.
hipError_t launch_rung_table_theta(const float *theta, float *alpha_out, const BaseTable &b, int W,
                                   RungTable *out, hipStream_t s);
// alpha_l = 0.5 + sigmoid(theta_l); dtheta_l = dalpha_l sigmoid(theta_l) (1 - sigmoid(theta_l)).
hipError_t launch_alpha_from_theta(const float *theta, float *alpha, int n, hipStream_t s);
hipError_t launch_dtheta(const float *theta, const float *dalpha, float *dtheta, int n, hipStream_t s);

// RoPE of one tensor (x1 == nullptr) or of two tensors in one launch: BH0 and BH1 rows
// (batch * heads), packed.  A table job (may be null) is carried by the launch.
hipError_t launch_rope(int dtype, int D, const void *x0, void *y0, const void *x1, void *y1, int BH0, int BH1, int T,
                       float rope_base, int transpose, hipStream_t s, const TableJob *job = nullptr);

}  // namespace fibattn
