// Device helpers shared by the score/decision kernels and the fused score + decision + compaction kernel: the
// per-token score of Eq. 2 (or its relative form) finished from the per-row partial sums of squares that the
// projection stage took from its fp32 accumulators.
#pragma once

#include "common.h"

namespace dash {

// Quarter qd (0..3) of the sum of a row's partial pairs: pairs qd, qd + 4, ... in order. The four quarters are added in order
// qd = 0..3, so a score has the same bits whoever finishes it.
template <int UNROLL = 4>
__device__ __forceinline__ float2 row_quarter(const float* __restrict__ partials, int cols, int fold, int n, int row, int qd) {
    float sd = 0.f, sx = 0.f;
    if (row < n) {
        const float2* src = reinterpret_cast<const float2*>(partials) + row;
        if (fold == 1) {
#pragma unroll UNROLL
            for (int p = qd; p < cols; p += 4) {
                const float2 v = src[(size_t)p * n];
                sd += v.x;
                sx += v.y;
            }
        } else {  // kNormFold neighbouring columns make up a partial: added in order, all loads of a few partials in flight
#pragma unroll UNROLL
            for (int c0 = qd * kNormFold; c0 < cols; c0 += 4 * kNormFold) {
                float2 v[kNormFold];
#pragma unroll
                for (int c = 0; c < kNormFold; ++c) {
                    v[c] = src[(size_t)min(c0 + c, cols - 1) * n];
                    if (c0 + c >= cols) v[c] = make_float2(0.f, 0.f);
                }
#pragma unroll
                for (int c = 1; c < kNormFold; ++c) {
                    v[0].x += v[c].x;
                    v[0].y += v[c].y;
                }
                sd += v[0].x;
                sx += v[0].y;
            }
        }
    }
    return make_float2(sd, sx);
}
__device__ __forceinline__ float2 add_quarters(float2 a, float2 b, float2 c, float2 d) {
    return make_float2(a.x + b.x + c.x + d.x, a.y + b.y + c.y + d.y);
}
// The same sum by one thread, in few registers.
__device__ __forceinline__ float2 row_sums(const float* __restrict__ partials, int cols, int fold, int n, int row) {
    float2 q[4];
#pragma unroll
    for (int qd = 0; qd < 4; ++qd) q[qd] = row_quarter<1>(partials, cols, fold, n, row, qd);
    return add_quarters(q[0], q[1], q[2], q[3]);
}

// Sum of the partial pairs of one row, taken by the four threads (row, q = 0..3) of a 256-thread workgroup that covers 64 rows.
__device__ __forceinline__ float2 row_sums_256(const float* __restrict__ partials, int cols, int fold, int n, int row_base,
                                               float2 (*red)[kChunkRows]) {
    const int r = threadIdx.x % kChunkRows, qd = threadIdx.x / kChunkRows;
    red[qd][r] = row_quarter(partials, cols, fold, n, row_base + r, qd);
    __syncthreads();
    // valid in every thread; callers use the copy of wave 0
    return add_quarters(red[0][r], red[1][r], red[2][r], red[3][r]);
}

__device__ __forceinline__ float score_from_sums(float2 t, int score_kind) {
    const float nd = sqrtf(t.x);
    if (score_kind == DASH_SCORE_ABS) return nd;
    return nd / fmaxf(sqrtf(t.y), kNormEps);
}

// Order-preserving map from fp32 to uint32 for the total order in which TopK ranks scores:
//   -inf < ... < -0.0 = +0.0 < ... < +inf < NaN   (every NaN, whatever its sign or payload, is one value).
// Eq. 3 ranks real numbers; this is the reading for the other values a float can hold: a NaN score ranks highest
// (the threshold rule keeps NaN rows as well, "score < tau" being false), the two zeros tie and are told apart
// by row like any tie.
__device__ __forceinline__ uint32_t order_key(float f) {
    if (f != f) return 0xFFFFFFFFu;
    const uint32_t b = __float_as_uint(f == 0.0f ? 0.0f : f);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

}  // namespace dash
