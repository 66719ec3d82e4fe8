// hoist_dev.h -- float32 matrix-core helpers, and a wave's hoisted rows on the
// float32 matrix cores (Sec. 5.2):
//   U[s] = (b_1 + W_1[:, :24] (b_p + W_p log1p(pipe[s])) + beta) scale
// for up to 4 consecutive stages s at once, with the rounding of a scalar chain
// of fused multiply-adds over ascending features and embeddings (one 16x16x4
// float32 matrix instruction adds four consecutive terms of the chain in
// ascending order, rounding each).  Bound by latency: 5 features' logarithms a
// lane and 40 matrix instructions of 32 cycles for its up to 4 stages, under the
// wait for the first stage's features.  For a kernel of one stage per wave the
// scalar chains of k_plain.hip are shorter (17 ragged queries' hoist 4.2 us, and
// 4.5 us with this).
#pragma once

#include "cm_internal.h"

namespace cm {
namespace hoist {

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ inline f32x4 mfma4(float a, float b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__device__ inline void swap32(float &a, float &b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false,
                                                    false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}

__device__ inline void swap16(float &a, float &b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false,
                                                    false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}

// A layer's output tile (lane group g = lane / 16 holds rows 4g .. 4g+3 of
// its column) as the next layer's operands: step t's operand is row 4t + g,
// the transpose of the 4 x 4 (group, register) grid.
__device__ inline void transpose4(f32x4 &v)
{
    float a = v[0], b = v[1], c = v[2], d = v[3];
    swap32(a, c);
    swap32(b, d);
    swap16(a, b);
    swap16(c, d);
    v = f32x4{a, b, c, d};
}

constexpr int ROWS = 4;                              // most stages of a call
constexpr int PASSES = (ROWS * FP + 63) / 64;        // logarithms of a lane

// The features of `rows` (1 .. ROWS) consecutive stages at p, held by a lane
// until hoist_rows: loads without a branch, past the last value the last one.
__device__ __forceinline__ void load_pipe(float (&v)[PASSES], const float *p, int rows, int lane)
{
    const auto *g = (const __attribute__((address_space(1))) float *)p;
    const int last = rows * FP - 1;
#pragma unroll
    for (int j = 0; j < PASSES; ++j) v[j] = g[min(lane + 64 * j, last)];
}

// The rows' hoisted vectors into lds[row][32], which is used for their
// logarithms first (ROWS * FP floats, this wave's alone; its LDS operations
// complete in order).
__device__ __forceinline__ void hoist_rows(const HoistPack *__restrict__ pk,
                                           const float (&v)[PASSES], int rows, float scale,
                                           float *lds, int lane)
{
    const int g = lane >> 4, n = lane & 15;
    f32x4 w[10];
#pragma unroll
    for (int k = 0; k < 10; ++k) w[k] = __builtin_bit_cast(f32x4, pk->w[k][lane]);
    f32x4 e0 = __builtin_bit_cast(f32x4, pk->bp[g]);
    f32x4 e1 = __builtin_bit_cast(f32x4, pk->bp[4 + g]);
    f32x4 h0 = __builtin_bit_cast(f32x4, pk->b1[g]);
    f32x4 h1 = __builtin_bit_cast(f32x4, pk->b1[4 + g]);
#pragma unroll
    for (int j = 0; j < PASSES; ++j)
        if (64 * j < rows * FP) lds[64 * j + lane] = log1pf(v[j]);
    __builtin_amdgcn_wave_barrier();
    const float *lp = lds + min(n, rows - 1) * FP + g;  // columns past the rows: the last one's
    float x[FP / 4];
#pragma unroll
    for (int t = 0; t < FP / 4; ++t) x[t] = lp[4 * t];
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int t = 0; t < FP / 4; ++t) {
        e0 = mfma4(w[t / 4][t % 4], x[t], e0);
        e1 = mfma4(w[(14 + t) / 4][(14 + t) % 4], x[t], e1);
    }
    transpose4(e0);
    transpose4(e1);
#pragma unroll
    for (int t = 0; t < E / 4; ++t) {
        const float e = t < 4 ? e0[t] : e1[t - 4];
        h0 = mfma4(w[(28 + t) / 4][(28 + t) % 4], e, h0);
        h1 = mfma4(w[(34 + t) / 4][(34 + t) % 4], e, h1);
    }
    const f32x4 b0 = __builtin_bit_cast(f32x4, pk->beta[g]);
    const f32x4 b1 = __builtin_bit_cast(f32x4, pk->beta[4 + g]);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        h0[j] = (h0[j] + b0[j]) * scale;
        h1[j] = (h1[j] + b1[j]) * scale;
    }
    if (n < rows) {
        f32x4 *out = reinterpret_cast<f32x4 *>(lds + n * H);
        out[g] = h0;
        out[4 + g] = h1;
    }
    __builtin_amdgcn_wave_barrier();
}

}  // namespace hoist
}  // namespace cm
