// k_fp8.hip -- the FP8 (e4m3) form of the cost model (Sec. 5.2) on the fp8
// matrix cores, and the encoder that turns raw schedule features into its
// e4m3 input codes (the log transform of Sec. 5.2 happens there, once per
// feature value).  The arithmetic lives in eval_fp8.h.
#include <algorithm>

#include "eval_fp8.h"

namespace cm {
namespace {

using namespace fp8eval;

template <bool kStage, bool kIndexed, bool kSpread, int kQ>
__device__ __forceinline__ void eval_body(const EvalLaunchOf<kQ> &L,
                                          const Fp8Pack *__restrict__ pk, const uint8_t *codes,
                                          const float *terms, const float *__restrict__ U,
                                          float *__restrict__ cost, float *__restrict__ stage,
                                          const int32_t *__restrict__ ridx, uint32_t rows)
{
    __shared__ bf16eval::GroupShared sh;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int q = query_at(L.nq, blockIdx.x, [&](int j) { return L.q[j].task0; });
    const EvalQ &E = L.q[q];
    QueryView8 Q;
    // memoized rows: codes is the row table and sched_off locates the row numbers
    Q.x = kIndexed ? codes : codes + E.sched_off;
    Q.ridx = kIndexed ? ridx + E.sched_off : nullptr;
    Q.rows = rows;
    Q.t = terms + E.terms_off;
    Q.u = U + E.u_off;
    Q.cost = cost + E.cost_off;
    Q.stage = kStage ? stage + E.stage_off : nullptr;
    Q.S = E.S;
    Q.N = E.N;
    Q.P = kSpread ? stage_parts(E.S) : E.parts;
    const Weights8 w = load_weights8(pk, lane);
    const int group = blockIdx.x - E.task0;
    if (kSpread && Q.P < E.parts)
        eval_group8<false, false, false, kSpread>(Q, group, wave, lane, w, sh);
    else
        eval_group8<false, kStage, kIndexed>(Q, group, wave, lane, w, sh);
}

template <bool kStage, bool kIndexed, int kQ>
__global__ __launch_bounds__(EVAL_WAVES * 64) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_eval_fp8(
    EvalLaunchOf<kQ> L, const Fp8Pack *__restrict__ pk, const uint8_t *codes, const float *terms,
    const float *__restrict__ U, float *__restrict__ cost, float *__restrict__ stage,
    const int32_t *__restrict__ ridx, uint32_t rows)
{
    eval_body<kStage, kIndexed, false>(L, pk, codes, terms, U, cost, stage, ridx, rows);
}

template <int kQ>
__global__ __launch_bounds__(EVAL_WAVES * 64) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_eval_fp8_spread(
    EvalLaunchOf<kQ> L, const Fp8Pack *__restrict__ pk, const uint8_t *codes, const float *terms,
    const float *__restrict__ U, float *__restrict__ cost, float *__restrict__ stage,
    const int32_t *__restrict__ ridx, uint32_t rows)
{
    eval_body<false, false, true>(L, pk, codes, terms, U, cost, stage, ridx, rows);
}

// e4m3 code of v: NaN -> 0x7F, magnitudes beyond 448 saturate (the
// conversion instruction itself gives NaN there), round to nearest even.
__device__ inline uint32_t e4m3_pair(float a, float b)
{
    const float ca = __builtin_amdgcn_fmed3f(a, -448.f, 448.f);
    const float cb = __builtin_amdgcn_fmed3f(b, -448.f, 448.f);
    uint32_t w = (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(ca, cb, 0, false) & 0xffffu;
    if (a != a) w = (w & 0xff00u) | 0x7fu;
    if (b != b) w = (w & 0x00ffu) | 0x7f00u;
    return w;
}

// log1p(x) in float32 within a few ulps, from the hardware base-2 logarithm:
// with u = 1 + x rounded, log(u) * x / (u - 1) cancels the rounding of u to
// first order (Goldberg's method, "What every computer scientist should know
// about floating-point arithmetic", 1991); u == 1 means log1p(x) = x to
// float32 precision, and for huge |u - 1| (whose reciprocal would underflow)
// the rounding of u no longer matters.  -1 gives -inf, below -1 NaN, +inf
// stays +inf.
__device__ inline float log1p_fast(float x)
{
    const float u = 1.f + x;
    const float d = u - 1.f;
    if (d == 0.f) return x;
    const float l = __builtin_amdgcn_logf(u) * 0.6931471805599453f;
    if (!(fabsf(d) < 0x1p100f)) return l;
    return l * (x * __builtin_amdgcn_rcpf(d));
}

__device__ inline uint32_t encode4(float4 x, float s)
{
    const uint32_t lo = e4m3_pair(log1p_fast(x.x) * s, log1p_fast(x.y) * s);
    const uint32_t hi = e4m3_pair(log1p_fast(x.z) * s, log1p_fast(x.w) * s);
    return lo | (hi << 16);
}

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int ENC_THREADS = 256;
constexpr int ENC_PER = 4;                                // quads of values per thread
constexpr int ENC_TILE = ENC_THREADS * ENC_PER * 4;       // values per workgroup and round
constexpr uint32_t ENC_LIMIT = 0x71800000u;               // bits of 2^100

// encode4 for values with bits below ENC_LIMIT (+0 <= x < 2^100) and a scale
// of at most 2^13, the same codes with fewer instructions: no NaN, no
// negative result and no huge u - 1 to select for, and where u == 1 (x at
// most 2^-24, a code of 0 at such a scale) the product is 0.  sl = ln 2 * s:
// a power of two scales every product alike.
__device__ inline float log1p_scaled(float x, float sl)
{
    const float u = 1.f + x;
    const float d = fmaxf(u - 1.f, 0x1p-24f);
    return (__builtin_amdgcn_logf(u) * sl) * (x * __builtin_amdgcn_rcpf(d));
}

__device__ inline uint32_t encode4_plain(f32x4 x, float sl)
{
    float y[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
        y[j] = __builtin_amdgcn_fmed3f(log1p_scaled(x[j], sl), 0.f, 448.f);
    return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(
        y[2], y[3], __builtin_amdgcn_cvt_pk_fp8_f32(y[0], y[1], 0, false), true);
}

// n values in whole tiles, a quad of values (one 16-byte load, one 4-byte
// store) per thread and step, so that a wave's loads and stores are
// contiguous; the last workgroup takes the values past the last tile.  Bound
// by memory (5 bytes a value) only while the arithmetic stays under about 100
// cycles a wave and value: a wave whose values are all plain (features are
// counts and ratios) takes the short form.  The features are read once
// (non-temporal), the codes are the evaluator's next input (kept in the
// caches).  168 M values: 127 us (6.6 TB/s) against 157 us with 64 contiguous bytes
// per thread and the general form for every value.  A workgroup per tile:
// 8,192 workgroups that loop take 5% more, non-temporal stores 8%.
__global__ __launch_bounds__(ENC_THREADS) void k_fp8_encode(const float *__restrict__ x, int64_t n,
                                                            float s, float sl,
                                                            uint8_t *__restrict__ codes)
{
    const int64_t tiles = n / ENC_TILE;
    const f32x4 *x4 = reinterpret_cast<const f32x4 *>(x);
    uint32_t *c4 = reinterpret_cast<uint32_t *>(codes);
    const int t = threadIdx.x;
    for (int64_t g = blockIdx.x; g < tiles; g += gridDim.x) {
        const int64_t v0 = g * (ENC_TILE / 4) + t;
        f32x4 v[ENC_PER];
        uint32_t most = 0;
#pragma unroll
        for (int j = 0; j < ENC_PER; ++j)
            v[j] = __builtin_nontemporal_load(x4 + v0 + j * ENC_THREADS);
#pragma unroll
        for (int j = 0; j < ENC_PER; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) most = max(most, __float_as_uint(v[j][e]));
        uint32_t o[ENC_PER];
        if (sl != 0.f && !__any(most >= ENC_LIMIT)) {
#pragma unroll
            for (int j = 0; j < ENC_PER; ++j) o[j] = encode4_plain(v[j], sl);
        } else {
#pragma unroll
            for (int j = 0; j < ENC_PER; ++j)
                o[j] = encode4(make_float4(v[j][0], v[j][1], v[j][2], v[j][3]), s);
        }
#pragma unroll
        for (int j = 0; j < ENC_PER; ++j) c4[v0 + j * ENC_THREADS] = o[j];
    }
    if (blockIdx.x == gridDim.x - 1)
        for (int64_t i = tiles * ENC_TILE + t; i < n; i += ENC_THREADS)
            codes[i] = (uint8_t)(e4m3_pair(log1p_fast(x[i]) * s, 0.f) & 0xffu);
}

}  // namespace

hipError_t launch_eval_fp8(const EvalLaunch &L, const Model &m, const uint8_t *codes,
                           const float *terms, const float *U, float *cost, float *stage,
                           hipStream_t st, const int32_t *ridx, uint32_t rows)
{
    if (L.ntasks == 0) return hipSuccess;
    const dim3 g(L.ntasks), b(EVAL_WAVES * 64);
    const Fp8Pack *pk = m.d_fp8;
    auto go = [&](auto few, auto many) {
        return launch_eval(few, many, g, b, st, L, pk, codes, terms, U, cost, stage, ridx, rows);
    };
    if (ridx && stage) return go(k_eval_fp8<true, true, QFEW>, k_eval_fp8<true, true, QMAX>);
    if (ridx) return go(k_eval_fp8<false, true, QFEW>, k_eval_fp8<false, true, QMAX>);
    if (stage) return go(k_eval_fp8<true, false, QFEW>, k_eval_fp8<true, false, QMAX>);
    for (int q = 0; q < L.nq; ++q)
        if (L.q[q].parts > stage_parts(L.q[q].S))
            return go(k_eval_fp8_spread<QFEW>, k_eval_fp8_spread<QMAX>);
    return go(k_eval_fp8<false, false, QFEW>, k_eval_fp8<false, false, QMAX>);
}

// x and codes must be 16-byte aligned (checked by the caller).
hipError_t launch_fp8_encode(const float *x, int64_t n, float in_scale, uint8_t *codes,
                             hipStream_t st)
{
    if (n == 0) return hipSuccess;
    const int64_t blocks = std::min<int64_t>(std::max<int64_t>(1, n / ENC_TILE), 1 << 30);
    // 0: the short form does not hold for this scale (its codes of tiny values
    // would differ, or its products underflow)
    const float sl = in_scale >= 0x1p-40f && in_scale <= 0x1p13f ? 0.6931471805599453f * in_scale : 0.f;
    hipLaunchKernelGGL(k_fp8_encode, dim3((unsigned)blocks), dim3(ENC_THREADS), 0, st, x, n,
                       in_scale, sl, codes);
    return hipGetLastError();
}

}  // namespace cm
