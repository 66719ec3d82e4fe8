// k_plain.hip -- per-stage hoist and the float32 evaluator.
//
// Hoist (one workgroup per stage): the algorithm features of a stage are the
// same for every candidate of the query, so their embedding and its share of
// the first layer are computed once per stage:
//   U[s] = W_1[:, :24] (W_p log1p(pipe[s]) + b_p) + b_1        (Sec. 5.2)
// plus W_1[:, 24:] b_s when the evaluator folds the schedule embedding into
// the first layer, times the hidden scale s_h of the FP8 form (1 else).
//
// Float32 evaluator: log1p of the 40 schedule features, the schedule
// embedding, the ReLU layer on the stacked embeddings, the ReLU coefficient
// layer and the dot product with the 8 cost terms (Sec. 5.2, App. B), on the
// float32 matrix cores, and a Kahan-compensated float32 sum over stages in
// ascending order.
#include <algorithm>

#include "cm_internal.h"
#include "hoist_dev.h"

namespace cm {
namespace {

using namespace hoist;

// One stage row of the hoist by a 64-thread workgroup: p = the stage's 56
// algorithm features, u = its 32 output floats.
__device__ inline void hoist_row(const float *__restrict__ params, const float *__restrict__ beta,
                                 int fold, float scale, const float *p, float *u, float *lp,
                                 float *ep)
{
    const int t = threadIdx.x;
    if (t < FP) lp[t] = log1pf(p[t]);
    __syncthreads();
    if (t < E) {
        const float *w = params + OFF_WP + t * FP;
        float a = params[OFF_BP + t];
        for (int f = 0; f < FP; ++f) a = fmaf(w[f], lp[f], a);
        ep[t] = a;
    }
    __syncthreads();
    if (t < H) {
        const float *w = params + OFF_W1 + t * 2 * E;
        float a = params[OFF_B1 + t];
        for (int e = 0; e < E; ++e) a = fmaf(w[e], ep[e], a);
        if (fold) a += beta[t];
        u[t] = a * scale;
    }
    __syncthreads();  // lp and ep are reused by the next row
}

template <int kQ>
__global__ __launch_bounds__(64) void k_hoist(EvalLaunchOf<kQ> L, const float *__restrict__ params,
                                              const float *__restrict__ beta, int fold,
                                              float scale, const float *__restrict__ pipe,
                                              float *__restrict__ U)
{
    __shared__ float lp[FP];
    __shared__ float ep[E];
    const int q = query_at(L.nq, blockIdx.x, [&](int j) { return L.q[j].hrow0; });
    const int s = blockIdx.x - L.q[q].hrow0;
    hoist_row(params, beta, fold, scale, pipe + L.q[q].pipe_off + (int64_t)s * FP,
              U + L.q[q].u_off + (int64_t)s * H, lp, ep);
}

// Hoist of a step: the rows of every query, grid-stride, from the device
// descriptors (the folded form of the bf16 and FP8 evaluators, with
// W_1[:, 24:] b_s folded in), times *scale when given (the FP8 form's s_h,
// read at run time so that a recorded launch follows the model's form).
__global__ __launch_bounds__(64) void k_hoist_step(const StepHead *__restrict__ h,
                                                   const StepQ *__restrict__ qs,
                                                   const float *__restrict__ params,
                                                   const float *__restrict__ beta,
                                                   const float *__restrict__ scale)
{
    __shared__ int32_t row0[STEP_MAX_QUERIES];
    __shared__ float lp[FP];
    __shared__ float ep[E];
    const int nq = h->nq, nrows = h->nrows;
    for (int j = threadIdx.x; j < nq; j += 64) row0[j] = qs[j].row0;
    __syncthreads();
    for (int r = blockIdx.x; r < nrows; r += gridDim.x) {
        // the last query whose first row is <= r
        int lo = 0, hi = nq - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (row0[mid] <= r) lo = mid;
            else hi = mid - 1;
        }
        const StepQ &D = qs[lo];
        const int s = r - row0[lo];
        hoist_row(params, beta, 1, scale ? *scale : 1.f, D.pipe + (int64_t)s * FP,
                  D.u + (int64_t)s * H, lp, ep);
    }
}

// The same for descriptors in the kernel's arguments, one row per workgroup.
__global__ __launch_bounds__(64) void k_hoist_step_value(StepArgs a,
                                                         const float *__restrict__ params,
                                                         const float *__restrict__ beta,
                                                         const float *__restrict__ scale)
{
    static_assert(STEP_VALUE_QUERIES <= 64, "one lane per query");
    __shared__ float lp[FP];
    __shared__ float ep[E];
    const int q = query_at(a.h.nq, blockIdx.x, [&](int j) { return a.q[j].row0; });
    const int s = blockIdx.x - a.q[q].row0;
    hoist_row(params, beta, 1, scale ? *scale : 1.f, a.q[q].pipe + (int64_t)s * FP,
              a.q[q].u + (int64_t)s * H, lp, ep);
}

// ---- float32 evaluator ----
// Every sum is the same chain of fused multiply-adds, in the same order, that
// a scalar walk over features, embedding and hidden units gives: one
// 16x16x4 float32 matrix instruction adds four consecutive terms of the chain
// in ascending order, rounding each (compared bit for bit with the fmaf chain
// over a million sums, subnormal ones included).  So the layers stay
// unfolded: bs + Ws x, then u + W1 es, then b2 + W2 h.

typedef __attribute__((address_space(3))) void lds_void;

// Packed operands of the first layer held by a lane for the whole launch (lane
// l: row l % 16, term 4t + l / 16 of step t) and its part of the accumulator
// seeds (rows 4 (l / 16) .. +3).  The other two layers' operands are read from
// LDS in each stage, where the logarithms need the registers.
struct Fp32Weights {
    float ws[2][10];
    f32x4 bs[2], b2;
};

__device__ inline Fp32Weights load_fp32(const Fp32Pack *__restrict__ pk, int lane)
{
    Fp32Weights W;
#pragma unroll
    for (int v = 0; v < 5; ++v) {
        const float4 x = pk->w[v][lane];
        const float w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) W.ws[(4 * v + j) / 10][(4 * v + j) % 10] = w[j];
    }
    const int g = lane >> 4;
    const float4 s0 = pk->bs[g], s1 = pk->bs[4 + g], s2 = pk->b2[g];
    W.bs[0] = f32x4{s0.x, s0.y, s0.z, s0.w};
    W.bs[1] = f32x4{s1.x, s1.y, s1.z, s1.w};
    W.b2 = f32x4{s2.x, s2.y, s2.z, s2.w};
    return W;
}

__device__ inline float relu32(float a) { return a < 0.f ? 0.f : a; }  // a NaN passes through

__device__ inline __amdgpu_buffer_rsrc_t rows_at(const float *p, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p), (short)0, bytes, 0x00020000);
}

// log1p(x) in float64, rounded to float32, and whether that may not be
// log1pf(x) (`unsure`).  With u = 1 + x in an interval of middle c and
// 1/c = inv rounded to float32, log(u) = -log(inv) + log1p(r) for
// r = x inv + (inv - 1), |r| < 2^-6.9, by five terms; in the interval at 1,
// inv = 1 and r = x, which keeps small x and 0 exact.  log1pf rounds to the
// other neighbour only where the value lies within its own error of the
// midpoint of two floats: over every float32 from 0 to 65,535 at most 0.0787,
// 0.0336, 0.0170, 0.0089 units in the last place for u of exponent 0, 1, 2,
// 3 .. 5 and 0.0041 above.  A value nearer to a midpoint than its entry's width
// (a little more) and any other x (negative, -0, larger, NaN) is left to
// log1pf, so that every result has its bits.
constexpr uint32_t LOG32_END = 0x477fff00u;  // 65,535

__device__ inline float log1p64(float x, const LogEntry &T, uint64_t &near, uint64_t &outside)
{
    const double inv = (double)T.inv;
    const double r = fma((double)x, inv, inv - 1.0);
    const double p = fma(r, fma(r, fma(r, 0.2, -0.25), 1.0 / 3.0), -0.5);
    const double y = fma(r * r, p, r) + T.log;
    // the 29 bits that float32 drops, as a distance from one half of its unit
    const uint32_t low = ((uint32_t)__builtin_bit_cast(uint64_t, y) << 3) + T.near;
    near = __builtin_amdgcn_ballot_w64(low <= 2 * T.near);  // 2^32 drops out of both
    outside = __builtin_amdgcn_ballot_w64(__float_as_uint(x) >= LOG32_END);
    return (float)y;
}

// log1pf of a wave's 10 values per lane: those that are not sure (2 to 3% of
// lognormal features) are gathered in the wave's list and go through log1pf
// 64 at a time.  Five table reads are in flight together, and a sure value's
// write to the list and its read go to a slot of its lane behind the list, so
// that there is no branch between them.
constexpr int LIST32 = 64 * 10;
__device__ __forceinline__ void log1p_wave(float (&x)[10], const LogEntry *tab, float *list)
{
    const int lane = threadIdx.x & 63;
    uint64_t mask[10];
    uint32_t slot[10];
    uint32_t n = 0;
#pragma unroll
    for (int half = 0; half < 10; half += 5) {
        LogEntry T[5];
#pragma unroll
        for (int t = 0; t < 5; ++t)
            T[t] = tab[(__float_as_uint(1.f + x[half + t]) >> (23 - LOG32_BITS)) & (LOG32_N - 1)];
#pragma unroll
        for (int t = half; t < half + 5; ++t) {
            uint64_t near, outside;
            const float y = log1p64(x[t], T[t - half], near, outside);
            const uint64_t m = near | outside;
            const uint32_t at = __builtin_amdgcn_mbcnt_hi(
                (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, n));
            slot[t] = __builtin_amdgcn_inverse_ballot_w64(m) ? at : (uint32_t)(LIST32 + lane);
            list[slot[t]] = x[t];
            n += (uint32_t)__popcll(m);
            mask[t] = m;
            x[t] = y;
        }
    }
    __builtin_amdgcn_wave_barrier();
    for (uint32_t j = lane; j < n; j += 64) list[j] = log1pf(list[j]);
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int half = 0; half < 10; half += 5) {
        float y[5];
#pragma unroll
        for (int t = 0; t < 5; ++t) y[t] = list[slot[half + t]];
        asm volatile("" : "+v"(y[0]), "+v"(y[1]), "+v"(y[2]), "+v"(y[3]), "+v"(y[4]));
#pragma unroll
        for (int t = 0; t < 5; ++t)
            x[half + t] = __builtin_amdgcn_inverse_ballot_w64(mask[half + t]) ? y[t] : x[half + t];
    }
}

// One stage of 16 candidates: x = log1p of features 4t + g of candidate
// lane % 16, u = the stage's hoisted units 4g .. +3 and 16 + 4g .. +3, tr =
// cost terms 4g .. 4g+3 of that candidate (g < 2).  Returns the stage's cost
// in lanes 16..31.
__device__ __forceinline__ float stage32(const float (&x)[10], const f32x4 (&u)[2], const f32x4 &tr,
                                         const Fp32Weights &W, const float4 (*wt)[64])
{
    const int lane = threadIdx.x & 63;
    float wl[20];  // W_1 (12) and W_2 (8)
#pragma unroll
    for (int v = 0; v < 5; ++v) {
        const float4 q = wt[v][lane];
        wl[4 * v] = q.x;
        wl[4 * v + 1] = q.y;
        wl[4 * v + 2] = q.z;
        wl[4 * v + 3] = q.w;
    }
    // matrix instructions first: the other waves' logarithms fill the cycles
    // between them (2% at 64 x 32,768)
    __builtin_amdgcn_s_setprio(1);
    f32x4 e0 = W.bs[0], e1 = W.bs[1];
#pragma unroll
    for (int t = 0; t < 10; ++t) {
        e0 = mfma4(W.ws[0][t], x[t], e0);
        e1 = mfma4(W.ws[1][t], x[t], e1);
    }
    transpose4(e0);
    transpose4(e1);
    f32x4 h0 = u[0], h1 = u[1];
#pragma unroll
    for (int t = 0; t < 6; ++t) {
        const float e = t < 4 ? e0[t] : e1[t - 4];
        h0 = mfma4(wl[t], e, h0);
        h1 = mfma4(wl[6 + t], e, h1);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        h0[j] = relu32(h0[j]);
        h1[j] = relu32(h1[j]);
    }
    transpose4(h0);
    transpose4(h1);
    f32x4 c = W.b2;
#pragma unroll
    for (int t = 0; t < 8; ++t) c = mfma4(wl[12 + t], t < 4 ? h0[t] : h1[t - 4], c);
    __builtin_amdgcn_s_setprio(0);
    // coefficients 0..3 of the chain in lane group 0, then 4..7 in group 1
    float v = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) v = fmaf(relu32(c[j]), tr[j], v);
    float w = v;
    swap16(v, w);  // v: group 0's partial sum in groups 0 and 1
#pragma unroll
    for (int j = 0; j < 4; ++j) v = fmaf(relu32(c[j]), tr[j], v);
    return v;
}

constexpr int F32_WAVES = 8;     // waves per workgroup
constexpr int F32_CHUNK = 128;   // stages between two rounds of summing
constexpr int F32_ROW = FS * 4;  // bytes of a feature row

struct Fp32Shared {
    uint4 xs[F32_WAVES][FP32_TILE * F32_ROW / 16];  // one stage's feature rows of each wave
    float v[2][F32_CHUNK][FP32_TILE];               // stage costs of two chunks
    float2 carry[FP32_TILE];                        // (sum, compensation) between chunks
    LogEntry log[LOG32_N];
    float4 w[5][64];                      // operands of the second and third layer
    float list[F32_WAVES][LIST32 + 64];  // values whose logarithm log1pf takes
};

// Loads of one wave's stage, issued one stage ahead of its arithmetic: the
// tile's 16 feature rows (2,560 contiguous bytes) straight into the wave's
// LDS block as whole cache lines, terms and hoisted units into registers.
__device__ __forceinline__ void issue32(const EvalQ &Q, const float *sched, const float *terms,
                                        const float *U, int s, int i0, int rows, int lane,
                                        uint4 *xsw, f32x4 (&u)[2], f32x4 &tr)
{
    constexpr int NT = 2;  // non-temporal: read exactly once
    const int64_t r = (int64_t)s * Q.N + i0;
    const auto xr = rows_at(sched + Q.sched_off + r * FS, rows * F32_ROW);
    const auto tq = rows_at(terms + Q.terms_off + r * C, rows * C * 4);
    const int g = lane >> 4, n = lane & 15;
    tr = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                       tq, n * (C * 4) + (g & 1) * 16, 0, NT));
    const float4 *ur = reinterpret_cast<const float4 *>(U + Q.u_off + (int64_t)s * H);
    u[0] = __builtin_bit_cast(f32x4, ur[g]);
    u[1] = __builtin_bit_cast(f32x4, ur[4 + g]);
    const int vo = lane * 16;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, (lds_void *)xsw, 16, vo, 0, 0, NT);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, (lds_void *)(xsw + 64), 16, vo + 1024, 0, 0, NT);
    if (lane < 32)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, (lds_void *)(xsw + 128), 16, vo + 2048, 0, 0,
                                                 NT);
}
static_assert(FP32_TILE * F32_ROW == 2560, "three copies of 1,024 + 1,024 + 512 bytes");

// A workgroup takes tiles of 16 candidates; its waves share a tile's stages
// (wave w: w, w + 8, ...), write the stage costs to LDS, and one wave, a
// different one for each chunk of stages, adds them in ascending order with
// compensation while the others go on.
// Bound by the vector ALU and the matrix cores, which overlap little: about 400
// vector instructions a wave and stage, 270 of them for the logarithms of its
// 10 values a lane (log1pf itself is 75 a value), and 40 matrix instructions of
// 32 cycles.  One query of 30 x 6,400: 515 us with one thread per candidate
// (100 waves, each a serial walk over the stages), 42 us in tiles with log1pf
// for every value, 31 us so; 4 x 64: 80, 6.5 and 6.0 us; 64 x 32,768 with its
// selection: 304 us with log1pf, 201 us so.
template <int kQ>
__global__ __launch_bounds__(F32_WAVES * 64) __attribute__((amdgpu_waves_per_eu(4, 4))) void
k_eval_fp32(EvalLaunchOf<kQ> L, const Fp32Pack *__restrict__ pk, const float *sched, const float *terms,
            const float *__restrict__ U, float *__restrict__ cost, float *__restrict__ stage)
{
    __shared__ Fp32Shared sh;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4, n = lane & 15;
    const Fp32Weights W = load_fp32(pk, lane);
    uint4 *xsw = sh.xs[wave];
    const float *xw = reinterpret_cast<const float *>(xsw);
    for (int i = threadIdx.x; i < LOG32_N; i += F32_WAVES * 64) sh.log[i] = pk->log[i];
    if (threadIdx.x < 5 * 64) sh.w[0][threadIdx.x] = pk->w[5][threadIdx.x];
    __syncthreads();
    int round = 0;
    for (int task = blockIdx.x; task < L.ntasks; task += gridDim.x) {
        const int q = query_at(L.nq, task, [&](int j) { return L.q[j].task0; });
        const EvalQ &Q = L.q[q];
        const int i0 = (task - Q.task0) * FP32_TILE;
        const int rows = min(FP32_TILE, Q.N - i0);
        for (int c0 = 0; c0 < Q.S; c0 += F32_CHUNK, ++round) {
            const int c1 = min(c0 + F32_CHUNK, Q.S);
            float(*vb)[FP32_TILE] = sh.v[round & 1];
            f32x4 u[2], tr;
            if (c0 + wave < c1) issue32(Q, sched, terms, U, c0 + wave, i0, rows, lane, xsw, u, tr);
            for (int s = c0 + wave; s < c1; s += F32_WAVES) {
                // the copy has landed (the compiler's own waits need not see
                // this read of the block)
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                float x[10];
#pragma unroll
                for (int t = 0; t < 10; ++t) x[t] = xw[n * FS + 4 * t + g];
                // the rows are in registers before the block is refilled
                asm volatile("" ::"v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(x[4]), "v"(x[5]),
                             "v"(x[6]), "v"(x[7]), "v"(x[8]), "v"(x[9])
                             : "memory");
                f32x4 u0[2] = {u[0], u[1]}, t0 = tr;
                if (s + F32_WAVES < c1)
                    issue32(Q, sched, terms, U, s + F32_WAVES, i0, rows, lane, xsw, u, tr);
                asm volatile("" ::: "memory");
                log1p_wave(x, sh.log, sh.list[wave]);
                const float v = stage32(x, u0, t0, W, sh.w);
                if (g == 1) {
                    vb[s - c0][n] = v;
                    if (stage && n < rows) stage[Q.stage_off + (int64_t)s * Q.N + i0 + n] = v;
                }
            }
            __syncthreads();
            // the chunk's sum; the next chunk's stage costs go to the other
            // buffer, and this wave reaches the next barrier only after it
            if (wave == (round & (F32_WAVES - 1)) && lane < FP32_TILE) {
                float sum = 0.f, comp = 0.f;
                if (c0) {
                    sum = sh.carry[lane].x;
                    comp = sh.carry[lane].y;
                }
                const int m = c1 - c0;
#pragma unroll 8
                for (int s = 0; s < m; ++s) {
                    const float y = vb[s][lane] - comp;
                    const float t = sum + y;
                    comp = (t - sum) - y;
                    sum = t;
                }
                if (c1 < Q.S) sh.carry[lane] = make_float2(sum, comp);
                else if (lane < rows) cost[Q.cost_off + i0 + lane] = sum;
            }
        }
    }
}

}  // namespace

hipError_t launch_hoist(const EvalLaunch &L, const Model &m, bool fold, float scale,
                        const float *pipe, float *U, hipStream_t st)
{
    if (L.nstages == 0) return hipSuccess;
    return launch_eval(k_hoist<QFEW>, k_hoist<QMAX>, dim3(L.nstages), dim3(64), st, L, m.d->params,
                       m.d->beta, fold ? 1 : 0, scale, pipe, U);
}

hipError_t launch_step_hoist(const StepHead *h, const StepQ *qs, const Model &m,
                             cm_precision prec, int grid, hipStream_t st)
{
    const float *scale = prec == CM_FP8 ? &m.d_fp8->uh : nullptr;
    hipLaunchKernelGGL(k_hoist_step, dim3(grid), dim3(64), 0, st, h, qs, m.d->params, m.d->beta,
                       scale);
    return hipGetLastError();
}

hipError_t launch_step_hoist(const StepArgs &a, const Model &m, cm_precision prec, hipStream_t st)
{
    if (a.h.nrows == 0) return hipSuccess;
    const float *scale = prec == CM_FP8 ? &m.d_fp8->uh : nullptr;
    hipLaunchKernelGGL(k_hoist_step_value, dim3(a.h.nrows), dim3(64), 0, st, a, m.d->params,
                       m.d->beta, scale);
    return hipGetLastError();
}

hipError_t launch_eval_fp32(const EvalLaunch &L, const Model &m, const float *sched,
                            const float *terms, const float *U, float *cost, float *stage,
                            hipStream_t st)
{
    if (L.ntasks == 0) return hipSuccess;
    // two workgroups of 8 waves fill a compute unit (4 waves per SIMD)
    const int grid = std::min(L.ntasks, 2 * m.cus);
    return launch_eval(k_eval_fp32<QFEW>, k_eval_fp32<QMAX>, dim3(grid), dim3(F32_WAVES * 64), st,
                       L, &m.d->fp32, sched, terms, U, cost, stage);
}

}  // namespace cm
