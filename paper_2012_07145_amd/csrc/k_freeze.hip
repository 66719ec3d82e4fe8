// k_freeze.hip -- freezing of the lowest-cost stages (Sec. 3.2): for the
// candidate a search kept, every stage except the ceil(log2 S) most costly
// ones has its schedule options frozen.  One workgroup per query ranks the
// candidate's per-stage costs by counting.
#include "cm_internal.h"

namespace cm {
namespace {

constexpr int FREEZE_THREADS = 1024;
constexpr int FREEZE_CHUNK = 2048;  // stage keys staged in LDS at a time

// Order-preserving key of a stage cost: ascending cost, -0 == +0, NaN after
// every number (all NaNs equal).
__device__ inline uint32_t cost_key(float v)
{
    if (v != v) return 0xffffffffu;
    if (v == 0.f) v = 0.f;
    const uint32_t u = __float_as_uint(v);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Ranking key of stage s: its cost's key, equal costs by lower index.
__device__ inline uint64_t stage_key(const float *v, int64_t N, int s)
{
    return ((uint64_t)cost_key(v[(int64_t)s * N]) << 32) | (uint32_t)s;
}

// Latency only: three dependent loads (candidate, its costs, the keys in LDS).
// `per` threads share a stage's count, as many as the workgroup has for the
// query's stages, so 100 stages take 13 comparisons a thread instead of the
// 8 x 100 of one thread per stage that walked a fixed 2,048-slot round: 80 us
// for 5 queries of 60 to 120 stages, 3.9 us so.
__global__ __launch_bounds__(FREEZE_THREADS) void k_freeze(FreezeLaunch L,
                                                           const float *__restrict__ stage,
                                                           const int32_t *__restrict__ cand,
                                                           int64_t cand_stride,
                                                           uint8_t *__restrict__ frozen)
{
    __shared__ uint64_t keys[FREEZE_CHUNK];
    const FreezeQ &Q = L.q[blockIdx.x];
    const int S = Q.S, t = threadIdx.x;
    const int64_t N = Q.N;
    const int c = cand[Q.cand_q * cand_stride];
    uint8_t *out = frozen + Q.flag_off;
    if (c < 0 || c >= Q.N) {  // no candidate kept: nothing is frozen
        for (int s = t; s < S; s += FREEZE_THREADS) out[s] = 0;
        return;
    }
    const int lg = S > 1 ? 32 - __clz(S - 1) : 0;  // ceil(log2 S): the stages left unfrozen
    const int nfreeze = S - lg;
    const float *v = stage + Q.stage_off + c;  // v[s * N]

    // per: a power of two of at most 64, so a stage's threads share a wave
    int lper = 0;
    while (lper < 6 && ((int64_t)S << (lper + 1)) <= FREEZE_THREADS) ++lper;
    const int per = 1 << lper, sub = t & (per - 1), slot = t >> lper;
    for (int base = 0; base < S; base += FREEZE_THREADS >> lper) {
        const int s = base + slot;
        const uint64_t mine = s < S ? stage_key(v, N, s) : 0;
        int rank = 0;  // stages ahead of s
        for (int t0 = 0; t0 < S; t0 += FREEZE_CHUNK) {
            const int nt = min(FREEZE_CHUNK, S - t0);
            if (base == 0 || S > FREEZE_CHUNK) {
                __syncthreads();
                for (int j = t; j < nt; j += FREEZE_THREADS) keys[j] = stage_key(v, N, t0 + j);
                __syncthreads();
            }
#pragma unroll 4
            for (int j = sub; j < nt; j += per) rank += keys[j] < mine;
        }
        for (int d = 1; d < per; d <<= 1) rank += __shfl_xor(rank, d);
        if (sub == 0 && s < S) out[s] = rank < nfreeze ? 1 : 0;
    }
}

}  // namespace

hipError_t launch_freeze(const FreezeLaunch &L, const float *stage, const int32_t *cand,
                         int64_t cand_stride, uint8_t *frozen, hipStream_t st)
{
    if (L.nq == 0) return hipSuccess;
    hipLaunchKernelGGL(k_freeze, dim3(L.nq), dim3(FREEZE_THREADS), 0, st, L, stage, cand,
                       cand_stride, frozen);
    return hipGetLastError();
}

}  // namespace cm
