// k_penalty.hip -- the known-bad-state penalty of the multi-pass search
// (Sec. 4.5): a candidate whose structural hash at the current pass's depth
// was seen before and judged unpromising gets a cost penalty, which moves it
// back in the beam before selection.
#include "cm_internal.h"

namespace cm {
namespace {

constexpr int SAMPLES = 1024;  // hashes of the bad set kept in LDS

// First position in a[0, n) (ascending) whose value is at least h.
template <class T>
__device__ inline int64_t lower_bound(const T *a, int64_t n, uint64_t h)
{
    int64_t lo = 0;
    while (n > 0) {
        const int64_t half = n >> 1;
        if (a[lo + half] < h) {
            lo += half + 1;
            n -= half + 1;
        } else {
            n = half;
        }
    }
    return lo;
}

// One thread per candidate of a query.  Every step-th hash
// of the bad set goes to LDS first, so that the bisection waits for memory
// only inside one step (not at all up to 1,024 hashes): 400 hashes and 17
// queries, 6.2 us with a walk over the queries and the bisection in memory,
// 4.1 us so.  512 threads share the samples: with 256, 1 M candidates against
// 100,000 hashes took 45.6 us a call (42.2 without samples, 39.3 so).
__global__ __launch_bounds__(PENALTY_THREADS) void k_penalty(PenaltyLaunch L,
                                                             const uint64_t *__restrict__ hashes,
                                                             const uint64_t *__restrict__ bad,
                                                             int64_t n_bad, int64_t step,
                                                             float penalty,
                                                             float *__restrict__ cost)
{
    __shared__ uint64_t sample[SAMPLES];
    const PenaltyQ &Q = L.q[query_at(L.nq, blockIdx.x, [&](int j) { return L.q[j].block0; })];
    const int64_t i = (int64_t)((int)blockIdx.x - Q.block0) * PENALTY_THREADS + threadIdx.x;
    const int64_t at = Q.cost_off + min(i, (int64_t)Q.N - 1);
    const uint64_t h = hashes[at];
    const float c = cost[at];
    const int ns = (int)((n_bad + step - 1) / step);  // <= SAMPLES
    for (int j = threadIdx.x; j < ns; j += PENALTY_THREADS) sample[j] = bad[j * step];
    __syncthreads();
    const int64_t below = lower_bound(sample, ns, h);  // samples under h
    bool hit = below < ns && sample[below] == h;
    if (!hit && step > 1 && below > 0) {
        const int64_t b0 = (below - 1) * step;
        const int64_t n = min(step, n_bad - b0);
        const int64_t k = lower_bound(bad + b0, n, h);
        hit = k < n && bad[b0 + k] == h;
    }
    if (hit && i < Q.N) cost[at] = c + penalty;
}

}  // namespace

hipError_t launch_penalty(const PenaltyLaunch &L, const uint64_t *hashes, const uint64_t *bad,
                          int64_t n_bad, float penalty, float *cost, hipStream_t st)
{
    if (L.nq == 0) return hipSuccess;
    if (L.blocks == 0 || n_bad == 0) return hipSuccess;
    const int64_t step = (n_bad + SAMPLES - 1) / SAMPLES;
    hipLaunchKernelGGL(k_penalty, dim3(L.blocks), dim3(PENALTY_THREADS), 0, st, L, hashes, bad,
                       n_bad, step, penalty, cost);
    return hipGetLastError();
}

}  // namespace cm
