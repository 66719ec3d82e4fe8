// k_step.hip -- the persistent step kernel: bf16 or FP8 evaluation of many
// ragged queries (Sec. 5.2) and each query's beam selection (Sec. 4, Sec. 4.4)
// in one launch.
//
// A grid of workgroups (8 waves each) whose size the batch may only reduce
// takes tasks from a device-wide queue: a workgroup's first task is its own
// number, and each further one costs an atomic add when the task before it
// ends.  A task is `gpt` consecutive row-tile groups of one query, evaluated
// exactly as the per-call kernels do (eval_bf16.h, eval_fp8.h), so the costs
// are bit-identical to them.
// Tasks never straddle a selection tile of TOPK_TILE candidates; the
// workgroup whose task completes a tile (an arrival count per tile) selects
// that tile's k best, and for a query of several tiles the last tile to
// finish merges their lists.  A query's selection therefore runs while other queries are
// still being evaluated.  All control words are left at zero when the
// kernel ends, so the next launch needs no clearing.
#include <algorithm>
#include <cstring>

#include "eval_bf16.h"
#include "eval_fp8.h"
#include "topk_dev.h"

namespace cm {
namespace {

using namespace bf16eval;
using namespace topk;

constexpr int NT = EVAL_WAVES * 64;

// Selection of tile `tile` of query q after the last of its tasks has
// arrived, and for a query of several tiles, the merge by the last tile.
__device__ __forceinline__ void select_tile(const StepQ &D, int q, int tile, int k, uint32_t *qcnt,
                            uint64_t *tpart, TopkShared<NT> &tsh, int &s_query_last)
{
    const int tid = threadIdx.x;
    constexpr int PER = TOPK_TILE / NT;
    uint32_t ord[PER];
    int nvalid;
    tile_orders<NT, PER, true>(D.cost, D.N, tile * TOPK_TILE, ord, nvalid);
    int nbest = tile_select<NT, PER>(
        ord, [&](int j) { return (uint32_t)(tile * TOPK_TILE + j * NT + sel_tid()); }, nvalid, k,
        tsh);
    bool write = true;
    if (D.ntiles > 1) {
        publish_list<NT>(tsh, nbest, k, tpart + (int64_t)(D.tile0 + tile) * k);
        __syncthreads();
        if (tid == 0) s_query_last = atomicAdd(&qcnt[q], 1u) == (uint32_t)(D.ntiles - 1);
        __syncthreads();
        write = s_query_last;
        if (write) {
            if (tid == 0) atomicExch(&qcnt[q], 0u);
            nbest = merge_lists<NT, PER>(tpart + (int64_t)D.tile0 * k, D.ntiles, TOPK_TILE, D.N, k, tsh);
        }
    }
    if (write) {
        write_beam<NT, true>(tsh, nbest, k, D.cost, D.idx, D.val);
        if (D.sidx) write_beam<NT, true>(tsh, nbest, k, D.cost, D.sidx, D.sval);
    }
}

// One task's evaluation: gpt row-tile groups of one query.
template <bool kSpread>
__device__ __forceinline__ void eval_task(const StepQ &D, int tq, int gpt, int wave, int lane,
                                          const Bf16Pack *__restrict__ pk, const Pairs &kp,
                                          const uint32_t *tab, GroupShared &gsh,
                                          const HoistPack *hp)
{
    QueryView Q;
    Q.x = static_cast<const uint16_t *>(D.x);
    Q.t = D.t;
    Q.u = D.u;
    Q.cost = D.cost;
    Q.S = D.S;
    Q.N = D.N;
    Q.P = stage_parts(D.S);
    const int group_rows = TILE_ROWS * (EVAL_WAVES / D.parts);
    if (hp) {
        Q.pipe = D.pipe;
        Q.hoist = hp;
    }
    const Weights w = load_weights(pk, lane);
    for (int g = 0; g < gpt; ++g) {
        const int group = tq * gpt + g;
        if (group * group_rows >= Q.N) break;  // uniform
        if (kSpread && Q.P < D.parts)
            eval_group<true, false, false, true>(Q, group, wave, lane, w, kp, tab, gsh);
        else
            eval_group<true>(Q, group, wave, lane, w, kp, tab, gsh);
        __syncthreads();  // the group's LDS is reused by the next group
    }
}

template <bool kSpread>
__device__ __forceinline__ void eval_task(const StepQ &D, int tq, int gpt, int wave, int lane,
                                          const Fp8Pack *__restrict__ pk, const Pairs &,
                                          const uint32_t *, GroupShared &gsh,
                                          const HoistPack *hp)
{
    fp8eval::QueryView8 Q;
    Q.x = static_cast<const uint8_t *>(D.x);
    Q.t = D.t;
    Q.u = D.u;
    Q.cost = D.cost;
    Q.S = D.S;
    Q.N = D.N;
    Q.P = stage_parts(D.S);
    const int group_rows = TILE_ROWS * (EVAL_WAVES / D.parts);
    if (hp) {
        Q.pipe = D.pipe;
        Q.hoist = hp;
        Q.uh = pk->uh;
    }
    const fp8eval::Weights8 w = fp8eval::load_weights8(pk, lane);
    for (int g = 0; g < gpt; ++g) {
        const int group = tq * gpt + g;
        if (group * group_rows >= Q.N) break;  // uniform
        if (kSpread && Q.P < D.parts)
            fp8eval::eval_group8<true, false, false, true>(Q, group, wave, lane, w, gsh);
        else
            fp8eval::eval_group8<true>(Q, group, wave, lane, w, gsh);
        __syncthreads();
    }
}

// LDS table of the log transform: the bf16 evaluator's only.
template <class Pack> struct LogTable { static constexpr int n = 1; };
template <> struct LogTable<Bf16Pack> { static constexpr int n = LOG_N; };

// The evaluation's and the selection's LDS are never in use at the same time
// (a workgroup-wide barrier separates every switch between them).
union StepShared {
    GroupShared g;
    TopkShared<NT> t;
};

template <bool kSpread, bool kOwn = false, class Pack>
__device__ __forceinline__ void step_body(const StepHead *__restrict__ h,
                                          const StepQ *__restrict__ qs, uint32_t *ctl,
                                          uint64_t *tpart, const Pack *__restrict__ pk,
                                          const HoistPack *__restrict__ hp = nullptr)
{
    __shared__ StepShared ssh;
    __shared__ uint32_t tab[LogTable<Pack>::n];
    GroupShared &gsh = ssh.g;
    TopkShared<NT> &tsh = ssh.t;
    __shared__ int32_t task0[STEP_MAX_QUERIES];
    __shared__ int s_next, s_tail, s_query_last;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nq = h->nq, ntasks = h->ntasks, k = h->k, gpt = h->gpt;
    uint32_t *qcnt = ctl + CTL_QCNT;
    uint32_t *tcnt = ctl + CTL_TCNT;
    unsigned long long *clk = reinterpret_cast<unsigned long long *>(ctl + CTL_CLK);

    // A workgroup's first task is its own number, and one without a task leaves
    // at once: a word that every workgroup of the grid adds to costs each of
    // them the others' additions (512 of them made an add and its return 4 to 5
    // us of a lone small query's 30).
    const int ngroups = min((int)gridDim.x, ntasks);
    int t = blockIdx.x;
    if (t >= ngroups) return;
    for (int j = tid; j < nq; j += NT) task0[j] = qs[j].task0;
    if constexpr (LogTable<Pack>::n > 1) load_table(tab, pk);
    if (tid == 0) atomicMin(&clk[0], (unsigned long long)__builtin_amdgcn_s_memrealtime());
    const Pairs kp = make_pairs();
    __syncthreads();
    while (t < ntasks) {
        // the query of task t: the last q with task0[q] <= t
        int lo = 0, hi = nq - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (task0[mid] <= t) lo = mid;
            else hi = mid - 1;
        }
        const int q = __builtin_amdgcn_readfirstlane(lo);
        const StepQ &D = qs[q];
        const int tq = t - D.task0;  // task within the query
        const int group_rows = TILE_ROWS * (EVAL_WAVES / D.parts);
        eval_task<kSpread>(D, tq, gpt, wave, lane, pk, kp, tab, gsh, kOwn ? hp : nullptr);
        // this task's costs (coherent stores) have completed before it counts
        // itself at its selection tile; the next task is taken only now, so
        // that the queue hands work to whichever workgroup is free first
        const int tpt = TOPK_TILE / (group_rows * gpt);  // tasks per tile
        const int tile = tq / tpt;
        wait_stores();
        __syncthreads();
        if (tid == 0) {
            const uint32_t need = (uint32_t)min(tpt, D.ntasks - tile * tpt);
            // the queue past the first tasks, while it holds any; a tile of one
            // task has no other workgroup to wait for
            uint32_t next = (uint32_t)ntasks, arrived = 0;
            if (ntasks > ngroups) next = (uint32_t)ngroups + atomicAdd(&ctl[CTL_NEXT], 1u);
            if (need > 1) arrived = atomicAdd(&tcnt[D.tile0 + tile], 1u);
            s_next = (int)next;
            s_tail = arrived == need - 1;
            if (need > 1 && arrived == need - 1) atomicExch(&tcnt[D.tile0 + tile], 0u);
        }
        __syncthreads();
        if (s_tail) {
            select_tile(D, q, tile, k, qcnt, tpart, tsh, s_query_last);
        }
        t = s_next;
        __syncthreads();  // s_next and s_tail are read; the selection's LDS is free
    }
    // the last workgroup to leave resets the queue for the next launch (every
    // other workgroup has made its final queue fetch before counting itself)
    // and publishes the launch's clock pair: its own leaving is the launch's
    // end, so that no workgroup waits for a maximum in memory
    if (tid == 0) {
        if (atomicAdd(&ctl[CTL_DONE], 1u) == (uint32_t)ngroups - 1) {
            unsigned long long *out = reinterpret_cast<unsigned long long *>(ctl + CTL_CLKOUT);
            const unsigned long long c0 = atomicExch(&clk[0], ~0ull);
            const unsigned long long c1 = __builtin_amdgcn_s_memrealtime();
            store_shared(&out[0], c0);
            store_shared(&out[1], c1);
            if (h->clk_out) {
                __hip_atomic_store(&h->clk_out[0], (uint64_t)c0, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_SYSTEM);
                __hip_atomic_store(&h->clk_out[1], (uint64_t)c1, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_SYSTEM);
            }
            atomicExch(&ctl[CTL_NEXT], 0u);
            atomicExch(&ctl[CTL_DONE], 0u);
        }
    }
}

__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_step_bf16(
    const StepHead *__restrict__ h, const StepQ *__restrict__ qs, uint32_t *ctl,
    uint64_t *tpart, const Bf16Pack *__restrict__ pk)
{
    step_body<false>(h, qs, ctl, tpart, pk);
}

__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_step_fp8(
    const StepHead *__restrict__ h, const StepQ *__restrict__ qs, uint32_t *ctl,
    uint64_t *tpart, const Fp8Pack *__restrict__ pk)
{
    step_body<false>(h, qs, ctl, tpart, pk);
}

__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4, 4))) void
k_step_bf16_value(StepArgs a, uint32_t *ctl, uint64_t *tpart, const Bf16Pack *__restrict__ pk)
{
    step_body<false>(&a.h, a.q, ctl, tpart, pk);
}

// A spread step has at most one workgroup per compute unit, so its waves may
// hold twice the registers where they need them.
template <bool kOwn>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2, 2))) void
k_step_bf16_spread(StepArgs a, uint32_t *ctl, uint64_t *tpart, const Bf16Pack *__restrict__ pk,
                   const HoistPack *__restrict__ hp)
{
    step_body<true, kOwn>(&a.h, a.q, ctl, tpart, pk, hp);
}

__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4, 4))) void
k_step_fp8_value(StepArgs a, uint32_t *ctl, uint64_t *tpart, const Fp8Pack *__restrict__ pk)
{
    step_body<false>(&a.h, a.q, ctl, tpart, pk);
}

template <bool kOwn>
__global__ __launch_bounds__(NT)
__attribute__((amdgpu_waves_per_eu(kOwn ? 2 : 4, kOwn ? 2 : 4))) void
k_step_fp8_spread(StepArgs a, uint32_t *ctl, uint64_t *tpart, const Fp8Pack *__restrict__ pk,
                  const HoistPack *__restrict__ hp)
{
    step_body<true, kOwn>(&a.h, a.q, ctl, tpart, pk, hp);
}

// Words of host memory as arguments (descriptors of a recorded call: a replay
// takes its arguments from the graph).
struct PutArgs {
    uint64_t w[NT - 64];
};
static_assert(sizeof(PutArgs) <= 4096 - 64, "kernel arguments");

__global__ __launch_bounds__(NT) void k_put(PutArgs a, int n, uint64_t *__restrict__ dst)
{
    if ((int)threadIdx.x < n) dst[threadIdx.x] = a.w[threadIdx.x];
}

}  // namespace

hipError_t launch_put(const void *src, size_t bytes, void *dst, hipStream_t st)
{
    constexpr size_t PART = sizeof(PutArgs);
    for (size_t at = 0; at < bytes; at += PART) {
        PutArgs a{};
        const size_t n = std::min(PART, bytes - at);
        std::memcpy(a.w, static_cast<const unsigned char *>(src) + at, n);
        hipLaunchKernelGGL(k_put, dim3(1), dim3(NT), 0, st, a, (int)(n / sizeof(uint64_t)),
                           reinterpret_cast<uint64_t *>(static_cast<unsigned char *>(dst) + at));
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_step(const StepHead *h, const StepQ *qs, uint32_t *ctl, uint64_t *tpart,
                       const Model &m, cm_precision prec, int grid, hipStream_t st)
{
    if (prec == CM_FP8)
        hipLaunchKernelGGL(k_step_fp8, dim3(grid), dim3(NT), 0, st, h, qs, ctl, tpart, m.d_fp8);
    else
        hipLaunchKernelGGL(k_step_bf16, dim3(grid), dim3(NT), 0, st, h, qs, ctl, tpart,
                           &m.d->bf16);
    return hipGetLastError();
}

hipError_t launch_step(const StepArgs &a, uint32_t *ctl, uint64_t *tpart, const Model &m,
                       cm_precision prec, int grid, hipStream_t st)
{
    grid = std::min(grid, a.h.ntasks);  // a workgroup without a task would only leave
    const bool own = a.h.spread == 2;
    if (prec == CM_FP8 && a.h.spread)
        hipLaunchKernelGGL(own ? k_step_fp8_spread<true> : k_step_fp8_spread<false>, dim3(grid),
                           dim3(NT), 0, st, a, ctl, tpart, m.d_fp8, &m.d->hoist);
    else if (prec == CM_FP8)
        hipLaunchKernelGGL(k_step_fp8_value, dim3(grid), dim3(NT), 0, st, a, ctl, tpart, m.d_fp8);
    else if (a.h.spread)
        hipLaunchKernelGGL(own ? k_step_bf16_spread<true> : k_step_bf16_spread<false>, dim3(grid),
                           dim3(NT), 0, st, a, ctl, tpart, &m.d->bf16, &m.d->hoist);
    else
        hipLaunchKernelGGL(k_step_bf16_value, dim3(grid), dim3(NT), 0, st, a, ctl, tpart,
                           &m.d->bf16);
    return hipGetLastError();
}

}  // namespace cm
