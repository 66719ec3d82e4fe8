// k_topk.hip -- per-query beam selection kernel (Sec. 4, Sec. 4.4): one
// workgroup per tile of a query's candidates, query descriptors passed by
// value; the selection itself is in topk_dev.h.
#include "topk_dev.h"

namespace cm {
namespace {

using namespace topk;

// 1,024 threads for every size: a larger workgroup reads more candidates in
// one tile, which saves lists and their merge, and places more keys at once.
// k = 32: 3.8 us at 64 candidates, 4.4 us at 1,024, 5.0 us at 4,096, 7.9 us at
// 16,384 and 10.7 us at 40,000 (three tiles); 256 threads in tiles of 4,096
// took 3.5, 4.6, 5.9, 9.6 and 22 us.
constexpr int NT = 1024;

__global__ __launch_bounds__(NT) void k_topk(TopkLaunch L, const float *__restrict__ cost,
                                             uint64_t *__restrict__ tpart,
                                             int32_t *__restrict__ tcnt,
                                             int32_t *__restrict__ idx_out,
                                             float *__restrict__ val_out)
{
    constexpr int TILE = TOPK_CALL_TILE, PER = TILE / NT;
    __shared__ TopkShared<NT> sh;
    __shared__ int last;
    const int t = threadIdx.x;
    const int q = query_at(L.nq, blockIdx.x, [&](int j) { return L.q[j].tile0; });
    const TopkQ &Q = L.q[q];
    const int tile = (int)blockIdx.x - Q.tile0;
    const int k = L.k;
    const float *c = cost + Q.cost_off;

    uint32_t ord[PER];
    int nvalid;
    tile_orders<NT, PER, false>(c, Q.N, tile * TILE, ord, nvalid);
    int nbest = tile_select<NT, PER>(
        ord, [&](int j) { return (uint32_t)(tile * TILE + j * NT + t); }, nvalid, k, sh);

    if (Q.ntiles > 1) {
        uint64_t *lists = tpart + (int64_t)Q.tile0 * k;
        publish_list<NT>(sh, nbest, k, lists + (int64_t)tile * k);
        __syncthreads();
        if (t == 0) last = atomicAdd(&tcnt[q], 1) == Q.ntiles - 1;
        __syncthreads();
        if (!last) return;
        nbest = merge_lists<NT, 4>(lists, Q.ntiles, TILE, Q.N, k, sh);
        if (t == 0) atomicExch(&tcnt[q], 0);
    }
    write_beam<NT, false>(sh, nbest, k, c, idx_out + (int64_t)Q.out_q * k,
                          val_out + (int64_t)Q.out_q * k);
}

}  // namespace

hipError_t launch_topk(const TopkLaunch &L, const float *cost, uint64_t *tpart, int32_t *tcnt,
                       int32_t *idx_out, float *val_out, hipStream_t st)
{
    if (L.ntasks == 0) return hipSuccess;
    hipLaunchKernelGGL(k_topk, dim3(L.ntasks), dim3(NT), 0, st, L, cost, tpart, tcnt,
                       idx_out, val_out);
    return hipGetLastError();
}

}  // namespace cm
