// topk_dev.h -- device code of per-query beam selection (Sec. 4: the search
// keeps the k best candidate states; Sec. 4.4: evaluated candidates are added
// to the beam), shared by the selection kernel and the tail of the
// persistent step kernel.
//
// Ranking key: 64 bits = (order-preserving image of the float32 cost) << 32 |
// candidate index.  -0 is mapped to +0 and every NaN to one quiet NaN that
// ranks after +inf, so the unsigned order of the keys is exactly "ascending
// cost, ties by lower index, NaN last", and keys are unique.
//
// One workgroup of NT threads selects over a tile of up to NT * PER
// candidates (element e = j*NT + thread):
//   1. every lane takes the minimum of its keys' cost halves; each wave whose
//      lanes all hold a candidate finds the m-th smallest of its 64 minima,
//      m = ceil(k / waves), by m wave minima; the largest of these is a
//      threshold with at least k keys at or under it, and for unordered costs
//      a few times k (tiles of at most max(128, 2k) candidates skip this: all
//      pass; in a larger one the full waves hold at least k keys);
//   2. keys under it are compacted into LDS, one atomic per wave;
//   3. each compacted key is placed by counting the compacted keys below it
//      (up to 8 threads share a key's count); keys placed at rank < k are the
//      k best, already in order.
// If many more than k keys pass (equal costs, costs in an order: the waves'
// minima then say little about each other), a second threshold takes every
// wave's minima from all over the tile, indices included (spread_threshold);
// if more than FILT still pass (few threads hold all the smallest keys), a
// workgroup-wide bitwise radix search finds the exact k-th key.
// A query with several tiles has each tile's sorted k best written to a
// device list; the last tile to finish selects again over those lists.
// All of it is latency: a chain of about six barriers.  The threshold by a
// bitonic sort of one 64-bit minimum per thread (36 exchanges, three of them
// through LDS) that this replaced made the selection of 6,400 candidates
// 18.5 us in two tiles of 4,096, against 5.7 us in one of 16,384, and
// of 17 queries of up to 4,096 12.4 us against 6.5 us.  In random order, that is:
// the sort gave every order the same time.  With the first threshold alone,
// equal or sorted costs of one query of 4,096 took 24 to 36 us a call at k = 32
// (the sort 7.6), of 100,000 34 to 43 (15.2), of 4,096 at k = 256 27 to 37
// (10.7); with the second one 7.6, 17 and 14, and random ones, which do not come
// to it, 7.5, 11.4 and 12.3 (8.8, 18.6 and 59.6).
#pragma once

#include "cm_internal.h"

namespace cm {
namespace topk {

constexpr uint64_t SENT = ~0ull;      // empty slot: ranks after every real key
constexpr uint32_t EMPTY = ~0u;       // its cost half
constexpr int FILT = 1024;            // compacted keys placed by counting
constexpr int CHEAP = 256;            // more than k + this are worth a better threshold
constexpr int ALL_PASS = 128;         // tiles of at most this many keys skip the threshold
static_assert(FILT >= 2 * CM_MAX_K && ALL_PASS <= CHEAP && CM_MAX_K <= CHEAP,
              "a merge round makes progress, all may pass without a threshold");

// Order-preserving image of a cost.
__device__ inline uint32_t cost_order(float c)
{
    uint32_t b = __float_as_uint(c);
    const uint32_t mag = b & 0x7fffffffu;
    if (mag == 0) b = 0;                          // -0 -> +0
    else if (mag > 0x7f800000u) b = 0x7fc00000u;  // any NaN -> one quiet NaN
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

__device__ inline uint64_t make_key(uint32_t order, uint32_t idx)
{
    return ((uint64_t)order << 32) | idx;
}

template <int NT>
struct TopkShared {
    static constexpr int WAVES = NT / 64;
    static_assert(NT >= CM_MAX_K, "one thread per output slot");
    uint64_t filt[FILT];
    uint64_t best[CM_MAX_K];
    uint32_t thr[WAVES];
    uint32_t nfilt;
    uint32_t cnt[2][WAVES];
    uint32_t red_and[WAVES], red_or[WAVES];
};

__device__ inline uint32_t wave_count(bool p) { return (uint32_t)__popcll(__ballot(p)); }

// The thread's index, opaque to the compiler: values derived from it (lane
// masks, partner addresses) are recomputed where they are used
// instead of being hoisted out of the persistent kernel's task loop, where
// they would stay live through the evaluation and spill.
__device__ inline int sel_tid()
{
    int t = (int)threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// ---------------------------------------------------------------- waves
template <int CTRL>
__device__ inline uint32_t dpp(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
}
constexpr int QUAD_XOR1 = 0xB1, QUAD_XOR2 = 0x4E, HALF_MIRROR = 0x141, MIRROR = 0x140;

// Minimum over the wave, in every lane: pairs, quads (lane ^ 1, ^ 2), then
// mirrored halves and rows of 16 lanes, then rows.
__device__ inline uint32_t wave_min(uint32_t v)
{
    v = min(v, dpp<QUAD_XOR1>(v));
    v = min(v, dpp<QUAD_XOR2>(v));
    v = min(v, dpp<HALF_MIRROR>(v));
    v = min(v, dpp<MIRROR>(v));
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = min((uint32_t)r[0], (uint32_t)r[1]);
    const auto h = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return min((uint32_t)h[0], (uint32_t)h[1]);
}

// Room for this wave's n keys in the compacted set (n uniform): its first slot.
template <int NT>
__device__ inline uint32_t reserve(TopkShared<NT> &sh, uint32_t n, int lane)
{
    uint32_t base = 0;
    if (lane == 0 && n) base = atomicAdd(&sh.nfilt, n);
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
}

__device__ inline uint32_t lanes_below(uint64_t mask)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// ---------------------------------------------------------------- workgroup
template <int NT>
__device__ inline uint32_t block_sum(uint32_t wave_value, TopkShared<NT> &sh, int &buf)
{
    const int tid = sel_tid();
    const int w = tid >> 6;
    if ((tid & 63) == 0) sh.cnt[buf][w] = wave_value;
    __syncthreads();
    uint32_t tot = 0;
#pragma unroll
    for (int j = 0; j < NT / 64; ++j) tot += sh.cnt[buf][j];
    buf ^= 1;
    return tot;
}

template <int NT, int PER>
__device__ uint32_t block_radix(const uint32_t (&val)[PER], const bool (&sel)[PER],
                                uint32_t &rank, TopkShared<NT> &sh, int &buf)
{
    uint32_t a = 0xffffffffu, o = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j)
        if (sel[j]) {
            a &= val[j];
            o |= val[j];
        }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
        a &= (uint32_t)__shfl_xor((int)a, d);
        o |= (uint32_t)__shfl_xor((int)o, d);
    }
    const int tid = sel_tid();
    const int w = tid >> 6;
    if ((tid & 63) == 0) {
        sh.red_and[w] = a;
        sh.red_or[w] = o;
    }
    __syncthreads();
    a = 0xffffffffu;
    o = 0;
#pragma unroll
    for (int j = 0; j < NT / 64; ++j) {
        a &= sh.red_and[j];
        o |= sh.red_or[j];
    }
    __syncthreads();
    const uint32_t diff = a ^ o;
    if (diff == 0) return a;
    const int hb = 31 - __clz(diff);
    uint32_t prefix = a & ~((2u << hb) - 1u);
    for (int b = hb; b >= 0; --b) {
        const uint32_t hmask = ~((2u << b) - 1u);
        uint32_t c = 0;
#pragma unroll
        for (int j = 0; j < PER; ++j)
            c += wave_count(sel[j] && ((val[j] ^ prefix) & hmask) == 0 && !((val[j] >> b) & 1u));
        const uint32_t cnt = block_sum(c, sh, buf);
        if (cnt < rank) {
            rank -= cnt;
            prefix |= 1u << b;
        }
    }
    return prefix;
}

// The k-th smallest key of the workgroup's registers (at least k real ones).
template <int NT, int PER, class Index>
__device__ uint64_t block_threshold(const uint32_t (&ord)[PER], Index index, int k,
                                    TopkShared<NT> &sh)
{
    int buf = 0;
    uint32_t rank = (uint32_t)k, idx[PER];
    bool sel[PER], eq[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        sel[j] = ord[j] != EMPTY;
        idx[j] = (uint32_t)index(j);
    }
    const uint32_t thi = block_radix<NT, PER>(ord, sel, rank, sh, buf);
    uint32_t c = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        eq[j] = sel[j] && ord[j] == thi;
        c += wave_count(eq[j]);
    }
    const uint32_t neq = block_sum(c, sh, buf);
    const uint32_t tlo = neq > rank ? block_radix<NT, PER>(idx, eq, rank, sh, buf) : 0xffffffffu;
    return ((uint64_t)thi << 32) | tlo;
}

// The compacted keys filt[0, n) in order: the min(n, k) smallest into
// sh.best, by counting.  Ends with a barrier.
template <int NT>
__device__ int place(int n, int k, TopkShared<NT> &sh)
{
    const int t = sel_tid();
    int lper = 0;  // 1, 2, 4 or 8 neighbouring threads share a key's count
    while (lper < 3 && (n << (lper + 1)) <= NT) ++lper;
    const int per = 1 << lper, sub = t & (per - 1);
    for (int base = 0; base < n; base += NT >> lper) {
        const int e = base + (t >> lper);
        const uint64_t mine = e < n ? sh.filt[e] : SENT;
        uint32_t r = 0;
#pragma unroll 4
        for (int j = sub; j < n; j += per) r += sh.filt[j] < mine;
        if (lper > 0) r += dpp<QUAD_XOR1>(r);
        if (lper > 1) r += dpp<QUAD_XOR2>(r);
        if (lper > 2) r += dpp<HALF_MIRROR>(r);
        if (sub == 0 && e < n && r < (uint32_t)k) sh.best[r] = mine;
    }
    __syncthreads();
    return min(n, k);
}

// The keys for which passes(cost order, j), compacted into sh.filt as far as
// they fit (nfilt is 0 and visible): their number.  Ends with a barrier.
template <int NT, int PER, class Index, class Passes>
__device__ __forceinline__ int compact(const uint32_t (&ord)[PER], Index index, int nvalid,
                                       Passes passes, TopkShared<NT> &sh)
{
    const int lane = sel_tid() & 63;
    uint32_t mine = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        if (j * NT >= nvalid) break;
        mine += wave_count(passes(ord[j], j));
    }
    uint32_t base = reserve(sh, mine, lane);
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        if (j * NT >= nvalid) break;
        const bool p = passes(ord[j], j);
        const uint64_t mask = __ballot(p);
        const uint32_t pos = base + lanes_below(mask);
        if (p && pos < FILT) sh.filt[pos] = make_key(ord[j], index(j));
        base += (uint32_t)__popcll(mask);
    }
    __syncthreads();
    return (int)sh.nfilt;
}

// A threshold with at least k keys at or under it, like the one of
// tile_select, but for costs that are equal or in an order: every thread's
// smallest key, index included, goes through LDS so that each wave holds every
// WAVES-th of them, and the m smallest of a wave's 64 are taken one by one.
// At most PER times as many keys pass as threads' minima do, which are k and a
// few.  (More than k threads hold a key.)  Leaves nfilt 0.
template <int NT, int PER, class Index>
__device__ uint64_t spread_threshold(const uint32_t (&ord)[PER], Index index, int k,
                                     TopkShared<NT> &sh)
{
    constexpr int W = NT / 64;
    static_assert(NT <= FILT && W <= CM_MAX_K, "scratch in the lists");
    const int t = sel_tid();
    const int lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    // spreads the strided reads over the banks
    auto at = [](int e) { return e ^ ((e >> 4) & 15); };
    uint64_t key = make_key(ord[0], (uint32_t)index(0));
#pragma unroll
    for (int j = 1; j < PER; ++j)  // of equal costs the first has the lowest index
        if (ord[j] < (uint32_t)(key >> 32)) key = make_key(ord[j], (uint32_t)index(j));
    __syncthreads();  // the number of keys that passed is read
    if (t == 0) sh.nfilt = 0;
    sh.filt[at(t)] = key;
    __syncthreads();
    key = sh.filt[at(lane * W + wave)];
    uint64_t w = 0;
    for (int i = (k + W - 1) / W; i > 0; --i) {
        const uint32_t hi = wave_min((uint32_t)(key >> 32));
        const uint32_t lo = wave_min((uint32_t)(key >> 32) == hi ? (uint32_t)key : ~0u);
        w = make_key(hi, lo);
        if (key == w) key = SENT;
    }
    if (lane == 0) sh.best[wave] = w;
    __syncthreads();
    uint64_t T = 0;
#pragma unroll
    for (int j = 0; j < W; ++j) T = max(T, sh.best[j]);
    return T;
}

// Select the k smallest keys of the workgroup into sh.best, ascending:
// element j*NT + thread has cost order ord[j] and candidate index(j); the
// nvalid first elements are real, the others EMPTY.  Returns min(k, nvalid).
template <int NT, int PER, class Index>
__device__ int tile_select(const uint32_t (&ord)[PER], Index index, int nvalid, int k,
                           TopkShared<NT> &sh)
{
    const int t = sel_tid();
    const int lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    if (t == 0) sh.nfilt = 0;
    uint32_t T = EMPTY - 1;  // every real key
    if (nvalid > max(ALL_PASS, 2 * k)) {
        const int full = min(NT, nvalid) / 64;  // waves that hold a key in every lane
        uint32_t w = 0;
        if (wave < full) {
            uint32_t m = ord[0];
#pragma unroll
            for (int j = 1; j < PER; ++j) m = min(m, ord[j]);
            for (int i = (k + full - 1) / full; i > 0; --i) {  // at most 64
                w = wave_min(m);
                if (m == w) m = EMPTY;
            }
        }
        if (lane == 0) sh.thr[wave] = w;
        __syncthreads();
        T = 0;
#pragma unroll
        for (int j = 0; j < NT / 64; ++j) T = max(T, sh.thr[j]);
        // 64 minima with repeats run out before m of them are taken
        T = min(T, EMPTY - 1);
    } else {
        __syncthreads();
    }
    int n = compact(ord, index, nvalid, [&](uint32_t o, int) { return o <= T; }, sh);
    // random costs come to 1.7 k and 100 keys, sorted ones to 1,000; up to 512 are
    // counted by two threads or more each
    if (n > CHEAP + k) {
        const uint64_t T2 = spread_threshold(ord, index, k, sh);
        n = compact(ord, index, nvalid,
                    [&](uint32_t o, int j) { return make_key(o, (uint32_t)index(j)) <= T2; }, sh);
    }
    if (n > FILT) {
        const uint64_t T2 = block_threshold<NT, PER>(ord, index, k, sh);
        __syncthreads();
        if (t == 0) sh.nfilt = 0;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const uint64_t key = make_key(ord[j], index(j));
            if (ord[j] != EMPTY && key <= T2) sh.filt[atomicAdd(&sh.nfilt, 1u)] = key;
        }
        __syncthreads();
        n = k;  // keys are unique: exactly k are at or under the k-th
    }
    return place<NT>(n, k, sh);
}

// This workgroup's tile list for the merge: k sorted keys (SENT past nbest),
// made visible to the merging workgroup.
template <int NT>
__device__ inline void publish_list(const TopkShared<NT> &sh, int nbest, int k, uint64_t *dst)
{
    const int t = sel_tid();
    if (t < k) store_shared(dst + t, t < nbest ? sh.best[t] : SENT);
    wait_stores();
}

// Select again over `ntiles` sorted per-tile lists of k keys at src (every
// list but the last is full; the last holds min(k, N - (ntiles - 1) * tile)
// real keys; written by other workgroups with store_shared) into sh.best.
// Returns min(k, N).
template <int NT, int PER>
__device__ int merge_lists(const uint64_t *src, int ntiles, int tile, int N, int k,
                           TopkShared<NT> &sh)
{
    const int t = sel_tid();
    const int total = (ntiles - 1) * k + min(k, N - (ntiles - 1) * tile);
    int nbest = 0;
    for (int base = 0; base < total;) {
        // the best so far, then as many new keys as fit
        const int nnew = min(total - base, NT * PER - nbest);
        uint32_t ord[PER], idx[PER];
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int e = j * NT + t;
            uint64_t key = SENT;
            if (e < nbest) key = sh.best[e];
            else if (e < nbest + nnew) key = load_shared(src + base + e - nbest);
            ord[j] = (uint32_t)(key >> 32);
            idx[j] = (uint32_t)key;
        }
        __syncthreads();  // best is read
        nbest = tile_select<NT, PER>(ord, [&](int j) { return idx[j]; }, nbest + nnew, k, sh);
        base += nnew;
    }
    return nbest;
}

// Cost orders of tile `beg`, beg + 1, ... of a query's costs c[0..N)
// (kShared: written by other workgroups of the same launch).
template <int NT, int PER, bool kShared>
__device__ inline void tile_orders(const float *c, int N, int beg, uint32_t (&ord)[PER],
                                   int &nvalid)
{
    nvalid = max(0, min(NT * PER, N - beg));
    float v[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int e = j * NT + sel_tid();
        v[j] = 0.f;
        if (e < nvalid) v[j] = kShared ? load_shared(c + beg + e) : c[beg + e];
    }
#pragma unroll
    for (int j = 0; j < PER; ++j)
        ord[j] = j * NT + sel_tid() < nvalid ? cost_order(v[j]) : EMPTY;
}

// Write the beam: idx[j] = query-local index, val[j] = its cost bit for bit,
// padded with (-1, +inf) past nbest.  The cost is its key's, except a zero or
// NaN, whose bits the key does not keep.
template <int NT, bool kShared>
__device__ inline void write_beam(const TopkShared<NT> &sh, int nbest, int k, const float *c,
                                  int32_t *idx, float *val)
{
    const int t = sel_tid();
    if (t < k) {
        int32_t id = -1;
        float v = __builtin_inff();
        if (t < nbest) {
            const uint64_t key = sh.best[t];
            const uint32_t o = (uint32_t)(key >> 32);
            id = (int32_t)(uint32_t)key;
            v = __uint_as_float((o & 0x80000000u) ? o & 0x7fffffffu : ~o);
            if (v == 0.f || v != v) v = kShared ? load_shared(c + id) : c[id];
        }
        idx[t] = id;
        val[t] = v;
    }
}

}  // namespace topk
}  // namespace cm
