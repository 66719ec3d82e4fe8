// cm_sample.hip -- hierarchical sampling (Sec. 3.1, Sec. 4.4): the options of
// every query are grouped into buckets of equal structural hash, and from a
// bucket of B options max(1, ceil(log2 B)) representatives are drawn at
// random without replacement -- the members with the smallest random keys,
// key i being the high 32 bits of output i of SplitMix64 (Steele, Lea and
// Flood 2014) seeded per query, equal keys by lower index.  The
// representatives' indices are written ascending, per query.
//
// On the device, a workgroup per chunk of 1,024 options of a query:
//   1. k_s_insert counts its chunk's hashes in an LDS hash table, adds each
//      distinct one once to the query's table in memory (open addressing, two
//      slots per option, so a probe always ends), and writes every option's
//      slot.  Few buckets hold most options, so counting in LDS first keeps
//      thousands of options off one memory word;
//   2. k_s_alloc gives every bucket of two or more a list of min(B, 256)
//      entries;
//   3. k_s_list puts the bucket's candidates there: all members of a bucket
//      of at most 32, else those with keys under (2r + 16) / B of the range
//      for r representatives (keys are uniform);
//   4. k_s_rank ranks each candidate among its list.  A bucket whose list came
//      out with fewer than r entries (the binomial tail gives 6 in 10^8 for
//      2,048 members, where it is largest) or more than it holds (under 1 in
//      10^50) is gathered again under a wider bound;
//   5. k_s_write places the kept options in index order and empties the
//      slots for the next call.
// Bound by latency and scattered access: five dependent kernels of 3 to 10 us.
// 17 queries of 700,000 options in all: 37 us; the three stable radix sorts,
// two scans and eight small kernels (73 launches) that this replaced took
// 508 us.  (Chunks of 2,048: 47 us.)  The tables are read and added to at
// random, so queries whose table no cache holds lose that: one query of 2^20
// options 0.22 ms (sorts 0.57), of 2^24 3.9 ms (3.3), of 2^27 39 ms (26).
#include <algorithm>
#include <cstring>
#include <memory>
#include <new>

#include "cm_internal.h"

namespace cm {
namespace {

struct SampleQ {
    int64_t base;    // first global option of the query
    int64_t off;     // hashes, selected indices at off
    uint64_t seed;
    int32_t n;
    int32_t chunk0;  // its first chunk; every query has at least one
};

constexpr int ST = 512;                // threads per block of the chunk kernels
constexpr int PER = 2;                 // options per thread
constexpr int CHUNK = ST * PER;        // options per chunk
constexpr int MASKS = CHUNK / 64;      // 64-option masks per chunk
constexpr int LSLOTS = 2 * CHUNK;      // slots of a chunk's LDS table
constexpr int32_t MAX_GRID = 1 << 22;  // workgroups of a launch, which takes under 2^32 threads
constexpr int GROUP = 512;             // chunks whose kept options are also summed together
constexpr int AT = 1024;               // threads per block of k_s_alloc
constexpr int LIST_MAX = 256;          // entries of a bucket's list
constexpr int LIST_ALL = 32;           // buckets of at most this many list every member
typedef unsigned long long u64;
constexpr u64 NO_HASH = ~0ull;  // empty slot; the hash of this value has a slot of its own

// Table of a call: query q's slots are 2 base + q .. + 2n, the last of them
// for the hash that marks an empty slot.
struct Table {
    u64 *key;
    int32_t *cnt;   // members of the slot's bucket
    uint32_t *off;  // its list's first entry
    int32_t *fill;  // candidates that came to its list
};

__device__ inline uint64_t mix64(uint64_t z)
{
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__device__ inline uint32_t option_key(uint64_t seed, uint32_t i)
{
    return (uint32_t)(mix64(seed + ((uint64_t)i + 1) * 0x9E3779B97F4A7C15ull) >> 32);
}

__device__ inline int64_t slots_of(const SampleQ &Q, int qi) { return 2 * Q.base + qi; }

// The query of chunk c: the last one whose chunk0 is <= c (ascending from 0).
// Each load and vote of the wave leaves a 64th of the range: one for up to 64
// queries, two for 4,096.  (A walk over all of them, 64 at a time, took 10.9 ms
// for 20,000 queries of 100 options and one of 5,000, this 0.42 ms.)
__device__ inline int query_of_chunk(const SampleQ *__restrict__ q, int nq, int c)
{
    const int lane = threadIdx.x & 63;
    int at = 0, n = nq;  // it is one of at .. at + n - 1
    while (n > 1) {
        const int step = (n + 63) >> 6;
        const int64_t e = (int64_t)lane * step;
        const bool before = q[at + (int)min(e, (int64_t)n - 1)].chunk0 <= c && e < n;
        const int last = __popcll(__ballot(before)) - 1;
        at += last * step;
        n = min(step, n - last * step);
    }
    return __builtin_amdgcn_readfirstlane(at);
}

// This thread's option j of the chunk from option i0 on; past the query's end
// its last one, so that loads need no branch (a load under a branch of its own
// is waited for there, one after the other).
__device__ inline uint32_t option(const SampleQ &Q, uint32_t i0, int j)
{
    return min(i0 + j * ST + threadIdx.x, (uint32_t)Q.n - 1);
}

// Representatives of a bucket of B.
__device__ inline int drawn(int B) { return B > 2 ? 32 - __clz(B - 1) : 1; }

// Largest key of a bucket's candidates.
__device__ inline uint32_t key_bound(int B, int r)
{
    if (B <= LIST_ALL) return 0xffffffffu;
    return (uint32_t)((float)(2 * r + 16) * (4294967040.f / (float)B));
}

// Count hash h in a chunk's LDS table (key[LSLOTS], cnt[LSLOTS + 1]): its slot,
// and whether this call is the one that took it.
__device__ inline uint32_t chunk_insert(u64 *key, uint32_t *cnt, u64 h, bool &fresh)
{
    uint32_t p = LSLOTS;
    fresh = false;
    if (h != NO_HASH) {
        p = (uint32_t)(mix64(h) >> 32) & (LSLOTS - 1);
        // at most half of the slots are ever taken
        for (int tries = 0; tries < LSLOTS; ++tries) {
            u64 k = *(volatile u64 *)&key[p];
            if (k == NO_HASH) {
                k = atomicCAS(&key[p], NO_HASH, h);
                fresh = k == NO_HASH;
            }
            if (fresh || k == h) break;
            p = (p + 1) & (LSLOTS - 1);
        }
    }
    const uint32_t before = atomicAdd(&cnt[p], 1u);
    if (p == LSLOTS) fresh = before == 0;
    return p;
}

// Descriptors of a call of at most VALUE_Q queries, passed to the first kernel
// by value; it leaves them in memory for the others.  Larger calls copy them
// from pinned memory ahead of it, which costs a copy, the event that guards
// the pinned block and the gaps around them: 5 us a call.  A replay of a
// recorded copy would read the block when it is another call's, so a recorded
// call passes them as arguments whatever their number (launch_put).
constexpr int VALUE_Q = 64;
struct SampleArgs {
    SampleQ q[VALUE_Q];
};

template <bool kByValue>
__global__ __launch_bounds__(ST) void k_s_insert(SampleArgs args, SampleQ *__restrict__ dq, int nq,
                                                 int chunk0,
                                                 const uint64_t *__restrict__ hashes, Table tb,
                                                 uint32_t *__restrict__ slot, uint32_t *arena)
{
    const SampleQ *q = kByValue ? args.q : dq;
    __shared__ u64 key[LSLOTS];
    __shared__ uint32_t cnt[LSLOTS + 1];  // members, then the slot in the query's table
    __shared__ uint16_t used[CHUNK + 1];
    __shared__ uint32_t nused;
    const int t = threadIdx.x, c = chunk0 + (int)blockIdx.x;
    if (c == 0 && t == 0) *arena = 0;
    if (kByValue && c == 0 && t < nq) dq[t] = args.q[t];
    const int qi = query_of_chunk(q, nq, c);
    const SampleQ Q = q[qi];
    const uint32_t i0 = (uint32_t)(c - Q.chunk0) * CHUNK;
    if (Q.n == 0) return;  // uniform: the query's one chunk is empty
    uint64_t h[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) h[j] = hashes[Q.off + option(Q, i0, j)];
    for (int p = t; p < LSLOTS; p += ST) {
        key[p] = NO_HASH;
        cnt[p] = 0;
    }
    if (t == 0) {
        cnt[LSLOTS] = 0;
        nused = 0;
    }
    __syncthreads();
    uint32_t at[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        at[j] = 0;
        if (i0 + j * ST + t >= (uint32_t)Q.n) continue;
        bool fresh;
        at[j] = chunk_insert(key, cnt, h[j], fresh);
        if (fresh) used[atomicAdd(&nused, 1u)] = (uint16_t)at[j];
    }
    __syncthreads();
    const int64_t s0 = slots_of(Q, qi);
    const uint32_t n2 = 2u * (uint32_t)Q.n;
    for (uint32_t e = t; e < nused; e += ST) {
        const uint32_t p = used[e];
        uint32_t x = n2;
        if (p < LSLOTS) {
            const u64 k = key[p];
            x = __umulhi((uint32_t)(mix64(k) >> 16), n2);
            // half of the slots are never taken; the count of tries ends the
            // walk also where calls that overlap against the rules fill them
            for (uint32_t tries = 0; tries < n2; ++tries) {
                const u64 old = atomicCAS(&tb.key[s0 + x], NO_HASH, k);
                if (old == NO_HASH || old == k) break;
                x = x + 1 == n2 ? 0 : x + 1;
            }
        }
        atomicAdd(&tb.cnt[s0 + x], (int32_t)cnt[p]);
        cnt[p] = x;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const uint32_t i = i0 + j * ST + t;
        if (i < (uint32_t)Q.n) slot[Q.base + i] = cnt[at[j]];
    }
}

// Inclusive sum over the wave's lanes up to this one.
__device__ inline uint32_t wave_scan(uint32_t v)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t o = (uint32_t)__shfl_up((int)v, d);
        if (lane >= d) v += o;
    }
    return v;
}

// Lists for four slots per thread; one addition to the arena per block.
__global__ __launch_bounds__(AT) void k_s_alloc(Table tb, int64_t slots, uint32_t *arena)
{
    __shared__ uint32_t part[AT / 64];
    __shared__ uint32_t first;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int64_t s = ((int64_t)blockIdx.x * AT + t) * 4;
    int32_t need[4] = {0, 0, 0, 0};
    if (s < slots) {  // the table's end is padded with empty slots
        const int4 c = *reinterpret_cast<const int4 *>(tb.cnt + s);
        const int32_t B[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) need[j] = B[j] > 1 ? min(B[j], LIST_MAX) : 0;
    }
    const uint32_t mine = (uint32_t)(need[0] + need[1] + need[2] + need[3]);
    const uint32_t upto = wave_scan(mine);
    if (lane == 63) part[wave] = upto;
    __syncthreads();
    uint32_t at = upto - mine, all = 0;
#pragma unroll
    for (int w = 0; w < AT / 64; ++w) {
        if (w < wave) at += part[w];
        all += part[w];
    }
    if (t == 0) first = all ? atomicAdd(arena, all) : 0;
    __syncthreads();
    at += first;
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (need[j]) {
            tb.off[s + j] = at;
            tb.fill[s + j] = 0;
            at += (uint32_t)need[j];
        }
}

__global__ __launch_bounds__(ST) void k_s_list(const SampleQ *__restrict__ q, int nq, int chunk0,
                                               Table tb,
                                               const uint32_t *__restrict__ slot,
                                               uint64_t *__restrict__ list)
{
    const int t = threadIdx.x, c = chunk0 + (int)blockIdx.x;
    const int qi = query_of_chunk(q, nq, c);
    const SampleQ Q = q[qi];
    const int64_t s0 = slots_of(Q, qi);
    const uint32_t i0 = (uint32_t)(c - Q.chunk0) * CHUNK;
    if (Q.n == 0) return;
    int64_t s[PER];
    int32_t B[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) s[j] = s0 + slot[Q.base + option(Q, i0, j)];
#pragma unroll
    for (int j = 0; j < PER; ++j) B[j] = tb.cnt[s[j]];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const uint32_t i = i0 + j * ST + t;
        if (i >= (uint32_t)Q.n || B[j] < 2) continue;
        const uint32_t k = option_key(Q.seed, i);
        if (k > key_bound(B[j], drawn(B[j]))) continue;
        const int pos = atomicAdd(&tb.fill[s[j]], 1);
        if (pos < min(B[j], LIST_MAX)) list[tb.off[s[j]] + pos] = ((uint64_t)k << 32) | i;
    }
}

constexpr int DIRECT = 8;  // lists of at most this many entries are ranked by one thread
constexpr int SHARE = 8;   // neighbouring threads that share a longer one

// Ranks a chunk's candidates in their lists.  A list is up to 256 scattered
// reads: short ones are read at once by the option's thread, the others'
// options are gathered in LDS and 8 threads read a list together, so that the
// chain of waits for memory stays at a few per round (one thread per option
// for all of them took 31 us instead of 11 us for 17 queries of 700,000
// options).
__global__ __launch_bounds__(ST) void k_s_rank(const SampleQ *__restrict__ q, int nq, int chunk0,
                                               Table tb,
                                               const uint32_t *__restrict__ slot,
                                               const uint64_t *__restrict__ list,
                                               u64 *__restrict__ mask, uint32_t *__restrict__ kept)
{
    struct Long {
        uint64_t mine;  // (key, index)
        uint32_t off;   // its list's first entry
        uint16_t f, r;  // entries (0: the list does not hold; off is then the slot), kept ones
    };
    __shared__ Long todo[CHUNK];
    __shared__ u64 ms[MASKS];
    __shared__ uint64_t found[CHUNK];
    __shared__ uint32_t ntodo, nfound, odd;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int c = chunk0 + (int)blockIdx.x;
    const int qi = query_of_chunk(q, nq, c);
    const SampleQ Q = q[qi];
    const int64_t s0 = slots_of(Q, qi);
    const uint32_t i0 = (uint32_t)(c - Q.chunk0) * CHUNK;
    if (Q.n == 0) {
        if (t < MASKS) mask[(int64_t)c * MASKS + t] = 0;
        if (t == 0) kept[c] = 0;
        return;
    }
    if (t == 0) ntodo = odd = 0;
    __syncthreads();
    int64_t s[PER];
    int32_t B[PER], f[PER];
    uint32_t off[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) s[j] = s0 + slot[Q.base + option(Q, i0, j)];
#pragma unroll
    for (int j = 0; j < PER; ++j) {  // fill and off mean something where B > 1
        B[j] = tb.cnt[s[j]];
        f[j] = tb.fill[s[j]];
        off[j] = tb.off[s[j]];
    }
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const uint32_t i = i0 + j * ST + t;
        const bool valid = i < (uint32_t)Q.n;
        bool keep = valid && B[j] == 1;
        if (valid && B[j] > 1) {
            const int r = drawn(B[j]);
            const uint32_t k = option_key(Q.seed, i);
            const uint64_t mine = ((uint64_t)k << 32) | i;
            if (f[j] < r || f[j] > min(B[j], LIST_MAX)) {
                todo[atomicAdd(&ntodo, 1u)] =
                    Long{mine, (uint32_t)(s[j] - s0), 0, (uint16_t)r};
                odd = 1;
            } else if (k <= key_bound(B[j], r)) {
                if (f[j] <= DIRECT) {
                    uint64_t v[DIRECT];
#pragma unroll
                    for (int e = 0; e < DIRECT; ++e) v[e] = list[off[j] + min(e, f[j] - 1)];
                    int rank = 0;
#pragma unroll
                    for (int e = 0; e < DIRECT; ++e) rank += e < f[j] && v[e] < mine;
                    keep = rank < r;
                } else {
                    todo[atomicAdd(&ntodo, 1u)] = Long{mine, off[j], (uint16_t)f[j], (uint16_t)r};
                }
            }
        }
        const u64 m = __ballot(keep);
        if (lane == 0) ms[j * (ST / 64) + wave] = m;
    }
    __syncthreads();
    const int n = (int)ntodo, sub = t & (SHARE - 1);
    for (int e = t / SHARE; e < n; e += ST / SHARE) {
        const Long L = todo[e];
        int rank = 0;
        for (int x = sub; x < L.f; x += 8 * SHARE) {
            uint64_t v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = list[L.off + min(x + j * SHARE, L.f - 1)];
#pragma unroll
            for (int j = 0; j < 8; ++j) rank += x + j * SHARE < L.f && v[j] < L.mine;
        }
#pragma unroll
        for (int d = 1; d < SHARE; d <<= 1) rank += __shfl_xor(rank, d);
        const uint32_t i = (uint32_t)L.mine - i0;
        if (sub == 0 && L.f > 0 && rank < L.r) atomicOr(&ms[i >> 6], 1ull << (i & 63));
    }
    __syncthreads();
    // Buckets whose list came out too short or too long, one after the other:
    // all threads gather the members under a wider bound, and rank the chunk's.
    // (A walk over the query by every option took 101 ms for one such bucket of
    // 256 in 1 M options, the whole call so 0.84 ms.)
    for (int e = 0; odd && e < n; ++e) {
        const Long L = todo[e];
        if (L.f > 0) continue;  // the same for all threads
        const int members = tb.cnt[s0 + L.off];
        const uint32_t bound = key_bound(members, L.r);
        const uint32_t wide = bound < 1u << 30 ? 4 * bound : ~0u;
        if (t == 0) nfound = 0;
        __syncthreads();
#pragma unroll 4
        for (uint32_t i = t; i < (uint32_t)Q.n; i += ST) {
            if (slot[Q.base + i] != L.off) continue;
            const uint32_t k = option_key(Q.seed, i);
            if (k > wide) continue;
            const uint32_t at = atomicAdd(&nfound, 1u);
            if (at < CHUNK) found[at] = ((uint64_t)k << 32) | i;
        }
        __syncthreads();
        const int m = (int)nfound;
        for (int x = e + t; x < n; x += ST) {
            const Long M = todo[x];
            if (M.f > 0 || M.off != L.off) continue;
            int rank = 0;
            if (m < L.r || m > CHUNK) {  // not even then: a walk by this thread
                for (uint32_t i = 0; i < (uint32_t)Q.n && rank < L.r; ++i)
                    if (slot[Q.base + i] == L.off)
                        rank += (((uint64_t)option_key(Q.seed, i) << 32) | i) < M.mine;
            } else if ((uint32_t)(M.mine >> 32) > wide) {
                rank = L.r;
            } else {
                for (int y = 0; y < m; ++y) rank += found[y] < M.mine;
            }
            const uint32_t i = (uint32_t)M.mine - i0;
            if (rank < L.r) atomicOr(&ms[i >> 6], 1ull << (i & 63));
            todo[x].f = 1;  // done; only this thread reads it before the barrier
        }
        __syncthreads();
    }
    if (wave == 0) {
        const u64 m = lane < MASKS ? ms[lane] : 0;
        if (lane < MASKS) mask[(int64_t)c * MASKS + lane] = m;
        uint32_t all = (uint32_t)__popcll(m);
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) all += (uint32_t)__shfl_xor((int)all, d);
        if (lane == 0) kept[c] = all;
    }
}

// What is kept in each GROUP of chunks, for k_s_write.
static_assert(GROUP == ST, "one chunk per thread");
__global__ __launch_bounds__(ST) void k_s_groups(const uint32_t *__restrict__ kept, int chunks,
                                                 uint32_t *__restrict__ group)
{
    __shared__ uint32_t part[ST / 64];
    const int t = threadIdx.x, e = blockIdx.x * GROUP + t;
    const uint32_t sum = wave_scan(e < chunks ? kept[e] : 0);
    if ((t & 63) == 63) part[t >> 6] = sum;
    __syncthreads();
    if (t == 0) {
        uint32_t all = 0;
#pragma unroll
        for (int w = 0; w < ST / 64; ++w) all += part[w];
        group[blockIdx.x] = all;
    }
}

__global__ __launch_bounds__(ST) void k_s_write(const SampleQ *__restrict__ q, int nq, int chunk0,
                                                int chunks, Table tb,
                                                const uint32_t *__restrict__ slot,
                                                const u64 *__restrict__ mask,
                                                const uint32_t *__restrict__ kept,
                                                const uint32_t *__restrict__ group,
                                                int32_t *__restrict__ out,
                                                int32_t *__restrict__ count)
{
    __shared__ uint32_t part[ST / 64], before[MASKS];
    __shared__ u64 ms[MASKS];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int c = chunk0 + (int)blockIdx.x;
    const int qi = query_of_chunk(q, nq, c);
    const SampleQ Q = q[qi];
    // Representatives of the query's chunks ahead of this one: by chunk up to two
    // groups, so that smaller calls need no sums of groups; past them whole
    // groups by their sums, or the work grows with the square of the options
    // (2^27 options in one query: 2^17 chunks, 8.6e9 reads).
    uint32_t sum = 0;
    int from = Q.chunk0;
    if (c - from > 2 * GROUP) {
        const int g0 = (from + GROUP - 1) / GROUP, g1 = c / GROUP;
        for (int e = from + t; e < g0 * GROUP; e += ST) sum += kept[e];
        for (int g = g0 + t; g < g1; g += ST) sum += group[g];
        from = g1 * GROUP;
    }
    for (int e = from + t; e < c; e += ST) sum += kept[e];
    sum = wave_scan(sum);
    if (lane == 63) part[wave] = sum;
    if (wave == 0) {
        const u64 m = lane < MASKS ? mask[(int64_t)c * MASKS + lane] : 0;
        const uint32_t n = (uint32_t)__popcll(m), upto = wave_scan(n);
        if (lane < MASKS) {
            ms[lane] = m;
            before[lane] = upto - n;
        }
    }
    __syncthreads();
    uint32_t base = 0;
#pragma unroll
    for (int w = 0; w < ST / 64; ++w) base += part[w];
    const int64_t s0 = slots_of(Q, qi);
    const uint32_t i0 = (uint32_t)(c - Q.chunk0) * CHUNK;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const u64 m = ms[j * (ST / 64) + wave];
        if (!((m >> lane) & 1)) continue;
        const uint32_t i = i0 + j * ST + t;
        const uint32_t pos = base + before[j * (ST / 64) + wave] +
                             (uint32_t)__popcll(m & ((1ull << lane) - 1));
        out[Q.off + pos] = (int32_t)i;
        // every bucket keeps a member, which empties its slot
        const int64_t s = s0 + slot[Q.base + i];
        tb.key[s] = NO_HASH;
        tb.cnt[s] = 0;
    }
    const bool last = c + 1 == chunks || (qi + 1 < nq && q[qi + 1].chunk0 == c + 1);
    if (last && t == 0) count[qi] = (int32_t)(base + kept[c]);
}

// Queries of at most one chunk: table, lists, ranks and the kept options'
// order all in one workgroup's LDS, one launch for the call.  20 options:
// 21.7 us with the five launches above (the host issues them), 9.6 us so; 1,024
// options 21.8 and 11.6 us.
template <bool kByValue>
__global__ __launch_bounds__(ST) void k_s_small(SampleArgs args, const SampleQ *__restrict__ dq,
                                                int query0,
                                                const uint64_t *__restrict__ hashes,
                                                int32_t *__restrict__ out,
                                                int32_t *__restrict__ count)
{
    __shared__ u64 key[LSLOTS];
    __shared__ uint32_t cnt[LSLOTS + 1], off[LSLOTS + 1], fill[LSLOTS + 1];
    __shared__ uint64_t list[CHUNK];
    __shared__ uint16_t slot[CHUNK];
    __shared__ uint32_t part[ST / 64], before[MASKS];
    __shared__ u64 ms[MASKS];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int qi = query0 + (int)blockIdx.x;
    const SampleQ Q = (kByValue ? args.q : dq)[qi];
    if (Q.n == 0) {
        if (t == 0) count[qi] = 0;
        return;
    }
    uint64_t h[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) h[j] = hashes[Q.off + option(Q, 0, j)];
    for (int p = t; p <= LSLOTS; p += ST) {
        if (p < LSLOTS) key[p] = NO_HASH;
        cnt[p] = 0;
        fill[p] = 0;
    }
    __syncthreads();
    uint32_t at[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        at[j] = 0;
        if (j * ST + t >= Q.n) continue;
        bool fresh;
        at[j] = chunk_insert(key, cnt, h[j], fresh);
        slot[j * ST + t] = (uint16_t)at[j];
    }
    __syncthreads();
    // lists: each bucket's room is its members', in slot order
    constexpr int SP = LSLOTS / ST;
    uint32_t room[SP], mine = 0;
#pragma unroll
    for (int j = 0; j < SP; ++j) mine += room[j] = cnt[t * SP + j];
    const uint32_t upto = wave_scan(mine);
    if (lane == 63) part[wave] = upto;
    __syncthreads();
    uint32_t first = upto - mine;
    for (int w = 0; w < wave; ++w) first += part[w];
#pragma unroll
    for (int j = 0; j < SP; ++j) {
        off[t * SP + j] = first;
        first += room[j];
    }
    if (t == ST - 1) off[LSLOTS] = first;
    __syncthreads();
    // candidates to their lists
    uint64_t me[PER];
    bool cand[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const uint32_t i = j * ST + t;
        const int B = (int)cnt[at[j]];
        const uint32_t k = option_key(Q.seed, i);
        me[j] = ((uint64_t)k << 32) | i;
        cand[j] = i < (uint32_t)Q.n && B > 1 && k <= key_bound(B, drawn(B));
        if (cand[j]) list[off[at[j]] + atomicAdd(&fill[at[j]], 1u)] = me[j];
    }
    __syncthreads();
    uint32_t sum = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int i = j * ST + t;
        const int B = (int)cnt[at[j]], r = drawn(B), f = (int)fill[at[j]];
        bool keep = i < Q.n && B == 1;
        if (i < Q.n && B > 1 && f < r) {  // too few candidates: all members
            int rank = 0;
            for (int e = 0; e < Q.n && rank < r; ++e)
                if (slot[e] == at[j])
                    rank += (((uint64_t)option_key(Q.seed, (uint32_t)e) << 32) | (uint32_t)e) <
                            me[j];
            keep = rank < r;
        } else if (cand[j]) {
            const uint64_t *l = list + off[at[j]];
            int rank = 0;
            for (int e = 0; e < f && rank < r; ++e) rank += l[e] < me[j];
            keep = rank < r;
        }
        const u64 m = __ballot(keep);
        if (lane == 0) ms[j * (ST / 64) + wave] = m;
    }
    __syncthreads();
    if (wave == 0) {
        const uint32_t n = lane < MASKS ? (uint32_t)__popcll(ms[lane]) : 0;
        sum = wave_scan(n);
        if (lane < MASKS) before[lane] = sum - n;
        if (lane == 63) count[qi] = (int32_t)sum;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const u64 m = ms[j * (ST / 64) + wave];
        if ((m >> lane) & 1)
            out[Q.off + before[j * (ST / 64) + wave] +
                (uint32_t)__popcll(m & ((1ull << lane) - 1))] = j * ST + t;
    }
}

__global__ __launch_bounds__(ST) void k_s_clear(Table tb, int64_t slots)
{
    for (int64_t s = (int64_t)blockIdx.x * ST + threadIdx.x; s < slots;
         s += (int64_t)gridDim.x * ST) {
        tb.key[s] = NO_HASH;
        tb.cnt[s] = 0;
    }
}

static_assert(sizeof(SampleQ) % 8 == 0, "whole words for launch_put");
static_assert(MASKS <= 64 && LSLOTS <= 65536, "one wave scans the masks, used[] holds slots");

}  // namespace
}  // namespace cm

struct cm_sampler {
    int device = 0;
    int32_t max_queries = 0;
    int64_t max_options = 0;
    int64_t slots = 0;            // table slots, padded for 16-byte reads
    cm::SampleQ *h_q = nullptr;   // pinned staging of the descriptors
    cm::SampleQ *d_q = nullptr;
    hipEvent_t staged = nullptr;  // the last copy out of h_q has been done
    unsigned char *d = nullptr;   // all device scratch
    cm::Table tb{};               // empty between calls
    bool clean = true;            // tb is empty once the calls so far, recorded ones aside, end
    uint32_t *slot = nullptr;     // per option: its slot in the query's part of the table
    uint64_t *list = nullptr;     // candidates of the buckets
    cm::u64 *mask = nullptr;      // kept options, 64 per word
    uint32_t *kept = nullptr;     // per chunk
    uint32_t *group = nullptr;    // per GROUP chunks
    uint32_t *arena = nullptr;    // list entries given out
};

namespace {

using cm::fail;

void free_sampler(cm_sampler *s)
{
    if (s->h_q) (void)hipHostFree(s->h_q);
    if (s->d_q) (void)hipFree(s->d_q);
    if (s->staged) (void)hipEventDestroy(s->staged);
    if (s->d) (void)hipFree(s->d);
}

int clear_blocks(int64_t slots)
{
    return (int)std::min<int64_t>((slots + cm::ST - 1) / cm::ST, 4096);
}

}  // namespace

extern "C" {

cm_status cm_sampler_create(int32_t max_queries, int64_t max_options, cm_sampler **out)
{
    using namespace cm;
    if (!out) return fail(CM_EINVAL, "out is NULL");
    *out = nullptr;
    if (max_queries < 1 || max_options < 1 || max_options > INT32_MAX - 1)
        return fail(CM_EINVAL, "max_queries must be >= 1 and max_options in [1, 2^31 - 2]");
    cm_sampler *s = new (std::nothrow) cm_sampler;
    if (!s) return fail(CM_ENOMEM, "host allocation failed");
    if (hipGetDevice(&s->device) != hipSuccess) {
        delete s;
        return fail(CM_EDEVICE, "no HIP device");
    }
    s->max_queries = max_queries;
    s->max_options = max_options;
    // the scratch, laid out from the widest element type down
    const int64_t T = max_options, chunks = T / CHUNK + max_queries;
    const int64_t groups = chunks / GROUP + 1;
    s->slots = (2 * T + max_queries + 3) / 4 * 4;
    const size_t bytes = (size_t)s->slots * (sizeof(u64) + 3 * sizeof(int32_t)) +
                         (size_t)T * (sizeof(uint64_t) + sizeof(uint32_t)) +
                         (size_t)chunks * (MASKS * sizeof(u64) + sizeof(uint32_t)) +
                         (size_t)groups * sizeof(uint32_t) + 64;
    bool ok = hipHostMalloc((void **)&s->h_q, sizeof(SampleQ) * max_queries, 0) == hipSuccess &&
              hipMalloc((void **)&s->d_q, sizeof(SampleQ) * max_queries) == hipSuccess &&
              hipEventCreateWithFlags(&s->staged, hipEventDisableTiming) == hipSuccess &&
              hipMalloc((void **)&s->d, bytes) == hipSuccess;
    if (ok) {
        unsigned char *p = s->d;
        auto take = [&p](size_t n) {
            unsigned char *at = p;
            p += n;
            return at;
        };
        // slots is a multiple of 4: cnt starts on a 16-byte boundary
        s->tb.key = (u64 *)take((size_t)s->slots * sizeof(u64));
        s->tb.cnt = (int32_t *)take((size_t)s->slots * sizeof(int32_t));
        s->tb.off = (uint32_t *)take((size_t)s->slots * sizeof(uint32_t));
        s->tb.fill = (int32_t *)take((size_t)s->slots * sizeof(int32_t));
        s->list = (uint64_t *)take((size_t)T * sizeof(uint64_t));
        s->mask = (u64 *)take((size_t)chunks * MASKS * sizeof(u64));
        s->slot = (uint32_t *)take((size_t)T * sizeof(uint32_t));
        s->kept = (uint32_t *)take((size_t)chunks * sizeof(uint32_t));
        s->group = (uint32_t *)take((size_t)groups * sizeof(uint32_t));
        s->arena = (uint32_t *)take(sizeof(uint32_t));
    }
    if (!ok) {
        (void)hipGetLastError();
        free_sampler(s);
        delete s;
        return fail(CM_ENOMEM, "sampler allocation failed");
    }
    hipLaunchKernelGGL(k_s_clear, dim3(clear_blocks(s->slots)), dim3(ST), 0, nullptr, s->tb,
                       s->slots);
    if (hipGetLastError() != hipSuccess || hipStreamSynchronize(nullptr) != hipSuccess) {
        (void)hipGetLastError();
        free_sampler(s);
        delete s;
        return fail(CM_EDEVICE, "sampler initialisation failed");
    }
    *out = s;
    return CM_OK;
}

cm_status cm_sampler_destroy(cm_sampler *s)
{
    if (!s) return fail(CM_EINVAL, "sampler is NULL");
    (void)hipDeviceSynchronize();
    free_sampler(s);
    delete s;
    return CM_OK;
}

cm_status cm_sample_buckets(cm_sampler *sp, const cm_batch *b, const uint64_t *hashes,
                            const uint64_t *seeds, int32_t *sel_idx, int32_t *sel_count,
                            cm_stream stream)
{
    using namespace cm;
    if (!sp || !b) return fail(CM_EINVAL, "sampler or batch is NULL");
    if (b->n_queries < 0) return fail(CM_EINVAL, "n_queries < 0");
    if (b->n_queries == 0) return CM_OK;
    if (!b->queries || !seeds) return fail(CM_EINVAL, "queries or seeds is NULL");
    if (b->n_queries > sp->max_queries)
        return fail(CM_E2BIG, "batch has %d queries, sampler holds %d", b->n_queries,
                    sp->max_queries);
    if (!sel_count) return fail(CM_EINVAL, "sel_count is NULL");
    int64_t T = 0;
    for (int32_t q = 0; q < b->n_queries; ++q) {
        const cm_query &Q = b->queries[q];
        if (Q.n_cands < 0) return fail(CM_EINVAL, "query %d: n_cands %d < 0", q, Q.n_cands);
        if (Q.cost_off < 0) return fail(CM_EINVAL, "query %d: negative cost_off", q);
        T += Q.n_cands;
    }
    if (T > sp->max_options)
        return fail(CM_E2BIG, "batch has %lld options, sampler holds %lld", (long long)T,
                    (long long)sp->max_options);
    if (T > 0 && (!hashes || !sel_idx)) return fail(CM_EINVAL, "hashes or sel_idx is NULL");
    int dev = -1;
    CM_HIP(hipGetDevice(&dev));
    if (dev != sp->device)
        return fail(CM_EINVAL, "sampler lives on device %d but device %d is current", sp->device,
                    dev);

    hipStream_t s = (hipStream_t)stream;
    const int nq = b->n_queries;
    const bool by_value = nq <= VALUE_Q;
    // On a stream under capture the call is recorded, not run: the pinned block,
    // its event and the table's state stay those of the last call.
    const bool recorded = capturing(s);
    SampleArgs args;
    std::unique_ptr<SampleQ[]> own(!by_value && recorded ? new (std::nothrow) SampleQ[nq]
                                                         : nullptr);
    SampleQ *const hq = by_value ? args.q : recorded ? own.get() : sp->h_q;
    if (!hq) return fail(CM_ENOMEM, "host allocation failed");
    if (!by_value && !recorded)
        CM_HIP(hipEventSynchronize(sp->staged));  // the last copy has left h_q
    int64_t base = 0;
    int32_t chunks = 0, most = 0;
    for (int q = 0; q < nq; ++q) {
        const cm_query &Q = b->queries[q];
        most = std::max(most, Q.n_cands);
        hq[q] = SampleQ{base, Q.cost_off, seeds[q], Q.n_cands, chunks};
        base += Q.n_cands;
        chunks += std::max(1, (int32_t)(((int64_t)Q.n_cands + CHUNK - 1) / CHUNK));
    }
    if (!by_value && recorded) {
        CM_HIP(launch_put(hq, sizeof(SampleQ) * nq, sp->d_q, s));
    } else if (!by_value) {
        CM_HIP(hipMemcpyAsync(sp->d_q, hq, sizeof(SampleQ) * nq, hipMemcpyHostToDevice, s));
        CM_HIP(hipEventRecord(sp->staged, s));
    }

    const dim3 t(ST);
    // one workgroup per query or chunk, in as many launches as they take
    auto launch = [](int32_t n, auto &&kernel) {
        for (int64_t at = 0; at < n; at += MAX_GRID) {
            kernel((int)at, dim3((unsigned)std::min<int64_t>(MAX_GRID, n - at)));
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    };
    if (most <= CHUNK) {
        CM_HIP(launch(nq, [&](int at, dim3 g) {
            if (by_value)
                hipLaunchKernelGGL(k_s_small<true>, g, t, 0, s, args, sp->d_q, at, hashes, sel_idx,
                                   sel_count);
            else
                hipLaunchKernelGGL(k_s_small<false>, g, t, 0, s, SampleArgs{}, sp->d_q, at, hashes,
                                   sel_idx, sel_count);
        }));
        return CM_OK;
    }
    if (!sp->clean) {  // an earlier call's launches failed
        hipLaunchKernelGGL(k_s_clear, dim3(clear_blocks(sp->slots)), dim3(ST), 0, s, sp->tb,
                           sp->slots);
        CM_HIP(hipGetLastError());
    }
    if (!recorded) sp->clean = false;
    CM_HIP(launch(chunks, [&](int at, dim3 g) {
        if (by_value)
            hipLaunchKernelGGL(k_s_insert<true>, g, t, 0, s, args, sp->d_q, nq, at, hashes, sp->tb,
                               sp->slot, sp->arena);
        else
            hipLaunchKernelGGL(k_s_insert<false>, g, t, 0, s, SampleArgs{}, sp->d_q, nq, at,
                               hashes, sp->tb, sp->slot, sp->arena);
    }));
    const int64_t slots = 2 * T + nq;
    hipLaunchKernelGGL(k_s_alloc, dim3((unsigned)((slots + 4 * AT - 1) / (4 * AT))), dim3(AT), 0,
                       s, sp->tb, slots, sp->arena);
    CM_HIP(hipGetLastError());
    CM_HIP(launch(chunks, [&](int at, dim3 g) {
        hipLaunchKernelGGL(k_s_list, g, t, 0, s, sp->d_q, nq, at, sp->tb, sp->slot, sp->list);
    }));
    CM_HIP(launch(chunks, [&](int at, dim3 g) {
        hipLaunchKernelGGL(k_s_rank, g, t, 0, s, sp->d_q, nq, at, sp->tb, sp->slot, sp->list,
                           sp->mask, sp->kept);
    }));
    if ((int64_t)most > (int64_t)2 * GROUP * CHUNK) {
        hipLaunchKernelGGL(k_s_groups, dim3((chunks + GROUP - 1) / GROUP), t, 0, s, sp->kept,
                           chunks, sp->group);
        CM_HIP(hipGetLastError());
    }
    CM_HIP(launch(chunks, [&](int at, dim3 g) {
        hipLaunchKernelGGL(k_s_write, g, t, 0, s, sp->d_q, nq, at, chunks, sp->tb, sp->slot,
                           sp->mask, sp->kept, sp->group, sel_idx, sel_count);
    }));
    if (!recorded) sp->clean = true;
    return CM_OK;
}

}  // extern "C"
