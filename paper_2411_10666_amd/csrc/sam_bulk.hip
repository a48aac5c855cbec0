// gfx950 kernels that build an automaton with the whole chip: of the corpus (arxiv 2411.10666,
// Section 3.1, Algorithm 2 Build-SAM), or of prompts too long for one workgroup's LDS.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sam_bulk_launch.h"

namespace sam {

namespace {

constexpr uint32_t kSort = 512;                  // threads of the kernels that sort
constexpr uint32_t kWaves = kSort / 64;
constexpr uint32_t kItems = kBulkTile / kSort;

struct BulkCtx {
    template <class F>
    __device__ __forceinline__ void lanes(F f) { f(threadIdx.x & 63); }
    __device__ __forceinline__ void wave_sync()
    {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    }
    // see bulk_long_walk
    template <class F>
    __device__ __forceinline__ uint32_t chain(uint32_t v, uint32_t down, F f, uint32_t *list, uint32_t &more, uint32_t &next)
    {
        const uint32_t lane = threadIdx.x & 63;
        const bool there = (uint64_t)lane * down <= v;
        const uint32_t s = there ? v - lane * down : 0;
        uint32_t link, kind;
        f(s, link, kind);
        const uint32_t above = (uint32_t)__shfl_up((int)link, 1);
        const unsigned long long follows = __ballot(lane == 0 || (there && above == s && s != v)),
                                 ends = __ballot(kind == 2), roots = __ballot(s == 0);
        uint32_t count = follows == ~0ull ? 64u : (uint32_t)__builtin_ctzll(~follows);
        more = 1;
        if (ends) {
            const uint32_t at = (uint32_t)__builtin_ctzll(ends);
            if (at < count) { count = at; more = 0; }
        }
        if (roots) {
            const uint32_t at = (uint32_t)__builtin_ctzll(roots);
            if (at < count) { count = at + 1; more = 0; }
        }
        if (lane < count) list[lane] = kind ? kNil : s;
        next = count ? (uint32_t)__shfl((int)link, (int)(count - 1)) : 0u;
        return count;
    }
    template <class U>
    __device__ __forceinline__ U cas(U *p, U expected, U v)
    {
        __hip_atomic_compare_exchange_strong(p, &expected, v, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
        return expected;
    }
    template <class U>
    __device__ __forceinline__ U add(U *p, U v)
    {
        return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ uint32_t lower(uint32_t *p, uint32_t v)
    {
        return __hip_atomic_fetch_min(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ void raise(uint32_t *p, uint32_t v)
    {
        __hip_atomic_fetch_max(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ void bit_or(uint32_t *p, uint32_t v)
    {
        __hip_atomic_fetch_or(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ uint32_t exch(uint32_t *p, uint32_t v)
    {
        return __hip_atomic_exchange(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ uint32_t fresh(uint32_t *p)
    {
        return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ uint32_t mulhi(uint32_t a, uint32_t b) { return __umulhi(a, b); }
    __device__ __forceinline__ uint32_t popc(uint32_t x) { return (uint32_t)__popc(x); }
    __device__ __forceinline__ uint32_t first(uint32_t x) { return (uint32_t)__builtin_ctz(x); }
    __device__ __forceinline__ uint32_t log2(uint32_t x) { return 31u - (uint32_t)__clz((int)x); }
};

// ---- where a text and its working arrays are -------------------------------------

// kListed: the prompts that the begin kernel has listed, else all of them, one after the other
template <class L, class Ix, bool kListed>
struct PromptSource {
    typedef Ix Index;
    typedef BulkTables<L> Store;
    static constexpr bool kCompact = L::kSlots == 16, kList = kListed;
    BatchView B;
    const int32_t *seq_map, *tokens;
    const int64_t *offsets;
    uint32_t lds_tokens, most;
    SeqMeta *list;

    __device__ __forceinline__ int sequence(uint32_t y) const { return seq_map ? seq_map[y] : (int)y; }
    __device__ __forceinline__ bool taken(uint32_t y) const
    {
        return bulk_takes(B, offsets[y + 1] - offsets[y], lds_tokens, most);
    }
    __host__ __device__ __forceinline__ char *rec(int b) const
    {
        return reinterpret_cast<char *>(B.dyn_rec) +
               (size_t)b * B.max_states * (kCompact ? sizeof(DynRecCompact) : sizeof(DynRec));
    }
    __host__ __device__ __forceinline__ char *slots(int b) const
    {
        return reinterpret_cast<char *>(B.dyn_slots) + (size_t)b * B.dyn_buckets * 128;
    }
    // the counts are where the sequence's own will be
    __device__ __forceinline__ uint32_t *counts(int b) const { return &B.meta[b].n_states; }
    __device__ __forceinline__ bool get(uint32_t y, BulkSeq<Ix> &q) const
    {
        if (kListed) y = list[y].listed;
        const int b = sequence(y);
        q.of = (uint32_t)b;
        const int64_t from = offsets[y], to = offsets[y + 1];
        q.n = B.meta[b].n;                   // (asked for with the offsets, not after them)
        if (!bulk_takes(B, to - from, lds_tokens, most) || q.n == 0) return false;
        q.tok = tokens + from;
        q.counts = counts(b);
        bulk_place(q, rec(b), slots(b), reinterpret_cast<char *>(B.dyn_text + (size_t)b * B.max_seq_len));
        return true;
    }
    __device__ __forceinline__ Store store(const BulkSeq<Ix> &q) const
    {
        return Store{rec((int)q.of), slots((int)q.of), B.dyn_buckets, q.tok, q.n};
    }
};

struct CorpusSource {
    typedef uint32_t Index;
    typedef BulkCorpus Store;
    const int32_t *tok;
    uint32_t n;
    BulkWork w;
    RootEnt *root;

    __device__ __forceinline__ bool get(uint32_t, BulkSeq<uint32_t> &q) const
    {
        q.n = n;
        q.tok = tok;
        q.counts = w.counts;
        bulk_place(q, w.first, w.second, w.third);
        return true;
    }
    // the transitions' table lies over the first region, of which the records need nothing any more
    __host__ __device__ __forceinline__ Store table() const
    {
        return Store{w.rec, reinterpret_cast<uint64_t *>(w.first),
                     reinterpret_cast<uint32_t *>(w.first + 16 * (size_t)n), 2 * n, root, tok, n};
    }
    __device__ __forceinline__ Store store(const BulkSeq<uint32_t> &) const { return table(); }
};

// ---- lanes working together ---------------------------------------------------------

__device__ __forceinline__ uint32_t lane_id() { return threadIdx.x & 63; }
__device__ __forceinline__ uint32_t uni(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }

__device__ __forceinline__ uint32_t wave_sums(uint32_t v)      // over the lower lanes and this one
{
    for (int d = 1; d < 64; d *= 2) {
        const uint32_t below = (uint32_t)__shfl_up((int)v, d);
        if (lane_id() >= (uint32_t)d) v += below;
    }
    return v;
}

__device__ __forceinline__ uint32_t wave_total(uint32_t v)
{
    for (int d = 32; d; d /= 2) v += (uint32_t)__shfl_xor((int)v, d);
    return v;
}

struct SortLds {
    uint32_t count[kWaves][256];
    uint32_t base[256];
    uint32_t part[kWaves];
};

// base[d] becomes the sum over the entries before d; all threads call it
__device__ __forceinline__ void exclusive_256(SortLds &s, uint32_t own, uint32_t plus)
{
    uint32_t upto = 0;
    if (threadIdx.x < 256) {
        upto = wave_sums(own);
        if (lane_id() == 63) s.part[threadIdx.x >> 6] = upto;
    }
    __syncthreads();
    if (threadIdx.x < 256) {
        uint32_t before = 0;
        for (uint32_t w = 0; w < (threadIdx.x >> 6); w++) before += s.part[w];
        s.base[threadIdx.x] = before + upto - own + plus;
    }
    __syncthreads();
}

// One stable pass over a tile [lo, hi): every wave ranks its own 256 items, 64 at a time, by eight
// ballots a digit; then the waves' counts are summed up.  base[d]: where the next item of
// digit d goes.
template <class K, class Load, class Put>
__device__ __forceinline__ void radix_tile(SortLds &s, uint32_t lo, uint32_t hi, uint32_t shift, Load load, Put put)
{
    const uint32_t wave = threadIdx.x >> 6, lane = lane_id();
    uint32_t *const count = s.count[wave];
    K key[kItems];
    uint32_t val[kItems], rank[kItems];
#pragma unroll
    for (uint32_t r = 0; r < kItems; r++) {
        const uint32_t at = lo + wave * (64 * kItems) + 64 * r + lane;
        key[r] = 0;
        val[r] = 0;
        if (at < hi) load(at, key[r], val[r]);
    }
#pragma unroll
    for (uint32_t r = 0; r < 4; r++) count[64 * r + lane] = 0;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (uint32_t r = 0; r < kItems; r++) {
        const uint32_t at = lo + wave * (64 * kItems) + 64 * r + lane, d = (uint32_t)(key[r] >> shift) & 255u;
        const bool on = at < hi;
        unsigned long long mask = __ballot(on);
#pragma unroll
        for (int bit = 0; bit < 8; bit++) {
            const unsigned long long set = __ballot((d >> bit) & 1u);
            mask &= ((d >> bit) & 1u) ? set : ~set;
        }
        const uint32_t below = (uint32_t)__popcll(mask & ((1ull << lane) - 1ull));
        uint32_t before = 0;
        if (on) before = count[d];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        __builtin_amdgcn_wave_barrier();
        if (on && below == 0) count[d] = before + (uint32_t)__popcll(mask);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        __builtin_amdgcn_wave_barrier();
        rank[r] = before + below;
    }
    __syncthreads();
    if (threadIdx.x < 256) {
        uint32_t run = s.base[threadIdx.x];
        for (uint32_t w = 0; w < kWaves; w++) {
            const uint32_t c = s.count[w][threadIdx.x];
            s.count[w][threadIdx.x] = run;
            run += c;
        }
        s.base[threadIdx.x] = run;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t r = 0; r < kItems; r++) {
        const uint32_t at = lo + wave * (64 * kItems) + 64 * r + lane, d = (uint32_t)(key[r] >> shift) & 255u;
        if (at < hi) put(count[d] + rank[r], key[r], val[r]);
    }
    __syncthreads();
}

// Starts of groups over sorted places [0, count) that are cut into tiles from lo to hi: for each
// place k, f(k, start, last), where a group starts at every place that differs(k) from the one
// before.  open: the start of the group that lo belongs to, if it does not start one.
template <class Differs, class F>
__device__ __forceinline__ void each_group(SortLds &s, uint32_t lo, uint32_t hi, uint32_t count, uint32_t open,
                                           Differs differs, F f)
{
    const uint32_t wave = threadIdx.x >> 6;
    for (uint32_t base = lo; base < hi; base += kSort) {
        const uint32_t k = base + threadIdx.x;
        const bool on = k < hi;
        // 1 + the nearest start up to here, 0: none in this wave
        uint32_t at = on && (k == 0 || differs(k)) ? k + 1 : 0;
        for (int d = 1; d < 64; d *= 2) {
            const uint32_t below = (uint32_t)__shfl_up((int)at, d);
            if (lane_id() >= (uint32_t)d && below > at) at = below;
        }
        if (lane_id() == 63) s.part[wave] = at;
        __syncthreads();
        uint32_t carry = open + 1, end = open + 1;
        for (uint32_t w = 0; w < kWaves; w++) {
            const uint32_t p = s.part[w];
            if (p > end) end = p;
            if (w < wave && p > carry) carry = p;
        }
        if (carry > at) at = carry;
        if (on) f(k, at - 1, k + 1 == count || differs(k + 1));
        open = end - 1;
        __syncthreads();
    }
}

// ---- the sort -------------------------------------------------------------------

// How many places of each digit every run of tiles has.
template <class Src>
__global__ __launch_bounds__(kSort) void bulk_hist_kernel(Src src, BulkSort sort, uint32_t pass)
{
    __shared__ uint32_t h[256];
    BulkSeq<typename Src::Index> q;
    if (!src.get(blockIdx.y, q)) return;
    const BulkCut cut = bulk_cut(q.n);
    if (blockIdx.x >= cut.blocks) return;
    if (threadIdx.x < 256) h[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t lo = blockIdx.x * cut.chunk, hi = q.n - lo > cut.chunk ? lo + cut.chunk : q.n;
    const uint64_t *const key = q.key(pass + 1);
    for (uint32_t i = lo + threadIdx.x; i < hi; i += kSort) {
        const uint64_t k = pass ? key[i] : bulk_key(q.tok, i, sort);
        atomicAdd(&h[(uint32_t)(k >> (8 * pass)) & 255u], 1u);
    }
    __syncthreads();
    if (threadIdx.x < 256) q.hist[blockIdx.x * 256 + threadIdx.x] = h[threadIdx.x];
}

// One pass, least significant digits first.  A workgroup sums up all the runs' counts by itself (256
// times as many words as there are runs, at most 256 of them, from the L2): that takes less than a
// launch.
template <class Src>
__global__ __launch_bounds__(kSort) void bulk_scatter_kernel(Src src, BulkSort sort, uint32_t pass)
{
    __shared__ SortLds s;
    BulkSeq<typename Src::Index> q;
    if (!src.get(blockIdx.y, q)) return;
    const BulkCut cut = bulk_cut(q.n);
    if (blockIdx.x >= cut.blocks) return;
    // (16 loads at a time in flight: one after the other they took longer than all the rest)
    const uint32_t digit = threadIdx.x & 255u, half = threadIdx.x >> 8;
    uint32_t all = 0, before = 0;
#pragma unroll 1
    for (uint32_t b = half; b < cut.blocks; b += 32) {
        uint32_t c[16];
#pragma unroll
        for (uint32_t j = 0; j < 16; j++) c[j] = b + 2 * j < cut.blocks ? q.hist[(b + 2 * j) * 256 + digit] : 0u;
#pragma unroll
        for (uint32_t j = 0; j < 16; j++) {
            all += c[j];
            before += b + 2 * j < blockIdx.x ? c[j] : 0u;
        }
    }
    if (half) { s.count[0][digit] = all; s.count[1][digit] = before; }
    __syncthreads();
    if (!half) { all += s.count[0][digit]; before += s.count[1][digit]; }
    exclusive_256(s, all, before);
    const uint32_t lo = blockIdx.x * cut.chunk, hi = q.n - lo > cut.chunk ? lo + cut.chunk : q.n;
    const uint64_t *const key = q.key(pass + 1);
    const uint32_t *const pos = q.pos(pass + 1);
    uint64_t *const to_key = q.key(pass);
    uint32_t *const to_pos = q.pos(pass);
    for (uint32_t t = lo; t < hi; t += kBulkTile)
        radix_tile<uint64_t>(
            s, t, hi - t > kBulkTile ? t + kBulkTile : hi, 8 * pass,
            [&](uint32_t at, uint64_t &k, uint32_t &v) {
                k = pass ? key[at] : bulk_key(q.tok, at, sort);
                v = pass ? pos[at] : at;
            },
            [&](uint32_t at, uint64_t k, uint32_t v) {
                to_key[at] = k;
                to_pos[at] = v;
            });
}

// A group of `size` places from `start` on is known in round `round`.
template <class I>
__device__ __forceinline__ void announce(const BulkSeq<I> &q, uint32_t round, uint32_t start, uint32_t size)
{
    if (size > 1) q.ctl[kCtlActive + round] = 1;
    if (size > kBulkLarge) {
        BulkCtx ctx;
        q.queue(round)[ctx.add(&q.ctl[kCtlQueued + round], 1u)] = start;
        ctx.raise(&q.ctl[kCtlLargest], size);
    }
}

// Groups of equal keys.
template <class Src>
__global__ __launch_bounds__(kSort) void bulk_groups_kernel(Src src, uint32_t first)
{
    __shared__ SortLds s;
    __shared__ uint32_t found;
    BulkSeq<typename Src::Index> q;
    if (!src.get(blockIdx.y, q)) return;
    const BulkCut cut = bulk_cut(q.n);
    if (blockIdx.x >= cut.blocks) return;
    const uint32_t lo = blockIdx.x * cut.chunk, hi = q.n - lo > cut.chunk ? lo + cut.chunk : q.n;
    const uint64_t *const key = q.key(first);
    auto differs = [&](uint32_t k) { return key[k] != key[k - 1]; };
    // the group that is open at lo starts at the nearest such place before it
    uint32_t open = 0;
    for (uint32_t end = lo; end;) {
        if (threadIdx.x == 0) found = 0;
        __syncthreads();
        const uint32_t k = end > threadIdx.x ? end - 1 - threadIdx.x : 0;
        if (k > 0 && differs(k)) atomicMax(&found, k);
        __syncthreads();
        open = found;
        __syncthreads();
        if (open) break;
        end = end > kSort ? end - kSort : 0;
    }
    each_group(s, lo, hi, q.n, open, differs, [&](uint32_t k, uint32_t start, bool last) {
        if (k != start) q.gs(0)[k] = start;
        if (last) {
            q.gs(0)[start] = kBulkStart | (k + 1 - start);
            announce(q, 0, start, k + 1 - start);
        }
        q.name[q.pos(first)[k]] = start;
        q.lev[k] = 0;
    });
}

// Sorts `size` places by their second names, 8 bits a pass, from key and pos into to_key and to_pos and
// back: in the former after an even number of passes.
__device__ void sort_places(SortLds &s, uint32_t *key, uint32_t *pos, uint32_t *to_key, uint32_t *to_pos, uint32_t size,
                            uint32_t passes)
{
    for (uint32_t pass = 0; pass < passes; pass++) {
        const uint32_t shift = 8 * pass < 32 ? 8 * pass : 24;      // a fifth pass sorts by the fourth's digit again
        if (threadIdx.x < 256) s.base[threadIdx.x] = 0;
        __syncthreads();
        for (uint32_t k = threadIdx.x; k < size; k += kSort) atomicAdd(&s.base[(key[k] >> shift) & 255u], 1u);
        __syncthreads();
        const uint32_t own = threadIdx.x < 256 ? s.base[threadIdx.x] : 0;
        __syncthreads();
        exclusive_256(s, own, 0);
        for (uint32_t t = 0; t < size; t += kBulkTile)
            radix_tile<uint32_t>(
                s, t, size - t > kBulkTile ? t + kBulkTile : size, shift,
                [&](uint32_t at, uint32_t &k, uint32_t &v) { k = key[at]; v = pos[at]; },
                [&](uint32_t at, uint32_t k, uint32_t v) { to_key[at] = k; to_pos[at] = v; });
        __syncthreads();
        uint32_t *const k = key, *const p = pos;
        key = to_key; pos = to_pos;
        to_key = k; to_pos = p;
    }
}

// Groups of the next round among the places from .. from + size of group g, sorted.
template <class I>
__device__ void part_sorted(SortLds &s, const BulkSeq<I> &q, uint32_t round, uint32_t g, uint32_t from, uint32_t size,
                            const uint32_t *key, const uint32_t *pos)
{
    uint32_t *const to_gs = q.gs(round + 1) + g + from;
    each_group(s, 0, size, size, 0, [&](uint32_t k) { return key[k] != key[k - 1]; },
               [&](uint32_t k, uint32_t start, bool last) {
                   if (k != start) to_gs[k] = g + from + start;
                   if (last) {
                       to_gs[start] = kBulkStart | (k + 1 - start);
                       announce(q, round + 1, g + from + start, k + 1 - start);
                   }
                   if (from + start) {
                       q.name[pos[k]] = g + from + start;
                       if (k == start) q.lev[g + from + start] = (uint8_t)(round + 1);
                   }
               });
    __syncthreads();
}

// The same for up to kCounted places that are not sorted: by counting, in LDS.
constexpr uint32_t kCounted = 256;
template <class I>
__device__ void part_counted(SortLds &s, const BulkSeq<I> &q, uint32_t round, uint32_t g, uint32_t from, uint32_t size,
                             const uint32_t *key, uint32_t *pos)
{
    const uint32_t k = threadIdx.x, own = k < size ? key[k] : 0, v = k < size ? pos[k] : 0;
    if (k < size) s.base[k] = own;
    __syncthreads();
    if (k < size) {
        uint32_t less = 0, same = 0, before = 0;
#pragma unroll 8
        for (uint32_t j = 0; j < size; j++) {
            const uint32_t x = s.base[j];
            less += x < own;
            same += x == own;
            before += x == own && j < k;
        }
        const uint32_t start = g + from + less;
        pos[less + before] = v;
        q.gs(round + 1)[start + before] = before ? start : kBulkStart | same;
        if (same > 1) q.ctl[kCtlActive + round + 1] = 1;
        if (from + less) {
            q.name[v] = start;
            if (!before) q.lev[start] = (uint8_t)(round + 1);
        }
    }
    __syncthreads();
}

// how many of the mask's bits belong to lower lanes
__device__ __forceinline__ uint32_t lower_bits(unsigned long long mask)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
}

// The places of group g that have the second name `pivot` to where they belong, those with smaller ones
// in front of them and those with larger ones from `more` on, into to_key and to_pos.  Returns how
// many are smaller.
template <class I>
__device__ uint32_t split_places(SortLds &s, const BulkSeq<I> &q, uint32_t first, uint32_t round, uint32_t g, uint32_t size,
                                 uint32_t pivot, uint32_t &more)
{
    constexpr uint32_t kEach = 4;                    // places of a thread at a time
    const uint32_t wave = uni(threadIdx.x >> 6), lane = lane_id();
    const uint32_t *const key = q.sec + g, *const pos = q.pos(first + round) + g;
    uint32_t *const to_key = q.sec2 + g, *const to_pos = q.pos(first + round + 1) + g;
    uint32_t less = 0, same = 0;
    for (uint32_t base = 0; base < size; base += kSort * kEach) {
        uint32_t k[kEach];
#pragma unroll
        for (uint32_t r = 0; r < kEach; r++) {
            const uint32_t at = base + r * kSort + threadIdx.x;
            k[r] = key[at < size ? at : size - 1];   // (no branches: all loads are under way at once)
            if (at >= size) k[r] = kNil;
        }
#pragma unroll
        for (uint32_t r = 0; r < kEach; r++) {
            less += k[r] < pivot;
            same += k[r] == pivot;
        }
    }
    less = wave_total(less);
    same = wave_total(same);
    if (lane == 0) { s.base[wave] = less; s.base[kWaves + wave] = same; }
    __syncthreads();
    less = same = 0;
    for (uint32_t w = 0; w < kWaves; w++) { less += s.base[w]; same += s.base[kWaves + w]; }
    less = uni(less);
    same = uni(same);
    more = less + same;
    const uint32_t start = g + less;
    uint32_t *const to_gs = q.gs(round + 1);
    uint32_t at_less = 0, at_same = 0, at_more = more;       // where the next tile's go
    // a wave takes 64 * kEach places side by side, and asks for the next ones before it stores these: a wait for
    // loads is one for all stores before them
    uint32_t next_k[kEach], next_v[kEach];
    auto ask = [&](uint32_t lo) {
#pragma unroll
        for (uint32_t r = 0; r < kEach; r++) {
            const uint32_t at = lo + 64 * r + lane, there = at < size ? at : size - 1;
            next_k[r] = key[there];
            next_v[r] = pos[there];
        }
    };
    ask(wave * (64 * kEach));
    for (uint32_t base = 0, turn = 0; base < size; base += kSort * kEach, turn ^= 1) {
        uint32_t k[kEach], v[kEach];
        uint32_t rank[kEach];                        // how many smaller ones of this wave are before it; equal ones above
        const uint32_t lo = base + wave * (64 * kEach);
#pragma unroll
        for (uint32_t r = 0; r < kEach; r++) {
            k[r] = lo + 64 * r + lane < size ? next_k[r] : kNil;
            v[r] = next_v[r];
        }
        ask(lo + kSort * kEach);
        uint32_t mine_less = 0, mine_same = 0;
#pragma unroll
        for (uint32_t r = 0; r < kEach; r++) {
            const unsigned long long is_less = __ballot(k[r] < pivot), is_same = __ballot(k[r] == pivot);
            rank[r] = (mine_less + lower_bits(is_less)) | (mine_same + lower_bits(is_same)) << 16;
            mine_less += (uint32_t)__popcll(is_less);
            mine_same += (uint32_t)__popcll(is_same);
        }
        // (the counts of the tile before are read until the barrier of the next one)
        uint32_t *const part = s.count[turn];
        if (lane == 0) { part[wave] = mine_less; part[kWaves + wave] = mine_same; }
        __syncthreads();
        uint32_t below = at_less, equal = at_same, above = at_more, all_less = 0, all_same = 0;
        for (uint32_t w = 0; w < kWaves; w++) {
            const uint32_t l = uni(part[w]), e = uni(part[kWaves + w]);
            if (w < wave) {
                below += l;
                equal += e;
                above += 64 * kEach - l - e;                 // (all of an earlier wave's are there)
            }
            all_less += l;
            all_same += e;
        }
#pragma unroll
        for (uint32_t r = 0; r < kEach; r++) {
            const uint32_t l = rank[r] & 0xFFFFu, e = rank[r] >> 16;
            if (lo + 64 * r + lane >= size) continue;
            if (k[r] == pivot) {
                const uint32_t place = equal + e;
                to_pos[less + place] = v[r];
                to_gs[start + place] = place ? start : kBulkStart | same;
                if (less) q.name[v[r]] = start;
            } else {
                const uint32_t place = k[r] < pivot ? below + l : above + 64 * r + lane - l - e;
                to_key[place] = k[r];
                to_pos[place] = v[r];
            }
        }
        at_less += all_less;
        at_same += all_same;
        at_more += kSort * kEach - all_less - all_same;      // (of the last tile: not used any more)
    }
    if (threadIdx.x == 0) {
        announce(q, round + 1, start, same);
        if (less) q.lev[start] = (uint8_t)(round + 1);
    }
    __syncthreads();
    return less;
}

// A round of a group that is too large for counting, by this workgroup alone: its places are sorted by
// their second names, in 3 passes or 5 (an odd number, so that they end in the buffers of the next round).
// In runs of a token and in short periods most of the group's second names are the same, round after
// round: there one pass takes those to their place, in front of them the smaller ones and behind the
// larger ones, and only these are sorted.  What bounds it is one workgroup's round trips, 2.3 us for 2048
// places.  (sam_build, ms, all places sorted / so / the host's builder: 700 000 equal tokens 101 / 25 / 39,
// 8 M of them 1350 / 305 / 556, 100 000 11.5 / 3.8 / 2.6, 700 000 in a period of two 54 / 15 / 41.
// sam_batch_reset of 600 prompts of 8000 equal tokens: 10.4 / 2.7, one workgroup each in all phases 3.1.)
template <class I>
__device__ void bulk_rank_large(SortLds &s, const BulkSeq<I> &q, uint32_t first, uint32_t round, uint32_t g)
{
    const uint32_t size = uni(q.gs(round)[g]) & ~kBulkStart, lane = lane_id();
    uint32_t *const key = q.sec + g, *const to_key = q.sec2 + g;
    uint32_t *const pos = q.pos(first + round) + g, *const to_pos = q.pos(first + round + 1) + g;
    // the most frequent of 64 second names, and how many of them it is
    const uint32_t sample = key[(uint64_t)size * lane / 64];
    uint32_t alike = 0;
    for (int d = 0; d < 64; d++) alike += (uint32_t)__shfl((int)sample, d) == sample;
    uint32_t most = alike;
    for (int d = 32; d; d /= 2) {
        const uint32_t other = (uint32_t)__shfl_xor((int)most, d);
        most = other > most ? other : most;
    }
    // split: what is smaller has come to the front, what is larger behind `more`
    uint32_t more = 0, count = size, passes = q.n < (1u << 24) ? 3 : 5;
    const bool split = uni(most) >= 32;
    if (split) {
        const uint32_t pivot = (uint32_t)__builtin_amdgcn_readlane((int)sample, __builtin_ctzll(__ballot(alike == most)));
        count = split_places(s, q, first, round, g, size, pivot, more);
        passes = q.n < (1u << 16) ? 2 : 4;
    }
    for (uint32_t from = 0;; from = more, count = size - more) {
        if (count > kCounted) {
            sort_places(s, (split ? to_key : key) + from, (split ? to_pos : pos) + from, (split ? key : to_key) + from,
                        (split ? pos : to_pos) + from, count, passes);
            part_sorted(s, q, round, g, from, count, to_key + from, to_pos + from);
        } else if (count) {
            part_counted(s, q, round, g, from, count, to_key + from, to_pos + from);
        }
        if (from == more) break;
    }
}

template <class Src>
__global__ __launch_bounds__(256) void bulk_gather_kernel(Src src, uint32_t first, uint32_t round, uint32_t h)
{
    BulkSeq<typename Src::Index> q;
    if (!src.get(blockIdx.y, q) || h >= q.n || !q.ctl[kCtlActive + round]) return;
    for (uint32_t k = blockIdx.x * 256 + threadIdx.x; k < q.n; k += gridDim.x * 256)
        bulk_gather(q, first, round, h, k);
}

// Workgroups 0 .. n_large-1 take the large groups, the others a run of places each.  The second names
// of a group lie side by side, so what bounds this is counting: 12 operations for four of them.  (72
// registers let seven waves into a SIMD; with the 107 that the large groups' part would take, four, the
// counting of 600 prompts of 8000 tokens takes 3 to 10 % longer.)
template <class Src>
__global__ __launch_bounds__(kSort) __attribute__((amdgpu_num_vgpr(72))) void bulk_rank_kernel(Src src, uint32_t first, uint32_t round, uint32_t h,
                                                         uint32_t n_large)
{
    __shared__ SortLds s;
    BulkSeq<typename Src::Index> q;
    if (!src.get(blockIdx.y, q) || h >= q.n || !q.ctl[kCtlActive + round]) return;
    if (blockIdx.x < n_large) {
        const uint32_t queued = q.ctl[kCtlQueued + round];
        for (uint32_t j = blockIdx.x; j < queued; j += n_large)
            bulk_rank_large(s, q, first, round, uni(q.queue(round)[j]));
        return;
    }
    bool more = false;
    for (uint32_t k = (blockIdx.x - n_large) * kSort + threadIdx.x; k < q.n; k += (gridDim.x - n_large) * kSort)
        more |= bulk_rank<false>(q, first, round, k);
    if (__any(more) && lane_id() == 0) q.ctl[kCtlActive + round + 1] = 1;
}

// ---- the tree -------------------------------------------------------------------

// Minima of 8, 64, 512 and 4096 common lengths.
template <class Src>
__global__ __launch_bounds__(kSort) void bulk_minima_kernel(Src src)
{
    typedef typename Src::Index I;
    __shared__ uint32_t part[kWaves];
    BulkSeq<I> q;
    if (!src.get(blockIdx.y, q)) return;
    const uint32_t count = ingest_pad(q.n), w = blockIdx.x * kSort + threadIdx.x, tops = q.ctl[kCtlTops];
    uint32_t size = ingest_first_mins(q.n);
    if (blockIdx.x * kSort >= size + 4672) return;               // covers the padding of the levels above
    uint32_t least = 0;
    if (w < count / 8) {
        const Eight<I> e = *reinterpret_cast<const Eight<I> *>(q.lcp + 8 * (size_t)w);
        least = e.v[0];
        for (int j = 1; j < 8; j++) least = e.v[j] < least ? e.v[j] : least;
    }
    if (w < size) q.mins1[w] = (I)least;
    for (uint32_t level = 2, bit = 1; level <= 4 && level <= tops; level++, bit *= 8) {
        size = ingest_pad(size / 8);
        if (level < 4) {
            for (uint32_t d = bit; d < 8 * bit; d *= 2) {
                const uint32_t other = (uint32_t)__shfl_xor((int)least, (int)d);
                least = other < least ? other : least;
            }
            const uint32_t at = w / (8 * bit);
            if (w % (8 * bit) == 0 && at < size) q.mins[q.ctl[kCtlLevel + level] + at] = (I)least;
        } else {
            if (lane_id() == 0) part[threadIdx.x >> 6] = least;
            __syncthreads();
            if (threadIdx.x == 0 && w / kSort < size) {
                for (uint32_t j = 1; j < kWaves; j++) least = part[j] < least ? part[j] : least;
                q.mins[q.ctl[kCtlLevel + 4] + w / kSort] = (I)least;
            }
        }
    }
}
static_assert(kSort == 512, "a workgroup finds the minima of 4096");

// The levels above them, by one workgroup.
template <class Src>
__global__ __launch_bounds__(kSort) void bulk_upper_minima_kernel(Src src)
{
    typedef typename Src::Index I;
    BulkSeq<I> q;
    if (!src.get(blockIdx.y, q)) return;
    const uint32_t tops = q.ctl[kCtlTops];
    uint32_t size = ingest_first_mins(q.n);
    for (uint32_t level = 2; level <= tops; level++) {
        const uint32_t real = size / 8;
        size = ingest_pad(real);
        if (level <= 4) continue;
        const I *const below = q.mins + q.ctl[kCtlLevel + level - 1];
        I *const out = q.mins + q.ctl[kCtlLevel + level];
        for (uint32_t w = threadIdx.x; w < size; w += kSort) {
            I least = 0;
            if (w < real) {
                least = below[8 * (size_t)w];
                for (int j = 1; j < 8; j++) least = below[8 * (size_t)w + j] < least ? below[8 * (size_t)w + j] : least;
            }
            out[w] = least;
        }
        __syncthreads();
    }
}

// Clones before each word of bits[]: sums of the runs of words, then their running sum.
template <class Src>
__global__ __launch_bounds__(kSort) void bulk_clone_sums_kernel(Src src)
{
    __shared__ uint32_t part[kWaves];
    BulkSeq<typename Src::Index> q;
    if (!src.get(blockIdx.y, q)) return;
    const uint32_t words = q.n / 32 + 1;
    const BulkCut cut = bulk_cut(words);
    if (blockIdx.x >= cut.blocks) return;
    const uint32_t lo = blockIdx.x * cut.chunk, hi = words - lo > cut.chunk ? lo + cut.chunk : words;
    uint32_t sum = 0;
    for (uint32_t w = lo + threadIdx.x; w < hi; w += kSort) sum += (uint32_t)__popc(q.bits[w]);
    sum = wave_total(sum);
    if (lane_id() == 0) part[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        sum = 0;
        for (uint32_t w = 0; w < kWaves; w++) sum += part[w];
        q.sums[blockIdx.x] = sum;
    }
}

template <class Src>
__global__ __launch_bounds__(kSort) void bulk_clone_ranks_kernel(Src src)
{
    __shared__ uint32_t part[kWaves];
    BulkSeq<typename Src::Index> q;
    if (!src.get(blockIdx.y, q)) return;
    const uint32_t words = q.n / 32 + 1;
    const BulkCut cut = bulk_cut(words);
    if (blockIdx.x >= cut.blocks) return;
    const uint32_t lo = blockIdx.x * cut.chunk, hi = words - lo > cut.chunk ? lo + cut.chunk : words;
    uint32_t run = 0;
    for (uint32_t b = 0; b < blockIdx.x; b++) run += q.sums[b];
    for (uint32_t base = lo; base < hi; base += kSort) {
        const uint32_t w = base + threadIdx.x, mine = w < hi ? (uint32_t)__popc(q.bits[w]) : 0u, upto = wave_sums(mine);
        if (lane_id() == 63) part[threadIdx.x >> 6] = upto;
        __syncthreads();
        uint32_t before = 0, all = 0;
        for (uint32_t j = 0; j < kWaves; j++) {
            all += part[j];
            before += j < (threadIdx.x >> 6) ? part[j] : 0u;
        }
        if (w < hi) q.rank[w] = run + before + upto - mine;
        run += all;
        __syncthreads();
    }
    if (threadIdx.x == 0 && hi == words) q.counts[kCntStates] = 1 + q.n + run;
}

// ---- phases in which every index works by itself ----------------------------------

enum class Phase { kOrder, kCommon, kInterval, kRepresent, kParent, kLeaf, kFirst, kSecond, kMark, kRecords, kSettle, kWalk };

// Three phases have hot spots: the nodes of frequent tokens, and the transitions between them, which
// thousands of positions ask for at once.  Atomics on one address follow each other, so these phases
// are launched in parts, a small one of the text first (part: in 64ths): the others read what it
// wrote and pass by.  (700 000 tokens of corpus: first ends 175 us in one launch, 70 in two; second
// ones 130, 40; walks 368, 300 in four.)
struct Part { uint32_t lo, hi; };
__host__ __device__ __forceinline__ uint32_t part_of(uint32_t count, uint32_t part)
{
    return part >= 64 ? count : (uint32_t)((uint64_t)count * part / 64);
}

// bulk_agree by a whole wave, 256 tokens a step: every lane compares four.
__device__ __forceinline__ uint32_t wave_agree(const int32_t *tok, uint32_t a, uint32_t b, uint32_t l)
{
    const uint32_t most = (a < b ? a : b) + 1;
    for (; l < most; l += 256) {
        const uint32_t at = l + 4 * lane_id();
        uint32_t upto = at;                              // how far this lane's four agree
        for (uint32_t j = 0; j < 4; j++)
            if (at + j < most && upto == at + j && tok[a - at - j] == tok[b - at - j]) upto++;
        const unsigned long long ends = __ballot(upto != at + 4);
        if (ends) return (uint32_t)__shfl((int)upto, __builtin_ctzll(ends));
    }
    return most;
}

template <Phase P, class Src>
__global__ __launch_bounds__(256) void bulk_phase_kernel(Src src, uint32_t tokens, Part part)
{
    typedef typename Src::Index I;
    BulkSeq<I> q;
    if (!src.get(blockIdx.y, q)) return;
    BulkCtx ctx;
    const uint32_t from = blockIdx.x * 256 + threadIdx.x, step = gridDim.x * 256;
    if constexpr (P == Phase::kCommon) {
        const uint32_t longest = bulk_longest(q, tokens);
        if (longest <= kBulkLong) {
            for (uint32_t c = from; c < (q.n + 7) / 8; c += step)
                bulk_common(q, tokens, 8, c, [&](uint32_t a, uint32_t b, uint32_t l) { return bulk_agree(q.tok, a, b, l); });
            return;
        }
        const uint32_t run = longest / 128, runs = (q.n + run - 1) / run;
        for (uint32_t c = from / 64; c < runs; c += step / 64)
            bulk_common(q, tokens, run, c, [&](uint32_t a, uint32_t b, uint32_t l) { return wave_agree(q.tok, a, b, l); });
    } else if constexpr (P == Phase::kSettle) {
        const auto out = src.store(q);
        const uint32_t states = q.counts[kCntStates];
        // what held working arrays is empty again, the text is the sequence's
        typedef typename Src::Store Store;
        uint4 *wipe;
        size_t wipes;
        if constexpr (sizeof(Store) == sizeof(BulkCorpus) && __is_same(Store, BulkCorpus)) {
            wipe = reinterpret_cast<uint4 *>(out.key);
            wipes = q.n;
            if (from == 0) out.root[(uint32_t)q.tok[0]].dst = 1;
        } else {
            wipe = reinterpret_cast<uint4 *>(out.slots);
            wipes = q.dirty / 16;
            int32_t *const text = src.B.dyn_text + (size_t)q.of * src.B.max_seq_len;
            for (uint32_t i = from; i < q.n; i += step) text[i] = q.tok[i];
        }
        for (size_t i = from; i < wipes; i += step) wipe[i] = make_uint4(kNil, kNil, kNil, kNil);
        for (uint32_t v = from; v < states; v += step) bulk_settle(ctx, q, out, states, v);
    } else if constexpr (P == Phase::kWalk) {
        auto out = src.store(q);
        const uint32_t states = q.counts[kCntStates];
        __shared__ uint32_t list[256], chain[2], total;
        out.chain = chain;
        if (threadIdx.x == 0) { total = 0; chain[0] = kNil; }
        __syncthreads();
        uint32_t made = 0;
        const uint32_t end = part_of(states, part.hi);
        for (uint32_t first = part_of(states, part.lo) + from - threadIdx.x % 64; first < end; first += step) {
            const uint32_t v = first + lane_id();
            BulkWalk w;
            w.i = w.v = w.u = 0;
            w.more = false;
            if (v < end) made += bulk_walk(ctx, q, out, states, v, w);
            for (unsigned long long left = __ballot(w.more); left; left &= left - 1) {
                const int lane = __builtin_ctzll(left);
                const BulkWalk one{(uint32_t)__shfl((int)w.i, lane), (uint32_t)__shfl((int)w.v, lane),
                                   (uint32_t)__shfl((int)w.u, lane), true};
                bulk_long_walk(ctx, q, out, states, one, list + (threadIdx.x & ~63u));
            }
        }
        made = wave_total(made);
        if (made && lane_id() == 0) atomicAdd(&total, made);
        __syncthreads();
        if (threadIdx.x == 0) {
            out.hang(ctx);
            if (total) ctx.add(&q.counts[kCntMade], total);
        }
    } else {
        const IngestTree<I> t = q.tree();
        if constexpr (P == Phase::kParent)
            for (uint32_t w = from; w < q.n / 32 + 1; w += step) q.bits[w] = 0;
        for (uint32_t i = part_of(q.n, part.lo) + from; i < part_of(q.n, part.hi); i += step) {
            if constexpr (P == Phase::kOrder) bulk_order(q, i);
            if constexpr (P == Phase::kInterval) t.interval(ctx, i);
            if constexpr (P == Phase::kRepresent) t.represent(i);
            if constexpr (P == Phase::kParent) t.parent(i);
            if constexpr (P == Phase::kLeaf) t.leaf_of(i);
            if constexpr (P == Phase::kFirst)
                if (!t.template first_end<true, true>(ctx, i)) ctx.bit_or(&q.counts[kCntCorrupt], 1u);
            if constexpr (P == Phase::kSecond) t.template second_end<true>(ctx, i);
            if constexpr (P == Phase::kMark) t.mark_clone(ctx, i);
            if constexpr (P == Phase::kRecords) bulk_records(ctx, q, t, src.store(q), i);
        }
    }
}

// ---- prompts: begin and end -----------------------------------------------------

// The text ends in front of its first token outside the vocabulary; until the end, meta->n says how
// long it is.  One workgroup a sequence; those that are taken make the list.
template <class Src>
__global__ __launch_bounds__(1024) void bulk_begin_kernel(Src src)
{
    __shared__ uint32_t first_bad, before;
    if (!src.taken(blockIdx.x)) return;
    const int b = src.sequence(blockIdx.x);
    const uint32_t count = (uint32_t)(src.offsets[blockIdx.x + 1] - src.offsets[blockIdx.x]), vocab = (uint32_t)src.B.vocab;
    const int32_t *const tok = src.tokens + src.offsets[blockIdx.x];
    uint32_t *const ctl = reinterpret_cast<uint32_t *>(src.B.dyn_text + (size_t)b * src.B.max_seq_len);
    if (threadIdx.x == 0) { first_bad = count; before = 0; }
    if (threadIdx.x < kBulkCtl) ctl[threadIdx.x] = 0;          // (where bulk_place has it)
    __syncthreads();
    for (uint32_t j = threadIdx.x; j < count; j += 1024)
        if ((uint32_t)tok[j] >= vocab) atomicMin(&first_bad, j);
    if (Src::kList)
        for (uint32_t y = threadIdx.x; y < blockIdx.x; y += 1024)
            if (src.taken(y)) atomicAdd(&before, 1u);
    __syncthreads();
    if (threadIdx.x == 0) {
        if (Src::kList) src.list[before].listed = blockIdx.x;
        SeqMeta *const meta = &src.B.meta[b];
        if (first_bad < count) {
            meta->status |= SAM_STATUS_TOKEN_BIT;
            atomicOr(src.B.status, SAM_STATUS_TOKEN_BIT);
        }
        meta->n = first_bad;
        if (first_bad) {
            ctl[kCtlTops] = bulk_levels(first_bad, ctl + kCtlLevel);
            for (uint32_t j = 0; j < kBulkCounts; j++) src.counts(b)[j] = 0;
        }
    }
}

template <class Src>
__global__ __launch_bounds__(64) void bulk_end_kernel(Src src, uint32_t n_seqs)
{
    const uint32_t y = blockIdx.x * 64 + threadIdx.x;
    BulkSeq<typename Src::Index> q;
    if (y >= n_seqs || !src.get(y, q)) return;
    const auto out = src.store(q);
    SeqMeta *const meta = &src.B.meta[q.of];
    if (q.counts[kCntCorrupt]) {
        meta->status |= SAM_STATUS_INTERNAL_BIT;
        atomicOr(src.B.status, SAM_STATUS_INTERNAL_BIT);
        meta->n = 0;                         // nothing of this sequence is valid from here on
        meta->n_states = 1;
        meta->last = 0;
        meta->n_trans = 0;
        return;
    }
    const uint32_t states = q.counts[kCntStates];
    // the last prefix is the last state but for a clone made with it
    uint32_t last = states - 1, len, link, endpos, itok;
    out.load(last, len, link, endpos, itok);
    if (len != q.n) last--;
    out.load(last, len, link, endpos, itok);
    const uint32_t P = link;
    out.load(P, len, link, endpos, itok);
    BulkCtx ctx;
    meta->last = last;
    meta->n_trans = q.counts[kCntMade] + states - 1;
    meta->s2 = P;
    meta->p_len = len; meta->p_link = link; meta->p_endpos = endpos;
    meta->p_head = out.head(ctx, P);
    meta->p_itok = itok; meta->p_idst = out.idst(P);
}

// ---- the corpus's tables ----------------------------------------------------------

__global__ void bulk_check_kernel(const int32_t *tok, uint32_t n, uint32_t vocab, uint32_t *at)
{
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x)
        if ((uint32_t)tok[i] >= vocab) atomicMin(at, i);
}

__global__ void bulk_corpus_begin_kernel(uint32_t *ctl, uint32_t *counts, uint32_t n)
{
    for (uint32_t j = threadIdx.x; j < kBulkCtl; j += blockDim.x) ctl[j] = 0;
    if (threadIdx.x < kBulkCounts) counts[threadIdx.x] = 0;
    __syncthreads();
    if (threadIdx.x == 0) ctl[kCtlTops] = bulk_levels(n, ctl + kCtlLevel);
}

// The transitions by index: of the states that come first in `states`, then of the table's slots.
__device__ __forceinline__ bool corpus_transition(const BulkCorpus &c, uint32_t states, uint64_t i, uint32_t &state,
                                                  uint32_t &token, uint32_t &dst)
{
    if (i < states) {
        const BulkCorpus::State r = c.rec[i];
        if (i == 0 || r.endpos >= c.n) return false;
        state = (uint32_t)i;
        token = (uint32_t)c.tok[r.endpos];
        dst = r.idst;
        return true;
    }
    const uint64_t key = c.key[i - states];
    if (key == ~(uint64_t)0) return false;
    state = (uint32_t)key;
    token = (uint32_t)(key >> 32);
    dst = c.dst[i - states];
    return true;
}

// A key goes into the first bucket on its way that has fewer than eight smaller ones, whatever the
// order in which they come: an insertion takes the place of the largest key of a full bucket if that
// is larger than its own, and goes on with that one.  A slot's key only ever falls, so a key that
// passes a bucket has eight smaller ones there for good.  (The file that a corpus is saved to holds
// this table: it is the same every time.)
__global__ __launch_bounds__(256) void bulk_table_keys_kernel(BulkCorpus c, uint32_t states, unsigned long long *slots,
                                                              uint64_t n_buckets)
{
    const uint64_t all = (uint64_t)states + c.n_slots;
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < all; i += (uint64_t)gridDim.x * 256) {
        uint32_t state, token, dst;
        if (!corpus_transition(c, states, i, state, token, dst)) continue;
        unsigned long long key = (unsigned long long)state | ((unsigned long long)token << 32);
        uint64_t b = bucket_of(hash_key(state, token), n_buckets);
        for (uint64_t left = n_buckets; left;) {
            unsigned long long *const bucket = slots + b * (2 * kBucketSlots);
            unsigned long long most = 0;
            int where = 0;
            for (int j = 0; j < kBucketSlots; j++) {
                const unsigned long long k = __hip_atomic_load(bucket + 2 * j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (k > most) { most = k; where = j; }
            }
            if (most < key) {                                   // eight smaller ones
                b = b + 1 == n_buckets ? 0 : b + 1;
                left--;
                continue;
            }
            if (atomicCAS(bucket + 2 * where, most, key) != most) continue;      // someone was faster: look again
            if (most == ~0ull) break;
            key = most;                                         // it goes on to the next bucket
            b = b + 1 == n_buckets ? 0 : b + 1;
            left--;
        }
    }
}

// The keys of a bucket in rising order, empty slots behind.
__global__ __launch_bounds__(256) void bulk_table_sort_kernel(ulonglong2 *slots, uint64_t n_buckets)
{
    for (uint64_t b = (uint64_t)blockIdx.x * 256 + threadIdx.x; b < n_buckets; b += (uint64_t)gridDim.x * 256) {
        unsigned long long k[kBucketSlots];
#pragma unroll
        for (int j = 0; j < kBucketSlots; j++) k[j] = slots[b * kBucketSlots + j].x;
        if (k[0] == ~0ull && k[1] == ~0ull) continue;
#pragma unroll
        for (int round = 0; round < kBucketSlots; round++)
#pragma unroll
            for (int j = round & 1; j + 1 < kBucketSlots; j += 2)
                if (k[j] > k[j + 1]) { const unsigned long long t = k[j]; k[j] = k[j + 1]; k[j + 1] = t; }
#pragma unroll
        for (int j = 0; j < kBucketSlots; j++) slots[b * kBucketSlots + j].x = k[j];
    }
}

// Targets and their end positions beside the keys.
__global__ __launch_bounds__(256) void bulk_table_targets_kernel(BulkCorpus c, uint32_t states, Slot *slots,
                                                                 uint64_t n_buckets)
{
    const uint64_t all = (uint64_t)states + c.n_slots;
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < all; i += (uint64_t)gridDim.x * 256) {
        uint32_t state, token, dst;
        if (!corpus_transition(c, states, i, state, token, dst)) continue;
        const unsigned long long key = (unsigned long long)state | ((unsigned long long)token << 32);
        uint64_t b = bucket_of(hash_key(state, token), n_buckets);
        bool found = false;
        for (uint64_t left = n_buckets; left && !found; left--) {
            for (int j = 0; j < kBucketSlots && !found; j++) {
                Slot *const s = slots + b * kBucketSlots + j;
                if (*reinterpret_cast<const unsigned long long *>(s) != key) continue;
                s->dst = dst;
                s->w = c.rec[dst].endpos;
                found = true;
            }
            b = b + 1 == n_buckets ? 0 : b + 1;
        }
    }
}

__global__ __launch_bounds__(256) void bulk_corpus_end_kernel(BulkCorpus c, uint32_t states, uint32_t vocab, LinkPair *pairs)
{
    for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < (states > vocab ? states : vocab); i += gridDim.x * 256) {
        if (i < states) {
            const uint32_t link = i ? c.rec[i].link : 0u;
            pairs[i] = LinkPair{link, c.rec[link].len};
            c.rec[i].idst = kNil;
        }
        if (i < vocab && c.root[i].dst) c.root[i].endpos = c.rec[c.root[i].dst].endpos;
    }
}

// ---- launching ----------------------------------------------------------------------

dim3 grid_for(uint64_t count, uint32_t per, uint32_t n_seqs, uint32_t most = 65536)
{
    const uint64_t want = (count + per - 1) / per;
    return dim3((uint32_t)(want < most ? (want ? want : 1) : most), n_seqs);
}

// runs of a text of n tokens, or of any shorter one
uint32_t most_runs(uint32_t n)
{
    const uint32_t tiles = (n + kBulkTile - 1) / kBulkTile;
    return tiles < kBulkBlocks ? tiles : kBulkBlocks;
}

// Everything between a text and its transitions, for texts of up to n tokens.
template <class Src>
void launch_phases(const Src &src, uint32_t n, uint32_t n_seqs, const BulkSort &sort, hipStream_t stream)
{
#define SAM_PART(P, COUNT, LO, HI)                                                                               \
    hipLaunchKernelGGL((bulk_phase_kernel<Phase::P, Src>), grid_for(((COUNT) * (uint64_t)(HI - LO) + 63) / 64, 256, n_seqs), \
                       dim3(256), 0, stream, src, sort.tokens, Part{LO, HI})
#define SAM_PHASE(P, COUNT) SAM_PART(P, COUNT, 0, 64)
#define SAM_PARTS(P, COUNT) do { SAM_PART(P, COUNT, 0, 3); SAM_PART(P, COUNT, 3, 64); } while (0)
    SAM_PHASE(kOrder, n);
    SAM_PHASE(kCommon, n / 8 + 1);
    hipLaunchKernelGGL((bulk_minima_kernel<Src>), dim3((ingest_first_mins(n) + 4672 + kSort - 1) / kSort, n_seqs), dim3(kSort),
                       0, stream, src);
    if (bulk_levels(n, nullptr) > 4)
        hipLaunchKernelGGL((bulk_upper_minima_kernel<Src>), dim3(1, n_seqs), dim3(kSort), 0, stream, src);
    SAM_PHASE(kInterval, n);
    SAM_PHASE(kRepresent, n);
    SAM_PHASE(kParent, n);
    SAM_PHASE(kLeaf, n);
    SAM_PARTS(kFirst, n);
    SAM_PARTS(kSecond, n);
    SAM_PHASE(kMark, n);
    const dim3 runs(most_runs(n / 32 + 1), n_seqs);
    if (runs.x > 1) hipLaunchKernelGGL((bulk_clone_sums_kernel<Src>), runs, dim3(kSort), 0, stream, src);
    hipLaunchKernelGGL((bulk_clone_ranks_kernel<Src>), runs, dim3(kSort), 0, stream, src);
    SAM_PHASE(kRecords, n);
    SAM_PHASE(kSettle, 2 * (uint64_t)n);
    SAM_PART(kWalk, 2 * (uint64_t)n, 0, 1);
    SAM_PART(kWalk, 2 * (uint64_t)n, 1, 4);
    SAM_PART(kWalk, 2 * (uint64_t)n, 4, 16);
    SAM_PART(kWalk, 2 * (uint64_t)n, 16, 64);
#undef SAM_PARTS
#undef SAM_PHASE
#undef SAM_PART
}

template <class Src>
void launch_sort(const Src &src, uint32_t n, uint32_t n_seqs, const BulkSort &sort, hipStream_t stream)
{
    const dim3 runs(most_runs(n), n_seqs);
    for (uint32_t pass = 0; pass < sort.passes; pass++) {
        hipLaunchKernelGGL((bulk_hist_kernel<Src>), runs, dim3(kSort), 0, stream, src, sort, pass);
        hipLaunchKernelGGL((bulk_scatter_kernel<Src>), runs, dim3(kSort), 0, stream, src, sort, pass);
    }
    hipLaunchKernelGGL((bulk_groups_kernel<Src>), runs, dim3(kSort), 0, stream, src, (sort.passes - 1) & 1);
}

template <class Src>
void launch_round(const Src &src, uint32_t n, uint32_t n_seqs, const BulkSort &sort, uint32_t round, uint32_t h,
                  hipStream_t stream)
{
    const uint32_t first = (sort.passes - 1) & 1, large = n / kBulkLarge < 64 ? n / kBulkLarge + 1 : (n < (1u << 20) ? 64 : 1024);
    hipLaunchKernelGGL((bulk_gather_kernel<Src>), grid_for(n, 256, n_seqs), dim3(256), 0, stream, src, first, round, h);
    dim3 g = grid_for(n, kSort, n_seqs);
    // (workgroups go to the XCDs in turn: an odd number of them for a text, or all texts' first ones, which take
    // the large groups, would meet on one of the eight)
    g.x = (g.x + large) | 1;
    hipLaunchKernelGGL((bulk_rank_kernel<Src>), g, dim3(kSort), 0, stream, src, first, round, h, large);
}

template <class Src>
hipError_t bulk_prompts(const BatchView &B, const int32_t *seq_map, int n_seqs, int n_listed, const int32_t *tokens,
                        const int64_t *offsets, uint32_t lds_tokens, uint32_t most, bool begin, hipStream_t stream)
{
    if (begin) {
        hipLaunchKernelGGL((bulk_begin_kernel<Src>), dim3(n_seqs), dim3(1024), 0, stream,
                           Src{B, seq_map, tokens, offsets, lds_tokens, most, B.meta});
        return hipGetLastError();
    }
    // workgroups find their sequence in the grid's second index, which ends at 65535
    const int all = Src::kList ? n_listed : n_seqs;
    for (int at = 0; at < all; at += 65535) {
        const int count = all - at < 65535 ? all - at : 65535;
        Src src{B, seq_map, tokens, offsets, lds_tokens, most, B.meta + at};
        if (!Src::kList) {
            src.offsets += at;
            if (seq_map) {
                src.seq_map += at;
            } else {                               // sequences at .. : the batch as if it began there
                src.B.dyn_text += (size_t)at * B.max_seq_len;
                src.B.dyn_rec = src.rec(at);
                src.B.dyn_slots = src.slots(at);
                src.B.meta += at;
            }
        }
        const BulkSort sort = bulk_sort_for((uint32_t)B.vocab, 32);
        launch_sort(src, most, (uint32_t)count, sort, stream);
        uint32_t round = 0;
        for (uint32_t h = sort.tokens; h < most; h *= 2, round++)
            launch_round(src, most, (uint32_t)count, sort, round, h, stream);
        launch_phases(src, most, (uint32_t)count, sort, stream);
        hipLaunchKernelGGL((bulk_end_kernel<Src>), dim3((count + 63) / 64), dim3(64), 0, stream, src, (uint32_t)count);
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_bulk_prompts(const BatchView &B, const int32_t *seq_map, int n_seqs, int n_listed, const int32_t *tokens,
                               const int64_t *offsets, uint32_t lds_tokens, uint32_t most, bool begin, hipStream_t stream)
{
#define SAM_BULK(L, I, LISTED) \
    bulk_prompts<PromptSource<L, I, LISTED>>(B, seq_map, n_seqs, n_listed, tokens, offsets, lds_tokens, most, begin, stream)
    if (B.compact) return n_listed ? SAM_BULK(IngestCompact, uint16_t, true) : SAM_BULK(IngestCompact, uint16_t, false);
    return n_listed ? SAM_BULK(IngestWide, uint32_t, true) : SAM_BULK(IngestWide, uint32_t, false);
#undef SAM_BULK
}

hipError_t bulk_check(const int32_t *tok, uint32_t n, uint32_t vocab, uint32_t *at, hipStream_t stream)
{
    hipLaunchKernelGGL(bulk_check_kernel, grid_for(n, 256, 1, 4096), dim3(256), 0, stream, tok, n, vocab, at);
    return hipGetLastError();
}

hipError_t bulk_corpus(const int32_t *tok, uint32_t n, uint32_t vocab, RootEnt *root, const BulkWork &w,
                       uint32_t *n_states, uint64_t *n_trans, bool *gave_up, hipStream_t stream)
{
    // to sort a group beyond this in full keeps one workgroup busy for a tenth of a second and more, each round
    constexpr uint32_t kMostLarge = 1u << 23;
    const CorpusSource src{tok, n, w, root};
    uint32_t ctl[kBulkCtl], counts[kBulkCounts];
    hipError_t e;
    *gave_up = false;
    hipLaunchKernelGGL(bulk_corpus_begin_kernel, dim3(1), dim3(256), 0, stream, reinterpret_cast<uint32_t *>(w.third), w.counts, n);
    const BulkSort sort = bulk_sort_for(vocab, 64);
    launch_sort(src, n, 1, sort, stream);
    uint32_t round = 0;
    for (uint64_t h = sort.tokens; h < n; h *= 2, round++) {
        if (n > kMostLarge) {
            if ((e = hipMemcpyAsync(ctl, w.third, sizeof(ctl), hipMemcpyDeviceToHost, stream)) != hipSuccess ||
                (e = hipStreamSynchronize(stream)) != hipSuccess)
                return e;
            if (!ctl[kCtlActive + round]) break;
            if (ctl[kCtlLargest] > kMostLarge) { *gave_up = true; return hipSuccess; }
        }
        launch_round(src, n, 1, sort, round, (uint32_t)h, stream);
    }
    launch_phases(src, n, 1, sort, stream);
    if ((e = hipGetLastError()) != hipSuccess ||
        (e = hipMemcpyAsync(counts, w.counts, sizeof(counts), hipMemcpyDeviceToHost, stream)) != hipSuccess ||
        (e = hipStreamSynchronize(stream)) != hipSuccess)
        return e;
    if (counts[kCntCorrupt]) *gave_up = true;
    *n_states = counts[kCntStates];
    *n_trans = (uint64_t)counts[kCntMade] + counts[kCntStates] - 1;
    return hipSuccess;
}

hipError_t bulk_corpus_tables(const int32_t *tok, uint32_t n, uint32_t vocab, uint32_t n_states, RootEnt *root,
                              const BulkWork &w, Slot *slots, uint64_t n_buckets, LinkPair *pairs, hipStream_t stream)
{
    const BulkCorpus c = CorpusSource{tok, n, w, root}.table();
    const dim3 all = grid_for((uint64_t)n_states + c.n_slots, 256, 1, 16384);
    hipLaunchKernelGGL(bulk_table_keys_kernel, all, dim3(256), 0, stream, c, n_states, (unsigned long long *)slots, n_buckets);
    hipLaunchKernelGGL(bulk_table_sort_kernel, grid_for(n_buckets, 256, 1, 16384), dim3(256), 0, stream, (ulonglong2 *)slots, n_buckets);
    hipLaunchKernelGGL(bulk_table_targets_kernel, all, dim3(256), 0, stream, c, n_states, slots, n_buckets);
    hipLaunchKernelGGL(bulk_corpus_end_kernel, grid_for(n_states > vocab ? n_states : vocab, 256, 1, 16384), dim3(256), 0, stream,
                       c, n_states, vocab, pairs);
    return hipGetLastError();
}

}  // namespace sam
