// gfx950 kernel that takes the prompts of fresh sequences whole (arxiv 2411.10666,
// Section 3.1: the dynamic automaton over prompt and generated tokens alike).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "sam_bulk_launch.h"
#include "sam_ingest.h"
#include "sam_prompt.h"
#include "sam_walk.h"

namespace sam {

// Extending a sequence token by token takes 0.6 to 1.2 us a token whatever the chip has
// free, so a prompt of 3000 tokens took 1.8 ms.  Built whole, by one workgroup with its
// working arrays in LDS (27 bytes a token, 16-bit indices), the bound is chains of dependent
// LDS and table accesses between about sixty barriers: the LDS pipeline is busy for 28 % of
// the cycles, the vector ALUs for 37 %.  Measured, sam_batch_reset: one prompt of 6000 tokens 222 us,
// 64 of 2048 137 us (1.2 ms token by token), 1024 of 2048 465 us, 1024 of 6000 1.19 ms (5.3 ms).  With
// the arrays in the sequence's own tables (prompts beyond LDS, where the whole chip does not take them,
// see launch_ingest) the bound is the rate at which one compute unit gets
// scattered requests to the L2 through, 0.5 to 0.6 a nanosecond: 12 prompts of 40 001 tokens
// 3.4 to 9.8 ms by their text (46 ms).  Of the 165 us that one workgroup needs for 6000 tokens, the sort takes 75, the
// intervals 19 and the transitions 61 (a compare-and-swap in the slot table each).  Two parts
// took longer: the nearest smaller values scanned in runs of 32 (130 us; now a tree of
// minima of 8, one 16-byte read a level, 19) and the transitions walking the records in
// memory instead of their copies in LDS (122 us, now 61).  Lanes that go on with the
// next position as soon as theirs has ended, instead of waiting for the longest path of their
// wave, took 218 against 218 us for one prompt of 6000 tokens, and 1.22 against 1.18 ms for 1024.

template <int T>
struct PromptCtx {
    static constexpr uint32_t kThreads = T;
    uint32_t tid;
    uint32_t *wsum;            // [T / 64]

    template <class F>
    __device__ __forceinline__ void each(uint32_t n, F f)
    {
        for (uint32_t i = tid; i < n; i += T) f(i);
    }
    template <class F>
    __device__ __forceinline__ void each_full(uint32_t n, F f)     // whole waves
    {
        for (uint32_t i = tid; i - tid < n; i += T) f(i, i < n);
    }
    // one wave for each index, with 64 words of part[] to itself
    template <class F>
    __device__ __forceinline__ void each_wave(uint32_t n, uint32_t *part, F f)
    {
        for (uint32_t i = tid / 64; i < n; i += T / 64) f(i, part + (tid & ~63u));
    }
    template <class F>
    __device__ __forceinline__ void lanes(F f) { f(tid & 63); }
    __device__ __forceinline__ void wave_sync()
    {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    }
    __device__ __forceinline__ void sync() { __syncthreads(); }
    template <class U>
    __device__ __forceinline__ U cas(U *p, U expected, U v)
    {
        __hip_atomic_compare_exchange_strong(p, &expected, v, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_WORKGROUP);
        return expected;
    }
    template <class U>
    __device__ __forceinline__ U add(U *p, U v)
    {
        return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __device__ __forceinline__ uint32_t lower(uint32_t *p, uint32_t v)
    {
        return __hip_atomic_fetch_min(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __device__ __forceinline__ void raise(uint32_t *p, uint32_t v)
    {
        __hip_atomic_fetch_max(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __device__ __forceinline__ void bit_or(uint32_t *p, uint32_t v)
    {
        __hip_atomic_fetch_or(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __device__ __forceinline__ uint32_t exch(uint32_t *p, uint32_t v)
    {
        return __hip_atomic_exchange(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __device__ __forceinline__ uint32_t fresh(uint32_t *p)
    {
        return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // a value that all threads have, as a scalar
    __device__ __forceinline__ uint32_t uniform(uint32_t x)
    {
        return (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
    }
    __device__ __forceinline__ uint32_t mulhi(uint32_t a, uint32_t b) { return __umulhi(a, b); }
    __device__ __forceinline__ uint32_t popc(uint32_t x) { return (uint32_t)__popc(x); }
    __device__ __forceinline__ uint32_t first(uint32_t x) { return (uint32_t)__builtin_ctz(x); }
    __device__ __forceinline__ uint32_t log2(uint32_t x) { return 31u - (uint32_t)__clz((int)x); }
    // sum over the lower lanes and this one
    __device__ __forceinline__ uint32_t wave_sums(uint32_t v)
    {
        for (int d = 1; d < 64; d *= 2) {
            const uint32_t below = (uint32_t)__shfl_up((int)v, d);
            if ((tid & 63) >= (uint32_t)d) v += below;
        }
        return v;
    }
    // where this lane's v places start in a counter that all lanes of the wave add to
    __device__ __forceinline__ uint32_t wave_add(uint32_t *p, uint32_t v)
    {
        const uint32_t upto = wave_sums(v);
        uint32_t base = 0;
        if ((tid & 63) == 63 && upto) base = add(p, upto);
        return (uint32_t)__shfl((int)base, 63) + upto - v;
    }
    // f(times) for a key: once for all lanes of the wave that have the same one, if they are 8 or
    // more, else once for each.  Atomics of a workgroup on one address of device memory follow
    // each other, and in a run of one token all pairs of a round are the same: 64 prompts of 9000
    // equal tokens took 4.6 ms with an insertion for each position, 1.1 with this.  (In LDS the
    // same brought 3 % for such texts and cost others 4 %.)
    template <class U, class F>
    __device__ __forceinline__ uint32_t together(U key, F f)
    {
        uint32_t r = 0;
        for (bool again = true; again;) {
            U first = (U)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)key);
            if constexpr (sizeof(U) == 8)
                first |= (U)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(key >> 32)) << 32;
            const uint64_t same = __ballot(key == first);
            const uint32_t count = (uint32_t)__popcll(same);
            const int lead = __builtin_ctzll(same);
            const bool shared = count >= 8;
            again = shared && key != first;
            if (!shared || (int)(tid & 63) == lead) r = f(shared ? count : 1u);
            if (key == first && shared) r = (uint32_t)__builtin_amdgcn_readlane((int)r, lead);
        }
        return r;
    }
    // part[i] becomes the sum of the entries before it; thread i reads entry i
    __device__ __forceinline__ void exclusive_sums(uint32_t *part)
    {
        const uint32_t v = part[tid], upto = wave_sums(v);
        if ((tid & 63) == 63) wsum[tid >> 6] = upto;
        __syncthreads();
        uint32_t before = 0;
        for (uint32_t w = 0; w < (tid >> 6); w++) before += wsum[w];
        part[tid] = before + upto - v;
    }
};

// How many tokens at the end of the prompt stand in front of corpus position `end` too, `known` of
// them known to: 64 a round trip (256 a round trip took less for long passages, but all prompts 1 %
// more, by the registers that it takes in the same kernel as the builds).
__device__ __forceinline__ uint32_t agree_back(const StaticView &S, const int32_t *tok, uint32_t n,
                                               uint32_t end, uint32_t known, int lane)
{
    const uint32_t most = n < end ? n : end;
    for (uint32_t base = known; base < most; base += 64) {
        const uint32_t j = base + lane, back = j < most ? j : most - 1;
        const unsigned long long differ = __ballot(tok[n - 1 - back] != S.text[end - 1 - back]);
        if (differ) {
            const uint32_t at = base + (uint32_t)__builtin_ctzll(differ);
            return uni(at < most ? at : most - 1);
        }
    }
    return most;
}

// The static cursor after a prompt belongs to the longest suffix of the prompt that occurs
// in the corpus, so the walk need not start at the first token: started at the root w
// tokens before the end it finds the longest such suffix of at most w tokens, and if that is
// shorter than w it is the one looked for.  48 tokens do for most prompts, but a batch waits for
// its longest walk.  If they match throughout, the corpus is compared with the prompt backwards
// from where they occur first, and the second window is one token longer than what agrees.  It is
// full too only if the prompt's end occurs elsewhere with more in front of it: further windows
// are at least four times as long.  Where more than half of the prompt agrees all of it is walked:
// a passage of the corpus costs one walk over it (0.15 to 0.3 us a token, 0.5 to 0.7 where
// matches break off).  (Windows of 48, 192, 768 ... tokens, each from the root: 256 passages of 3073
// tokens 2.2 ms, now 1.0 (token by token 1.9); 256 prompts of 1024 with matches of up to 272: 0.50,
// now 0.18.)
__device__ __forceinline__ void static_tail(const StaticView &S, const int32_t *tok, uint32_t n,
                                            uint32_t vocab, int lane, uint32_t &s, uint32_t &l,
                                            uint32_t &e, uint32_t &fault, bool use_asm)
{
    for (uint32_t w = n < 48 ? n : 48;;) {
        s = 0; l = 0; e = 0;
        static_feed(S, tok + (n - w), w, vocab, lane, s, l, e, fault, use_asm);
        if (uni(l) < w || w == n || fault) return;
        const uint32_t next = agree_back(S, tok, n, uni(e) & ~kWideBit, w, lane) + 1;
        w = w == 48 || next > 4 * w ? next : 4 * w;
        if (w > n || next > n / 2) w = n;
    }
}

// Fresh sequences (just reset) take their prompts.  Workgroups 0 .. n_static-1 walk the
// corpus automaton, one wave per sequence; workgroup n_static + i builds the automaton of prompt
// i's sequence (n_static is a multiple of 8: where all sequences of a batch take prompts, in
// their order, it runs on the XCD on which their steps will find the tables).  The walks
// reserve the builds' LDS without using it; beside the builds they cost little (1024 prompts
// of 2048 tokens 465 us without a corpus, 447 over one of 4 M tokens, whose prompts repeat less).  A
// token outside the vocabulary ends its prompt.
template <bool kCompact, bool kAsm, int T>
__global__ __launch_bounds__(T) void sam_prompt_kernel(StaticView S, BatchView B,
                                                          const int32_t *__restrict__ seq_map,
                                                          int n_seqs, int n_static,
                                                          const int32_t *__restrict__ tokens,
                                                          const int64_t *__restrict__ offsets,
                                                          uint32_t lds_tokens, uint32_t max_tokens,
                                                          uint32_t bulk_tokens)
{
    extern __shared__ __align__(16) char lds[];
    __shared__ uint32_t bad, wsum[T / 64];
    const uint32_t vocab = (uint32_t)B.vocab;
    const int lane = threadIdx.x & 63;
    const bool walks = (int)blockIdx.x < n_static;
    const int i = walks ? (int)blockIdx.x * (T / 64) + (int)(threadIdx.x >> 6)
                        : (int)blockIdx.x - n_static;
    if (i >= n_seqs) return;
    const int b = seq_map ? seq_map[i] : i;
    SeqMeta *meta = &B.meta[b];
    const int32_t *tok = tokens + offsets[i];
    const int64_t count = offsets[i + 1] - offsets[i];
    if (count <= 0) return;
    if (count > (int64_t)B.max_seq_len || count > (int64_t)max_tokens) {
        if (!walks && threadIdx.x == 0) {
            meta->status |= SAM_STATUS_CAPACITY_BIT;
            atomicOr(B.status, SAM_STATUS_CAPACITY_BIT);
        }
        return;
    }
    const bool bulk = bulk_tokens && bulk_takes(B, count, lds_tokens, bulk_tokens);
    if (!walks && bulk) return;
    uint32_t n = (uint32_t)count;
    if (walks) {
        uint32_t first = n;
        if (bulk) first = uni(meta->n);                  // found by then, by a whole workgroup
        else for (uint32_t base = 0; base < n && first == n; base += 256) {
            uint32_t at = n;
#pragma unroll
            for (int u = 3; u >= 0; u--) {
                const uint32_t j = base + 64 * u + lane;
                if (j < n && (uint32_t)tok[j] >= vocab) at = j;
            }
            if (__any(at < n))
                for (int d = 32; d; d /= 2) {
                    const uint32_t other = (uint32_t)__shfl_xor((int)at, d);
                    at = other < at ? other : at;
                }
            first = uni(at);
        }
        n = first;
        uint32_t s = 0, l = 0, e = 0, fault = 0;
        if (n) static_tail(S, tok, n, vocab, lane, s, l, e, fault, kAsm);
        if (lane == 0) {
            meta->s1 = s; meta->l1 = l; meta->e1 = e;
            if (fault & SAM_STATUS_INTERNAL_BIT) atomicOr(B.status, SAM_STATUS_INTERNAL_BIT);
        }
        return;
    }

    if (threadIdx.x == 0) bad = n;
    __syncthreads();
    for (uint32_t j = threadIdx.x; j < n; j += T)
        if ((uint32_t)tok[j] >= vocab) atomicMin(&bad, j);
    __syncthreads();
    const uint32_t first_bad = bad;
    if (first_bad < n && threadIdx.x == 0) {
        meta->status |= SAM_STATUS_TOKEN_BIT;
        atomicOr(B.status, SAM_STATUS_TOKEN_BIT);
    }
    n = first_bad;
    if (n == 0) return;
    typedef typename std::conditional<kCompact, IngestCompact, IngestWide>::type IL;
    typedef typename std::conditional<kCompact, uint16_t, uint32_t>::type I;
    typedef typename std::conditional<kCompact, uint32_t, uint64_t>::type K;
    const IngestSeq q{tok, n, B.dyn_text + (size_t)b * B.max_seq_len,
                      reinterpret_cast<char *>(B.dyn_rec) +
                          (size_t)b * B.max_states * (kCompact ? sizeof(DynRecCompact) : sizeof(DynRec)),
                      reinterpret_cast<char *>(B.dyn_slots) + (size_t)b * B.dyn_buckets * 128, B.dyn_buckets};
    PromptCtx<T> ctx{threadIdx.x, wsum};
    uint32_t *small;
    if (n <= lds_tokens) {
        IngestArrays<uint16_t, uint32_t> A;
        ingest_place_lds(A, lds, n);
        small = A.small;
        ingest_build<IL, true>(ctx, q, A);
    } else {
        IngestArrays<I, K> A;
        ingest_place_tables(A, q, lds, n);
        small = A.small;
        ingest_build<IL, false>(ctx, q, A);
    }
    if (threadIdx.x == 0) {
        if (small[121]) {
            meta->status |= SAM_STATUS_INTERNAL_BIT;
            atomicOr(B.status, SAM_STATUS_INTERNAL_BIT);
            return;                          // nothing of this sequence is valid from here on
        }
        const uint32_t last = small[123], P = IL::link(q.rec, last);
        uint32_t len, link, endpos, itok;
        IL::load(q.rec, P, len, link, endpos, itok);
        meta->n = n; meta->n_states = small[124]; meta->last = last; meta->n_trans = small[125];
        meta->s2 = P;
        meta->p_len = len; meta->p_link = link; meta->p_endpos = endpos;
        meta->p_head = IL::head(ctx, q.rec, P);
        meta->p_itok = itok; meta->p_idst = IL::idst(q.rec, P);
    }
}

hipError_t launch_ingest(const StaticView &S, const BatchView &B, const int32_t *seq_map,
                         int n_seqs, const int32_t *tokens, const int64_t *offsets,
                         const int64_t *host_offsets, int64_t most, hipStream_t stream)
{
    auto one_by_one = [&] {
        return launch_feed(S, B, seq_map, n_seqs, tokens, offsets, nullptr, nullptr, nullptr,
                           nullptr, nullptr, stream);
    };
    auto prompt = [&](int i) { return host_offsets[i + 1] - host_offsets[i]; };
    PromptSizes sizes = {n_seqs, 0, host_offsets[n_seqs] - host_offsets[0], 0};
    for (int i = 0; i < n_seqs; i++)
        if (prompt(i) > sizes.longest) sizes.longest = prompt(i);
    sizes.most = most > sizes.longest ? most : sizes.longest;
    int dev = 0, lds_limit = 0, n_cu = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess)
        e = hipDeviceGetAttribute(&lds_limit, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
    if (e == hipSuccess)
        e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    const size_t room = (size_t)lds_limit - 256;             // the kernel's own words
    // the most tokens whose working arrays fit
    uint32_t fit = 0, over = kIngestIdx16 + 1;
    while (over - fit > 1) {
        const uint32_t mid = (fit + over) / 2;
        if (ingest_lds_bytes(mid) <= room) fit = mid; else over = mid;
    }
    int64_t n_beyond = 0;
    if (sizes.longest > fit)
        for (int i = 0; i < n_seqs; i++) n_beyond += prompt(i) > fit;
    if (!prompts_whole(sizes, n_beyond, n_cu)) return one_by_one();
    const uint32_t max_tokens = (uint32_t)sizes.most;
    uint32_t lds_tokens = (uint32_t)sizes.longest < fit ? (uint32_t)sizes.longest : fit;
    size_t bytes = ingest_lds_bytes(lds_tokens);
    if (max_tokens > lds_tokens) {
        const size_t small = B.compact ? ingest_small_bytes<uint16_t>(max_tokens, true)
                                       : ingest_small_bytes<uint32_t>(max_tokens, true);
        bytes = small > bytes ? small : bytes;
        const size_t rec_bytes = (size_t)B.max_states * (B.compact ? sizeof(DynRecCompact) : sizeof(DynRec)),
                     slot_bytes = (size_t)B.dyn_buckets * 128;
        if (!(B.compact ? ingest_tables_fit<uint16_t, uint32_t>(max_tokens, rec_bytes, slot_bytes)
                        : ingest_tables_fit<uint32_t, uint64_t>(max_tokens, rec_bytes, slot_bytes)) || bytes > room) {
            // (small tables have too little room beside the fixed parts)
            if (max_tokens > fit) return one_by_one();
            lds_tokens = max_tokens;
            bytes = ingest_lds_bytes(lds_tokens);
        }
    }
    // Prompts beyond LDS are built by the whole chip, phase by phase, wherever their tables have room for
    // that: one workgroup each is bound by the scattered accesses of its compute unit even where there
    // are more of them than units.  sam_batch_reset, chip / workgroups, ms, tokens
    // = 32 000 u^5 of a uniform u:
    //   1 x 6500  0.30 / 0.46    1 x 16 000  0.35 / 1.2    1 x 100 000  0.60 / 8.2    12 x 40 000  0.65 / 3.3
    //   64 x 30 000  1.5 / 3.0   256 x 9000  1.38 / 1.38   600 x 8000  2.5 / 2.9
    // (period of 150: 1 x 6500 0.47 / 1.1, 12 x 40 000 1.4 / 9.4, 600 x 8000 3.6 / 7.1; of one token only:
    // 1 x 6500 0.58 / 0.64, 12 x 40 000 1.6 / 5.2, 256 x 9000 1.67 / 1.55, 600 x 8000 2.6 / 3.1; that and another token:
    // 1 x 6500 1.07 / 2.18, 12 x 40 001 4.4 / 14.9, 600 x 8000 3.4 / 9.0; u^3 with copies of up to 200 tokens: 12 x 40 001
    // 0.96 / 6.9).
    // The launches cover the prompts that are taken, which the begin kernel lists (one of 7000 among 1279 of 64
    // tokens: 0.44 ms, of 100 000 1.5; with workgroups for all prompts 0.79 and 8.3; one workgroup each
    // 0.51 and 8.9).  Few of them that one workgroup each builds while the others are built are left to
    // that: the chip's phases follow the others' builds, and take 0.3 ms and more (chip / workgroups, ms, one of
    // 6500 tokens among 1024 of 500 0.46 / 0.49, of 2000 0.66 / 0.58, of 4000 0.97 / 0.73; one of 9000 0.48 /
    // 0.67, 0.66 / 0.76, 0.96 / 0.90; 64 of 6500 0.62 / 0.73, 0.82 / 0.91, 1.13 / 1.24).
    // (A call that may be captured covers all prompts, by the host's longest: replayed with longer ones
    // it leaves those to one workgroup each.)
    uint32_t bulk_tokens = n_beyond > 0 && lds_tokens >= kBulkLdsTokens && !B.no_bulk ? (uint32_t)sizes.longest : 0u;
    int n_listed = 0;
    if (bulk_tokens && most == 0) {
        int64_t others = sizes.total;
        for (int i = 0; i < n_seqs; i++)
            if (bulk_takes(B, prompt(i), lds_tokens, bulk_tokens)) {
                n_listed++;
                others -= prompt(i);
            }
        if (n_listed == 0 || (n_listed < 32 && sizes.longest < 4000 + others / 800)) bulk_tokens = n_listed = 0;
        if (n_listed == n_seqs) n_listed = 0;
    }
    if (bulk_tokens && (e = launch_bulk_prompts(B, seq_map, n_seqs, n_listed, tokens, offsets, lds_tokens, bulk_tokens, true,
                                                stream)) != hipSuccess)
        return e;
    // workgroups for the corpus: a wave each sequence, a multiple of 8 workgroups
    auto walks = [&](int waves) { return B.has_static ? (((n_seqs + waves - 1) / waves + 7) & ~7) : 0; };
    const int threads = short_prompts(sizes, walks(16), n_cu) ? 256 : 1024, n_static = walks(threads / 64);
#define SAM_LAUNCH_PROMPT_T(COMPACT, ASM, T)                                                     \
    hipLaunchKernelGGL((sam_prompt_kernel<COMPACT, ASM, T>), dim3(n_static + n_seqs), dim3(T),    \
                       bytes, stream, S, B, seq_map, n_seqs, n_static, tokens, offsets,          \
                       lds_tokens, max_tokens, bulk_tokens)
#define SAM_LAUNCH_PROMPT(COMPACT, ASM)                                                          \
    do {                                                                                        \
        if (threads == 256) SAM_LAUNCH_PROMPT_T(COMPACT, ASM, 256);                              \
        else SAM_LAUNCH_PROMPT_T(COMPACT, ASM, 1024);                                            \
    } while (0)
    const bool cxx = B.no_asm || (S.n_buckets >> 32);
    if (B.compact) {
        if (cxx) SAM_LAUNCH_PROMPT(true, false); else SAM_LAUNCH_PROMPT(true, true);
    } else {
        if (cxx) SAM_LAUNCH_PROMPT(false, false); else SAM_LAUNCH_PROMPT(false, true);
    }
#undef SAM_LAUNCH_PROMPT
#undef SAM_LAUNCH_PROMPT_T
    if ((e = hipGetLastError()) != hipSuccess || !bulk_tokens) return e;
    return launch_bulk_prompts(B, seq_map, n_seqs, n_listed, tokens, offsets, lds_tokens, bulk_tokens, false, stream);
}

}  // namespace sam
