// A prompt's automaton built whole (sam_ingest.h, its phases run one after the other on the
// CPU) against the token-by-token host builder: ids, lengths, links, end positions and every
// transition.  The tables and the LDS block have exactly the sizes that the library gives them:
// an access outside one of them is seen by AddressSanitizer.  The working arrays lie in there one
// behind the other; an access past the end of one lands in the next and shows, if at all,
// as a difference.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <random>
#include <string>
#include <vector>

#include "../paper_2411_10666_amd/csrc/sam_host.h"
#include "../paper_2411_10666_amd/csrc/sam_ingest.h"

using namespace sam;

template <uint32_t T>
struct CpuCtx {
    static constexpr uint32_t kThreads = T;
    uint32_t widest = 0;                   // the most indices that a phase runs over
    uint32_t swaps = 0, most_swaps = 0;    // compare-and-swaps that one index makes, one after the other
    template <class F> void each(uint32_t n, F f)
    {
        if (n > widest) widest = n;
        for (uint32_t i = 0; i < n; i++) {
            swaps = 0;
            f(i);
            if (swaps > most_swaps) most_swaps = swaps;
        }
    }
    template <class F> void each_wave(uint32_t n, uint32_t *part, F f) { for (uint32_t i = 0; i < n; i++) f(i, part); }
    template <class F> void lanes(F f) { for (uint32_t i = 0; i < 64; i++) f(i); }
    void wave_sync() {}
    template <class U, class F> uint32_t together(U, F f) { return f(1); }
    template <class F> void each_full(uint32_t n, F f) { for (uint32_t i = 0; i < n; i++) f(i, true); }
    void sync() {}
    template <class U> U cas(U *p, U expected, U v) { swaps++; const U old = *p; if (old == expected) *p = v; return old; }
    template <class U> U add(U *p, U v) { const U old = *p; *p = (U)(old + v); return old; }
    uint32_t lower(uint32_t *p, uint32_t v) { const uint32_t old = *p; if (v < old) *p = v; return old; }
    void raise(uint32_t *p, uint32_t v) { if (v > *p) *p = v; }
    void bit_or(uint32_t *p, uint32_t v) { *p |= v; }
    uint32_t exch(uint32_t *p, uint32_t v) { const uint32_t old = *p; *p = v; return old; }
    uint32_t fresh(uint32_t *p) { return *p; }
    uint32_t uniform(uint32_t x) { return x; }
    uint32_t mulhi(uint32_t a, uint32_t b) { return (uint32_t)(((uint64_t)a * b) >> 32); }
    uint32_t popc(uint32_t x) { return (uint32_t)__builtin_popcount(x); }
    uint32_t first(uint32_t x) { return (uint32_t)__builtin_ctz(x); }
    uint32_t log2(uint32_t x) { return 31u - (uint32_t)__builtin_clz(x); }
    uint32_t wave_add(uint32_t *p, uint32_t v) { return add(p, v); }
    void exclusive_sums(uint32_t *part)
    {
        uint32_t sum = 0;
        for (uint32_t i = 0; i < T; i++) { const uint32_t v = part[i]; part[i] = sum; sum += v; }
    }
};

static int bad(const char *what, uint32_t n, uint32_t at)
{
    printf("%s differs: %u tokens, at %u\n", what, n, at);
    return 1;
}

struct Aligned {
    void *p;
    explicit Aligned(size_t bytes, int fill) : p(aligned_alloc(128, (bytes + 127) / 128 * 128)) { memset(p, fill, bytes); }
    ~Aligned() { free(p); }
};

template <class IL, bool kLds, class I, class K, uint32_t T>
static int one(const std::vector<int32_t> &x, int32_t vocab, uint32_t max_seq_len)
{
    const uint32_t n = (uint32_t)x.size();
    constexpr bool compact = IL::kSlots == 16;
    const size_t rec_bytes = (size_t)(2 * max_seq_len + 2) * (compact ? sizeof(DynRecCompact) : sizeof(DynRec));
    const size_t slot_bytes = (size_t)dynamic_slots_for(max_seq_len) * (compact ? sizeof(SlotCompact) : sizeof(Slot));
    const uint32_t n_buckets = (uint32_t)(slot_bytes / 128);
    // the library leaves such prompts to the token-by-token kernel; long ones always fit
    if (!kLds && !ingest_tables_fit<I, K>(n, rec_bytes, (size_t)n_buckets * 128))
        return n < 2000 ? 0 : bad("room", n, 0);
    Aligned rec(rec_bytes, 0x5A), slots((size_t)n_buckets * 128, 0xFF), text((size_t)max_seq_len * 4, 0);
    Aligned lds(kLds ? ingest_lds_bytes(n) : ingest_small_bytes<I>(n, true), 0xA5);
    const IngestSeq q{x.data(), n, (int32_t *)text.p, rec.p, slots.p, n_buckets};
    IngestArrays<I, K> A;
    if constexpr (kLds) ingest_place_lds(A, (char *)lds.p, n);
    else ingest_place_tables(A, q, (char *)lds.p, n);
    CpuCtx<T> ctx;
    ingest_build<IL, kLds>(ctx, q, A);

    HostSam h;
    std::string err;
    if (h.build(x.data(), n, vocab, err) != 0) return bad(err.c_str(), n, 0);
    // no phase works on more than the prompt's own share of the tables, however large they are
    if (ctx.widest > 6 * n + 1024) return bad("widest phase", n, ctx.widest);
    // (linear probing in a table that is 0.8 full: some hundred)
    if (ctx.most_swaps > (n < 10000 ? 500u : 3000u)) return bad("swaps in a row", n, ctx.most_swaps);
    if (A.small[124] != h.n_states) return bad("states", n, A.small[124]);
    if (A.small[125] != h.n_trans) return bad("transitions", n, A.small[125]);
    if (memcmp(text.p, x.data(), (size_t)n * 4)) return bad("text", n, 0);
    if (h.len[A.small[123]] != n) return bad("last state", n, A.small[123]);
    uint64_t seen = 0;
    for (uint32_t v = 0; v < h.n_states; v++) {
        uint32_t len, link, endpos, itok;
        IL::load(rec.p, v, len, link, endpos, itok);
        if (len != h.len[v]) return bad("length", n, v);
        if (link != h.link[v]) return bad("link", n, v);
        if (endpos != h.endpos[v]) return bad("end position", n, v);
        if (itok != kNil) {
            if (h.find(v, itok) != IL::idst(rec.p, v)) return bad("inline transition", n, v);
            seen++;
        }
        for (uint32_t at = IL::head(ctx, rec.p, v); at != kNil; seen++) {
            if (at >= n_buckets * IL::kSlots) return bad("slot", n, v);
            uint32_t state, token, dst, next;
            if (compact) {
                const SlotCompact &s = ((const SlotCompact *)slots.p)[at];
                state = s.key >> 17; token = s.key & 0x1FFFFu; dst = s.dst;
                next = s.next == 0xFFFFu ? kNil : s.next;
            } else {
                const Slot &s = ((const Slot *)slots.p)[at];
                state = s.state; token = s.token; dst = s.dst; next = s.w;
            }
            if (state != v || h.find(v, token) != dst) return bad("transition", n, v);
            at = next;
        }
    }
    return seen == h.n_trans ? 0 : bad("transition lists", n, (uint32_t)seen);
}

// Tables that something else writes to, or that are too small: every loop ends, and says so.
struct MeddlingCtx : CpuCtx<256> {
    uint32_t syncs = 0, at = 0, states = 0;
    uint32_t *rec = nullptr;
    void sync()
    {
        if (++syncs != at) return;
        for (uint32_t v = 0; v < states; v++) rec[4 * v] = 0xFFFFu | (v << 16);      // links that lead nowhere
    }
};

static int guards()
{
    const uint32_t n = 3000, cap = 3000;
    std::mt19937 rng(7);
    std::vector<int32_t> x(n);
    for (int32_t &t : x) t = (int32_t)(rng() % 3);
    uint32_t syncs[2], caught[2] = {0, 0};
    // left alone but for a slot table of two buckets (run 0), left alone (1), meddled with at
    // each of the last barriers; arrays in LDS and in the tables
    for (uint32_t k = 0; k < 20; k++) {
        const uint32_t run = k / 2;
        const bool lds = k % 2 == 0;
        const uint32_t n_buckets = run == 0 ? 2 : (uint32_t)(dynamic_slots_for(cap) / 16);
        if (!lds && (run == 0 || run > 5)) continue;        // before that the records hold other arrays
        Aligned rec((2 * cap + 2) * sizeof(DynRecCompact), 0x5A), slots((size_t)n_buckets * 128, 0xFF), text(cap * 4, 0);
        Aligned mem(lds ? ingest_lds_bytes(n) : ingest_small_bytes<uint16_t>(n, true), 0xA5);
        const IngestSeq q{x.data(), n, (int32_t *)text.p, rec.p, slots.p, n_buckets};
        IngestArrays<uint16_t, uint32_t> A;
        if (lds) ingest_place_lds(A, (char *)mem.p, n);
        else ingest_place_tables(A, q, (char *)mem.p, n);
        MeddlingCtx ctx;
        ctx.rec = (uint32_t *)rec.p;
        ctx.states = n;
        ctx.at = run < 2 ? 0 : syncs[lds] - (run - 2);
        if (lds) ingest_build<IngestCompact, true>(ctx, q, A);
        else ingest_build<IngestCompact, false>(ctx, q, A);
        if (run == 0 && !A.small[121]) return bad("guard of the slot table", n, run);
        if (run == 1 && A.small[121]) return bad("guard, nothing wrong", n, run);
        if (run == 1) syncs[lds] = ctx.syncs;
        if (run > 1 && A.small[121]) caught[lds]++;
    }
    return caught[0] && caught[1] ? 0 : bad("guards of the links", n, caught[0]);
}

// Calls that are faster token by token stay so (256 compute units; the measured sizes stand with
// the rule), the others are taken whole.
static int rules()
{
    // the most that fits into 160 KB of LDS beside the kernel's own words
    if (ingest_lds_bytes(6144) > 163840 - 256 || ingest_lds_bytes(6145) <= 163840 - 256)
        return bad("LDS", 6144, (uint32_t)ingest_lds_bytes(6144));
    struct { int64_t n_seqs, longest, mean, n_beyond; bool whole; } calls[] = {
        {1, 63, 63, 0, false}, {1, 64, 64, 0, true}, {1024, 64, 64, 0, true}, {1280, 64, 20, 0, true},
        {2048, 64, 64, 0, false}, {8192, 64, 64, 0, false}, {16384, 87, 87, 0, false}, {2048, 88, 88, 0, true},
        {8192, 96, 96, 0, true}, {16384, 128, 128, 0, true}, {2048, 128, 20, 0, true}, {3000, 64, 20, 0, false},
        {3000, 96, 20, 0, true}, {8192, 64, 20, 0, false}, {8192, 128, 20, 0, false}, {8192, 256, 20, 0, true},
        {4096, 6000, 6000, 0, true}, {1024, 8000, 8000, 1024, true}, {2048, 6300, 6300, 2048, false},
        {2048, 16000, 16000, 2048, false}, {4096, 8000, 300, 100, true}, {1500, 20000, 20000, 1500, true},
        {2048, 20000, 20000, 2048, false}, {1536, 40000, 40000, 1536, false}, {512, 40000, 40000, 512, true},
        {1, 1 << 18, 1 << 18, 1, true}, {1, (1 << 18) + 1, (1 << 18) + 1, 1, false},
    };
    for (auto &c : calls) {
        const PromptSizes p = {c.n_seqs, c.longest, c.mean * c.n_seqs, c.longest};
        if (prompts_whole(p, c.n_beyond, 256) != c.whole) return bad("rule", (uint32_t)c.n_seqs, (uint32_t)c.longest);
    }
    PromptSizes p = {64, 100, 64, (1 << 18) + 1};              // may be longer when the kernel runs
    if (prompts_whole(p, 0, 256)) return bad("rule of replayed calls", 100, 0);
    struct { int64_t n_seqs, longest, n_walks; bool small; } sizes[] = {
        {240, 256, 16, false}, {241, 256, 16, true}, {256, 257, 16, false}, {256, 256, 0, false}, {257, 512, 0, true},
        {257, 513, 0, false}, {512, 1024, 0, false}, {513, 1024, 0, true}, {513, 1025, 40, false},
    };
    for (auto &c : sizes) {
        const PromptSizes q = {c.n_seqs, c.longest, c.longest, c.longest};
        if (short_prompts(q, c.n_walks, 256) != c.small) return bad("rule of threads", (uint32_t)c.n_seqs, (uint32_t)c.longest);
    }
    return 0;
}

int main()
{
    if (guards() || rules()) return 1;
    std::mt19937 rng(5);
    const uint32_t sizes[] = {1, 2, 3, 7, 8, 9, 63, 64, 65, 255, 256, 257, 511, 513, 1023, 1024, 1025, 2500, 6200};
    for (const uint32_t n : sizes)
        for (int kind = 0; kind < 9; kind++)
            for (const int32_t vocab : {2, 60, 9000}) {
                std::vector<int32_t> x(n);
                for (uint32_t i = 0; i < n; i++) {
                    const double u = rng() / 4294967296.0;
                    x[i] = kind == 2 ? vocab - 1 : kind == 3 ? (int32_t)(i % 7) % vocab
                         : kind == 4 ? (i % 2 ? (int32_t)(i / 2) % vocab : 0) : (int32_t)(u * u * u * vocab);
                }
                if (kind == 1)                                  // copies of earlier spans
                    for (uint32_t i = 20; i < n; i += 1 + rng() % 40) {
                        const uint32_t from = rng() % i;
                        const uint32_t back = i - from;
                        for (uint32_t k = rng() % 80; k && i < n; k--, i++) x[i] = x[i - back];
                    }
                // long walks: a run and another token, a period of two and another token, two runs
                // with different tokens around them, a run that is three quarters of the text
                if (kind >= 5)
                    for (uint32_t i = 0; i < n; i++) {
                        const int32_t a = vocab - 1;
                        if (kind == 5) x[i] = i + 1 == n ? 0 : a;
                        if (kind == 6) x[i] = i + 1 == n ? vocab / 2 : (int32_t)(i % 2) * a;
                        if (kind == 7) x[i] = i == 0 || i + 1 == n || i == n / 2 ? (int32_t)(i % 5) % vocab : a;
                        if (kind == 8 && i < n * 3 / 4) x[i] = 0;
                    }
                const uint32_t cap = n + rng() % 20;
                if (one<IngestCompact, true, uint16_t, uint32_t, 1024>(x, vocab, cap) ||
                    one<IngestWide, true, uint16_t, uint32_t, 256>(x, vocab, cap))
                    return 1;
                if (n >= 64 && (one<IngestCompact, false, uint16_t, uint32_t, 1024>(x, vocab, cap) ||
                                one<IngestWide, false, uint32_t, uint64_t, 1024>(x, vocab, cap)))
                    return 1;
            }
    // long ones: where the 16-bit indices end and the names' levels begin, up to the longest taken
    // whole; copies, a run, and periods whose pairs crowd into few buckets
    for (const uint32_t n : {16365u, 16366u, 16367u, 40001u, 65536u, 65537u, 131072u, 262143u, 262144u})
        for (int kind = 0; kind < 5; kind++) {
            std::vector<int32_t> x(n);
            for (int32_t &t : x) t = (int32_t)(rng() % 3000);
            const uint32_t period = kind == 2 ? 130 : kind == 3 ? (uint32_t)(n / 500) : n;
            for (uint32_t i = period; i < n; i++) x[i] = x[i - period];
            if (kind == 1) for (uint32_t i = 1; i + 1 < n; i++) x[i] = 0;
            if (kind == 4)
                for (uint32_t i = 20; i < n; i += 1 + rng() % 40) {
                    const uint32_t back = i - rng() % i;
                    for (uint32_t k = rng() % 6000; k && i < n; k--, i++) x[i] = x[i - back];
                }
            if ((n <= kIngestIdx16 && one<IngestCompact, false, uint16_t, uint32_t, 1024>(x, 3000, n)) ||
                one<IngestWide, false, uint32_t, uint64_t, 1024>(x, 3000, n))
                return 1;
        }
    // a short prompt in a long sequence's tables
    for (const uint32_t n : {64u, 700u, 3000u}) {
        std::vector<int32_t> x(n);
        for (int32_t &t : x) t = (int32_t)(rng() % 9);
        if (one<IngestCompact, false, uint16_t, uint32_t, 1024>(x, 9, 16366) ||
            one<IngestWide, false, uint32_t, uint64_t, 1024>(x, 9, 200000))
            return 1;
    }
    printf("ok\n");
    return 0;
}
