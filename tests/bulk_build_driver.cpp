// An automaton built by phases over the whole chip (sam_bulk.h, the phases run one after the other on
// the CPU) against the token-by-token host builder: ids, lengths, links, end positions and every
// transition, into a sequence's own tables in both layouts and into the corpus's.  What lanes or
// workgroups do together has a plain form here: std::sort for the radix passes, counting for
// groups of any size, loops for the minima and the running sums, one link after the other for the
// states that a wave guesses (the kernels' own forms are compared with the host builder on the GPU).
// The regions have exactly the sizes that the library gives them: an access outside one is seen by
// AddressSanitizer.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <sanitizer/asan_interface.h>

#include <algorithm>
#include <random>
#include <string>
#include <vector>

#include "../paper_2411_10666_amd/csrc/sam_bulk.h"
#include "../paper_2411_10666_amd/csrc/sam_host.h"

using namespace sam;

struct CpuCtx {
    template <class F> void lanes(F f) { for (uint32_t i = 0; i < 64; i++) f(i); }
    void wave_sync() {}
    template <class F> uint32_t chain(uint32_t v, uint32_t down, F f, uint32_t *list, uint32_t &more, uint32_t &next)
    {
        uint32_t count = 0, link = 0;
        for (more = 1; count < 64 && more; count++) {
            const uint32_t s = count ? link : v;
            if (count && (uint64_t)count * down > v) break;
            if (count && s != v - count * down) break;
            uint32_t kind, up;
            f(s, up, kind);
            if (kind == 2) { more = 0; break; }
            list[count] = kind ? kNil : s;
            link = up;
            if (s == 0) more = 0;
        }
        next = link;
        return count;
    }
    template <class U> U cas(U *p, U expected, U v) { const U old = *p; if (old == expected) *p = v; return old; }
    template <class U> U add(U *p, U v) { const U old = *p; *p = (U)(old + v); return old; }
    uint32_t lower(uint32_t *p, uint32_t v) { const uint32_t old = *p; if (v < old) *p = v; return old; }
    void bit_or(uint32_t *p, uint32_t v) { *p |= v; }
    uint32_t exch(uint32_t *p, uint32_t v) { const uint32_t old = *p; *p = v; return old; }
    uint32_t fresh(uint32_t *p) { return *p; }
    uint32_t mulhi(uint32_t a, uint32_t b) { return (uint32_t)(((uint64_t)a * b) >> 32); }
    uint32_t popc(uint32_t x) { return (uint32_t)__builtin_popcount(x); }
    uint32_t first(uint32_t x) { return (uint32_t)__builtin_ctz(x); }
    uint32_t log2(uint32_t x) { return 31u - (uint32_t)__builtin_clz(x); }
};

static int bad(const char *what, uint32_t n, uint32_t at)
{
    printf("%s differs: %u tokens, at %u\n", what, n, at);
    return 1;
}

struct Aligned {
    char *p;
    size_t bytes;
    Aligned(size_t b, int fill) : p((char *)aligned_alloc(128, room(b))), bytes(b)
    {
        memset(p, fill, b);
        // what the block has behind the region is out of bounds too
        ASAN_POISON_MEMORY_REGION(p + b, room(b) - b);
    }
    ~Aligned()
    {
        ASAN_UNPOISON_MEMORY_REGION(p + bytes, room(bytes) - bytes);
        free(p);
    }
    static size_t room(size_t b) { return (b + 127) / 128 * 128; }
};

// what the kernels with lanes working together do
template <class I>
static void sort_by_tokens(BulkSeq<I> &q, const BulkSort &s, uint32_t first)
{
    const uint32_t n = q.n;
    std::vector<std::pair<uint64_t, uint32_t>> a(n);
    for (uint32_t i = 0; i < n; i++) a[i] = {bulk_key(q.tok, i, s), i};
    std::sort(a.begin(), a.end());
    for (uint32_t k = 0; k < n; k++) { q.key(first)[k] = a[k].first; q.pos(first)[k] = a[k].second; }
    for (uint32_t k = 0, start = 0; k < n; k++) {
        if (k && q.key(first)[k] != q.key(first)[k - 1]) start = k;
        if (k != start) q.gs(0)[k] = start;
        if (k + 1 == n || q.key(first)[k + 1] != q.key(first)[k]) q.gs(0)[start] = kBulkStart | (k + 1 - start);
        if (k != start) q.ctl[kCtlActive] = 1;
        q.name[q.pos(first)[k]] = start;
        q.lev[k] = 0;
    }
}

template <class I>
static void minima(BulkSeq<I> &q)
{
    q.ctl[kCtlTops] = bulk_levels(q.n, q.ctl + kCtlLevel);
    const I *below = q.lcp;
    uint32_t count = ingest_pad(q.n);
    for (uint32_t level = 1; level <= q.ctl[kCtlTops]; level++) {
        I *const out = level == 1 ? q.mins1 : q.mins + q.ctl[kCtlLevel + level];
        const uint32_t real = count / 8, padded = ingest_pad(real);
        for (uint32_t w = 0; w < padded; w++) {
            I least = 0;
            if (w < real) least = *std::min_element(below + 8 * w, below + 8 * w + 8);
            out[w] = least;
        }
        below = out;
        count = padded;
    }
}

// everything up to the records; the number of states
template <class I, class S>
static uint32_t states_of(CpuCtx &ctx, BulkSeq<I> &q, uint32_t vocab, uint32_t key_bits, const S &out)
{
    const uint32_t n = q.n;
    memset(q.ctl, 0, 4 * kBulkCtl);
    memset(q.counts, 0, 4 * kBulkCounts);
    const BulkSort sort = bulk_sort_for(vocab, key_bits);
    const uint32_t first = (sort.passes - 1) & 1;
    sort_by_tokens(q, sort, first);
    uint32_t round = 0;
    for (uint32_t h = sort.tokens; q.ctl[kCtlActive + round] && h < n; h *= 2, round++) {
        for (uint32_t k = 0; k < n; k++) bulk_gather(q, first, round, h, k);
        for (uint32_t k = 0; k < n; k++)
            if (bulk_rank<true>(q, first, round, k)) q.ctl[kCtlActive + round + 1] = 1;
    }
    for (uint32_t i = 0; i < n; i++) bulk_order(q, i);
    const uint32_t longest = bulk_longest(q, sort.tokens), run = longest > kBulkLong ? longest / 128 : 8;
    for (uint32_t c = 0; c <= (n - 1) / run; c++)
        bulk_common(q, sort.tokens, run, c, [&](uint32_t a, uint32_t b, uint32_t l) { return bulk_agree(q.tok, a, b, l); });
    minima(q);
    const IngestTree<I> t = q.tree();
    for (uint32_t k = 0; k < n; k++) t.interval(ctx, k);
    for (uint32_t k = 0; k < n; k++) t.represent(k);
    for (uint32_t k = 0; k < n; k++) t.parent(k);
    for (uint32_t k = 0; k < n / 32 + 1; k++) q.bits[k] = 0;
    for (uint32_t k = 0; k < n; k++) t.leaf_of(k);
    for (uint32_t k = 0; k < n; k++) t.template first_end<true>(ctx, k);
    for (uint32_t k = 0; k < n; k++) t.second_end(ctx, k);
    for (uint32_t k = 0; k < n; k++) t.mark_clone(ctx, k);
    uint32_t sum = 0;
    for (uint32_t w = 0; w < n / 32 + 1; w++) { q.rank[w] = sum; sum += ctx.popc(q.bits[w]); }
    for (uint32_t k = 0; k < n; k++) bulk_records(ctx, q, t, out, k);
    return q.counts[kCntStates] = 1 + n + sum;
}

template <class I, class S>
static void transitions(CpuCtx &ctx, BulkSeq<I> &q, S out, uint32_t states)
{
    uint32_t list[64], chain[2] = {kNil, kNil};
    out.chain = chain;
    for (uint32_t v = 0; v < states; v++) {
        BulkWalk w;
        q.counts[kCntMade] += bulk_walk(ctx, q, out, states, v, w);
        if (w.more) bulk_long_walk(ctx, q, out, states, w, list);
        if (v % 300 == 299) {                        // as if a workgroup ended here
            out.hang(ctx);
            chain[0] = kNil;
        }
    }
    out.hang(ctx);
}

template <class IL, class I>
static int tables(const HostSam &h, const std::vector<int32_t> &x, int32_t vocab, uint32_t max_seq_len, uint32_t key_bits)
{
    const uint32_t n = (uint32_t)x.size();
    constexpr bool compact = IL::kSlots == 16;
    const size_t rec_bytes = (size_t)(2 * max_seq_len + 2) * (compact ? sizeof(DynRecCompact) : sizeof(DynRec));
    const uint32_t n_buckets = (uint32_t)(dynamic_slots_for(max_seq_len) * (compact ? sizeof(SlotCompact) : sizeof(Slot)) / 128);
    Aligned rec(rec_bytes, 0x5A), slots((size_t)n_buckets * 128, 0xFF), text((size_t)max_seq_len * 4, 0x77);
    if (!bulk_tables_fit<I>(n, max_seq_len, rec_bytes, (size_t)n_buckets * 128)) return bad("room", n, max_seq_len);
    BulkSeq<I> q;
    q.tok = x.data();
    q.n = n;
    uint32_t counts[kBulkCounts];
    q.counts = counts;
    bulk_place(q, rec.p, slots.p, text.p);
    const BulkTables<IL> out{rec.p, slots.p, n_buckets, x.data(), n};
    CpuCtx ctx;
    const uint32_t states = states_of(ctx, q, (uint32_t)vocab, key_bits, out);
    memset(slots.p, 0xFF, q.dirty);
    memcpy(text.p, x.data(), 4 * (size_t)n);
    for (uint32_t v = 0; v < states; v++) bulk_settle(ctx, q, out, states, v);
    transitions(ctx, q, out, states);
    if (q.counts[kCntCorrupt]) return bad("guard", n, 0);
    if (states != h.n_states) return bad("states", n, states);
    if (q.counts[kCntMade] + states - 1 != h.n_trans) return bad("transitions", n, q.counts[kCntMade]);
    uint64_t seen = 0;
    for (uint32_t v = 0; v < h.n_states; v++) {
        uint32_t len, link, endpos, itok;
        IL::load(rec.p, v, len, link, endpos, itok);
        if (len != h.len[v] || link != h.link[v] || endpos != h.endpos[v]) return bad("state", n, v);
        if (itok != kNil) {
            if (h.find(v, itok) != IL::idst(rec.p, v)) return bad("inline transition", n, v);
            seen++;
        }
        for (uint32_t at = IL::head(ctx, rec.p, v); at != kNil; seen++) {
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

static int corpus(const HostSam &h, const std::vector<int32_t> &x, int32_t vocab, uint32_t key_bits)
{
    const uint32_t n = (uint32_t)x.size();
    Aligned first(bulk_first_bytes(n), 0x5A), second(bulk_second_bytes<uint32_t>(n), 0x5B), third(bulk_third_bytes(n), 0x5C),
        rec(16 * (2 * (size_t)n + 1), 0x5D);
    uint32_t counts[kBulkCounts];
    std::vector<RootEnt> root((size_t)vocab, RootEnt{0, 0});
    BulkSeq<uint32_t> q;
    q.tok = x.data();
    q.n = n;
    q.counts = counts;
    bulk_place(q, first.p, second.p, third.p);
    // the open-addressed table lies over the first region
    const BulkCorpus out{(BulkCorpus::State *)rec.p, (uint64_t *)first.p, (uint32_t *)(first.p + 16 * (size_t)n), 2 * n,
                         root.data(), x.data(), n};
    CpuCtx ctx;
    const uint32_t states = states_of(ctx, q, (uint32_t)vocab, key_bits, out);
    memset(first.p, 0xFF, 16 * (size_t)n);
    root[(size_t)x[0]].dst = 1;
    for (uint32_t v = 0; v < states; v++) bulk_settle(ctx, q, out, states, v);
    transitions(ctx, q, out, states);
    if (q.counts[kCntCorrupt]) return bad("corpus: guard", n, 0);
    if (states != h.n_states) return bad("corpus: states", n, states);
    if (q.counts[kCntMade] + states - 1 != h.n_trans) return bad("corpus: transitions", n, q.counts[kCntMade]);
    uint64_t seen = 0;
    for (uint32_t v = 0; v < states; v++) {
        const BulkCorpus::State &s = out.rec[v];
        if (s.len != h.len[v] || s.link != h.link[v] || s.endpos != h.endpos[v]) return bad("corpus: state", n, v);
        if (v && s.endpos < n) {
            if (h.find(v, (uint32_t)x[s.endpos]) != s.idst) return bad("corpus: first transition", n, v);
            seen++;
        }
    }
    for (uint32_t at = 0; at < out.n_slots; at++)
        if (out.key[at] != ~(uint64_t)0) {
            if (h.find((uint32_t)out.key[at], (uint32_t)(out.key[at] >> 32)) != out.dst[at]) return bad("corpus: transition", n, at);
            seen++;
        }
    for (int32_t t = 0; t < vocab; t++) {
        if ((root[t].dst ? root[t].dst : kNil) != h.find(0, (uint32_t)t)) return bad("corpus: root", n, (uint32_t)t);
        seen += root[t].dst != 0;
    }
    return seen == h.n_trans ? 0 : bad("corpus: all transitions", n, (uint32_t)seen);
}

int main()
{
    std::mt19937 rng(5);
    const uint32_t sizes[] = {1, 2, 3, 7, 8, 9, 63, 64, 65, 255, 257, 511, 513, 1023, 1025, 2500, 4096, 9000};
    for (const uint32_t n : sizes)
        for (int kind = 0; kind < 9; kind++)
            for (const int32_t vocab : {1, 2, 60, 9000, 140000}) {
                if (n > 3000 && (vocab != 9000 || kind == 2 || kind == 3 || kind == 8)) continue;
                std::vector<int32_t> x(n);
                for (uint32_t i = 0; i < n; i++) {
                    const double u = rng() / 4294967296.0;
                    x[i] = kind == 2 ? vocab - 1 : kind == 3 ? (int32_t)(i % 7) % vocab
                         : kind == 4 ? (i % 2 ? (int32_t)(i / 2) % vocab : 0) : (int32_t)(u * u * u * vocab);
                }
                if (kind == 1)                                  // copies of earlier spans
                    for (uint32_t i = 20; i < n; i += 1 + rng() % 40) {
                        const uint32_t back = i - rng() % i;
                        for (uint32_t k = rng() % 300; k && i < n; k--, i++) x[i] = x[i - back];
                    }
                if (kind >= 5)
                    for (uint32_t i = 0; i < n; i++) {          // long walks
                        const int32_t a = vocab - 1;
                        if (kind == 5) x[i] = i + 1 == n ? 0 : a;
                        if (kind == 6) x[i] = i + 1 == n ? vocab / 2 : (int32_t)(i % 2) * a;
                        if (kind == 7) x[i] = i == 0 || i + 1 == n || i == n / 2 ? (int32_t)(i % 5) % vocab : a;
                        if (kind == 8 && i < n * 3 / 4) x[i] = 0;
                    }
                HostSam h;
                std::string err;
                if (h.build(x.data(), n, vocab, err) != 0) return bad(err.c_str(), n, 0);
                for (const uint32_t most : {2u, 32u, 64u}) {
                    if (n > 2000 && most != 64) continue;       // quadratic without large groups
                    if (corpus(h, x, vocab, most)) return 1;
                    const uint32_t cap = (n > kBulkLdsTokens ? n : kBulkLdsTokens) + 3 + rng() % 2 * 77;
                    if (cap <= 16366 && vocab <= 131072 && tables<IngestCompact, uint16_t>(h, x, vocab, cap, most)) return 1;
                    if (tables<IngestWide, uint32_t>(h, x, vocab, cap, most)) return 1;
                }
            }
    printf("ok\n");
    return 0;
}
