// An automaton built from its whole text at once; here a prompt's, by one workgroup.
//
// Online extension (Algorithm 2) is a serial chain: one token after the other, each with
// two or three dependent memory round trips.  A prompt is known in full, though, and what
// the chain leaves behind is fixed by the text alone:
//
//   * the states are the prefixes of the text and the strings that occur with two
//     different tokens in front of them; the suffix links form the compressed trie of
//     all prefixes read BACKWARDS (the suffix tree of the reversed text);
//   * a prefix state's id is its step's first new id; the state of a string w that is no
//     prefix is cloned in the step in which w first occurs with a second token in front
//     of it, i.e. at the second smallest of the first end positions of w's children in
//     that tree, and at most one state is cloned in a step;
//   * min_endpos of a state is the smallest prefix in its subtree;
//   * (v, t) leads to the state on the suffix path of the prefix x[..i+1] whose lengths
//     include len(v) + 1, for any occurrence of v that ends at i and is followed by t.
//
// So the workgroup sorts the reversed prefixes by doubling (names of the last h tokens
// before every position; equal pairs of names get equal names for 2h), takes the common
// lengths of neighbours, finds every interval's parent by the nearest smaller values,
// numbers the states, and inserts the transitions with compare-and-swap.  Children are in
// no particular order (a tree has none), so a round of the sort is a hash table of pairs
// and no radix passes.  Everything is exact: tokens and names are compared, never hashes.
//
// Written as phases over an index range with a barrier between them (Ctx::each,
// Ctx::sync); nothing is carried from one phase to the next in a thread, so the same
// source also runs phase by phase on the CPU.
#pragma once
#include <stdint.h>

#include <type_traits>

#include "sam_layout.h"

#if defined(__HIPCC__)
#define SAM_HD __host__ __device__ __forceinline__
#else
#define SAM_HD inline
#endif

namespace sam {

constexpr uint32_t kIngestMaxTokens = 1u << 18;      // beyond: the serial kernel
constexpr uint32_t kIngestIdx16 = 16366;             // the most tokens that 16-bit indices do for

// What the host knows of the prompts of a call.
struct PromptSizes {
    int64_t n_seqs;
    int64_t longest;     // tokens; what the launch is made for
    int64_t total;
    int64_t most;        // what a prompt may have when the kernel runs: more than `longest` where
                         // the host has not read the device's offsets itself (a captured call that
                         // is replayed with other prompts)
};

// Are the prompts of a call taken whole, or token by token?  n_beyond: how many are too long for
// LDS.  Whole, the about sixty barriers take what the serial loops need for 64 tokens as long
// as all workgroups run at once; token by token, sequences share compute units better.  Measured
// on 256 compute units, sam_batch_reset, token by token against whole (us):
//   64 tokens     1 sequence 80 / 77   1024: 96 / 88   1536: 104 / 93, over a corpus 109 / 112
//                 2048: 120 / 133   8192: 234 / 264   16384: 432 / 518
//   76 tokens     2048: 119 / 128   4096: 179 / 171   8192: 276 / 277, over a corpus 299 / 318
//   88 tokens     2048: 125 / 132   4096: 193 / 183   8192: 300 / 288, over a corpus 336 / 331
//   96 tokens     2048: 135 / 134   4096: 210 / 188   8192: 340 / 294
//   20 tokens and one of n    2048, n = 64: 92 / 97, 128: 130 / 96   3000, n = 64: 100 / 104, 96: 112 / 106
//                 8192, n = 64: 121 / 173, 128: 153 / 174, 256: 237 / 176
//   beyond LDS    6300 tokens: 1024: 6176 / 5550   1280: 6473 / 6861   1536: 6822 / 8190   2048: 7615 / 10771
//                 16000: 1280: 19655 / 18764   1536: 20385 / 21944   40000: 1280: 76443 / 79013   1536: 78160 / 94476
//                 20000 (wide layout, half the working set): 1280: 36934 / 31489   1536: 37795 / 37370
inline bool prompts_whole(const PromptSizes &p, int64_t n_beyond, int64_t n_cu)
{
    if (p.longest < 64 || p.most > (int64_t)kIngestMaxTokens) return false;
    if (p.n_seqs > 5 * n_cu) {
        if (p.longest < 88) return false;
        // mostly short ones: each costs a workgroup its barriers
        if (p.total < 32 * p.n_seqs && p.longest < 64 + 8 * p.n_seqs / (3 * n_cu)) return false;
    }
    return n_beyond <= (p.longest > kIngestIdx16 && p.longest <= 32768 ? 6 : 5) * n_cu;
}

// Do they get workgroups of 256 threads, or of 1024?  Of 1024 one fits on a compute unit (69 to 81 VGPRs
// a thread; bound to 64, so that two fit where LDS allows it, 257 prompts of 1025 tokens take
// 188 us instead of 184, 1024 of 1500 455 instead of 446), so it is 256 where there are more workgroups than compute units (n_walks of them walk
// the corpus automaton) and the prompts are so short that 256 threads suffice.  Measured, 1024
// against 256 threads: 256 prompts of 256 tokens 88 against 90 us, over a corpus 120 against 103, of
// 512 130 against 134, of 1024 (no corpus) 121 against 155; 300 of 64 97 against 78, of 256 116
// against 96, of 1024 164 against 181; 512 of 512 137 against 127, of 1024 178 against 195; 640 of 1024
// 223 against 207; 1024 of 64 150 against 82, of 512 215 against 152, of 1024 287 against 250, of
// 1500 387 against 422.
inline bool short_prompts(const PromptSizes &p, int64_t n_walks, int64_t n_cu)
{
    return (p.n_seqs + n_walks > n_cu && p.longest <= 256) || (p.n_seqs > n_cu && p.longest <= 512) ||
           (p.n_seqs > 2 * n_cu && p.longest <= 1024);
}

struct IngestSeq {
    const int32_t *tok;        // the prompt, every token inside the vocabulary
    uint32_t n;                // tokens, >= 1
    int32_t *text;
    void *rec;                 // record table of the sequence
    void *slots;               // slot table
    uint32_t n_buckets;
};

// ---- the two table layouts, as single threads write them ----------------------

struct IngestWide {
    static constexpr uint32_t kSlots = 8;
    static constexpr bool kHead16 = false;       // slot indices beyond 16 bits
    static SAM_HD void fill_next(void *, uint32_t, uint32_t, uint32_t) {}
    static SAM_HD void store_head(void *, uint32_t, uint32_t) {}
    static SAM_HD void store(void *rec, uint32_t s, uint32_t len, uint32_t link, uint32_t endpos,
                             uint32_t itok, uint32_t idst)
    {
        DynRec *r = reinterpret_cast<DynRec *>(rec) + s;
        r->len = len; r->link = link; r->endpos = endpos; r->head = kNil;
        r->itok = itok; r->idst = idst;
    }
    static SAM_HD void store_idst(void *rec, uint32_t s, uint32_t dst)
    {
        (reinterpret_cast<DynRec *>(rec) + s)->idst = dst;
    }
    static SAM_HD uint32_t len(const void *rec, uint32_t s) { return (reinterpret_cast<const DynRec *>(rec) + s)->len; }
    static SAM_HD uint32_t link(const void *rec, uint32_t s) { return (reinterpret_cast<const DynRec *>(rec) + s)->link; }
    static SAM_HD void load(const void *rec, uint32_t s, uint32_t &len, uint32_t &link, uint32_t &endpos,
                            uint32_t &itok)
    {
        const DynRec *r = reinterpret_cast<const DynRec *>(rec) + s;
        len = r->len; link = r->link; endpos = r->endpos; itok = r->itok;
    }
    static SAM_HD uint32_t idst(const void *rec, uint32_t s) { return (reinterpret_cast<const DynRec *>(rec) + s)->idst; }
    // claim the slot for (p, t): 0 claimed, 1 the key was there already, 2 another key
    template <class C>
    static SAM_HD int claim(C &ctx, void *slots, uint32_t at, uint32_t p, uint32_t t)
    {
        const uint64_t key = (uint64_t)p | ((uint64_t)t << 32);
        const uint64_t old = ctx.cas(reinterpret_cast<uint64_t *>(reinterpret_cast<Slot *>(slots) + at), ~(uint64_t)0, key);
        return old == ~(uint64_t)0 ? 0 : (old == key ? 1 : 2);
    }
    // what a plain read says of the slot: 0 empty (or claimed meanwhile), 1 and 2 as above
    static SAM_HD int peek(const void *slots, uint32_t at, uint32_t p, uint32_t t)
    {
        const uint64_t seen = *reinterpret_cast<const uint64_t *>(reinterpret_cast<const Slot *>(slots) + at);
        return seen == ~(uint64_t)0 ? 0 : (seen == ((uint64_t)p | ((uint64_t)t << 32)) ? 1 : 2);
    }
    template <class C>
    static SAM_HD void fill(C &ctx, void *rec, void *slots, uint32_t at, uint32_t p, uint32_t, uint32_t dst)
    {
        Slot *s = reinterpret_cast<Slot *>(slots) + at;
        s->dst = dst;
        s->w = ctx.exch(&(reinterpret_cast<DynRec *>(rec) + p)->head, at);
    }
    template <class C>
    static SAM_HD uint32_t head(C &ctx, void *rec, uint32_t s)
    {
        return ctx.fresh(&(reinterpret_cast<DynRec *>(rec) + s)->head);
    }
    // transitions of the root that were chained apart: one more, and the whole chain into the root's list
    static SAM_HD void link_slot(void *slots, uint32_t at, uint32_t dst, uint32_t next)
    {
        Slot *s = reinterpret_cast<Slot *>(slots) + at;
        s->dst = dst;
        s->w = next;
    }
    template <class C>
    static SAM_HD void hang(C &ctx, void *rec, void *slots, uint32_t head, uint32_t tail)
    {
        (reinterpret_cast<Slot *>(slots) + tail)->w = ctx.exch(&reinterpret_cast<DynRec *>(rec)->head, head);
    }
};

struct IngestCompact {
    static constexpr uint32_t kSlots = 16;
    static constexpr bool kHead16 = true;
    static SAM_HD void fill_next(void *slots, uint32_t at, uint32_t dst, uint32_t next)
    {
        (reinterpret_cast<uint32_t *>(slots) + 2 * (size_t)at)[1] = (dst & 0xFFFFu) | (next << 16);
    }
    static SAM_HD void store_head(void *rec, uint32_t s, uint32_t head)
    {
        reinterpret_cast<uint16_t *>(rec)[8 * (size_t)s + 3] = (uint16_t)head;
    }
    static SAM_HD uint32_t widen(uint32_t v16) { return v16 == 0xFFFFu ? kNil : v16; }
    static SAM_HD void store(void *rec, uint32_t s, uint32_t len, uint32_t link, uint32_t endpos,
                             uint32_t itok, uint32_t idst)
    {
        uint32_t *r = reinterpret_cast<uint32_t *>(rec) + 4 * (size_t)s;
        r[0] = (len & 0xFFFFu) | (link << 16);
        r[1] = (endpos & 0xFFFFu) | 0xFFFF0000u;
        r[2] = itok;
        r[3] = idst & 0xFFFFu;
    }
    static SAM_HD void store_idst(void *rec, uint32_t s, uint32_t dst)
    {
        (reinterpret_cast<uint32_t *>(rec) + 4 * (size_t)s)[3] = dst & 0xFFFFu;
    }
    static SAM_HD uint32_t len(const void *rec, uint32_t s) { return (reinterpret_cast<const uint32_t *>(rec) + 4 * (size_t)s)[0] & 0xFFFFu; }
    static SAM_HD uint32_t link(const void *rec, uint32_t s) { return widen((reinterpret_cast<const uint32_t *>(rec) + 4 * (size_t)s)[0] >> 16); }
    static SAM_HD void load(const void *rec, uint32_t s, uint32_t &len, uint32_t &link, uint32_t &endpos,
                            uint32_t &itok)
    {
        const uint32_t *r = reinterpret_cast<const uint32_t *>(rec) + 4 * (size_t)s;
        const uint32_t a = r[0], b = r[1];
        len = a & 0xFFFFu; link = widen(a >> 16); endpos = b & 0xFFFFu; itok = r[2];
    }
    static SAM_HD uint32_t idst(const void *rec, uint32_t s) { return (reinterpret_cast<const uint32_t *>(rec) + 4 * (size_t)s)[3]; }
    template <class C>
    static SAM_HD int claim(C &ctx, void *slots, uint32_t at, uint32_t p, uint32_t t)
    {
        const uint32_t key = (p << 17) | t;
        const uint32_t old = ctx.cas(reinterpret_cast<uint32_t *>(slots) + 2 * (size_t)at, kNil, key);
        return old == kNil ? 0 : (old == key ? 1 : 2);
    }
    static SAM_HD int peek(const void *slots, uint32_t at, uint32_t p, uint32_t t)
    {
        const uint32_t seen = reinterpret_cast<const uint32_t *>(slots)[2 * (size_t)at];
        return seen == kNil ? 0 : (seen == ((p << 17) | t) ? 1 : 2);
    }
    // the head shares its word with the end position, which does not change
    template <class C>
    static SAM_HD void fill(C &ctx, void *rec, void *slots, uint32_t at, uint32_t p, uint32_t endpos,
                            uint32_t dst)
    {
        const uint32_t old = ctx.exch(reinterpret_cast<uint32_t *>(rec) + 4 * (size_t)p + 1,
                                      (endpos & 0xFFFFu) | (at << 16));
        (reinterpret_cast<uint32_t *>(slots) + 2 * (size_t)at)[1] = (dst & 0xFFFFu) | (old & 0xFFFF0000u);
    }
    template <class C>
    static SAM_HD uint32_t head(C &ctx, void *rec, uint32_t s)
    {
        return widen(ctx.fresh(reinterpret_cast<uint32_t *>(rec) + 4 * (size_t)s + 1) >> 16);
    }
    static SAM_HD void link_slot(void *slots, uint32_t at, uint32_t dst, uint32_t next) { fill_next(slots, at, dst, next & 0xFFFFu); }
    // the root's end position is 0
    template <class C>
    static SAM_HD void hang(C &ctx, void *rec, void *slots, uint32_t head, uint32_t tail)
    {
        const uint32_t old = ctx.exch(reinterpret_cast<uint32_t *>(rec) + 1, head << 16);
        reinterpret_cast<uint16_t *>(slots)[4 * (size_t)tail + 3] = (uint16_t)(old >> 16);
    }
};

// The slot of (v, t) in the table: 0 claimed now, 1 it was there, 2 the table is full.  kPeek: slots
// are read before they are tried.
template <class L, bool kPeek = false, class C>
SAM_HD int ingest_claim(C &ctx, void *slots, uint32_t n_buckets, uint32_t v, uint32_t t, uint32_t &at)
{
    const uint32_t hsh = dyn_hash(v, t);
    uint32_t b = ctx.mulhi(hsh, n_buckets);
    int got = 2;
    for (uint32_t left = n_buckets; left && got == 2; left--) {
        for (uint32_t j = 0; j < L::kSlots && got == 2; j++) {
            at = b * L::kSlots + ((hsh + j) & (L::kSlots - 1));
            if (kPeek) got = L::peek(slots, at, v, t);
            if (!kPeek || got == 0) got = L::claim(ctx, slots, at, v, t);
        }
        b = b + 1 == n_buckets ? 0 : b + 1;
    }
    return got;
}

// ---- working arrays -------------------------------------------------------------
//
// I: index type (16 bits up to kIngestIdx16 tokens), K: a pair of names.

template <class I, class K>
struct IngestArrays {
    // sort
    K        *key;       // [h_size] pairs of names (empty: all ones)
    K        *val;       // [h_size] lower half: positions that have it; upper: where they start
    K        *cursor;    // [n] a bucket of a group: lower half its positions, then their start;
                         // upper half the first of its pairs (+ 1) in key[]
    I        *grp;       // [n] name of position i = start of its group; top bit: alone in it
    I        *slot;      // [n] where its pair is in key[]
    I        *next;      // [h_size] the next pair (+ 1) of the same bucket
    I        *size;      // [n] size of the group that starts here
    uint32_t *lo, *hi;   // [n] least and largest second name in it (32-bit indices only)
    I        *name1;     // [n] names of single tokens (unused if the text is read instead)
    uint8_t  *lev;       // [n] round in which a group came to start here
    uint32_t  h_size;
    // tree; boundary k lies between places k-1 and k of the sorted order
    I        *sa;        // [n]
    I        *lcp;       // [n]
    I        *node;      // [n]
    I        *tab;       // [2n]
    I        *par;       // [n]
    I        *pfx;       // [n]
    I        *leaf;      // [n]
    uint32_t *m;         // [n]
    uint32_t *sec;       // [n]
    I        *names;     // [7][stride] names of the last 16 * 4^j tokens (tables in device memory only)
    uint32_t  stride;    // n rounded up to 16
    size_t    dirty;     // bytes of the slot table that held any of this (tables in device memory only)
    // the states, once their records are written, and the text (all in LDS only)
    uint32_t *state;     // [2n + 1][2] len | link << 16, min_endpos | head << 16
    int32_t  *text;      // [n]
    // always in LDS
    I        *mins1;     // minima of 8 boundaries each (with device-memory tables: there)
    I        *mins;      // the levels above, 8 to 1, one behind the other; part[] says where
    uint32_t *bits;      // [n / 32 + 1] steps that clone
    uint32_t *rank;      // [n / 32 + 1] clones before the word
    uint32_t *small;     // [128] flags and results
    uint32_t *part;      // [kIngestParts] partial sums
};

// A walk up the suffix links of more than kLongWalk states goes on by waves (below), kWalks of
// them at most: the states of all walks that bring a new token are fewer than three a token.
constexpr uint32_t kLongWalk = 32, kWalks = 32;
constexpr uint32_t kIngestParts = 1024;      // at least one for every thread of a workgroup

SAM_HD uint32_t ingest_h_size(uint32_t n) { return n + n / 4 + 64; }

struct IngestBump {
    char *p;
    template <class T>
    SAM_HD T *take(size_t count)
    {
        T *r = reinterpret_cast<T *>(p);
        p += (count * sizeof(T) + 15) / 16 * 16;
        return r;
    }
};

// Minima over runs of 8, 64, 512 ... boundaries.  Every level is padded with zeros to whole
// runs and has at least one of them, so a search to the right always ends.
SAM_HD uint32_t ingest_pad(uint32_t count) { return (count / 8 + 1) * 8; }
SAM_HD uint32_t ingest_first_mins(uint32_t n) { return ingest_pad(ingest_pad(n) / 8); }
SAM_HD uint32_t ingest_upper_mins(uint32_t n)
{
    uint32_t sum = 0;
    for (uint32_t c = ingest_first_mins(n); c > 8; sum += c) c = ingest_pad(c / 8);
    return sum;
}

template <class I>
SAM_HD size_t ingest_small_bytes(uint32_t n, bool mins)
{
    const size_t w = n / 32 + 1;
    return 512 + 4 * kIngestParts + 2 * ((w * 4 + 15) / 16 * 16) +
           (mins ? (ingest_upper_mins(n) * sizeof(I) + 15) / 16 * 16 : 0);
}

template <class I, class K>
SAM_HD void ingest_place_small(IngestArrays<I, K> &A, IngestBump &b, uint32_t n)
{
    A.small = b.take<uint32_t>(128);
    A.part = b.take<uint32_t>(kIngestParts);
    A.bits = b.take<uint32_t>(n / 32 + 1);
    A.rank = b.take<uint32_t>(n / 32 + 1);
}

// All of it in LDS.  The tree's arrays lie over the sort's: what overlaps is never
// alive at the same time (node over grp, pfx over name1, the rest over the hash table).
SAM_HD size_t ingest_lds_bytes(uint32_t n)
{
    const size_t h = ingest_h_size(n);
    auto up = [](size_t x) { return (x + 15) / 16 * 16; };
    const size_t sort = 2 * up(4 * h) + up(2 * h) + up(4 * (size_t)n) + 2 * up(2 * (size_t)n);
    const size_t tree = 3 * up(2 * (size_t)n) + up(2 * (size_t)ingest_pad(n)) + 2 * up(4 * (size_t)n) +
                        up(2 * (size_t)ingest_first_mins(n)) + up(2 * (size_t)ingest_upper_mins(n));
    const size_t all = up(n) + 2 * up(2 * (size_t)n) + (sort > tree ? sort : tree);
    const size_t state = up(8 * (2 * (size_t)n + 1)) + up(4 * (size_t)n);
    return ingest_small_bytes<uint16_t>(n, false) + (all > state ? all : state);
}

SAM_HD void ingest_place_lds(IngestArrays<uint16_t, uint32_t> &A, char *lds, uint32_t n)
{
    IngestBump b{lds};
    ingest_place_small(A, b, n);
    const IngestBump common = b;
    A.h_size = ingest_h_size(n);
    A.lev = b.take<uint8_t>(n);
    A.name1 = b.take<uint16_t>(n);
    A.grp = b.take<uint16_t>(n);
    A.pfx = A.name1;
    A.node = A.grp;
    IngestBump t = b;
    A.key = b.take<uint32_t>(A.h_size);
    A.val = b.take<uint32_t>(A.h_size);
    A.next = b.take<uint16_t>(A.h_size);
    A.cursor = b.take<uint32_t>(n);
    A.slot = b.take<uint16_t>(n);
    A.size = b.take<uint16_t>(n);
    A.sa = t.take<uint16_t>(n);
    A.lcp = t.take<uint16_t>(ingest_pad(n));
    A.par = t.take<uint16_t>(n);
    A.leaf = t.take<uint16_t>(n);
    A.m = t.take<uint32_t>(n);
    A.tab = reinterpret_cast<uint16_t *>(A.m);
    A.sec = t.take<uint32_t>(n);
    A.mins1 = t.take<uint16_t>(ingest_first_mins(n));
    A.mins = t.take<uint16_t>(ingest_upper_mins(n));
    IngestBump u = common;                 // after the records are written
    A.state = u.take<uint32_t>(2 * (2 * (size_t)n + 1));
    A.text = u.take<int32_t>(n);
}

// Levels of names that n tokens have: 16, 64, 256 ... of them at a time.
SAM_HD uint32_t ingest_name_levels(uint32_t n)
{
    uint32_t levels = 0;
    for (uint32_t w = 16; w < n; w *= 4) levels++;
    return levels;
}

// The large arrays in the sequence's own tables, which hold nothing yet: 16 indices a
// token in the record table, 8 in the slot table (plus its 64 spare slots).  What the
// records are written from is in the slot table; the part of it that was used is emptied again
// afterwards.
template <class I, class K>
SAM_HD void ingest_place_tables(IngestArrays<I, K> &A, const IngestSeq &q, char *lds, uint32_t n)
{
    IngestBump s{lds};
    ingest_place_small(A, s, n);
    A.mins = s.take<I>(ingest_upper_mins(n));
    A.state = nullptr;
    A.text = nullptr;
    A.names = nullptr;
    A.h_size = ingest_h_size(n);
    A.name1 = nullptr;
    IngestBump r{reinterpret_cast<char *>(q.rec)};
    A.grp = r.take<I>(n);
    A.lev = r.take<uint8_t>(n);
    IngestBump r2 = r;                     // the sort's arrays, and then the tree's
    A.key = r.take<K>(A.h_size);
    A.val = r.take<K>(A.h_size);
    A.cursor = r.take<K>(n);
    A.slot = r.take<I>(n);
    A.next = r.take<I>(A.h_size);
    A.size = r.take<I>(n);
    if (sizeof(I) == 4) {
        A.lo = r.take<uint32_t>(n);
        A.hi = r.take<uint32_t>(n);
    }
    A.sa = r2.take<I>(n);
    A.node = r2.take<I>(n);
    A.tab = r2.take<I>(2 * (size_t)n);
    A.mins1 = r2.take<I>(ingest_first_mins(n));
    IngestBump t{reinterpret_cast<char *>(q.slots)};
    A.lcp = t.take<I>(ingest_pad(n));
    A.names = reinterpret_cast<I *>(t.p);  // names live until lcp is known, the rest after it
    A.stride = (n + 15) & ~15u;
    A.par = t.take<I>(n);
    A.pfx = t.take<I>(n);
    A.leaf = t.take<I>(n);
    A.m = t.take<uint32_t>(n);
    A.sec = t.take<uint32_t>(n);
    const size_t rest = (size_t)(t.p - reinterpret_cast<char *>(q.slots)),
                 names = (size_t)(reinterpret_cast<char *>(A.names + ingest_name_levels(n) * (size_t)A.stride) -
                                  reinterpret_cast<char *>(q.slots));
    A.dirty = names > rest ? names : rest;
}

// Do the working arrays of n tokens fit into tables of these sizes?  (They do unless the
// slot table is smaller than usual.)
template <class I, class K>
inline bool ingest_tables_fit(uint32_t n, size_t rec_bytes, size_t slot_bytes)
{
    const size_t h = ingest_h_size(n), N = n;
    auto up = [](size_t x) { return (x + 15) / 16 * 16; };
    const size_t sort = 2 * up(sizeof(K) * h) + up(sizeof(I) * h) + up(sizeof(K) * N) + 2 * up(sizeof(I) * N) +
                        (sizeof(I) == 4 ? 2 * up(4 * N) : 0);
    const size_t tree = 2 * up(sizeof(I) * N) + up(2 * sizeof(I) * N) + up(sizeof(I) * ingest_first_mins(n));
    const size_t names = ingest_name_levels(n) * sizeof(I) * ((N + 15) / 16 * 16);
    const size_t rest = 3 * up(sizeof(I) * N) + 2 * up(4 * N);
    return up(sizeof(I) * N) + up(N) + (sort > tree ? sort : tree) <= rec_bytes &&
           up(sizeof(I) * ingest_pad(n)) + (names > rest ? names : rest) <= slot_bytes;
}

template <class I>
struct alignas(16) Eight { I v[8]; };

// ---- the tree of a sorted order -------------------------------------------------

// From the common lengths of neighbours in the sorted order to the states' ids: what one index
// does in each phase.  The phases are in this order, with a barrier between any two.
template <class I>
struct IngestTree {
    static constexpr I kNone = (I)~(I)0, kRoot = (I)(kNone - 1);
    uint32_t n;
    const I *sa;             // [n] position in each place of the sorted order
    const I *lcp;            // [ingest_pad(n)] common length with the place before, zeros behind
    I *node, *tab, *par, *pfx, *leaf;
    uint32_t *m, *sec;
    const I *mins1, *mins;   // minima of 8, and the levels above
    const uint32_t *level_at;      // where level j >= 2 starts in mins
    uint32_t tops;           // the highest level
    uint32_t *bits;
    const uint32_t *rank;

    // of the run that holds entry `at` of a level: which entries are below l
    SAM_HD uint32_t run_mask(uint32_t level, uint32_t at, uint32_t l) const
    {
        const I *p = level == 0 ? lcp : (level == 1 ? mins1 : mins + level_at[level]);
        const Eight<I> e = *reinterpret_cast<const Eight<I> *>(p + (at & ~7u));
        uint32_t mask = 0;
        for (int j = 0; j < 8; j++) mask |= (e.v[j] < l ? 1u : 0u) << j;
        return mask;
    }
    // the nearest boundary left of k with less than l (there is one: lcp[0] = 0), and right
    template <class C>
    SAM_HD uint32_t smaller_left(C &ctx, uint32_t k, uint32_t l) const
    {
        uint32_t level = 0, at = k, mask;
        while (!(mask = run_mask(level, at, l) & ((1u << (at & 7)) - 1u)) && level < tops) { at >>= 3; level++; }
        at = (at & ~7u) + ctx.log2(mask | 1u);
        for (; level; level--) {
            at *= 8;
            at += ctx.log2(run_mask(level - 1, at, l) | 1u);
        }
        return at;
    }
    template <class C>
    SAM_HD uint32_t smaller_right(C &ctx, uint32_t k, uint32_t l) const
    {
        uint32_t level = 0, at = k, mask;
        while (!(mask = run_mask(level, at, l) & (0xFEu << (at & 7)) & 0xFFu) && level < tops) { at >>= 3; level++; }
        at = (at & ~7u) + ctx.first(mask | 0x80u);
        for (; level; level--) {
            at *= 8;
            at += ctx.first(run_mask(level - 1, at, l) | 0x80u);
        }
        return at < n ? at : n;
    }
    SAM_HD uint32_t at_or_zero(uint32_t k) const { return k < n ? lcp[k] : 0u; }

    // Interval of boundary k: from lb to rb, the nearest boundaries with a smaller value.
    // Of the intervals that share lb only the widest has lcp[lb] >= lcp[rb], of those that
    // share rb only the widest of the others: one index each, in tab[].
    template <class C>
    SAM_HD void interval(C &ctx, uint32_t k) const
    {
        const uint32_t l = lcp[k];
        if (l == 0) { node[k] = kNone; return; }
        const uint32_t lb = smaller_left(ctx, k, l), rb = smaller_right(ctx, k, l);
        const bool left = lcp[lb] >= at_or_zero(rb);
        const uint32_t id = left ? lb : n + rb;
        tab[id] = (I)k;                                // any boundary of the interval will do
        node[k] = (I)id;
        par[k] = (I)(left ? lb : rb);
    }
    SAM_HD void represent(uint32_t k) const { if (lcp[k]) node[k] = tab[node[k]]; }
    SAM_HD void parent(uint32_t k) const
    {
        const bool rep = lcp[k] && node[k] == (I)k;
        par[k] = !rep ? kNone : (lcp[par[k]] == 0 ? kRoot : node[par[k]]);
        pfx[k] = kNone;
        m[k] = kNil;
        sec[k] = kNil;
    }
    SAM_HD void leaf_of(uint32_t k) const
    {
        const uint32_t i = sa[k], lk = lcp[k], rk = at_or_zero(k + 1), l = lk > rk ? lk : rk;
        I v = kRoot;
        if (l) {
            v = node[lk >= rk ? k : k + 1];
            // the prefix is as long as what it shares with a neighbour: it is that node
            if (l == i + 1) { pfx[v] = (I)i; v = par[v]; }
        }
        leaf[i] = v;
    }
    // first end positions: every prefix goes up until a smaller one has been there.  False: more
    // nodes than there are (kGuard).  kPeek: what others wrote before is read first (it only falls).
    template <bool kGuard, bool kPeek = false, class C>
    SAM_HD bool first_end(C &ctx, uint32_t i) const
    {
        uint32_t left = n + 1;
        for (I v = leaf[i]; v != kRoot && pfx[v] == kNone; v = par[v]) {
            if (kPeek && m[v] < i) break;
            if (ctx.lower(&m[v], i) < i) break;
            if (kGuard && !--left) return false;
        }
        return true;
    }
    // and the second: of the first ones of a node's children
    template <bool kPeek = false, class C>
    SAM_HD void second_end(C &ctx, uint32_t i) const
    {
        const I v = leaf[i];
        if (v != kRoot && pfx[v] == kNone && m[v] != i && !(kPeek && sec[v] < i)) ctx.lower(&sec[v], i);
        const I p = par[i];
        if (p != kNone && pfx[i] == kNone && p != kRoot && pfx[p] == kNone && m[p] != m[i] &&
            !(kPeek && sec[p] < m[i]))
            ctx.lower(&sec[p], m[i]);
    }
    SAM_HD bool cloned(uint32_t k) const { return par[k] != kNone && pfx[k] == kNone; }
    template <class C>
    SAM_HD void mark_clone(C &ctx, uint32_t k) const
    {
        if (cloned(k)) ctx.bit_or(&bits[sec[k] >> 5], 1u << (sec[k] & 31));
    }
    // ids, once rank[] has the running sum over bits[]
    template <class C>
    SAM_HD uint32_t prefix_id(C &ctx, uint32_t i) const
    {
        return 1 + i + rank[i >> 5] + ctx.popc(bits[i >> 5] & ((1u << (i & 31)) - 1u));
    }
    template <class C>
    SAM_HD uint32_t node_id(C &ctx, I v) const
    {
        if (v == kRoot) return 0;
        return pfx[v] != kNone ? prefix_id(ctx, pfx[v]) : prefix_id(ctx, sec[v]) + 1;
    }
};

// ---- the build --------------------------------------------------------------------

SAM_HD uint32_t ingest_hash(uint32_t k)
{
    k *= 0x9E3779B1u;
    k ^= k >> 15;
    return k * 0x2C1B3C6Du;
}
SAM_HD uint32_t ingest_hash(uint64_t k) { return ingest_hash((uint32_t)k ^ (uint32_t)(k >> 32) * 0x85EBCA77u); }

// Results: small[123] id of the last prefix, small[124] states, small[125] transitions,
// small[121] not 0: a loop that follows table contents ran into its guard (only if something
// else wrote to the tables meanwhile), the automaton is not to be used.
template <class L, bool kLds, class I, class K, class C>
SAM_HD void ingest_build(C &ctx, const IngestSeq &q, const IngestArrays<I, K> &A)
{
    const uint32_t n = q.n, hs = A.h_size;
    constexpr K kEmpty = (K)~(K)0;
    constexpr uint32_t kHalf = sizeof(K) * 4;
    constexpr I kAlone = (I)((I)1 << (sizeof(I) * 8 - 1));
    constexpr K kLow = (K)(((K)1 << kHalf) - 1);
    uint32_t *const small = A.small;
    uint32_t *const active = small;                  // [32] one flag per round
    const uint32_t words = n / 32 + 1;
    auto corrupt = [&] { ctx.bit_or(&small[121], 1u); };

    auto insert = [&](K key) -> uint32_t {
        auto put = [&](uint32_t times) -> uint32_t {
            uint32_t at = ctx.mulhi(ingest_hash(key), hs), left = hs;
            for (; left; left--) {
                const K old = ctx.cas(&A.key[at], kEmpty, key);
                if (old == kEmpty || old == key) break;
                at = at + 1 == hs ? 0 : at + 1;
            }
            if (!kLds && !left) corrupt();
            ctx.add(&A.val[at], (K)times);
            return at;
        };
        if (kLds) return put(1);
        return ctx.together(key, put);
    };

    // names of single tokens
    ctx.each(128, [&](uint32_t i) { small[i] = 0; });
    ctx.each(words, [&](uint32_t i) { A.bits[i] = 0; });
    ctx.each(hs, [&](uint32_t i) { A.key[i] = kEmpty; A.val[i] = 0; });
    ctx.sync();
    ctx.each(n, [&](uint32_t i) {
        const int32_t t = q.tok[i];
        q.text[i] = t;
        A.slot[i] = (I)insert((K)(uint32_t)t);
    });
    ctx.sync();
    ctx.each_full(hs, [&](uint32_t i, bool on) {
        const uint32_t c = on ? (uint32_t)A.val[i] : 0u;
        const uint32_t start = ctx.wave_add(&small[127], c);
        if (c) {
            A.val[i] = (K)(((K)start << kHalf) | c);
            A.lev[start] = 0;
        }
    });
    ctx.sync();
    auto take_names = [&](uint32_t i, uint32_t round) -> uint32_t {
        const K v = A.val[A.slot[i]];
        const uint32_t g = (uint32_t)(v >> kHalf), c = (uint32_t)(v & kLow);
        A.grp[i] = (I)(c == 1 ? g | (uint32_t)kAlone : g);
        A.size[g] = (I)c;
        if (c > 1) active[round] = 1;
        return g;
    };
    ctx.each(n, [&](uint32_t i) {
        const uint32_t g = take_names(i, 0);
        if (kLds) A.name1[i] = (I)g;
    });
    ctx.sync();

    // Names of the last 2h tokens from those of the last h.  The order inside a group is
    // that of the second names.  A group of c positions has c buckets, which cut the range of
    // second names evenly; a running sum over all buckets says where each starts, and the few
    // different pairs in one bucket (no more than c, nor than names in its range, hence no
    // more than about the square root of n) are compared with each other.  In a long text of one
    // period, say 134 tokens of 200 000, they are that many (251 ms; token by token 129): from the
    // first round on in which more than kCrowd pairs met in a bucket, the buckets of a group cut
    // the range of its own second names (52 ms).
    constexpr bool kSpread = sizeof(I) == 4;
    constexpr uint32_t kCrowd = 32;
    uint32_t *const crowded = small + 32;            // [32] one flag per round
    const uint32_t shift = ctx.log2(n) + 1;          // second names are 0 .. n
    auto bucket_of_pair = [&](auto spread, K key) -> uint32_t {
        const uint32_t g = (uint32_t)(key >> kHalf), second = (uint32_t)(key & kLow), size = A.size[g];
        if constexpr (decltype(spread)::value) {
            // rises with the second name, which is all that it has to
            const float width = (float)size / (float)(A.hi[g] - A.lo[g] + 1u);
            const uint32_t at = (uint32_t)((float)(second - A.lo[g]) * width);
            return g + (at < size ? at : size - 1u);
        }
        return g + (uint32_t)(((uint64_t)second * size) >> shift);
    };
    constexpr uint32_t kRuns = C::kThreads;          // of the running sum, one for each thread
    static_assert(kRuns <= kIngestParts, "part[] holds one sum for each thread");
    const uint32_t prun = (n + kRuns - 1) / kRuns;
    // all pairs of a round are in key[]: where each starts goes into the upper half of its val[]
    // (two bodies: the test for one in every bucket_of_pair cost 2 % of 12 x 40 000 tokens)
    auto rank_pairs = [&](auto spread, uint32_t round) {
        ctx.each(hs, [&](uint32_t i) {
            const K key = A.key[i];
            if (key != kEmpty) ctx.add(&A.cursor[bucket_of_pair(spread, key)], A.val[i]);
        });
        ctx.sync();
        ctx.each(kRuns, [&](uint32_t c) {
            uint32_t sum = 0;
            for (uint32_t k = c * prun; k < (c + 1) * prun && k < n; k++) sum += (uint32_t)A.cursor[k];
            A.part[c] = sum;
        });
        ctx.sync();
        ctx.exclusive_sums(A.part);
        ctx.each(kRuns, [&](uint32_t c) {
            uint32_t sum = A.part[c];
            for (uint32_t k = c * prun; k < (c + 1) * prun && k < n; k++) {
                const uint32_t mine = (uint32_t)A.cursor[k];
                A.cursor[k] = sum;
                sum += mine;
            }
        });
        ctx.sync();
        ctx.each(hs, [&](uint32_t i) {
            const K key = A.key[i];
            if (key == kEmpty) return;
            K *const w = &A.cursor[bucket_of_pair(spread, key)];
            for (K seen = *w;;) {
                A.next[i] = (I)(seen >> kHalf);
                const K old = ctx.cas(w, seen, (K)((seen & kLow) | ((K)(i + 1) << kHalf)));
                if (old == seen) break;
                seen = old;
            }
        });
        ctx.sync();
        ctx.each(hs, [&](uint32_t i) {
            const K key = A.key[i];
            if (key == kEmpty) return;
            const K w = A.cursor[bucket_of_pair(spread, key)];
            uint32_t start = (uint32_t)(w & kLow), left = hs;
            for (uint32_t j = (uint32_t)(w >> kHalf); j; j = A.next[j - 1]) {
                if (A.key[j - 1] < key) start += (uint32_t)(A.val[j - 1] & kLow);
                if (!kLds && !--left) { corrupt(); return; }
            }
            if (kSpread && (decltype(spread)::value || hs - left > kCrowd)) crowded[round] = 1;
            A.val[i] |= (K)((K)start << kHalf);
            if (start != (uint32_t)(key >> kHalf)) A.lev[start] = (uint8_t)round;
        });
        ctx.sync();
    };
    uint32_t round = 1;
    for (uint32_t h = 1; h < n; h *= 2, round++) {
        if (!active[round - 1]) break;
        if (!kLds && h >= 16 && (ctx.log2(h) & 1) == 0) {
            const uint32_t j = (ctx.log2(h) - 4) / 2;
            if (j < 7) ctx.each(n, [&](uint32_t i) { A.names[j * A.stride + i] = A.grp[i]; });
        }
        ctx.each(hs, [&](uint32_t i) { A.key[i] = kEmpty; A.val[i] = 0; });
        const bool spread = kSpread && round > 1 && ctx.uniform(crowded[round - 1]);
        ctx.each(n, [&](uint32_t i) { A.cursor[i] = 0; });
        if (kSpread && spread) ctx.each(n, [&](uint32_t i) { A.lo[i] = kNil; A.hi[i] = 0; });
        ctx.sync();
        ctx.each(n, [&](uint32_t i) {
            const I g = A.grp[i];
            if (g & kAlone) { A.cursor[g & (I)~kAlone] = 1; return; }
            const uint32_t second = i >= h ? (uint32_t)(A.grp[i - h] & (I)~kAlone) + 1u : 0u;
            A.slot[i] = (I)insert((K)(((K)g << kHalf) | (K)second));
        });
        ctx.sync();
        if (kSpread && spread) {
            ctx.each(hs, [&](uint32_t i) {
                const K key = A.key[i];
                if (key == kEmpty) return;
                ctx.lower(&A.lo[key >> kHalf], (uint32_t)(key & kLow));
                ctx.raise(&A.hi[key >> kHalf], (uint32_t)(key & kLow));
            });
            ctx.sync();
        }
        if constexpr (kSpread) {
            if (spread) rank_pairs(std::true_type{}, round);
            else rank_pairs(std::false_type{}, round);
        } else {
            rank_pairs(std::false_type{}, round);
        }
        ctx.each(n, [&](uint32_t i) {
            if (!(A.grp[i] & kAlone)) take_names(i, round);
        });
        ctx.sync();
    }
    // sorted order, and the common length of neighbours: at least h tokens if their groups
    // parted in the round that took h to 2h, and fewer than 2h
    ctx.each(n, [&](uint32_t i) { A.sa[A.grp[i] & (I)~kAlone] = (I)i; });
    ctx.sync();
    ctx.each(n, [&](uint32_t k) {
        const uint32_t r = A.lev[k];
        uint32_t l = 0;
        if (k > 0 && r > 0) {
            l = 1u << (r - 1);
            const uint32_t a = A.sa[k - 1], b = A.sa[k];
            const uint32_t most = (a < b ? a : b) + 1;
            if (kLds) {
                while (l < most && A.name1[a - l] == A.name1[b - l]) l++;
            } else {
                // strides of 16 * 4^j tokens by their names, the last few token by token
                for (int j = 6; j >= 0; j--) {
                    const uint32_t w = 16u << (2 * j);
                    if (w >= (1u << (r - 1)) * 2u) continue;          // not named, or too long
                    while (l + w <= most) {
                        const I *const nj = A.names + (uint32_t)j * A.stride;
                        const I x = nj[a - l], y = nj[b - l];
                        if (x != y) break;
                        l += w;
                    }
                }
                while (l < most && q.tok[a - l] == q.tok[b - l]) l++;
            }
        }
        A.lcp[k] = (I)l;
    });
    ctx.sync();
    ctx.each(ingest_pad(n) - n, [&](uint32_t k) { A.lcp[n + k] = 0; });
    ctx.sync();
    uint32_t *const level_at = A.part;               // where level j >= 2 starts in mins
    uint32_t tops = 1;
    {
        const I *below = A.lcp;
        uint32_t count = ingest_pad(n);
        I *out = A.mins1;
        for (;;) {
            const uint32_t real = count / 8, padded = ingest_pad(real);
            ctx.each(padded, [&](uint32_t w) {
                I least = 0;
                if (w < real) {
                    const Eight<I> e = *reinterpret_cast<const Eight<I> *>(below + 8 * w);
                    least = e.v[0];
                    for (int j = 1; j < 8; j++) least = e.v[j] < least ? e.v[j] : least;
                }
                out[w] = least;
            });
            if (tops >= 2) ctx.each(1, [&](uint32_t) { level_at[tops] = (uint32_t)(out - A.mins); });
            ctx.sync();
            if (padded == 8) break;
            below = out;
            out = tops == 1 ? A.mins : out + padded;
            count = padded;
            tops++;
        }
    }
    const IngestTree<I> tree{n, A.sa, A.lcp, A.node, A.tab, A.par, A.pfx, A.leaf, A.m, A.sec, A.mins1, A.mins,
                             level_at, tops, A.bits, A.rank};
    ctx.each(n, [&](uint32_t k) { tree.interval(ctx, k); });
    ctx.sync();
    ctx.each(n, [&](uint32_t k) { tree.represent(k); });
    ctx.sync();
    ctx.each(n, [&](uint32_t k) { tree.parent(k); });
    ctx.sync();
    ctx.each(n, [&](uint32_t k) { tree.leaf_of(k); });
    ctx.sync();
    ctx.each(n, [&](uint32_t i) { if (!tree.template first_end<!kLds>(ctx, i)) corrupt(); });
    ctx.sync();
    ctx.each(n, [&](uint32_t i) { tree.second_end(ctx, i); });
    ctx.sync();
    ctx.each(n, [&](uint32_t k) { tree.mark_clone(ctx, k); });
    ctx.sync();
    // ids
    uint32_t *const part = small + 64;               // [60]: sums of runs of words
    constexpr uint32_t kParts = 56;
    const uint32_t run = (words + kParts - 1) / kParts;
    auto run_of = [&](uint32_t c, uint32_t &lo, uint32_t &hi) {
        lo = c * run; hi = lo + run;
        if (lo > words) lo = words;
        if (hi > words) hi = words;
    };
    ctx.each(kParts, [&](uint32_t c) {
        uint32_t lo, hi, sum = 0;
        run_of(c, lo, hi);
        for (uint32_t w = lo; w < hi; w++) sum += ctx.popc(A.bits[w]);
        part[c] = sum;
    });
    ctx.sync();
    ctx.each(kParts, [&](uint32_t c) {
        uint32_t lo, hi, sum = 0;
        run_of(c, lo, hi);
        for (uint32_t j = 0; j < c; j++) sum += part[j];
        for (uint32_t w = lo; w < hi; w++) { A.rank[w] = sum; sum += ctx.popc(A.bits[w]); }
        if (c == kParts - 1) small[124] = 1 + n + sum;
    });
    ctx.sync();
    auto prefix_id = [&](uint32_t i) -> uint32_t { return tree.prefix_id(ctx, i); };
    auto node_id = [&](I v) -> uint32_t { return tree.node_id(ctx, v); };
    // records, with the transition of the first occurrence inline
    ctx.each(n, [&](uint32_t i) {
        const uint32_t id = prefix_id(i);
        if (i == 0) L::store(q.rec, 0, 0, kNil, 0, (uint32_t)q.tok[0], 1);
        const bool more = i + 1 < n;
        L::store(q.rec, id, i + 1, node_id(A.leaf[i]), i + 1, more ? (uint32_t)q.tok[i + 1] : kNil,
                 more ? prefix_id(i + 1) : 0u);
        if (tree.cloned(i))
            L::store(q.rec, prefix_id(A.sec[i]) + 1, A.lcp[i], node_id(A.par[i]), A.m[i] + 1,
                     (uint32_t)q.tok[A.m[i] + 1], 0u);
    });
    ctx.sync();
    const uint32_t states = small[124];
    if (kLds) {
        // the walks below read the states and the text from LDS
        ctx.each(states, [&](uint32_t v) {
            uint32_t len, link, endpos, itok;
            L::load(q.rec, v, len, link, endpos, itok);
            A.state[2 * v] = len | (link << 16);
            A.state[2 * v + 1] = endpos | 0xFFFF0000u;
        });
        ctx.each(n, [&](uint32_t i) { A.text[i] = q.tok[i]; });
        ctx.sync();
        // LDS is this workgroup's alone, but what was just read went through the tables: links that
        // lead to shorter states end at the root
        ctx.each(states, [&](uint32_t v) {
            const uint32_t up = A.state[2 * v] >> 16;
            if (v && (up >= states || (A.state[2 * up] & 0xFFFFu) >= (A.state[2 * v] & 0xFFFFu))) corrupt();
        });
        ctx.sync();
        if (small[121]) return;
    } else {
        // What of the slot table held the arrays above is emptied again, about 20 bytes a token
        // (24 to 32 with 32-bit indices); the rest, which may be far larger, still is empty.
        uint64_t *const s = reinterpret_cast<uint64_t *>(q.slots);
        ctx.each((uint32_t)(A.dirty / 8), [&](uint32_t i) { s[i] = ~(uint64_t)0; });
    }
    // the root's link reads as kNil or, from LDS, as 0xFFFF; nothing asks for it
    auto link_of = [&](uint32_t v) -> uint32_t { return kLds ? A.state[2 * v] >> 16 : L::link(q.rec, v); };
    auto len_of = [&](uint32_t v) -> uint32_t { return kLds ? A.state[2 * v] & 0xFFFFu : L::len(q.rec, v); };
    // The state that holds w tokens of the suffix path of u (u is that long, w > 0).
    auto ancestor = [&](uint32_t u, uint32_t w) -> uint32_t {
        for (uint32_t left = states;;) {
            const uint32_t up = link_of(u);
            if (len_of(up) < w) return u;
            u = up;
            if (!kLds && !--left) { corrupt(); return u; }
        }
    };
    // inline targets of the clones: they are the ids that follow a prefix with its bit set
    ctx.each(n, [&](uint32_t i) {
        if (!((A.bits[i >> 5] >> (i & 31)) & 1u)) return;
        const uint32_t v = prefix_id(i) + 1;
        uint32_t len, link, endpos, itok;
        if (kLds) {
            len = len_of(v);
            endpos = A.state[2 * v + 1] & 0xFFFFu;
        } else {
            L::load(q.rec, v, len, link, endpos, itok);
        }
        L::store_idst(q.rec, v, ancestor(prefix_id(endpos), len + 1));
    });
    ctx.sync();
    // All other transitions.  Position i brings the token t behind it to every state on its
    // suffix path, up to one that has it from an earlier comer: that one goes on from there.
    // A state whose first occurrence ends at i has t inline already, and only i passes it.
    auto token = [&](uint32_t i) -> uint32_t { return (uint32_t)(kLds ? A.text[i] : q.tok[i]); };
    auto look = [&](uint32_t v, uint32_t &len, uint32_t &link, uint32_t &endpos, uint32_t &itok) {
        if (kLds) {
            const uint32_t a = A.state[2 * v];
            len = a & 0xFFFFu;
            link = a >> 16;
            endpos = A.state[2 * v + 1] & 0xFFFFu;
            itok = (uint32_t)A.text[endpos];
        } else {
            L::load(q.rec, v, len, link, endpos, itok);
        }
    };
    auto claim = [&](uint32_t v, uint32_t t, uint32_t &at) -> int {
        const int got = ingest_claim<L>(ctx, q.slots, q.n_buckets, v, t, at);
        if (got == 2) corrupt();
        return got;
    };
    auto enter = [&](uint32_t at, uint32_t v, uint32_t endpos, uint32_t dst) {
        if (kLds && L::kHead16)
            L::fill_next(q.slots, at, dst, ctx.exch(&A.state[2 * v + 1], endpos | (at << 16)) >> 16);
        else
            L::fill(ctx, q.rec, q.slots, at, v, endpos, dst);
    };
    uint32_t *const walks = small;                   // [kWalks][3] walks handed over
    ctx.each(n - 1, [&](uint32_t i) {
        const uint32_t t = token(i + 1);
        uint32_t u = prefix_id(i + 1), v = link_of(prefix_id(i)), made = 0;
        for (uint32_t step = 1;; step++) {
            uint32_t len, link, endpos, itok, at = 0;
            look(v, len, link, endpos, itok);
            if (itok == t) {
                if (endpos != i + 1) break;
            } else {
                if (claim(v, t, at)) break;
                u = ancestor(u, len + 1);
                enter(at, v, endpos, u);
                made++;
            }
            if (v == 0) break;
            v = link;
            if (step == kLongWalk) {
                const uint32_t k = ctx.add(&small[122], 1u);
                if (k < kWalks) { walks[3 * k] = i; walks[3 * k + 1] = v; walks[3 * k + 2] = u; break; }
            }
            if (!kLds && step == states) { corrupt(); break; }
        }
        if (made) ctx.add(&small[126], made);
    });
    ctx.sync();
    // The end of a long run of one token, or of a short period, brings a new token to as many
    // states as the run is long; a position that walks alone gets one compare-and-swap after the
    // other through.  So a walk of more than kLongWalk states is handed over to a wave: 64 states
    // at a time are listed by their links and then tried together.  It goes on if the last of
    // them was still without the token; whoever has the token at one of the others meets it at
    // the next one up and stops there.  (5999 equal tokens and another one: 5.9 ms with the walk left
    // to its position, 2.2 ms; 3.4 ms token by token.)
    ctx.each_wave(small[122] < kWalks ? small[122] : kWalks, A.part, [&](uint32_t k, uint32_t *list) {
        const uint32_t i = walks[3 * k], t = token(i + 1);
        uint32_t v = walks[3 * k + 1], u = walks[3 * k + 2];
        for (uint32_t left = states;; left--) {
            if (!kLds && !left) { corrupt(); break; }
            uint32_t count = 0;
            bool more = true, last_tried = false;
            while (more && count < 64) {
                uint32_t len, link, endpos, itok;
                look(v, len, link, endpos, itok);
                last_tried = itok != t;
                if (!last_tried && endpos != i + 1) { more = false; break; }
                list[count++] = last_tried ? v : kNil;
                more = v != 0;
                v = link;
            }
            ctx.wave_sync();
            ctx.lanes([&](uint32_t lane) {
                if (lane >= count || list[lane] == kNil) return;
                const uint32_t w = list[lane];
                uint32_t len, link, endpos, itok, at = 0, to = kNil;
                if (claim(w, t, at) == 0) {
                    look(w, len, link, endpos, itok);
                    to = ancestor(u, len + 1);
                    enter(at, w, endpos, to);
                    ctx.add(&small[126], 1u);
                }
                list[lane] = to;
            });
            ctx.wave_sync();
            if (!more) break;
            if (last_tried) {
                u = list[63];
                if (u == kNil) break;
            }
            ctx.wave_sync();
        }
    });
    if (kLds && L::kHead16) {
        ctx.sync();
        ctx.each(states, [&](uint32_t v) {
            const uint32_t head = A.state[2 * v + 1] >> 16;
            if (head != 0xFFFFu) L::store_head(q.rec, v, head);
        });
    }
    ctx.sync();
    ctx.each(1, [&](uint32_t) {
        small[125] = small[126] + small[124] - 1;
        small[123] = prefix_id(n - 1);
    });
    ctx.sync();
}

}  // namespace sam
