// An automaton built by the whole chip at once: of the corpus, or of prompts too long for
// one workgroup's LDS.
//
// The method is the one of sam_ingest.h: the suffix links form the tree of the sorted
// reversed prefixes, the ids follow from it, the transitions are inserted in any order.
// What differs is who does it and how the order is found.  Every phase is a launch of its own
// over all positions of all texts, so the barrier between phases is the launch boundary; and
// the sort is a radix sort by the last few tokens (as many as fit into 64 bits), followed by
// doubling rounds in which a position only counts the smaller second names of its own group, which
// lie side by side: one random access a position and round, against eight or so for the hash
// tables that one workgroup uses.
//
// This file holds the layout of the working arrays and what one index does in each phase, so the
// same source also runs on the CPU; the phases that need lanes working together (the radix
// sort, running sums, minima) are in sam_bulk.hip.
#pragma once
#include <stdint.h>
#include <string.h>

#include "sam_ingest.h"

namespace sam {

constexpr uint32_t kBulkTile = 2048;         // places that a workgroup sorts at a time
constexpr uint32_t kBulkBlocks = 256;        // runs of whole tiles that a text is cut into, at most
constexpr uint32_t kBulkLarge = 1024;        // groups beyond are sorted by a workgroup each
constexpr uint32_t kBulkStart = 0x80000000u; // gs[]: a group starts here, its size below; else: where
constexpr uint32_t kBulkAlone = kBulkStart | 1u;
constexpr uint32_t kBulkLdsTokens = 4096;    // never for texts that are sure to fit into LDS

constexpr uint32_t kBulkWalk = 32;           // steps of a walk that a lane makes alone

// words of a text's control block, up to the states
enum : uint32_t {
    kCtlActive = 0,          // [32] round r has groups to part
    kCtlQueued = 32,         // [32] large ones among them
    kCtlTops = 64, kCtlLargest,    // levels of minima; size of the largest group that was queued
    kCtlLevel = 72,          // [16] where the levels start
    kBulkCtl = 96
};
// and of its counts, to the end
enum : uint32_t { kCntStates, kCntCorrupt, kCntMade, kBulkCounts };

struct BulkCut { uint32_t blocks, chunk; };
SAM_HD BulkCut bulk_cut(uint32_t count)
{
    const uint32_t tiles = (count + kBulkTile - 1) / kBulkTile, per = (tiles + kBulkBlocks - 1) / kBulkBlocks;
    return BulkCut{(tiles + per - 1) / per, per * kBulkTile};
}

// The sort by the last tokens: `tokens` of them, `bits` each, in passes of 8 bits; the pass p writes
// the buffers p & 1.  A name of h = tokens << r tokens is what round r starts from.
struct BulkSort { uint32_t tokens, bits, passes; };
// As many tokens as key_bits hold (64 at most), two if they do not hold two.
inline BulkSort bulk_sort_for(uint32_t vocab, uint32_t key_bits)
{
    uint32_t bits = 1;
    while (bits < 32 && (vocab >> bits)) bits++;               // values 0 .. vocab
    const uint32_t tokens = key_bits / bits > 2 ? key_bits / bits : 2;
    return BulkSort{tokens, bits, (tokens * bits + 7) / 8};
}

template <class I>
struct BulkSeq {
    const int32_t *tok;      // every token inside the vocabulary
    uint32_t n;
    uint32_t of;             // the sequence
    uint32_t *counts;
    uint32_t *ctl;
    uint64_t *key0, *key1;   // [n] the last tokens, the very last on top
    uint32_t *pos0, *pos1;   // [n] sorted positions; round r reads pos(first + r), writes the other
    uint32_t *gs0, *gs1;     // [n] by place: start and size of its group; round r reads gs(r)
    uint32_t *sec, *sec2;    // [n] by place: second name
    uint32_t *name;          // [n] by position: start of its group
    uint8_t  *lev;           // [n] by place: 1 + the round in which a group came to start here
    uint32_t *queue0, *queue1;     // starts of large groups; round r reads queue(r)
    uint32_t *hist, *sums;
    I *sa, *lcp, *node, *tab, *par, *pfx, *leaf, *mins1, *mins;
    uint32_t *m, *second, *bits, *rank;
    size_t dirty;            // bytes of the second region that are used

    // (not arrays: their index is no constant)
    SAM_HD uint64_t *key(uint32_t k) const { return k & 1 ? key1 : key0; }
    SAM_HD uint32_t *pos(uint32_t k) const { return k & 1 ? pos1 : pos0; }
    SAM_HD uint32_t *gs(uint32_t k) const { return k & 1 ? gs1 : gs0; }
    SAM_HD uint32_t *queue(uint32_t k) const { return k & 1 ? queue1 : queue0; }

    SAM_HD IngestTree<I> tree() const
    {
        return IngestTree<I>{n, sa, lcp, node, tab, par, pfx, leaf, m, second, mins1, mins,
                             ctl + kCtlLevel, ctl[kCtlTops], bits, rank};
    }
};

SAM_HD size_t bulk_up(size_t x) { return (x + 15) / 16 * 16; }

// Three regions.  The first: 32 bytes a token and 96; the records, where they lie over it, are
// written when nothing of it is needed any more.  The second: 24 bytes a token and 192 (16 with 16-bit
// indices), which the records are written from.  The third: see bulk_third_bytes; a sequence's text, which
// is written after the records.  What lies over each other is never alive together: the group arrays
// over the keys once the first groups are known, the tree over the sort (but not over name[], which
// the common lengths are found from), lev[] under second[].
SAM_HD size_t bulk_first_bytes(size_t n) { return 32 * n + 96; }
template <class I>
SAM_HD size_t bulk_second_bytes(size_t n) { return (4 * sizeof(I) + 8) * n + 192; }
SAM_HD size_t bulk_third_bytes(uint32_t n)
{
    return 4 * kBulkCtl + bulk_up(4 * 256 * (size_t)bulk_cut(n).blocks) + 2 * bulk_up(4 * (size_t)(n / kBulkLarge + 1)) +
           2 * bulk_up(4 * (size_t)(n / 32 + 1)) + 4 * kBulkBlocks;
}

// Do n tokens' working arrays fit into a sequence's own tables?  (With 16-bit indices they do if there is
// room for three more tokens.)
template <class I>
SAM_HD bool bulk_tables_fit(uint32_t n, uint32_t max_seq_len, size_t rec_bytes, size_t slot_bytes)
{
    return max_seq_len >= kBulkLdsTokens && n <= max_seq_len && bulk_first_bytes(n) <= rec_bytes &&
           bulk_second_bytes<I>(n) <= slot_bytes && bulk_third_bytes(n) <= 4 * (size_t)max_seq_len;
}

template <class I>
SAM_HD void bulk_place(BulkSeq<I> &q, char *first, char *second, char *third)
{
    const size_t n = q.n;
    IngestBump a{first};
    q.pos0 = a.take<uint32_t>(n);
    q.pos1 = a.take<uint32_t>(n);
    q.gs0 = a.take<uint32_t>(n);
    q.name = a.take<uint32_t>(n);
    IngestBump k = a;
    q.key0 = a.take<uint64_t>(n);
    q.key1 = a.take<uint64_t>(n);
    q.gs1 = k.take<uint32_t>(n);
    q.sec = k.take<uint32_t>(n);
    q.sec2 = k.take<uint32_t>(n);
    IngestBump t{first};
    q.sa = t.take<I>(n);
    q.node = t.take<I>(n);
    q.tab = t.take<I>(2 * n);
    q.mins1 = t.take<I>(ingest_first_mins(q.n));
    q.mins = t.take<I>(ingest_upper_mins(q.n));
    IngestBump b{second};
    q.lcp = b.take<I>(ingest_pad(q.n));
    q.par = b.take<I>(n);
    q.pfx = b.take<I>(n);
    q.leaf = b.take<I>(n);
    q.m = b.take<uint32_t>(n);
    q.second = b.take<uint32_t>(n);
    q.lev = reinterpret_cast<uint8_t *>(q.second);
    q.dirty = (size_t)(b.p - second);
    IngestBump c{third};
    q.ctl = c.take<uint32_t>(kBulkCtl);
    q.hist = c.take<uint32_t>(256 * (size_t)bulk_cut(q.n).blocks);
    q.queue0 = c.take<uint32_t>(n / kBulkLarge + 1);
    q.queue1 = c.take<uint32_t>(n / kBulkLarge + 1);
    q.bits = c.take<uint32_t>(n / 32 + 1);
    q.rank = c.take<uint32_t>(n / 32 + 1);
    q.sums = c.take<uint32_t>(kBulkBlocks);
}

// Levels of minima above the common lengths of n places, and where each starts.
SAM_HD uint32_t bulk_levels(uint32_t n, uint32_t *at)
{
    uint32_t tops = 1, where = 0;
    for (uint32_t c = ingest_first_mins(n); c > 8;) {
        c = ingest_pad(c / 8);
        tops++;
        if (at) at[tops] = where;
        where += c;
    }
    return tops;
}

// The last `tokens` tokens of the prefix that ends at i; nothing (0) in front of the text.
SAM_HD uint64_t bulk_key(const int32_t *tok, uint32_t i, const BulkSort &s)
{
    uint64_t k = 0;
    for (uint32_t j = 0; j < s.tokens; j++)
        k = (k << (s.bits & 63)) | (i >= j ? (uint64_t)((uint32_t)tok[i - j] + 1u) : 0u);
    return k;
}

// ---- the phases: what one index does ---------------------------------------------

// Rounds.  Second names of the places whose group is not down to one.
template <class I>
SAM_HD void bulk_gather(const BulkSeq<I> &q, uint32_t first, uint32_t round, uint32_t h, uint32_t k)
{
    if (q.gs(round)[k] == kBulkAlone) return;
    const uint32_t i = q.pos(first + round)[k];
    q.sec[k] = i >= h ? q.name[i - h] + 1u : 0u;
}

struct Four { uint32_t v[4]; };

// Counts the smaller second names of the own group, and the equal ones before its own place: the
// new place.  Groups beyond kBulkLarge are left to bulk_rank_large (kAll: they are not).  True: the
// new group has others.
template <bool kAll, class I>
SAM_HD bool bulk_rank(const BulkSeq<I> &q, uint32_t first, uint32_t round, uint32_t k)
{
    const uint32_t *const gs = q.gs(round), *const pos = q.pos(first + round);
    uint32_t *const to_gs = q.gs(round + 1), *const to_pos = q.pos(first + round + 1);
    const uint32_t v = gs[k];
    if (v == kBulkAlone) {
        to_gs[k] = v;
        to_pos[k] = pos[k];
        return false;
    }
    const uint32_t g = v & kBulkStart ? k : v, size = gs[g] & ~kBulkStart;
    if (!kAll && size > kBulkLarge) return false;
    const uint32_t *const sec = q.sec + g, own = k - g, mine = sec[own];
    uint32_t less = 0, same = 0, before = 0, j = 0;
    for (; j + 4 <= size; j += 4) {
        Four f;
        memcpy(&f, sec + j, sizeof(f));
        for (uint32_t u = 0; u < 4; u++) {
            less += f.v[u] < mine;
            same += f.v[u] == mine;
            before += f.v[u] == mine && j + u < own;
        }
    }
    for (; j < size; j++) {
        less += sec[j] < mine;
        same += sec[j] == mine;
        before += sec[j] == mine && j < own;
    }
    const uint32_t i = pos[k], start = g + less;
    to_pos[start + before] = i;
    to_gs[start + before] = before ? start : kBulkStart | same;
    if (less) {
        q.name[i] = start;
        if (!before) q.lev[start] = (uint8_t)(round + 1);
    }
    return same > 1;
}

// All names are places now.
template <class I>
SAM_HD void bulk_order(const BulkSeq<I> &q, uint32_t i) { q.sa[q.name[i]] = (I)i; }

// How many tokens the prefixes that end at a and b have in common at their ends, `l` of them known to.
SAM_HD uint32_t bulk_agree(const int32_t *tok, uint32_t a, uint32_t b, uint32_t l)
{
    const uint32_t most = (a < b ? a : b) + 1;
    while (l + 4 <= most) {
        Four x, y;
        memcpy(&x, tok + (a - l - 3), sizeof(x));
        memcpy(&y, tok + (b - l - 3), sizeof(y));
        if (x.v[3] != y.v[3]) return l;
        if (x.v[2] != y.v[2]) return l + 1;
        if (x.v[1] != y.v[1]) return l + 2;
        if (x.v[0] != y.v[0]) return l + 3;
        l += 4;
    }
    while (l < most && tok[a - l] == tok[b - l]) l++;
    return l;
}

// Common lengths of a run of positions with the place before theirs, the last position first: one
// whose successor has L of them has L - 1 at least, and one that parted in round r has tokens << r.
// Where there are long ones (more than kBulkLong tokens) a wave takes a run, 256 tokens a step, and the
// runs grow with the longest: what the first position of each compares stays a few tokens for each
// position, and texts that repeat in large are not quadratic.
constexpr uint32_t kBulkLong = 1024;
template <class I>
SAM_HD uint32_t bulk_longest(const BulkSeq<I> &q, uint32_t tokens)      // not less than half of it
{
    uint32_t h = tokens;
    for (uint32_t r = 0; r < 32 && q.ctl[kCtlActive + r] && h < q.n; r++) h *= 2;
    return h;
}

template <class I, class Agree>
SAM_HD void bulk_common(const BulkSeq<I> &q, uint32_t tokens, uint32_t run, uint32_t c, Agree agree)
{
    const uint32_t lo = c * run, hi = q.n - lo > run ? lo + run : q.n;
    uint32_t l = 0;
    for (uint32_t i = hi; i-- > lo;) {
        const uint32_t k = q.name[i];
        l = l ? l - 1 : 0;
        if (k == 0) {
            l = 0;
        } else {
            const uint32_t r = q.lev[k], known = r ? tokens << (r - 1) : 0;
            l = agree(i, (uint32_t)q.sa[k - 1], l > known ? l : known);
        }
        q.lcp[k] = (I)l;
    }
    if (lo == 0)
        for (uint32_t k = q.n; k < ingest_pad(q.n); k++) q.lcp[k] = 0;
}

// ---- where the states go ----------------------------------------------------------

// A sequence's own tables.
template <class L>
struct BulkTables {
    void *rec, *slots;
    uint32_t n_buckets;
    const int32_t *tok;
    uint32_t n;
    // The root gets a transition for every different token of the text, and exchanges of its list's head
    // follow each other: a workgroup chains its own in LDS ([0] the last slot, kNil at first; [1] the
    // first one) and hangs the chain into the root's list at its end.  (Walks of 12 prompts of 40 001
    // tokens, vocabulary 32 000: 325 us with an exchange for each, 190 so; 512 of 8000 1.47 ms, 1.30.)
    uint32_t *chain = nullptr;

    SAM_HD void store(uint32_t s, uint32_t len, uint32_t link, uint32_t endpos, uint32_t itok, uint32_t idst) const
    {
        L::store(rec, s, len, link, endpos, itok, idst);
    }
    SAM_HD void load(uint32_t s, uint32_t &len, uint32_t &link, uint32_t &endpos, uint32_t &itok) const
    {
        L::load(rec, s, len, link, endpos, itok);
    }
    SAM_HD void len_link(uint32_t s, uint32_t &len, uint32_t &link) const
    {
        len = L::len(rec, s);
        link = L::link(rec, s);
    }
    SAM_HD uint32_t idst(uint32_t s) const { return L::idst(rec, s); }
    template <class C>
    SAM_HD uint32_t head(C &ctx, uint32_t s) const { return L::head(ctx, rec, s); }
    SAM_HD void store_idst(uint32_t s, uint32_t dst) const { L::store_idst(rec, s, dst); }
    template <class C>
    SAM_HD int claim(C &ctx, uint32_t v, uint32_t t, uint32_t &at) const
    {
        return ingest_claim<L, true>(ctx, slots, n_buckets, v, t, at);
    }
    template <class C>
    SAM_HD void enter(C &ctx, uint32_t at, uint32_t v, uint32_t, uint32_t endpos, uint32_t dst) const
    {
        if (v) { L::fill(ctx, rec, slots, at, v, endpos, dst); return; }
        const uint32_t before = ctx.exch(&chain[0], at);
        if (before == kNil) chain[1] = at;
        L::link_slot(slots, at, dst, before);
    }
    template <class C>
    SAM_HD void hang(C &ctx) const
    {
        if (chain[0] != kNil) L::hang(ctx, rec, slots, chain[0], chain[1]);
    }
};

// The corpus: states of 16 bytes {length, link, min_endpos, target of the transition that follows
// the first occurrence}; the root's transitions in a table by token, the others in an
// open-addressed one that the tables of the library are made from afterwards.
struct BulkCorpus {
    struct State { uint32_t len, link, endpos, idst; };
    State *rec;
    uint64_t *key;           // [n_slots] state | token << 32, all ones: empty
    uint32_t *dst;           // [n_slots]
    uint32_t n_slots;
    RootEnt *root;
    const int32_t *tok;
    uint32_t n;
    uint32_t *chain = nullptr;   // none is needed: the root's are in a table by token

    SAM_HD void store(uint32_t s, uint32_t len, uint32_t link, uint32_t endpos, uint32_t, uint32_t idst) const
    {
        rec[s] = State{len, link, endpos, idst};
    }
    SAM_HD void load(uint32_t s, uint32_t &len, uint32_t &link, uint32_t &endpos, uint32_t &itok) const
    {
        const State r = rec[s];
        len = r.len; link = r.link; endpos = r.endpos;
        itok = r.endpos < n ? (uint32_t)tok[r.endpos] : kNil;
    }
    SAM_HD void len_link(uint32_t s, uint32_t &len, uint32_t &link) const
    {
        len = rec[s].len;
        link = rec[s].link;
    }
    SAM_HD uint32_t idst(uint32_t s) const { return rec[s].idst; }
    SAM_HD void store_idst(uint32_t s, uint32_t dst) const { rec[s].idst = dst; }
    template <class C>
    SAM_HD int claim(C &ctx, uint32_t v, uint32_t t, uint32_t &at) const
    {
        if (v == 0) return root[t].dst || ctx.cas(&root[t].dst, 0u, kNil) ? 1 : 0;
        const uint64_t mine = (uint64_t)v | ((uint64_t)t << 32);
        at = ctx.mulhi(hash_key(v, t), n_slots);
        for (uint32_t left = n_slots; left; left--) {
            uint64_t old = key[at];
            if (old == ~(uint64_t)0) old = ctx.cas(&key[at], ~(uint64_t)0, mine);
            if (old == ~(uint64_t)0) return 0;
            if (old == mine) return 1;
            at = at + 1 == n_slots ? 0 : at + 1;
        }
        return 2;
    }
    template <class C>
    SAM_HD void enter(C &, uint32_t at, uint32_t v, uint32_t t, uint32_t, uint32_t to) const
    {
        if (v == 0) root[t].dst = to;
        else dst[at] = to;
    }
    template <class C>
    SAM_HD void hang(C &) const {}
};

// ---- states and transitions -------------------------------------------------------

// Records, with the transition of the first occurrence: of a prefix to the next one, and of the
// others the prefix on whose suffix path its target lies, for the time being.
template <class S, class C, class I>
SAM_HD void bulk_records(C &ctx, const BulkSeq<I> &q, const IngestTree<I> &t, const S &out, uint32_t i)
{
    const bool more = i + 1 < q.n;
    const uint32_t id = t.prefix_id(ctx, i);
    if (i == 0) out.store(0, 0, kNil, 0, (uint32_t)q.tok[0], 1);
    out.store(id, i + 1, t.node_id(ctx, t.leaf[i]), i + 1, more ? (uint32_t)q.tok[i + 1] : kNil,
              more ? t.prefix_id(ctx, i + 1) : 0u);
    if (t.cloned(i)) {
        const uint32_t first = t.m[i];
        out.store(t.prefix_id(ctx, t.sec[i]) + 1, t.lcp[i], t.node_id(ctx, t.par[i]), first + 1,
                  (uint32_t)q.tok[first + 1], t.prefix_id(ctx, first + 1));
    }
}

// Climbs a suffix path: the state that holds w tokens of it, for one w after the other (falling, > 0).
// What it knows of the next state up stays, so a w that the state itself answers costs no access.
template <class S>
struct BulkPath {
    const S &out;
    uint32_t states, u, up, up_len, up_link;

    SAM_HD BulkPath(const S &o, uint32_t n, uint32_t from) : out(o), states(n), u(from), up(0), up_len(0), up_link(0)
    {
        uint32_t len;
        if (u >= states) return;
        out.len_link(u, len, up);
        if (up < states) out.len_link(up, up_len, up_link);
    }
    // false: a link that leads nowhere, or more of them than there are states
    SAM_HD bool climb(uint32_t w)
    {
        if (u >= states || up >= states) return false;
        for (uint32_t left = states; up_len >= w; left--) {
            if (!left || up_link >= states) return false;
            u = up;
            up = up_link;
            out.len_link(up, up_len, up_link);
        }
        return true;
    }
};

template <class S, class C, class I>
SAM_HD void bulk_settle(C &ctx, const BulkSeq<I> &q, const S &out, uint32_t states, uint32_t v)
{
    uint32_t len, link, endpos, itok;
    out.load(v, len, link, endpos, itok);
    if (v == 0 || len == endpos) return;
    BulkPath<S> path(out, states, out.idst(v));
    if (!path.climb(len + 1)) ctx.bit_or(&q.counts[kCntCorrupt], 1u);
    out.store_idst(v, path.u);
}

// The transitions of all occurrences but the first: a prefix brings the token behind it to every
// state on its suffix path, up to one that has it from an earlier comer, which goes on from there.
// A state whose first occurrence this is has the token already, and only this prefix passes it.
struct BulkWalk {
    uint32_t i, v, u;        // the prefix ends at i; v: the next state; u: on the target's suffix path
    bool more;               // not at its end after kBulkWalk states
};

// Returns how many it made.
template <class S, class C, class I>
SAM_HD uint32_t bulk_walk(C &ctx, const BulkSeq<I> &q, const S &out, uint32_t states, uint32_t prefix, BulkWalk &w)
{
    uint32_t len, link, endpos, itok;
    w.more = false;
    out.load(prefix, len, link, endpos, itok);
    if (prefix == 0 || len != endpos || len >= q.n) return 0;
    const uint32_t i = len - 1, t = (uint32_t)q.tok[len];
    uint32_t v = link, made = 0;
    if (v >= states) { ctx.bit_or(&q.counts[kCntCorrupt], 1u); return 0; }
    BulkPath<S> path(out, states, out.idst(prefix));
    out.load(v, len, link, endpos, itok);
    for (uint32_t step = 1;; step++) {
        // the next state's record travels while this one's slot is looked at
        uint32_t len2 = 0, link2 = 0, endpos2 = 0, itok2 = 0, at = 0;
        if (v && link < states) out.load(link, len2, link2, endpos2, itok2);
        if (itok == t) {
            if (endpos != i + 1) break;
        } else {
            const int got = out.claim(ctx, v, t, at);
            if (got == 1) break;
            if (got == 2 || !path.climb(len + 1)) { ctx.bit_or(&q.counts[kCntCorrupt], 1u); break; }
            out.enter(ctx, at, v, t, endpos, path.u);
            made++;
        }
        if (v == 0) break;
        v = link;
        if (v >= states) { ctx.bit_or(&q.counts[kCntCorrupt], 1u); break; }
        if (step == kBulkWalk) {
            w.i = i;
            w.v = v;
            w.u = path.u;
            w.more = true;
            break;
        }
        len = len2; link = link2; endpos = endpos2; itok = itok2;
    }
    return made;
}

// A longer walk goes on by the whole wave: 64 states at a time are listed by their links and then
// tried together (the end of a long run of one token brings a new one to as many states as the run is
// long).  In a run or a short period the links go down by the same
// number of states again and again, so the list is guessed from the last link and holds as far as
// the links say so: 64 states a round trip there, at least one elsewhere.  list: 64 words of the wave's
// own.
template <class S, class C, class I>
SAM_HD void bulk_long_walk(C &ctx, const BulkSeq<I> &q, const S &out, uint32_t states, const BulkWalk &w, uint32_t *list)
{
    const uint32_t i = w.i, t = (uint32_t)q.tok[i + 1];
    uint32_t v = w.v, u = w.u, down = 1;
    auto corrupt = [&] { ctx.bit_or(&q.counts[kCntCorrupt], 1u); };
    for (uint32_t left = states;; left--) {
        if (!left || v >= states) { corrupt(); break; }
        // how many of v, v - down, v - 2 down ... follow each other by their links, up to the first
        // that has the token from an earlier comer or is the root
        uint32_t more, next;
        const uint32_t count = ctx.chain(v, down, [&](uint32_t s, uint32_t &link, uint32_t &kind) {
            uint32_t len, endpos, itok;
            out.load(s, len, link, endpos, itok);
            // 0 to be tried, 1 has it from this prefix, 2 from an earlier comer: the end
            kind = itok != t ? 0u : (endpos == i + 1 ? 1u : 2u);
        }, list, more, next);
        // list[0 .. count): the states, kNil for those not to be tried
        ctx.wave_sync();
        const bool last_tried = count && list[count - 1] != kNil;
        ctx.wave_sync();
        ctx.lanes([&](uint32_t lane) {
            if (lane >= count || list[lane] == kNil) return;
            const uint32_t s = list[lane];
            uint32_t len, link, endpos, itok, at = 0, to = kNil;
            const int got = out.claim(ctx, s, t, at);
            if (got == 2) corrupt();
            if (got == 0) {
                out.load(s, len, link, endpos, itok);
                BulkPath<S> path(out, states, u);
                if (!path.climb(len + 1)) corrupt();
                to = path.u;
                out.enter(ctx, at, s, t, endpos, to);
                ctx.add(&q.counts[kCntMade], 1u);
            }
            list[lane] = to;
        });
        ctx.wave_sync();
        if (!more) break;
        if (last_tried) {
            u = list[count - 1];
            if (u == kNil || u >= states) break;
        }
        const uint32_t at = v - (count - 1) * down;      // the last one listed
        down = at > next ? at - next : 1;
        v = next;
        ctx.wave_sync();
    }
}

}  // namespace sam
