// Launchers of the builds over the whole chip (sam_bulk.hip).
#pragma once
#include "sam_bulk.h"
#include "sam_device.h"

namespace sam {

// Fresh sequences (launch_reset before) take those of their prompts that have more than lds_tokens
// tokens and fit their tables (bulk_takes); `most`: what a prompt may have by then.  n_listed: how many
// these are, where the host knows for sure, or 0: the launches cover all prompts.  begin: only looks
// for tokens outside the vocabulary, and makes the list; meta->n is how many there are in front of the
// first, from then on.
hipError_t launch_bulk_prompts(const BatchView &B, const int32_t *seq_map, int n_seqs, int n_listed, const int32_t *tokens,
                               const int64_t *offsets, uint32_t lds_tokens, uint32_t most, bool begin, hipStream_t stream);

__host__ __device__ __forceinline__ bool bulk_takes(const BatchView &B, int64_t count, uint32_t lds_tokens, uint32_t most)
{
    if (count <= (int64_t)lds_tokens || count > (int64_t)most || count > (int64_t)B.max_seq_len) return false;
    const size_t rec = (size_t)B.max_states * (B.compact ? sizeof(DynRecCompact) : sizeof(DynRec)),
                 slots = (size_t)B.dyn_buckets * 128;
    return B.compact ? bulk_tables_fit<uint16_t>((uint32_t)count, B.max_seq_len, rec, slots)
                     : bulk_tables_fit<uint32_t>((uint32_t)count, B.max_seq_len, rec, slots);
}

// Working memory of a corpus build, in device memory of the caller's.
struct BulkWork {
    char *first, *second, *third;      // bulk_first_bytes, bulk_second_bytes<uint32_t>, bulk_third_bytes
    uint32_t *counts;                  // kBulkCounts words
    BulkCorpus::State *rec;            // [2n + 1]
};
// The states and transitions of the corpus; reads the counts back (synchronises).  gave_up: it has groups
// that are too large to sort here.
hipError_t bulk_corpus(const int32_t *tok, uint32_t n, uint32_t vocab, RootEnt *root, const BulkWork &w,
                       uint32_t *n_states, uint64_t *n_trans, bool *gave_up, hipStream_t stream);
// All transitions but the root's into the table of n_buckets (all bytes 0xFF before), in an order that
// the keys alone decide; end positions into it and into root; link pairs; the states as the host
// keeps them (their last word all ones).
hipError_t bulk_corpus_tables(const int32_t *tok, uint32_t n, uint32_t vocab, uint32_t n_states, RootEnt *root,
                              const BulkWork &w, Slot *slots, uint64_t n_buckets, LinkPair *pairs, hipStream_t stream);
// Position of the first token outside [0, vocab), n if there is none (*at: device, set to n before).
hipError_t bulk_check(const int32_t *tok, uint32_t n, uint32_t vocab, uint32_t *at, hipStream_t stream);

}  // namespace sam
