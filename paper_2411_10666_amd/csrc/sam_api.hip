// C ABI of the library (see include/sam.h): argument checks, device memory and
// kernel launches.  All arithmetic of the method runs in the kernels
// (sam_kernels.hip) and, for the corpus automaton, in the host builder
// (sam_host.cpp).
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include <atomic>
#include <mutex>
#include <new>
#include <string>
#include <thread>
#include <vector>

#include "../../include/sam.h"
#include "sam_bulk_launch.h"
#include "sam_device.h"
#include "sam_host.h"
#include "sam_membench.h"
#include "sam_prompt.h"

using namespace sam;

namespace {

thread_local std::string g_err;
int g_layout_override = 0;   // bit 0: always the wide layout, bit 1: tight slot tables,
                             // bit 2: C++ token loops, bit 3: corpus table beyond 4 GiB,
                             // bit 4: scout waves whatever the batch size, bit 5: never,
                             // bit 6: corpora on the device whatever their size,
                             // bit 7: no builds by the whole chip, bits 8 to 10: see build_malloc
// Scout waves look at a step's row ahead of the walks.  They pay where there is something to look at and
// the walks would wait for it: the more, the longer the rows (the walks of a row are a chain, the
// scouts' look-ups are not) and the longer the sequences (a short one's tables are in the caches from
// the step before).  Measured, time with scouts over time without, rows of up to 4 / 8 / 16, small corpora:
//   64 x 1000 tokens      1.04 1.01      1 x 3000        1.05 1.01     1 x 13 000        0.99 0.94
//   64 x 3000        1.04 1.01 0.98      8 x 5000        1.00 0.96     8 x 13 000        0.96 0.91
//   64 x 4000        1.03 0.99 0.97     32 x 9000   1.00 0.95 0.92   128 x 2500     1.03 1.00 0.98
//   64 x 9000        0.99 0.95 0.92     32 x 13 500 0.98 0.94 0.91   128 x 5000     1.02 0.99 0.96
//   1024 x 1000      1.04 1.01 0.98    256 x 10 000 0.97            1024 x 8000     0.97 (1024 x 7500, 6: 0.94)
//   of up to 2: 1.0 to 1.13; of 3: 256 x 10 000 0.99, 12 x 41 000 1.00, 1 x 41 000 1.02; of 12: 1 x 5500 1.01, 8 x 4000
//   0.98; of 24: 64 x 480 0.98, 8 x 1000 0.98; of 64: 1 x 500 1.00, 256 x 300 0.99
// so the line is drawn at the tokens of a sequence times the square of a row's (8: 3900, 16: 980), three
// times as high where all tables together stay in the caches, and dropped beyond the L2 (32 MB) for all but
// short sequences.  A corpus makes no difference while the last-level cache (256 MB) holds it; walks over a larger one miss in it,
// and with 128 sequences and more scouts pay for short ones too (over 7 GB, rows of up to 8 / 16: 128 x 1600 0.97
// 0.95, 256 x 800 0.97 0.94, 1024 x 210 1.00 0.96; 128 x 800 1.02 1.01, 64 x 1000 1.05 1.03).
// They stop paying once the walking waves
// alone fill the chip: with more than six sequences per compute unit the scouts take wave slots and
// issue cycles from other sequences' walks (1024 sequences on 256 units over 6 GB of
// tables -9 % per step with scouts, 1536 -6 %, 2048 +9 %, 4096 +19 %, 8192 +27 %).
constexpr int     kScoutMaxSeqPerCu = 6;
bool scouts_pay(int64_t seq_len, int64_t accept, int64_t batch, int64_t table_bytes, int64_t corpus_bytes)
{
    if (accept < 4) return false;
    const int64_t reach = seq_len * accept * accept, mb = 1 << 20;
    return (reach >= 250000 && table_bytes >= 4 * mb) || reach >= 850000 ||
           (table_bytes >= 40 * mb && seq_len >= 2500) ||
           (corpus_bytes > 256 * mb && batch >= 128 && accept >= 8 && table_bytes >= 10 * mb);
}
// buckets of 128 bytes that make a transition table of 4.5 GiB
constexpr uint64_t kHugeTableBuckets = (1ull << 25) + (1ull << 22);
// Does the device build this corpus?  From 10 000 tokens on: about fifty launches and a few allocations
// take what the host needs for those (sam_build, device / host, ms, Zipf text: 5000 tokens 0.62 / 0.38,
// 10 000 0.68 / 0.65, 20 000 0.79 / 1.24, 100 000 1.6 / 6.2, 700 000 6.3 / 102, 6 M 23 / 1304; a large corpus'
// copy to the host goes by the machine: 4.3 to 8.2 for 700 000).
// Text that repeats is what the host is fast at (it stays in its caches) and the device slow: more rounds of the
// sort, large groups that one workgroup takes each, and behind a run or a short period one wave that brings the next
// token to as many states as the run is long.  So 16 places are looked at, whether what follows them is what was
// there d tokens before:
// - Where a share of them repeats, at a distance of up to 1024, the line is at 10 000 + 45 000 times that share
//   (a period of 150: 20 000 tokens 1.01 / 0.74, 60 000 1.62 / 1.91; runs in a quarter of the text: 15 000 0.93 / 0.88,
//   25 000 1.23 / 1.39; in half of it: 30 000 1.80 / 1.56, 40 000 1.98 / 2.13).
// - Where one stretch over its period is more than a quarter of the text, at 250 000 (a run of half the text and then
//   other text: 100 000 7.2 / 5.0, 200 000 15 / 10, 300 000 23 / 25; a period of 2: 100 000 5.3 / 3.6, 250 000 14.6 / 15.4; of
//   5: 100 000 2.9 / 3.4).
// - Where it is more than 0.6 of it and ends before the text does, at 600 000 (a run and another token: 300 000 31 / 20,
//   500 000 54 / 43, 1 M 101 / 104; of three quarters: 300 000 28 / 19, 500 000 45 / 44; to the end of the text: 300 000
//   11 / 15).
bool device_builds(const int32_t *x, int64_t n)
{
    if (g_layout_override & 128) return false;
    if (g_layout_override & 64) return true;
    if (n < 10000) return false;
    if (n >= 600000) return true;
    constexpr int kLooks = 16, kSame = 16;
    const int64_t most = n < 64000 ? 1024 : 4;       // (longer periods only move the first line)
    int repeats = 0, run = 0;
    int64_t before = 0, reach = 0;
    bool inner = false;
    for (int k = 1; k <= kLooks; k++) {
        const int32_t *const at = x + (n - kSame) * k / kLooks;     // the last one is the text's end
        int64_t d = 1;
        while (d <= most && d <= at - x && !(at[-d] == at[0] && memcmp(at - d, at, kSame * sizeof(int32_t)) == 0)) d++;
        if (d > most || d > at - x) d = 0;
        run = d && d == before ? run + 1 : 1;
        before = d;
        if (!d) continue;
        repeats++;
        if (run * n / kLooks / d > reach) {
            reach = run * n / kLooks / d;
            inner = k < kLooks;
        }
    }
    if (n < 10000 + 45000 * repeats / kLooks) return false;
    if (reach > n / 4 && n < 250000) return false;
    return !(10 * reach > 6 * n && inner);
}
HostSam::ProgressFn g_progress = nullptr;
void *g_progress_user = nullptr;

int fail(int code, const std::string &msg)
{
    g_err = msg;
    return code;
}

int fail_hip(const char *what, hipError_t e)
{
    g_err = std::string(what) + ": " + hipGetErrorString(e);
    return e == hipErrorOutOfMemory ? SAM_ENOMEM : SAM_EDEVICE;
}

#define HIP_TRY(expr)                                      \
    do {                                                   \
        hipError_t e_ = (expr);                            \
        if (e_ != hipSuccess) return fail_hip(#expr, e_);  \
    } while (0)

}  // namespace

// Table space of the batch made by sam_batch_init_noalloc: device memory that is
// part of the loaded code object, so no call ever has to allocate it.  Every GPU
// the library runs on holds its own copy at its own address for the life of the
// process.  In host code the name below is only a handle for hipGetSymbolAddress;
// the address kernels and fills receive is the one that call returns.
constexpr size_t kNoAllocBytes = (size_t)SAM_NOALLOC_MAX_BYTES;
static __device__ __align__(256) unsigned char g_noalloc_scratch[kNoAllocBytes];

struct sam_corpus {
    HostSam    host;
    bool       on_device = false;
    int        device = -1;
    StaticView view = {};
    void      *d_text = nullptr, *d_linkrec = nullptr, *d_root = nullptr, *d_slots = nullptr;
    void      *d_topk = nullptr;
    int64_t    device_bytes = 0;
};

struct sam_batch {
    const sam_corpus *corpus = nullptr;
    BatchView         view = {};
    int64_t           device_bytes = 0;
    int               noalloc_device = -1;   // >= 0: lives in that device's fixed buffer
};

namespace {

// one fixed-buffer batch per device: its handle, the buffer's device address
// (looked up once per device) and whether the handle is handed out
constexpr int kMaxDevices = 64;
struct NoAllocSlot {
    sam_batch      handle;
    unsigned char *base = nullptr;
    bool           busy = false;
};
NoAllocSlot g_noalloc[kMaxDevices];
std::mutex  g_noalloc_mu;

}  // namespace

// Address of the current device's copy of the fixed buffer, looked up once per
// device with that device current (the first lookup makes the runtime load this
// file's device code on that GPU, which is when the buffer comes to exist there).
// Call with g_noalloc_mu held.
static hipError_t noalloc_base_locked(int dev, unsigned char **base)
{
    NoAllocSlot &slot = g_noalloc[dev];
    if (!slot.base) {
        void *p = nullptr;
        hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(g_noalloc_scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        slot.base = (unsigned char *)p;
    }
    *base = slot.base;
    return hipSuccess;
}

extern "C" {

const char *sam_last_error(void) { return g_err.c_str(); }

#ifndef SAM_BUILD_ID
#define SAM_BUILD_ID "unknown"
#endif
const char *sam_build_id(void) { return SAM_BUILD_ID; }

static void corpus_release_device(sam_corpus *c)
{
    if (c->d_text) (void)hipFree(c->d_text);
    if (c->d_linkrec) (void)hipFree(c->d_linkrec);
    if (c->d_root) (void)hipFree(c->d_root);
    if (c->d_slots) (void)hipFree(c->d_slots);
    if (c->d_topk) (void)hipFree(c->d_topk);
    c->d_text = c->d_linkrec = c->d_root = c->d_slots = c->d_topk = nullptr;
}

// Device memory that corpus_finish works in, the caller's: the link pairs, a bit for every state
// and a count.  done: an allocation that is not read once the records are made (the pairs lie in it).
struct FinishScratch {
    const LinkPair     *pairs;
    uint32_t           *wide;
    unsigned long long *count;
    void              **done;
};
static size_t wide_bytes(uint32_t n_states) { return ((size_t)n_states + 31) / 32 * sizeof(uint32_t); }

// Device memory of sam_build.  Testing: the request that bits 8 to 10 of the layout override name finds none.
enum BuildMemory { kNoRequest, kText, kRoot, kWork, kMarks, kSlots, kRecords, kTable };
static bool build_malloc(BuildMemory which, void **p, size_t bytes)
{
    *p = nullptr;
    if (which == ((g_layout_override >> 8) & 7)) return false;
    if (hipMalloc(p, bytes) == hipSuccess) return true;
    (void)hipGetLastError();
    *p = nullptr;
    return false;
}

// What is on the device already: text, the root's transitions, the table of all others, the link
// pairs and room for the state records, which are made from them, as is the walks' table.
static int corpus_finish(sam_corpus *c, const FinishScratch &w)
{
    const HostSam &h = c->host;
    const size_t b_text = (size_t)h.n_tokens * sizeof(int32_t);
    const size_t b_lr = (size_t)h.n_states * sizeof(LinkRec);
    const size_t b_root = (size_t)h.vocab * sizeof(RootEnt);
    // link pairs -> 32-byte state records with two transitions inline
    hipError_t e = hipMemset(w.wide, 0, wide_bytes(h.n_states));
    if (e == hipSuccess)
        e = launch_staterec(w.pairs, (Slot *)c->d_slots, (RootEnt *)c->d_root, (LinkRec *)c->d_linkrec,
                            w.wide, h.n_states, h.n_buckets * kBucketSlots, (uint32_t)h.vocab, nullptr);
    // The walks only ever look up transitions of wide states (a narrow state's record
    // holds all of its own): the table they probe is rebuilt with those alone, at load
    // 0.5, and the full one freed.  (Not in the testing mode that wants a table beyond
    // 4 GiB.)
    uint64_t n_buckets = h.n_buckets;
    if (e == hipSuccess && (g_layout_override & 8) == 0) {
        unsigned long long n_wide = 0;
        void *d_new = nullptr;
        e = hipMemset(w.count, 0, sizeof(*w.count));
        if (e == hipSuccess)
            e = launch_count_wide((const Slot *)c->d_slots, w.wide, h.n_buckets * kBucketSlots, w.count, nullptr);
        if (e == hipSuccess) e = hipMemcpy(&n_wide, w.count, sizeof(n_wide), hipMemcpyDeviceToHost);
        const uint64_t nb_new = (2 * (uint64_t)n_wide + 64 + kBucketSlots - 1) / kBucketSlots;
        if (e == hipSuccess && nb_new < h.n_buckets) {
            const size_t b_new = (size_t)nb_new * kBucketSlots * sizeof(Slot);
            if (!build_malloc(kTable, &d_new, b_new)) {
                // no room for a second table beside all the rest: what is not read any more makes room (the
                // count was waited for, so the records are made)
                (void)hipFree(*w.done);
                *w.done = nullptr;
                if (hipMalloc(&d_new, b_new) != hipSuccess) {
                    // still none: the full one serves
                    (void)hipGetLastError();
                    d_new = nullptr;
                }
            }
            if (d_new) {
                e = launch_fill_empty(d_new, b_new, nullptr);
                if (e == hipSuccess)
                    e = launch_compact_slots((const Slot *)c->d_slots, w.wide,
                                             h.n_buckets * kBucketSlots, (Slot *)d_new, nb_new,
                                             nullptr);
                if (e == hipSuccess) e = hipDeviceSynchronize();
                if (e == hipSuccess) {
                    (void)hipFree(c->d_slots);
                    c->d_slots = d_new;
                    n_buckets = nb_new;
                } else {
                    (void)hipFree(d_new);
                }
            }
        }
    }
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (e != hipSuccess) return fail_hip("sam_build: state records", e);
    c->view.n_buckets = n_buckets;
    c->view.text = (const int32_t *)c->d_text;
    c->view.linkrec = (const LinkRec *)c->d_linkrec;
    c->view.root = (const RootEnt *)c->d_root;
    c->view.slots = (const Slot *)c->d_slots;
    c->view.n_tokens = (uint32_t)h.n_tokens;
    c->view.n_states = h.n_states;
    c->device_bytes = (int64_t)(b_text + b_lr + b_root + (size_t)n_buckets * kBucketSlots * sizeof(Slot));
    c->on_device = true;
    if (c->device >= 0 && c->device < kMaxDevices) {
        // a set-up call: do the one-time lookup of the fixed buffer here, so that a later
        // sam_batch_init_noalloc on this device has nothing left to load
        std::lock_guard<std::mutex> lock(g_noalloc_mu);
        unsigned char *unused = nullptr;
        (void)noalloc_base_locked(c->device, &unused);
    }
    return SAM_OK;
}

static int corpus_upload(sam_corpus *c)
{
    const HostSam &h = c->host;
    std::vector<LinkPair> lr;
    try {
        h.make_linkrec(lr);
    } catch (const std::bad_alloc &) {
        return fail(SAM_ENOMEM, "sam_build: out of host memory for the link records");
    }
    const size_t b_text = (size_t)h.n_tokens * sizeof(int32_t);
    const size_t b_root = (size_t)h.vocab * sizeof(RootEnt);
    const size_t b_slots = (size_t)h.n_buckets * kBucketSlots * sizeof(Slot);
    const size_t b_pairs = (size_t)h.n_states * sizeof(LinkPair);
    HIP_TRY(hipGetDevice(&c->device));
    HIP_TRY(hipMalloc(&c->d_text, b_text));
    HIP_TRY(hipMalloc(&c->d_root, b_root));
    HIP_TRY(hipMalloc(&c->d_slots, b_slots));
    HIP_TRY(hipMalloc(&c->d_linkrec, (size_t)h.n_states * sizeof(LinkRec)));
    HIP_TRY(hipMemcpy(c->d_text, h.text.data(), b_text, hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(c->d_root, h.root.data(), b_root, hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(c->d_slots, h.slots, b_slots, hipMemcpyHostToDevice));
    const size_t b_wide = bulk_up(wide_bytes(h.n_states));
    void *pairs = nullptr, *marks = nullptr;
    hipError_t e = hipMalloc(&pairs, b_pairs);
    if (e == hipSuccess) e = hipMalloc(&marks, b_wide + sizeof(unsigned long long));
    if (e == hipSuccess) e = hipMemcpy(pairs, lr.data(), b_pairs, hipMemcpyHostToDevice);
    const int rc = e != hipSuccess ? fail_hip("sam_build: state records", e)
                                   : corpus_finish(c, {(const LinkPair *)pairs, (uint32_t *)marks,
                                                       (unsigned long long *)((char *)marks + b_wide), &pairs});
    if (pairs) (void)hipFree(pairs);
    if (marks) (void)hipFree(marks);
    return rc;
}

// A copy to host memory that is not pinned goes through the runtime's staging buffers at the rate of one
// thread's memcpy (17 GB/s).  Here the device fills one half of a pinned buffer while several threads
// empty the other: 48 MB in about 1.1 ms instead of 2.8.  (Threads with a stream and a part of the copy each:
// 2.7 ms, most of it the first stream's creation.)
static hipError_t copy_down(void *dst, const void *src, size_t bytes)
{
    constexpr size_t kHalf = 8u << 20;
    constexpr int kThreads = 6;
    char *stage = nullptr;
    if (bytes < kHalf || hipHostMalloc((void **)&stage, 2 * kHalf, hipHostMallocDefault) != hipSuccess) {
        (void)hipGetLastError();
        return hipMemcpy(dst, src, bytes, hipMemcpyDeviceToHost);
    }
    const size_t chunks = (bytes + kHalf - 1) / kHalf;
    auto size_of = [&](size_t k) { return k + 1 < chunks ? kHalf : bytes - k * kHalf; };
    std::atomic<size_t> ready(0);                        // chunks that have come
    std::atomic<size_t> emptied[kThreads];               // chunks that each thread has copied its slice of
    for (auto &done : emptied) done.store(0);
    std::atomic<bool> stop(false);
    int workers = 0;
    auto work = [&](int t) {
        for (size_t k = 0; k < chunks; k++) {
            while (ready.load(std::memory_order_acquire) <= k) {
                if (stop.load()) return;
                std::this_thread::yield();
            }
            const size_t part = (kHalf / kThreads + 4095) / 4096 * 4096, lo = t * part;
            const size_t hi = t + 1 < kThreads && lo + part < size_of(k) ? lo + part : size_of(k);
            if (lo < hi) memcpy((char *)dst + k * kHalf + lo, stage + (k & 1) * kHalf + lo, hi - lo);
            emptied[t].store(k + 1, std::memory_order_release);
        }
    };
    std::thread pool[kThreads];
    try {
        for (; workers < kThreads; workers++) pool[workers] = std::thread(work, workers);
    } catch (...) {
    }
    hipError_t e = workers == kThreads ? hipSuccess : hipErrorOutOfMemory;
    auto fill = [&](size_t k) {
        return hipMemcpyAsync(stage + (k & 1) * kHalf, (const char *)src + k * kHalf, size_of(k), hipMemcpyDeviceToHost, nullptr);
    };
    if (e == hipSuccess) e = fill(0);
    for (size_t k = 0; k < chunks && e == hipSuccess; k++) {
        if ((e = hipStreamSynchronize(nullptr)) != hipSuccess) break;
        ready.store(k + 1, std::memory_order_release);
        // the other half is free once every thread has its slice of the chunk before this one
        for (auto &done : emptied)
            while (done.load(std::memory_order_acquire) < k) std::this_thread::yield();
        if (k + 1 < chunks) e = fill(k + 1);
    }
    if (e != hipSuccess) stop.store(true);
    for (int t = 0; t < workers; t++) pool[t].join();
    (void)hipHostFree(stage);
    // no threads to be had: the plain way
    return workers == kThreads ? e : hipMemcpy(dst, src, bytes, hipMemcpyDeviceToHost);
}

// Build-SAM on the device: the host receives what its own builder would have made, but for the order
// of the keys in the transition table.  *done false: no room for it, or nothing for it; the host
// builds.
static int corpus_build_device(sam_corpus *c, const int32_t *tokens, int64_t n, int32_t vocab, bool *done)
{
    *done = false;
    const uint64_t n_buckets = static_buckets_for(n), n_slots = n_buckets * kBucketSlots;
    if (n_slots >= 0xFFFFFFFFull) return SAM_OK;
    bool room = false;             // the thread below writes it: it outlives scratch, which waits for the thread
    struct Scratch {
        void *work = nullptr, *marks = nullptr;
        std::thread host;
        ~Scratch()
        {
            if (host.joinable()) host.join();
            if (work) (void)hipFree(work);
            if (marks) (void)hipFree(marks);
        }
    } scratch;
    // every failure to allocate on the device ends here: what was allocated is freed, the host builds
    auto none = [&] {
        if (scratch.host.joinable()) scratch.host.join();
        corpus_release_device(c);
        c->host.~HostSam();
        new (&c->host) HostSam();
        return SAM_OK;
    };
    HIP_TRY(hipGetDevice(&c->device));
    hipError_t e;
    const uint32_t un = (uint32_t)n;
    BulkWork w;
    if (!build_malloc(kText, &c->d_text, (size_t)n * sizeof(int32_t)) ||
        !build_malloc(kRoot, &c->d_root, (size_t)vocab * sizeof(RootEnt)))
        return none();
    const size_t b1 = bulk_first_bytes(un), b2 = bulk_up(bulk_second_bytes<uint32_t>(un)), b3 = bulk_up(bulk_third_bytes(un)),
                 br = (2 * (size_t)n + 1) * sizeof(BulkCorpus::State);
    if (!build_malloc(kWork, &scratch.work, bulk_up(b1) + b2 + br) ||
        !build_malloc(kMarks, &scratch.marks, b3 + 4 * kBulkCounts))
        return none();
    w.first = (char *)scratch.work;
    w.second = w.first + bulk_up(b1);
    w.rec = (BulkCorpus::State *)(w.second + b2);
    w.third = (char *)scratch.marks;
    w.counts = (uint32_t *)(w.third + b3);
    // the host's memory is made ready while the device works
    try {
        scratch.host = std::thread([&] { room = c->host.reserve_for_copy(tokens, n, vocab, n_buckets); });
    } catch (...) {
        room = c->host.reserve_for_copy(tokens, n, vocab, n_buckets);
    }
    uint32_t at = un;
    HIP_TRY(hipMemcpy(c->d_text, tokens, (size_t)n * sizeof(int32_t), hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(w.counts, &at, sizeof(at), hipMemcpyHostToDevice));
    HIP_TRY(bulk_check((const int32_t *)c->d_text, un, (uint32_t)vocab, w.counts, nullptr));
    HIP_TRY(hipMemcpy(&at, w.counts, sizeof(at), hipMemcpyDeviceToHost));
    if (at < un)
        return fail(SAM_ETOKEN, "sam_build: corpus token " + std::to_string(tokens[at]) + " at position " +
                                    std::to_string(at) + " is outside [0, vocab)");
    HIP_TRY(hipMemset(c->d_root, 0, (size_t)vocab * sizeof(RootEnt)));
    uint32_t n_states = 0;
    uint64_t n_trans = 0;
    bool gave_up = false;
    HIP_TRY(bulk_corpus((const int32_t *)c->d_text, un, (uint32_t)vocab, (RootEnt *)c->d_root, w, &n_states, &n_trans,
                        &gave_up, nullptr));
    if (gave_up) return none();
    if (g_progress) g_progress("finalize", 0, (int64_t)n_slots, g_progress_user);
    // (the last two requests that the build cannot do without, and the most memory that it holds: about
    // 207 bytes a token, where the host's build needs 130)
    if (!build_malloc(kSlots, &c->d_slots, n_slots * sizeof(Slot)) ||
        !build_malloc(kRecords, &c->d_linkrec, (size_t)n_states * sizeof(LinkRec)))
        return none();
    // the second region (24 bytes a token) and the third (a quarter) are free again
    LinkPair *const d_pairs = (LinkPair *)w.second;
    const FinishScratch finish = {d_pairs, (uint32_t *)w.third, (unsigned long long *)w.counts, &scratch.work};
    e = launch_fill_empty(c->d_slots, n_slots * sizeof(Slot), nullptr);
    if (e == hipSuccess)
        e = bulk_corpus_tables((const int32_t *)c->d_text, un, (uint32_t)vocab, n_states, (RootEnt *)c->d_root, w,
                               (Slot *)c->d_slots, n_buckets, d_pairs, nullptr);
    if (scratch.host.joinable()) scratch.host.join();
    if (e == hipSuccess && !room) {
        return fail(SAM_ENOMEM, "sam_build: out of host memory for the automaton");
    }
    static_assert(sizeof(HostState) == sizeof(BulkCorpus::State), "states are copied as they are");
    if (g_progress) g_progress("upload", 0, 1, g_progress_user);       // the other way round, here
    HostSam &h = c->host;
    h.n_states = n_states;
    h.n_trans = n_trans;
    h.st.set_size(n_states);
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (e == hipSuccess) e = copy_down(h.slots, c->d_slots, n_slots * sizeof(Slot));
    if (e == hipSuccess) e = copy_down(&h.st[0], w.rec, (size_t)n_states * sizeof(HostState));
    if (e == hipSuccess) e = hipMemcpy(h.root.data(), c->d_root, (size_t)vocab * sizeof(RootEnt), hipMemcpyDeviceToHost);
    if (e != hipSuccess) return fail_hip("sam_build: tables", e);
    const int rc = corpus_finish(c, finish);
    *done = rc == SAM_OK;
    return rc;
}

static int build_common(const int32_t *tokens, int64_t n, int32_t vocab, bool upload,
                        sam_corpus **out)
{
    if (!out) return fail(SAM_EINVAL, "sam_build: out is NULL");
    *out = nullptr;
    sam_corpus *c = new (std::nothrow) sam_corpus;
    if (!c) return fail(SAM_ENOMEM, "sam_build: out of host memory");
    if (upload && tokens && n >= 1 && n <= 0x7FFFFFFELL && vocab >= 1 && (g_layout_override & 8) == 0 &&
        device_builds(tokens, n)) {
        bool done = false;
        if (g_progress) g_progress("build", 0, n, g_progress_user);
        const int rc = corpus_build_device(c, tokens, n, vocab, &done);
        if (rc != SAM_OK || done) {
            if (rc != SAM_OK) {
                corpus_release_device(c);
                delete c;
                return rc;
            }
            *out = c;
            return SAM_OK;
        }
    }
    std::string err;
    int rc;
    try {
        rc = c->host.build(tokens, n, vocab, err, g_progress, g_progress_user,
                           (g_layout_override & 8) ? kHugeTableBuckets : 0);
    } catch (const std::bad_alloc &) {
        rc = SAM_ENOMEM;
        err = "sam_build: out of host memory";
    }
    if (rc != SAM_OK) {
        delete c;
        return fail(rc, err);
    }
    if (upload) {
        if (g_progress) g_progress("upload", 0, 1, g_progress_user);
        rc = corpus_upload(c);
        if (rc != SAM_OK) {
            corpus_release_device(c);
            delete c;
            return rc;
        }
    }
    *out = c;
    return SAM_OK;
}

int sam_build(const int32_t *corpus_tokens, int64_t n_tokens, int32_t vocab, sam_corpus **out)
{
    return build_common(corpus_tokens, n_tokens, vocab, true, out);
}

int sam_build_host_only(const int32_t *corpus_tokens, int64_t n_tokens, int32_t vocab,
                        sam_corpus **out)
{
    return build_common(corpus_tokens, n_tokens, vocab, false, out);
}

int sam_corpus_save(const sam_corpus *c, const char *path)
{
    if (!c || !path) return fail(SAM_EINVAL, "sam_corpus_save: NULL argument");
    std::string err;
    const int rc = c->host.save(path, err);
    return rc == SAM_OK ? SAM_OK : fail(rc, err);
}

static int load_common(const char *path, bool upload, sam_corpus **out)
{
    if (!out || !path) return fail(SAM_EINVAL, "sam_corpus_load: NULL argument");
    *out = nullptr;
    sam_corpus *c = new (std::nothrow) sam_corpus;
    if (!c) return fail(SAM_ENOMEM, "sam_corpus_load: out of host memory");
    std::string err;
    int rc;
    try {
        rc = c->host.load(path, err);
    } catch (const std::bad_alloc &) {
        rc = SAM_ENOMEM;
        err = "sam_corpus_load: out of host memory";
    }
    if (rc != SAM_OK) {
        delete c;
        return fail(rc, err);
    }
    if (upload) {
        rc = corpus_upload(c);
        if (rc != SAM_OK) {
            corpus_release_device(c);
            delete c;
            return rc;
        }
    }
    *out = c;
    return SAM_OK;
}

int sam_corpus_load(const char *path, sam_corpus **out) { return load_common(path, true, out); }

int sam_corpus_load_host_only(const char *path, sam_corpus **out)
{
    return load_common(path, false, out);
}

int sam_corpus_info(const sam_corpus *c, int64_t *n_states, int64_t *n_trans,
                    int64_t *device_bytes)
{
    if (!c) return fail(SAM_EINVAL, "sam_corpus_info: corpus is NULL");
    if (n_states) *n_states = c->host.n_states;
    if (n_trans) *n_trans = (int64_t)c->host.n_trans;
    if (device_bytes) *device_bytes = c->device_bytes;
    return SAM_OK;
}

int sam_corpus_export(const sam_corpus *c, int32_t *length, int32_t *link, int32_t *min_endpos)
{
    if (!c) return fail(SAM_EINVAL, "sam_corpus_export: corpus is NULL");
    const HostSam &h = c->host;
    for (uint32_t s = 0; s < h.n_states; s++) {
        if (length) length[s] = (int32_t)h.len[s];
        if (link) link[s] = h.link[s] == kNil ? -1 : (int32_t)h.link[s];
        if (min_endpos) min_endpos[s] = (int32_t)h.endpos[s];
    }
    return SAM_OK;
}

int sam_corpus_find(const sam_corpus *c, int64_t state, int32_t token, int64_t *target)
{
    if (!c || !target) return fail(SAM_EINVAL, "sam_corpus_find: NULL argument");
    if (state < 0 || state >= (int64_t)c->host.n_states || token < 0 || token >= c->host.vocab)
        return fail(SAM_EINVAL, "sam_corpus_find: state or token out of range");
    const uint32_t d = c->host.find((uint32_t)state, (uint32_t)token);
    *target = d == kNil ? -1 : (int64_t)d;
    return SAM_OK;
}

int sam_corpus_build_topk(sam_corpus *c, int32_t k)
{
    if (!c) return fail(SAM_EINVAL, "sam_corpus_build_topk: corpus is NULL");
    std::string err;
    int rc;
    try {
        rc = c->host.build_topk(k, err, g_progress, g_progress_user);
    } catch (const std::bad_alloc &) {
        rc = SAM_ENOMEM;
        err = "sam_corpus_build_topk: out of host memory";
    }
    if (rc != SAM_OK) return fail(rc, err);
    if (c->on_device) {
        int dev = -1;
        HIP_TRY(hipGetDevice(&dev));
        if (dev != c->device)
            return fail(SAM_EINVAL, "sam_corpus_build_topk: the corpus lives on another device");
        const size_t bytes = c->host.topk.size() * sizeof(TopEnt);
        HIP_TRY(hipDeviceSynchronize());     // no launch may still read the old table
        if (c->d_topk) {
            c->device_bytes -= (int64_t)((size_t)c->host.n_states * c->view.top_k * sizeof(TopEnt));
            (void)hipFree(c->d_topk);
            c->d_topk = nullptr;
            c->view.topk = nullptr;
            c->view.top_k = 0;
        }
        HIP_TRY(hipMalloc(&c->d_topk, bytes));
        HIP_TRY(hipMemcpy(c->d_topk, c->host.topk.data(), bytes, hipMemcpyHostToDevice));
        c->view.topk = (const TopEnt *)c->d_topk;
        c->view.top_k = k;
        c->device_bytes += (int64_t)bytes;
    }
    return SAM_OK;
}

int sam_corpus_export_topk(const sam_corpus *c, uint64_t *freq, int32_t *token, int32_t *target,
                           float *prob)
{
    if (!c) return fail(SAM_EINVAL, "sam_corpus_export_topk: corpus is NULL");
    const HostSam &h = c->host;
    if (h.top_k < 1) return fail(SAM_EINVAL, "sam_corpus_export_topk: no top-k table was built");
    const size_t n = (size_t)h.n_states * h.top_k;
    if (freq)
        for (uint32_t s = 0; s < h.n_states; s++) freq[s] = h.freq[s];
    for (size_t i = 0; i < n; i++) {
        const TopEnt &e = h.topk[i];
        if (token) token[i] = e.dst ? (int32_t)e.token : -1;
        if (target) target[i] = e.dst ? (int32_t)e.dst : -1;
        if (prob) prob[i] = e.prob;
    }
    return SAM_OK;
}

void sam_corpus_free(sam_corpus *c)
{
    if (!c) return;
    corpus_release_device(c);
    delete c;
}

static void batch_release(sam_batch *b)
{
    if (b->noalloc_device >= 0) {
        // nothing to free: the tables are the device's fixed buffer
        std::lock_guard<std::mutex> lock(g_noalloc_mu);
        g_noalloc[b->noalloc_device].busy = false;
        return;
    }
    if (b->view.dyn_text) (void)hipFree(b->view.dyn_text);
    if (b->view.dyn_rec) (void)hipFree(b->view.dyn_rec);
    if (b->view.dyn_slots) (void)hipFree(b->view.dyn_slots);
    if (b->view.meta) (void)hipFree(b->view.meta);
    if (b->view.status) (void)hipFree(b->view.status);
    delete b;
}

// Argument checks shared by the two init calls; resolves the vocabulary.
static int batch_check_args(const char *fn, const sam_corpus *corpus, const int32_t *prompt_tokens,
                            const int64_t *prompt_offsets, int32_t batch, int32_t &vocab,
                            int32_t max_seq_len, int32_t max_accept, int32_t draft_len)
{
    const std::string f(fn);
    if (!prompt_tokens || !prompt_offsets)
        return fail(SAM_EINVAL, f + ": prompt_tokens / prompt_offsets is NULL");
    if (batch < 1) return fail(SAM_EINVAL, f + ": batch must be >= 1");
    if (max_seq_len < 1 || max_seq_len > (1 << 28))
        return fail(SAM_EINVAL, f + ": max_seq_len must be in 1 .. 2^28");
    if (max_accept < 1 || max_accept > 4096)
        return fail(SAM_EINVAL, f + ": max_accept must be in 1 .. 4096");
    if (draft_len < 1 || draft_len > 1024)
        return fail(SAM_EINVAL, f + ": draft_len must be in 1 .. 1024");
    if (corpus && !corpus->on_device)
        return fail(SAM_EINVAL, f + ": corpus was built host-only");
    if (corpus) {
        int dev = -1;
        HIP_TRY(hipGetDevice(&dev));
        if (dev != corpus->device)
            return fail(SAM_EINVAL, f + ": the corpus lives on device " +
                                        std::to_string(corpus->device) + ", the current device is " +
                                        std::to_string(dev));
        vocab = corpus->host.vocab;
    }
    if (vocab < 1) return fail(SAM_EINVAL, f + ": vocab must be >= 1");
    return SAM_OK;
}

static int batch_check_offsets(const char *fn, const int64_t *offs, int32_t batch,
                               int32_t max_seq_len)
{
    const std::string f(fn);
    if (offs[0] < 0) return fail(SAM_EINVAL, f + ": prompt_offsets[0] < 0");
    for (int32_t b = 0; b < batch; b++) {
        const int64_t len = offs[b + 1] - offs[b];
        if (len < 0) return fail(SAM_EINVAL, f + ": prompt_offsets must not decrease");
        if (len > max_seq_len)
            return fail(SAM_ECAPACITY, f + ": prompt " + std::to_string(b) + " has " +
                                           std::to_string(len) + " tokens, max_seq_len is " +
                                           std::to_string(max_seq_len));
    }
    return SAM_OK;
}

// Sizes of the per-sequence tables for these parameters.
struct BatchBytes { size_t text, rec, slots, meta; };

static BatchBytes batch_configure(BatchView &v, const sam_corpus *corpus, int32_t batch,
                                  int32_t vocab, int32_t max_seq_len, int32_t max_accept,
                                  int32_t draft_len, int32_t l_bias)
{
    const bool has_static = corpus != nullptr;
    v.batch = batch;
    v.vocab = vocab;
    v.max_seq_len = (uint32_t)max_seq_len;
    v.max_states = 2u * (uint32_t)max_seq_len + 2u;
    v.compact = ((g_layout_override & 1) == 0 && max_seq_len <= kCompactMaxSeqLen &&
                 vocab <= kCompactMaxVocab) ? 1 : 0;
    // a sequence never holds more than max_seq_len - 1 transitions in its slots
    const uint64_t dyn_slots = (g_layout_override & 2)
                                   ? ((uint64_t)max_seq_len + 16 + 15) / 16 * 16
                                   : dynamic_slots_for(max_seq_len);
    const size_t slot_bytes = v.compact ? sizeof(SlotCompact) : sizeof(Slot);
    const size_t rec_bytes = v.compact ? sizeof(DynRecCompact) : sizeof(DynRec);
    v.dyn_buckets = (uint32_t)(dyn_slots * slot_bytes / 128);
    v.max_accept = max_accept;
    v.draft_len = draft_len;
    v.l_bias = l_bias;
    v.l_threshold = -1;
    v.no_asm = (g_layout_override & 4) ? 1 : 0;
    v.no_bulk = (g_layout_override & 128) ? 1 : 0;
    int dev = 0, n_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        n_cu = 0;                          // unknown: no upper limit
    v.has_static = has_static ? 1 : 0;
    BatchBytes b;
    b.text = (size_t)batch * max_seq_len * sizeof(int32_t);
    b.rec = (size_t)batch * v.max_states * rec_bytes;
    b.slots = (size_t)batch * v.dyn_buckets * 128;
    b.meta = (size_t)batch * sizeof(SeqMeta);
    const bool scouts_fit = n_cu <= 0 || (int64_t)batch <= (int64_t)n_cu * kScoutMaxSeqPerCu;
    const bool pay = scouts_pay(max_seq_len, max_accept, batch, (int64_t)(b.text + b.rec + b.slots),
                                corpus ? corpus->device_bytes : 0);
    v.scout = ((g_layout_override & 32) == 0 && ((g_layout_override & 16) || (scouts_fit && pay))) ? 1 : 0;
    return b;
}

int sam_batch_init(const sam_corpus *corpus, const int32_t *prompt_tokens,
                   const int64_t *prompt_offsets, int32_t batch, int32_t vocab,
                   int32_t max_seq_len, int32_t max_accept, int32_t draft_len, int32_t l_bias,
                   void *hip_stream, sam_batch **out)
{
    if (!out) return fail(SAM_EINVAL, "sam_batch_init: out is NULL");
    *out = nullptr;
    int rc = batch_check_args("sam_batch_init", corpus, prompt_tokens, prompt_offsets, batch,
                              vocab, max_seq_len, max_accept, draft_len);
    if (rc != SAM_OK) return rc;
    hipStream_t stream = (hipStream_t)hip_stream;

    // the offsets decide how far each wave reads: check them before any launch
    std::vector<int64_t> offs;
    try {
        offs.resize((size_t)batch + 1);
    } catch (const std::bad_alloc &) {
        return fail(SAM_ENOMEM, "sam_batch_init: out of host memory");
    }
    HIP_TRY(hipMemcpyAsync(offs.data(), prompt_offsets, offs.size() * sizeof(int64_t),
                           hipMemcpyDeviceToHost, stream));
    HIP_TRY(hipStreamSynchronize(stream));
    rc = batch_check_offsets("sam_batch_init", offs.data(), batch, max_seq_len);
    if (rc != SAM_OK) return rc;

    sam_batch *bt = new (std::nothrow) sam_batch;
    if (!bt) return fail(SAM_ENOMEM, "sam_batch_init: out of host memory");
    bt->corpus = corpus;
    BatchView &v = bt->view;
    const BatchBytes bb = batch_configure(v, corpus, batch, vocab, max_seq_len, max_accept,
                                          draft_len, l_bias);
    hipError_t e;
    if ((e = hipMalloc((void **)&v.dyn_text, bb.text)) != hipSuccess ||
        (e = hipMalloc((void **)&v.dyn_rec, bb.rec)) != hipSuccess ||
        (e = hipMalloc((void **)&v.dyn_slots, bb.slots)) != hipSuccess ||
        (e = hipMalloc((void **)&v.meta, bb.meta)) != hipSuccess ||
        (e = hipMalloc((void **)&v.status, 256)) != hipSuccess) {
        batch_release(bt);
        return fail_hip("sam_batch_init: hipMalloc", e);
    }
    bt->device_bytes = (int64_t)(bb.text + bb.rec + bb.slots + bb.meta + 256);
    StaticView S = corpus ? corpus->view : StaticView{};
    if ((e = hipMemsetAsync(v.dyn_slots, 0xFF, bb.slots, stream)) != hipSuccess ||
        (e = launch_reset(v, nullptr, batch, stream)) != hipSuccess ||
        (e = launch_ingest(S, v, nullptr, batch, prompt_tokens, prompt_offsets,
                           offs.data(), 0, stream)) != hipSuccess ||
        (e = hipStreamSynchronize(stream)) != hipSuccess) {
        batch_release(bt);
        return fail_hip("sam_batch_init: prompt ingest", e);
    }
    uint32_t st = 0;
    if ((e = hipMemcpy(&st, v.status, sizeof(st), hipMemcpyDeviceToHost)) != hipSuccess) {
        batch_release(bt);
        return fail_hip("sam_batch_init: status read", e);
    }
    if (st & SAM_STATUS_TOKEN) {
        batch_release(bt);
        return fail(SAM_ETOKEN, "sam_batch_init: a prompt token is outside [0, vocab)");
    }
    *out = bt;
    return SAM_OK;
}

int sam_batch_init_noalloc(const sam_corpus *corpus, const int32_t *prompt_tokens,
                           const int64_t *prompt_offsets, const int64_t *prompt_offsets_host,
                           int32_t batch, int32_t vocab, int32_t max_seq_len, int32_t max_accept,
                           int32_t draft_len, int32_t l_bias, void *hip_stream, sam_batch **out)
{
    static const char *fn = "sam_batch_init_noalloc";
    if (!out) return fail(SAM_EINVAL, "sam_batch_init_noalloc: out is NULL");
    *out = nullptr;
    if (!prompt_offsets_host)
        return fail(SAM_EINVAL, "sam_batch_init_noalloc: prompt_offsets_host is NULL");
    int rc = batch_check_args(fn, corpus, prompt_tokens, prompt_offsets, batch, vocab, max_seq_len,
                              max_accept, draft_len);
    if (rc != SAM_OK) return rc;
    rc = batch_check_offsets(fn, prompt_offsets_host, batch, max_seq_len);
    if (rc != SAM_OK) return rc;
    hipStream_t stream = (hipStream_t)hip_stream;
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices)
        return fail(SAM_EINVAL, "sam_batch_init_noalloc: device index beyond " +
                                    std::to_string(kMaxDevices - 1));

    BatchView v = {};
    const BatchBytes bb = batch_configure(v, corpus, batch, vocab, max_seq_len, max_accept,
                                          draft_len, l_bias);
    auto up = [](size_t x) { return (x + 255) / 256 * 256; };
    const size_t o_text = 0, o_rec = o_text + up(bb.text), o_slots = o_rec + up(bb.rec),
                 o_meta = o_slots + up(bb.slots), o_status = o_meta + up(bb.meta),
                 need = o_status + 256;
    if (need > kNoAllocBytes)
        return fail(SAM_EINVAL, "sam_batch_init_noalloc: these sizes need " + std::to_string(need) +
                                    " bytes of table space, the fixed buffer holds " +
                                    std::to_string(kNoAllocBytes) +
                                    " (use sam_batch_init for larger batches)");

    NoAllocSlot &slot = g_noalloc[dev];
    unsigned char *base = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_noalloc_mu);
        if (slot.busy)
            return fail(SAM_EINVAL, "sam_batch_init_noalloc: the fixed buffer of this device is in "
                                    "use by a batch that has not been freed");
        hipError_t e = noalloc_base_locked(dev, &base);
        if (e != hipSuccess) return fail_hip("sam_batch_init_noalloc: address of the fixed buffer", e);
        slot.busy = true;
    }
    v.dyn_text = (int32_t *)(base + o_text);
    v.dyn_rec = base + o_rec;
    v.dyn_slots = base + o_slots;
    v.meta = (SeqMeta *)(base + o_meta);
    v.status = (uint32_t *)(base + o_status);
    sam_batch *bt = &slot.handle;
    bt->corpus = corpus;
    bt->view = v;
    bt->device_bytes = (int64_t)need;
    bt->noalloc_device = dev;
    // the buffer keeps what the last batch left: empty the slot tables, then fresh
    // records, cursors and status word (the reset kernel), then the prompts
    StaticView S = corpus ? corpus->view : StaticView{};
    // the device's offsets are read when the kernel runs; in a captured graph they may be others
    // by then, up to what a sequence holds
    hipError_t e;
    if ((e = launch_fill_empty(v.dyn_slots, bb.slots, stream)) != hipSuccess ||
        (e = launch_reset(v, nullptr, batch, stream)) != hipSuccess ||
        (e = launch_ingest(S, v, nullptr, batch, prompt_tokens, prompt_offsets, prompt_offsets_host,
                           max_seq_len, stream)) != hipSuccess) {
        batch_release(bt);
        return fail_hip("sam_batch_init_noalloc: launch", e);
    }
    *out = bt;
    return SAM_OK;
}

int sam_batch_step(sam_batch *bt, const int32_t *accepted, const int32_t *counts,
                   int32_t *match_len, int32_t *draft, int32_t *draft_len, int32_t *source,
                   void *hip_stream)
{
    if (!bt) return fail(SAM_EINVAL, "sam_batch_step: batch is NULL");
    if (!accepted || !counts || !match_len || !draft || !draft_len || !source)
        return fail(SAM_EINVAL, "sam_batch_step: NULL buffer");
    StaticView S = bt->corpus ? bt->corpus->view : StaticView{};
    hipError_t e = launch_feed(S, bt->view, nullptr, bt->view.batch, accepted, nullptr, counts,
                               match_len, draft, draft_len, source, (hipStream_t)hip_stream);
    if (e != hipSuccess) return fail_hip("sam_batch_step: launch", e);
    return SAM_OK;
}

int sam_batch_replay(sam_batch *bt, int32_t n_steps, const int32_t *accepted, const int32_t *counts,
                     int32_t *match_len, int32_t *draft, int32_t *draft_len, int32_t *source,
                     void *hip_stream)
{
    if (!bt) return fail(SAM_EINVAL, "sam_batch_replay: batch is NULL");
    if (!accepted || !counts || !match_len || !draft || !draft_len || !source)
        return fail(SAM_EINVAL, "sam_batch_replay: NULL buffer");
    if (n_steps < 1) return fail(SAM_EINVAL, "sam_batch_replay: n_steps must be >= 1");
    StaticView S = bt->corpus ? bt->corpus->view : StaticView{};
    hipError_t e = launch_replay(S, bt->view, n_steps, accepted, counts, match_len, draft,
                                 draft_len, source, (hipStream_t)hip_stream);
    if (e != hipSuccess) return fail_hip("sam_batch_replay: launch", e);
    return SAM_OK;
}

int sam_membench(int32_t kind, int64_t size, int64_t count, int32_t workgroups, double *result)
{
    if (!result) return fail(SAM_EINVAL, "sam_membench: result is NULL");
    std::string err;
    const int rc = membench(kind, size, count, workgroups, result, err);
    return rc == SAM_OK ? SAM_OK : fail(rc, err);
}

int sam_batch_tree_draft(sam_batch *bt, int32_t max_size, int32_t *tokens, int32_t *parents,
                         float *probs, int32_t *sizes, void *hip_stream)
{
    if (!bt) return fail(SAM_EINVAL, "sam_batch_tree_draft: batch is NULL");
    if (!tokens || !parents || !probs || !sizes)
        return fail(SAM_EINVAL, "sam_batch_tree_draft: NULL buffer");
    if (!bt->corpus || !bt->corpus->view.topk)
        return fail(SAM_EINVAL, "sam_batch_tree_draft: the batch has no corpus with a top-k "
                                "table (sam_corpus_build_topk)");
    if (max_size < 1 || max_size > kMaxTreeSize)
        return fail(SAM_EINVAL, "sam_batch_tree_draft: max_size must be in 1 .. " +
                                    std::to_string(kMaxTreeSize));
    hipError_t e = launch_tree(bt->corpus->view, bt->view, max_size, tokens, parents, probs,
                               sizes, (hipStream_t)hip_stream);
    if (e != hipSuccess) return fail_hip("sam_batch_tree_draft: launch", e);
    return SAM_OK;
}

int sam_batch_reset(sam_batch *bt, const int32_t *slots, int32_t n_slots,
                    const int32_t *prompt_tokens, const int64_t *prompt_offsets, void *hip_stream)
{
    if (!bt) return fail(SAM_EINVAL, "sam_batch_reset: batch is NULL");
    if (!slots || !prompt_tokens || !prompt_offsets)
        return fail(SAM_EINVAL, "sam_batch_reset: NULL buffer");
    const BatchView &v = bt->view;
    if (n_slots < 1 || n_slots > v.batch)
        return fail(SAM_EINVAL, "sam_batch_reset: n_slots must be in 1 .. batch");
    hipStream_t stream = (hipStream_t)hip_stream;
    std::vector<int32_t> hs;
    std::vector<int64_t> offs;
    std::vector<char> seen;
    try {
        hs.resize((size_t)n_slots);
        offs.resize((size_t)n_slots + 1);
        seen.assign((size_t)v.batch, 0);
    } catch (const std::bad_alloc &) {
        return fail(SAM_ENOMEM, "sam_batch_reset: out of host memory");
    }
    HIP_TRY(hipMemcpyAsync(hs.data(), slots, hs.size() * sizeof(int32_t), hipMemcpyDeviceToHost,
                           stream));
    HIP_TRY(hipMemcpyAsync(offs.data(), prompt_offsets, offs.size() * sizeof(int64_t),
                           hipMemcpyDeviceToHost, stream));
    HIP_TRY(hipStreamSynchronize(stream));
    if (offs[0] < 0) return fail(SAM_EINVAL, "sam_batch_reset: prompt_offsets[0] < 0");
    for (int32_t i = 0; i < n_slots; i++) {
        if (hs[i] < 0 || hs[i] >= v.batch)
            return fail(SAM_EINVAL, "sam_batch_reset: slot " + std::to_string(hs[i]) +
                                        " is outside the batch");
        if (seen[hs[i]])
            return fail(SAM_EINVAL, "sam_batch_reset: slot " + std::to_string(hs[i]) +
                                        " is listed twice");
        seen[hs[i]] = 1;
        const int64_t len = offs[i + 1] - offs[i];
        if (len < 0) return fail(SAM_EINVAL, "sam_batch_reset: prompt_offsets must not decrease");
        if (len > (int64_t)v.max_seq_len)
            return fail(SAM_ECAPACITY, "sam_batch_reset: prompt " + std::to_string(i) + " has " +
                                           std::to_string(len) + " tokens, max_seq_len is " +
                                           std::to_string(v.max_seq_len));
    }
    StaticView S = bt->corpus ? bt->corpus->view : StaticView{};
    hipError_t e;
    if ((e = launch_reset(v, slots, n_slots, stream)) != hipSuccess ||
        (e = launch_ingest(S, v, slots, n_slots, prompt_tokens, prompt_offsets,
                           offs.data(), 0, stream)) != hipSuccess)
        return fail_hip("sam_batch_reset: launch", e);
    return SAM_OK;
}

int sam_batch_debug(const sam_batch *bt, int32_t *s1, int32_t *l1, int32_t *s2, int32_t *l2,
                    void *hip_stream)
{
    if (!bt) return fail(SAM_EINVAL, "sam_batch_debug: batch is NULL");
    hipError_t e = launch_debug(bt->view, s1, l1, s2, l2, nullptr, nullptr, nullptr,
                                (hipStream_t)hip_stream);
    if (e != hipSuccess) return fail_hip("sam_batch_debug: launch", e);
    return SAM_OK;
}

int sam_batch_sizes(const sam_batch *bt, int32_t *text_len, int32_t *n_states, int32_t *n_trans,
                    void *hip_stream)
{
    if (!bt) return fail(SAM_EINVAL, "sam_batch_sizes: batch is NULL");
    hipError_t e = launch_debug(bt->view, nullptr, nullptr, nullptr, nullptr, text_len, n_states,
                                n_trans, (hipStream_t)hip_stream);
    if (e != hipSuccess) return fail_hip("sam_batch_sizes: launch", e);
    return SAM_OK;
}

int sam_batch_status(const sam_batch *bt, uint32_t *status, void *hip_stream)
{
    if (!bt || !status) return fail(SAM_EINVAL, "sam_batch_status: NULL argument");
    hipStream_t stream = (hipStream_t)hip_stream;
    HIP_TRY(hipMemcpyAsync(status, bt->view.status, sizeof(uint32_t), hipMemcpyDeviceToHost,
                           stream));
    HIP_TRY(hipStreamSynchronize(stream));
    return SAM_OK;
}

int sam_batch_set_threshold(sam_batch *bt, int32_t l_threshold)
{
    if (!bt) return fail(SAM_EINVAL, "sam_batch_set_threshold: batch is NULL");
    bt->view.l_threshold = l_threshold < 0 ? -1 : l_threshold;
    return SAM_OK;
}

int sam_set_progress_callback(sam_progress_fn fn, void *user)
{
    g_progress = fn;
    g_progress_user = user;
    return SAM_OK;
}

int sam_set_layout_override(int mode)
{
    if (mode < 0 || mode > 2047) return fail(SAM_EINVAL, "sam_set_layout_override: mode is 0 .. 2047");
    g_layout_override = mode;
    return SAM_OK;
}

int sam_batch_info(const sam_batch *bt, int64_t *device_bytes)
{
    if (!bt || !device_bytes) return fail(SAM_EINVAL, "sam_batch_info: NULL argument");
    *device_bytes = bt->device_bytes;
    return SAM_OK;
}

void sam_batch_free(sam_batch *bt)
{
    if (!bt) return;
    batch_release(bt);
}

}  // extern "C"
