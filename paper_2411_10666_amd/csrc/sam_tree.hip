// gfx950 kernel for tree drafts from the static automaton (arxiv 2411.10666,
// Section 3.2 and Algorithm 4: best-first expansion over the top-k successors
// that Algorithm 3 computed on the host).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sam_device.h"

namespace sam {

namespace {

__device__ __forceinline__ uint32_t uni(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}

// Maximum of a value over the 64 lanes: data-parallel-primitive moves that the compiler
// folds into the maximum itself (0 is what a lane without a partner compares with), within
// rows of 16 lanes and then row by row; the last lane has it.
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t x)
{
#define SAM_DPP_MAX(ctrl, rows)                                                                    \
    do {                                                                                           \
        const uint32_t y = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, ctrl, rows, 0xF, false); \
        x = x > y ? x : y;                                                                         \
    } while (0)
    SAM_DPP_MAX(0xB1, 0xF);       // lanes i ^ 1
    SAM_DPP_MAX(0x4E, 0xF);       // lanes i ^ 2
    SAM_DPP_MAX(0x141, 0xF);      // 7 - i in each half row
    SAM_DPP_MAX(0x140, 0xF);      // 15 - i in each row
    SAM_DPP_MAX(0x142, 0xA);      // rows 1 and 3: the last lane of the row before
    SAM_DPP_MAX(0x143, 0xC);      // rows 2 and 3: the last lane of row 1
#undef SAM_DPP_MAX
    return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
}

}  // namespace

// Tree draft by best-first expansion over the top-k successors (Algorithm 4),
// one wavefront per sequence.  Entry number i of the priority queue (in the order of the
// pushes) belongs to lane i % 64, row i / 64.  The largest probability comes first and, among
// equals, the entry pushed first.
//
// A pop is one dependent memory read (the table row of the popped state's k children) and
// the work between its arrival and the next request.  The lanes that will hold the
// children request them, so they arrive where they stay.  Of the children only the first
// can be the next pop (a row is ordered by falling probability, and the product with the
// parent's probability keeps that order), and the best of the entries already queued was
// found while the request travelled: when the row is here, one product, two lane reads and
// a compare give the next state, and its row is requested before anything else is done.
// Queueing the children and the search for the best entry follow in that request's shadow.
// Tokens and parents go to LDS when pushed, the popped entries too, and come back once, when
// the draft is written out.
// Probabilities are float products rounded once per edge.  The rest of a pop's 0.45 us is
// the row's round trip (a 69 MB table; a call of 256 drafts of 40 entries, k = 4: 18 us).
// Asking for the row of the queue's best entry ahead, in case
// the next pop is that one, cost 2.4 us a call: the two requests are waited for together.
//
// The queue has two forms, because the search has to stay in the shadow.  Up to 128 entries: two
// rows in registers, probability bits (0: popped or not there yet) and state.  More: rows in
// LDS, below.  Measured (us a call from the host, 64 drafts, states from the L2; all rows in
// registers, a queue in LDS that is scanned at each pop, the two forms here): 128 entries of k = 8
// 143, 83, 67; of k = 4 96, 83, 67; of k = 1 (two rows) 63, 84, 63, and 67 with the second form; 40
// entries of k = 8 37, 39, 34; of k = 4 34, 39, 34.
constexpr int kRegisterRows = 2;
__global__ __launch_bounds__(64) void sam_tree_kernel(StaticView S, BatchView B, int max_size,
                                                       int32_t *__restrict__ tokens,
                                                       int32_t *__restrict__ parents,
                                                       float *__restrict__ probs,
                                                       int32_t *__restrict__ sizes)
{
    __shared__ int32_t qtok[64 * kRegisterRows];
    __shared__ int32_t qpar[64 * kRegisterRows];
    __shared__ int32_t oidx[kMaxTreeSize];
    __shared__ float   oprob[kMaxTreeSize];
    const int b = blockIdx.x;
    const int lane = threadIdx.x;
    const SeqMeta m = B.meta[b];
    const int k = S.top_k;
    int dn = 0;
    if (m.n > 0) {
        uint32_t prob[kRegisterRows], state[kRegisterRows];
#pragma unroll
        for (int r = 0; r < kRegisterRows; r++) { prob[r] = 0; state[r] = 0; }
        if (lane == 0) {
            qtok[0] = B.dyn_text[(size_t)b * B.max_seq_len + m.n - 1];
            qpar[0] = -1;
        }
        int qn = 1;
        uint32_t st = (uint32_t)__builtin_amdgcn_readfirstlane((int)m.s1);
        uint32_t p = __float_as_uint(1.0f);
        int idx = 0;                                     // the popped entry
        // Lane (first + j) % 64 asks for child j, the other lanes for child 0 once more: no
        // branch, so the result stays in the registers it arrives in until it is needed.
        auto request = [&](uint32_t of, int first) {
            const int j = (lane - first) & 63;
            return S.topk[(size_t)of * (uint32_t)k + (uint32_t)(j < k ? j : 0)];
        };
        TopEnt e = request(st, qn);
        uint32_t best = 0, best_state = 0;               // of the queue, the popped entry left out
        int best_at = 0;
        for (;;) {
            oidx[dn] = idx;                              // (every lane writes the same)
            oprob[dn] = __uint_as_float(p);
            dn++;
            if (dn == max_size) break;
            const int mine_no = (lane - qn) & 63;
            const bool valid = e.dst != 0 && mine_no < k;
            const uint32_t pn = valid ? __float_as_uint(__fmul_rn(__uint_as_float(p), e.prob)) : 0u;
            const uint32_t first_p = (uint32_t)__builtin_amdgcn_readlane((int)pn, qn & 63);
            const uint32_t first_state = (uint32_t)__builtin_amdgcn_readlane((int)e.dst, qn & 63);
            const bool child = first_p > best;           // a tie goes to the entry pushed earlier
            if (!child && best == 0) break;              // nothing left
            // the number a child in this lane takes (the compares below never meet -1)
            const int slot = valid ? qn + mine_no : -1;
            idx = (int)uni((uint32_t)(child ? qn : best_at));
            qn = (int)uni((uint32_t)(qn + __popcll(__ballot(valid))));
            st = uni(child ? first_state : best_state);
            p = uni(child ? first_p : best);
            const TopEnt coming = request(st, qn);
            if (valid) {
                qtok[slot] = (int32_t)e.token;
                qpar[slot] = dn - 1;
            }
#pragma unroll
            for (int r = 0; r < kRegisterRows; r++) {
                const bool here = slot == 64 * r + lane;
                prob[r] = here ? pn : prob[r];
                state[r] = here ? e.dst : state[r];
                prob[r] = idx == 64 * r + lane ? 0u : prob[r];       // popped
            }
            // The best of the queue.  Among equals the entry pushed first is the one in the
            // lowest register that has one, and there in the lowest lane.
            uint32_t mine = prob[0];
#pragma unroll
            for (int r = 1; r < kRegisterRows; r++) mine = prob[r] > mine ? prob[r] : mine;
            best = wave_max_u32(mine);
#pragma unroll
            for (int r = kRegisterRows - 1; r >= 0; r--) {
                const unsigned long long holders = __ballot(prob[r] == best);
                const int from = __builtin_ctzll(holders | (1ull << 63));
                const uint32_t its = (uint32_t)__builtin_amdgcn_readlane((int)state[r], from);
                best_at = holders ? 64 * r + from : best_at;
                best_state = holders ? its : best_state;
            }
            // Only here is the row waited for: as plain assignments these moves (and the wait
            // for the row with them) end up in front of the search.
            asm volatile("v_mov_b32 %0, %3\n\tv_mov_b32 %1, %4\n\tv_mov_b32 %2, %5"
                         : "=&v"(e.token), "=&v"(e.dst), "=&v"(e.prob)
                         : "v"(coming.token), "v"(coming.dst), "v"(coming.prob), "s"(best));
        }
    }
    __syncthreads();
    for (int i = lane; i < max_size; i += 64) {
        const bool have = i < dn;
        const int q = have ? oidx[i] : 0;
        tokens[(size_t)b * max_size + i] = have ? qtok[q] : -1;
        parents[(size_t)b * max_size + i] = have ? qpar[q] : -1;
        probs[(size_t)b * max_size + i] = have ? oprob[i] : 0.0f;
    }
    if (lane == 0) sizes[b] = dn;
}

// More than 128 entries: the rows are in LDS, and every lane keeps the best entry of its own column in
// registers.  A push changes that by one compare; a pop of a queued entry makes the one lane it
// came from read its column again.
template <int R>
__global__ __launch_bounds__(64) void sam_tree_large_kernel(StaticView S, BatchView B, int max_size,
                                                             int32_t *__restrict__ tokens,
                                                             int32_t *__restrict__ parents,
                                                             float *__restrict__ probs,
                                                             int32_t *__restrict__ sizes)
{
    __shared__ uint32_t qprob[64 * R];                   // 0: popped
    __shared__ uint32_t qstate[64 * R];
    __shared__ int32_t  qtok[64 * R];
    __shared__ int32_t  qpar[64 * R];
    __shared__ int32_t  oidx[kMaxTreeSize];
    __shared__ float    oprob[kMaxTreeSize];
    const int b = blockIdx.x;
    const int lane = threadIdx.x;
    const SeqMeta m = B.meta[b];
    const int k = S.top_k;
    int dn = 0;
    if (m.n > 0) {
        if (lane == 0) {
            qtok[0] = B.dyn_text[(size_t)b * B.max_seq_len + m.n - 1];
            qpar[0] = -1;
            qprob[0] = 0;
        }
        int qn = 1;
        uint32_t st = (uint32_t)__builtin_amdgcn_readfirstlane((int)m.s1);
        uint32_t p = __float_as_uint(1.0f);
        int idx = 0;
        auto request = [&](uint32_t of, int first) {
            const int j = (lane - first) & 63;
            return S.topk[(size_t)of * (uint32_t)k + (uint32_t)(j < k ? j : 0)];
        };
        TopEnt e = request(st, qn);
        uint32_t mine = 0, my_state = 0;                 // this lane's best
        int my_row = 0;
        uint32_t best = 0, best_state = 0;
        int best_at = 0;
        for (;;) {
            oidx[dn] = idx;
            oprob[dn] = __uint_as_float(p);
            dn++;
            if (dn == max_size) break;
            const int mine_no = (lane - qn) & 63;
            const bool valid = e.dst != 0 && mine_no < k;
            const uint32_t pn = valid ? __float_as_uint(__fmul_rn(__uint_as_float(p), e.prob)) : 0u;
            const uint32_t first_p = (uint32_t)__builtin_amdgcn_readlane((int)pn, qn & 63);
            const uint32_t first_state = (uint32_t)__builtin_amdgcn_readlane((int)e.dst, qn & 63);
            const bool child = first_p > best;
            if (!child && best == 0) break;
            const int slot = qn + mine_no;
            idx = (int)uni((uint32_t)(child ? qn : best_at));
            qn = (int)uni((uint32_t)(qn + __popcll(__ballot(valid))));
            st = uni(child ? first_state : best_state);
            p = uni(child ? first_p : best);
            const TopEnt coming = request(st, qn);
            if (valid) {
                const bool stays = slot != idx;
                qprob[slot] = stays ? pn : 0u;
                qstate[slot] = e.dst;
                qtok[slot] = (int32_t)e.token;
                qpar[slot] = dn - 1;
                if (stays && pn > mine) { mine = pn; my_state = e.dst; my_row = slot >> 6; }
            }
            if (!child && lane == (idx & 63)) {
                qprob[idx] = 0;
                mine = 0;
                for (int r = 0; 64 * r + lane < qn; r++) {
                    const uint32_t other = qprob[64 * r + lane];
                    if (other > mine) { mine = other; my_row = r; }
                }
                my_state = qstate[64 * my_row + lane];
            }
            best = wave_max_u32(mine);
            // among equals the entry pushed first: the lowest row, and there the lowest lane
            unsigned long long holders = __ballot(mine == best);
            if (holders & (holders - 1)) {
                const uint32_t row = 0xFFFFu - wave_max_u32(mine == best ? 0xFFFFu - (uint32_t)my_row : 0u);
                holders = __ballot(mine == best && my_row == (int)row);
            }
            const int from = __builtin_ctzll(holders | (1ull << 63));
            best_at = 64 * (int)__builtin_amdgcn_readlane(my_row, from) + from;
            best_state = (uint32_t)__builtin_amdgcn_readlane((int)my_state, from);
            asm volatile("v_mov_b32 %0, %3\n\tv_mov_b32 %1, %4\n\tv_mov_b32 %2, %5"
                         : "=&v"(e.token), "=&v"(e.dst), "=&v"(e.prob)
                         : "v"(coming.token), "v"(coming.dst), "v"(coming.prob), "s"(best));
        }
    }
    __syncthreads();
    for (int i = lane; i < max_size; i += 64) {
        const bool have = i < dn;
        const int q = have ? oidx[i] : 0;
        tokens[(size_t)b * max_size + i] = have ? qtok[q] : -1;
        parents[(size_t)b * max_size + i] = have ? qpar[q] : -1;
        probs[(size_t)b * max_size + i] = have ? oprob[i] : 0.0f;
    }
    if (lane == 0) sizes[b] = dn;
}

hipError_t launch_tree(const StaticView &S, const BatchView &B, int max_size, int32_t *tokens,
                       int32_t *parents, float *probs, int32_t *sizes, hipStream_t stream)
{
    // entries that can ever be pushed: the start and k children of every pop but the last
    const int most = 1 + (max_size - 1) * S.top_k;
#define SAM_LAUNCH_TREE(...)                                                                   \
    hipLaunchKernelGGL((__VA_ARGS__), dim3(B.batch), dim3(64), 0, stream, S, B, max_size,      \
                       tokens, parents, probs, sizes)
    static_assert(1 + (kMaxTreeSize - 1) * kMaxTopK <= 64 * 16, "the largest queue");
    // (8 and 16 rows differ in LDS only: 16 bytes an entry, 10 drafts a compute unit at 16 rows)
    if (most <= 64 * kRegisterRows) SAM_LAUNCH_TREE(sam_tree_kernel);
    else if (most <= 64 * 8) SAM_LAUNCH_TREE(sam_tree_large_kernel<8>);
    else SAM_LAUNCH_TREE(sam_tree_large_kernel<16>);
#undef SAM_LAUNCH_TREE
    return hipGetLastError();
}

}  // namespace sam
