// The walk over the corpus automaton (arxiv 2411.10666: Algorithm 1 Transfer), as one wave
// does it: in C++ and, for corpora below 2^32 buckets, in gfx950 assembly.  Shared by the
// kernels that feed tokens one by one and the one that takes prompts whole.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sam_device.h"

namespace sam {

namespace {

__device__ __forceinline__ uint32_t uni(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}

__device__ __forceinline__ uint32_t lane_get(uint32_t v, int src_lane)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)v, src_lane);
}

// Keep a wave-uniform value materialised at this point of the program, so the
// load that produced it cannot be moved below.
__device__ __forceinline__ void pin_s(uint32_t &v)
{
    asm volatile("" : "+s"(v));
}

// Same for a per-lane value.  Used on the step's token vector: once the load has
// landed before the token loop, reading a lane of it inside the loop no longer
// makes the wave wait for the stores of the previous token.
__device__ __forceinline__ void pin_v(uint32_t &v)
{
    asm volatile("" : "+v"(v));
}

__device__ __forceinline__ void order_memory()
{
    // stores and later loads of one wavefront reach memory in program order;
    // this only stops the compiler from moving them across each other
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
}

// ---- static automaton: Transfer (Algorithm 1) -----------------------------

// Feed one token.  (s, l) is the cursor, e = min_endpos(s) with the wide flag of s
// in bit 31 (a state is wide if it has transitions beyond the two in its record).
__device__ __forceinline__ void static_transfer(const StaticView &S, uint32_t t, int lane,
                                                uint32_t &s, uint32_t &l, uint32_t &e,
                                                uint32_t &fault)
{
    // every suffix-link hop shortens the match, so l + 1 rounds always suffice;
    // the bound only matters if the tables were corrupted
    for (uint32_t guard = l + 2; ; guard--) {
        if (guard == 0) { fault |= SAM_STATUS_INTERNAL_BIT; s = 0; l = 0; e = 0; return; }
        if (s == 0) {
            const uint2 r = reinterpret_cast<const uint2 *>(S.root)[t];
            uint32_t d = uni(r.x), ep = uni(r.y);
            pin_s(ep);
            if (d) { s = d; e = ep; l = 1; }
            else   { l = 0; e = 0; }
            return;
        }
        // the record answers for a state with at most two transitions; a wide state's
        // bucket is requested together with it
        const bool wide = (e & kWideBit) != 0;
        const LinkRec lr = S.linkrec[s];
        uint64_t b = 0;
        uint4 sl = make_uint4(kNil, kNil, 0, 0);
        if (wide) {
            b = bucket_of(hash_key(s, t), S.n_buckets);
            sl = reinterpret_cast<const uint4 *>(S.slots)[b * kBucketSlots + (lane & 7)];
        }
        if (uni(lr.itok) == t) {
            s = uni(lr.idst); e = uni(lr.iendpos); l += 1;
            return;
        }
        if (uni(lr.itok2) == t) {
            s = uni(lr.idst2); e = uni(lr.iendpos2); l += 1;
            return;
        }
        uint32_t nlink = uni(lr.link), nlen = uni(lr.lenlink);
        pin_s(nlink);
        bool hit = false;
        if (wide) {
            uint32_t mh = (uint32_t)__ballot(sl.x == s && sl.y == t) & 0xFFu;
            uint32_t me = (uint32_t)__ballot(sl.x == kNil) & 0xFFu;
            pin_s(mh);
            for (uint64_t left = S.n_buckets; left; left--) {
                if (mh) {
                    const int j = __builtin_ctz(mh);
                    s = lane_get(sl.z, j);
                    e = lane_get(sl.w, j);
                    l += 1;
                    hit = true;
                    break;
                }
                if (me) break;
                b = (b + 1 == S.n_buckets) ? 0 : b + 1;
                sl = reinterpret_cast<const uint4 *>(S.slots)[b * kBucketSlots + (lane & 7)];
                mh = (uint32_t)__ballot(sl.x == s && sl.y == t) & 0xFFu;
                me = (uint32_t)__ballot(sl.x == kNil) & 0xFFu;
            }
        }
        if (hit) return;
        s = nlink;
        l = nlen & ~kWideBit;
        e = nlen & kWideBit;
    }
}
// Transfer (Algorithm 1) over tokens tv[i .. m) in gfx950 assembly: the same
// steps as static_transfer, about a third of the instructions.  Lanes 0..7 fetch
// the 8 slots of a bucket, the suffix-link record travels with the bucket.  i:
// index of the next token (in/out); on return i == m or tv[i] is outside the
// vocabulary.  Needs n_buckets < 2^32.
//   s64 t   s65 t * c2   s66 link-hop guard   s67 bucket-sweep guard
//   s68:69 s70:71 addresses / compare results   s72 hash   s73 bucket
//   s74 hit mask   s75 empty mask   s76:77 compare result   s78 s79 scratch
//   v41 zero   v42:45 slot {state, token, dst, endpos}   s88..s95 state record   v46:47 root entry
__device__ __forceinline__ void static_feed_asm(uint32_t slots_lo, uint32_t slots_hi,
                                                uint32_t lr_lo, uint32_t lr_hi, uint32_t root_lo,
                                                uint32_t root_hi, uint32_t nb, uint32_t m,
                                                uint32_t vocab, uint32_t tv, uint32_t lane16,
                                                uint32_t &i, uint32_t &st, uint32_t &l,
                                                uint32_t &e, uint32_t &flt)
{
    asm volatile(
        "s_mov_b64 s[96:97], exec\n\t"
        "s_mov_b64 exec, 0xff\n\t"
        "v_mov_b32 v41, 0\n"
        "L_stok_%=:\n\t"
        "v_readlane_b32 s64, %[tv], %[i]\n\t"
        "s_add_u32 s66, %[l], 2\n\t"            // every link hop shortens the match
        "s_cmp_ge_u32 s64, %[vocab]\n\t"
        "s_cbranch_scc1 L_sexit_%=\n\t"
        "s_mul_i32 s65, s64, 0x85ebca77\n"
        "L_stry_%=:\n\t"
        "s_sub_u32 s66, s66, 1\n\t"
        "s_cbranch_scc1 L_scorrupt_%=\n\t"
        "s_cmp_eq_u32 %[st], 0\n\t"
        "s_cbranch_scc1 L_sroot_%=\n\t"
        // the state's record {itok, idst, iendpos, itok2, idst2, iendpos2, link, lenlink}.
        // It comes through the scalar cache (the table is read-only), which has its own
        // counter: vector loads return in order, so a record behind a bucket in the same
        // queue could not arrive before it.  Bit 31 of e says whether the state is wide;
        // if not, its record holds all its transitions and no bucket is requested.
        "s_lshl_b32 s68, %[st], 5\n\t"
        "s_lshr_b32 s69, %[st], 27\n\t"
        "s_add_u32 s68, s68, %[lr_lo]\n\t"
        "s_addc_u32 s69, s69, %[lr_hi]\n\t"
        "s_load_dwordx8 s[88:95], s[68:69], 0x0\n\t"
        "s_bitcmp1_b32 %[e], 31\n\t"
        "s_cbranch_scc0 L_srec_%=\n\t"
        "s_mul_i32 s72, %[st], 0x9e3779b1\n\t"
        "s_add_u32 s72, s72, s65\n\t"
        "s_lshr_b32 s79, s72, 15\n\t"
        "s_xor_b32 s72, s72, s79\n\t"
        "s_mul_i32 s72, s72, 0x2c1b3c6d\n\t"
        "s_lshr_b32 s79, s72, 12\n\t"
        "s_xor_b32 s72, s72, s79\n\t"
        "s_mul_i32 s72, s72, 0x297a2d39\n\t"
        "s_lshr_b32 s79, s72, 15\n\t"
        "s_xor_b32 s72, s72, s79\n\t"
        "s_mul_hi_u32 s73, s72, %[nb]\n\t"
        "s_mov_b32 s67, %[nb]\n\t"
        "s_lshl_b32 s70, s73, 7\n\t"
        "s_lshr_b32 s71, s73, 25\n\t"
        "s_add_u32 s70, s70, %[slots_lo]\n\t"
        "s_addc_u32 s71, s71, %[slots_hi]\n\t"
        "global_load_dwordx4 v[42:45], %[lane16], s[70:71]\n\t"
        // the record is here before the bucket (often from a line the last token
        // already brought in): if it repeats the transition asked for, the bucket is
        // not waited for at all
        "s_waitcnt lgkmcnt(0)\n\t"
        "s_cmp_eq_u32 s88, s64\n\t"
        "s_cbranch_scc1 L_sinline_%=\n\t"
        "s_cmp_eq_u32 s91, s64\n\t"
        "s_cbranch_scc1 L_sinline2_%=\n\t"
        "s_branch L_swait_%=\n"
        "L_srec_%=:\n\t"
        "s_waitcnt lgkmcnt(0)\n\t"
        "s_cmp_eq_u32 s88, s64\n\t"
        "s_cbranch_scc1 L_sinline_%=\n\t"
        "s_cmp_eq_u32 s91, s64\n\t"
        "s_cbranch_scc1 L_sinline2_%=\n\t"
        "s_branch L_smiss_%=\n"
        "L_sload_%=:\n\t"
        "s_lshl_b32 s70, s73, 7\n\t"
        "s_lshr_b32 s71, s73, 25\n\t"
        "s_add_u32 s70, s70, %[slots_lo]\n\t"
        "s_addc_u32 s71, s71, %[slots_hi]\n\t"
        "global_load_dwordx4 v[42:45], %[lane16], s[70:71]\n"
        "L_swait_%=:\n\t"
        "s_waitcnt vmcnt(0)\n\t"
        "v_cmp_eq_u32 vcc, %[st], v42\n\t"
        "v_cmp_eq_u32 s[76:77], s64, v43\n\t"
        "v_cmp_eq_u32 s[70:71], -1, v42\n\t"
        "s_and_b32 s74, vcc_lo, s76\n\t"
        "s_mov_b32 s75, s70\n\t"
        "s_cmp_lg_u32 s74, 0\n\t"
        "s_cbranch_scc1 L_shit_%=\n\t"
        "s_cmp_lg_u32 s75, 0\n\t"
        "s_cbranch_scc1 L_smiss_%=\n\t"
        // bucket full of other keys: go on in the next one
        "s_sub_u32 s67, s67, 1\n\t"
        "s_cbranch_scc1 L_scorrupt_%=\n\t"
        "s_add_u32 s73, s73, 1\n\t"
        "s_cmp_eq_u32 s73, %[nb]\n\t"
        "s_cselect_b32 s73, 0, s73\n\t"
        "s_branch L_sload_%=\n"
        "L_shit_%=:\n\t"
        "s_ff1_i32_b32 s78, s74\n\t"
        "s_add_u32 %[l], %[l], 1\n\t"
        "v_readlane_b32 %[st], v44, s78\n\t"
        "v_readlane_b32 %[e], v45, s78\n\t"
        "s_branch L_sdone_%=\n"
        "L_sinline_%=:\n\t"
        "s_add_u32 %[l], %[l], 1\n\t"
        "s_mov_b32 %[st], s89\n\t"
        "s_mov_b32 %[e], s90\n\t"
        "s_branch L_sdone_%=\n"
        "L_sinline2_%=:\n\t"
        "s_add_u32 %[l], %[l], 1\n\t"
        "s_mov_b32 %[st], s92\n\t"
        "s_mov_b32 %[e], s93\n\t"
        "s_branch L_sdone_%=\n"
        "L_smiss_%=:\n\t"
        "s_mov_b32 %[st], s94\n\t"              // follow the suffix link
        "s_and_b32 %[l], s95, 0x7fffffff\n\t"
        "s_and_b32 %[e], s95, 0x80000000\n\t"   // its wide flag; its end position is not needed
        "s_branch L_stry_%=\n"
        "L_sroot_%=:\n\t"
        "s_lshl_b32 s68, s64, 3\n\t"
        "s_add_u32 s68, s68, %[root_lo]\n\t"
        "s_addc_u32 s69, %[root_hi], 0\n\t"
        "global_load_dwordx2 v[46:47], v41, s[68:69]\n\t"
        "s_waitcnt vmcnt(0)\n\t"
        "v_readfirstlane_b32 s78, v46\n\t"
        "v_readfirstlane_b32 s79, v47\n\t"
        "s_cmp_eq_u32 s78, 0\n\t"
        "s_cbranch_scc1 L_snone_%=\n\t"
        "s_mov_b32 %[st], s78\n\t"
        "s_mov_b32 %[e], s79\n\t"
        "s_mov_b32 %[l], 1\n\t"
        "s_branch L_sdone_%=\n"
        "L_snone_%=:\n\t"
        "s_mov_b32 %[l], 0\n\t"
        "s_mov_b32 %[e], 0\n"
        "L_sdone_%=:\n\t"
        "s_add_u32 %[i], %[i], 1\n\t"
        "s_cmp_lt_u32 %[i], %[m]\n\t"
        "s_cbranch_scc1 L_stok_%=\n\t"
        "s_branch L_sexit_%=\n"
        "L_scorrupt_%=:\n\t"
        "s_or_b32 %[flt], %[flt], 8\n\t"
        "s_mov_b32 %[st], 0\n\t"
        "s_mov_b32 %[l], 0\n\t"
        "s_mov_b32 %[e], 0\n"
        "L_sexit_%=:\n\t"
        "s_waitcnt vmcnt(0)\n\t"
        "s_mov_b64 exec, s[96:97]\n\t"
        : [i] "+s"(i), [st] "+s"(st), [l] "+s"(l), [e] "+s"(e), [flt] "+s"(flt)
        : [slots_lo] "s"(slots_lo), [slots_hi] "s"(slots_hi), [lr_lo] "s"(lr_lo),
          [lr_hi] "s"(lr_hi), [root_lo] "s"(root_lo), [root_hi] "s"(root_hi), [nb] "s"(nb),
          [m] "s"(m), [vocab] "s"(vocab), [tv] "v"(tv), [lane16] "v"(lane16)
        : "memory", "vcc", "scc",
          "s64", "s65", "s66", "s67", "s68", "s69", "s70", "s71", "s72", "s73", "s74", "s75",
          "s76", "s77", "s78", "s79", "s88", "s89", "s90", "s91", "s92", "s93", "s94", "s95",
          "s96", "s97",
          "v41", "v42", "v43", "v44", "v45", "v46", "v47");
}

// Wave 0: feed `count` tokens to the static cursor; stops in front of a token
// outside the vocabulary (wave 1 reports it).
__device__ __forceinline__ void static_feed(const StaticView &S, const int32_t *tok, int64_t count,
                                            uint32_t vocab, int lane, uint32_t &s, uint32_t &l,
                                            uint32_t &e, uint32_t &fault, bool use_asm,
                                            bool have_first = false, uint32_t first = 0)
{
    bool stop = false;
    const bool in_asm = use_asm;          // the launcher sends corpora beyond 2^32 buckets to C++
    for (int64_t base = 0; base < count && !stop; base += 64) {
        const int m = (int)((count - base) < 64 ? (count - base) : 64);
        uint32_t tv;
        if (have_first && base == 0) tv = first;     // fetched by the caller with its other loads
        else tv = lane < m ? (uint32_t)tok[base + lane] : 0u;
        pin_v(tv);
        if (in_asm) {
            const uint64_t a_sl = (uint64_t)S.slots, a_lr = (uint64_t)S.linkrec,
                           a_rt = (uint64_t)S.root;
            uint32_t i = 0, flt = 0;
            uint32_t a_s = uni(s), a_l = uni(l), a_e = uni(e);
            static_feed_asm(uni((uint32_t)a_sl), uni((uint32_t)(a_sl >> 32)), uni((uint32_t)a_lr),
                            uni((uint32_t)(a_lr >> 32)), uni((uint32_t)a_rt),
                            uni((uint32_t)(a_rt >> 32)), uni((uint32_t)S.n_buckets),
                            uni((uint32_t)m), uni(vocab), tv, (uint32_t)(lane & 7) * 16u, i, a_s,
                            a_l, a_e, flt);
            s = a_s; l = a_l; e = a_e;
            fault |= flt;
            if ((int)i < m) stop = true;
        } else {
            for (int i = 0; i < m; i++) {
                const uint32_t t = lane_get(tv, i);
                if (t >= vocab) { stop = true; break; }
                static_transfer(S, t, lane, s, l, e, fault);
            }
        }
    }
}

}  // namespace

}  // namespace sam
