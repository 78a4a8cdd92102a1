// Wavefront-level primitives for gfx950 (64 lanes).  They act inside one wavefront; a workgroup may hold several.
// Every function here must be called by all 64 lanes in wave-uniform control flow.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#define EST_DEV __device__ __forceinline__
#define EST_DEV_NOINLINE __device__ __attribute__((noinline))
#define EST_UNROLL _Pragma("unroll")
#define EST_CHECK(cond) ((void)0)
#define EST_CHK_ORDER_INIT() ((void)0)
#define EST_CHK_ORDER(tag) ((void)0)

namespace wv {

EST_DEV uint32_t lane() { return threadIdx.x & 63u; }

EST_DEV uint64_t ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }

// value of v in lane src (src may differ per lane)
EST_DEV uint32_t shfl(uint32_t v, uint32_t src) {
    return (uint32_t)__builtin_amdgcn_ds_bpermute((int)(src << 2), (int)v);
}

// lane l hands v to lane dst (0..63): the value a lane was handed, 0 where it was handed none.  Lanes that hand to the same lane
// must hand it the same value.
EST_DEV uint32_t push(uint32_t v, uint32_t dst) {
    return (uint32_t)__builtin_amdgcn_ds_permute((int)(dst << 2), (int)v);
}

// value of v in lane l; l must be the same in every lane
EST_DEV uint32_t bcast(uint32_t v, uint32_t l) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)__builtin_amdgcn_readfirstlane((int)l));
}

// is this lane's bit set in m?  (m must be the same in every lane; the mask is used as the lane
// predicate directly, no vector instruction is spent on it)
EST_DEV bool lane_in(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// The same for a mask known when compiling, written into scalar registers where it is used: left to itself the compiler
// makes the masks of all sorting networks before the loop they are in, and they spill: two reads and two writes of a vector lane
// per use instead of two scalar moves, and a dozen registers gone where they do not (spilled scalar registers of the simulation
// kernel 247 -> 153; with the rows exchanged by permlane swaps and an emission's batch starts found by one push, sweeps take 4 to 7 % less).
template <uint64_t M>
EST_DEV bool lane_in_const() {
    uint32_t lo, hi;
    asm volatile("s_mov_b32 %0, %1" : "=s"(lo) : "i"((int32_t)(uint32_t)M));
    asm volatile("s_mov_b32 %0, %1" : "=s"(hi) : "i"((int32_t)(uint32_t)(M >> 32)));
    return __builtin_amdgcn_inverse_ballot_w64(((uint64_t)hi << 32) | lo);
}

// value of lane-1 (lane 0 keeps its own) / of lane+1 (lane 63 keeps its own: shl1)
EST_DEV uint32_t shr1(uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x138, 0xF, 0xF, false); }
EST_DEV uint32_t shl1(uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x130, 0xF, 0xF, false); }
// value of lane ^ 1, ^ 2, ^ 4, ^ 8 (data-parallel-primitive moves inside a row of 16 lanes; every
// lane has a source, so no previous value is carried)
EST_DEV uint32_t xor1(uint32_t v) { return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, true); }
EST_DEV uint32_t xor2(uint32_t v) { return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, true); }
EST_DEV uint32_t xor8(uint32_t v) { return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x128, 0xF, 0xF, true); }
// the values of the two lanes l and l ^ 16 (l ^ 32): a that of the lower one, b that of the upper one, in both lanes
EST_DEV void pair16(uint32_t v, uint32_t &a, uint32_t &b) {
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    a = r[0];
    b = r[1];
}
EST_DEV void pair32(uint32_t v, uint32_t &a, uint32_t &b) {
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    a = r[0];
    b = r[1];
}
EST_DEV uint32_t xor4(uint32_t v) {
    const uint32_t down = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x124, 0xF, 0xF, true);  // from lane-4 (mod 16)
    const uint32_t up = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x12C, 0xF, 0xF, true);    // from lane+4 (mod 16)
    return lane_in_const<0xF0F0F0F0F0F0F0F0ull>() ? down : up;
}

// number of set bits of m below this lane's position (m must be the same in every lane)
EST_DEV uint32_t rank_below(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// v, hidden from the optimiser: what is computed from the result inside a loop is not moved out of the loop
// (where it would hold registers for the whole loop)
EST_DEV uint32_t opaque(uint32_t v) {
    asm volatile("" : "+v"(v));
    return v;
}

// the value of the first lane, in a scalar register (for a value the compiler already knows to be the same in every
// lane this costs nothing)
EST_DEV uint32_t uniform(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }

// The helpers below take operands that are the same in every lane and work on the scalar unit.  Their operands go
// through uniform() first: where the compiler keeps such a value in a vector register (it does when it cannot
// prove the value uniform), the scalar-register operand of the instruction text would otherwise not assemble.

// 1 when a >= b (a == b), else 0, for operands that are the same in every lane: a scalar compare whose result is an
// integer in a scalar register (several tests combined with & and | then cost one branch, and no lane masks)
EST_DEV uint32_t flag_ge(uint32_t a, uint32_t b) {
    uint32_t r;
    a = uniform(a); b = uniform(b);
    asm("s_cmp_ge_u32 %1, %2\n\ts_cselect_b32 %0, 1, 0" : "=s"(r) : "s"(a), "s"(b) : "scc");
    return r;
}
EST_DEV uint32_t flag_eq(uint32_t a, uint32_t b) {
    uint32_t r;
    a = uniform(a); b = uniform(b);
    asm("s_cmp_eq_u32 %1, %2\n\ts_cselect_b32 %0, 1, 0" : "=s"(r) : "s"(a), "s"(b) : "scc");
    return r;
}

// v with lane l replaced by x (l and x the same in every lane, l < 64): v_writelane_b32, reached through its
// compiler intrinsic (this compiler declares no builtin for it), so wait states and m0 are the compiler's business.
extern "C" __device__ uint32_t est_llvm_writelane(uint32_t x, uint32_t l, uint32_t v) __asm("llvm.amdgcn.writelane");
EST_DEV uint32_t set_lane(uint32_t v, uint32_t x, uint32_t l) { return est_llvm_writelane(x, l, v); }

// min(t + d, 2^32 - 1) for operands that are the same in every lane, on the scalar unit (the compiler's own
// saturating add exists on the vector unit only, with a trip there and back)
EST_DEV uint32_t sat_add_uniform(uint32_t t, uint32_t d) {
    uint32_t r;
    t = uniform(t); d = uniform(d);
    asm("s_add_u32 %0, %1, %2\n\ts_cselect_b32 %0, -1, %0" : "=s"(r) : "s"(t), "s"(d) : "scc");
    return r;
}

// The batch-by-batch recurrence of a batched queue, for as many batches as the window decides.  rdy: ready times of the
// window's queries, ascending (2^32-1 in the lanes beyond the window's w queries); F: the times the replicas are free
// again, ascending, 2^32-1 beyond the last one; Lrot: lane l holds the latency of a batch of l queries (lane 0 that of 64).
// A batch starts at T = max(earliest free time, ready time of query a), takes the queries ready by then, up to B, and
// completes at e = T + latency, at most 2^32-1; e goes into the sorted F in place of the earliest entry (with the right
// neighbour n of every lane: the middle one of F, n and e, which is n below the place of e, e at it and F above it).
// Every batch leaves e in lane K of gend and a bit at its first query in heads.
//
// What bounds it is the latency of one chain and, on a full device, the issue slots of both units: per batch 7 vector and 10
// scalar instructions, one branch.  A stage whose queue forms 2.5 queries per batch spends a third of its instructions
// here.  (With the first queries written lane by lane as well, the neighbour taken by a minimum and a maximum, the clamp and
// both ends of the window tested per batch: 9 and 15.)  Wait states: the DPP source F was written three instructions
// earlier, lane selects come from scalar instructions.

// The loop for a step in which no time can reach 2^32-1 (a < w and K < K_end on entry): it ends, with a < w, before a batch at
// whose start the whole window is ready or that may need a lane from K_end on.  One test per batch: the queries ready
// at its start are fewer than the window holds and than the first query plus the lanes left (every batch takes a query at least,
// so the lanes last as long as that holds); the second bound moves on with the batches formed.
EST_DEV void form_batches_inside(uint32_t rdy, uint32_t Lrot, uint32_t B, uint32_t w, uint32_t K_end, uint32_t &F, uint32_t &gend,
                                 uint64_t &heads, uint32_t &a, uint32_t &K) {
    uint32_t t, u, c, m, z, x = 0xFFFFFFFFu;
    B = uniform(B); w = uniform(w); K_end = uniform(K_end);
    asm volatile("s_mov_b32 %[m], m0\n\t"
                 "s_mov_b32 m0, %[K]\n\t"
                 "v_readfirstlane_b32 %[t], %[F]\n\t"
                 "v_readlane_b32 %[u], %[rdy], %[a]\n\t"
                 "v_mov_b32_dpp %[x], %[F] wave_shl:1 row_mask:0xf bank_mask:0xf\n\t"
                 "s_max_u32 %[t], %[t], %[u]\n\t"
                 "v_cmp_ge_u32 vcc, %[t], %[rdy]\n\t"
                 "s_bcnt1_i32_b64 %[c], vcc\n\t"
                 "s_branch 2f\n"
                 "1:\n\t"
                 "s_sub_u32 %[u], %[c], %[a]\n\t"
                 "s_min_u32 %[u], %[u], %[B]\n\t"
                 "v_readlane_b32 %[c], %[L], %[u]\n\t"
                 "s_bitset1_b64 %[heads], %[a]\n\t"
                 "s_add_u32 %[a], %[a], %[u]\n\t"
                 "s_add_u32 %[t], %[t], %[c]\n\t"
                 "v_med3_u32 %[F], %[F], %[x], %[t]\n\t"
                 "v_readlane_b32 %[u], %[rdy], %[a]\n\t"
                 "v_writelane_b32 %[gend], %[t], m0\n\t"
                 "s_add_u32 m0, m0, 1\n\t"
                 "v_readfirstlane_b32 %[t], %[F]\n\t"
                 "v_mov_b32_dpp %[x], %[F] wave_shl:1 row_mask:0xf bank_mask:0xf\n\t"
                 "s_max_u32 %[t], %[t], %[u]\n\t"
                 "v_cmp_ge_u32 vcc, %[t], %[rdy]\n\t"
                 "s_bcnt1_i32_b64 %[c], vcc\n\t"
                 "s_cmp_lt_u32 %[c], %[z]\n\t"
                 "s_cbranch_scc1 1b\n"
                 "2:\n\t"
                 "s_sub_u32 %[z], %[Ke], m0\n\t"
                 "s_add_u32 %[z], %[z], %[a]\n\t"
                 "s_min_u32 %[z], %[z], %[w]\n\t"
                 "s_cmp_lt_u32 %[c], %[z]\n\t"
                 "s_cbranch_scc1 1b\n\t"
                 "s_mov_b32 %[K], m0\n\t"
                 "s_mov_b32 m0, %[m]\n\t"
                 "s_nop 1"
                 : [F] "+v"(F), [gend] "+v"(gend), [heads] "+s"(heads), [a] "+s"(a), [K] "+s"(K), [t] "=&s"(t), [u] "=&s"(u),
                   [c] "=&s"(c), [x] "+v"(x), [m] "=&s"(m), [z] "=&s"(z)
                 : [rdy] "v"(rdy), [L] "v"(Lrot), [B] "s"(B), [w] "s"(w), [Ke] "s"(K_end)
                 : "vcc", "scc");
}

// The loop without conditions (a < w and K < K_end on entry): it ends when the window or the lanes below K_end are used up, or
// before a batch that is not full while wf or more queries are ready (more members may follow).  Batches that start at
// 2^32-1 may count lanes beyond the window: a can end up larger than w.
EST_DEV void form_batches(uint32_t rdy, uint32_t Lrot, uint32_t B, uint32_t w, uint32_t wf, uint32_t K_end, uint32_t &F, uint32_t &gend,
                          uint64_t &heads, uint32_t &a, uint32_t &K) {
    uint32_t t, u, c, m, x = 0xFFFFFFFFu;
    B = uniform(B); w = uniform(w); wf = uniform(wf); K_end = uniform(K_end);
    asm volatile("s_mov_b32 %[m], m0\n\t"
                 "s_mov_b32 m0, %[K]\n\t"
                 "s_nop 1\n"
                 "1:\n\t"
                 "v_readfirstlane_b32 %[t], %[F]\n\t"
                 "v_readlane_b32 %[u], %[rdy], %[a]\n\t"
                 "v_mov_b32_dpp %[x], %[F] wave_shl:1 row_mask:0xf bank_mask:0xf\n\t"
                 "s_max_u32 %[t], %[t], %[u]\n\t"
                 "v_cmp_ge_u32 vcc, %[t], %[rdy]\n\t"
                 "s_bcnt1_i32_b64 %[c], vcc\n\t"
                 "s_sub_u32 %[u], %[c], %[a]\n\t"
                 "s_min_u32 %[u], %[u], %[B]\n\t"
                 "s_cmp_ge_u32 %[c], %[wf]\n\t"
                 "s_cbranch_scc1 3f\n"
                 "2:\n\t"
                 "v_readlane_b32 %[c], %[L], %[u]\n\t"
                 "s_bitset1_b64 %[heads], %[a]\n\t"
                 "s_add_u32 %[t], %[t], %[c]\n\t"
                 "s_cselect_b32 %[t], -1, %[t]\n\t"
                 "s_add_u32 %[a], %[a], %[u]\n\t"
                 "v_med3_u32 %[F], %[F], %[x], %[t]\n\t"
                 "v_writelane_b32 %[gend], %[t], m0\n\t"
                 "s_add_u32 m0, m0, 1\n\t"
                 "s_cmp_lt_u32 %[a], %[w]\n\t"
                 "s_cbranch_scc0 4f\n\t"
                 "s_cmp_lt_u32 m0, %[Ke]\n\t"
                 "s_cbranch_scc1 1b\n\t"
                 "s_branch 4f\n"
                 "3:\n\t"
                 "s_cmp_eq_u32 %[u], %[B]\n\t"
                 "s_cbranch_scc1 2b\n"
                 "4:\n\t"
                 "s_mov_b32 %[K], m0\n\t"
                 "s_mov_b32 m0, %[m]\n\t"
                 "s_nop 1"
                 : [F] "+v"(F), [gend] "+v"(gend), [heads] "+s"(heads), [a] "+s"(a), [K] "+s"(K), [t] "=&s"(t), [u] "=&s"(u),
                   [c] "=&s"(c), [x] "+v"(x), [m] "=&s"(m)
                 : [rdy] "v"(rdy), [L] "v"(Lrot), [B] "s"(B), [w] "s"(w), [wf] "s"(wf), [Ke] "s"(K_end)
                 : "vcc", "scc");
}

EST_DEV uint32_t min_u32(uint32_t v) {
#pragma unroll
    for (uint32_t d = 32; d >= 1; d >>= 1) {
        uint32_t o = shfl(v, lane() ^ d);
        v = o < v ? o : v;
    }
    return uniform(v);
}
EST_DEV uint32_t max_u32(uint32_t v) { return ~min_u32(~v); }

// (moves inside the rows of 16 lanes, then one scalar read per row: no trip through the LDS crossbar)
EST_DEV uint32_t sum_u32(uint32_t v) {
    v += xor1(v);
    v += xor2(v);
    v += (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x124, 0xF, 0xF, true);  // + lane-4 (mod 16)
    v += xor8(v);
    return bcast(v, 0) + bcast(v, 16) + bcast(v, 32) + bcast(v, 48);
}

// exclusive prefix sum over lanes: shifts by 1, 2, 4, 8 inside the rows of 16 lanes (zeros come in at the row's
// start), then the totals of the rows before a lane's own are added from scalar registers.  (Carrying the row
// totals across with row broadcasts instead measured 5 % slower on the whole sweep.)
EST_DEV uint32_t prefix_excl_u32(uint32_t v) {
    uint32_t x = v;
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, true);  // row_shr:1
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, true);  // row_shr:2
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, true);  // row_shr:4
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, true);  // row_shr:8
    const uint32_t t0 = bcast(x, 15), t1 = t0 + bcast(x, 31), t2 = t1 + bcast(x, 47);
    const uint32_t row = lane() >> 4;
    const uint32_t before = row == 0u ? 0u : row == 1u ? t0 : row == 2u ? t1 : t2;
    return x + before - v;
}

// Make earlier memory writes (global and LDS) of any lane visible to later reads of any lane
// of this wavefront.
EST_DEV void sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// The same for LDS only: earlier LDS writes of any lane are visible to later LDS reads of any lane of
// this wavefront.  Does not wait for outstanding global loads or stores.
EST_DEV void sync_lds() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// A word that another wavefront of the workgroup may write or read (the same address and value in every lane).  Whoever stores such
// a word after a sync() shows with it what it wrote before: a wavefront issues its memory operations in the order of the code,
// LDS answers them in that order, and one compute unit's loads and stores of global memory reach its cache in it.  What is used or
// overwritten only where the loaded word allows it comes after the load by itself; where two such words have to be read in a
// certain order, the second one's index goes through after().  (Acquires at workgroup scope instead also wait for the wavefront's own
// stores under way, 1 % on calls with few candidates; a barrier for all of the compiler's memory operations makes it load the plan's fields
// again, 1 to 2 % on shared runs.)
EST_DEV uint32_t after(uint32_t v, uint32_t first) {  // v, known only once first is
    asm volatile("" : "+v"(v) : "v"(first));
    return v;
}
EST_DEV uint32_t load_shared(const uint32_t *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); }
EST_DEV void store_shared(uint32_t *p, uint32_t v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); }

EST_DEV void lds_add(uint32_t *p, uint32_t v) { atomicAdd(p, v); }
// (by one lane) the word before: compare and swap, fetch and add
EST_DEV uint32_t lds_cas(uint32_t *p, uint32_t expect, uint32_t v) { return atomicCAS(p, expect, v); }
EST_DEV uint32_t lds_fetch_add(uint32_t *p, uint32_t v) { return atomicAdd(p, v); }
EST_DEV void atomic_or_u64(uint64_t *p, uint64_t v) { atomicOr((unsigned long long *)p, (unsigned long long)v); }
EST_DEV void atomic_or_u32(uint32_t *p, uint32_t v) { atomicOr(p, v); }
EST_DEV void atomic_add_u32(uint32_t *p, uint32_t v) { atomicAdd(p, v); }
EST_DEV void atomic_max_u32(uint32_t *p, uint32_t v) { atomicMax(p, v); }
EST_DEV uint32_t fetch_add_u32(uint32_t *p, uint32_t v) { return atomicAdd(p, v); }
EST_DEV uint64_t ticks() { return wall_clock64(); }
EST_DEV void atomic_add_u64(uint64_t *p, uint64_t v) { atomicAdd((unsigned long long *)p, (unsigned long long)v); }

}  // namespace wv
