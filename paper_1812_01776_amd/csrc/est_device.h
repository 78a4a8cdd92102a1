// Device code of the batched Estimator: the 64-lane wavefronts of a workgroup simulate a few candidate
// configurations end to end.  Written against the wv:: primitives only, so that the same text
// also compiles for a lock-step CPU emulation used by the host-side checks of the kernel logic.
//
// The simulated system is the centralized batched queue of arXiv 1812.01776 (Section 3, serving
// system requirements; Section 2.1, maximum batch size; Section 4.2, event order).  Because
// queues are unbounded and the DAG is feed-forward, a stage depends only on its own input
// stream ordered by (ready time, query index); the global event order of Section 4.2 is
// reproduced by running every stage over its ordered stream:
//
//   SCAN   one stage.  Walk the stage's input stream; a batch starts at T = max(earliest replica
//          free time, ready time of the first waiting query), takes every waiting query with
//          ready <= T up to the maximum batch size, and completes at T + L(actual size)
//          (Section 4.2: latency from the profile for a batch of the given size; Section 2.1: the
//          whole batch returns together).  Completed batches are emitted to the output stream in
//          (completion time, query index) order.
//   MERGE  builds a stage's input stream from the output streams of the query's nearest visited
//          ancestors: a query that skips a stage passes through it in zero time (Section 4.1,
//          scale factor / conditional control flow) and a stage with several parents is ready at
//          the maximum of their completions.
//   LAT    a MERGE into the virtual sink: latency = completion - arrival (Section 4.2), and the
//          SLO miss count (Section 2: latencies must be below the constraint).
//
// Streams are per-candidate rings of 64-bit keys (time << 32 | query index) in global memory,
// so that comparing keys compares (time, query index).  An operation runs until it needs input that is not
// there yet or output space that is not free yet, and tells its neighbours on the way how far it is; who runs which
// operation when is the driver's business (below).
#pragma once
#include "est_types.h"

namespace estdev {

EST_DEV uint32_t umin(uint32_t a, uint32_t b) { return a < b ? a : b; }
EST_DEV uint32_t umax(uint32_t a, uint32_t b) { return a > b ? a : b; }
EST_DEV uint32_t popc64(uint64_t x) { return (uint32_t)__builtin_popcountll(x); }
EST_DEV uint32_t ctz64(uint64_t x) { return (uint32_t)__builtin_ctzll(x); }
EST_DEV uint64_t lanes_below(uint32_t l) { return l >= 64 ? ~0ull : ((1ull << l) - 1ull); }

// Saturating clock: every computed time is min(true time, horizon = 2^32 - 1).
EST_DEV uint32_t sat_add(uint32_t t, uint32_t d) {
    uint32_t e = t + d;
    return e < t ? 0xFFFFFFFFu : e;
}

// LDS of one wavefront while it merges, for a plan whose widest merge has k sources: see merge_run.
// Size: EST_LDS_MERGE_BYTES(k).

struct Ctx {
    const EstSimArgs *a;
    const EstPlan *P;
    uint32_t *st;
    uint64_t *rings;
    uint32_t *rep;
    uint32_t *slots;
    uint8_t *tab;  // time tables of the merges that join several streams
    uint32_t *lat;
    const EstStageCfg *cfg;
    uint64_t *lds;
    uint32_t t;  // candidate index
    // streams taken from another candidate's captured run instead of this one's scratch (bit per ring)
    uint64_t memo_rings;
    const uint64_t *cap_rings;
};

// Diagnostics record of candidate t and stage s: EST_DBG_WORDS words (unused, ticks in the stage's scan, steps,
// queries in steps, of which: batch by batch with four or more queries per batch, unused, one-per-batch, batch by batch
// otherwise; then ticks spent in steps of the kinds: batch by batch with four or more, unused, one-per-batch, batch by
// batch otherwise, backlog or horizon, unused; then ticks in the batch-by-batch recurrence and the batches it formed).
// The record of stage EST_MAX_STAGES-1 holds what belongs to no stage: ticks in merges, in the sink, in the
// selection, merge rounds, merge output elements, merge calls, scan calls.
EST_DEV uint64_t *est_dbg_rec(const EstSimArgs *a, uint32_t t, uint32_t s) {
    return a->dbg_ticks + a->n_cfg + ((uint64_t)t * EST_MAX_STAGES + s) * EST_DBG_WORDS;
}

// Ring cursors and the other state words of a candidate, in LDS, are written by the operation that owns them and read
// by its neighbours, which may run in another wavefront of the workgroup at the same time: they are read and written
// through these (the value is the same in every lane).
EST_DEV uint32_t ld_st(const uint32_t *p) { return wv::load_shared(p); }
EST_DEV void st_st(uint32_t *p, uint32_t v) { wv::store_shared(p, v); }

struct View {
    const uint64_t *base;
    uint32_t mask, wr, fin;
};

template <bool MEMO>
EST_DEV View view_of(const Ctx &c, int32_t ring) {
    View v;
    if (ring == EST_SRC_TRACE) {
        v.base = c.a->trace_keys;
        v.mask = 0xFFFFFFFFu;
        v.wr = c.a->n;
        v.fin = 1;
    } else if (MEMO && ((c.memo_rings >> ring) & 1ull)) {  // a whole stream somebody else produced; cursors were preset
        const EstRing &R = c.a->cap_plan->rings[ring];
        v.base = c.cap_rings + R.off;
        v.mask = R.cap_mask;
        v.wr = ld_st(&c.st[c.P->wr_off + ring]);
        v.fin = 1;
    } else {
        const EstRing &R = c.P->rings[ring];
        v.base = c.rings + R.off;
        v.mask = R.cap_mask;
        const uint32_t f = ld_st(&c.st[c.P->fin_off + ring]);  // (before the cursor: a stream seen as ended is seen whole)
        v.fin = f != 0u;
        v.wr = ld_st(&c.st[wv::after(c.P->wr_off + ring, f)]);
    }
    return v;
}

// The same with the scalars marked as identical in every lane (they are: one address, one value), which
// keeps everything computed from them in scalar registers.
template <bool MEMO>
EST_DEV View uniform_view_of(const Ctx &c, int32_t ring) {
    View v = view_of<MEMO>(c, ring);
    v.mask = wv::uniform(v.mask);
    v.wr = wv::uniform(v.wr);
    v.fin = wv::uniform(v.fin);
    return v;
}

// Free elements of a ring: capacity minus the distance to its slowest consumer.
EST_DEV uint32_t ring_space(const Ctx &c, int32_t ring, uint32_t wr) {
    const EstRing &R = c.P->rings[ring];
    uint32_t used = 0;
    for (uint32_t i = 0; i < R.n_cons; ++i) used = umax(used, wr - ld_st(&c.st[c.P->rd_off + R.cons_edge[i]]));
    EST_CHECK(used <= R.cap_mask + 1u);
    return R.cap_mask + 1u - used;
}

// Lanes that keep the smaller value in the compare-exchange step (k, j) of a bitonic network:
// those whose bit j and bit k are both clear or both set.
constexpr uint64_t keep_min_mask(uint32_t k, uint32_t j) {
    uint64_t m = 0;
    for (uint32_t l = 0; l < 64; ++l)
        if (((l & j) == 0) == ((l & k) == 0)) m |= 1ull << l;
    return m;
}

// Ascending bitonic sort of the values of lanes 0 .. width-1 (width a power of two, the same in
// every lane; lanes beyond it take part but their result is not used).
template <uint32_t K, uint32_t J>
EST_DEV uint32_t cmpx(uint32_t v, uint32_t o) {
    const uint32_t lo = umin(v, o), hi = umax(v, o);
    return wv::lane_in_const<keep_min_mask(K, J)>() ? lo : hi;
}
template <uint32_t K, uint32_t J>
EST_DEV uint32_t cmpx_rows(uint32_t v) {  // J = 16 or 32
    uint32_t a, b;
    if (J == 16) wv::pair16(v, a, b); else wv::pair32(v, a, b);
    return cmpx<K, J>(a, b);
}
EST_DEV uint32_t sort_lanes(uint32_t v, uint32_t width) {
    v = cmpx<2, 1>(v, wv::xor1(v));
    if (width <= 2) return v;
    v = cmpx<4, 2>(v, wv::xor2(v));
    v = cmpx<4, 1>(v, wv::xor1(v));
    if (width <= 4) return v;
    v = cmpx<8, 4>(v, wv::xor4(v));
    v = cmpx<8, 2>(v, wv::xor2(v));
    v = cmpx<8, 1>(v, wv::xor1(v));
    if (width <= 8) return v;
    v = cmpx<16, 8>(v, wv::xor8(v));
    v = cmpx<16, 4>(v, wv::xor4(v));
    v = cmpx<16, 2>(v, wv::xor2(v));
    v = cmpx<16, 1>(v, wv::xor1(v));
    if (width <= 16) return v;
    v = cmpx_rows<32, 16>(v);
    v = cmpx<32, 8>(v, wv::xor8(v));
    v = cmpx<32, 4>(v, wv::xor4(v));
    v = cmpx<32, 2>(v, wv::xor2(v));
    v = cmpx<32, 1>(v, wv::xor1(v));
    if (width <= 32) return v;
    v = cmpx_rows<64, 32>(v);
    v = cmpx_rows<64, 16>(v);
    v = cmpx<64, 8>(v, wv::xor8(v));
    v = cmpx<64, 4>(v, wv::xor4(v));
    v = cmpx<64, 2>(v, wv::xor2(v));
    v = cmpx<64, 1>(v, wv::xor1(v));
    return v;
}

// Ascending bitonic sort of one 64-bit key per lane over all 64 lanes.
template <uint32_t K, uint32_t J>
EST_DEV uint64_t cmpx64(uint64_t v, uint32_t ohi, uint32_t olo) {
    const uint64_t o = ((uint64_t)ohi << 32) | olo;
    return ((o < v) == wv::lane_in_const<keep_min_mask(K, J)>()) ? o : v;
}
template <uint32_t K, uint32_t J>
EST_DEV uint64_t cmpx64_rows(uint64_t v) {  // J = 16 or 32
    uint32_t ahi, alo, bhi, blo;
    if (J == 16) { wv::pair16((uint32_t)(v >> 32), ahi, bhi); wv::pair16((uint32_t)v, alo, blo); }
    else { wv::pair32((uint32_t)(v >> 32), ahi, bhi); wv::pair32((uint32_t)v, alo, blo); }
    return cmpx64<K, J>(((uint64_t)ahi << 32) | alo, bhi, blo);
}
template <uint32_t K>
EST_DEV uint64_t sort_merge64(uint64_t v) {  // the compare-exchange steps (K, K/2), ..., (K, 1)
    if (K >= 64) v = cmpx64_rows<K, 32>(v);
    if (K >= 32) v = cmpx64_rows<K, 16>(v);
    if (K >= 16) v = cmpx64<K, 8>(v, wv::xor8((uint32_t)(v >> 32)), wv::xor8((uint32_t)v));
    if (K >= 8) v = cmpx64<K, 4>(v, wv::xor4((uint32_t)(v >> 32)), wv::xor4((uint32_t)v));
    if (K >= 4) v = cmpx64<K, 2>(v, wv::xor2((uint32_t)(v >> 32)), wv::xor2((uint32_t)v));
    return cmpx64<K, 1>(v, wv::xor1((uint32_t)(v >> 32)), wv::xor1((uint32_t)v));
}
EST_DEV uint64_t sort_lanes64(uint64_t v) {
    v = sort_merge64<2>(v);
    v = sort_merge64<4>(v);
    v = sort_merge64<8>(v);
    v = sort_merge64<16>(v);
    v = sort_merge64<32>(v);
    return sort_merge64<64>(v);
}

// ------------------------------------------------------------------------------------------ SCAN
//
// Per-wavefront working set of a scan.  In registers, one entry per lane:
//   F       the time every replica is free again, ascending (2^32-1 beyond the last replica); which replica is which
//           does not matter, so a free time is all there is to a replica;
//   gend, ginfo   the pending batches -- dispatched, not yet passed on -- ascending by completion time: lane l < nG
//           holds the completion time, and the number of members << 8 | the member slot.  The lanes from nG on hold
//           the numbers of the free slots.
// In LDS:
//   in-ring   128 or 256 keys (EstPlan::scan_ring): the next elements of the stage's input stream, refilled from the
//             source ring in chunks (and filtered on the way, when only some elements of the source visit the stage);
//   slots     EstPlan::slot_words words cut into slots of B (the candidate's maximum batch size at the stage): the
//             query indices of the members of the pending batches.
// A step looks at a window of up to 64 input elements.  First whatever is pending and certain to finish before anything
// dispatched from here on leaves: everything that completes before lim = T0 + Lmin, T0 the start of the next batch, Lmin
// the shortest latency of the stage.  Then the next batches are formed -- all of them become pending; only steps in
// which every query is a batch of its own write their results directly.

// Query indices of the lanes in M (a prefix), which are in consecutive groups gid, each group's sorted ascending.
// Indices that span less than 2^26 around the first one are sorted as 32-bit (group, index) pairs.
EST_DEV uint32_t sort_groups(uint32_t gid, uint32_t q, uint64_t M) {
    const bool valid = wv::lane_in(M);
    const uint32_t base = wv::uniform(q) - (1u << 25), d = q - base;
    if ((M & wv::ballot(d >= (1u << 26))) == 0) {
        const uint32_t k = sort_lanes(valid ? ((gid << 26) | d) : 0xFFFFFFFFu, 64);
        return (k & ((1u << 26) - 1u)) + base;
    }
    return (uint32_t)sort_lanes64(valid ? (((uint64_t)gid << 32) | q) : ~0ull);
}

// The smallest power of two that is at least n (n from 1 to 64), at least 2
EST_DEV uint32_t pow2_at_least(uint32_t n) { return n <= 2u ? 2u : 1u << (32u - (uint32_t)__builtin_clz(n - 1u)); }

// Pending batches k0 .. k1-1, which all complete at the same time mv and have more than 64 members in all, written to
// out[wr ...] merged by query index: every batch is sorted in its slot, then every member finds its place among all of
// them by binary searches.
EST_DEV void emit_big_tie(uint32_t B, uint32_t *lslots, uint32_t k0, uint32_t k1, uint32_t mv, uint32_t ginfo, uint64_t *out,
                          uint32_t omask, uint32_t wr) {
    const uint32_t ln = wv::lane();
    for (uint32_t k = k0; k < k1; ++k) {
        const uint32_t gi = wv::bcast(ginfo, k), cr = gi >> 8, at = (gi & 0xFFu) * B + ln;
        const uint32_t x = ln < cr ? lslots[at] : 0xFFFFFFFFu;  // (query indices stay below 2^31)
        const uint32_t xs = sort_lanes(x, pow2_at_least(cr));
        wv::sync_lds();
        if (ln < cr) lslots[at] = xs;
    }
    wv::sync_lds();
    const uint64_t tkey = (uint64_t)mv << 32;
    for (uint32_t k = k0; k < k1; ++k) {
        const uint32_t gi = wv::bcast(ginfo, k), cr = gi >> 8;
        const uint32_t x = ln < cr ? lslots[(gi & 0xFFu) * B + ln] : 0u;
        uint32_t rank = ln;
        for (uint32_t k2 = k0; k2 < k1; ++k2) {
            const uint32_t g2 = wv::bcast(ginfo, k2);
            if (k2 == k || ln >= cr) continue;
            const uint32_t *s2 = lslots + (g2 & 0xFFu) * B;
            uint32_t lo = 0, hi = g2 >> 8;
            while (lo < hi) {
                const uint32_t mid = (lo + hi) >> 1;
                if (s2[mid] < x) lo = mid + 1; else hi = mid;
            }
            rank += lo;
        }
        if (ln < cr) out[(wr + rank) & omask] = tkey | x;
    }
}

// Pass on, in (completion time, query index) order, the members of the first nE pending batches (at least one; no
// batch that stays completes at the same time as one of them), as far as the output ring has room; returns the number
// of batches passed on.  Output positions are handled 64 at a time: a position finds its batch by counting the set bits
// of a mask of the batches' first positions, and members that leave at the same time are put in query order only where
// they are not in it already.  (Times clamped at the horizon need no order: everything downstream of a clamped time is
// clamped too.)
EST_DEV uint32_t emit_pending(uint32_t B, uint32_t *lslots, uint32_t nE, uint32_t gend, uint32_t ginfo, uint64_t *out,
                              uint32_t omask, uint32_t &wr, uint32_t &space) {
    const uint32_t ln = wv::lane();
    const uint32_t cnt = ln < nE ? ginfo >> 8 : 0u;
    const uint32_t off = wv::prefix_excl_u32(cnt);
    uint32_t total = wv::bcast(off, nE - 1u) + wv::bcast(cnt, nE - 1u);
    const uint64_t tied = lanes_below(nE) & ~1ull & wv::ballot(gend == wv::shr1(gend)) & wv::ballot(gend != 0xFFFFFFFFu);
    if (total > space) {
        nE = popc64(lanes_below(nE) & wv::ballot(off + cnt <= space));  // (a prefix; batches that tie leave together)
        while (nE > 0 && ((tied >> nE) & 1ull)) --nE;
        if (nE == 0) return 0;
        total = wv::bcast(off, nE - 1u) + wv::bcast(cnt, nE - 1u);
    }
    const uint32_t pk = (ginfo & 0xFFu) | (off << 8);
    for (uint32_t k0 = 0, o0 = 0; k0 < nE;) {
        uint32_t k1 = nE, o1 = total;
        if (total - o0 > 64u) {
            k1 = popc64(lanes_below(nE) & wv::ballot(off + cnt <= o0 + 64u));
            while (k1 > k0 && ((tied >> k1) & 1ull)) --k1;  // (k1 < nE)
            if (k1 == k0) {
                for (k1 = k0 + 1u; k1 < nE && ((tied >> k1) & 1ull);) ++k1;
                emit_big_tie(B, lslots, k0, k1, wv::bcast(gend, k0), ginfo, out, omask, wr + o0);
                o0 = k1 < nE ? wv::bcast(off, k1) : total;
                k0 = k1;
                continue;
            }
            o1 = wv::bcast(off, k1);
        }
        const uint32_t n = o1 - o0;
        const uint64_t KM = lanes_below(k1) & ~lanes_below(k0);
        const bool mine = wv::lane_in(KM);
        const uint32_t pos = off - o0;  // first position of my batch in this chunk
        const uint64_t H = wv::ballot(wv::push(1u, mine ? pos : 0u) != 0u);
        const uint32_t kl = k0 + wv::rank_below(H >> 1);  // my batch (bit 0 of H is set)
        const uint32_t e = wv::shfl(gend, kl), y = wv::shfl(pk, kl);
        uint32_t q = ln < n ? lslots[(y & 0xFFu) * B + (o0 + ln - (y >> 8))] : 0u;
        const uint32_t qp = wv::shr1(q);
        uint64_t Hg = H;  // first positions of the groups that leave at the same time
        if (tied & KM) {
            const uint32_t ep = wv::shr1(e);
            Hg = wv::ballot(e != ep) | 1ull;
        }
        if (lanes_below(n) & ~Hg & wv::ballot(qp > q)) q = sort_groups(wv::rank_below(Hg >> 1), q, lanes_below(n));
        if (ln < n) out[(wr + o0 + ln) & omask] = ((uint64_t)e << 32) | q;
        k0 = k1;
        o0 = o1;
    }
    wr += total;
    space -= total;
    return nE;
}

enum { PUBLISH = 256 };  // elements a scan writes before it tells its neighbours

// Returns whether the operation has finished for good.
template <bool DIAG, bool MEMO>
EST_DEV bool scan_run(const Ctx &c, const EstOp &op) {
    const uint32_t ln = wv::lane();
    const EstPlan &P = *c.P;
    const uint32_t s = op.stage;
    const EstStageCfg sc = c.cfg[s];
    // (values read from memory are the same in every lane; saying so keeps what is computed from them in
    // scalar registers, off the vector unit)
    const uint32_t B = wv::uniform(sc.batch), R = wv::uniform(sc.replicas);
    EST_CHECK(B >= 1 && B <= op.b_max && R >= 1 && R <= op.r_max);
    const uint32_t *Ltab = c.a->lat_us + ((uint64_t)s * c.a->dag->H + sc.hw) * c.a->dag->Bmax;
    const uint32_t Lmine = ln < B ? Ltab[ln] : 0u;  // lane l holds L(l+1)
    const uint32_t Lrot = wv::shfl(Lmine, ln - 1u);  // lane l holds L(l), lane 0 L(64)
    const uint32_t L1 = wv::bcast(Lmine, 0);
    const uint32_t Lmin = wv::min_u32(ln < B ? Lmine : 0xFFFFFFFFu);
    const uint32_t Lmax = wv::max_u32(ln < B ? Lmine : 0u);
    // window and free times below this: 64 batches one after the other stay below the horizon
    const uint32_t t_inside = Lmax < (1u << 26) ? 0xFFFFFFFFu - 64u * Lmax : 0u;
    const bool mono = Lmin == L1;  // no batch is faster than a single query
    const uint32_t SW = wv::uniform(P.slot_words);
    const uint32_t nslots = umin(64u, SW / B);  // (at least R)
    EST_CHECK(nslots >= R);
    uint32_t *g_free = c.rep + op.rep_off, *g_end = g_free + 64, *g_info = g_free + 128, *g_n = g_free + 192;  // g_n: pending batches, staged keys
    uint32_t *g_slots = c.slots + op.slot_off;
    uint64_t *lkey = c.lds;
    const uint32_t RING = wv::uniform(P.scan_ring), rmask = RING - 1u;
    uint32_t *lslots = (uint32_t *)(c.lds + RING);
    const uint8_t *acc = c.a->acc + (uint64_t)op.acc_idx * c.a->acc_stride;
    const uint32_t filtered = wv::uniform(op.filtered);
    const uint32_t inv_b = (65536u + B - 1u) / B, inv_r = (65536u + R - 1u) / R;

    const bool isrep = ln < R;
    uint32_t F = isrep ? g_free[ln] : 0xFFFFFFFFu;
    uint32_t gend = g_end[ln], ginfo = g_info[ln];
    uint32_t nG = wv::uniform(g_n[0]);
    uint32_t lhead = 0, ltail = wv::uniform(g_n[1]);  // in-ring: consumed / filled
    uint64_t *g_keys = (uint64_t *)(g_slots + SW);
    if (nG)  // members still pending: back into LDS
        for (uint32_t i = ln; i < SW; i += 64) lslots[i] = g_slots[i];
    for (uint32_t i = ln; i < ltail; i += 64) lkey[i] = g_keys[i];  // and what had been staged
    wv::sync_lds();

    View in = view_of<MEMO>(c, op.src_ring[0]);
    in.mask = wv::uniform(in.mask);
    in.wr = wv::uniform(in.wr);
    in.fin = wv::uniform(in.fin);
    uint32_t rraw = wv::uniform(c.st[P.rd_off + op.src_edge[0]]);  // next source position to read
    const EstRing &OR = P.rings[op.out_ring];
    uint64_t *out = c.rings + OR.off;
    const uint32_t omask = wv::uniform(OR.cap_mask);
    uint32_t wr = wv::uniform(c.st[P.wr_off + op.out_ring]);
    uint32_t space = wv::uniform(ring_space(c, op.out_ring, wr));
    bool finished = false;
    uint32_t wr_pub = wr;  // what the readers have been told
    EST_CHK_ORDER_INIT();  // (host-side emulation only: everything written from here on is verified to be in order, step by step)
    uint32_t sat_skip = 0;     // steps to go before the backlog front end is tried again
    uint32_t single_skip = 0;  // the same for one query per batch
    uint32_t cf_skip = 0;      // and for its closed forms
    uint64_t d_blkl = 0, d_blkk = 0;  // diagnostics: ticks in the batch-by-batch recurrence, batches it formed
    uint64_t d_tk[6] = {0, 0, 0, 0, 0, 0}, tk0 = 0;  // diagnostics: ticks by the kind of step that ended the iteration
    uint32_t d_b1 = 0, d_b1e = 0, d_sat = 0, d_sate = 0, d_hz = 0, d_blk = 0, d_blke = 0, d_grp = 0, d_grpe = 0;  // diagnostics

    for (;;) {
        uint32_t staged = ltail - lhead;
        if (staged < 64 && rraw != in.wr) {
            // refill: as much of the source as the ring has room for beside what is staged (up to three loads of 64
            // elements, issued together)
            const uint32_t left = umin(umin(in.wr - rraw, RING - staged), 192u);
            const uint32_t w0 = umin(left, 64u), w1 = left > 64 ? umin(left - 64, 64u) : 0u,
                           w2 = left > 128 ? umin(left - 128, 64u) : 0u;
            const uint64_t k0 = ln < w0 ? in.base[(rraw + ln) & in.mask] : 0ull;
            const uint64_t k1 = ln < w1 ? in.base[(rraw + 64 + ln) & in.mask] : 0ull;
            const uint64_t k2 = ln < w2 ? in.base[(rraw + 128 + ln) & in.mask] : 0ull;
            // (lane masks are combined as scalars: one vector compare per term)
            uint64_t A0 = lanes_below(w0), A1 = lanes_below(w1), A2 = lanes_below(w2);
            bool a0 = ln < w0, a1 = ln < w1, a2 = ln < w2;
            if (filtered) {  // (lanes beyond a window hold key 0: query 0 exists)
                const bool f0 = (acc[(uint32_t)k0] & 1u) != 0u, f1 = (acc[(uint32_t)k1] & 1u) != 0u, f2 = (acc[(uint32_t)k2] & 1u) != 0u;
                A0 &= wv::ballot(f0); A1 &= wv::ballot(f1); A2 &= wv::ballot(f2);
                a0 = a0 && f0; a1 = a1 && f1; a2 = a2 && f2;
            }
            const uint32_t i0 = (ltail + wv::rank_below(A0)) & rmask;
            ltail += popc64(A0);
            const uint32_t i1 = (ltail + wv::rank_below(A1)) & rmask;
            ltail += popc64(A1);
            const uint32_t i2 = (ltail + wv::rank_below(A2)) & rmask;
            ltail += popc64(A2);
            if (a0) lkey[i0] = k0;
            if (a1) lkey[i1] = k1;
            if (a2) lkey[i2] = k2;
            rraw += w0 + w1 + w2;
            EST_CHECK(ltail - lhead <= RING);
            // What has been written so far is in place (the loads just waited for were issued after it): tell the readers,
            // and the producer what has been read, so that both can run beside this operation.
            if (wr - wr_pub >= PUBLISH) {
                wv::sync();
                if (ln == 0) {
                    st_st(&c.st[P.wr_off + op.out_ring], wr);
                    st_st(&c.st[P.rd_off + op.src_edge[0]], rraw);
                }
                wr_pub = wr;
            }
            wv::sync_lds();
            continue;
        }
        if (staged < 64 && !in.fin) {
            // the producer may have gone on meanwhile
            const uint32_t fin2 = wv::uniform(ld_st(&c.st[P.fin_off + op.src_ring[0]]));
            const uint32_t wr2 = wv::uniform(ld_st(&c.st[wv::after(P.wr_off + op.src_ring[0], fin2)]));
            if (fin2 || wr2 != in.wr) {
                in.fin = fin2 ? 1u : 0u;
                in.wr = wr2;
                wv::sync();
                continue;
            }
        }
        if (staged == 0 && !in.fin) break;
        // a step may pass on a window of 64 queries: with less room than that in the output ring, let the reader run
        // first rather than squeeze batches through
        if (staged != 0 && space < 64u) {
            space = wv::uniform(ring_space(c, op.out_ring, wr));  // the reader may have gone on meanwhile
            if (space < 64u) break;
        }
        if (DIAG) tk0 = wv::ticks();
        const uint32_t w = umin(staged, 64u);
        const uint64_t key = ln < w ? lkey[(lhead + ln) & rmask] : ~0ull;
        const uint32_t rdy = (uint32_t)(key >> 32);
        const uint32_t q = (uint32_t)key;
        EST_CHECK(ln == 0 || ln >= w || rdy == 0xFFFFFFFFu || key > lkey[(lhead + ln - 1) & rmask]);  // input is ordered
        const uint32_t f0 = wv::uniform(F), r0 = wv::uniform(rdy);
        const uint32_t T0 = umax(f0, r0);  // the next batch starts here (the horizon when the input has ended)
        // ---- what nothing dispatched from here on can overtake leaves
        {
            const uint32_t lim = wv::sat_add_uniform(T0, Lmin);
            const uint64_t late = ~lanes_below(nG) | (T0 == 0xFFFFFFFFu ? 0ull : wv::ballot(gend >= lim));
            const uint32_t nE = late ? ctz64(late) : 64u;
            if (nE > 0) {
                const uint32_t d = emit_pending(B, lslots, nE, gend, ginfo, out, omask, wr, space);
                EST_CHK_ORDER(4);
                if (d) {
                    nG -= d;
                    // the batches passed on go to the end of the lanes: their slots are free
                    const uint32_t src = ln + d < nslots ? ln + d : ln + d - nslots;
                    gend = wv::shfl(gend, src);
                    ginfo = wv::shfl(ginfo, src);
                    wv::sync_lds();
                }
                if (d < nE) break;  // wait for the consumer
            }
        }
        if (staged == 0) {  // input exhausted for good, and nothing is in flight any more
            finished = true;
            break;
        }
        if (T0 == 0xFFFFFFFFu) {
            // Every replica is busy up to the horizon, or the input is clamped there: whatever is still queued starts and
            // ends at the horizon, where order no longer matters.
            const uint32_t m = umin(w, space);
            if (m == 0) break;
            if (ln < m) out[(wr + ln) & omask] = 0xFFFFFFFF00000000ull | q;
            wr += m;
            space -= m;
            lhead += m;
            d_hz += m;
            if (DIAG) d_tk[4] += wv::ticks() - tk0;
            continue;
        }
        const uint32_t last = wv::flag_ge(64u, staged) & wv::flag_eq(rraw, in.wr) & in.fin;  // the window holds the end of the input
        if (nG == 0 && L1 > 0 && mono) {
            if (space < 64u) continue;
            if (cf_skip == 0 && w >= 32 && R <= 31) {
                // Closed forms for a whole window of queries that are each a batch of their own, checked with one
                // vote and left to the steps below when they do not hold.  Query i runs on the replica that served
                // query i-R (the table's entry i for the first R).
                //   Nobody waits: every query finds that replica free again by the time it is ready, ready[i] >=
                //   ready[i-R] + L(1) (for B > 1 no two queries may become ready together): end[i] = ready[i] + L(1).
                //   Everybody waits (B = 1): ready[i] <= end[i-R], so end[i] = free[i mod R] + (i div R + 1) L(1), as
                //   long as these ascend strictly (they do while the free times lie within one L(1) of each other;
                //   equal completion times would have to be put in query order).
                const uint64_t WM = lanes_below(w);
                const uint32_t back = ln >= R && ln < w ? (uint32_t)(lkey[(lhead + ln - R) & rmask] >> 32) : 0u;
                const uint32_t prev1 = ln < R ? F : sat_add(back, L1);
                uint64_t ok1 = WM & wv::ballot(prev1 <= rdy);
                if (B > 1) ok1 &= wv::ballot(rdy != wv::shl1(rdy)) | ~lanes_below(w - 1u);
                uint32_t m = 0, x = 0;
                if (ok1 == WM) {
                    m = (B > 1 && !last) ? w - 1u : w;  // (for B > 1 the last query may yet be joined by the next)
                    x = sat_add(rdy, L1);
                } else if (B == 1) {
                    const uint32_t lo = wv::opaque(ln);
                    const uint32_t kd = (lo * inv_r) >> 16, km = lo - kd * R;
                    const uint64_t st = (uint64_t)wv::shfl(F, km) + (uint64_t)kd * L1;  // when my replica is free for me
                    const uint64_t en = st + L1;
                    x = en >= 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)en;
                    const uint32_t xp = wv::shr1(x);
                    if ((WM & ~(wv::ballot((uint64_t)rdy <= st) & wv::ballot(x != 0xFFFFFFFFu) & (wv::ballot(x > xp) | 1ull))) == 0) m = w;
                }
                if (m >= R && wv::bcast(x, m - 1u) != 0xFFFFFFFFu) {
                    if (ln < m) out[(wr + ln) & omask] = ((uint64_t)x << 32) | q;
                    wr += m;
                    space -= m;
                    EST_CHK_ORDER(9);
                    const uint32_t tnew = wv::shfl(x, ln + m - R);  // the table becomes the last R completion times
                    if (isrep) F = tnew;
                    lhead += m;
                    ++d_b1; d_b1e += m;
                    if (DIAG) d_tk[2] += wv::ticks() - tk0;
                    continue;
                }
                cf_skip = 6;
            } else if (cf_skip) {
                --cf_skip;
            }
            // With larger batch sizes the same evaluation holds as long as no query waits and no two become
            // ready together: then every query is a batch of its own, started on arrival.
            const bool single = B > 1 && single_skip == 0 && w >= 16;
            if (B == 1 || single) {
                // Maximum batch size 1: every query is its own batch and the service time is the constant
                // L(1), so completions keep the input order and query i runs on the replica that served
                // query i-R:  end_i = max(ready_i, end_{i-R}) + L(1).  The sorted replica table is exactly
                // (end_{i-R}, ..., end_{i-1}), so a whole window is evaluated at once with a max-plus
                // scan of stride R.  Nothing is pending: results are written out immediately.
                uint32_t x = sat_add(umax(rdy, isrep ? F : 0u), L1);
                for (uint32_t d = R, mul = 1; d < 64; d <<= 1, mul <<= 1) {
                    const uint32_t y = wv::shfl(x, ln - d);
                    const uint32_t inc = (uint64_t)mul * L1 > 0xFFFFFFFFull ? 0xFFFFFFFFu : mul * L1;
                    if (ln >= d) x = umax(x, sat_add(y, inc));
                }
                uint32_t m = w;
                bool sorted = true;
                if (single) {
                    // the leading queries that start on arrival, each alone at its ready time (the one after
                    // it must be seen to become ready later); completion times then ascend strictly, and
                    // whatever is dispatched later finishes later still
                    const uint32_t rnext = wv::shl1(rdy);
                    const uint64_t gm = lanes_below(w) & wv::ballot(x == sat_add(rdy, L1)) & wv::ballot(x != 0xFFFFFFFFu) &
                                        ((wv::ballot(rdy != rnext) & lanes_below(w - 1u)) | (last ? 1ull << (w - 1u) : 0ull));
                    m = gm == ~0ull ? 64u : ctz64(~gm);
                    if (m < 12) {
                        single_skip = 6;  // not the regime: leave it alone for a few steps
                        m = 0;
                    }
                } else {
                    // Queries that complete at the same time leave ordered by query index.  Since
                    // end_i > end_{i-R}, such a run has at most R members; a shorter run at the end of what
                    // can be written now may continue with the next query, and is kept back until that is
                    // known (times clamped at the horizon need no order).
                    const uint32_t xp = wv::shr1(x);
                    const uint32_t qp = wv::shr1(q);
                    const uint64_t bnd = (lanes_below(w) & wv::ballot(x != xp)) | 1ull;  // starts of runs
                    const uint32_t s0 = 63u - (uint32_t)__builtin_clzll(bnd & lanes_below(m));  // start of the run of lane m-1
                    const uint32_t xl = wv::bcast(x, m - 1u);
                    if (!(last || xl == 0xFFFFFFFFu || m - s0 >= R)) m = s0;
                    if (m == 0) break;  // wait for the rest of the run
                    sorted = (lanes_below(m) & ~1ull & wv::ballot(x == xp) & wv::ballot(q < qp) & wv::ballot(x != 0xFFFFFFFFu)) == 0;
                }
                if (m > 0) {
                    uint64_t okey = ln < m ? (((uint64_t)x << 32) | q) : ~0ull;
                    if (!sorted) okey = sort_lanes64(okey);
                    if (ln < m) out[(wr + ln) & omask] = okey;
                    wr += m;
                    space -= m;
                    ++d_b1; d_b1e += m;
                    if (DIAG) d_tk[2] += wv::ticks() - tk0;
                    EST_CHK_ORDER(1);
                    // the table becomes the last R completion times
                    const uint32_t keep = R > m ? R - m : 0u;  // old entries that stay
                    const uint32_t told = wv::shfl(F, ln + m);
                    const uint32_t tnew = wv::shfl(x, ln + m - R);
                    if (isrep) F = ln < keep ? told : tnew;
                    // (old entries that stay ended by some earlier start + L(1): no later than the new ends)
                    const uint32_t fbefore = wv::shr1(F);
                    EST_CHECK(ln == 0 || !isrep || F >= fbefore);
                    (void)fbefore;
                    lhead += m;
                    continue;
                }
            }
            if (single_skip) --single_skip;
        }
        // ---- form the next batches: heads = first queries of the batches, a = queries taken, gend in the lanes nG .. K-1 =
        //      completion time of every new batch, F = the new free times
        uint32_t K = nG, a = 0, kind = 3;
        uint64_t heads = 0;
        if (sat_skip == 0 && B >= 2 && w >= 2 * B && wv::bcast(rdy, B - 1) <= f0) {
            // Backlog: while the queue holds a full batch whenever a replica frees, the replicas take
            // full batches in rotation.  With the free times f_0 <= ... <= f_{R-1} < f_0 + L(B), batch k
            // (queries kB .. kB+B-1 of the window) starts at f_k, where f_k = f_{k-R} + L(B) for k >= R,
            // provided its last member is ready by then.  The leading batches that satisfy this are all
            // dispatched at once.
            const uint32_t LB = wv::bcast(Lmine, B - 1);
            if (wv::bcast(F, R - 1) < wv::sat_add_uniform(f0, LB)) {
                const uint32_t lo = wv::opaque(ln);
                const uint32_t kb = (lo * inv_b) >> 16;        // my batch
                const uint32_t kd = (kb * inv_r) >> 16, km = kb - kd * R;
                const uint64_t ft = (uint64_t)wv::shfl(F, km) + (uint64_t)kd * LB;
                const uint32_t fk = ft >= 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)ft;
                const uint32_t e = sat_add(fk, LB);
                const uint32_t nfull = umin((w * inv_b) >> 16, nslots - nG);
                const uint32_t lastr = wv::shfl(rdy, kb * B + B - 1u);
                const uint64_t okm = lanes_below(nfull * B) & wv::ballot(lastr <= fk) & wv::ballot(e != 0xFFFFFFFFu);
                const uint32_t nl = okm == ~0ull ? 64u : ctz64(~okm);  // a multiple of B: the test is per batch
                const uint32_t nacc = (nl * inv_b) >> 16;
                if (nacc >= 2) {
                    a = nacc * B;
                    K = nG + nacc;
                    kind = 4;
                    heads = lanes_below(a) & wv::ballot(lo == kb * B);
                    const uint32_t first = (ln - nG) * B, en = wv::shfl(e, first);
                    if (ln >= nG && ln < K) gend = en;
                    // the entries not taken, then the last min(nacc, R) batches
                    const uint32_t nn = umin(nacc, R);
                    const uint32_t oe = wv::shfl(F, ln + nn), ne = wv::shfl(e, (nacc - R + ln) * B);
                    if (isrep) F = ln + nn < R ? oe : ne;
                }
            }
            if (a == 0) sat_skip = 4;
        } else if (sat_skip) {
            --sat_skip;
        }
        if (a == 0) {
            // batch by batch; a batch that is not full is decided once a query ready later is in view, or none can follow
            const uint64_t tkl = DIAG ? wv::ticks() : 0;
            if (umax(wv::bcast(rdy, w - 1u), wv::bcast(F, R - 1u)) < t_inside)
                wv::form_batches_inside(rdy, Lrot, B, w, nslots, F, gend, heads, a, K);
            if (K < nslots) wv::form_batches(rdy, Lrot, B, w, last ? 65u : w, nslots, F, gend, heads, a, K);
            a = umin(a, w);
            if (DIAG) { d_blkl += wv::ticks() - tkl; d_blkk += K - nG; }
            if (a == 0) break;  // undecidable: wait for input
        }
        // ---- the new batches become pending: members to their slots, sizes, everything in order of completion
        {
            const uint32_t kb = nG + wv::rank_below(heads >> 1);  // my batch's lane (query 0 starts the first)
            const bool head = wv::lane_in(heads);
            const uint32_t vA = wv::push(head ? ln : 0u, head ? kb : nG);  // first query of the lane's batch (the first of all at query 0)
            const uint32_t pk = wv::shfl((ginfo & 0xFFu) | (vA << 8), kb);
            if (ln < a) lslots[(pk & 0xFFu) * B + (ln - (pk >> 8))] = q;
            const uint32_t anext = wv::shl1(vA);
            const uint32_t cnt = (ln + 1u == K ? a : anext) - vA;
            if (ln >= nG && ln < K) ginfo = (ginfo & 0xFFu) | (cnt << 8);
            if (kind == 3 && a >= 4u * (K - nG)) kind = 0;
            nG = K;
            EST_CHECK(nG <= nslots);
            const uint32_t gprev = wv::shr1(gend);
            if (lanes_below(nG) & ~1ull & wv::ballot(gprev > gend)) {
                const uint32_t base = T0, d = gend - base;  // (everything pending completes after T0)
                uint32_t from;
                if ((lanes_below(nG) & wv::ballot(d >= (1u << 26))) == 0) {
                    from = sort_lanes(ln < nG ? ((d << 6) | ln) : 0xFFFFFFFFu, pow2_at_least(nG)) & 63u;
                } else {
                    from = (uint32_t)sort_lanes64(ln < nG ? (((uint64_t)gend << 32) | ln) : ~0ull) & 63u;
                }
                if (ln >= nG) from = ln;  // (the free slots stay where they are)
                gend = wv::shfl(gend, from);
                ginfo = wv::shfl(ginfo, from);
            }
            wv::sync_lds();
            lhead += a;
            if (kind == 4) { ++d_sat; d_sate += a; } else if (kind == 0) { ++d_grp; d_grpe += a; } else { ++d_blk; d_blke += a; }
            if (DIAG) d_tk[kind] += wv::ticks() - tk0;
        }
    }

    if (DIAG && c.a->dbg_ticks && ln == 0) {
        uint64_t *pc = est_dbg_rec(c.a, c.t, s);  // per candidate and stage (one writer: no atomics)
        pc[2] += d_b1 + d_sat + d_blk + d_grp; pc[3] += d_b1e + d_sate + d_hz + d_blke + d_grpe;
        pc[4] += d_grpe; pc[6] += d_b1e; pc[7] += d_blke;
        for (uint32_t i = 0; i < 6; ++i) pc[8 + i] += d_tk[i];
        pc[14] += d_blkl; pc[15] += d_blkk;
        wv::atomic_add_u64(&est_dbg_rec(c.a, c.t, EST_MAX_STAGES - 1)[6], 1);
    }
    // back to memory: the free times, the pending batches and their members, the cursors
    if (isrep) g_free[ln] = F;
    g_end[ln] = gend;
    g_info[ln] = ginfo;
    const uint32_t left_over = ltail - lhead;
    if (ln == 0) { g_n[0] = nG; g_n[1] = left_over; }
    if (nG)
        for (uint32_t i = ln; i < SW; i += 64) g_slots[i] = lslots[i];
    for (uint32_t i = ln; i < left_over; i += 64) g_keys[i] = lkey[(lhead + i) & rmask];
    wv::sync();  // what was written to the output ring is in place before its cursor moves
    if (ln == 0) {
        st_st(&c.st[P.rd_off + op.src_edge[0]], rraw);
        st_st(&c.st[P.wr_off + op.out_ring], wr);
        if (finished) st_st(&c.st[P.fin_off + op.out_ring], EST_FIN);
    }
    return finished;
}

// ------------------------------------------------------------------------------------------ MERGE

// Keys clamped at the horizon may appear in any order inside a stream (see emit_pending); for merging
// they are ordered by (source, staging index) instead of by query index.
EST_DEV uint64_t eff_key(uint64_t key, uint32_t j, uint32_t l) {
    return (uint32_t)(key >> 32) == 0xFFFFFFFFu ? (0xFFFFFFFF00000000ull | (uint64_t)(j << 8) | l) : key;
}

// Staged elements per source of a merge (LDS ring), how many of them a round looks at, sources whose loads are issued
// together.  (62 and not 64: a merge of four then fits the LDS of six wavefronts per SIMD.)
enum { MERGE_RING = 128, MERGE_WIN = 62, MERGE_GROUP = 4 };

template <bool DIAG, bool MEMO>
EST_DEV bool merge_run(const Ctx &c, const EstOp &op) {
    const uint32_t ln = wv::lane();
    const EstPlan &P = *c.P;
    const uint32_t K = wv::uniform(op.n_src);
    const bool is_lat = wv::uniform(op.type) == EST_OP_LAT;
    const uint8_t *acc = c.a->acc + (uint64_t)op.acc_idx * c.a->acc_stride;
    uint64_t *out = nullptr;
    uint32_t omask = 0, wr, space = 0xFFFFFFFFu;
    if (is_lat) {
        wr = wv::uniform(c.st[P.miss_off + 1]);
    } else {
        const EstRing &OR = P.rings[op.out_ring];
        out = c.rings + OR.off;
        omask = wv::uniform(OR.cap_mask);
        wr = wv::uniform(c.st[P.wr_off + op.out_ring]);
        space = wv::uniform(ring_space(c, op.out_ring, wr));
    }
    uint32_t miss = 0, wr_pub = wr;
    uint32_t d_rounds = 0, d_elems = 0;  // diagnostics
    bool finished = false;

    if (K == 1 && !op.has_cnt) {
        // one source, every query fed by it alone: filter and copy, four windows of 64 at a time (their
        // loads are issued together)
        View sv = uniform_view_of<MEMO>(c, op.src_ring[0]);
        uint32_t rc = wv::uniform(c.st[P.rd_off + op.src_edge[0]]);
        const uint32_t slo = wv::uniform(c.a->slo_us);
        for (;;) {
            if (!is_lat && space < 256u) {
                space = wv::uniform(ring_space(c, op.out_ring, wr));
                if (space < 256u) break;  // wait for the consumer
            }
            if (sv.wr - rc < 256u && !sv.fin) {  // the producer may have gone on meanwhile
                sv = uniform_view_of<MEMO>(c, op.src_ring[0]);
                wv::sync();
            }
            if (rc == sv.wr) {
                finished = sv.fin != 0;
                break;
            }
            const uint32_t left = sv.wr - rc;
            uint64_t key[4];
            uint32_t av[4], arr[4];
EST_UNROLL
            for (uint32_t u = 0; u < 4; ++u) key[u] = u * 64u + ln < left ? sv.base[(rc + u * 64u + ln) & sv.mask] : 0ull;
EST_UNROLL
            for (uint32_t u = 0; u < 4; ++u) av[u] = acc[(uint32_t)key[u]];  // (idle lanes look at query 0)
            if (is_lat) {
EST_UNROLL
                for (uint32_t u = 0; u < 4; ++u) arr[u] = c.a->arrival[(uint32_t)key[u]];
            }
EST_UNROLL
            for (uint32_t u = 0; u < 4; ++u) {
                const bool a = u * 64u + ln < left && (av[u] & 1u) != 0u;
                const uint64_t A = wv::ballot(a);
                const uint32_t pos = wr + wv::rank_below(A);
                if (a) {
                    if (is_lat) {
                        const uint32_t l = (uint32_t)(key[u] >> 32) - arr[u];
                        c.lat[c.a->lat_by_qid ? (uint32_t)key[u] : pos] = l;
                        miss += l > slo;
                    } else {
                        out[pos & omask] = key[u];
                    }
                }
                const uint32_t na = popc64(A);
                wr += na;
                if (!is_lat) space -= na;
            }
            rc += umin(left, 256u);
            if (wr - wr_pub >= 2048u) {
                wv::sync();
                if (ln == 0) {
                    if (!is_lat) st_st(&c.st[P.wr_off + op.out_ring], wr);
                    st_st(&c.st[P.rd_off + op.src_edge[0]], rc);
                }
                wr_pub = wr;
            }
        }
        if (ln == 0) st_st(&c.st[P.rd_off + op.src_edge[0]], rc);
    } else {
        // Several sources.  A query fed by several of them is ready at the largest of its times: of its
        // elements only the one with the largest key (time, query; equal times: the higher source) is passed
        // on.  Every accepted element leaves its time in its source's table when it is staged; an entry
        // still unset reads as the horizon.  Sources are consumed in key order, so when an element is
        // consumed every element of the same query with a smaller key has been staged already, and an
        // element whose partner is unset or larger is not the last.  No counting, no read-modify-write.
        //
        // LDS: per source a ring of MERGE_RING staged keys (uint64) | per source MERGE_WIN passed-on keys (uint64) |
        // per source MERGE_RING accept masks (uint8).  The per-source scalars live in two vector registers, one
        // lane per (field, source): reading one is a lane read into a scalar register, not a trip to LDS.
        const uint32_t KS = P.max_src;
        uint64_t *rkey = c.lds;
        uint64_t *lst = c.lds + KS * MERGE_RING;
        uint8_t *racc = (uint8_t *)(lst + KS * MERGE_WIN);
        enum { F_RD = 0, F_WR = 8, F_FIN = 16, F_HEAD = 24, F_TAIL = 32, F_MASK = 40, F_BLO = 48, F_BHI = 56,  // va: lane = field + source
               F_NFIN = 0, F_CONS = 8 };                                                                    // vb: passed on / consumed this round
        uint32_t va = 0, vb = 0;
        const uint32_t tab_mask = wv::uniform(op.tab_mask), tab_len = wv::uniform(op.tab_len);
        uint32_t *tab0 = (uint32_t *)(c.tab + op.tab_off);
        for (uint32_t j = 0; j < K; ++j) {
            const View sv = uniform_view_of<MEMO>(c, op.src_ring[j]);
            const uint64_t bp = (uint64_t)(uintptr_t)sv.base;
            va = wv::set_lane(va, wv::uniform(c.st[P.rd_off + op.src_edge[j]]), F_RD + j);
            va = wv::set_lane(va, sv.wr, F_WR + j);
            va = wv::set_lane(va, sv.fin, F_FIN + j);
            va = wv::set_lane(va, sv.mask, F_MASK + j);
            va = wv::set_lane(va, wv::uniform((uint32_t)bp), F_BLO + j);
            va = wv::set_lane(va, wv::uniform((uint32_t)(bp >> 32)), F_BHI + j);
        }
        for (;;) {
            if (!is_lat && space < 64u * K) {
                space = wv::uniform(ring_space(c, op.out_ring, wr));
                if (space < 64u * K) break;  // wait for the consumer
            }
            // ---- refill: every source with no more than a window staged takes up to 64 further elements; the
            //      loads of all sources are issued before any is used.  (Refilling all of them only once one had run
            //      low: fewer trips to memory but shorter windows, 5 to 9 % slower.)
            bool any = false;
            for (uint32_t j0 = 0; j0 < K; j0 += MERGE_GROUP) {
                uint64_t kx[MERGE_GROUP];
                uint32_t wx[MERGE_GROUP], ax[MERGE_GROUP];
                bool some = false;
EST_UNROLL
                for (uint32_t u = 0; u < MERGE_GROUP; ++u) {
                    const uint32_t j = j0 + u;
                    wx[u] = 0;
                    kx[u] = 0;
                    if (j < K) {
                        const uint32_t staged = wv::bcast(va, F_TAIL + j) - wv::bcast(va, F_HEAD + j);
                        const uint32_t rd = wv::bcast(va, F_RD + j), left = wv::bcast(va, F_WR + j) - rd;
                        if (staged <= 64u && left > 0u) {
                            const uint64_t *base = (const uint64_t *)(uintptr_t)(((uint64_t)wv::bcast(va, F_BHI + j) << 32) | wv::bcast(va, F_BLO + j));
                            const uint32_t smask = wv::bcast(va, F_MASK + j);
                            wx[u] = umin(64u, left);
                            if (ln < wx[u]) kx[u] = base[(rd + ln) & smask];
                            some = true;
                        }
                    }
                }
                if (!some) continue;
                any = true;
EST_UNROLL
                for (uint32_t u = 0; u < MERGE_GROUP; ++u) ax[u] = (wx[u] && ln < wx[u]) ? acc[(uint32_t)kx[u]] : 0u;
EST_UNROLL
                for (uint32_t u = 0; u < MERGE_GROUP; ++u) {
                    const uint32_t j = j0 + u;
                    if (!wx[u]) continue;
                    uint32_t am = ax[u];
                    if (!((am >> j) & 1u)) am = 0;  // not for this stage, or superseded by a nearer ancestor
                    if (((tab_mask >> j) & 1u) && (am & (am - 1u)))
                        tab0[(uint64_t)__builtin_popcount(tab_mask & ((1u << j) - 1u)) * tab_len + (uint32_t)kx[u]] = (uint32_t)(kx[u] >> 32);
                    const uint32_t tl = wv::bcast(va, F_TAIL + j);
                    const uint32_t at = j * MERGE_RING + ((tl + ln) & (MERGE_RING - 1u));
                    if (ln < wx[u]) {
                        rkey[at] = kx[u];
                        racc[at] = (uint8_t)am;
                    }
                    va = wv::set_lane(va, tl + wx[u], F_TAIL + j);
                    va = wv::set_lane(va, wv::bcast(va, F_RD + j) + wx[u], F_RD + j);
                }
            }
            if (wr - wr_pub >= 512u) {  // tell the neighbours how far this operation is
                wv::sync();
                for (uint32_t j = 0; j < K; ++j) {
                    const uint32_t back = wv::bcast(va, F_RD + j) - (wv::bcast(va, F_TAIL + j) - wv::bcast(va, F_HEAD + j));
                    if (ln == 0) st_st(&c.st[P.rd_off + op.src_edge[j]], back);
                }
                if (ln == 0 && !is_lat) st_st(&c.st[P.wr_off + op.out_ring], wr);
                wr_pub = wr;
            }
            if (any) wv::sync();  // (tables and staged elements: written above, read below by other lanes)
            // ---- the window of every source: its first MERGE_WIN staged elements
            uint32_t more = 0, total = 0;  // more, bit j: source j may hold elements beyond its window
            bool blocked = false, clamped = false;
            uint64_t bound = ~0ull;  // everything up to the smallest last key of a source that may hold more is final
            for (uint32_t j = 0; j < K; ++j) {
                const uint32_t h = wv::bcast(va, F_HEAD + j), staged = wv::bcast(va, F_TAIL + j) - h;
                const uint32_t w = umin((uint32_t)MERGE_WIN, staged);
                const bool has_more = staged > (uint32_t)MERGE_WIN || wv::bcast(va, F_RD + j) != wv::bcast(va, F_WR + j) || !wv::bcast(va, F_FIN + j);
                if (has_more) more |= 1u << j;
                total += w;
                if (w == 0) {
                    blocked = blocked || has_more;
                } else {
                    const uint64_t lk = rkey[j * MERGE_RING + ((h + w - 1u) & (MERGE_RING - 1u))];
                    const uint32_t tl = wv::uniform((uint32_t)(lk >> 32)), ql = wv::uniform((uint32_t)lk);
                    clamped = clamped || tl == 0xFFFFFFFFu;
                    if (has_more) {
                        const uint64_t last = eff_key(((uint64_t)tl << 32) | ql, j, w - 1u);
                        bound = last < bound ? last : bound;
                    }
                }
            }
            if (blocked || total == 0) {
                if (!blocked && more == 0) {
                    finished = true;
                    break;
                }
                // the producers may have gone on meanwhile
                bool news = false;
                for (uint32_t j = 0; j < K; ++j) {
                    if (wv::bcast(va, F_FIN + j)) continue;
                    const View sv = uniform_view_of<MEMO>(c, op.src_ring[j]);
                    if (sv.wr != wv::bcast(va, F_WR + j) || sv.fin) news = true;
                    va = wv::set_lane(va, sv.wr, F_WR + j);
                    va = wv::set_lane(va, sv.fin, F_FIN + j);
                }
                if (!news) break;
                wv::sync();
                continue;
            }
            // ---- which of the consumed elements are passed on (the table look-ups of all sources are issued together)
            uint32_t n_out = 0;
            for (uint32_t j0 = 0; j0 < K; j0 += MERGE_GROUP) {
                uint64_t kx[MERGE_GROUP];
                uint32_t amx[MERGE_GROUP], t2x[MERGE_GROUP];
                bool px[MERGE_GROUP];
                uint32_t hard = 0;  // bit u: some element of the source has more than one partner
EST_UNROLL
                for (uint32_t u = 0; u < MERGE_GROUP; ++u) {
                    const uint32_t j = j0 + u;
                    kx[u] = 0; amx[u] = 0; t2x[u] = 0; px[u] = false;
                    if (j < K) {
                        const uint32_t h = wv::bcast(va, F_HEAD + j);
                        const uint32_t w = umin((uint32_t)MERGE_WIN, wv::bcast(va, F_TAIL + j) - h);
                        const uint32_t at = j * MERGE_RING + ((h + ln) & (MERGE_RING - 1u));
                        if (ln < w) { kx[u] = rkey[at]; amx[u] = racc[at]; }
                        const uint64_t x = clamped ? eff_key(kx[u], j, ln) : kx[u];
                        const bool consumed = ln < w && x <= bound;  // a prefix of the window: a source's keys ascend
                        const uint32_t mj = popc64(wv::ballot(consumed));
                        vb = wv::set_lane(vb, mj, F_CONS + j);
                        px[u] = consumed && amx[u] != 0u;
                        const uint32_t others = amx[u] & ~(1u << j);
                        if (px[u] && others != 0u) {
                            const uint32_t j2 = (uint32_t)__builtin_ctz(others);
                            t2x[u] = tab0[(uint64_t)__builtin_popcount(tab_mask & ((1u << j2) - 1u)) * tab_len + (uint32_t)kx[u]];
                        }
                        if (wv::ballot(px[u] && (others & (others - 1u)) != 0u)) hard |= 1u << u;
                    }
                }
EST_UNROLL
                for (uint32_t u = 0; u < MERGE_GROUP; ++u) {
                    const uint32_t j = j0 + u;
                    if (j < K) {
                        const uint32_t t = (uint32_t)(kx[u] >> 32);
                        const uint32_t others = amx[u] & ~(1u << j);
                        bool pass = px[u];
                        if (pass && others != 0u) {
                            const uint32_t j2 = (uint32_t)__builtin_ctz(others);
                            if (!(t2x[u] < t || (t2x[u] == t && j2 < j))) pass = false;
                        }
                        if ((hard >> u) & 1u) {  // more than two parents: the remaining partners one by one
                            for (uint32_t j2 = 0; j2 < K; ++j2) {
                                const bool need = pass && j2 != j && ((others >> j2) & 1u);
                                if (!wv::ballot(need)) continue;
                                const uint32_t t2 = need ? tab0[(uint64_t)__builtin_popcount(tab_mask & ((1u << j2) - 1u)) * tab_len + (uint32_t)kx[u]] : 0u;
                                if (need && !(t2 < t || (t2 == t && j2 < j))) pass = false;
                            }
                        }
                        const uint64_t F = wv::ballot(pass);
                        const uint32_t fr = wv::rank_below(F);
                        if (pass) lst[j * MERGE_WIN + fr] = kx[u];
                        vb = wv::set_lane(vb, popc64(F), F_NFIN + j);
                        n_out += popc64(F);
                    }
                }
            }
            ++d_rounds; d_elems += n_out;
            wv::sync_lds();
            // ---- place the passed-on elements.  As many as a wavefront has lanes: the lists are merged one after the other,
            //      each put behind what is there with its order reversed, so that the last six steps of a sorting network
            //      are left; no trip to LDS depends on another, and the output is written in one piece.  More of them, or
            //      times clamped at the horizon: every element's rank in its own list plus the smaller elements of the others
            //      (a search is six dependent trips to LDS per pair of lists).  A join sets the pace of a candidate that has a
            //      workgroup to itself; its rounds pass on 51 elements on average on the ten-stage pipeline, in 6.0 us when
            //      all were placed by searches.  97 candidates x 99,991 queries of the fork and join 16.0 -> 13.1 ms, one of
            //      ten stages x 20,011 2.91 -> 2.58 ms, the grid of 12,288 x 100,003 189 -> 183 ms.
            if (n_out <= 64u && !clamped) {
                uint64_t rk = ~0ull;
                uint32_t have = 0;
                for (uint32_t j = 0; j < K; ++j) {
                    const uint32_t nf = wv::bcast(vb, F_NFIN + j);
                    if (nf == 0) continue;
                    const uint32_t at = have ? 63u - ln : ln;
                    if (at < nf) rk = lst[j * MERGE_WIN + at];
                    if (have) rk = sort_merge64<64>(rk);
                    have += nf;
                }
                if (ln < n_out) {
                    if (is_lat) {
                        const uint32_t q = (uint32_t)rk;
                        const uint32_t l = (uint32_t)(rk >> 32) - c.a->arrival[q];
                        c.lat[c.a->lat_by_qid ? q : wr + ln] = l;
                        miss += l > c.a->slo_us;
                    } else {
                        out[(wr + ln) & omask] = rk;
                    }
                }
            } else {
                for (uint32_t j = 0; j < K; ++j) {
                    const uint32_t nf = wv::bcast(vb, F_NFIN + j);
                    if (nf == 0) continue;
                    const bool have = ln < nf;
                    const uint64_t rk = have ? lst[j * MERGE_WIN + ln] : 0ull;
                    uint32_t rank = ln;
                    for (uint32_t j2 = 0; j2 < K; ++j2) {
                        const uint32_t n2 = wv::bcast(vb, F_NFIN + j2);
                        if (j2 == j || n2 == 0) continue;
                        const uint64_t *l2 = lst + j2 * MERGE_WIN;
                        const uint32_t top = 1u << (31u - (uint32_t)__builtin_clz(n2));  // the largest power of two within the list
                        uint32_t lo = 0;  // elements of list j2 below rk (no two lists hold the same key: one element per query is passed on)
                        if (!clamped) {
                            for (uint32_t step = top; step >= 1; step >>= 1) {
                                const uint32_t i = lo + step;
                                const bool in = i <= n2;
                                const uint64_t y = l2[in ? i - 1u : 0u];
                                if (in && y < rk) lo = i;
                            }
                        } else {
                            const uint64_t x = eff_key(rk, j, ln);
                            for (uint32_t step = top; step >= 1; step >>= 1) {
                                const uint32_t i = lo + step;
                                const bool in = i <= n2;
                                const uint64_t y = eff_key(l2[in ? i - 1u : 0u], j2, in ? i - 1u : 0u);
                                if (in && y < x) lo = i;
                            }
                        }
                        rank += lo;
                    }
                    if (have) {
                        const uint32_t pos = wr + rank;
                        if (is_lat) {
                            const uint32_t q = (uint32_t)rk;
                            const uint32_t l = (uint32_t)(rk >> 32) - c.a->arrival[q];
                            c.lat[c.a->lat_by_qid ? q : pos] = l;
                            miss += l > c.a->slo_us;
                        } else {
                            out[pos & omask] = rk;
                        }
                    }
                }
            }
            wr += n_out;
            if (!is_lat) space -= n_out;  // (a reader may have made more room since: looked up again when this runs short)
            for (uint32_t j = 0; j < K; ++j) va = wv::set_lane(va, wv::bcast(va, F_HEAD + j) + wv::bcast(vb, F_CONS + j), F_HEAD + j);
            wv::sync_lds();
        }
        // staged but not consumed: read again next time
        for (uint32_t j = 0; j < K; ++j) {
            const uint32_t back = wv::bcast(va, F_RD + j) - (wv::bcast(va, F_TAIL + j) - wv::bcast(va, F_HEAD + j));
            if (ln == 0) st_st(&c.st[P.rd_off + op.src_edge[j]], back);
        }
    }

    if (DIAG && c.a->dbg_ticks && ln == 0) {
        uint64_t *po = est_dbg_rec(c.a, c.t, EST_MAX_STAGES - 1);
        wv::atomic_add_u64(&po[3], d_rounds); wv::atomic_add_u64(&po[4], d_elems); wv::atomic_add_u64(&po[5], 1);
    }
    const uint32_t miss_all = is_lat ? wv::sum_u32(miss) : 0u;
    wv::sync();  // what was written to the output ring is in place before its cursor moves
    if (ln == 0) {
        if (is_lat) {
            st_st(&c.st[P.miss_off + 1], wr);
            st_st(&c.st[P.miss_off], ld_st(&c.st[P.miss_off]) + miss_all);
        } else {
            st_st(&c.st[P.wr_off + op.out_ring], wr);
            if (finished) st_st(&c.st[P.fin_off + op.out_ring], EST_FIN);
        }
    }
    return finished;
}

// ------------------------------------------------------------------------------------------ driver
//
// A workgroup of a.waves wavefronts works on up to a.per_group candidates at a time (one scratch slot each).  Wavefront
// w < per_group takes a candidate from the launch's work counter whenever slot w is free, and prefers that candidate's
// operations; a wavefront whose own candidate has nothing it could run, or that has none (fewer candidates than
// wavefronts, or none left), runs an operation of another candidate of the workgroup.  An operation is run by one wavefront at
// a time (a lock per operation); what it needs is in the slot's memory, so any wavefront can go on with it.  So a
// candidate alone in its workgroup runs as a pipeline over all of its wavefronts, and the last candidates of a launch are
// finished by everybody.  (What bounds a call with few candidates is its slowest single simulation, and what a sweep loses
// at its end are the wavefronts without a candidate.  With one wavefront per candidate, or the operations of a candidate
// cut beforehand into four runs for a workgroup of four, against this: 16 candidates x 10^6 queries of the ten-stage pipeline
// 341 -> 130 ms, 4,500 x 50,000 62 -> 49 ms, 12,288 x 100,000 255 -> 206 ms.)
//
// Control words in LDS.  Of the workgroup: [0] no candidates are left, [1] how many wavefronts are running something (low 8
// bits) and how often one has finished (above); then the plan's lists of state words to watch.
// Of a slot: candidate, phase, operations done, memoised rings (two words), spare; then per operation its lock (0 free,
// 1 running, 2 done) and what it had seen when it was last entered; then the candidate's state words.
enum { G_DRAINED = 0, G_WORK = 1, G_WORDS = 4, C_T = 0, C_PHASE = 1, C_DONE = 2, C_MEMO = 3, C_T0 = 5, C_LOCK = 6 };
enum { PH_EMPTY = 0, PH_INIT = 1, PH_RUN = 2 };
enum { STEP_IDLE = 0, STEP_WORKED = 1, STEP_END = 2 };

struct Pool {
    const EstSimArgs *a;
    uint32_t *gw, *ctl;
    const uint16_t *woff, *watch;
};

EST_DEV Pool make_pool(const EstSimArgs &a, uint32_t *lds) {
    Pool p;
    p.a = &a;
    p.gw = lds;
    p.woff = (const uint16_t *)(lds + G_WORDS);
    p.watch = p.woff + EST_WATCH_HEAD(a.n_ops);
    p.ctl = lds + G_WORDS + EST_WATCH_WORDS(a.n_ops, a.n_watch);
    return p;
}

EST_DEV uint32_t *slot_ctl(const Pool &p, uint32_t j) { return p.ctl + j * p.a->ctl_words; }
EST_DEV uint32_t *slot_state(const Pool &p, uint32_t j) { return p.ctl + j * p.a->ctl_words + C_LOCK + 2u * p.a->n_ops; }

// By one lane: something begins, and ends, to run in this workgroup (the start of a candidate, an operation with the selection
// that may follow it).  It is said before the slot or the operation is taken, so there is no moment at which only the taker
// knows; a taker that comes too late takes it back.
EST_DEV void work_begin(const Pool &p) { wv::lds_add(&p.gw[G_WORK], 1u); }
EST_DEV void work_end(const Pool &p) { wv::lds_add(&p.gw[G_WORK], 0xFFu); }  // (one fewer running, one more finished)
EST_DEV void work_cancel(const Pool &p) { wv::lds_add(&p.gw[G_WORK], 0xFFFFFFFFu); }

// What a wavefront remembers between two looks that found nothing to do.
struct Wait {
    uint32_t idle, still, seen;
};

// Whether to give up, after a look that found nothing: limit looks in a row during which nobody in the workgroup ran
// anything or finished anything.  How long a wavefront itself goes without work says nothing: a pipeline of two operations
// leaves two of four wavefronts idle for as long as its trace lasts.
EST_DEV bool stuck(const Pool &p, Wait &w, uint32_t limit) {
    const uint32_t v = wv::uniform(ld_st(&p.gw[G_WORK]));
    if ((v & 0xFFu) != 0u || v != w.seen) {
        w.seen = v;
        w.still = 0;
        return false;
    }
    return ++w.still > limit;
}

// By one wavefront, before any other starts.
EST_DEV void pool_setup(const Pool &p) {
    const uint32_t ln = wv::lane();
    const EstSimArgs &a = *p.a;
    if (ln < G_WORDS) p.gw[ln] = 0;
    if (a.n > 0) {
        uint16_t *wo = (uint16_t *)p.woff, *wt = (uint16_t *)p.watch;
        for (uint32_t i = ln; i <= a.n_ops; i += 64) wo[i] = a.plan->watch_off[i];
        for (uint32_t i = ln; i < a.n_watch; i += 64) wt[i] = a.plan->watch[i];
    }
    for (uint32_t j = 0; j < a.per_group; ++j) {
        if (ln == 0) slot_ctl(p, j)[C_PHASE] = PH_EMPTY;
        for (uint32_t i = ln; i < a.n_ops; i += 64) slot_ctl(p, j)[C_LOCK + i] = 2;
    }
    wv::sync_lds();
}

EST_DEV Ctx make_ctx(const EstSimArgs &a, uint32_t t, uint32_t slot, uint32_t *st, uint64_t *lds) {
    Ctx c;
    c.a = &a;
    c.P = a.plan;
    c.st = st;
    c.rings = a.rings + (uint64_t)slot * a.ring_stride;
    c.rep = a.rep + (uint64_t)slot * a.rep_stride;
    c.slots = a.slots + (uint64_t)slot * a.slot_stride;
    c.tab = a.tabs + (uint64_t)slot * a.tab_stride;
    c.lat = a.lat + (uint64_t)(a.lat_by_qid ? t : slot) * a.lat_stride;
    c.cfg = a.cfg + (uint64_t)t * a.dag->S;
    c.lds = lds;
    c.t = t;
    c.memo_rings = 0;
    c.cap_rings = nullptr;
    return c;
}

// A candidate's scratch before its first operation: cursors and flags zero, every replica idle at t = 0, every member
// slot free, no element of any joined stream looked at yet.
template <bool DIAG, bool MEMO>
EST_DEV void slot_init(const Pool &p, uint32_t j, uint32_t t, uint32_t slot) {
    const uint32_t ln = wv::lane();
    const EstSimArgs &a = *p.a;
    const EstPlan &P = *a.plan;
    uint32_t *ctl = slot_ctl(p, j), *st = slot_state(p, j);
    const Ctx c = make_ctx(a, t, slot, st, nullptr);
    for (uint32_t i = C_LOCK + 2u * a.n_ops + ln; i < a.ctl_words; i += 64) ctl[i] = 0;
    // (what an operation had seen when it was last entered: a reader of the trace is ready at once)
    for (uint32_t i = ln; i < a.n_ops; i += 64) ctl[C_LOCK + a.n_ops + i] = P.ops[i].from_trace ? 0x80000000u : 0u;
    for (uint64_t i = ln; i < a.rep_stride; i += 64) c.rep[i] = 0;
    wv::sync();
    for (uint32_t opi = 0; opi < a.n_ops; ++opi) {
        const EstOp &op = P.ops[opi];
        if (op.type == EST_OP_SCAN) c.rep[op.rep_off + 128 + ln] = ln;
    }
    {
        uint32_t *tw = (uint32_t *)c.tab;
        for (uint64_t i = ln; i < a.tab_stride / 4; i += 64) tw[i] = 0xFFFFFFFFu;
    }
    uint32_t done = 0;
    uint64_t mr = 0;
    if (MEMO) {
        // Operations this candidate does not run count as done.  In a replay the streams they would have
        // produced are complete already in the captured run of the candidate's base: point the readers
        // there and preset the write cursors to the captured lengths.
        const uint64_t skip = a.skip_ops[t];
        const bool replay = a.cap_rings != nullptr;
        const uint32_t b = replay ? a.base_of[t] : 0u;
        const uint32_t *cs = replay ? a.cap_state + (uint64_t)b * a.cap_state_stride : nullptr;
        for (uint32_t opi = 0; opi < a.n_ops; ++opi) {
            if (!((skip >> opi) & 1ull)) continue;
            const int32_t r = P.ops[opi].out_ring;
            ++done;
            if (replay && r >= 0) {
                mr |= 1ull << r;
                if (ln == 0) {
                    st[P.wr_off + r] = cs[P.wr_off + r];
                    st[P.fin_off + r] = EST_FIN;
                }
            }
        }
    }
    if (ln == 0) {
        ctl[C_T] = t;
        ctl[C_DONE] = done;
        ctl[C_MEMO] = (uint32_t)mr;
        ctl[C_MEMO + 1] = (uint32_t)(mr >> 32);
        if (DIAG && a.dbg_ticks) ctl[C_T0] = (uint32_t)wv::ticks();
        st_st(&ctl[C_PHASE], PH_RUN);
    }
    wv::sync();
    // Last of all the locks, which have stood at "done" since the slot's previous candidate: a wavefront that still takes
    // the slot for that one's finds either nothing to run or the new candidate complete.  It may even finish the new one
    // and empty the slot before this wavefront goes on, so from here on the slot's words are not this wavefront's to write.
    for (uint32_t i = ln; i < a.n_ops; i += 64)
        st_st(&ctl[C_LOCK + i], MEMO && i < 64u && ((a.skip_ops[t] >> i) & 1ull) ? 2u : 0u);
    wv::sync_lds();
}

// Locks an operation of the candidate in slot j that has something new to work on: at least a.quantum elements or the
// end of a stream more than when it was last entered (anything at all while no other operation of the candidate is running).
// Operations are looked at from index `from` on, round and round.  Returns its index, or n_ops.
EST_DEV uint32_t pick_op(const Pool &p, uint32_t j, uint32_t from) {
    const uint32_t ln = wv::lane();
    const EstSimArgs &a = *p.a;
    const uint32_t n_ops = a.n_ops;
    uint32_t *ctl = slot_ctl(p, j);
    const uint32_t *st = slot_state(p, j);
    for (uint32_t base = 0; base < n_ops; base += 64) {
        const uint32_t l = base + ln;
        const bool in = l < n_ops;
        const uint32_t lock = in ? ld_st(&ctl[C_LOCK + l]) : 2u, seen = in ? ld_st(&ctl[C_LOCK + n_ops + l]) : 0u;
        const uint32_t o = in ? p.woff[l] : 0u, k = in ? p.woff[l + 1u] - o : 0u;
        uint32_t sum = 0;
        for (uint32_t i = 0; i < a.max_watch; ++i)
            if (i < k) sum += ld_st(&st[p.watch[o + i]]);
        const uint64_t idle = wv::ballot(lock == 0u);
        uint64_t ready = idle & wv::ballot(sum - seen >= a.quantum);
        if (ready == 0 && wv::ballot(lock == 1u) == 0 && n_ops <= 64u) ready = idle & wv::ballot(sum != seen);
        if (n_ops > 64u) ready = idle & wv::ballot(sum != seen);
        while (ready) {
            const uint64_t later = from > base && from - base < 64u ? ready & ~lanes_below(from - base) : ready;
            const uint32_t i = ctz64(later ? later : ready);
            uint32_t got = 0;
            if (ln == i) {
                work_begin(p);
                got = wv::lds_cas(&ctl[C_LOCK + l], 0u, 1u) == 0u ? 1u : 0u;
                if (got) st_st(&ctl[C_LOCK + n_ops + l], sum);
                else work_cancel(p);
            }
            if (wv::bcast(got, i)) return base + i;
            ready &= ~(1ull << i);
        }
    }
    return n_ops;
}

EST_DEV void select_wave(const EstSimArgs &a, uint32_t t, uint32_t slot, uint32_t miss, uint64_t *lds);

// One step of a wavefront: start a candidate, or run one operation, or find nothing to do.  group: index of the workgroup;
// at: where the search for an operation starts; lds: the wavefront's own area.
template <bool DIAG, bool MEMO>
EST_DEV uint32_t pool_step(const Pool &p, uint32_t group, uint32_t wave, uint32_t &at, uint64_t *lds) {
    const uint32_t ln = wv::lane();
    const EstSimArgs &a = *p.a;
    const uint32_t K = a.per_group, n_ops = a.n_ops;
    const uint32_t home = wave < K ? wave : wave % K;
    if (wave < K && group * K + home < a.n_slots && wv::uniform(ld_st(&slot_ctl(p, home)[C_PHASE])) == PH_EMPTY && wv::uniform(ld_st(&p.gw[G_DRAINED])) == 0u) {
        uint32_t *ctl = slot_ctl(p, home);
        uint32_t t = 0;
        if (ln == 0) {
            work_begin(p);
            st_st(&ctl[C_PHASE], PH_INIT);
            t = wv::fetch_add_u32(&a.status->next_cfg, 1u);
        }
        t = wv::bcast(t, 0);
        if (t >= a.n_cfg) {
            if (ln == 0) {
                st_st(&ctl[C_PHASE], PH_EMPTY);
                st_st(&p.gw[G_DRAINED], 1u);
                work_end(p);
            }
        } else {
            if (MEMO && a.order) t = a.order[t];
            slot_init<DIAG, MEMO>(p, home, t, (MEMO && a.slot_by_cfg) ? t : group * K + home);
            if (ln == 0) work_end(p);
            at = 0;
            if (n_ops > 0) return STEP_WORKED;
        }
    }
    const uint32_t ph = ln < K ? ld_st(&slot_ctl(p, ln)[C_PHASE]) : (uint32_t)PH_EMPTY;
    const uint64_t run = wv::ballot(ph == PH_RUN);
    if (wv::ballot(ph != PH_EMPTY) == 0 && wv::uniform(ld_st(&p.gw[G_DRAINED])) != 0u) return STEP_END;
    uint32_t j = home, opi = n_ops;
    for (uint32_t i = 0; i < K; ++i) {
        j = home + i < K ? home + i : home + i - K;
        if (!((run >> j) & 1ull)) continue;
        opi = pick_op(p, j, i == 0 ? at : 0u);
        if (opi < n_ops || n_ops == 0) break;
    }
    if (opi == n_ops && !(n_ops == 0 && ((run >> home) & 1ull) && wave == home)) return STEP_IDLE;
    wv::sync();  // (what the operation's last runner and its neighbours left)
    uint32_t *ctl = slot_ctl(p, j), *st = slot_state(p, j);
    const uint32_t t = wv::uniform(ld_st(&ctl[C_T]));
    const uint32_t slot = (MEMO && a.slot_by_cfg) ? t : group * K + j;
    bool whole = n_ops == 0;  // the candidate is through
    if (n_ops > 0) {
        Ctx c = make_ctx(a, t, slot, st, lds);
        if (MEMO) {
            c.memo_rings = ((uint64_t)wv::uniform(ctl[C_MEMO + 1]) << 32) | wv::uniform(ctl[C_MEMO]);
            if (a.cap_rings) c.cap_rings = a.cap_rings + (uint64_t)a.base_of[t] * a.cap_ring_stride;
        }
        const EstOp &op = a.plan->ops[opi];
        const uint64_t k0 = (DIAG && a.dbg_ticks) ? wv::ticks() : 0;
        const bool fin = wv::uniform(op.type) == EST_OP_SCAN ? scan_run<DIAG, MEMO>(c, op) : merge_run<DIAG, MEMO>(c, op);
        if (DIAG && a.dbg_ticks && ln == 0) {
            const uint64_t dt = wv::ticks() - k0;
            if (op.type == EST_OP_SCAN) est_dbg_rec(&a, t, op.stage)[1] += dt;
            else wv::atomic_add_u64(&est_dbg_rec(&a, t, EST_MAX_STAGES - 1)[op.type == EST_OP_LAT ? 1 : 0], dt);
        }
        wv::sync();  // (everything the operation leaves is in place before somebody else may enter it)
        uint32_t nd = 0;
        if (ln == 0) {
            if (fin) nd = wv::lds_fetch_add(&ctl[C_DONE], 1u) + 1u;
            st_st(&ctl[C_LOCK + opi], fin ? 2u : 0u);
        }
        whole = fin && wv::bcast(nd, 0) == n_ops;
        at = opi + 1u < n_ops ? opi + 1u : 0u;
    }
    if (whole) {
        wv::sync();
        const uint64_t k1 = (DIAG && a.dbg_ticks) ? wv::ticks() : 0;
        if (MEMO && a.slot_by_cfg)  // a captured run: its stream lengths stay with it
            for (uint32_t i = ln; i < a.plan->state_words; i += 64) a.state[(uint64_t)slot * a.state_stride + i] = st[i];
        if (!a.lat_by_qid) select_wave(a, t, slot, a.n > 0 ? wv::uniform(ld_st(&st[a.plan->miss_off])) : 0u, lds);
        if (DIAG && a.dbg_ticks && ln == 0) {
            wv::atomic_add_u64(&est_dbg_rec(&a, t, EST_MAX_STAGES - 1)[2], wv::ticks() - k1);
            a.dbg_ticks[t] = (uint32_t)wv::ticks() - ctl[C_T0];
        }
        wv::sync();
        if (ln == 0) st_st(&ctl[C_PHASE], PH_EMPTY);
    }
    if (ln == 0 && n_ops > 0) work_end(p);
    return STEP_WORKED;
}

// ------------------------------------------------------------------------------------------ P99

// Nearest-rank P99 of one candidate's latencies by a 4-pass radix select (8 bits per pass), one
// wavefront per candidate, plus the candidate's cost = sum over stages of replicas x price
// (Section 6, cost model).
EST_DEV void select_wave(const EstSimArgs &a, uint32_t t, uint32_t slot, uint32_t miss, uint64_t *lds) {
    const uint32_t ln = wv::lane();
    const EstStageCfg *cfg = a.cfg + (uint64_t)t * a.dag->S;
    if (ln == 0) {
        uint64_t cost = 0;
        for (uint32_t s = 0; s < a.dag->S; ++s)
            cost += (uint64_t)cfg[s].replicas * a.cost_uusd_hr[(uint64_t)s * a.dag->H + cfg[s].hw];
        a.cost[t] = cost;
    }
    if (!a.have_lat) return;
    const uint32_t *lat = a.lat + (uint64_t)slot * a.lat_stride;
    uint32_t *hist = (uint32_t *)lds;  // 256 bins
    const uint32_t n = a.n;
    uint32_t k = (uint32_t)(((uint64_t)99 * n + 99) / 100);  // 1-based rank, ceil(0.99 n)
    uint32_t prefix = 0;
    for (int pass = 3; pass >= 0; --pass) {
        const uint32_t shift = (uint32_t)pass * 8;
        for (uint32_t i = ln; i < 256; i += 64) hist[i] = 0;
        wv::sync_lds();
        for (uint32_t i0 = 0; i0 < n; i0 += 512) {  // eight loads in flight per lane
            uint32_t v[8];
EST_UNROLL
            for (uint32_t u = 0; u < 8; ++u) {
                const uint32_t i = i0 + u * 64u + ln;
                v[u] = i < n ? lat[i] : 0u;
            }
EST_UNROLL
            for (uint32_t u = 0; u < 8; ++u) {
                const bool match = i0 + u * 64u + ln < n && (pass == 3 || (v[u] >> (shift + 8)) == (prefix >> (shift + 8)));
                if (match) wv::lds_add(&hist[(v[u] >> shift) & 255u], 1u);
            }
        }
        wv::sync_lds();
        // lane l owns bins 4l .. 4l+3
        const uint32_t h0 = hist[4 * ln], h1 = hist[4 * ln + 1], h2 = hist[4 * ln + 2], h3 = hist[4 * ln + 3];
        const uint32_t mine = h0 + h1 + h2 + h3;
        const uint32_t before = wv::prefix_excl_u32(mine);
        const uint64_t hit = wv::ballot(before < k && k <= before + mine);
        EST_CHECK(popc64(hit) == 1);
        const uint32_t hl = ctz64(hit);
        uint32_t digit = 0, kk = 0;
        if (ln == hl) {
            uint32_t r = k - before;  // rank inside my four bins
            if (r <= h0) { digit = 4 * ln; kk = r; }
            else if (r <= h0 + h1) { digit = 4 * ln + 1; kk = r - h0; }
            else if (r <= h0 + h1 + h2) { digit = 4 * ln + 2; kk = r - h0 - h1; }
            else { digit = 4 * ln + 3; kk = r - h0 - h1 - h2; }
        }
        digit = wv::bcast(digit, hl);
        k = wv::bcast(kk, hl);
        prefix |= digit << shift;
        wv::sync_lds();
    }
    if (ln == 0) {
        a.p99[t] = prefix;
        a.miss[t] = miss;
    }
}

// ------------------------------------------------------------------------------------------ preprocessing

// Nearest visited ancestors of every stage (and of the virtual sink, index S) for one query:
// bit p = the completion of stage p feeds the stage directly, bit EST_TRACE_BIT = the arrival does.
// A member that is an ancestor of another member is left out: times never decrease along a path of the
// pipeline (a skipped stage passes its ready time on), so its completion is no later than the other's and never
// decides the maximum (Section 4.1, conditional control flow: a query that takes one branch of a fork and skips
// the other is fed by that branch alone, not also by the stage before the fork).
EST_DEV void nearest_sets(const EstDag &d, uint32_t mask, uint64_t *nv) {
    uint64_t anc[EST_MAX_STAGES + 1];  // every ancestor of the stage, and the arrival
    for (uint32_t c = 0; c <= d.S; ++c) {
        uint64_t s = 0, a = 1ull << EST_TRACE_BIT;
        const uint32_t b = d.parent_off[c], e = d.parent_off[c + 1];
        if (b == e) s = 1ull << EST_TRACE_BIT;
        for (uint32_t i = b; i < e; ++i) {
            const uint32_t p = d.parent_idx[i];
            s |= ((mask >> p) & 1u) ? (1ull << p) : nv[p];
            a |= (1ull << p) | anc[p];
        }
        uint64_t dominated = 0;
        for (uint64_t t = s & ~(1ull << EST_TRACE_BIT); t; t &= t - 1) dominated |= anc[__builtin_ctzll(t)];
        nv[c] = s & ~dominated;
        anc[c] = a;
    }
}

// Pass 1 over the trace (thread tid of nthreads, strided): monotonicity, per-stage source unions,
// visit counts.
EST_DEV void prep1_thread(const EstPrepArgs &a, uint32_t tid, uint32_t nthreads) {
    const EstDag &d = *a.dag;
    uint64_t uni[EST_MAX_STAGES + 1], muni[EST_MAX_STAGES + 1];
    uint32_t cntv[EST_MAX_STAGES + 1];
    uint64_t multi = 0;  // bit c: some visiting query of stage c has more than one nearest visited ancestor
    bool bad = false;
    for (uint32_t c = 0; c <= d.S; ++c) { uni[c] = 0; muni[c] = 0; cntv[c] = 0; }
    for (uint64_t q = tid; q < a.n; q += nthreads) {
        const uint32_t m = a.mask[q];
        if (q > 0 && a.arrival[q] < a.arrival[q - 1]) bad = true;
        uint64_t nv[EST_MAX_STAGES + 1];
        nearest_sets(d, m, nv);
        for (uint32_t c = 0; c <= d.S; ++c) {
            if (c < d.S && !((m >> c) & 1u)) continue;
            uni[c] |= nv[c];
            cntv[c]++;
            if (__builtin_popcountll(nv[c]) > 1) {
                multi |= 1ull << c;
                muni[c] |= nv[c];
            }
        }
    }
    for (uint32_t c = 0; c <= d.S; ++c) {
        if (cntv[c]) {
            wv::atomic_or_u64(&a.status->src_union[c], uni[c]);
            wv::atomic_add_u32(&a.status->n_visit[c], cntv[c]);
            if ((multi >> c) & 1ull) {
                wv::atomic_or_u32(&a.status->multi[c], 1u);
                wv::atomic_or_u64(&a.status->multi_union[c], muni[c]);
            }
        }
    }
    if (bad) wv::atomic_or_u32(&a.status->bad_trace, 1u);
    if (tid == 0 && a.n > 0) a.status->last_arrival = a.arrival[a.n - 1];
}

// Pass 2: the key stream of the trace, and for every merge operation the per-query accept mask:
// bit j set = source j of the operation is one of the query's nearest visited ancestors.
EST_DEV void prep2_thread(const EstPrepArgs &a, uint32_t tid, uint32_t nthreads) {
    const EstDag &d = *a.dag;
    for (uint64_t q = tid; q < a.n; q += nthreads) {
        const uint32_t m = a.mask[q];
        a.trace_keys[q] = ((uint64_t)a.arrival[q] << 32) | q;
        uint64_t nv[EST_MAX_STAGES + 1];
        nearest_sets(d, m, nv);
        for (uint32_t i = 0; i < a.n_acc; ++i) {
            const uint32_t c = a.acc_stage[i];
            uint8_t bits = 0;
            if (c == d.S || ((m >> c) & 1u)) {
                for (uint64_t s = nv[c]; s; s &= s - 1) {
                    const uint32_t src = (uint32_t)__builtin_ctzll(s);
                    bits |= (uint8_t)(1u << a.acc_slot_of_src[c][src]);
                }
            }
            a.acc[(uint64_t)i * a.acc_stride + q] = bits;
        }
    }
}

// Range check of every configuration entry and the per-stage maxima that size the scratch.
EST_DEV void cfg_thread(const EstCfgArgs &a, uint32_t tid, uint32_t nthreads) {
    const EstDag &d = *a.dag;
    uint32_t rmax[EST_MAX_STAGES], bmax[EST_MAX_STAGES];
    bool bad = false;
    for (uint32_t s = 0; s < d.S; ++s) { rmax[s] = 0; bmax[s] = 0; }
    for (uint64_t i = tid; i < a.n_cfg; i += nthreads) {
        for (uint32_t s = 0; s < d.S; ++s) {
            const EstStageCfg e = a.cfg[i * d.S + s];
            if (e.hw >= d.H || e.batch < 1 || e.batch > d.Bmax || e.replicas < 1 || e.replicas > EST_MAX_REPLICAS) bad = true;
            rmax[s] = umax(rmax[s], e.replicas);
            bmax[s] = umax(bmax[s], e.batch);
        }
    }
    for (uint32_t s = 0; s < d.S; ++s) {
        if (rmax[s]) wv::atomic_max_u32(&a.status->r_max[s], rmax[s]);
        if (bmax[s]) wv::atomic_max_u32(&a.status->b_max[s], bmax[s]);
    }
    if (bad) wv::atomic_or_u32(&a.status->bad_cfg, 1u);
}

// Traffic envelope of the trace (Section 5, "traffic envelopes"): for every window width the largest
// number of arrivals in any half-open window [t, t + width).  The maximum is attained by a window
// that starts at an arrival.  One wavefront takes one width and the queries [j0, j1), 64 at a time: lane l the window
// that starts at query j0 + l.  Window ends ascend with the query, so the end of the block before bounds the block's from
// below, and the end of its last window, found by the whole wavefront (64 probes at a time, first a growing distance
// apart, then ever closer), bounds them from above; between the two every lane bisects.
// What bounds it are dependent loads, about ten per block of 64 windows, and how many wavefronts wait for theirs at the same
// time: all widths at once are some ten thousand.  (With a thread per 16 consecutive queries, which searched for its first
// window of every width and moved the ends on one arrival at a time, 2 x 10^6 arrivals and 10 widths took 0.62 ms; now 0.45 ms.  The whole
// call 3.67 -> 1.46 ms.)

// First index in [lo, n) whose arrival is at or after limit, n if there is none; lo and limit the same in every lane.
EST_DEV uint32_t first_at_or_after(const uint32_t *arrival, uint32_t n, uint32_t lo, uint64_t limit) {
    const uint32_t ln = wv::lane();
    uint32_t shift = 0;  // probes are 2^shift apart; everything below lo is before the limit
    for (;;) {
        const uint64_t at = (uint64_t)lo + (((uint64_t)ln + 1u) << shift) - 1u;
        const bool before = at < n && (uint64_t)arrival[at < n ? at : n - 1u] < limit;
        const uint32_t k = popc64(wv::ballot(before));  // (a prefix of the lanes: arrivals ascend)
        lo += k << shift;
        if (k < 64u) {  // the answer is within 2^shift elements from lo
            if (shift == 0u) return lo;
            shift = shift > 6u ? shift - 6u : 0u;
        } else if (shift < 24u) {
            shift += 6u;
        }
    }
}

EST_DEV void envelope_wave(const EstEnvArgs &a, uint32_t win, uint32_t j0, uint32_t j1) {
    const uint32_t ln = wv::lane(), n = (uint32_t)a.n;
    const uint64_t width = a.win_us[win];
    uint32_t best = 0, end = j0;
    for (uint32_t j = j0; j < j1; j += 64) {
        const uint32_t m = umin(64u, j1 - j), mine = j + umin(ln, m - 1u);
        const uint64_t limit = (uint64_t)a.arrival[mine] + width;
        const uint64_t top = (uint64_t)a.arrival[j + m - 1u] + width;
        uint32_t lo = umax(end, mine + 1u);  // (a window holds the arrival it starts at)
        end = first_at_or_after(a.arrival, n, umax(end, j + m), top);
        uint32_t hi = end;
        while (wv::ballot(lo < hi)) {
            const uint32_t mid = lo + ((hi - lo) >> 1);
            const bool before = lo < hi && (uint64_t)a.arrival[mid] < limit;
            if (lo < hi) { if (before) lo = mid + 1u; else hi = mid; }
        }
        best = umax(best, lo - mine);
    }
    best = wv::max_u32(best);
    if (ln == 0 && best > a.max_queries[win]) wv::atomic_max_u32(&a.max_queries[win], best);
}

}  // namespace estdev
