// fused.h -- the persistent fused kernel (paper Section 3.2 and Section 4.1
// "Fused kernel composition"): each workgroup claims (plan, mini-block range)
// work items from a device queue; its waves each take one 256-row mini block
// at a time, decode the referenced columns straight from where the chunks
// rest (HBM or pinned host memory mapped into the device), filter, and queue
// the surviving row ids in LDS; full batches of 64 survivors are probed
// against the dimension hash tables (LDS copies for small ones) and
// aggregated into a per-workgroup LDS table.  The last workgroup to finish
// writes the records to the host buffer -- nothing is materialised in
// between (group tables above kEmitEntries entries go out through emit_kernel).
#pragma once
#include "device.h"

namespace dpf {
namespace {

// ---------------------------------------------------------------------------
// Stage B: probes, value loads and aggregation of one row per lane.  m and i
// may differ between lanes (rows queued from several mini blocks).  gagg is
// the plan's group table in device memory.
// ---------------------------------------------------------------------------
template <bool kHash>
__device__ __forceinline__ void stage_b(CQ& Q, uint8_t* smem_shared, unsigned long long* gagg, LdsSlots sv, int m,
                                        int i, bool active, bool& ok_hdr) {
    bool ok = active;
    const int nprobes = Q.nprobes;
    for (int j = 0; j < nprobes; ++j) {
        if (__ballot(ok) == 0) return;
        CPR& P = Q.probes[j];
        if (ok) {
            CC& fc = Q.cols[P.fk_col];
            int64_t fk = decode_at(fc, m, i, ok_hdr);
            if (fc.enc == ENC_DICT) fk = dict_value(fc, fk, ok_hdr);
            if (fk < INT32_MIN || fk > INT32_MAX || !filter_maybe(P.h, smem_shared, fk)) {
                ok = false;  // certainly absent
                continue;
            }
            // The key-range bitmap answers membership exactly: it settles a
            // probe that needs no payload, and keeps non-members (most rows
            // of a selective join) away from the hash table's random reads.
            if (P.h.bits) {
                if (!bitmap_has(P.h, smem_shared, fk)) {
                    ok = false;
                    continue;
                }
                if (P.pay_slot[0] < 0 && P.pay_slot[1] < 0) continue;
            }
            const bool lds = P.h.lds_off >= 0;
            int slot = lds ? hash_find<true>(P.h, smem_shared, fk) : hash_find<false>(P.h, smem_shared, fk);
            ok = slot >= 0;
            if (ok) {
                for (int k = 0; k < P.h.npay; ++k) {
                    if (P.pay_slot[k] < 0) continue;
                    int64_t pv = lds ? hash_payload<true>(P.h, smem_shared, k, slot)
                                     : hash_payload<false>(P.h, smem_shared, k, slot);
                    sv.set(P.pay_slot[k], pv);
                }
            }
        }
    }
    if (!ok) return;
    // Fact values for slots 0..nloads-1, two slots at a time: the group's
    // loads go out in three rounds (mini-block headers, packed words,
    // dictionary entries), so that a flush waits for memory three times a
    // group rather than three times a slot; a DELTA column (a running sum)
    // decodes on its own.
    const int nloads = Q.nloads;
    constexpr int kGrp = 2;
#pragma unroll 1
    for (int g0 = 0; g0 < nloads; g0 += kGrp) {
        uint32_t w0[kGrp], w1[kGrp];
        int64_t base[kGrp];
#pragma unroll
        for (int k = 0; k < kGrp; ++k) {
            if (g0 + k < nloads) {
                CC& c = Q.cols[Q.loads[g0 + k].col];
                w0[k] = ro(c.woff)[m];
                w1[k] = ro(c.woff)[m + 1];
                base[k] = ro(c.base)[m];
            }
        }
        uint64_t u[kGrp];
#pragma unroll
        for (int k = 0; k < kGrp; ++k) {
            if (g0 + k < nloads) {
                CC& c = Q.cols[Q.loads[g0 + k].col];
                if (c.enc == ENC_DELTA) {
                    u[k] = (uint64_t)decode_at(c, m, i, ok_hdr);
                } else {
                    // the checks of mb_hdr: a corrupt header must not steer a load
                    const uint32_t nw = w1[k] - w0[k];
                    const bool hok = (w0[k] <= w1[k]) && (w1[k] <= c.nwords) && ((nw & 7u) == 0) && (nw <= 512u);
                    ok_hdr = ok_hdr && hok;
                    const int b = hok ? (int)(nw >> 3) : 0;
                    u[k] = (uint64_t)base[k] +
                           (b ? bits_at(ro(c.words) + (hok ? w0[k] : 0u), (uint32_t)i * (uint32_t)b, b) : 0);
                }
            }
        }
#pragma unroll
        for (int k = 0; k < kGrp; ++k) {
            if (g0 + k < nloads) {
                CL& Ld = Q.loads[g0 + k];
                int64_t x = (int64_t)u[k];
                if (Ld.dict_val) x = dict_value(Q.cols[Ld.col], x, ok_hdr);
                sv.set(g0 + k, x);
            }
        }
    }
    int64_t g;
    if (!group_index(Q, sv, g)) { ok_hdr = false; return; }
    if (!aggregate_row<kHash>(Q, smem_shared, gagg, sv, g)) ok_hdr = false;
}

// ---------------------------------------------------------------------------
// One mini block of one plan, by one wave (stage A), survivors queued
// ---------------------------------------------------------------------------
struct WaveArea {
    const uint32_t* tab;  // [32] the workgroup's string-scan table
    uint32_t* pend;    // [kPendCap] queued surviving row ids
    int64_t* slots;    // [kMaxSlots][kWave] stage-B values
    uint32_t* offs;    // [260] string row offsets
    uint32_t* first1;  // [256] leftmost s1 start per row
    uint32_t* last2;   // [256] rightmost s2 start + 1 per row
    uint4* recs;       // [kRecCap] string words with a prefix hit
};

template <bool kHash>
__device__ __forceinline__ void flush_pending(CQ& Q, uint8_t* smem_shared, unsigned long long* gagg, const WaveArea& W,
                                              int& npend, int lane, bool& ok_hdr) {
    wave_lds_sync();
    for (int base = 0; base < npend; base += kWave) {
        int idx = base + lane;
        bool act = idx < npend;
        uint32_t row = W.pend[act ? idx : 0];
        stage_b<kHash>(Q, smem_shared, gagg, LdsSlots{W.slots + lane}, (int)(row >> 8), (int)(row & 255u), act,
                       ok_hdr);
    }
    npend = 0;
    wave_lds_sync();
}

template <bool kHash>
__device__ __forceinline__ void queue_survivors(CQ& Q, uint8_t* smem_shared, unsigned long long* gagg, const WaveArea& W,
                                                int64_t row0, uint32_t mask, int lane, int& npend, bool& ok_hdr) {
    if (__ballot(mask != 0) == 0) return;
    // Queue survivors (wave ballot + mbcnt compaction).
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        bool bit = (mask >> k) & 1u;
        uint64_t b = __ballot(bit);
        if (bit) W.pend[npend + bits_below(b)] = (uint32_t)(row0 + 64 * k + lane);
        npend += (int)__popcll(b);
    }
    if (npend >= kWave) flush_pending<kHash>(Q, smem_shared, gagg, W, npend, lane, ok_hdr);
}

// Stage A of mini block m: returns the mask of rows passing every atom (row
// 64 k + lane -> bit k).  kEager: the plan's one string atom comes last and
// its loads are issued before the integer atoms run, so both wait for memory
// once, together.
template <bool kEager, int kStr>
__device__ __forceinline__ uint32_t filter_tile(CQ& Q, const uint8_t* smem_shared, const WaveArea& W, int m, int lane,
                                                int nvalid, bool& ok_hdr) {
    uint32_t mask = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) mask |= (uint32_t)(64 * k + lane < nvalid) << k;
    const StrLds L{W.tab, W.offs, W.first1, W.last2, W.recs};
    const int npreds = Q.npreds;
    CP& PL = Q.preds[npreds - 1];
    StrTile S;
    if (kEager) str_begin(Q.cols[PL.col], m, lane, S);
    int64_t v[4];
    int last_col = -1;
    for (int a = 0; a < (kEager ? npreds - 1 : npreds); ++a) {
        CP& P = Q.preds[a];
        if (!kEager && P.kind == PK_STR) {
            if (!kStr) {
                ok_hdr = false;  // unreachable: the launch picks the string instantiation
                return 0;
            } else if (kStr == 2 && Q.cols[P.col].enc == ENC_FSST) {
                mask &= fsst_pred(Q, Q.cols[P.col], m, lane, nvalid, reinterpret_cast<uint8_t*>(W.offs), smem_shared,
                                  ok_hdr);
            } else {
                // (the table is loaded for the plan's last atom only)
                if (str_mode(P.n1, P.n2) == kStrShifted)
                    mask &= str_pred<kStrShifted>(Q.cols[P.col], P, m, lane, nvalid, L, ok_hdr);
                else
                    mask &= str_pred<kStrMasked>(Q.cols[P.col], P, m, lane, nvalid, L, ok_hdr);
            }
        } else {
            const int z = zone_test(Q.cols[P.col], P, m);
            if (z == 1) continue;
            if (z == 0) return 0;
            if (P.col != last_col) {
                ok_hdr &= decode_dense(Q.cols[P.col], m, lane, v);
                last_col = P.col;
            }
            mask &= eval_int_pred(P, Q.in_vals, v);
        }
        if (__ballot(mask != 0) == 0) return 0;  // no survivor in this mini block
    }
    if (kEager) {
        const int mode = PL.tab_rot ? kStrTable : str_mode(PL.n1, PL.n2);
        if (mode == kStrTable)
            mask &= str_finish<kStrTable>(Q.cols[PL.col], PL, lane, nvalid, S, L, ok_hdr);
        else if (mode == kStrShifted)
            mask &= str_finish<kStrShifted>(Q.cols[PL.col], PL, lane, nvalid, S, L, ok_hdr);
        else
            mask &= str_finish<kStrMasked>(Q.cols[PL.col], PL, lane, nvalid, S, L, ok_hdr);
    }
    return mask;
}

// Rows of mask (row 64 k + lane -> bit k) of mini block m whose first
// probe finds its key.
__device__ __forceinline__ uint32_t member_tile(CQ& Q, const uint8_t* smem_shared, int m, int lane, uint32_t mask,
                                                bool& ok_hdr) {
    CPR& P0 = Q.probes[0];
    CC& fc = Q.cols[P0.fk_col];
    int64_t fk[4];
    ok_hdr &= decode_dense(fc, m, lane, fk);
    if (fc.enc == ENC_DICT)
#pragma unroll
        for (int k = 0; k < 4; ++k) fk[k] = (mask >> k) & 1u ? dict_value(fc, fk[k], ok_hdr) : 0;
    return P0.h.lds_off >= 0 ? hash_member4<true>(P0.h, smem_shared, fk, mask)
                             : hash_member4<false>(P0.h, smem_shared, fk, mask);
}

template <int kStr, bool kHash>
__device__ __forceinline__ void process_tile(CQ& Q, uint8_t* smem_shared, unsigned long long* gagg, const WaveArea& W,
                                             int m, int lane, int& npend, bool& ok_hdr) {
    const int64_t row0 = (int64_t)m * kMB;
    const int nvalid = (int)min((int64_t)kMB, Q.nrows - row0);
    const int npreds = Q.npreds;

    if (npreds == 0 && Q.nprobes == 0) {
        // Neither a fact predicate nor a join: every valid row goes straight
        // to stage B.
        for (int k = 0; k < 4; ++k) {
            if (64 * k >= nvalid) break;
            int i = 64 * k + lane;
            stage_b<kHash>(Q, smem_shared, gagg, LdsSlots{W.slots + lane}, m, i, i < nvalid, ok_hdr);
        }
        return;
    }
    if (npreds == 0) return;  // probes without predicates: semi_tiles handles those plans
    // (an FSST atom is never the eager one: its plan has fs_pred >= 0)
    uint32_t mask =
        Q.nint_preds == npreds - 1 && Q.preds[npreds - 1].kind == PK_STR && Q.fs_pred < 0
            ? (kStr ? filter_tile<true, kStr>(Q, smem_shared, W, m, lane, nvalid, ok_hdr) : (ok_hdr = false, 0u))
            : filter_tile<false, kStr>(Q, smem_shared, W, m, lane, nvalid, ok_hdr);
    // The first (most selective) probe's membership test joins stage A: its
    // foreign keys are decoded for the whole mini block with coalesced
    // loads, so stage B gets only the rows that find their key (and probes
    // them again for payloads), not every row that passed the filters.
    if (Q.nprobes > 0 && __ballot(mask != 0)) mask = member_tile(Q, smem_shared, m, lane, mask, ok_hdr);
    queue_survivors<kHash>(Q, smem_shared, gagg, W, row0, mask, lane, npend, ok_hdr);
}

// Semi-join stage A of one mini block whose foreign keys issue_dense read:
// the first (most selective) probe filters; its survivors are probed again,
// with payloads, in stage B.
template <bool kHash>
__device__ __forceinline__ void semi_tile(CQ& Q, uint8_t* smem_shared, unsigned long long* gagg, const WaveArea& W,
                                          int m, int lane, const RawDense& R, int& npend, bool& ok_hdr) {
    const int64_t row0 = (int64_t)m * kMB;
    const int nvalid = (int)min((int64_t)kMB, Q.nrows - row0);
    uint32_t mask = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) mask |= (uint32_t)(64 * k + lane < nvalid) << k;
    CPR& P0 = Q.probes[0];
    CC& fc = Q.cols[P0.fk_col];
    int64_t fk[4];
    ok_hdr &= finish_dense(fc, R, lane, fk);
    if (fc.enc == ENC_DICT)
#pragma unroll
        for (int k = 0; k < 4; ++k) fk[k] = (mask >> k) & 1u ? dict_value(fc, fk[k], ok_hdr) : 0;
    mask = P0.h.lds_off >= 0 ? hash_member4<true>(P0.h, smem_shared, fk, mask)
                             : hash_member4<false>(P0.h, smem_shared, fk, mask);
    queue_survivors<kHash>(Q, smem_shared, gagg, W, row0, mask, lane, npend, ok_hdr);
}

// The semi-join tiles m0, m0 + nw, ... < m1 of one wave, two in flight: the
// next tile's keys are loaded while the current one is probed.
template <bool kHash>
__device__ __forceinline__ void semi_tiles(CQ& Q, uint8_t* smem_shared, unsigned long long* gagg, const WaveArea& W,
                                           int m0, int m1, int nw, int lane, int& npend, bool& ok_hdr) {
    CC& fc = Q.cols[Q.probes[0].fk_col];
    RawDense A, B;
    if (m0 < m1) issue_dense(fc, m0, lane, A);
    for (int m = m0; m < m1; m += 2 * nw) {
        const int m2 = m + nw;
        dense_ready(A);  // as seg_ready: wait for A before B's loads are issued
        if (m2 < m1) issue_dense(fc, m2, lane, B);
        semi_tile<kHash>(Q, smem_shared, gagg, W, m, lane, A, npend, ok_hdr);
        if (m2 >= m1) break;
        dense_ready(B);
        if (m2 + nw < m1) issue_dense(fc, m2 + nw, lane, A);
        semi_tile<kHash>(Q, smem_shared, gagg, W, m2, lane, B, npend, ok_hdr);
    }
}


// Per-wave LDS: (plans with fact predicates) the survivor queue, then one
// region shared by the stage-B value slots and the string predicate's row
// offsets, s1 / s2 starts and hit queue -- a wave never uses both at once
// (a mini block's string test finishes before its survivors are queued).
constexpr size_t kSlotBytes = kMaxSlots * kWave * 8;
constexpr size_t kStrBytes = 260 * 4 + 2 * 256 * 4 + kRecCap * 16;

__host__ __device__ constexpr size_t wave_area_bytes(bool str_stage, bool pend_stage) {
    return (pend_stage ? kPendCap * 4 : 0) + (str_stage && kStrBytes > kSlotBytes ? kStrBytes : kSlotBytes);
}

__device__ __forceinline__ WaveArea wave_area(uint8_t* p, const uint32_t* tab, bool pend_stage) {
    WaveArea W;
    W.tab = tab;
    W.pend = reinterpret_cast<uint32_t*>(p);
    uint8_t* shared = p + (pend_stage ? kPendCap * 4 : 0);
    W.slots = reinterpret_cast<int64_t*>(shared);
    W.offs = reinterpret_cast<uint32_t*>(shared);
    W.first1 = W.offs + 260;
    W.last2 = W.first1 + 256;
    W.recs = reinterpret_cast<uint4*>(W.last2 + 256);
    return W;
}

// Merge the workgroup's LDS group table into the plan's global table.  The
// device-scope adds return their old values, which the caller folds into a
// sink: once the sink is known the adds have been performed.
__device__ unsigned long long flush_lds_agg(CQ& Q, uint8_t* smem_shared, unsigned long long* gagg) {
    if (!Q.agg_lds) return 0;
    const int64_t n = Q.ngroups * Q.nacc;
    unsigned long long* T = reinterpret_cast<unsigned long long*>(smem_shared + Q.agg_lds_off);
    unsigned long long sink = 0;
    for (int64_t e = threadIdx.x; e < n; e += blockDim.x) {
        unsigned long long x = T[e];
        if (x) sink += atomicAdd(gagg + e, x);
        T[e] = 0;
    }
    return sink;
}

// Load a plan's LDS-resident dimension tables.
__device__ __forceinline__ void load_lds_tables(CQ& Q, uint8_t* smem_shared) {
    for (int j = 0; j < Q.nprobes; ++j) {
        CH& h = Q.probes[j].h;
        if (h.bits_lds_off >= 0) {
            cptr<uint4> src = (cptr<uint4>)h.bits;
            uint4* dst = reinterpret_cast<uint4*>(smem_shared + h.bits_lds_off);
            const uint32_t n = (uint32_t)((h.bspan + 127) / 128);  // 16-byte units
            for (uint32_t e = threadIdx.x; e < n; e += blockDim.x) dst[e] = ld4(src, e);
        }
        if (h.filt_lds_off >= 0) {
            cptr<uint4> src = (cptr<uint4>)h.filt;
            uint4* dst = reinterpret_cast<uint4*>(smem_shared + h.filt_lds_off);
            const uint32_t n = (1u << h.flog2) / 128u;  // 16-byte units
            for (uint32_t e = threadIdx.x; e < n; e += blockDim.x) dst[e] = ld4(src, e);
        }
        if (h.lds_off < 0) continue;
        cptr<uint4> src = (cptr<uint4>)h.keys;
        uint4* dst = reinterpret_cast<uint4*>(smem_shared + h.lds_off);
        for (uint32_t e = threadIdx.x; e < h.bytes / 16u; e += blockDim.x) dst[e] = ld4(src, e);
    }
}

// The plan's whole LDS state: string table, dimension tables, a cleared group
// table.
__device__ void load_lds_state(CQ& Q, uint8_t* smem_shared, uint32_t* str_tab) {
    if (Q.npreds > 0 && threadIdx.x < 32) {
        CP& PL = Q.preds[Q.npreds - 1];
        if (PL.kind == PK_STR && PL.tab_rot) str_tab[threadIdx.x] = PL.tab[threadIdx.x];
    }
    load_lds_tables(Q, smem_shared);
    if (Q.agg_lds) {
        const int64_t n = Q.ngroups * Q.nacc;
        unsigned long long* T = reinterpret_cast<unsigned long long*>(smem_shared + Q.agg_lds_off);
        for (int64_t e = threadIdx.x; e < n; e += blockDim.x) T[e] = 0;
    }
}

// ---------------------------------------------------------------------------
// Work queue.  Workgroup i runs on XCD i % 8 (round-robin dispatch), and each
// XCD has its own L2, so a single queue head would serialise every claim of
// the grid on one device-coherent atomic.  Instead the items are split into
// eight contiguous ranges with one head each: a workgroup takes items of
// its XCD's range, then of the others.  Completion counts per XCD and then across XCDs.
// The dispatch rule only affects speed: any workgroup may take any item.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t* ctr(const BatchArgs& a, int i) { return a.counters + i * kCounterStride; }

// A claim, by one whole wave: n(x) items in XCD x's range.  Returns the item's
// place in its range x, -1 when all are taken.  A workgroup's first item is its
// place among those homed on its XCD; those after the last workgroup's are
// claimed.  (Claims on one head are served one at a time, about 0.1 us each: 5M
// comments, an item a workgroup, took 99 us with first items claimed too, 93
// without.)  Then the other ranges.  A lone plan with a few items a workgroup
// reads the heads of all that are left together: one after the other they kept
// every workgroup for seven waits at the launch's end (40,000 rows: 40.3 us,
// now 38.0).  With many items (a.walk) ranges end at different times, and a
// workgroup looks for the next one often: there one head a look, or the reads
// hold up the claims (two scans of 2.2M rows and four joins over 1M in one
// batch: 113 us together, 99 so).
template <class N>
__device__ __forceinline__ int claim(const BatchArgs& a, int home, uint32_t& drained, bool first, int lane, N n, int& x) {
    auto given = [&](int y) { return (int)gridDim.x > y ? (int)((gridDim.x - 1u - (uint32_t)y) / kXcds + 1u) : 0; };
    auto left = [&](int y) { return (uint32_t)max((int)n(y) - given(y), 0); };  // to be claimed
    x = home;
    if (first && blockIdx.x / kXcds < n(home)) return (int)(blockIdx.x / kXcds);
    for (;;) {
        if (!((drained >> x) & 1u) && left(x) > 0) {
            uint32_t j = 0;
            if (lane == 0) j = atomicAdd(ctr(a, x), 1u);
            j = (uint32_t)__builtin_amdgcn_readfirstlane((int)j);
            if (j < left(x)) return (int)j + given(x);
        }
        drained |= 1u << x;
        const uint32_t rest = ~drained & ((1u << kXcds) - 1u);
        if (rest == 0) return -1;
        const uint32_t from = (rest >> home) | (rest << (kXcds - home));
        x = (home + __builtin_ctz(from)) & (kXcds - 1);  // the next after home
        const uint32_t look = a.walk ? 1u << x : rest;
        uint32_t h = ~0u;
        if (lane < kXcds && ((look >> lane) & 1u))
            h = __hip_atomic_load(ctr(a, lane), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        drained |= look & ~(uint32_t)__ballot(h < left(lane & (kXcds - 1)));  // (x itself: the next turn passes it by)
    }
}

__device__ __forceinline__ int claim_item(const BatchArgs& a, int home, uint32_t& drained, bool first, int lane, int total) {
    int x;
    auto start = [&](int y) { return (uint32_t)((int64_t)total * y / kXcds); };
    const int j = claim(a, home, drained, first, lane, [&](int y) { return start(y + 1) - start(y); }, x);
    return j < 0 ? -1 : (int)start(x) + j;
}

// Claims of a lone plan: each XCD's eighth of its mini blocks (a pruned plan's:
// of its surviving blocks') is cut into large items and, at its end, small ones
// so that all workgroups end together (24M-row summary: 185 us with one size,
// 179 so).  Every XCD has the same items; the last ones' may be empty.  False:
// none left.
__device__ __forceinline__ bool claim_guided(const BatchArgs& a, int home, uint32_t& drained, bool first, int lane, int& mb0,
                                             int& mb1) {
    int x;
    const int j = claim(a, home, drained, first, lane, [&](int) { return (uint32_t)a.xcd_items; }, x);
    if (j < 0) return false;
    const bool big = j < a.xcd_big;
    mb0 = x * a.xcd_mb + (big ? j * a.mb_per_item : a.xcd_big * a.mb_per_item + (j - a.xcd_big) * a.small_mb);
    mb1 = min(mb0 + (big ? a.mb_per_item : a.small_mb), min((x + 1) * a.xcd_mb, a.guided_mb));
    return true;
}

// The workgroup's next item: its number (-1: none), and of a guided one its mini
// blocks.
template <bool kGuided>
__device__ __forceinline__ void next_item(const BatchArgs& a, int32_t* ctrl, int home, uint32_t& drained, bool first, int wave,
                                          int lane, int total_items, int& item, int& mb0, int& mb1) {
    __syncthreads();
    if (wave == 0) {
        if (kGuided && a.guided_mb) item = claim_guided(a, home, drained, first, lane, mb0, mb1) ? 0 : -1;
        else item = claim_item(a, home, drained, first, lane, total_items);
        if (lane == 0) {
            ctrl[0] = item;
            if (kGuided) {
                ctrl[4] = mb0;
                ctrl[5] = mb1;
            }
        }
    }
    __syncthreads();
    item = uniform_i32(ctrl[0]);
    if (kGuided) {
        mb0 = uniform_i32(ctrl[4]);
        mb1 = uniform_i32(ctrl[5]);
    }
}

// True for the workgroup that finishes last (call after a fence).
__device__ __forceinline__ bool finish_last(const BatchArgs& a, int home) {
    const uint32_t nhome = (gridDim.x - 1u - (uint32_t)home) / kXcds + 1u;  // workgroups homed on this XCD
    if (atomicAdd(ctr(a, kXcds + home), 1u) != nhome - 1u) return false;
    __threadfence();
    const uint32_t nx = gridDim.x < (uint32_t)kXcds ? gridDim.x : (uint32_t)kXcds;
    return atomicAdd(ctr(a, 2 * kXcds), 1u) == nx - 1u;
}

// Mini blocks [mb0, mb1) of a plan's work item t: a slice of the plan, or,
// after chunk pruning, a slice of one surviving block.
__device__ __forceinline__ void item_range(const BatchArgs& a, CQ& Q, int t, int& mb0, int& mb1) {
    if (Q.live) {
        const int ipc = (Q.prune_mb + a.mb_per_item - 1) / a.mb_per_item;  // items per block
        const int j = t / ipc;
        const int blk = ro(Q.live)[j];
        mb0 = blk * Q.prune_mb + (t - j * ipc) * a.mb_per_item;
        mb1 = min(min(mb0 + a.mb_per_item, (blk + 1) * Q.prune_mb), Q.nmb);
    } else {
        mb0 = t * a.mb_per_item;
        mb1 = min(mb0 + a.mb_per_item, Q.nmb);
    }
}

// The end of a launch, entered by every workgroup once its global effects
// have been performed: the last one in emits the plans' group tables and
// resets the work queue.
__device__ __forceinline__ void finish_launch(const BatchArgs& a, int32_t* ctrl, int home, int nw, int wave, int lane) {
    if (threadIdx.x == 0) ctrl[1] = finish_last(a, home) ? 1 : 0;
    __syncthreads();
    if (!ctrl[1]) return;
    __threadfence();
    // One wave a plan where the batch has more plans than the workgroup waves
    // (each plan's copy is mostly one wait for memory), else all threads on
    // each plan in turn.  Larger tables are left to emit_kernel.
    const bool by_wave = a.nq >= nw;
    for (int qi = by_wave ? wave : 0; qi < a.nq; qi += by_wave ? nw : 1) {
        CQ& Q = *ro(a.q[qi]);
        if (!Q.emit_copy) continue;
        emit_table(Q, reinterpret_cast<unsigned long long*>(a.agg[qi]), a.status[qi],
                   by_wave ? lane : (int)threadIdx.x, by_wave ? kWave : (int)blockDim.x);
    }
    if (threadIdx.x < 2 * kXcds + 1)  // every other workgroup has left: reset for the next launch
        __hip_atomic_store(ctr(a, threadIdx.x), 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __threadfence_system();
}

// ---------------------------------------------------------------------------
// The persistent fused kernel (4, 8 or 16 waves per workgroup)
// ---------------------------------------------------------------------------
// kStr: 0 no string atom in the batch, 1 string atoms on VARLEN columns, 2
// also an FSST atom.  kHash: some plan aggregates into a hash group table.
template <int kStr, bool kHash>
__global__ __launch_bounds__(16 * kWave) __attribute__((amdgpu_waves_per_eu(kStr == 2 ? 5 : 6, 8))) void fused_kernel(BatchArgs a) {
    extern __shared__ __align__(16) uint8_t smem[];
    // Static LDS: its address is known when the kernel is compiled, so the
    // string scan's table reads take it as an immediate offset.
    __shared__ __align__(16) uint32_t str_tab[kLdsStrTabBytes / 4];
    int32_t* ctrl = reinterpret_cast<int32_t*>(smem);
    uint8_t* shared_area = smem + kLdsCtrlBytes;
    const bool str_stage = a.str_stage != 0;
    const int lane = lane_id();
    const int wave = uniform_i32(threadIdx.x >> 6);  // uniform: mini-block headers become scalar loads
    const int nw = uniform_i32((int)(blockDim.x >> 6));
    const bool pend_stage = a.pend_stage != 0;
    const WaveArea W =
        wave_area(shared_area + a.lds_shared + (size_t)wave * wave_area_bytes(str_stage, pend_stage), str_tab,
                  pend_stage);
    const int total_items = a.item_start[a.nq];

    const int home = (int)(blockIdx.x % kXcds);
    uint32_t drained = 0;  // wave 0: item ranges found empty
    unsigned long long sink = 0;  // old values of this thread's device-scope atomics
    bool direct = false;          // some plan aggregated straight into global memory
    int cur = -1;
    int fs_chunk = -1;  // chunk whose FSST code tables are in LDS
    bool ok_hdr = true;
    int npend = 0;
    for (bool first = true;; first = false) {
        int item = 0, mb0 = 0, mb1 = 0;
        next_item<kStr == 1>(a, ctrl, home, drained, first, wave, lane, total_items, item, mb0, mb1);
        if (item < 0) break;
        int qi = 0;
        while (qi + 1 < a.nq && a.item_start[qi + 1] <= item) ++qi;
        qi = uniform_i32(qi);
        CQ& Q = *ro(a.q[qi]);
        unsigned long long* const gagg = reinterpret_cast<unsigned long long*>(a.agg[qi]);
        if (qi != cur) {
            if (cur >= 0) {
                unsigned long long* const cagg = reinterpret_cast<unsigned long long*>(a.agg[cur]);
                // Queued survivors stay valid across the items of one plan:
                // they go to stage B when the queue fills, at a plan switch
                // (before the plan's LDS state is replaced) and at the end.
                // The string instantiation also flushes at every item's end:
                // its survivors are few, and a full flush in the middle of an
                // item keeps the workgroup's other waves waiting at the next
                // item's barrier (measured: without string atoms, deferring
                // is faster; with them, flushing per item).
                if (npend) flush_pending<kHash>(*ro(a.q[cur]), shared_area, cagg, W, npend, lane, ok_hdr);
                __syncthreads();
                sink += flush_lds_agg(*ro(a.q[cur]), shared_area, cagg);
                if (!ok_hdr) sink += atomicOr(a.status[cur], ST_CORRUPT);
                ok_hdr = true;
            }
            __syncthreads();
            load_lds_state(Q, shared_area, str_tab);
            if (kStr == 2) fsst_load_dfa(Q, shared_area);
            fs_chunk = -1;
            __syncthreads();
            cur = qi;
            direct |= Q.agg_lds == 0;
        }
        const bool guided = kStr == 1 && a.guided_mb;
        if (!guided) item_range(a, Q, item - a.item_start[qi], mb0, mb1);
        if (Q.npreds == 0 && Q.nprobes > 0) {
            semi_tiles<kHash>(Q, shared_area, gagg, W, mb0 + wave, mb1, nw, lane, npend, ok_hdr);
        } else if (kStr == 2 && Q.fs_pred >= 0) {
            // FSST: the item's mini blocks chunk by chunk, each chunk's code
            // tables built once by the workgroup
            const int mbpc = max(Q.cols[Q.preds[Q.fs_pred].col].mbpc, 1);
            for (int s0 = mb0; s0 < mb1;) {
                const int k = s0 / mbpc;
                const int s1 = min(mb1, (k + 1) * mbpc);
                if (k != fs_chunk) {
                    __syncthreads();
                    fsst_load_chunk(Q, shared_area, k);
                    __syncthreads();
                    fs_chunk = k;
                }
                for (int m = s0 + wave; m < s1; m += nw)
                    process_tile<kStr, kHash>(Q, shared_area, gagg, W, m, lane, npend, ok_hdr);
                s0 = s1;
            }
        } else {
            for (int v = mb0 + wave; v < mb1; v += nw) {
                int m = v;
                if (guided && Q.live) {  // v counts the surviving blocks' mini blocks
                    const int j = v / Q.prune_mb;
                    m = ro(Q.live)[j] * Q.prune_mb + (v - j * Q.prune_mb);
                    if (m >= Q.nmb) continue;
                }
                process_tile<kStr, kHash>(Q, shared_area, gagg, W, m, lane, npend, ok_hdr);
            }
        }
        if (kStr && npend) flush_pending<kHash>(Q, shared_area, gagg, W, npend, lane, ok_hdr);
    }
    if (cur >= 0) {
        unsigned long long* const cagg = reinterpret_cast<unsigned long long*>(a.agg[cur]);
        if (npend) flush_pending<kHash>(*ro(a.q[cur]), shared_area, cagg, W, npend, lane, ok_hdr);
        __syncthreads();
        sink += flush_lds_agg(*ro(a.q[cur]), shared_area, cagg);
        if (!ok_hdr) sink += atomicOr(a.status[cur], ST_CORRUPT);
    }
    // Last workgroup out emits every plan's records and resets the queue.
    // Publishing: the workgroup's global effects are device-scope atomics,
    // which are coherent across XCDs; waiting for their returned values
    // (the sink) orders them before the completion count, so the costly
    // agent-scope release fence (an L2 writeback) is needed only where rows
    // were aggregated straight into global memory with plain-result atomics.
    if (direct) __threadfence();
    if (sink == ~0ull) ctrl[3] = 1;  // consumes every returned value
    __syncthreads();
    finish_launch(a, ctrl, home, nw, wave, lane);
}

// Two instantiations per string mode, each mode compiled in a source file of
// its own: only batches with a hash group table carry its probing code in
// stage B (its mere presence there slowed the star join by 3%).
template <int kStr, bool kHash>
hipError_t launch_fused_kernel(const BatchArgs& a, int waves, int grid, size_t lds_bytes, hipStream_t s) {
    static bool attr_set = false;
    if (!attr_set) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&fused_kernel<kStr, kHash>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024 - (int)kLdsStrTabBytes);
        attr_set = true;
    }
    hipLaunchKernelGGL((fused_kernel<kStr, kHash>), dim3(grid), dim3(waves * kWave), lds_bytes, s, a);
    return hipGetLastError();
}

template <int kStr>
hipError_t launch_fused_mode(const BatchArgs& a, int waves, int grid, size_t lds_bytes, hipStream_t s) {
    return a.agg_hash ? launch_fused_kernel<kStr, true>(a, waves, grid, lds_bytes, s)
                      : launch_fused_kernel<kStr, false>(a, waves, grid, lds_bytes, s);
}

}  // namespace
}  // namespace dpf
