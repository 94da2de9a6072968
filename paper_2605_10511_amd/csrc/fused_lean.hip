// fused_lean.hip -- the fused kernel for batches whose plans carry every
// value in 32 bits (LeanPlan: no probes, integer atoms only, each group key and
// measure an offset of less than 2^32 from its column's minimum, packed in 32
// bits or fewer).  fused.h has the general kernel; both share the work queue, the
// group tables and the emission.
//
// What bounds it: latency and instruction issue, not bandwidth (60M-row filter
// 1.4 TB/s, 24M-row summary 0.8 TB/s of the 5.7 a plain read reaches; counters: a
// mini block of the filter takes 263 vector and 266 scalar instructions, its
// waves wait half of their cycles).  The
// general kernel decodes to 64 bits, reads its descriptors with chains of
// scalar loads for every mini block and again for every 64 surviving rows, and
// adds each row to a group table that all lanes of a workgroup share, or to
// device memory.  Here
//  * the headers of a wave's next 16 mini blocks are read, checked and turned
//    into code-space bounds by one lane each (lean_setup), so that a mini
//    block costs one LDS read per column instead of a chain of scalar loads;
//  * the packed words of up to four mini blocks are copied to LDS straight from
//    memory, 16 bytes a lane, all columns in flight together (lean_load_group);
//    a lane's four rows are then dword pairs, a funnel shift and a bit extract
//    in 32 bits, and a range atom is a subtract and a compare;
//  * row sets are four wave masks in scalar registers;
//  * a mini block that keeps kDenseMin rows or more is aggregated in place from
//    its staged words; fewer survivors are queued and gathered, 256 at a time;
//  * the workgroup's LDS group table has up to 8 copies side by side, lanes
//    spread over them, so that rows of the same group do not meet in one
//    address;
//  * rows of a wave that all fall in one group of a table in device memory
//    (a sorted group key) are summed across the wave before one lane adds.
// Before and after, kernel time: 60M-row filter 472 -> 208 us, 24M-row summary
// 730 -> 157 us, revenue per day over 10M sorted rows 3,400 -> 91 us.
#include "fused.h"

namespace dpf {
namespace {

using CLC = const DPF_AS_CONST LeanMore;
using CLA = const DPF_AS_CONST LeanAcc;
using CLT = const DPF_AS_CONST LeanTerm;
#define DPF_AS_GLOBAL __attribute__((address_space(1)))
#define DPF_AS_LDS __attribute__((address_space(3)))
typedef DPF_AS_GLOBAL unsigned long long gu64;

// Rows a mini block must keep for its value columns to be staged and the rows
// aggregated in place.  At 32 of 256 rows (60M-row filter) gathering took 260
// us, staging 363.  The other scans measured keep far more or far fewer rows a
// mini block: 48 and 64 instead of 96 made no difference to them.
constexpr int kDenseMin = 96;
// The same where the value columns are there already (the first mini blocks of
// a scan): 40,000 rows in 40.3 us, with 48 in 41.8.
constexpr int kStagedMin = 16;

// Header record of a column's mini block: x, y: the address of its packed
// words (48 bits), above it the width (8 bits) and flags; z, w: an atom's low
// bound and span of passing packed values, or a value column's base - ref and
// its smallest difference.
enum : uint32_t {  // in y
    kHdrGeneral = 1u << 24,  // decode with decode_dense (checks the header again)
    kHdrAll = 1u << 25,      // every row passes the atom
    kHdrNone = 1u << 26,     // no row does
    kHdrDelta = 1u << 27,    // DELTA of width 0 or 1
};
__device__ __forceinline__ uint32_t hdr_width(uint32_t y) { return (y >> 16) & 127u; }
__device__ __forceinline__ cptr<uint8_t> hdr_words(uint32_t x, uint32_t y) {
    return (cptr<uint8_t>)(((uint64_t)(y & 0xFFFFu) << 32) | x);
}

// The packed words of up to four mini blocks are staged together: one wait for
// memory, one walk of the entries for 1,024 rows.  Of the atoms the first
// kLeanAhead are read that way, the others decoded one by one.
constexpr int kGroup = 4;
constexpr int kLeanAhead = 3;

struct LeanWave {
    uint16_t* rows;  // [kLeanQueue] queued rows, counted from the first of the 16 mini blocks
    uint4* recs;     // [entry][kLeanTiles] header records
    uint8_t* stage;  // packed words of a group of mini blocks (LeanEnt::stage_off)
    const LeanEnt* ents;  // the workgroup's copy of the plan's entries
    int group;       // mini blocks staged together: 4, 2 or 1
    uint32_t lr;     // copies of the plan's LDS group table: 2^lr
};

// The same value, unknown to the compiler: what is computed from it is not
// hoisted out of the loops into registers that the whole kernel then carries.
__device__ __forceinline__ int here(int x) {
    asm volatile("" : "+v"(x));
    return x;
}

__device__ __forceinline__ bool in_mask(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// Header records of mini blocks m0 .. m0 + nt - 1 for every entry, 8 entries
// x 16 mini blocks a step, two a lane.  Returns the mini blocks that no row
// survives.  slow: some atom needs decode_dense.  A corrupt header of an
// atom's column is reported here, unless an earlier atom settled the mini
// block.
__device__ __forceinline__ uint32_t lean_setup(CQ& Q, const LeanWave& W, int m0, int nt, int lane,
                                               bool& slow, bool& ok_hdr) {
    lane = here(lane);
    constexpr int kSub = kWave / kLeanTiles, kPer = 2;  // entries a step: kSub x kPer
    const int t = lane & (kLeanTiles - 1), m = m0 + t, sub = lane / kLeanTiles;
    const int nents = Q.lean.nents, npreds = Q.npreds;
    uint32_t dead = 0;
    slow = npreds > kLeanAhead;
    for (int e0 = 0; e0 < nents; e0 += kSub * kPer) {
        LeanEnt c[kPer];
        uint32_t w0[kPer], w1[kPer];
        int64_t base[kPer], dmin[kPer];
        bool act[kPer];
#pragma unroll
        for (int h = 0; h < kPer; ++h) {
            const int e = e0 + h * kSub + sub;
            act[h] = e < nents && t < nt;
            c[h] = W.ents[e < nents ? e : 0];
            const int mm = t < nt ? m : m0;
            w0[h] = ro(c[h].woff)[mm];
            w1[h] = ro(c[h].woff)[mm + 1];
            base[h] = ro(c[h].base)[mm];
            dmin[h] = 0;
            if (c[h].enc == ENC_DELTA) dmin[h] = ro(c[h].dmin)[mm];
        }
#pragma unroll
        for (int h = 0; h < kPer; ++h) {
            const int e = e0 + h * kSub + sub;
            const bool delta = c[h].enc == ENC_DELTA;
            const uint32_t maxw = (uint32_t)c[h].maxw;
            const uint32_t nw = w1[h] - w0[h];
            const bool hok = (w0[h] <= w1[h]) & (w1[h] <= c[h].nwords) & ((nw & 7u) == 0) & (nw <= 512u);  // as mb_hdr
            const uint32_t b = hok ? nw >> 3 : 0u;
            const uint64_t addr = (uint64_t)(c[h].words + (hok ? w0[h] : 0u));
            uint32_t meta = ((uint32_t)(addr >> 32) & 0xFFFFu) | b << 16 | (hok ? 0u : kHdrGeneral), x, y;
            const bool pred = e < npreds;
            // an atom: the zone test of zone_test, one mini block a lane
            const int64_t plo = c[h].lo, phi = c[h].hi;
            const int64_t kLim = int64_t(1) << 61, kDLim = int64_t(1) << 31;
            const bool ne = c[h].kind == PK_NE;
            const bool known = ((c[h].kind == PK_RANGE) | ne) & hok & (b <= 32) & (base[h] < kLim) & (base[h] > -kLim) &
                               (dmin[h] < kDLim) & (dmin[h] > -kDLim);
            const int64_t span = (int64_t)((uint64_t(1) << (b & 63u)) - 1);
            const int64_t d = known ? dmin[h] * (kMB - 1) : 0;
            const int64_t lo = base[h] + (d < 0 ? d : 0);
            const int64_t hi = base[h] + (d < 0 ? 0 : d) + (delta ? span * (kMB - 1) : span);
            const bool all = known & (ne ? (hi < plo) | (lo > plo) : (lo >= plo) & (hi <= phi));
            const bool zero = known & !all & (ne ? lo == hi : (hi < plo) | (lo > phi));
            const bool fast = known & !delta & (b <= maxw);
            const bool gen = !all & !zero & !fast;
            if (pred) {
                // undecided: packed value v passes iff v - x <= y (mod 2^32)
                const uint32_t l32 = plo <= base[h] ? 0u : (uint32_t)((uint64_t)plo - (uint64_t)base[h]);
                const uint32_t h32 = phi >= hi ? (uint32_t)span : (uint32_t)((uint64_t)phi - (uint64_t)base[h]);
                x = ne ? (uint32_t)((uint64_t)plo - (uint64_t)base[h]) + 1u : l32;
                y = ne ? 0xFFFFFFFEu : h32 - l32;
                meta |= (all ? kHdrAll : 0u) | (zero ? kHdrNone : 0u) | (gen ? kHdrGeneral : 0u);
            } else {
                // (a bad header stays kHdrGeneral alone: decode_dense and lean_at report it)
                meta |= delta ? (!hok || b > 1 ? kHdrGeneral : kHdrDelta) : b > maxw ? kHdrGeneral : 0u;
                x = (uint32_t)(uint64_t)base[h] - (uint32_t)(uint64_t)plo;
                y = (uint32_t)(uint64_t)dmin[h];
            }
            if (act[h]) W.recs[e * kLeanTiles + t] = make_uint4((uint32_t)addr, meta, x, y);
            slow |= __ballot(act[h] & pred & gen) != 0;
            const uint64_t nb = __ballot(act[h] & pred & zero), bb = __ballot(act[h] & pred & !hok);
            if (nb | bb) {
#pragma unroll
                for (int j = 0; j < kSub; ++j) {  // the atoms in order
                    constexpr uint32_t kAllTiles = (1u << kLeanTiles) - 1u;
                    if ((uint32_t)(bb >> (kLeanTiles * j)) & ~dead & kAllTiles) ok_hdr = false;
                    dead |= (uint32_t)(nb >> (kLeanTiles * j)) & kAllTiles;
                }
            }
        }
    }
    wave_lds_sync();
    return dead;
}

__device__ __forceinline__ uint4 uniform_rec(const uint4& r) {
    return make_uint4((uint32_t)uniform_i32((int)r.x), (uint32_t)uniform_i32((int)r.y), (uint32_t)uniform_i32((int)r.z),
                      (uint32_t)uniform_i32((int)r.w));
}

__device__ __forceinline__ uint4 lean_rec(const LeanWave& W, int e, int t) {
    return uniform_rec(W.recs[e * kLeanTiles + t]);
}

// The lane's four rows' values of b <= kLeanWidth bits: the 64 rows between them
// are 2 b whole dwords, so all four sit at bit (lane b) & 31 of a pair of dwords.
__device__ __forceinline__ void lean_unpack(const uint8_t* stage, uint32_t b, int lane, uint32_t v[4]) {
    const uint32_t bp = (uint32_t)lane * b, sh = bp & 31u;
    const uint8_t* p = stage + ((bp >> 5) << 2);
    const uint32_t keep = b ? ~0u >> (32u - b) : 0u;
    uint64_t w[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) w[k] = *reinterpret_cast<const u64_a4*>(p + (uint32_t)k * 8u * b);
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = __builtin_amdgcn_alignbit((uint32_t)(w[k] >> 32), (uint32_t)w[k], sh) & keep;
}

// ---------------------------------------------------------------------------
// Aggregation of R rows a lane (row sets mk[r]), values u[r][slot].
// ---------------------------------------------------------------------------
// Values of R rows a lane.
template <int R>
struct Rows {
    uint32_t v[kMaxSlots * R];  // slot s of row r: v[s R + r]
    __device__ __forceinline__ uint32_t& operator[](int i) { return v[i]; }
    __device__ __forceinline__ uint32_t operator[](int i) const { return v[i]; }
};

// Slot s (wave-uniform) of R rows: a branch to the register that holds it.
// (The empty asm of each case is its own, or the compiler merges the cases
// into one indexed load of a copy of u in scratch.)
template <int R>
__device__ __forceinline__ void lean_get(const Rows<R> u, int s, uint32_t x[R]) {
    switch (s) {
#define DPF_SLOT(i)                                            \
    case i:                                                    \
        _Pragma("unroll") for (int r = 0; r < R; ++r) {        \
            x[r] = u[i * R + r];                                 \
            asm volatile("; slot " #i : "+v"(x[r]));           \
        }                                                      \
        break;
        DPF_SLOT(0) DPF_SLOT(1) DPF_SLOT(2) DPF_SLOT(3) DPF_SLOT(4) DPF_SLOT(5) DPF_SLOT(6)
        default:
#pragma unroll
            for (int r = 0; r < R; ++r) {
                x[r] = u[7 * R + r];
                asm volatile("; slot 7" : "+v"(x[r]));
            }
#undef DPF_SLOT
    }
}

// A factor's value in R rows, in 32 bits (it is known to fit).
template <int R>
__device__ __forceinline__ void lean_term32(CLT& T, const Rows<R> u, uint32_t x[R]) {
    const uint32_t c = (uint32_t)T.c;
    if (T.slot < 0) {
#pragma unroll
        for (int r = 0; r < R; ++r) x[r] = c;
        return;
    }
    lean_get<R>(u, T.slot, x);
    if (T.mk == 1) {
#pragma unroll
        for (int r = 0; r < R; ++r) x[r] += c;
    } else if (T.mk == -1) {
#pragma unroll
        for (int r = 0; r < R; ++r) x[r] = c - x[r];
    } else {
        const uint32_t mul = (uint32_t)T.mul;
#pragma unroll
        for (int r = 0; r < R; ++r) x[r] = x[r] * mul + c;
    }
}

template <int R>
__device__ __forceinline__ void lean_value(CLA& A, const Rows<R> u, uint64_t val[R]) {
    uint32_t x[R];
    if (A.cls == 0) {  // one factor x + c
        const uint64_t c = (uint64_t)A.t[0].c;
#pragma unroll
        for (int r = 0; r < R; ++r) x[r] = 0;
        if (A.t[0].slot >= 0) lean_get<R>(u, A.t[0].slot, x);
#pragma unroll
        for (int r = 0; r < R; ++r) val[r] = (uint64_t)x[r] + c;
    } else if (A.cls == 3) {  // the last value times one more factor in [0, 2^24)
        lean_term32<R>(A.t[A.nterms - 1], u, x);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t hi = ((uint32_t)(val[r] >> 32) & 0xFFFFFFu) * (x[r] & 0xFFFFFFu);
            val[r] = (uint64_t)(uint32_t)val[r] * (uint64_t)x[r] + ((uint64_t)hi << 32);
        }
    } else if (A.cls == 1) {  // factors in [0, 2^24): 24-bit multiplies
        lean_term32<R>(A.t[0], u, x);
#pragma unroll
        for (int r = 0; r < R; ++r) val[r] = x[r];
        if (A.nterms > 1) {
            uint32_t y[R];
            lean_term32<R>(A.t[1], u, y);
#pragma unroll
            for (int r = 0; r < R; ++r) val[r] = (uint64_t)(x[r] & 0xFFFFFFu) * (uint64_t)(y[r] & 0xFFFFFFu);
        }
        if (A.nterms > 2) {
            uint32_t y[R];
            lean_term32<R>(A.t[2], u, y);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const uint32_t hi = ((uint32_t)(val[r] >> 32) & 0xFFFFFFu) * (y[r] & 0xFFFFFFu);
                val[r] = (uint64_t)(uint32_t)val[r] * (uint64_t)y[r] + ((uint64_t)hi << 32);
            }
        }
    } else {
#pragma unroll
        for (int r = 0; r < R; ++r) val[r] = 1;
        for (int t = 0; t < A.nterms; ++t) {
            const uint64_t mul = (uint64_t)A.t[t].mul, c = (uint64_t)A.t[t].c;
#pragma unroll
            for (int r = 0; r < R; ++r) x[r] = 0;
            if (A.t[t].slot >= 0) lean_get<R>(u, A.t[t].slot, x);
#pragma unroll
            for (int r = 0; r < R; ++r) val[r] *= (uint64_t)x[r] * mul + c;  // slot < 0: mul * 0 + c
        }
    }
}

// Adds the rows to a table in device memory, one group of the rows at a time
// while a group has kRunMin rows: they are summed over the wave, accumulator a
// left in lane a, and added by one instruction.  The rest goes row by row.
// (Summing a run costs about 30 instructions an accumulator; rows of one group
// added one by one meet on one address.)
constexpr uint32_t kRunMin = 8;

// Entry e of a direct table (at most 2^22 groups x 12 accumulators): a 32-bit
// byte offset, so that the scalar base takes no address registers a lane.
__device__ __forceinline__ gu64* row_at(gu64* T, uint32_t e) {
    uint32_t o = e * 8u;
    asm volatile("" : "+v"(o));
    return (gu64*)((DPF_AS_GLOBAL uint8_t*)T + o);
}

template <int R>
__device__ __forceinline__ void lean_add_global(CQ& Q, const Rows<R> u, const uint64_t mk[R], const uint32_t g[R],
                                                gu64* T, int lane) {
    const int nacc = Q.nacc;
    uint64_t rem[R];
#pragma unroll
    for (int r = 0; r < R; ++r) rem[r] = mk[r];
    for (;;) {
        uint64_t any = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) any |= rem[r];
        if (any == 0) return;
        uint32_t g0 = 0;
#pragma unroll
        for (int r = R - 1; r >= 0; --r)
            if (rem[r]) g0 = (uint32_t)__builtin_amdgcn_readlane((int)g[r], __builtin_ctzll(rem[r]));
        uint64_t sel[R];
        uint32_t rows = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            sel[r] = __ballot(g[r] == g0) & rem[r];
            rows += (uint32_t)__popcll(sel[r]);
        }
        const bool run = rows >= kRunMin;
        uint64_t mine = rows;
        if (!run) {
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (in_mask(rem[r]))
                    __hip_atomic_fetch_add(row_at(T, g[r] * (uint32_t)nacc), 1ull, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
        }
        uint64_t val[R];
        for (int a = 1; a < nacc; ++a) {
            lean_value<R>(Q.lean.accs[a], u, val);
            if (run) {
                uint64_t s = 0;
#pragma unroll
                for (int r = 0; r < R; ++r) s += in_mask(sel[r]) ? val[r] : 0ull;
                const uint64_t tot = readlane_u64(wave_incl_scan_u64(s), kWave - 1);
                if (lane == a) mine = tot;
            } else {
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (in_mask(rem[r]))
                        __hip_atomic_fetch_add(row_at(T, g[r] * (uint32_t)nacc + (uint32_t)a),
                                               (unsigned long long)val[r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        if (!run) return;
        if (lane < nacc)
            __hip_atomic_fetch_add(row_at(T, g0 * (uint32_t)nacc + (uint32_t)lane), (unsigned long long)mine, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int r = 0; r < R; ++r) rem[r] &= ~sel[r];
    }
}

template <int R, bool kHash>
__device__ __forceinline__ void lean_aggregate(CQ& Q, uint8_t* smem_shared, unsigned long long* gagg, uint32_t lr,
                                               const Rows<R> u, uint64_t mk[R], int lane, bool& ok_hdr) {
    const int nacc = Q.nacc, nkeys = Q.nkeys;
    uint64_t bad = 0;
    if (kHash && Q.agg_hash) {
        // group indices of up to 62 bits, added row by row
        uint64_t g64[R];
#pragma unroll
        for (int r = 0; r < R; ++r) g64[r] = 0;
        for (int k = 0; k < nkeys; ++k) {
            CK& K = Q.keys[k];
            uint32_t x[R];
            lean_get<R>(u, K.slot, x);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const uint64_t out = __ballot((uint64_t)x[r] >= (uint64_t)K.card) & mk[r];
                bad |= out;
                mk[r] &= ~out;
                g64[r] += (uint64_t)x[r] * (uint64_t)K.stride;
            }
        }
        gu64* at[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            at[r] = (gu64*)gagg;
            if (!in_mask(mk[r])) continue;
            const int64_t row = agg_row(Q, gagg, (int64_t)g64[r]);
            if (row < 0) {
                ok_hdr = false;
            } else {
                at[r] += (uint64_t)row * (uint32_t)nacc;
                __hip_atomic_fetch_add(at[r], 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        uint64_t val[R];
        for (int a = 1; a < nacc; ++a) {
            lean_value<R>(Q.lean.accs[a], u, val);
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (in_mask(mk[r]) && ok_hdr)
                    __hip_atomic_fetch_add(at[r] + a, (unsigned long long)val[r], __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
        }
        if (bad) ok_hdr = false;
        return;
    }
    uint32_t g[R];
#pragma unroll
    for (int r = 0; r < R; ++r) g[r] = 0;
    // key slots one after the other, each from its own registers
    const uint32_t keys = (uint32_t)Q.lean.keys;
#pragma unroll
    for (int s = 0; s < kMaxSlots; ++s) {
        if (!((keys >> s) & 1u)) continue;
        const uint32_t last = Q.lean.key_last[s], stride = Q.lean.key_stride[s] & 0xFFFFFFu;
        uint64_t out[R], any = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            out[r] = __ballot(u[s * R + r] > last) & mk[r];
            any |= out[r];
            g[r] += (u[s * R + r] & 0xFFFFFFu) * stride;  // the table has at most 2^22 groups
        }
        if (any) {
            bad = any;
#pragma unroll
            for (int r = 0; r < R; ++r) mk[r] &= ~out[r];
        }
    }
    if (bad) ok_hdr = false;
    if (!Q.agg_lds) {
        lean_add_global<R>(Q, u, mk, g, (gu64*)gagg, lane);
        return;
    }
    // Copies side by side: entry e of the table at e << lr, the lane's copy in
    // it.  Rows that are not in the set go to a group after the last one,
    // which nobody reads: no branch per row and accumulator.
    const uint32_t lr3 = lr + 3u;
    uint8_t* const T = smem_shared + Q.agg_lds_off;
    uint32_t at[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint32_t gr = in_mask(mk[r]) ? g[r] : (uint32_t)Q.ngroups;
        at[r] = ((gr * (uint32_t)nacc) << lr3) + ((lane << 3) & ((1u << lr3) - 1u));
        atomicAdd(reinterpret_cast<unsigned long long*>(T + at[r]), 1ull);
    }
    // Sums of one slot's plain values: by slot, so that each reads its
    // register directly (their constants are added when the table leaves LDS).
    const uint32_t plain = (uint32_t)Q.lean.plain;
#pragma unroll
    for (int s = 0; s < kMaxSlots; ++s) {
        if (!((plain >> s) & 1u)) continue;
        uint8_t* const Ta = T + ((uint32_t)Q.lean.plain_acc[s] << lr3);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            // (widened here: left to itself the compiler keeps every value
            // as a 64-bit register pair from its decode on)
            uint32_t x = u[s * R + r];
            asm volatile("" : "+v"(x));
            atomicAdd(reinterpret_cast<unsigned long long*>(Ta + at[r]), (unsigned long long)x);
        }
    }
    const int nprod = Q.lean.nprod;
    uint64_t val[R];
    for (int j = 0; j < nprod; ++j) {
        const int a = Q.lean.prod_acc[j];
        lean_value<R>(Q.lean.accs[a], u, val);
        uint8_t* const Ta = T + ((uint32_t)a << lr3);
#pragma unroll
        for (int r = 0; r < R; ++r)
            atomicAdd(reinterpret_cast<unsigned long long*>(Ta + at[r]), (unsigned long long)val[r]);
    }
}

// The packed words of the group of mini blocks t0 .. (nt mini blocks have
// records), for the entries of mask, to the staging area: a column's mini
// blocks follow each other in memory, so a group's are one contiguous copy,
// loaded straight into LDS (no registers, all columns in flight together).
// Gathered from memory, each lane's word is an access of its own, 64 to an
// instruction: 770 accesses a mini block of the 60M-row filter.
// place: lane 4 e + g gets the place in LDS of entry e's mini block t0 + g.
// Returns the entries whose words are not there (a mini block to be decoded
// another way; entries from 16 on).
__device__ __forceinline__ uint32_t lean_load_group(const LeanWave& W, int t0, int nt, uint32_t mask, int lane,
                                                    uint32_t& place) {
    lane = here(lane);
    const int ng = min(W.group, nt - t0);
    // lane 4 e + g: entry e, mini block t0 + g
    const int e = lane / kGroup, g = lane & (kGroup - 1);
    const bool in = ((mask >> e) & 1u) && g < ng;
    const uint2 xy = *reinterpret_cast<const uint2*>(&W.recs[in ? e * kLeanTiles + t0 + g : 0]);
    const uint2 src = *reinterpret_cast<const uint2*>(&W.ents[in ? e : 0].stage_off);  // {place, copy}, for one mini block
    const uint32_t xa = (uint32_t)__shfl((int)xy.x, lane & ~(kGroup - 1), kWave);
    const uint32_t end = xy.x - xa + 32u * hdr_width(xy.y);
    // (a copy that a value column shares is made even where the atom needs none)
    const uint64_t want_b = __ballot(in && (src.y == 2 || !(xy.y & (kHdrAll | kHdrNone))));
    const uint64_t wide_b = __ballot(in && end > W.ents[in ? e : 0].stage_sz * (uint32_t)W.group);
    const uint64_t odd_b = __ballot(in && (xy.y & (kHdrGeneral | kHdrDelta))) | wide_b;
    wave_lds_sync();  // the words of the last group have been read
    if (in) place = src.x * (uint32_t)W.group + (xy.x - xa);
    uint32_t odd = mask & ~0xFFFFu;
    for (uint32_t left = mask & 0xFFFFu; left; left &= left - 1u) {
        const int a = __builtin_ctz(left);
        const bool no = ((odd_b >> (kGroup * a)) & 0xFull) != 0;
        if (no) odd |= 1u << a;
        const uint32_t copy = (uint32_t)__builtin_amdgcn_readlane((int)src.y, kGroup * a);
        if (copy == 0 || (no && copy != 2) || ((wide_b >> (kGroup * a)) & 0xFull) || ((want_b >> (kGroup * a)) & 0xFull) == 0)
            continue;
        const uint32_t n = (uint32_t)__builtin_amdgcn_readlane((int)end, kGroup * a + ng - 1);
        const uint32_t x = (uint32_t)__builtin_amdgcn_readlane((int)xy.x, kGroup * a);
        const uint32_t y = (uint32_t)__builtin_amdgcn_readlane((int)xy.y, kGroup * a);
        const uint32_t to = (uint32_t)__builtin_amdgcn_readlane((int)src.x, kGroup * a) * (uint32_t)W.group;
        DPF_AS_GLOBAL uint8_t* p = (DPF_AS_GLOBAL uint8_t*)(((uint64_t)(y & 0xFFFFu) << 32) | x);
        for (uint32_t o = 0; o < n; o += 1024u) {
            uint32_t at = (uint32_t)lane * 16u + o;
            if (at < n)
                __builtin_amdgcn_global_load_lds(p + at, (DPF_AS_LDS uint8_t*)(W.stage + to + o), 16, 0, 0);
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    wave_lds_sync();
    return odd;
}

// ---------------------------------------------------------------------------
// A mini block in place: every value column decoded from the staging area
// (odd: but for these entries).
// ---------------------------------------------------------------------------
__device__ __forceinline__ void lean_dense(CQ& Q, const LeanWave& W, int m, int t, const uint64_t mk[4], uint32_t odd,
                                           uint32_t place, int g, int lane, Rows<4>& u, bool& ok_hdr) {
    lane = here(lane);
    const int nloads = Q.nloads, e0 = Q.lean.load0;
    const uint4 rec = W.recs[(e0 + max(min(lane, nloads - 1), 0)) * kLeanTiles + t];  // lane s: slot s
    const uint32_t no = odd >> e0;
    uint32_t other = 0, dict = 0;
#pragma unroll
    for (int s = 0; s < kMaxSlots; ++s) {
        if (s >= nloads) continue;
        if (!((no >> s) & 1u)) {
            const uint32_t rx = (uint32_t)__builtin_amdgcn_readlane((int)place, kGroup * (e0 + s) + g);
            const uint32_t ry = (uint32_t)__builtin_amdgcn_readlane((int)rec.y, s);
            const uint32_t rz = (uint32_t)__builtin_amdgcn_readlane((int)rec.z, s);
            uint32_t v[4];
            lean_unpack(W.stage + rx, hdr_width(ry), lane, v);
#pragma unroll
            for (int k = 0; k < 4; ++k) u[s * 4 + k] = v[k] + rz;
        } else {
            other |= 1u << s;
        }
    }
    dict = (uint32_t)Q.lean.dicts;
    for (uint32_t left = other | dict; left; left &= left - 1u) {
        const int j = __builtin_ctz(left);
        CLC& c = Q.lean.more[e0 + j];
        uint32_t y[4] = {0, 0, 0, 0};
        if ((other >> j) & 1u) {
            const uint4 r = lean_rec(W, e0 + j, t);
            if (!(r.y & kHdrDelta)) {
                int64_t v[4];
                ok_hdr &= decode_dense(Q.cols[c.col], m, lane, v);
#pragma unroll
                for (int k = 0; k < 4; ++k) y[k] = (uint32_t)((uint64_t)v[k] - (uint64_t)c.ref);
            } else {
                // DELTA of width 0 or 1: 64 rows' differences are one scalar
                // word, and the running sum is a count of its bits
                cptr<uint32_t> w = ro(c.words) + ro(c.woff)[m];
                uint32_t carry = r.z;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint64_t d = hdr_width(r.y) ? ((uint64_t)w[2 * k + 1] << 32) | w[2 * k] : 0ull;
                    y[k] = (uint32_t)(64 * k + lane) * r.w + carry + bits_below(d) + (in_mask(d) ? 1u : 0u);
                    carry += (uint32_t)__popcll(d);
                }
            }
        } else {
#pragma unroll
            for (int s = 0; s < kMaxSlots; ++s)
#pragma unroll
                for (int k = 0; k < 4; ++k) y[k] = s == j ? u[s * 4 + k] : y[k];
        }
        if (c.dict) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                uint32_t x = 0;
                if (in_mask(mk[k])) {
                    if (y[k] < (uint32_t)c.ndict) x = (uint32_t)((uint64_t)ro(c.dict)[y[k]] - (uint64_t)c.dref);
                    else ok_hdr = false;
                }
                y[k] = x;
            }
        }
#pragma unroll
        for (int s = 0; s < kMaxSlots; ++s)
#pragma unroll
            for (int k = 0; k < 4; ++k) u[s * 4 + k] = s == j ? y[k] : u[s * 4 + k];
    }
}

// u of row i of mini block m, any encoding and width.  A DELTA row is a sum of
// up to 255 packed differences: of width 1 (a sorted column of slowly rising
// values) it is a count of set bits.
__device__ __forceinline__ uint32_t lean_at(CQ& Q, CLC& c, int m, int i, bool& ok_hdr) {
    const MbHdr h = mb_hdr(Q.cols[c.col], m);
    ok_hdr = ok_hdr && h.ok;
    if (c.enc == ENC_DELTA && h.b == 1) {
        uint32_t sum = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int n = i + 1 - 32 * j;  // rows of word j that count
            const uint32_t keep = n >= 32 ? ~0u : n > 0 ? (1u << n) - 1u : 0u;
            sum += __popc(h.w[j] & keep);
        }
        return (uint32_t)((uint64_t)h.base - (uint64_t)c.ref) + sum + (uint32_t)i * (uint32_t)(uint64_t)ro(c.dmin)[m];
    }
    return (uint32_t)((uint64_t)decode_at(Q.cols[c.col], m, i, ok_hdr) - (uint64_t)c.ref);
}

// ---------------------------------------------------------------------------
// Up to 256 queued rows of the current 16 mini blocks four a
// lane, row[r] (counted from mini block c0) where mk[r] has the lane: values gathered by their records.
// All loads go out before any is used; the records are read twice instead of
// held.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void lean_gather(CQ& Q, const LeanWave& W, int c0, const uint32_t row[4],
                                            const uint64_t mk[4], Rows<4>& u, bool& ok_hdr) {
    const int nloads = Q.nloads, e0 = Q.lean.load0;
    constexpr int kAt = 2;
    uint32_t other = 0;
    // Two slots at a time: what four have in flight does not fit the registers.  The packed values come as pairs of aligned dwords:
    // lanes whose rows are near each other then share an access, which dwords
    // at any byte do not.
#pragma unroll
    for (int s0 = 0; s0 < kMaxSlots; s0 += kAt) {
        if (s0 >= nloads) continue;
        uint64_t w[kAt][4];
#pragma unroll
        for (int s = 0; s < kAt; ++s) {
            if (s0 + s >= nloads) continue;
            uint64_t other_b = 0;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const uint32_t t = in_mask(mk[r]) ? row[r] >> 8 : 0u;
                const uint2 xy = *reinterpret_cast<const uint2*>(&W.recs[(e0 + s0 + s) * kLeanTiles + t]);
                const bool fast = in_mask(mk[r]) && !(xy.y & (kHdrGeneral | kHdrDelta));
                other_b |= __ballot(!fast) & mk[r];
                w[s][r] = 0;
                if (fast) w[s][r] = *(cptr<u64_a4>)(hdr_words(xy.x, xy.y) + ((((row[r] & 255u) * hdr_width(xy.y)) >> 5) << 2));
            }
            if (other_b) other |= 1u << (s0 + s);
        }
#pragma unroll
        for (int s = 0; s < kAt; ++s) {
            if (s0 + s >= nloads) continue;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const uint32_t t = in_mask(mk[r]) ? row[r] >> 8 : 0u;
                const uint4 rec = W.recs[(e0 + s0 + s) * kLeanTiles + t];
                const uint32_t b = hdr_width(rec.y);
                const uint32_t v = __builtin_amdgcn_alignbit((uint32_t)(w[s][r] >> 32), (uint32_t)w[s][r],
                                                             ((row[r] & 255u) * b) & 31u);
                u[(s0 + s) * 4 + r] = (b < 32u ? __builtin_amdgcn_ubfe(v, 0u, b) : v) + rec.z;  // (it takes 5 bits of b)
            }
        }
    }
    other |= (uint32_t)Q.lean.dicts;
    for (uint32_t left = other; left; left &= left - 1u) {
        const int j = __builtin_ctz(left);
        CLC& c = Q.lean.more[e0 + j];
#pragma unroll 1
        for (int r = 0; r < 4; ++r) {
            uint32_t v = 0, rw = 0;
            uint64_t m = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (q == r) { rw = row[q]; m = mk[q]; }
#pragma unroll
            for (int s = 0; s < kMaxSlots; ++s)
#pragma unroll
                for (int q = 0; q < 4; ++q) v = s == j && q == r ? u[s * 4 + q] : v;
            if (in_mask(m)) {
                const uint32_t y = W.recs[(e0 + j) * kLeanTiles + (rw >> 8)].y;
                if (y & (kHdrGeneral | kHdrDelta)) v = lean_at(Q, c, c0 + (int)(rw >> 8), (int)(rw & 255u), ok_hdr);
                if (c.dict) {
                    uint32_t x = 0;
                    if (v < (uint32_t)c.ndict) x = (uint32_t)((uint64_t)ro(c.dict)[v] - (uint64_t)c.dref);
                    else ok_hdr = false;
                    v = x;
                }
            }
#pragma unroll
            for (int s = 0; s < kMaxSlots; ++s)
#pragma unroll
                for (int q = 0; q < 4; ++q) u[s * 4 + q] = s == j && q == r ? v : u[s * 4 + q];
        }
    }
}

// Mini blocks t0 .. t1 - 1 by one wave.  values: the last mini block needed the
// value columns staged, so the next group's come with its atoms'.
template <bool kHash>
__device__ __forceinline__ void lean_slice(CQ& Q, uint8_t* smem_shared, unsigned long long* gagg, const LeanWave& W,
                                           int t0, int t1, int lane, bool& values, bool& ok_hdr) {
    const int npreds = Q.npreds;
    const uint32_t amask = (1u << min(npreds, kLeanAhead)) - 1u;  // the atoms that are staged
    const uint32_t vmask = ((1u << Q.lean.nents) - 1u) & ~((1u << Q.lean.load0) - 1u);
    for (int c0 = t0; c0 < t1; c0 += kLeanTiles) {
        const int nt = min(kLeanTiles, t1 - c0);
        uint32_t odd = 0, have = 0;  // entries without staged words; staged entries
        bool slow = false;
        wave_lds_sync();  // the records of the last mini blocks have been read
        uint32_t todo = ((1u << nt) - 1u) & ~lean_setup(Q, W, c0, nt, lane, slow, ok_hdr);  // mini blocks not yet taken
        todo = (uint32_t)uniform_i32((int)todo);
        const int group = W.group;
        int grp = -1;        // group of mini blocks in the staging area
        uint32_t place = 0;  // its places there
        int nrow = 0;       // queued rows of the 16 mini blocks
        for (;;) {
            Rows<4> u;
            uint64_t mk[4];
            // (the records are about to be replaced: all rows)
            if (nrow >= (todo == 0 ? 1 : 4 * kWave)) {
                wave_lds_sync();
                const int n = min(nrow, 4 * kWave);
                nrow -= n;
                uint32_t row[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int left = n - 64 * r;
                    mk[r] = left >= 64 ? ~0ull : left > 0 ? (1ull << left) - 1ull : 0ull;
                    row[r] = (uint32_t)W.rows[nrow + (64 * r + lane < n ? 64 * r + lane : 0)];
                }
                lean_gather(Q, W, c0, row, mk, u, ok_hdr);
                wave_lds_sync();
            } else if (todo == 0) {
                break;
            } else {
                const int t = __builtin_ctz(todo), m = c0 + t;
                todo &= todo - 1u;
                if (t / group != grp) {
                    grp = t / group;
                    have = amask | (values ? vmask : 0u);
                    odd = lean_load_group(W, grp * group, nt, have, lane, place);
                }
                // lane a: the record of entry a
                const uint4 rec = W.recs[min(lane, max(npreds - 1, 0)) * kLeanTiles + t];
                const int nvalid = (int)min((int64_t)kMB, Q.nrows - (int64_t)m * kMB);
                const int g = t - grp * group;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int n = nvalid - 64 * k;
                    mk[k] = n >= 64 ? ~0ull : n > 0 ? (1ull << n) - 1ull : 0ull;
                }
#pragma unroll
                for (int a = 0; a < kLeanAhead; ++a) {
                    if (a >= npreds || ((odd >> a) & 1u)) continue;
                    const uint32_t ry = (uint32_t)__builtin_amdgcn_readlane((int)rec.y, a);
                    if (ry & kHdrAll) continue;  // (kHdrNone: a dead mini block, not here)
                    const uint32_t rx = (uint32_t)__builtin_amdgcn_readlane((int)place, kGroup * a + g);
                    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)rec.z, a);
                    const uint32_t span = (uint32_t)__builtin_amdgcn_readlane((int)rec.w, a);
                    uint32_t v[4];
                    lean_unpack(W.stage + rx, hdr_width(ry), lane, v);
#pragma unroll
                    for (int k = 0; k < 4; ++k) mk[k] &= __ballot(v[k] - lo <= span);
                }
                if ((mk[0] | mk[1] | mk[2] | mk[3]) == 0) continue;
                if (slow || (odd & amask)) {
                    for (int p = 0; p < npreds; ++p) {
                        const uint32_t meta = lean_rec(W, p, t).y;
                        if ((meta & kHdrAll) || (p < kLeanAhead && !((odd >> p) & 1u))) continue;
                        int64_t v[4];
                        ok_hdr &= decode_dense(Q.cols[Q.preds[p].col], m, lane, v);
                        const uint32_t f = eval_int_pred(Q.preds[p], Q.in_vals, v);
#pragma unroll
                        for (int k = 0; k < 4; ++k) mk[k] &= __ballot((f >> k) & 1u);
                        if ((mk[0] | mk[1] | mk[2] | mk[3]) == 0) break;
                    }
                    if ((mk[0] | mk[1] | mk[2] | mk[3]) == 0) continue;
                }
                const int n0 = (int)__popcll(mk[0]), n1 = (int)__popcll(mk[1]);
                const int n2 = (int)__popcll(mk[2]), n3 = (int)__popcll(mk[3]);
                const int nlive = n0 + n1 + n2 + n3;
                values = nlive >= kDenseMin;
                if (nlive < ((have & vmask) == vmask ? kStagedMin : kDenseMin)) {
                    const uint32_t row = (uint32_t)(t * kMB + lane);
                    if (in_mask(mk[0])) W.rows[nrow + bits_below(mk[0])] = (uint16_t)row;
                    nrow += n0;
                    if (in_mask(mk[1])) W.rows[nrow + bits_below(mk[1])] = (uint16_t)(row + 64);
                    nrow += n1;
                    if (in_mask(mk[2])) W.rows[nrow + bits_below(mk[2])] = (uint16_t)(row + 128);
                    nrow += n2;
                    if (in_mask(mk[3])) W.rows[nrow + bits_below(mk[3])] = (uint16_t)(row + 192);
                    nrow += n3;
                    continue;
                }
                if (vmask && (have & vmask) == 0) {
                    odd |= lean_load_group(W, grp * group, nt, vmask, lane, place);
                    have |= vmask;
                }
                lean_dense(Q, W, m, t, mk, odd, place, g, lane, u, ok_hdr);
            }
            lean_aggregate<4, kHash>(Q, smem_shared, gagg, W.lr, u, mk, lane, ok_hdr);
        }
    }
}

// Adds the workgroup's LDS group table, its copies summed and the plain sums'
// constants applied, to the plan's table in device memory.  Returns a sink of
// the old values, as flush_lds_agg does.
__device__ unsigned long long lean_flush_agg(CQ& Q, uint8_t* smem_shared, unsigned long long* gagg, uint32_t lr) {
    if (!Q.agg_lds) return 0;
    const uint32_t nacc = (uint32_t)Q.nacc, n = ((uint32_t)Q.ngroups * nacc) << lr;
    const unsigned long long* T = reinterpret_cast<const unsigned long long*>(smem_shared + Q.agg_lds_off);
    unsigned long long sink = 0;
    for (uint32_t e0 = 0; e0 < n; e0 += blockDim.x) {  // whole waves: the copies are summed across lanes
        const uint32_t e = e0 + threadIdx.x, i = e >> lr, a = i % nacc;
        unsigned long long x = 0;
        if (e < n) x = T[e] + (unsigned long long)Q.lean.fold[a] * T[((i - a) << lr) + (e & ((1u << lr) - 1u))];
        for (uint32_t d = 1; d < (1u << lr); d <<= 1) x += __shfl_xor(x, (int)d, kWave);
        if (e < n && (e & ((1u << lr) - 1u)) == 0 && x) sink += atomicAdd(gagg + i, x);
    }
    return sink;
}

// ---------------------------------------------------------------------------
// The kernel: work items as in fused_kernel, an item's mini blocks cut into
// one run a wave.
// ---------------------------------------------------------------------------
template <bool kHash>
__global__ __launch_bounds__(16 * kWave) __attribute__((amdgpu_waves_per_eu(4, 8))) void lean_kernel(BatchArgs a) {
    extern __shared__ __align__(16) uint8_t smem[];
    int32_t* ctrl = reinterpret_cast<int32_t*>(smem);
    uint8_t* shared_area = smem + kLdsCtrlBytes;
    const int lane = lane_id();
    const int wave = uniform_i32(threadIdx.x >> 6);
    const int nw = uniform_i32((int)(blockDim.x >> 6));
    LeanWave W;
    {
        uint8_t* p = shared_area + a.lds_shared + (size_t)a.lean_ents * sizeof(LeanEnt);
        W.ents = reinterpret_cast<const LeanEnt*>(shared_area + a.lds_shared);
        p += (size_t)wave * lean_wave_bytes(a.lean_ents, a.lean_stage);
        W.recs = reinterpret_cast<uint4*>(p);
        p += (size_t)a.lean_ents * kLeanTiles * 16;
        W.rows = reinterpret_cast<uint16_t*>(p);
        W.stage = p + kLeanQueue * 2;
        W.group = a.lean_group;
        W.lr = 0;
    }
    const int total_items = a.item_start[a.nq];
    const int home = (int)(blockIdx.x % kXcds);
    uint32_t drained = 0;
    unsigned long long sink = 0;
    int cur = -1;
    bool ok_hdr = true, values = true;
    const bool guided = a.guided_mb != 0;
    for (bool first = true;; first = false) {
        int item = 0, mb0 = 0, mb1 = 0;
        next_item<true>(a, ctrl, home, drained, first, wave, lane, total_items, item, mb0, mb1);
        int qi = 0;
        if (item >= 0) {
            while (qi + 1 < a.nq && a.item_start[qi + 1] <= item) ++qi;
            qi = uniform_i32(qi);
        }
        if (cur >= 0 && (item < 0 || qi != cur)) {  // leaving a plan
            CQ& Q = *ro(a.q[cur]);
            sink += lean_flush_agg(Q, shared_area, reinterpret_cast<unsigned long long*>(a.agg[cur]), W.lr);
            if (!ok_hdr) sink += atomicOr(a.status[cur], ST_CORRUPT);
            ok_hdr = true;
            __syncthreads();
        }
        if (item < 0) break;
        CQ& Q = *ro(a.q[qi]);
        if (qi != cur) {
            W.lr = (uint32_t)min(Q.lean.log2r, a.lean_log2r);
            if (!Q.lean.stage_first) values = false;
            cptr<uint4> src = (cptr<uint4>)&Q.lean.ents[0];
            uint4* dst = reinterpret_cast<uint4*>(shared_area + a.lds_shared);
            for (uint32_t e = threadIdx.x; e < (uint32_t)Q.lean.nents * sizeof(LeanEnt) / 16; e += blockDim.x)
                dst[e] = ld4(src, e);
            if (Q.agg_lds) {
                const uint32_t n = ((uint32_t)Q.ngroups * (uint32_t)Q.nacc) << W.lr;
                unsigned long long* T = reinterpret_cast<unsigned long long*>(shared_area + Q.agg_lds_off);
                for (uint32_t e = threadIdx.x; e < n; e += blockDim.x) T[e] = 0;
            }
            __syncthreads();
            cur = qi;
        }
        if (!guided) item_range(a, Q, item - a.item_start[qi], mb0, mb1);
        const int per = (mb1 - mb0 + nw - 1) / nw;
        const int t1 = min(mb1, mb0 + (wave + 1) * per);
        // (a guided item of a pruned plan counts the surviving blocks' mini
        // blocks: its run may lie in several of them)
        const bool blocks = guided && Q.live;
        for (int v = mb0 + wave * per; v < t1;) {
            int s0 = v, s1 = t1;
            if (blocks) {
                const int j = v / Q.prune_mb, off = v - j * Q.prune_mb;
                s0 = ro(Q.live)[j] * Q.prune_mb + off;
                s1 = s0 + min(t1 - v, Q.prune_mb - off);
                v += s1 - s0;
                s1 = min(s1, Q.nmb);
            } else {
                v = t1;
            }
            lean_slice<kHash>(Q, shared_area, reinterpret_cast<unsigned long long*>(a.agg[qi]), W, s0, s1, lane, values, ok_hdr);
        }
    }
    // Publishing, as in fused_kernel: every global effect is a device-scope
    // atomic.  Those with a result are waited for through the sink; those
    // without (rows added straight to device memory) by their count, which
    // needs no L2 writeback: no plain store has to become visible.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (sink == ~0ull) ctrl[3] = 1;  // consumes every returned value
    __syncthreads();
    finish_launch(a, ctrl, home, nw, wave, lane);
}

template <bool kHash>
hipError_t launch_lean_kernel(const BatchArgs& a, int waves, int grid, size_t lds_bytes, hipStream_t s) {
    static bool attr_set = false;
    if (!attr_set) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&lean_kernel<kHash>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        attr_set = true;
    }
    hipLaunchKernelGGL((lean_kernel<kHash>), dim3(grid), dim3(waves * kWave), lds_bytes, s, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_lean(const BatchArgs& a, int waves, int grid, size_t lds_bytes, hipStream_t s) {
    if (waves != 4 && waves != 8 && waves != 16) return hipErrorInvalidValue;
    return a.agg_hash ? launch_lean_kernel<true>(a, waves, grid, lds_bytes, s)
                      : launch_lean_kernel<false>(a, waves, grid, lds_bytes, s);
}

}  // namespace dpf
