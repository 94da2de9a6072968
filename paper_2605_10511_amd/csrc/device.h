// device.h -- device code that several kernels share: decoding of encoded
// columns, integer and string predicates, hash probes and aggregation into a
// group table.  Included by each kernel source; everything has internal
// linkage there.
//
// Work mapping inside a mini block: lane l of a wave owns rows l, l+64,
// l+128, l+192, so every load instruction of the wave covers a contiguous
// run of packed bits (row i sits at bit i * width).
#pragma once
#include <hip/hip_runtime.h>

#include "dpf_internal.h"

namespace dpf {
namespace {

// Descriptors and encoded columns are read-only during a launch, so the
// kernels read them through the constant address space: wave-uniform reads
// (headers, descriptor fields) become scalar loads and per-lane reads become
// global loads, never flat ones.
#define DPF_AS_CONST __attribute__((address_space(4)))
template <class T>
using cptr = const DPF_AS_CONST T*;
template <class T>
__device__ __forceinline__ cptr<T> ro(const T* p) { return (cptr<T>)p; }
using CQ = const DPF_AS_CONST DevQuery;
using CC = const DPF_AS_CONST DevCol;
using CP = const DPF_AS_CONST DevPred;
using CH = const DPF_AS_CONST DevHash;
using CPR = const DPF_AS_CONST DevProbe;
using CL = const DPF_AS_CONST DevLoad;
using CK = const DPF_AS_CONST DevKey;
using CT = const DPF_AS_CONST DevTerm;
using CA = const DPF_AS_CONST DevAcc;
using CHB = const DPF_AS_CONST HashBuildArgs;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 ld4(cptr<uint4> g, uint32_t i) {
    const u32x4 t = ((cptr<u32x4>)g)[i];
    return make_uint4(t.x, t.y, t.z, t.w);
}

constexpr int kPendCap = 320;   // per-wave survivor queue (64 pending + one mini block)
constexpr int kSegIters = 2;    // 16-byte string loads per lane per segment (2 KB per wave, double-buffered)
constexpr int kRecCap = 64;     // per-wave queue of string words with a prefix hit (16 B each)

// ---------------------------------------------------------------------------
// Wave helpers
// ---------------------------------------------------------------------------
__device__ __forceinline__ int lane_id() { return __lane_id(); }

__device__ __forceinline__ uint32_t bits_below(uint64_t b) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u));
}

__device__ __forceinline__ int32_t uniform_i32(int32_t x) { return __builtin_amdgcn_readfirstlane(x); }

__device__ __forceinline__ uint64_t readlane_u64(uint64_t x, int l) {
    uint32_t lo = __builtin_amdgcn_readlane((uint32_t)x, l);
    uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(x >> 32), l);
    return ((uint64_t)hi << 32) | lo;
}

// Cross-lane moves through DPP (GFX9 data-parallel primitives): no address
// registers, no LDS.  A lane whose source is outside the pattern, or whose
// row is masked off, receives 0.
constexpr int kDppRowShr1 = 0x111, kDppRowShr2 = 0x112, kDppRowShr4 = 0x114, kDppRowShr8 = 0x118;
constexpr int kDppWaveShl1 = 0x130;  // lane i receives lane i + 1
constexpr int kDppWaveShr1 = 0x138;  // lane i receives lane i - 1
constexpr int kDppRowBcast15 = 0x142, kDppRowBcast31 = 0x143;

template <int kCtrl, int kRowMask = 0xf>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, kCtrl, kRowMask, 0xf, false);
}

template <int kCtrl, int kRowMask = 0xf>
__device__ __forceinline__ uint64_t dpp_u64(uint64_t x) {
    const uint32_t lo = dpp_u32<kCtrl, kRowMask>((uint32_t)x);
    const uint32_t hi = dpp_u32<kCtrl, kRowMask>((uint32_t)(x >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// Inclusive wave scans: shifts 1, 2, 4, 8 inside each 16-lane row, then lane
// 15 of a row is added to the next row and lane 31 to rows 2 and 3.
__device__ __forceinline__ uint32_t wave_incl_scan_u32(uint32_t x) {
    x += dpp_u32<kDppRowShr1>(x);
    x += dpp_u32<kDppRowShr2>(x);
    x += dpp_u32<kDppRowShr4>(x);
    x += dpp_u32<kDppRowShr8>(x);
    x += dpp_u32<kDppRowBcast15, 0xa>(x);
    x += dpp_u32<kDppRowBcast31, 0xc>(x);
    return x;
}

__device__ __forceinline__ uint64_t wave_incl_scan_u64(uint64_t x) {
    x += dpp_u64<kDppRowShr1>(x);
    x += dpp_u64<kDppRowShr2>(x);
    x += dpp_u64<kDppRowShr4>(x);
    x += dpp_u64<kDppRowShr8>(x);
    x += dpp_u64<kDppRowBcast15, 0xa>(x);
    x += dpp_u64<kDppRowBcast31, 0xc>(x);
    return x;
}

// Orders this wave's LDS accesses (a wave's LDS operations complete in issue
// order; the fence keeps the compiler from moving them across).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// ---------------------------------------------------------------------------
// Bit unpacking (paper Section 3.4.1 and 4.1: FOR with a per-mini-block base
// and bit width; the 64-bit variant reads through a wider window)
// ---------------------------------------------------------------------------
typedef uint64_t u64_a4 __attribute__((aligned(4)));

__device__ __forceinline__ uint64_t bits_at(cptr<uint32_t> w, uint32_t bitpos, int b) {
    cptr<uint32_t> p = w + (bitpos >> 5);
    uint32_t sh = bitpos & 31u;
    uint64_t x = *(cptr<u64_a4>)p >> sh;
    if (b > 32) {
        uint64_t hi = p[2];
        if (sh) x |= hi << (64 - sh);
    }
    return b >= 64 ? x : (x & ((uint64_t(1) << b) - 1));
}

struct MbHdr {
    int64_t base;
    cptr<uint32_t> w;
    int b;
    bool ok;
};

// Mini-block header with consistency checks (a corrupt header must not
// steer a load out of bounds).
__device__ __forceinline__ MbHdr mb_hdr(CC& c, int m) {
    MbHdr h;
    uint32_t w0 = ro(c.woff)[m], w1 = ro(c.woff)[m + 1];
    uint32_t nw = w1 - w0;
    h.ok = (w0 <= w1) && (w1 <= c.nwords) && ((nw & 7u) == 0) && (nw <= 512u);
    h.b = (int)(nw >> 3);
    h.base = ro(c.base)[m];
    h.w = ro(c.words) + (h.ok ? w0 : 0);
    if (!h.ok) h.b = 0;
    return h;
}

// Dense decode of the wave's four rows (64k + lane) of mini block m.
// DICT columns yield codes; VARLEN yields lengths.  Returns false on a
// corrupt header.
// Dense decode in two steps, so that a wave can have the loads of several
// mini blocks in flight: issue_dense reads the header and the packed words
// (raw 64-bit windows, or the full values for widths above 32), and
// finish_dense unpacks them (DELTA: a wave scan).
struct RawDense {
    MbHdr h;
    int64_t dmin;
    uint64_t raw[4];
    uint32_t sh[4];
};

__device__ __forceinline__ void issue_dense(CC& c, int m, int lane, RawDense& R) {
    R.h = mb_hdr(c, m);
    R.dmin = c.enc == ENC_DELTA ? ro(c.dmin)[m] : 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t bitpos = (uint32_t)(64 * k + lane) * (uint32_t)R.h.b;
        R.sh[k] = bitpos & 31u;
        if (R.h.b == 0) {
            R.raw[k] = 0;
        } else if (R.h.b <= 32) {
            R.raw[k] = *(cptr<u64_a4>)(R.h.w + (bitpos >> 5));
        } else {
            R.raw[k] = bits_at(R.h.w, bitpos, R.h.b);
            R.sh[k] = 0;
        }
    }
}

__device__ __forceinline__ bool finish_dense(CC& c, const RawDense& R, int lane, int64_t v[4]) {
    const MbHdr& h = R.h;
    uint64_t u[4];
    const uint64_t mask = h.b >= 64 ? ~uint64_t(0) : ((uint64_t(1) << h.b) - 1);
#pragma unroll
    for (int k = 0; k < 4; ++k) u[k] = h.b == 0 ? 0 : ((R.raw[k] >> R.sh[k]) & mask);
    if (c.enc == ENC_DELTA) {
        // value_i = anchor + i * dmin + sum_{j <= i} packed_j  (packed_0 = 0)
        const uint64_t dmin = (uint64_t)R.dmin;
        uint64_t carry = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            uint64_t s = h.b ? wave_incl_scan_u64(u[k]) : 0;
            uint32_t i = 64 * k + lane;
            v[k] = (int64_t)((uint64_t)h.base + (uint64_t)i * dmin + carry + s);
            if (h.b) carry += readlane_u64(s, 63);
        }
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = (int64_t)((uint64_t)h.base + u[k]);
    }
    return h.ok;
}

// An empty use of R's packed words: their loads must be complete here.
__device__ __forceinline__ void dense_ready(const RawDense& R) {
#pragma unroll
    for (int k = 0; k < 4; ++k) asm volatile("" ::"v"(R.raw[k]));
}

__device__ __forceinline__ bool decode_dense(CC& c, int m, int lane, int64_t v[4]) {
    RawDense R;
    issue_dense(c, m, lane, R);
    return finish_dense(c, R, lane, v);
}

// Value of row i of mini block m (random access).  DELTA sums the packed
// differences up to i.
__device__ __forceinline__ int64_t decode_at(CC& c, int m, int i, bool& ok) {
    MbHdr h = mb_hdr(c, m);
    ok = ok && h.ok;
    if (c.enc == ENC_DELTA) {
        uint64_t s = 0;
        if (h.b)
            for (int j = 1; j <= i; ++j) s += bits_at(h.w, (uint32_t)j * (uint32_t)h.b, h.b);
        return (int64_t)((uint64_t)h.base + (uint64_t)i * (uint64_t)ro(c.dmin)[m] + s);
    }
    uint64_t u = h.b ? bits_at(h.w, (uint32_t)i * (uint32_t)h.b, h.b) : 0;
    return (int64_t)((uint64_t)h.base + u);
}

// DICT code -> value (bounds-checked).
__device__ __forceinline__ int64_t dict_value(CC& c, int64_t code, bool& ok) {
    if (code < 0 || code >= c.ndict) { ok = false; return 0; }
    return ro(c.dict)[code];
}

// ---------------------------------------------------------------------------
// Zone test from the mini-block header alone.  A FOR mini block holds values
// in [base, base + 2^b - 1]; a DELTA one, anchor + i * dmin + (a sum of i
// packed differences in [0, 2^b - 1]) for i < 256.  When that interval lies
// inside a range atom every row passes, when it misses the atom none does,
// and the column need not be decoded (the paper's zone maps, Section 3.4,
// at mini-block granularity and with no bytes beyond the header).
// Returns 1: all rows pass, 0: none, -1: undecided.  Wave-uniform (scalar).
// ---------------------------------------------------------------------------
__device__ __forceinline__ int zone_test(CC& c, CP& p, int m) {
    if (p.kind != PK_RANGE && p.kind != PK_NE) return -1;
    const MbHdr h = mb_hdr(c, m);
    // int64 is exact here: |base| < 2^61, width <= 32, |dmin| < 2^31, so the
    // interval ends stay below 2^62 in magnitude.  Otherwise: undecided.
    const int64_t kLim = int64_t(1) << 61;
    if (!h.ok || h.b > 32 || h.base >= kLim || h.base <= -kLim) return -1;
    const int64_t span = h.b ? (int64_t)((uint64_t(1) << h.b) - 1) : 0;
    int64_t lo = h.base, hi = h.base;
    if (c.enc == ENC_DELTA) {
        const int64_t dmin = ro(c.dmin)[m];
        if (dmin >= (int64_t(1) << 31) || dmin <= -(int64_t(1) << 31)) return -1;
        const int64_t d = dmin * (kMB - 1);
        if (d < 0) lo += d; else hi += d;
        hi += span * (kMB - 1);
    } else {
        hi += span;
    }
    if (p.kind == PK_RANGE) {
        if (lo >= p.lo && hi <= p.hi) return 1;
        if (hi < p.lo || lo > p.hi) return 0;
        return -1;
    }
    if (hi < p.lo || lo > p.lo) return 1;  // NE: the excluded value is outside
    if (lo == hi) return 0;                // every row equals it
    return -1;
}

// ---------------------------------------------------------------------------
// Integer predicates on four dense values -> 4-bit mask
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t eval_int_pred(CP& p, cptr<int64_t> in_vals,
                                                  const int64_t v[4]) {
    uint32_t mk = 0;
    const int kind = p.kind;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        bool t;
        if (kind == PK_RANGE) {
            t = v[k] >= p.lo && v[k] <= p.hi;
        } else if (kind == PK_NE) {
            t = v[k] != p.lo;
        } else if (kind == PK_INMASK) {
            t = v[k] >= 0 && v[k] < 64 && ((p.mask >> (uint64_t)v[k]) & 1u);
        } else if (kind == PK_INLIST) {
            t = false;
            for (int j = 0; j < p.n_in; ++j) t |= v[k] == in_vals[p.in_off + j];
        } else {
            t = false;
        }
        mk |= (uint32_t)t << k;
    }
    return mk;
}

// ---------------------------------------------------------------------------
// String predicate "s1 then s2" (LIKE '%s1%s2%', paper Section 4.1) over one
// mini block, byte-parallel.
//
// The mini block's heap is read into registers in 2 KB segments of 16-byte
// loads, two segments in turn (the next one loads while the current one is
// compared): each lane holds four consecutive words, and the two words after
// them come from the next lane by a DPP lane shift.  At every byte position
// the 4-byte window is compared with the first 4 bytes of s1 and of s2
// (three byte-aligns and eight compares per word; the hit masks combine in
// scalar registers), so a chance match costs nothing until a whole 4-byte
// prefix agrees.  A word with such a hit is queued in LDS with its two
// successors; after the last segment the queued words are checked together,
// one per lane, against 8-byte windows (the rest of a longer pattern from
// memory), mapped to their row by binary search over the row offsets (LDS),
// and kept as the row's leftmost s1 start and rightmost s2 start.  A row
// contains s1 then s2 iff some s2 start b and s1 start a satisfy b >= a +
// |s1|, that is iff rightmost s2 >= leftmost s1 + |s1|.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int row_of(const uint32_t* offs, uint32_t p) {
    int lo = 0, hi = 255;  // largest r with offs[r] <= p
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (offs[mid] <= p) lo = mid; else hi = mid - 1;
    }
    return lo;
}

template <class S, class Wp>
__device__ __forceinline__ bool bytes_eq(S s, Wp w, int from, int n) {
    for (int i = from; i < n; ++i)
        if (s[i] != w[i]) return false;
    return true;
}

struct StrPattern {
    uint64_t p8, m8;  // first min(n, 8) bytes, little endian, and their mask
};

__device__ __forceinline__ StrPattern make_pattern(cptr<uint8_t> w, int n) {
    StrPattern P;
    P.p8 = *(cptr<uint64_t>)w;  // bytes past n are zero
    P.m8 = n >= 8 ? ~uint64_t(0) : ((uint64_t(1) << (8 * n)) - 1);
    P.p8 &= P.m8;
    return P;
}

struct StrLds {
    const uint32_t* tab;  // [32] the workgroup's copy of DevPred::tab (kStrTable)
    uint32_t* offs;    // [257] row start offsets within the mini block's heap
    uint32_t* first1;  // [256] leftmost s1 start (0xffffffff: none)
    uint32_t* last2;   // [256] rightmost s2 start + 1 (0: none)
    uint4* recs;       // [kRecCap] words with a prefix hit: {byte offset, word, next, the one after}
};

// Records an s1 and/or s2 start at heap position pos of the mini block: the
// row comes from a binary search over the row offsets; a word longer than 8
// bytes is checked in full where it rests.
__device__ __forceinline__ void note_start(const StrLds& L, uint32_t pos, bool m1, bool m2, CP& p,
                                           cptr<uint8_t> hs) {
    const int r = row_of(L.offs, pos);
    const uint32_t rend = L.offs[r + 1];
    if (m1 && pos + (uint32_t)p.n1 <= rend && (p.n1 <= 8 || bytes_eq(hs + pos, p.s1, 8, p.n1)))
        atomicMin(&L.first1[r], pos);
    if (m2 && pos + (uint32_t)p.n2 <= rend && (p.n2 <= 8 || bytes_eq(hs + pos, p.s2, 8, p.n2)))
        atomicMax(&L.last2[r], pos + 1);
}

// Tests 4 byte positions with 8-byte windows: q is the byte offset of word
// e0 from the 16-byte-aligned start, e1/e2 the two words after it, and the
// positions are q + kFirst .. q + kFirst + 3.
template <int kFirst>
__device__ __forceinline__ void check_word(const StrLds& L, uint32_t q, uint32_t e0, uint32_t e1, uint32_t e2,
                                           uint32_t s0, uint32_t total, const StrPattern& P1, const StrPattern& P2,
                                           CP& p, cptr<uint8_t> hs) {
    uint32_t k1 = 0, k2 = 0;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int sh = kFirst + t;  // 0..4
        const uint32_t lo = sh == 0 ? e0 : sh == 4 ? e1 : __builtin_amdgcn_alignbit(e1, e0, 8 * (sh & 3));
        const uint32_t hi = sh == 0 ? e1 : sh == 4 ? e2 : __builtin_amdgcn_alignbit(e2, e1, 8 * (sh & 3));
        const uint64_t win8 = (uint64_t)lo | ((uint64_t)hi << 32);
        const uint32_t qt = q + (uint32_t)sh;
        const bool inr = qt >= s0 && qt - s0 < total;
        k1 |= (uint32_t)(inr && (win8 & P1.m8) == P1.p8) << t;
        k2 |= (uint32_t)(inr && (win8 & P2.m8) == P2.p8) << t;
    }
    for (uint32_t k = k1 | k2; k; k &= k - 1) {
        const int t = __builtin_ctz(k);
        note_start(L, q + (uint32_t)(kFirst + t) - s0, (k1 >> t) & 1u, (k2 >> t) & 1u, p, hs);
    }
}

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// One mini block's string test between issuing its loads and using them.
// One heap segment in registers: lane l holds bytes [16 (base + it * 64 + l),
// +16) in W[it]; tx, ty are the two words after the segment (for lane 63).
struct Seg {
    uint4 W[kSegIters];
    uint32_t tx, ty;
};

struct StrTile {
    Seg cur;               // the segment being compared (the first, after str_begin)
    uint64_t lraw[4];      // packed lengths of rows 4 lane .. 4 lane + 3, unshifted
    cptr<uint4> g;         // 16-byte-aligned start of the heap bytes
    const uint8_t* gp;     // the same address, generic
    uint64_t h0, h1;       // heap byte range of the mini block
    int64_t lbase;         // minimum length
    uint32_t lsh;          // bit offset of row 4 lane's length in lraw[0]
    int b;                 // length bit width
    bool ok;
};

// Buffer resource over [p, p + nbytes): raw (stride 0) 32-bit words; a load
// whose VGPR offset + immediate offset lies past nbytes returns zeros.
constexpr int kRawBufferWord3 = 0x00020000;

// Loads heap vectors base .. base + 511 of the tile (vector v = bytes
// [16 v, 16 v + 16) from the 16-byte-aligned start) into W; vectors past
// nvec read as zero through the buffer range check.  The per-lane offset is
// the only VGPR address; the slots differ by immediate offsets.
__device__ __forceinline__ void load_segment(Seg& G, const StrTile& S, uint32_t base, uint32_t nvec, int lane) {
    const uint32_t nbytes = (nvec + 1u - base) * 16u;
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(S.gp + (uint64_t)base * 16u), 0, (int)nbytes, kRawBufferWord3);
    // The empty asm keeps the compiler from hoisting one offset register per
    // slot out of the loops: the slot offsets must stay immediates.
    int vo = lane * 16;
    asm volatile("" : "+v"(vo));
    const int vo2 = vo + 4096;
#pragma unroll
    for (int it = 0; it < kSegIters; ++it) {
        const int off = it * kWave * 16;  // below 4096: immediate on vo; else on vo2
        const u32x4 t = off < 4096 ? __builtin_amdgcn_raw_buffer_load_b128(r, vo + off, 0, 0)
                                   : __builtin_amdgcn_raw_buffer_load_b128(r, vo2 + (off - 4096), 0, 0);
        G.W[it] = make_uint4(t.x, t.y, t.z, t.w);
    }
    const uint32_t vt = base + kSegIters * kWave;  // wave-uniform: scalar load
    G.tx = G.ty = 0;
    if (vt <= nvec) {
        const u32x2 t = ((cptr<u32x2>)S.g)[2 * vt];
        G.tx = t.x;
        G.ty = t.y;
    }
}

// Issues the loads of mini block m's lengths and first heap segment.
__device__ __forceinline__ void str_begin(CC& c, int m, int lane, StrTile& S) {
    const MbHdr h = mb_hdr(c, m);
    S.h0 = ro(c.hoff)[m];
    S.h1 = ro(c.hoff)[m + 1];
    S.ok = h.ok && h.b <= 32 && S.h0 <= S.h1 && S.h1 <= c.heap_bytes && (S.h1 - S.h0) < (uint64_t(1) << 30);
    S.b = S.ok ? h.b : 0;
    S.lbase = h.base;
    const uint64_t a0 = S.h0 & ~uint64_t(15);
    S.g = (cptr<uint4>)(c.heap + a0);
    S.gp = c.heap + a0;
    const uint32_t nvec = S.ok ? (uint32_t)((S.h1 - a0 + 15u) >> 4) : 0u;
    // lengths: row 4 lane + j at bit (4 lane + j) b; one 8-byte window per row
    const uint32_t bp = 4u * (uint32_t)lane * (uint32_t)S.b;
    S.lsh = bp & 31u;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t pj = bp + (uint32_t)j * (uint32_t)S.b;
        S.lraw[j] = S.b ? *(cptr<u64_a4>)(h.w + (pj >> 5)) : 0;
    }
    if (S.ok) {
        load_segment(S.cur, S, 0, nvec, lane);
    } else {
#pragma unroll
        for (int it = 0; it < kSegIters; ++it) S.cur.W[it] = make_uint4(0u, 0u, 0u, 0u);
        S.cur.tx = S.cur.ty = 0;
    }
}

// An empty use of every word of G: the loads that fill G must be complete
// here, so the compares that follow need no wait of their own.
__device__ __forceinline__ void seg_ready(const Seg& G) {
#pragma unroll
    for (int it = 0; it < kSegIters; ++it)
        asm volatile("" ::"v"(G.W[it].x), "v"(G.W[it].y), "v"(G.W[it].z), "v"(G.W[it].w));
}

// Neighbour words of lane's segment slot it: the next lane's first two words
// (for lane 63, those of the next slot's lane 0, or the words after the
// segment).
__device__ __forceinline__ void next_words(const Seg& S, int it, int lane, uint32_t& nx, uint32_t& nx2) {
    nx = dpp_u32<kDppWaveShl1>(S.W[it].x);
    nx2 = dpp_u32<kDppWaveShl1>(S.W[it].y);
    uint32_t lx = S.tx, ly = S.ty;
    if (it + 1 < kSegIters) {
        lx = __builtin_amdgcn_readlane(S.W[it + 1 < kSegIters ? it + 1 : it].x, 0);
        ly = __builtin_amdgcn_readlane(S.W[it + 1 < kSegIters ? it + 1 : it].y, 0);
    }
    if (lane == kWave - 1) { nx = lx; nx2 = ly; }
}

// Checks queued hit words, one per lane (all lanes at once: a wave pays
// for the check once per batch of hits, not once per hit).
// A record {q, e0, e1, e2} stands for the starts q + kFirst .. + 3.
template <int kFirst>
__device__ __forceinline__ void drain_records(const StrLds& L, int nrec, uint32_t s0, uint32_t total,
                                              const StrPattern& P1, const StrPattern& P2, CP& p,
                                              cptr<uint8_t> hs, int lane) {
    wave_lds_sync();
    for (int j = lane; j < nrec; j += kWave) {
        const uint4 r = L.recs[j];
        check_word<kFirst>(L, r.x, r.y, r.z, r.w, s0, total, P1, P2, p, hs);
    }
    wave_lds_sync();
}

// Scan modes of the string test:
//   kStrMasked  (a word under 4 bytes): 4-byte windows at every byte, masked;
//   kStrShifted (words of 4 bytes or more): 4-byte windows at every byte
//               (a word and its three byte-aligns);
//   kStrTable   (both words of 7 bytes or more, with a table): every
//               occurrence covers a whole 4-byte-aligned word, which then
//               equals one of the word's four 4-byte shifts; each aligned
//               word is looked up in the 32-slot LDS table of the eight
//               shifts (DevPred::tab), one read and one compare a word, and
//               the neighbour words are gathered only on a hit.
enum : int { kStrMasked = 0, kStrShifted = 1, kStrTable = 2 };

__device__ __forceinline__ int str_mode(int n1, int n2) { return (n1 < 4 || n2 < 4) ? kStrMasked : kStrShifted; }

// Returns the 4-bit match mask of the lane's rows (row 64 k + lane -> bit k)
// for the mini block whose loads str_begin issued; clears ok on corruption.
// kOffsReady: the caller has written the row offsets (L.offs[0..256]) from
// materialised string offsets, and S carries no packed lengths.
template <int kMode, bool kOffsReady = false>
__device__ __forceinline__ uint32_t str_finish(CC& c, CP& p, int lane, int nvalid, StrTile& S,
                                               const StrLds& L, bool& ok) {
    if (!S.ok) { ok = false; return 0; }
    uint32_t* const offs = L.offs;
    const uint32_t s0 = (uint32_t)(S.h0 & 15u);
    const uint32_t nvec = (uint32_t)((S.h1 - (S.h0 - s0) + 15u) >> 4);
    if (kOffsReady) {
        reinterpret_cast<uint4*>(L.first1)[lane] = make_uint4(~0u, ~0u, ~0u, ~0u);
        reinterpret_cast<uint4*>(L.last2)[lane] = make_uint4(0u, 0u, 0u, 0u);
    } else {
    // Row offsets: lane l takes rows 4l..4l+3, so one wave scan suffices.
    uint32_t len[4], lsum = 0;
    const uint64_t lmask = (uint64_t(1) << S.b) - 1;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t sh = (S.lsh + (uint32_t)j * (uint32_t)S.b) & 31u;
        const uint32_t u = (uint32_t)((S.lraw[j] >> sh) & lmask);
        len[j] = 4 * lane + j < nvalid ? (uint32_t)S.lbase + u : 0u;
        lsum += len[j];
    }
    const uint32_t incl = wave_incl_scan_u32(lsum);
    const uint32_t total = __builtin_amdgcn_readlane(incl, 63);
    {
        uint32_t o = incl - lsum;
        uint4 ov;
        ov.x = o;
        ov.y = o + len[0];
        ov.z = ov.y + len[1];
        ov.w = ov.z + len[2];
        reinterpret_cast<uint4*>(offs)[lane] = ov;
        // Materialised here (the empty asm keeps the compiler from hoisting
        // the constant registers out of the tile loop, where they spilled).
        uint32_t ones = ~0u, zero = 0u;
        asm volatile("" : "+v"(ones), "+v"(zero));
        reinterpret_cast<uint4*>(L.first1)[lane] = make_uint4(ones, ones, ones, ones);
        reinterpret_cast<uint4*>(L.last2)[lane] = make_uint4(zero, zero, zero, zero);
    }
    if (lane == 0) offs[256] = total;
    if ((uint64_t)total != S.h1 - S.h0) { ok = false; return 0; }
    }

    const StrPattern P1 = make_pattern(p.s1, p.n1), P2 = make_pattern(p.s2, p.n2);
    // The first 4 bytes of each word (masked for kStrMasked).
    const uint32_t k1 = (uint32_t)P1.m8, k2 = (uint32_t)P2.m8;
    const uint32_t q1 = (uint32_t)P1.p8, q2 = (uint32_t)P2.p8;
    cptr<uint8_t> hs = ro(c.heap + S.h0);
    const uint32_t total_b = (uint32_t)(S.h1 - S.h0);
    int nrec = 0;
    // Window modes: does a word's 4-byte prefix start in x (x1: the word
    // after it), at x or one of its three byte-aligns?
    auto word_hit = [&](uint32_t x, uint32_t x1) -> bool {
        const uint32_t w1 = __builtin_amdgcn_alignbit(x1, x, 8);
        const uint32_t w2 = __builtin_amdgcn_alignbit(x1, x, 16);
        const uint32_t w3 = __builtin_amdgcn_alignbit(x1, x, 24);
        if (kMode == kStrMasked)
            return ((x & k1) == q1) | ((w1 & k1) == q1) | ((w2 & k1) == q1) | ((w3 & k1) == q1) |
                   ((x & k2) == q2) | ((w1 & k2) == q2) | ((w2 & k2) == q2) | ((w3 & k2) == q2);
        return (x == q1) | (w1 == q1) | (w2 == q1) | (w3 == q1) | (x == q2) | (w1 == q2) | (w2 == q2) | (w3 == q2);
    };
    // A record {q, x, y, z} holds the 12 bytes from offset q and stands for
    // 4 starts: q .. q + 3 in the window modes; q + 1 .. q + 4 for kStrTable,
    // whose hit on the aligned word y means a start in the 3 bytes before y
    // or at y itself.
    constexpr int kFirst = kMode == kStrTable ? 1 : 0;
    auto push = [&](bool cnd, uint32_t q, uint32_t x, uint32_t y, uint32_t z) {
        const uint64_t hb = __builtin_amdgcn_ballot_w64(cnd);
        if (hb) {
            const int nh = (int)__popcll(hb);
            if (nrec + nh > kRecCap) {
                drain_records<kFirst>(L, nrec, s0, total_b, P1, P2, p, hs, lane);
                nrec = 0;
            }
            if (cnd) L.recs[nrec + bits_below(hb)] = make_uint4(q, x, y, z);
            nrec += nh;
        }
    };
    uint32_t tail = 0;  // last word of the previous segment (lane 63's fourth)
    // Hot loop over one segment.  A word with a prefix hit queues its record
    // in LDS (a rare, wave-uniform branch); kStrTable gathers the
    // neighbouring words only then.
    const uint32_t rot = p.tab_rot;
    auto scan = [&](const Seg& G, uint32_t base) {
#pragma unroll
        for (int it = 0; it < kSegIters; ++it) {
            if (base + (uint32_t)it * kWave > nvec) break;  // slots past the mini block hold zeros
            const uint4 w = G.W[it];
            const uint32_t q0 = (base + (uint32_t)it * kWave + (uint32_t)lane) * 16u;
            uint32_t nx = 0, nx2 = 0;
            if (kMode != kStrTable) next_words(G, it, lane, nx, nx2);
            const uint32_t e[6] = {w.x, w.y, w.z, w.w, nx, nx2};
            if (kMode != kStrTable) {
#pragma unroll
                for (int wd = 0; wd < 4; ++wd) {
                    const bool h = word_hit(e[wd], e[wd + 1]);
                    if (__builtin_amdgcn_ballot_w64(h)) push(h, q0 + 4u * (uint32_t)wd, e[wd], e[wd + 1], e[wd + 2]);
                }
                continue;
            }
            // kStrTable: the four table reads first, so that they wait together.
            uint32_t t[4];
#pragma unroll
            for (int wd = 0; wd < 4; ++wd) {
                const uint32_t y = e[wd] ^ __builtin_amdgcn_alignbit(e[wd], e[wd], rot);
                t[wd] = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const uint8_t*>(L.tab) + (y & 0x7Cu));
            }
            // one wave vote for the four words: hits are rare
            if (!__builtin_amdgcn_ballot_w64((t[0] == e[0]) | (t[1] == e[1]) | (t[2] == e[2]) | (t[3] == e[3])))
                continue;
#pragma unroll
            for (int wd = 0; wd < 4; ++wd) {
                const bool h = t[wd] == e[wd];
                if (!__builtin_amdgcn_ballot_w64(h)) continue;
                // The word before: the previous lane's last (lane 0: the
                // previous slot's lane 63, or the segment before's); the word
                // after: the next lane's first for the lane's last word.
                uint32_t xp, y1;
                if (wd) {
                    xp = e[wd - 1];
                } else {
                    const uint32_t prev = it ? __builtin_amdgcn_readlane(G.W[it ? it - 1 : 0].w, 63) : tail;
                    xp = (uint32_t)__builtin_amdgcn_update_dpp((int)prev, (int)w.w, kDppWaveShr1, 0xf, 0xf, false);
                }
                if (wd < 3) {
                    y1 = e[wd + 1];
                } else {
                    uint32_t b;
                    next_words(G, it, lane, y1, b);
                }
                push(h, q0 + 4u * (uint32_t)wd - 4u, xp, e[wd], y1);
            }
        }
        if (kMode == kStrTable) tail = __builtin_amdgcn_readlane(G.W[kSegIters - 1].w, 63);
    };
    // Two segment buffers in turn: the next segment's loads are in flight
    // while the current one is compared.  seg_ready makes the wait for the
    // current buffer explicit before the next loads are issued: left to the
    // compiler, the join after a conditional load merges the two paths'
    // outstanding-load counts, and the wait before the compares would then
    // also cover the loads just issued.
    constexpr uint32_t kSeg = kSegIters * kWave;
    Seg other;
    for (uint32_t base = 0;; base += 2 * kSeg) {
        const bool more1 = base + kSeg < nvec;
        seg_ready(S.cur);
        if (more1) load_segment(other, S, base + kSeg, nvec, lane);
        scan(S.cur, base);
        if (!more1) break;
        const bool more2 = base + 2 * kSeg < nvec;
        seg_ready(other);
        if (more2) load_segment(S.cur, S, base + 2 * kSeg, nvec, lane);
        scan(other, base + kSeg);
        if (!more2) break;
    }
    if (nrec) drain_records<kFirst>(L, nrec, s0, total_b, P1, P2, p, hs, lane);
    wave_lds_sync();
    uint32_t res = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        int i = 64 * k + lane;
        uint32_t f = L.first1[i], e = L.last2[i];
        bool hit = i < nvalid && f != 0xFFFFFFFFu && e != 0u && (uint64_t)(e - 1) >= (uint64_t)f + p.n1;
        res |= (uint32_t)hit << k;
    }
    return res;
}

template <int kMode>
__device__ __forceinline__ uint32_t str_pred(CC& c, CP& p, int m, int lane, int nvalid, const StrLds& L,
                                             bool& ok) {
    StrTile S;
    str_begin(c, m, lane, S);
    return str_finish<kMode>(c, p, lane, nvalid, S, L, ok);
}

// ---------------------------------------------------------------------------
// FSST strings (Sections 3.4.2 and 4.1): each chunk carries a table of up to
// 255 symbols of 1..8 bytes; a record is a run of one-byte codes, code 255
// escaping the literal byte after it.  The string test never writes a
// decoded byte: LIKE '%s1%s2%' is a byte automaton D with S = |s1| + |s2|
// + 1 states (the two words' Knuth-Morris-Pratt automata in sequence, built
// with the plan), and the workgroup lifts it to the chunk's codes,
//     T[q][c] = the state D reaches from q over the bytes of symbol c,
// so that a lane steps one code per LDS byte read.  The escape joins the
// same table: T[q][255] = S + q, whose row is D itself (the literal byte's
// step), and codes the chunk does not define lead to a sink row 2S.  T has
// 2S + 1 rows of 256 bytes (DevQuery::fs_lds_off); rows S .. 2S are loaded
// with the plan, rows 0 .. S-1 for every chunk.
// ---------------------------------------------------------------------------

// Rows S .. 2S of the plan's code table: the byte automaton and the sink.
__device__ void fsst_load_dfa(CQ& Q, uint8_t* smem_shared) {
    if (Q.fs_pred < 0) return;
    const uint32_t S = (uint32_t)Q.fs_states;
    uint8_t* T = smem_shared + Q.fs_lds_off;
    cptr<uint4> src = (cptr<uint4>)Q.fs_dfa;
    uint4* dst = reinterpret_cast<uint4*>(T + S * 256);
    for (uint32_t e = threadIdx.x; e < S * 16; e += blockDim.x) dst[e] = ld4(src, e);
    for (uint32_t e = threadIdx.x; e < 256; e += blockDim.x) T[2 * S * 256 + e] = (uint8_t)(2 * S);
}

// Rows 0 .. S-1 of the code table for chunk k (rows S .. 2S in place).
__device__ void fsst_load_chunk(CQ& Q, uint8_t* smem_shared, int k) {
    CP& P = Q.preds[Q.fs_pred];
    CC& c = Q.cols[P.col];
    const uint32_t S = (uint32_t)Q.fs_states;
    uint8_t* T = smem_shared + Q.fs_lds_off;
    const uint8_t* D = T + S * 256;
    cptr<uint8_t> tab = ro(c.symtab) + (size_t)k * (256 * 8 + 256);
    for (uint32_t code = threadIdx.x; code < 256; code += blockDim.x) {
        const uint64_t sv = ((cptr<uint64_t>)tab)[code];
        const uint32_t L = code < 255 ? (uint32_t)tab[256 * 8 + code] : 0u;
        for (uint32_t q = 0; q < S; ++q) {
            uint32_t st;
            if (code == 255) {
                st = S + q;
            } else if (L == 0 || L > 8) {
                st = 2 * S;
            } else {
                st = q;
                for (uint32_t b = 0; b < L; ++b) st = D[st * 256 + (uint32_t)((sv >> (8 * b)) & 0xFF)];
            }
            T[q * 256 + code] = (uint8_t)st;
        }
    }
}

// A lane's run of codes through a 48-byte register window x:y:z of the
// heap (x at byte offset A from base, 16-byte aligned, A <= pos < A + 16):
// a peek reads x and y only, so the load that refills z has the 16 bytes of
// y to work through before it is waited for.  Offsets are 32-bit, relative
// to the 16-byte-aligned start of the mini block's codes; the heap is
// padded, so the window's loads stay inside it while pos is at most the
// mini block's end.
struct CodeReader {
    cptr<uint4> base;
    uint32_t pos, A;
    uint4 x, y, z;
    __device__ __forceinline__ void init(const uint8_t* heap, uint64_t h0, uint32_t p) {
        const uint64_t a0 = h0 & ~uint64_t(15);
        base = (cptr<uint4>)(heap + a0);
        pos = (uint32_t)(h0 - a0) + p;
        A = pos & ~15u;
        x = ld4(base, A >> 4);
        y = ld4(base, (A >> 4) + 1u);
        z = ld4(base, (A >> 4) + 2u);
    }
    // the next 4 code bytes, first in the low byte
    // (two-way selects: a four-way pick by o >> 2 compiles to a stack copy
    // of the window and an indexed load)
    __device__ __forceinline__ uint32_t peek4() const {
        const uint32_t o = pos - A;
        const bool half = (o & 8u) != 0;
        const uint32_t a0 = half ? x.z : x.x, a1 = half ? x.w : x.y, b0 = half ? y.x : x.z;
        const uint32_t lo = __builtin_amdgcn_alignbyte(a1, a0, o & 3u);
        const uint32_t hi = __builtin_amdgcn_alignbyte(b0, a1, o & 3u);
        return (o & 4u) ? hi : lo;
    }
    // the next 16 code bytes, four per word (a: the first four)
    __device__ __forceinline__ void peek16(uint32_t& a, uint32_t& b, uint32_t& c, uint32_t& d) const {
        const uint32_t o = pos - A;
        const bool half = (o & 8u) != 0, q = (o & 4u) != 0;
        const uint32_t B0 = half ? x.z : x.x, B1 = half ? x.w : x.y, B2 = half ? y.x : x.z, B3 = half ? y.y : x.w;
        const uint32_t B4 = half ? y.z : y.x, B5 = half ? y.w : y.y;
        const uint32_t c0 = q ? B1 : B0, c1 = q ? B2 : B1, c2 = q ? B3 : B2, c3 = q ? B4 : B3, c4 = q ? B5 : B4;
        a = __builtin_amdgcn_alignbyte(c1, c0, o & 3u);
        b = __builtin_amdgcn_alignbyte(c2, c1, o & 3u);
        c = __builtin_amdgcn_alignbyte(c3, c2, o & 3u);
        d = __builtin_amdgcn_alignbyte(c4, c3, o & 3u);
    }
    // the next 8 code bytes (a: the first four)
    __device__ __forceinline__ void peek8(uint32_t& a, uint32_t& b) const {
        const uint32_t o = pos - A;
        const bool half = (o & 8u) != 0, q = (o & 4u) != 0;
        const uint32_t B0 = half ? x.z : x.x, B1 = half ? x.w : x.y, B2 = half ? y.x : x.z, B3 = half ? y.y : x.w;
        const uint32_t c0 = q ? B1 : B0, c1 = q ? B2 : B1, c2 = q ? B3 : B2;
        a = __builtin_amdgcn_alignbyte(c1, c0, o & 3u);
        b = __builtin_amdgcn_alignbyte(c2, c1, o & 3u);
    }
    __device__ __forceinline__ void advance(uint32_t n) {
        pos += n;
        if (pos - A < 16) return;
        if (pos - A < 32) {
            x = y;
            y = z;
            A += 16;
            z = ld4(base, (A >> 4) + 2u);
        } else {
            A = pos & ~15u;
            x = ld4(base, A >> 4);
            y = ld4(base, (A >> 4) + 1u);
            z = ld4(base, (A >> 4) + 2u);
        }
    }
};

// Code lengths of rows 4 lane .. 4 lane + 3 of FSST mini block m (rows from
// nvalid on: 0) and the mini block's code range; false on a corrupt header.
__device__ __forceinline__ bool fsst_lengths(CC& c, int m, int lane, int nvalid, uint32_t rl[4], uint32_t& lsum,
                                             uint32_t& incl, uint64_t& h0) {
    const MbHdr h = mb_hdr(c, m);
    h0 = ro(c.hoff)[m];
    const uint64_t h1 = ro(c.hoff)[m + 1];
    if (!(h.ok && h.b <= 32 && h0 <= h1 && h1 <= c.heap_bytes && (h1 - h0) < (uint64_t(1) << 30))) return false;
    lsum = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int r = 4 * lane + j;
        rl[j] = r < nvalid ? (uint32_t)h.base + (uint32_t)(h.b ? bits_at(h.w, (uint32_t)r * (uint32_t)h.b, h.b) : 0) : 0u;
        lsum += rl[j];
    }
    incl = wave_incl_scan_u32(lsum);
    return (uint64_t)__builtin_amdgcn_readlane(incl, 63) == h1 - h0;
}

// The string atom on FSST mini block m: returns the mask of rows that
// contain s1 and, after its leftmost end, s2 (row 64 k + lane -> bit k).
// Lane l takes rows 4 l .. 4 l + 3, whose codes are contiguous in the heap,
// sixteen codes per step.  fl: 256 bytes of the wave's LDS for the
// transposition.
__device__ __forceinline__ uint32_t fsst_pred(CQ& Q, CC& c, int m, int lane, int nvalid, uint8_t* fl,
                                              const uint8_t* smem_shared, bool& ok) {
    // The table is the first thing in the shared area (fs_lds_off == 0), so
    // its address is a constant and a step's LDS address is one byte
    // permute: {code, state, 0, 0}.
    const uint8_t* T = smem_shared;
    const uint32_t S = (uint32_t)Q.fs_states, acc = S - 1;
    uint32_t rl[4], lsum, incl;
    uint64_t h0;
    if (!fsst_lengths(c, m, lane, nvalid, rl, lsum, incl, h0)) { ok = false; return 0; }
    CodeReader R;
    R.init(c.heap, h0, incl - lsum);
    uint32_t res = 0;
#pragma unroll 1
    for (int r = 0; r < 4; ++r) {
        // (a select, not rl[r]: a dynamic index would put rl in scratch)
        uint32_t rem = r == 0 ? rl[0] : r == 1 ? rl[1] : r == 2 ? rl[2] : rl[3];
        uint32_t st = 0;
        while (rem) {
            // sixteen codes a step (most records take one or two): the
            // states after 1 .. 16 codes, then the one after nq of them
            uint32_t qa, qb, qc, qd;
            R.peek16(qa, qb, qc, qd);
            const uint32_t nq = min(rem, 16u);
            auto step = [&](uint32_t s, uint32_t w, uint32_t sel) -> uint32_t {
                return T[__builtin_amdgcn_perm(s, w, sel)];
            };
            const uint32_t x0 = step(st, qa, 0x0c0c0400u), x1 = step(x0, qa, 0x0c0c0401u);
            const uint32_t x2 = step(x1, qa, 0x0c0c0402u), x3 = step(x2, qa, 0x0c0c0403u);
            const uint32_t x4 = step(x3, qb, 0x0c0c0400u), x5 = step(x4, qb, 0x0c0c0401u);
            const uint32_t x6 = step(x5, qb, 0x0c0c0402u), x7 = step(x6, qb, 0x0c0c0403u);
            const uint32_t x8 = step(x7, qc, 0x0c0c0400u), x9 = step(x8, qc, 0x0c0c0401u);
            const uint32_t x10 = step(x9, qc, 0x0c0c0402u), x11 = step(x10, qc, 0x0c0c0403u);
            const uint32_t x12 = step(x11, qd, 0x0c0c0400u), x13 = step(x12, qd, 0x0c0c0401u);
            const uint32_t x14 = step(x13, qd, 0x0c0c0402u);
            uint32_t x15 = step(x14, qd, 0x0c0c0403u);
            // (an empty use keeps the last reads unconditional: the compiler
            // otherwise branches on nq around them)
            asm volatile("" : "+v"(x15));
            {
                // a select tree on the bits of nq - 1
                const uint32_t i = nq - 1u;
                const bool b0 = (i & 1u) != 0, b1 = (i & 2u) != 0, b2 = (i & 4u) != 0, b3 = (i & 8u) != 0;
                const uint32_t t0 = b0 ? x1 : x0, t1 = b0 ? x3 : x2, t2 = b0 ? x5 : x4, t3 = b0 ? x7 : x6;
                const uint32_t t4 = b0 ? x9 : x8, t5 = b0 ? x11 : x10, t6 = b0 ? x13 : x12, t7 = b0 ? x15 : x14;
                const uint32_t u0 = b1 ? t1 : t0, u1 = b1 ? t3 : t2, u2 = b1 ? t5 : t4, u3 = b1 ? t7 : t6;
                const uint32_t v0 = b2 ? u1 : u0, v1 = b2 ? u3 : u2;
                st = b3 ? v1 : v0;
            }
            // matched: the rest of the record is skipped
            const uint32_t adv = st == acc ? rem : nq;
            rem -= adv;
            R.advance(adv);
        }
        if (st >= S) ok = false;  // an escape without its byte, or a code the table does not define
        res |= (uint32_t)(st == acc) << r;
    }
    // rows 4 lane + j -> rows 64 k + lane, through LDS
    reinterpret_cast<uint32_t*>(fl)[lane] =
        (res & 1u) | ((res >> 1) & 1u) << 8 | ((res >> 2) & 1u) << 16 | ((res >> 3) & 1u) << 24;
    wave_lds_sync();
    uint32_t mask = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) mask |= (uint32_t)(fl[64 * k + lane] != 0) << k;
    wave_lds_sync();
    return mask;
}

// ---------------------------------------------------------------------------
// Value slots carried by a surviving row.  Fact-column loads occupy slots
// 0..nloads-1, probe payloads the slots after them.  In the fused kernel the
// slots live in the wave's LDS area (one int64 column per lane, so runtime
// slot ids cost nothing); the fragmented kernels keep them in registers.
// ---------------------------------------------------------------------------
struct LdsSlots {
    int64_t* p;  // this lane's slot 0; slot s at p[s * kWave]
    __device__ __forceinline__ void set(int id, int64_t x) const { p[id * kWave] = x; }
    __device__ __forceinline__ int64_t get(int id) const { return p[id * kWave]; }
};

struct RegSlots {
    int64_t v[kMaxSlots];
    __device__ __forceinline__ void set(int id, int64_t x) {
#pragma unroll
        for (int i = 0; i < kMaxSlots; ++i)
            if (i == id) v[i] = x;
    }
    __device__ __forceinline__ int64_t get(int id) const {
        int64_t x = 0;
#pragma unroll
        for (int i = 0; i < kMaxSlots; ++i)
            if (i == id) x = v[i];
        return x;
    }
};

__device__ __forceinline__ uint32_t hash32(int32_t key, int log2cap) {
    return log2cap ? ((uint32_t)key * 0x9E3779B1u) >> (32 - log2cap) : 0u;
}

// Linear-probing lookup; returns the slot or -1.
template <bool kLds>
__device__ __forceinline__ int hash_find(CH& h, const uint8_t* smem_shared, int64_t key) {
    if (key < INT32_MIN || key > INT32_MAX || key == kEmptyKey) return -1;
    const int32_t k = (int32_t)key;
    const int32_t* lkeys = reinterpret_cast<const int32_t*>(smem_shared + h.lds_off);
    cptr<int32_t> gkeys = ro(h.keys);
    uint32_t s = hash32(k, h.log2cap);
    for (uint32_t n = 0; n <= h.cap_mask; ++n) {
        int32_t x = kLds ? lkeys[s] : gkeys[s];
        if (x == k) return (int)s;
        if (x == kEmptyKey) return -1;
        s = (s + 1) & h.cap_mask;
    }
    return -1;
}

// LDS filter test: false means the key is certainly absent.
__device__ __forceinline__ bool filter_maybe(CH& h, const uint8_t* smem_shared, int64_t key) {
    if (h.filt_lds_off < 0) return true;
    const uint32_t b = filter_bit((int32_t)key, h.flog2), b2 = filter_bit2((int32_t)key, h.flog2);
    const uint32_t* f = reinterpret_cast<const uint32_t*>(smem_shared + h.filt_lds_off);
    const uint32_t w = f[b >> 5];  // b2 lies in the same word
    return ((w >> (b & 31)) & (w >> (b2 & 31)) & 1u) != 0;
}

// Key-range bitmap test (the table has one: h.bits != nullptr).
__device__ __forceinline__ bool bitmap_has(CH& h, const uint8_t* smem_shared, int64_t key) {
    const uint64_t d = (uint64_t)key - (uint64_t)h.bmin;
    if (d >= h.bspan) return false;
    const uint32_t w = h.bits_lds_off >= 0
                           ? reinterpret_cast<const uint32_t*>(smem_shared + h.bits_lds_off)[d >> 5]
                           : ro(h.bits)[d >> 5];
    return (w >> (d & 31)) & 1u;
}

// The same test on the bitmap in device memory (kernels without the fused
// kernel's LDS copies).
__device__ __forceinline__ bool bitmap_has_global(CH& h, int64_t key) {
    const uint64_t d = (uint64_t)key - (uint64_t)h.bmin;
    return d < h.bspan && ((ro(h.bits)[d >> 5] >> (d & 31)) & 1u);
}

// Membership of the lane's four keys (mask bit k: row 64 k + lane is live):
// four independent bit tests when the table has a bitmap, else the hash
// chains probed in lockstep so that their loads are in flight together.
template <bool kLds>
__device__ __forceinline__ uint32_t hash_member4(CH& h, const uint8_t* smem_shared, const int64_t key[4],
                                                 uint32_t live) {
    if (h.filt_lds_off >= 0) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (key[k] < INT32_MIN || key[k] > INT32_MAX || !filter_maybe(h, smem_shared, key[k])) live &= ~(1u << k);
        if (__ballot(live != 0) == 0) return 0;
    }
    if (h.bits) {
        uint32_t found = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            found |= (uint32_t)(((live >> k) & 1u) && bitmap_has(h, smem_shared, key[k])) << k;
        return found;
    }
    const int32_t* lkeys = reinterpret_cast<const int32_t*>(smem_shared + h.lds_off);
    cptr<int32_t> gkeys = ro(h.keys);
    uint32_t slot[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if (key[k] < INT32_MIN || key[k] > INT32_MAX || key[k] == kEmptyKey) live &= ~(1u << k);
        slot[k] = hash32((int32_t)key[k], h.log2cap);
    }
    uint32_t found = 0;
    for (uint32_t n = 0; n <= h.cap_mask && __ballot(live != 0); ++n) {
        int32_t x[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) x[k] = (live >> k) & 1u ? (kLds ? lkeys[slot[k]] : gkeys[slot[k]]) : kEmptyKey;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (!((live >> k) & 1u)) continue;
            if (x[k] == (int32_t)key[k]) {
                found |= 1u << k;
                live &= ~(1u << k);
            } else if (x[k] == kEmptyKey) {
                live &= ~(1u << k);
            } else {
                slot[k] = (slot[k] + 1) & h.cap_mask;
            }
        }
    }
    return found;
}

template <bool kLds>
__device__ __forceinline__ int64_t hash_payload(CH& h, const uint8_t* smem_shared, int k,
                                                int slot) {
    if (kLds) {
        // payload arrays follow the keys at the same relative offsets
        const uint8_t* base = smem_shared + h.lds_off + ((const uint8_t*)h.pay[k] - (const uint8_t*)h.keys);
        return h.pay64[k] ? reinterpret_cast<const int64_t*>(base)[slot]
                          : (int64_t)reinterpret_cast<const int32_t*>(base)[slot];
    }
    cptr<uint8_t> base = ro((const uint8_t*)h.pay[k]);
    return h.pay64[k] ? ((cptr<int64_t>)base)[slot] : (int64_t)((cptr<int32_t>)base)[slot];
}

// ---------------------------------------------------------------------------
// Aggregation of one surviving row into the (LDS or global) group table
// ---------------------------------------------------------------------------
template <class S>
__device__ __forceinline__ bool group_index(CQ& Q, const S& sv, int64_t& g) {
    g = 0;
    for (int k = 0; k < Q.nkeys; ++k) {
        CK& K = Q.keys[k];
        int64_t d = sv.get(K.slot) - K.min;
        if (d < 0 || d >= K.card) return false;
        g += d * K.stride;
    }
    return true;
}

template <class S>
__device__ __forceinline__ int64_t acc_value(CA& A, const S& sv) {
    int64_t prod = 1;
    for (int t = 0; t < A.nterms; ++t) {
        CT& T = A.t[t];
        int64_t x = T.slot >= 0 ? T.mul * sv.get(T.slot) + T.add : T.add;
        prod *= x;
    }
    return prod;
}

// Row of group g in the group table T: g itself (direct table), or the
// slot that g holds in the hash table, claimed with a compare-and-swap on
// the first free slot of its linear probe sequence (-1: no slot free, which
// the table's size rules out).
__device__ __forceinline__ int64_t agg_row(CQ& Q, unsigned long long* T, int64_t g) {
    if (!Q.agg_hash) return g;
    const uint64_t n = (uint64_t)Q.ngroups, mask = n - 1;
    unsigned long long* K = T + n * (uint64_t)Q.nacc;
    const unsigned long long key = (unsigned long long)g + 1ull;
    uint64_t h = ((uint64_t)key * 0x9E3779B97F4A7C15ull) >> 17;
    for (uint64_t t = 0; t < n; ++t) {
        h &= mask;
        unsigned long long k = __hip_atomic_load(&K[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (k == 0ull) k = atomicCAS(&K[h], 0ull, key);
        if (k == 0ull || k == key) return (int64_t)h;
        ++h;
    }
    return -1;
}

// false: the hash group table had no free slot.  kHash: the batch has a
// plan with a hash group table (only those instantiations carry its code).
template <bool kHash, class S>
__device__ __forceinline__ bool aggregate_row(CQ& Q, uint8_t* smem_shared, unsigned long long* gagg, const S& sv,
                                              int64_t g) {
    const int nacc = Q.nacc;
    unsigned long long* T = Q.agg_lds
        ? reinterpret_cast<unsigned long long*>(smem_shared + Q.agg_lds_off) + g * nacc
        : gagg + g * nacc;
    if constexpr (kHash) {
        if (Q.agg_hash) {
            const int64_t r = agg_row(Q, gagg, g);
            if (r < 0) return false;
            T = gagg + r * nacc;
        }
    }
    atomicAdd(&T[0], 1ull);
    for (int a = 1; a < nacc; ++a) atomicAdd(&T[a], (unsigned long long)acc_value(Q.accs[a], sv));
    return true;
}

__device__ __forceinline__ unsigned long long ld_acq(const unsigned long long* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Copy a small direct group table T to the plan's pinned host buffer (paper
// Section 3.1: the aggregate is returned to the host) and clear it and the
// status word for the next execution.  The table goes out whole, empty
// groups included: the host drops those.  A compaction would put a count, a
// position and then one load after the other in series for each group, about
// 1 us each; here all loads of up to four entries a thread wait once.  Run
// by nthreads threads (tid among them) after every workgroup has finished.
__device__ void emit_table(CQ& Q, unsigned long long* T, uint32_t* status, int tid, int nthreads) {
    const int n = (int)Q.ngroups * Q.nacc;  // at most kEmitEntries
    int64_t* out = Q.host_out + 2;
    for (int e0 = tid; e0 < n; e0 += 4 * nthreads) {
        unsigned long long v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = e0 + k * nthreads < n ? ld_acq(&T[e0 + k * nthreads]) : 0ull;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (e0 + k * nthreads < n) {
                out[e0 + k * nthreads] = (int64_t)v[k];
                T[e0 + k * nthreads] = 0;
            }
    }
    if (tid == 0) {
        const uint32_t st = __hip_atomic_exchange(status, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        Q.host_out[0] = (int64_t)st;
        Q.host_out[1] = 1;  // the table is present
    }
}
}  // namespace
}  // namespace dpf
