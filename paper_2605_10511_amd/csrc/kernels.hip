// kernels.hip -- gfx950 kernels of the data-path-fusion query library other
// than the fused one (fused.h).
//
//  * hash_count / hash_insert: the build side (Section 3.1, Kernel #1).
//  * emit_kernel: the records of a large group table to the host.
//  * frag_*: the plan as separate kernels with materialised intermediates
//    (Section 5.1, the multi-kernel baseline).
#include "device.h"

namespace dpf {
namespace {

// ---------------------------------------------------------------------------
// Hash build (dimension scan -> filter -> insert)
//
// Two scans of the build side: hash_count sizes the table, hash_insert fills
// it.  Both are bound by latency: a wave has few mini blocks (three, for a
// dimension of 6M rows), and each is a chain of dependent reads.  So a mini
// block that a filter leaves empty reads nothing more, the four rows of a
// lane walk their probe and insert chains in lockstep (one wait for four
// rows), and the count's results are reduced per workgroup before they meet
// in device memory: one set of atomics a thread, all on the same six words,
// took 0.6 of the 0.7 ms that a joined build over 6M orders took in all
// (now count and insert 0.17 ms together).
// ---------------------------------------------------------------------------

// Slots of the lane's four keys in a table in device memory (-1: absent);
// live: the rows to look up (bit k).  Returns the rows found.
__device__ __forceinline__ uint32_t hash_slots4(CH& h, const int64_t key[4], uint32_t live, int slot[4]) {
    uint32_t s[4], found = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        slot[k] = -1;
        if (key[k] < INT32_MIN || key[k] > INT32_MAX || key[k] == kEmptyKey) live &= ~(1u << k);
        s[k] = hash32((int32_t)key[k], h.log2cap);
    }
    if (h.bits) {  // membership settles most rows of a selective join
        uint32_t in = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) in |= (uint32_t)(((live >> k) & 1u) && bitmap_has_global(h, key[k])) << k;
        live = in;
    }
    cptr<int32_t> keys = ro(h.keys);
    for (uint32_t n = 0; n <= h.cap_mask && __ballot(live != 0); ++n) {
        int32_t x[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) x[k] = (live >> k) & 1u ? keys[s[k]] : kEmptyKey;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (!((live >> k) & 1u)) continue;
            if (x[k] == (int32_t)key[k]) {
                found |= 1u << k;
                slot[k] = (int)s[k];
                live &= ~(1u << k);
            } else if (x[k] == kEmptyKey) {
                live &= ~(1u << k);
            } else {
                s[k] = (s[k] + 1) & h.cap_mask;
            }
        }
    }
    return found;
}

// Qualifying rows of mini block m (row 64 k + lane -> bit k), with their keys
// and payloads.
__device__ __forceinline__ uint32_t hash_tile_mask(CHB& A, int m, int lane, int nvalid,
                                                   int64_t key[4], int64_t pay[2][4], bool& ok) {
    uint32_t mask = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) mask |= (uint32_t)(64 * k + lane < nvalid) << k;
    // every header is checked, also of columns that the filters leave unread
    ok &= mb_hdr(A.cols[A.key_col], m).ok;
    for (int j = 0; j < A.npay; ++j)
        if (A.pay_src[j] < 0) ok &= mb_hdr(A.cols[A.pay_col[j]], m).ok;
    for (int p = 0; p < A.npreds; ++p) ok &= mb_hdr(A.cols[A.preds[p].col], m).ok;
    for (int s = 0; s < A.nsub; ++s) ok &= mb_hdr(A.cols[A.sub[s].fk_col], m).ok;
    int64_t v[4];
    for (int p = 0; p < A.npreds; ++p) {
        CP& P = A.preds[p];
        const int z = zone_test(A.cols[P.col], P, m);
        if (z == 1) continue;
        if (z == 0) return 0;
        ok &= decode_dense(A.cols[P.col], m, lane, v);
        mask &= eval_int_pred(P, A.in_vals, v);
        if (__ballot(mask != 0) == 0) return 0;
    }
    // A joined build side (Section 3.1, Kernel #2): each row must find its
    // foreign key in every probed table; payloads may come from those tables.
    for (int s = 0; s < A.nsub; ++s) {
        CPR& P = A.sub[s];
        CC& fc = A.cols[P.fk_col];
        int64_t fk[4];
        int slot[4];
        ok &= decode_dense(fc, m, lane, fk);
        if (fc.enc == ENC_DICT)
#pragma unroll
            for (int k = 0; k < 4; ++k) fk[k] = dict_value(fc, fk[k], ok);
        mask &= hash_slots4(P.h, fk, mask, slot);
        if (__ballot(mask != 0) == 0) return 0;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            if (j >= A.npay || A.pay_src[j] != s) continue;
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if ((mask >> k) & 1u) pay[j][k] = hash_payload<false>(P.h, nullptr, A.pay_col[j], slot[k]);
        }
    }
    CC& kc = A.cols[A.key_col];
    ok &= decode_dense(kc, m, lane, key);
    if (kc.enc == ENC_DICT)
#pragma unroll
        for (int k = 0; k < 4; ++k) key[k] = dict_value(kc, key[k], ok);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        if (j >= A.npay || A.pay_src[j] >= 0) continue;  // taken from a probe above
        CC& pc = A.cols[A.pay_col[j]];
        ok &= decode_dense(pc, m, lane, pay[j]);
        if (pc.enc == ENC_DICT)
#pragma unroll
            for (int k = 0; k < 4; ++k) pay[j][k] = dict_value(pc, pay[j][k], ok);
    }
    return mask;
}

// Minimum (kMax: maximum) over the wave, in every lane.
template <bool kMax>
__device__ __forceinline__ long long wave_minmax(long long x) {
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const long long y = __shfl_xor(x, d, kWave);
        x = kMax ? max(x, y) : min(x, y);
    }
    return x;
}

__global__ __launch_bounds__(kBlock) void hash_count_kernel(const HashBuildArgs* __restrict__ args) {
    __shared__ long long part[kWaves][7];
    CHB& A = *ro(args);
    const int lane = lane_id();
    const int wave = uniform_i32((int)(threadIdx.x >> 6));
    const int gw = uniform_i32((int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6));  // wave-uniform
    const int nw = (gridDim.x * blockDim.x) >> 6;
    bool ok = true;
    long long cnt = 0;
    long long mn0 = INT64_MAX, mx0 = INT64_MIN, mn1 = INT64_MAX, mx1 = INT64_MIN, mn2 = INT64_MAX, mx2 = INT64_MIN;
    for (int m = gw; m < A.nmb; m += nw) {
        const int nvalid = (int)min((int64_t)kMB, A.nrows - (int64_t)m * kMB);
        int64_t key[4], pay[2][4];
        uint32_t mask = hash_tile_mask(A, m, lane, nvalid, key, pay, ok);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (!((mask >> k) & 1u)) continue;
            cnt += 1;
            mn0 = min(mn0, (long long)key[k]);
            mx0 = max(mx0, (long long)key[k]);
            if (A.npay > 0) { mn1 = min(mn1, (long long)pay[0][k]); mx1 = max(mx1, (long long)pay[0][k]); }
            if (A.npay > 1) { mn2 = min(mn2, (long long)pay[1][k]); mx2 = max(mx2, (long long)pay[1][k]); }
        }
    }
    // wave, then workgroup, then one atomic per value and workgroup
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) cnt += __shfl_xor(cnt, d, kWave);
    mn0 = wave_minmax<false>(mn0);
    mx0 = wave_minmax<true>(mx0);
    if (A.npay > 0) { mn1 = wave_minmax<false>(mn1); mx1 = wave_minmax<true>(mx1); }
    if (A.npay > 1) { mn2 = wave_minmax<false>(mn2); mx2 = wave_minmax<true>(mx2); }
    const bool bad = __ballot(!ok) != 0;
    if (lane == 0) {
        part[wave][0] = cnt;
        part[wave][1] = mn0; part[wave][2] = mx0;
        part[wave][3] = mn1; part[wave][4] = mx1;
        part[wave][5] = mn2; part[wave][6] = mx2;
        if (bad) atomicOr(A.status, ST_CORRUPT);
    }
    __syncthreads();
    const int j = threadIdx.x;
    if (j < 7) {
        long long x = part[0][j];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) {
            const long long y = part[w][j];
            x = j == 0 ? x + y : (j & 1) ? min(x, y) : max(x, y);
        }
        if (j == 0) {
            if (x) atomicAdd(A.count, (unsigned long long)x);
        } else if (j & 1) {
            if (x != INT64_MAX) atomicMin(&A.mm[j - 1], x);
        } else if (x != INT64_MIN) {
            atomicMax(&A.mm[j - 1], x);
        }
    }
}

__global__ __launch_bounds__(kBlock) void hash_insert_kernel(const HashBuildArgs* __restrict__ args, HashTableArgs t) {
    CHB& A = *ro(args);
    const int lane = lane_id();
    const int gw = uniform_i32((int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6));  // wave-uniform
    const int nw = (gridDim.x * blockDim.x) >> 6;
    bool ok = true;
    uint32_t flags = 0;
    for (int m = gw; m < A.nmb; m += nw) {
        const int nvalid = (int)min((int64_t)kMB, A.nrows - (int64_t)m * kMB);
        int64_t key[4], pay[2][4];
        const uint32_t mask = hash_tile_mask(A, m, lane, nvalid, key, pay, ok);
        uint32_t live = mask, won = 0, s[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (((live >> k) & 1u) && (key[k] < INT32_MIN || key[k] > INT32_MAX || key[k] == kEmptyKey)) {
                flags |= ST_UNSUPPORTED;
                live &= ~(1u << k);
            }
            s[k] = hash32((int32_t)key[k], t.log2cap);
        }
        for (uint32_t n = 0; __ballot(live != 0); ++n) {
            if (n > t.cap_mask) { flags |= live ? ST_CAPACITY : 0u; break; }
            int32_t prev[4];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if ((live >> k) & 1u) prev[k] = atomicCAS(&t.keys[s[k]], kEmptyKey, (int32_t)key[k]);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (!((live >> k) & 1u)) continue;
                if (prev[k] == kEmptyKey) {
                    won |= 1u << k;
                    live &= ~(1u << k);
                } else if (prev[k] == (int32_t)key[k]) {
                    flags |= ST_DUPLICATE;
                    live &= ~(1u << k);
                } else {
                    s[k] = (s[k] + 1) & t.cap_mask;
                }
            }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (!((won >> k) & 1u)) continue;
            const int32_t kk = (int32_t)key[k];
            if (t.bits) {
                const uint64_t d = (uint64_t)(key[k] - t.bmin);
                atomicOr(&t.bits[d >> 5], 1u << (d & 31));
            }
            if (t.filt) {
                const uint32_t fb = filter_bit(kk, t.flog2), fb2 = filter_bit2(kk, t.flog2);
                atomicOr(&t.filt[fb >> 5], (1u << (fb & 31)) | (1u << (fb2 & 31)));  // both in one word
            }
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                if (j >= A.npay) continue;
                if (t.pay64[j]) reinterpret_cast<int64_t*>(t.pay[j])[s[k]] = pay[j][k];
                else reinterpret_cast<int32_t*>(t.pay[j])[s[k]] = (int32_t)pay[j][k];
            }
        }
    }
    if (!ok) flags |= ST_CORRUPT;
    if (flags) atomicOr(A.status, flags);
}

// An empty table: its keys, then zeros (bitmap and filter) to the end.
__global__ void hash_clear_kernel(int32_t* p, int64_t nkeys, int64_t zero_from, int64_t nwords) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < nwords; i += (int64_t)gridDim.x * blockDim.x) {
        if (i < nkeys) p[i] = kEmptyKey;
        else if (i >= zero_from) p[i] = 0;
    }
}

// Bandwidth probe (measurement only, not on the query path): every lane
// streams 16-byte loads over [p, p + n16 * 16) in a grid-stride loop, four
// loads in flight, and folds them into one word that is stored only when it
// equals the caller's value `key`, so that no load can be dropped.
__global__ __launch_bounds__(256) void stream_read_kernel(const uint4* __restrict__ p, uint64_t n16,
                                                           uint32_t key, uint32_t* __restrict__ sink) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    cptr<u32x4> v = (cptr<u32x4>)p;
    uint32_t acc = 0;
    for (; i + 3 * stride < n16; i += 4 * stride) {
        const u32x4 x0 = v[i], x1 = v[i + stride], x2 = v[i + 2 * stride], x3 = v[i + 3 * stride];
        acc ^= (x0.x ^ x0.y ^ x0.z ^ x0.w) + (x1.x ^ x1.y ^ x1.z ^ x1.w) + (x2.x ^ x2.y ^ x2.z ^ x2.w) +
               (x3.x ^ x3.y ^ x3.z ^ x3.w);
    }
    for (; i < n16; i += stride) {
        const u32x4 x = v[i];
        acc ^= x.x ^ x.y ^ x.z ^ x.w;
    }
    if (acc == key) sink[0] = acc;
}

// Writes the non-empty groups of a large or hashed group table to the plan's
// pinned host buffer and clears them and the status words for the next
// execution.  Bound by the scan of the slots (32 MB for 2^22 hash slots) and
// the records' way over the host link, so the slots are cut into slabs of
// kEmitSlab over many workgroups; one workgroup alone took 21 ms for 2^22
// slots.  Each workgroup reserves a slab's output with one atomic.  The
// buffer is one array per record field (the group, then each accumulator):
// a wave's stores are then contiguous runs of 8 bytes a lane, where whole
// records would cross the link as scattered 8-byte writes.  The host orders
// the groups.  status: [bits, records so far, finished workgroups].
constexpr int kEmitBlock = 1024, kEmitSlots = 8, kEmitSlab = kEmitBlock * kEmitSlots;

__global__ __launch_bounds__(kEmitBlock) void emit_kernel(const DevQuery* __restrict__ q, unsigned long long* T,
                                                          uint32_t* status) {
    __shared__ uint32_t wcnt[kEmitBlock / kWave];
    __shared__ uint32_t base_s;
    CQ& Q = *ro(q);
    const int nacc = Q.nacc;
    const int64_t G = Q.ngroups;
    unsigned long long* const K = Q.agg_hash ? T + G * nacc : nullptr;
    int64_t* const out = Q.host_out + 2;
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    for (int64_t s0 = (int64_t)blockIdx.x * kEmitSlab; s0 < G; s0 += (int64_t)gridDim.x * kEmitSlab) {
        unsigned long long key[kEmitSlots], cnt[kEmitSlots];
#pragma unroll
        for (int k = 0; k < kEmitSlots; ++k) {
            const int64_t g = s0 + k * kEmitBlock + threadIdx.x;
            key[k] = g < G ? (K ? K[g] : (unsigned long long)g + 1ull) : 0ull;
        }
        uint32_t mine = 0;
#pragma unroll
        for (int k = 0; k < kEmitSlots; ++k) {
            const int64_t g = s0 + k * kEmitBlock + threadIdx.x;
            cnt[k] = key[k] ? T[g * nacc] : 0ull;
            if (K && key[k]) K[g] = 0;
        }
#pragma unroll
        for (int k = 0; k < kEmitSlots; ++k) mine += (uint32_t)__popcll(__ballot(cnt[k] != 0));  // the wave's
        if (lane == 0) wcnt[wave] = mine;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t t = 0;
            for (int w = 0; w < kEmitBlock / kWave; ++w) { const uint32_t x = wcnt[w]; wcnt[w] = t; t += x; }
            base_s = t ? atomicAdd(&status[1], t) : 0u;
        }
        __syncthreads();
        uint32_t o = base_s + wcnt[wave];
#pragma unroll
        for (int k = 0; k < kEmitSlots; ++k) {
            const uint64_t b = __ballot(cnt[k] != 0);
            if (cnt[k]) {
                const int64_t g = s0 + k * kEmitBlock + threadIdx.x;
                const int64_t pos = o + bits_below(b);
                out[pos] = (int64_t)(key[k] - 1ull);
                out[G + pos] = (int64_t)cnt[k];
                T[g * nacc] = 0;
                for (int a = 1; a < nacc; ++a) {
                    out[(1 + a) * G + pos] = (int64_t)T[g * nacc + a];
                    T[g * nacc + a] = 0;
                }
            }
            o += (uint32_t)__popcll(b);
        }
        __syncthreads();  // wcnt and base_s are rewritten by the next slab
    }
    // Thread 0 has the values its reservations returned, so they precede its
    // count here: the last one reads the total.
    if (threadIdx.x == 0 && atomicAdd(&status[2], 1u) == gridDim.x - 1u) {
        Q.host_out[1] = (int64_t)atomicExch(&status[1], 0u);
        Q.host_out[0] = (int64_t)atomicExch(&status[0], 0u);
        atomicExch(&status[2], 0u);
        __threadfence_system();
    }
}

template <typename T>
__global__ void fill_kernel(T* p, T v, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// ---------------------------------------------------------------------------
// Fragmented execution: one kernel per step, intermediates in HBM.  Each
// kernel is the straightforward data-parallel form of its step, with
// workgroup-level aggregation of its atomics.
// ---------------------------------------------------------------------------
// Decode one integer column to int64 (codes for DICT).
__global__ __launch_bounds__(kBlock) void frag_decode_int(const DevQuery* __restrict__ q, int c, int64_t* out) {
    CQ& Q = *ro(q);
    CC& C = Q.cols[c];
    const int lane = lane_id();
    const int gw = uniform_i32((int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6));  // wave-uniform
    const int nw = (gridDim.x * blockDim.x) >> 6;
    bool ok = true;
    for (int m = gw; m < Q.nmb; m += nw) {
        int64_t v[4];
        ok &= decode_dense(C, m, lane, v);
        for (int k = 0; k < 4; ++k) {
            int64_t r = (int64_t)m * kMB + 64 * k + lane;
            if (r < Q.nrows) out[r] = v[k];
        }
    }
    if (!ok) atomicOr(Q.status, ST_CORRUPT);
}

// Decode a string column: offsets [nrows + 1] and a copy of the bytes.
__global__ __launch_bounds__(kBlock) void frag_decode_str(const DevQuery* __restrict__ q, int c, int64_t* off,
                                                           uint8_t* bytes) {
    CQ& Q = *ro(q);
    CC& C = Q.cols[c];
    const int lane = lane_id();
    const int gw = uniform_i32((int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6));  // wave-uniform
    const int nw = (gridDim.x * blockDim.x) >> 6;
    bool ok = true;
    for (int m = gw; m < Q.nmb; m += nw) {
        const int nvalid = (int)min((int64_t)kMB, Q.nrows - (int64_t)m * kMB);
        MbHdr h = mb_hdr(C, m);
        ok &= h.ok;
        uint64_t h0 = ro(C.hoff)[m], h1 = ro(C.hoff)[m + 1];
        if (!(h0 <= h1 && h1 <= C.heap_bytes)) { ok = false; continue; }
        uint64_t carry = h0;
        for (int k = 0; k < 4; ++k) {
            int i = 64 * k + lane;
            uint64_t len = (i < nvalid) ? (uint64_t)h.base + (h.b ? bits_at(h.w, (uint32_t)i * h.b, h.b) : 0) : 0;
            uint64_t s = wave_incl_scan_u64(len);
            if (i < nvalid) off[(int64_t)m * kMB + i] = (int64_t)(carry + s - len);
            carry += readlane_u64(s, 63);
        }
        if (carry != h1) ok = false;
        // copy the bytes: 16-byte pieces where both sides are aligned
        uint64_t b = h0;
        while (b < h1 && (b & 15)) {
            if (b + lane < h1 && ((b + lane) & ~uint64_t(15)) == (b & ~uint64_t(15))) bytes[b + lane] = ro(C.heap)[b + lane];
            b = (b | 15) + 1;
        }
        for (uint64_t v = b + 16 * (uint64_t)lane; v + 16 <= h1; v += 16 * kWave)
            *reinterpret_cast<uint4*>(bytes + v) = ld4((cptr<uint4>)(C.heap + v), 0);
        uint64_t tail = b + ((h1 > b ? h1 - b : 0) & ~uint64_t(15));
        if (tail + lane < h1) bytes[tail + lane] = ro(C.heap)[tail + lane];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) off[Q.nrows] = (int64_t)Q.cols[c].heap_bytes;
    if (!ok) atomicOr(Q.status, ST_CORRUPT);
}

// FSST record decode (Section 4.1): one wave per mini block, lane l on rows
// 4 l .. 4 l + 3.  Pass 1 walks the codes for the decoded record lengths and
// a wave prefix sum gives every row's output offset; pass 2 decodes the
// records in parallel into an LDS staging window, copied out with
// coalesced stores (a mini block larger than the window takes several
// windows).  Each wave takes a contiguous run of mini blocks and keeps the
// symbol table of the current chunk in its LDS.  Both passes take eight
// codes a step, so that their table reads are issued together.  The window
// (7.5 KiB, above the 6.8 KiB that 256 rows of the string workload's
// comments decode to) lets four workgroups share a CU's LDS.
constexpr int kFsstStage = 7680;
// + 16: the spill of the last 8-byte symbol write, and the copy-out's
// read-ahead dword
constexpr size_t kFsstDecodeWaveBytes = 256 * 8 + 256 + kFsstStage + 16;
// an 8-byte store at any byte address (gfx950's LDS takes unaligned access)
typedef uint64_t u64_ua __attribute__((aligned(1)));

__global__ __launch_bounds__(kBlock) void frag_decode_fsst(const DevQuery* __restrict__ q, int c, int64_t* off,
                                                           uint8_t* bytes) {
    extern __shared__ __align__(16) uint8_t smem[];
    CQ& Q = *ro(q);
    CC& C = Q.cols[c];
    const int lane = lane_id();
    const int wave = uniform_i32(threadIdx.x >> 6);
    uint8_t* wa = smem + (size_t)wave * kFsstDecodeWaveBytes;
    uint64_t* sym = reinterpret_cast<uint64_t*>(wa);
    uint8_t* len = wa + 256 * 8;
    uint8_t* stage = wa + 256 * 8 + 256;
    const int nw = gridDim.x * kWaves;
    const int gw = blockIdx.x * kWaves + wave;
    const int per = (Q.nmb + nw - 1) / nw;
    const int m0 = gw * per, m1 = min(Q.nmb, m0 + per);
    const int mbpc = max(C.mbpc, 1);
    int chunk = -1;
    bool ok = true;
    for (int m = m0; m < m1; ++m) {
        const int nvalid = (int)min((int64_t)kMB, Q.nrows - (int64_t)m * kMB);
        if (m / mbpc != chunk) {
            chunk = m / mbpc;
            cptr<uint8_t> tab = ro(C.symtab) + (size_t)chunk * (256 * 8 + 256);
            wave_lds_sync();
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int e = 64 * j + lane;
                const uint32_t le = e < 255 ? min((uint32_t)tab[256 * 8 + e], 8u) : 0u;
                // bytes past a symbol's length are zero in LDS (code 255: none)
                sym[e] = ((cptr<uint64_t>)tab)[e] & (le >= 8u ? ~0ull : (1ull << (8 * le)) - 1ull);
                len[e] = (uint8_t)le;
            }
            wave_lds_sync();
        }
        uint32_t rl[4], lsum, incl;
        uint64_t h0;
        if (!fsst_lengths(C, m, lane, nvalid, rl, lsum, incl, h0)) { ok = false; continue; }
        const uint64_t d0 = ro(C.doff)[m], d1 = ro(C.doff)[m + 1];
        if (!(d0 <= d1 && d1 <= C.str_bytes)) { ok = false; continue; }
        // pass 1: decoded lengths, the lane's four rows' codes as one run,
        // eight codes a step (a literal counts 1 byte; the bytes before each
        // row boundary are summed on the side).  A code of length 0 and an
        // escape as the lane's last code mark the column corrupt.
        CodeReader R;
        R.init(C.heap, h0, incl - lsum);
        bool esc = false;
        const uint32_t c1 = rl[0], c2 = c1 + rl[1], c3 = c2 + rl[2];
        uint32_t n = 0, n1 = 0, n2 = 0, n3 = 0;
        for (uint32_t i = 0; i < lsum;) {
            uint32_t qa, qb;
            R.peek8(qa, qb);
            const uint32_t nq = min(lsum - i, 8u);
            uint32_t l[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) l[j] = len[((j < 4 ? qa : qb) >> (8 * (j & 3))) & 0xFFu];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const uint32_t cd = ((j < 4 ? qa : qb) >> (8 * (j & 3))) & 0xFFu;
                const bool act = (uint32_t)j < nq;
                const bool lit = esc;
                ok = ok && !(act && !lit && cd != 255u && l[j] == 0);
                const uint32_t cb = act ? (lit ? 1u : l[j]) : 0u;
                const uint32_t k = i + j;
                n += cb;
                n1 += k < c1 ? cb : 0u;
                n2 += k < c2 ? cb : 0u;
                n3 += k < c3 ? cb : 0u;
                esc = act ? (!lit && cd == 255u) : esc;
            }
            i += nq;
            R.advance(nq);
        }
        if (esc) { ok = false; esc = false; }
        const uint32_t dl[4] = {n1, n2 - n1, n3 - n2, n - n3};
        const uint32_t dsum = n;
        const uint32_t dincl = wave_incl_scan_u32(dsum);
        const uint32_t dtotal = __builtin_amdgcn_readlane(dincl, 63);
        if ((uint64_t)dtotal != d1 - d0) { ok = false; continue; }
        uint32_t start = dincl - dsum;
        {
            uint32_t o = start;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int r = 4 * lane + j;
                if (r < nvalid) off[(int64_t)m * kMB + r] = (int64_t)(d0 + o);
                o += dl[j];
            }
        }
        // pass 2: decode window by window.  A symbol is stored as one
        // unaligned 8-byte LDS write (its padding bytes are overwritten by
        // the next symbol); a lane's last writes can spill up to 7 zero bytes
        // into the next lane's first bytes, so after the window every lane
        // writes its first 7 bytes again, exactly.
        const uint32_t dend = start + dsum;
        for (uint32_t w0 = 0; w0 < dtotal; w0 += kFsstStage) {
            const uint32_t wn = min((uint32_t)kFsstStage, dtotal - w0);
            const uint32_t wend = w0 + wn;
            const bool here = start < wend && dend > w0;
            if (here) {
                R.init(C.heap, h0, incl - lsum);
                uint32_t d = start;  // decoded position of the next byte
                uint32_t rem = lsum;
                while (rem && d < wend) {
                    uint32_t qa, qb;
                    R.peek8(qa, qb);
                    const uint32_t nq = min(rem, 8u);
                    uint64_t sv[8];
                    uint32_t l[8];
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const uint32_t cd = ((j < 4 ? qa : qb) >> (8 * (j & 3))) & 0xFFu;
                        sv[j] = sym[cd];
                        l[j] = len[cd];
                    }
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        if ((uint32_t)j < nq) {
                            const uint32_t cd = ((j < 4 ? qa : qb) >> (8 * (j & 3))) & 0xFFu;
                            const uint32_t L = esc ? 1u : l[j];
                            const uint64_t v = esc ? (uint64_t)cd : sv[j];
                            esc = !esc && cd == 255u;
                            if (d - w0 < wn) {
                                *reinterpret_cast<u64_ua*>(stage + (d - w0)) = v;
                            } else if (d < w0 && d + L > w0) {  // a symbol across the window's start
                                for (uint32_t b = w0 - d; b < L; ++b) stage[d + b - w0] = (uint8_t)(v >> (8 * b));
                            }
                            d += L;
                        }
                    }
                    rem -= nq;
                    R.advance(nq);
                }
                esc = false;
            }
            wave_lds_sync();
            // the lane's first bytes (at most 7), which the previous lanes'
            // spill may have zeroed, decoded again and stored byte by byte
            if (here && start >= w0) {
                const uint32_t hend = min(min(dend, start + 7u), wend);
                R.init(C.heap, h0, incl - lsum);
                uint32_t d = start, rem = lsum;
                while (rem && d < hend) {
                    const uint32_t cd = R.peek4() & 0xFFu;
                    uint32_t L = len[cd];
                    uint64_t v = sym[cd];
                    if (cd == 255u && rem > 1) {
                        R.advance(1);
                        --rem;
                        v = R.peek4() & 0xFFu;
                        L = 1;
                    }
                    for (uint32_t b = 0; b < L && d + b < hend; ++b) stage[d + b - w0] = (uint8_t)(v >> (8 * b));
                    d += L;
                    --rem;
                    R.advance(1);
                }
            }
            wave_lds_sync();
            // copy-out: bytes up to a 4-byte boundary of the destination,
            // then whole dwords (two aligned LDS dwords realigned), then the
            // tail
            uint8_t* dst = bytes + d0 + w0;
            const uint32_t head = min(wn, (uint32_t)((4u - ((uintptr_t)dst & 3u)) & 3u));
            if ((uint32_t)lane < head) dst[lane] = stage[lane];
            const uint32_t nd = (wn - head) >> 2;
            uint32_t* dw = reinterpret_cast<uint32_t*>(dst + head);
            const uint32_t* sw = reinterpret_cast<const uint32_t*>(stage);
            for (uint32_t i = lane; i < nd; i += kWave) {
                const uint32_t so = head + 4u * i;
                dw[i] = __builtin_amdgcn_alignbyte(sw[(so >> 2) + 1], sw[so >> 2], so & 3u);
            }
            for (uint32_t i = head + 4u * nd + lane; i < wn; i += kWave) dst[i] = stage[i];
            wave_lds_sync();
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) off[Q.nrows] = (int64_t)C.str_bytes;
    if (!ok) atomicOr(Q.status, ST_CORRUPT);
}

__global__ void frag_filter_int(const DevQuery* __restrict__ q, int pi, const int64_t* vals, uint8_t* flags,
                                int first) {
    CQ& Q = *ro(q);
    CP& P = Q.preds[pi];
    for (int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; r < Q.nrows;
         r += (int64_t)gridDim.x * blockDim.x) {
        int64_t v4[4] = {vals[r], 0, 0, 0};
        bool t = eval_int_pred(P, Q.in_vals, v4) & 1u;
        flags[r] = (uint8_t)((first ? 1 : flags[r]) & t);
    }
}

// The string atom over the materialised column: the same heap scan as the
// fused kernel's string test (aligned-word table or byte windows), one wave
// per 256 rows, reading the decoded offsets and the copied bytes (mcol: the
// column's descriptor with its heap pointing at that copy); one flag per row.
template <int kMode>
__global__ __launch_bounds__(kBlock) void frag_filter_str(const DevQuery* __restrict__ q, const DevCol* __restrict__ mcol,
                                                          int pi, const int64_t* __restrict__ off, uint8_t* flags,
                                                          int first) {
    extern __shared__ __align__(16) uint8_t smem[];
    __shared__ __align__(16) uint32_t tab[32];
    CQ& Q = *ro(q);
    CP& P = Q.preds[pi];
    CC& C = *ro(mcol);
    if (threadIdx.x < 32) tab[threadIdx.x] = P.tab[threadIdx.x];
    __syncthreads();
    const int lane = lane_id();
    const int wave = uniform_i32(threadIdx.x >> 6);
    uint8_t* wa = smem + (size_t)wave * (260 * 4 + 2 * 256 * 4 + kRecCap * 16);
    uint32_t* offs = reinterpret_cast<uint32_t*>(wa);
    const StrLds L{tab, offs, offs + 260, offs + 516, reinterpret_cast<uint4*>(offs + 772)};
    bool ok = true;
    for (int m = blockIdx.x * kWaves + wave; m < Q.nmb; m += gridDim.x * kWaves) {
        const int64_t row0 = (int64_t)m * kMB;
        const int nvalid = (int)min((int64_t)kMB, Q.nrows - row0);
        StrTile S;
        S.h0 = (uint64_t)ro(off)[row0];
        S.h1 = (uint64_t)ro(off)[row0 + nvalid];
        S.ok = S.h0 <= S.h1 && S.h1 <= C.heap_bytes && (S.h1 - S.h0) < (uint64_t(1) << 30);
        const uint64_t a0 = S.h0 & ~uint64_t(15);
        S.g = (cptr<uint4>)(C.heap + a0);
        S.gp = C.heap + a0;
        const uint32_t nvec = S.ok ? (uint32_t)((S.h1 - a0 + 15u) >> 4) : 0u;
        if (S.ok) load_segment(S.cur, S, 0, nvec, lane);
        // row offsets within the mini block, from the materialised offsets
        uint4 ov;
        const int64_t rb = row0 + 4 * lane;
        const int64_t rend = row0 + nvalid;
        ov.x = (uint32_t)((uint64_t)ro(off)[min(rb, rend)] - S.h0);
        ov.y = (uint32_t)((uint64_t)ro(off)[min(rb + 1, rend)] - S.h0);
        ov.z = (uint32_t)((uint64_t)ro(off)[min(rb + 2, rend)] - S.h0);
        ov.w = (uint32_t)((uint64_t)ro(off)[min(rb + 3, rend)] - S.h0);
        reinterpret_cast<uint4*>(offs)[lane] = ov;
        if (lane == 0) offs[256] = (uint32_t)(S.h1 - S.h0);
        const uint32_t mask = str_finish<kMode, true>(C, P, lane, nvalid, S, L, ok);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int i = 64 * k + lane;
            if (i >= nvalid) continue;
            const int64_t r = row0 + i;
            const bool prev = first ? true : flags[r] != 0;
            flags[r] = (uint8_t)(prev && ((mask >> k) & 1u));
        }
        wave_lds_sync();
    }
    if (!ok) atomicOr(Q.status, ST_CORRUPT);
}

// flags -> row list (order not preserved; aggregation is order-free).  One
// global atomic per workgroup step of 1024 rows.
// Output space is reserved once per tile of kFragTile rows (16 per thread):
// one device-scope atomic on the list's counter per tile.  With one per
// 64- or 1,024-row step the atomics on that single counter serialised the
// kernels.
constexpr int kFragRows = 16;
constexpr int kFragTile = kBlock * kFragRows;

// Per wave: its survivors' count from the per-lane keep bits (bit k: row k
// of the lane), then the tile's reservation; returns the wave's first slot.
__device__ __forceinline__ unsigned long long frag_reserve(uint32_t keep, unsigned long long* count, int lane,
                                                           int wave) {
    __shared__ uint32_t wcnt[kWaves];
    __shared__ unsigned long long base_s;
    uint32_t c = 0;
#pragma unroll
    for (int k = 0; k < kFragRows; ++k) c += (uint32_t)__popcll(__ballot((keep >> k) & 1u));
    if (lane == 0) wcnt[wave] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t t = 0;
        for (int w = 0; w < kWaves; ++w) { const uint32_t x = wcnt[w]; wcnt[w] = t; t += x; }
        base_s = t ? atomicAdd(count, (unsigned long long)t) : 0;
    }
    __syncthreads();
    const unsigned long long o = base_s + wcnt[wave];
    __syncthreads();  // wcnt and base_s are rewritten by the next tile
    (void)lane;
    return o;
}

__global__ __launch_bounds__(kBlock) void frag_compact(const DevQuery* __restrict__ q, const uint8_t* flags,
                                                       FragRow* rows, unsigned long long* count) {
    CQ& Q = *ro(q);
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    for (int64_t t0 = (int64_t)blockIdx.x * kFragTile; t0 < Q.nrows; t0 += (int64_t)gridDim.x * kFragTile) {
        uint32_t keep = 0;
#pragma unroll
        for (int k = 0; k < kFragRows; ++k) {
            const int64_t r = t0 + (int64_t)k * kBlock + threadIdx.x;
            keep |= (uint32_t)(r < Q.nrows && flags[r]) << k;
        }
        unsigned long long o = frag_reserve(keep, count, lane, wave);
#pragma unroll
        for (int k = 0; k < kFragRows; ++k) {
            const bool f = (keep >> k) & 1u;
            const uint64_t b = __ballot(f);
            if (f) rows[o + bits_below(b)] = (FragRow)(t0 + (int64_t)k * kBlock + threadIdx.x);
            o += (uint32_t)__popcll(b);
        }
    }
}

// all rows -> row list (plans without a fact predicate)
__global__ void frag_iota(const DevQuery* __restrict__ q, FragRow* rows, unsigned long long* count) {
    CQ& Q = *ro(q);
    for (int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; r < Q.nrows;
         r += (int64_t)gridDim.x * blockDim.x)
        rows[r] = (FragRow)r;
    if (blockIdx.x == 0 && threadIdx.x == 0) *count = (unsigned long long)Q.nrows;
}

// Probe j: keep listed rows whose key is found; carry the earlier payload
// arrays along and append this probe's payloads.
__global__ __launch_bounds__(kBlock) void frag_probe(const DevQuery* __restrict__ q, int j, const int64_t* fkvals,
                                                     const FragRow* rin, const unsigned long long* nin,
                                                     FragRow* rout, unsigned long long* nout,
                                                     const FragBuffers fb, int src, int npay_before) {
    CQ& Q = *ro(q);
    CPR& P = Q.probes[j];
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const int64_t n = (int64_t)*nin;
    CC& fc = Q.cols[P.fk_col];
    for (int64_t t0 = (int64_t)blockIdx.x * kFragTile; t0 < n; t0 += (int64_t)gridDim.x * kFragTile) {
        uint32_t keep = 0;
        int slot[kFragRows];
#pragma unroll
        for (int k = 0; k < kFragRows; ++k) {
            const int64_t e = t0 + (int64_t)k * kBlock + threadIdx.x;
            slot[k] = -1;
            if (e < n) {
                int64_t fk = fkvals[(int64_t)rin[e]];
                bool okd = true;
                if (fc.enc == ENC_DICT) fk = dict_value(fc, fk, okd);
                // the same bitmap pre-test as the fused kernel's stage B
                if (!P.h.bits || bitmap_has_global(P.h, fk)) slot[k] = hash_find<false>(P.h, nullptr, fk);
            }
            keep |= (uint32_t)(slot[k] >= 0) << k;
        }
        unsigned long long o = frag_reserve(keep, nout, lane, wave);
#pragma unroll
        for (int k = 0; k < kFragRows; ++k) {
            const bool f = (keep >> k) & 1u;
            const uint64_t b = __ballot(f);
            if (f) {
                const int64_t e = t0 + (int64_t)k * kBlock + threadIdx.x;
                const unsigned long long w = o + bits_below(b);
                rout[w] = rin[e];
                for (int t = 0; t < npay_before; ++t) fb.pay[1 - src][t][w] = fb.pay[src][t][e];
                for (int p = 0; p < P.h.npay; ++p)
                    fb.pay[1 - src][npay_before + p][w] = hash_payload<false>(P.h, nullptr, p, slot[k]);
            }
            o += (uint32_t)__popcll(b);
        }
    }
}

// Aggregate the final row list: fact values gathered from the decoded
// columns, payloads from the aligned arrays; small group tables are
// accumulated per workgroup in LDS first.
__global__ __launch_bounds__(kBlock) void frag_aggregate(const DevQuery* __restrict__ q, const FragRow* rows,
                                                         const unsigned long long* nrows_list, const FragBuffers fb,
                                                         int src) {
    __shared__ unsigned long long tab[4096];
    CQ& Q = *ro(q);
    const int64_t n = (int64_t)*nrows_list;
    const bool local = !Q.agg_hash && Q.ngroups * Q.nacc <= 4096;
    if (local)
        for (int e = threadIdx.x; e < Q.ngroups * Q.nacc; e += blockDim.x) tab[e] = 0;
    __syncthreads();
    bool okall = true;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t r = (int64_t)rows[e];
        RegSlots sv;
        for (int s = 0; s < kMaxSlots; ++s) sv.v[s] = 0;
        int pidx = 0;
        for (int j = 0; j < Q.nprobes; ++j) {
            for (int k = 0; k < Q.probes[j].h.npay; ++k) {
                int sl = Q.probes[j].pay_slot[k];
                if (sl >= 0) sv.set(sl, fb.pay[src][pidx][e]);
                ++pidx;
            }
        }
        for (int l = 0; l < Q.nloads; ++l) {
            CL& Ld = Q.loads[l];
            int64_t x = fb.dec[Ld.col][r];
            if (Ld.dict_val) x = dict_value(Q.cols[Ld.col], x, okall);
            sv.set(l, x);
        }
        int64_t g;
        if (!group_index(Q, sv, g)) { okall = false; continue; }
        unsigned long long* T;
        if (local) {
            T = &tab[g * Q.nacc];
        } else {
            unsigned long long* A = reinterpret_cast<unsigned long long*>(Q.agg);
            const int64_t row = agg_row(Q, A, g);
            if (row < 0) { okall = false; continue; }
            T = A + row * Q.nacc;
        }
        atomicAdd(&T[0], 1ull);
        for (int a = 1; a < Q.nacc; ++a) atomicAdd(&T[a], (unsigned long long)acc_value(Q.accs[a], sv));
    }
    __syncthreads();
    if (local)
        for (int e = threadIdx.x; e < Q.ngroups * Q.nacc; e += blockDim.x)
            if (tab[e]) atomicAdd(reinterpret_cast<unsigned long long*>(Q.agg) + e, tab[e]);
    if (!okall) atomicOr(Q.status, ST_CORRUPT);
}

__global__ __launch_bounds__(kBlock) void frag_emit(const DevQuery* __restrict__ q) {
    CQ& Q = *ro(q);
    emit_table(Q, reinterpret_cast<unsigned long long*>(Q.agg), Q.status, threadIdx.x, blockDim.x);
    __threadfence_system();
}

__global__ void frag_reset_counts(unsigned long long* c, int n) {
    if ((int)threadIdx.x < n) c[threadIdx.x] = 0;
}
}  // namespace

hipError_t launch_hash_count(const HashBuildArgs* d_args, int grid, hipStream_t s) {
    hipLaunchKernelGGL(hash_count_kernel, dim3(grid), dim3(kBlock), 0, s, d_args);
    return hipGetLastError();
}

hipError_t launch_hash_insert(const HashBuildArgs* d_args, const HashTableArgs& t, int grid, hipStream_t s) {
    hipLaunchKernelGGL(hash_insert_kernel, dim3(grid), dim3(kBlock), 0, s, d_args, t);
    return hipGetLastError();
}

hipError_t launch_hash_clear(int32_t* p, int64_t nkeys, int64_t zero_from, int64_t nwords, hipStream_t s) {
    const int64_t blocks = (nwords + 255) / 256;
    hipLaunchKernelGGL(hash_clear_kernel, dim3((int)(blocks < 4096 ? blocks : 4096)), dim3(256), 0, s, p, nkeys,
                       zero_from, nwords);
    return hipGetLastError();
}

hipError_t launch_stream_read(const void* p, uint64_t bytes, uint32_t key, uint32_t* sink, int grid,
                              hipStream_t s) {
    hipLaunchKernelGGL(stream_read_kernel, dim3(grid), dim3(256), 0, s, reinterpret_cast<const uint4*>(p),
                       (uint64_t)(bytes / 16), key, sink);
    return hipGetLastError();
}

hipError_t launch_emit(const DevQuery* d_q, const DevQuery& h_q, int64_t* agg, uint32_t* status, hipStream_t s) {
    const int64_t slabs = (h_q.ngroups + kEmitSlab - 1) / kEmitSlab;
    hipLaunchKernelGGL(emit_kernel, dim3((int)(slabs < 1024 ? slabs : 1024)), dim3(kEmitBlock), 0, s, d_q,
                       reinterpret_cast<unsigned long long*>(agg), status);
    return hipGetLastError();
}

hipError_t launch_fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t s) {
    int64_t blocks = (n + 255) / 256;
    int grid = (int)(blocks < 4096 ? blocks : 4096);
    if (grid < 1) grid = 1;
    hipLaunchKernelGGL(fill_kernel<int32_t>, dim3(grid), dim3(256), 0, s, p, v, n);
    return hipGetLastError();
}

hipError_t launch_fill_i64(int64_t* p, int64_t v, int64_t n, hipStream_t s) {
    int64_t blocks = (n + 255) / 256;
    int grid = (int)(blocks < 4096 ? blocks : 4096);
    if (grid < 1) grid = 1;
    hipLaunchKernelGGL(fill_kernel<int64_t>, dim3(grid), dim3(256), 0, s, p, v, n);
    return hipGetLastError();
}

int run_fragmented(const DevQuery* d_q, const DevQuery& Q, const FragBuffers& fb, hipStream_t s) {
    int launches = 0;
    const int grid = 2048;
    auto chk = [&]() { ++launches; return hipGetLastError() == hipSuccess; };
    hipLaunchKernelGGL(frag_reset_counts, dim3(1), dim3(64), 0, s, fb.counts, kMaxProbes + 2);
    if (!chk()) return -1;
    // 1) decompression kernels: every referenced column, fully materialised
    bool needed[kMaxCols] = {};
    for (int p = 0; p < Q.npreds; ++p) needed[Q.preds[p].col] = true;
    for (int j = 0; j < Q.nprobes; ++j) needed[Q.probes[j].fk_col] = true;
    for (int l = 0; l < Q.nloads; ++l) needed[Q.loads[l].col] = true;
    for (int c = 0; c < Q.ncols; ++c) {
        if (!needed[c]) continue;
        if (Q.cols[c].enc == ENC_VARLEN) {
            hipLaunchKernelGGL(frag_decode_str, dim3(grid), dim3(kBlock), 0, s, d_q, c, fb.str_off[c],
                               fb.str_bytes[c]);
        } else if (Q.cols[c].enc == ENC_FSST) {
            hipLaunchKernelGGL(frag_decode_fsst, dim3(grid), dim3(kBlock), kWaves * kFsstDecodeWaveBytes, s, d_q, c,
                               fb.str_off[c], fb.str_bytes[c]);
        } else {
            hipLaunchKernelGGL(frag_decode_int, dim3(grid), dim3(kBlock), 0, s, d_q, c, fb.dec[c]);
        }
        if (!chk()) return -1;
    }
    // 2) one filter kernel per predicate, then compaction to a row list
    for (int p = 0; p < Q.npreds; ++p) {
        const int c = Q.preds[p].col;
        if (Q.preds[p].kind == PK_STR) {
            const DevPred& P = Q.preds[p];
            const int mode = P.tab_rot ? kStrTable : (P.n1 < 4 || P.n2 < 4) ? kStrMasked : kStrShifted;
            const size_t lds = (size_t)kWaves * (260 * 4 + 2 * 256 * 4 + kRecCap * 16);
            const int64_t wgs = ((int64_t)Q.nmb + kWaves - 1) / kWaves;
            const int sgrid = (int)(wgs < 2048 ? (wgs > 0 ? wgs : 1) : 2048);
            if (mode == kStrTable)
                hipLaunchKernelGGL(frag_filter_str<kStrTable>, dim3(sgrid), dim3(kBlock), lds, s, d_q, fb.str_col[c], p,
                                   fb.str_off[c], fb.flags, p == 0 ? 1 : 0);
            else if (mode == kStrShifted)
                hipLaunchKernelGGL(frag_filter_str<kStrShifted>, dim3(sgrid), dim3(kBlock), lds, s, d_q, fb.str_col[c], p,
                                   fb.str_off[c], fb.flags, p == 0 ? 1 : 0);
            else
                hipLaunchKernelGGL(frag_filter_str<kStrMasked>, dim3(sgrid), dim3(kBlock), lds, s, d_q, fb.str_col[c], p,
                                   fb.str_off[c], fb.flags, p == 0 ? 1 : 0);
        } else
            hipLaunchKernelGGL(frag_filter_int, dim3(grid), dim3(256), 0, s, d_q, p, fb.dec[c], fb.flags,
                               p == 0 ? 1 : 0);
        if (!chk()) return -1;
    }
    if (Q.npreds > 0)
        hipLaunchKernelGGL(frag_compact, dim3(grid), dim3(kBlock), 0, s, d_q, fb.flags, fb.rows[0], &fb.counts[0]);
    else
        hipLaunchKernelGGL(frag_iota, dim3(grid), dim3(256), 0, s, d_q, fb.rows[0], &fb.counts[0]);
    if (!chk()) return -1;
    // 3) one probe kernel per dimension
    int src = 0, npay = 0;
    for (int j = 0; j < Q.nprobes; ++j) {
        hipLaunchKernelGGL(frag_probe, dim3(grid), dim3(kBlock), 0, s, d_q, j, fb.dec[Q.probes[j].fk_col],
                           fb.rows[src], &fb.counts[j], fb.rows[1 - src], &fb.counts[j + 1], fb, src, npay);
        if (!chk()) return -1;
        npay += Q.probes[j].h.npay;
        src = 1 - src;
    }
    // 4) aggregation and 5) result emission
    hipLaunchKernelGGL(frag_aggregate, dim3(grid), dim3(kBlock), 0, s, d_q, fb.rows[src], &fb.counts[Q.nprobes],
                       fb, src);
    if (!chk()) return -1;
    if (Q.emit_copy) {
        hipLaunchKernelGGL(frag_emit, dim3(1), dim3(kBlock), 0, s, d_q);
        if (!chk()) return -1;
    } else {
        if (launch_emit(d_q, Q, Q.agg, Q.status, s) != hipSuccess) return -1;
        ++launches;
    }
    return launches;
}

}  // namespace dpf
