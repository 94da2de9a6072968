// dpf_internal.h -- descriptors shared by the host runtime and the gfx950
// kernels.  A plan is flattened into one DevQuery in device memory; the
// persistent kernel reads it with scalar (wave-uniform) loads.
#pragma once
#include <stdint.h>

#include <hip/hip_runtime.h>

namespace dpf {

constexpr int kMB = 256;          // values per mini block
constexpr int kWave = 64;         // CDNA wavefront
constexpr int kWaves = 4;         // waves per workgroup
constexpr int kBlock = kWave * kWaves;
constexpr int kMaxCols = 16;      // fact columns per plan
constexpr int kMaxPreds = 12;     // predicate atoms per plan
constexpr int kMaxProbes = 4;     // probes per plan
constexpr int kMaxSlots = 8;      // values carried per surviving row
constexpr int kMaxKeys = 4;       // group-by keys
constexpr int kMaxAccs = 12;      // accumulators (count + sums)
constexpr int kMaxTerms = 3;      // factors per aggregate product
constexpr int kMaxIn = 64;        // IN-list values per plan
constexpr int kMaxWord = 32;      // bytes per string-predicate word
constexpr int kMaxBatch = 64;     // plans per fused launch
constexpr int kMaxHashCols = 8;   // dimension columns per hash build
constexpr int kMaxHashPreds = 8;  // dimension predicates per hash build
constexpr int64_t kMaxGroups = int64_t(1) << 22;  // direct-indexed group table limit
constexpr int64_t kMaxHashSlots = int64_t(1) << 22;  // hash group table limit (slots)
// A direct group table of at most this many entries (groups x accumulators)
// is copied to the host whole by the fused kernel's last workgroup; a larger
// or hashed one is compacted by emit_kernel, a second launch (about 5 us,
// the time that workgroup takes to copy this many entries).
constexpr int64_t kEmitEntries = 8192;
constexpr int64_t kMaxGroupDomain = int64_t(1) << 62;  // group index + 1 fits int64
constexpr int32_t kEmptyKey = INT32_MIN;
constexpr int kXcds = 8;             // XCDs per device; workgroup i is dispatched to XCD i % 8
constexpr int kCounterStride = 32;   // 32-bit words between work-queue counters (128-byte lines)
constexpr int kCounterWords = (2 * kXcds + 1) * kCounterStride;

enum : int32_t { ENC_FOR = 1, ENC_DELTA = 2, ENC_DICT = 3, ENC_VARLEN = 4, ENC_FSST = 6 };

// Device view of one encoded column (all arrays indexed by global mini block).
struct DevCol {
    const int64_t* base;    // [nmb] FOR base | DELTA anchor | DICT code base | VARLEN min length
    const uint32_t* woff;   // [nmb + 1] first word of each mini block's packed data
    const uint32_t* words;  // packed values, LSB first, value i at bit i * width
    const int64_t* dmin;    // DELTA: [nmb] minimum first difference
    const uint64_t* hoff;   // VARLEN, FSST: [nmb + 1] byte offset of the mini block's strings (codes)
    const uint8_t* heap;    // VARLEN: string bytes; FSST: codes (padded)
    const int64_t* dict;    // DICT: [ndict] sorted distinct values
    const uint64_t* doff;   // FSST: [nmb + 1] decoded byte offset of each mini block
    const uint8_t* symtab;  // FSST: per chunk, sym[256] (uint64) then len[256] (uint8)
    int64_t nrows;
    uint64_t heap_bytes;
    uint64_t str_bytes;     // VARLEN, FSST: decoded string bytes
    uint32_t nwords;
    int32_t nmb;
    int32_t enc;
    int32_t ndict;
    int32_t mbpc;           // mini blocks per chunk (FSST: mini block m uses table m / mbpc)
    int32_t pad;
};

enum : int32_t { PK_RANGE = 1, PK_NE = 2, PK_INMASK = 3, PK_INLIST = 4, PK_STR = 5, PK_FALSE = 6 };

// One conjunctive atom, already rewritten into the column's code space
// (dictionary columns compare codes).
struct DevPred {
    int32_t col;
    int32_t kind;
    int64_t lo, hi;     // RANGE: lo <= x <= hi; NE: x != lo
    uint64_t mask;      // INMASK: bit c set -> code c qualifies (codes < 64)
    int32_t in_off;     // INLIST: values in_vals[in_off .. in_off + n_in)
    int32_t n_in;
    int32_t n1, n2;     // STR: word lengths
    uint8_t s1[kMaxWord];
    uint8_t s2[kMaxWord];
    // STR with both words of at least 7 bytes: lookup table of the aligned-
    // word test.  The eight 4-byte shifts (bytes [j, j + 4), j < 4) of s1
    // and s2 sit at slot str_slot(x, tab_rot); a free slot i holds a word
    // whose slot is not i, so a word x is a shift iff tab[str_slot(x)] == x.
    // tab_rot = 0: no rotation separates the shifts (no table).
    uint32_t tab_rot;
    uint32_t tab[32];
};

// Slot of a 4-byte word in DevPred::tab: bits 2..6 of x ^ rotr(x, r).
__host__ __device__ inline uint32_t str_slot(uint32_t x, uint32_t r) {
    return ((x ^ ((x >> r) | (x << ((32u - r) & 31u)))) & 0x7Cu) >> 2;
}

// Workgroup LDS of the fused kernel: the string-scan table (DevPred::tab of
// the plan's last atom, static LDS), then, dynamic, control words, the
// shared area and the per-wave areas.
constexpr size_t kLdsCtrlBytes = 64;
constexpr size_t kLdsStrTabBytes = 128;
constexpr size_t kLdsHeadBytes = kLdsCtrlBytes + kLdsStrTabBytes;  // counted against the CU's LDS

// Open-addressing table: int32 keys (kEmptyKey = free), payload arrays
// follow the key array in the same allocation.  When the qualifying keys
// span at most kMaxBitmapBits values, a membership bitmap over [bmin, bmin +
// bspan) follows as well: a probe that needs no payload tests one bit.
constexpr uint64_t kMaxBitmapBits = uint64_t(1) << 25;  // 4 MB
struct DevHash {
    const int32_t* keys;
    const void* pay[2];
    const uint32_t* bits;  // nullptr: no bitmap
    int64_t bmin;
    uint64_t bspan;
    uint32_t cap_mask;
    int32_t log2cap;
    int32_t npay;
    int32_t pay64[2];   // payload k stored as int64 (else int32)
    int32_t lds_off;    // >= 0: byte offset of the workgroup's LDS copy
    uint32_t bytes;     // keys + payloads
    // Two-hash bit filter over the keys (small tables only): a probe of a
    // table left in HBM first tests the workgroup's LDS copy of the filter.
    const uint32_t* filt;  // nullptr: none
    int32_t flog2;         // filter bits = 2^flog2
    int32_t filt_lds_off;  // >= 0: byte offset of the LDS copy
    int32_t bits_lds_off;  // >= 0: byte offset of an LDS copy of the bitmap
};
constexpr int kMaxFilterLog2 = 18;  // 32 KB
// The filter's two bit positions, both in one 32-bit word (a blocked
// filter: one LDS read a probe): top bits of 24-bit products, a full-rate
// multiply on the GPU where a 32-bit one issues at quarter rate.  Keys that
// differ only above bit 23 share their bits: more false positives, never a
// missed key.
__host__ __device__ inline uint32_t filter_bit(int32_t key, int flog2) {
    return (((uint32_t)key & 0xFFFFFFu) * 0x2545F5u) >> (32 - flog2);
}
__host__ __device__ inline uint32_t filter_bit2(int32_t key, int flog2) {
    return (filter_bit(key, flog2) & ~31u) | (((((uint32_t)key & 0xFFFFFFu) * 0x9E3779u) + 0x7F4A7C15u) >> 27);
}

struct DevProbe {
    int32_t fk_col;
    int32_t pay_slot[2];  // value slot receiving payload k (-1: unused)
    DevHash h;
};

struct DevLoad { int32_t col, slot, dict_val, pad; };  // fact column -> value slot (DICT: code or value)
struct DevKey { int32_t slot; int32_t pad; int64_t min, card, stride; };
struct DevTerm { int32_t slot; int32_t pad; int64_t mul, add; };  // slot < 0: constant add
struct DevAcc { int32_t nterms; int32_t pad; DevTerm t[kMaxTerms]; };

enum : uint32_t { ST_CORRUPT = 1u, ST_CAPACITY = 2u, ST_UNSUPPORTED = 4u, ST_DUPLICATE = 8u };

// The plan as the lean kernel reads it (fused_lean.hip): values carried as
// 32-bit offsets u = value - ref.
constexpr int kLeanTiles = 16;    // mini blocks whose headers a wave prepares at a time
constexpr int kLeanEnts = kMaxPreds + kMaxSlots;
constexpr int kLeanWidth = 32;    // widest packed value: what a shift of up to 31 leaves of a dword pair
// Copies of an LDS group table: at most 8, in 8 KB.  (6 groups: the 24M-row
// summary took 204 us with 4 copies, 166 with 8, 164 with 16; the 60M-row filter
// 216, 215 and 224, 266 with 32.)
constexpr int kMaxLeanLog2r = 3;
constexpr int kLeanAggBytes = 8 * 1024;

struct LeanEnt {            // one column as an atom or a value slot reads it
    const uint32_t* words;
    const uint32_t* woff;
    const int64_t* base;
    const int64_t* dmin;
    int64_t lo, hi;         // atom: its range (lo: the excluded value); else lo: u = decoded value - lo
                            // (with a dictionary: u is the code, lo 0)
    uint32_t nwords;
    int32_t enc;
    int32_t kind;           // atom: PK_*
    int32_t maxw;           // widest mini block of the column, at most kLeanWidth
    // Staging area of the column's packed words, for one mini block: its place
    // in the wave's, whether this entry copies them (0: an entry before it with
    // the same column does; 2: for a later one too), its bytes.
    uint32_t stage_off, stage_copy, stage_sz;
    uint32_t pad;
};
static_assert(sizeof(LeanEnt) == 80, "copied to LDS in 16-byte units");
struct LeanMore {           // what only the rarer paths need of an entry
    const uint32_t* words;
    const uint32_t* woff;
    const int64_t* dmin;
    int64_t ref;
    const int64_t* dict;    // value slot of a DICT column's values: u = dict[code] - dref
    int64_t dref;
    int32_t enc;
    int32_t ndict;
    int32_t col;            // index into DevQuery::cols
};
struct LeanTerm {           // factor mul * u + c (slot < 0: c)
    int32_t slot;
    int32_t mk;             // mul when it is 1 or -1, else 0
    int64_t mul, c;
};
struct LeanAcc {
    int32_t nterms;
    // 0: u + c; 1: every factor in [0, 2^24); 2: general; 3: as 1, and the
    // factors but the last are those of the accumulator before it
    int32_t cls;
    LeanTerm t[kMaxTerms];
};
struct LeanPlan {
    int32_t ok;             // the plan qualifies
    int32_t nents;          // entries: atoms, then value slots
    int32_t load0;          // first value slot's entry
    int32_t log2r;          // copies of the LDS group table: up to 2^log2r
    int32_t stage_bytes;    // a wave's staging area for the packed words of one mini block
    int32_t dicts;          // value slots that hold a DICT column's values: bits
    int32_t stage_first;    // a wave's first mini blocks have their value columns staged with the atoms'
    // Direct group tables: the key slots (bits), each with its largest value
    // and its stride.
    int32_t keys;
    uint32_t key_last[kMaxSlots];
    uint32_t key_stride[kMaxSlots];
    alignas(16) LeanEnt ents[kLeanEnts];
    LeanMore more[kLeanEnts];
    LeanAcc accs[kMaxAccs];
    // In the LDS group table, a sum of a slot's plain values u + c is kept as
    // the sum of u (slot s in accumulator plain_acc[s], where plain has bit s)
    // and c times the group's rows is added when the table leaves LDS (fold).
    // The other accumulators are prod_acc[0 .. nprod).
    int32_t plain;
    int32_t nprod;
    int32_t plain_acc[kMaxSlots];
    int32_t prod_acc[kMaxAccs];
    int64_t fold[kMaxAccs];
};

// Queued rows of a wave: fewer than 256 and those of a mini block of fewer than
// kDenseMin (fused_lean.hip).
constexpr int kLeanQueue = 384;
// A wave's LDS: header records, queue, staging area.
__host__ __device__ constexpr size_t lean_wave_bytes(int ents, int stage) {
    return (size_t)ents * kLeanTiles * 16 + kLeanQueue * 2 + (size_t)stage;
}
struct DevQuery {
    int64_t nrows;
    int32_t nmb;
    int32_t ncols;
    DevCol cols[kMaxCols];
    int32_t npreds;  // integer atoms first, then string atoms
    int32_t nint_preds;
    DevPred preds[kMaxPreds];
    int64_t in_vals[kMaxIn];
    int32_t nprobes;
    int32_t nloads;
    DevProbe probes[kMaxProbes];
    DevLoad loads[kMaxSlots];
    int32_t nkeys;
    int32_t nacc;    // accumulator 0 is the row count
    DevKey keys[kMaxKeys];
    DevAcc accs[kMaxAccs];
    // Group table: ngroups rows of nacc accumulators, zero between
    // executions.  Direct (agg_hash 0): row g is group index g.  Hash
    // (agg_hash 1, a group-key domain above kMaxGroups): ngroups is a power
    // of two at least twice the groups the table can receive, and ngroups
    // keys follow the accumulators (group index + 1; 0: empty slot), placed
    // by linear probing.
    int64_t ngroups;
    int64_t* agg;
    int32_t agg_lds;     // accumulate in the workgroup's LDS table first
    int32_t agg_lds_off; // byte offset of that table
    int32_t lds_shared;  // LDS bytes of this plan's shared area (hashes + table)
    int32_t has_str;
    int32_t agg_hash;
    int32_t emit_copy;   // the last workgroup copies the whole table to the host (kEmitEntries)
    // The string atom on an FSST column (index into preds, -1: none): its
    // byte automaton (fs_states rows of 256 next states, device memory) and
    // the byte offset of its code table ((2 fs_states + 1) rows of 256) in
    // the shared area.
    int32_t fs_pred;
    int32_t fs_lds_off;
    int32_t fs_states;
    int32_t fs_pad;
    const uint8_t* fs_dfa;
    uint32_t* status;    // device: status bits (ST_*), emit_kernel's record and workgroup counts
    // Device address of the pinned output: [status, 1, group table] (emit_copy),
    // else [status, records, groups[ngroups], accumulator 0[ngroups], ...].
    int64_t* host_out;
    // Chunk pruning: null, or the ascending indices of the blocks of
    // prune_mb mini blocks that the zone maps do not exclude; the fused
    // kernel's work items then cover those blocks only.
    const int32_t* live;
    int32_t nlive;
    int32_t prune_mb;
    LeanPlan lean;
};

// Bytes of a plan's group table: the accumulators, and the keys of a hash
// table.
inline size_t agg_table_bytes(const DevQuery& q) {
    return (size_t)q.ngroups * (size_t)(q.nacc + (q.agg_hash ? 1 : 0)) * 8;
}

struct BatchArgs {
    const DevQuery* q[kMaxBatch];
    // Per plan: its group table (agg_table_bytes, zero between
    // executions) and its status word, in the plan's workspace or in the
    // library's static scratch area.
    int64_t* agg[kMaxBatch];
    uint32_t* status[kMaxBatch];
    int32_t item_start[kMaxBatch + 1];
    int32_t nq;
    int32_t mb_per_item;
    uint32_t* counters;   // kCounterWords: per XCD x, the claim head of item range x (line x) and
                          // its finished workgroups (line 8 + x); finished XCDs (line 16)
    int32_t lds_shared;   // max lds_shared over the batch
    int32_t str_stage;    // per-wave string staging present (2: some plan has an FSST atom)
    int32_t pend_stage;   // per-wave survivor queue present (some plan has a fact predicate or a probe)
    int32_t agg_hash;     // some plan aggregates into a hash group table
    int32_t lean_ents;    // lean kernel: most entries of a plan
    int32_t lean_stage;   // a wave's staging bytes
    int32_t lean_group;   // mini blocks staged together: 4, 2 or 1
    int32_t lean_log2r;   // copies of an LDS group table: at most 2^lean_log2r
    // A lone plan's guided items (else guided_mb 0): its mini blocks (of its
    // surviving blocks); those of an XCD, from x * xcd_mb on (the last XCDs' may
    // be fewer or none); an XCD's items, the first xcd_big of mb_per_item mini
    // blocks, the rest of small_mb.
    int32_t guided_mb;
    int32_t xcd_mb;
    int32_t xcd_items;
    int32_t xcd_big;
    int32_t small_mb;
    int32_t walk;         // claims look at the other item ranges one by one
};

// Hash build over a dimension table (optionally joined: the rows must find
// their foreign keys in the tables of sub[], probed from device memory).
struct HashBuildArgs {
    DevCol cols[kMaxHashCols];
    int32_t ncols;
    int32_t npreds;
    DevPred preds[kMaxHashPreds];
    int64_t in_vals[kMaxIn];
    int32_t key_col;
    int32_t npay;
    int32_t pay_col[2];   // column, or (pay_src >= 0) payload index of sub[pay_src]
    int32_t pay_src[2];   // -1: a column of cols
    int32_t nsub;
    DevProbe sub[2];
    int32_t nmb;
    int32_t pad;
    int64_t nrows;
    // outputs
    unsigned long long* count;  // qualifying rows
    long long* mm;              // [0..1] key min/max, [2..5] payload min/max
    uint32_t* status;
};

// The table that the insert pass fills.
struct HashTableArgs {
    int32_t* keys;
    void* pay[2];
    int32_t pay64[2];
    uint32_t cap_mask;
    int32_t log2cap;
    uint32_t* bits;     // membership bitmap (nullptr: none)
    int64_t bmin;
    uint32_t* filt;     // bit filter (nullptr: none)
    int32_t flog2;
};

// Launchers.  Each returns the hipError_t of the launch.
// waves: 4, 8 or 16 waves per workgroup.  launch_fused picks the instantiation
// for the batch's string atoms (str_stage), each in a source file of its own.
hipError_t launch_fused(const BatchArgs& a, int waves, int grid, size_t lds_bytes, hipStream_t s);
hipError_t launch_fused_str(const BatchArgs& a, int waves, int grid, size_t lds_bytes, hipStream_t s);
hipError_t launch_fused_fsst(const BatchArgs& a, int waves, int grid, size_t lds_bytes, hipStream_t s);
// The lean kernel: every plan of the batch has lean.ok.
hipError_t launch_lean(const BatchArgs& a, int waves, int grid, size_t lds_bytes, hipStream_t s);
// Per-wave LDS the fused kernel needs (survivor queue, string row offsets).
size_t fused_wave_area_bytes(bool str, bool pend);
hipError_t launch_hash_count(const HashBuildArgs* d_args, int grid, hipStream_t s);
hipError_t launch_hash_insert(const HashBuildArgs* d_args, const HashTableArgs& t, int grid, hipStream_t s);
// p[0 .. nkeys) = kEmptyKey, p[zero_from .. nwords) = 0.
hipError_t launch_hash_clear(int32_t* p, int64_t nkeys, int64_t zero_from, int64_t nwords, hipStream_t s);
// Emits and clears a group table that the fused kernel does not copy itself
// (emit_copy 0).  status: the plan's status words.
hipError_t launch_emit(const DevQuery* d_q, const DevQuery& h_q, int64_t* agg, uint32_t* status, hipStream_t s);
hipError_t launch_fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t s);
// Bandwidth probe: grid x 256 lanes read bytes (a multiple of 16) at p.
hipError_t launch_stream_read(const void* p, uint64_t bytes, uint32_t key, uint32_t* sink, int grid,
                              hipStream_t s);
hipError_t launch_fill_i64(int64_t* p, int64_t v, int64_t n, hipStream_t s);

// Fragmented (multi-kernel) execution of one plan.  Row lists hold row ids
// as uint32: plans cover at most 2^32 - 1 rows, and every decoded array is
// indexed with the id widened to 64 bits.
typedef uint32_t FragRow;
static_assert(sizeof(FragRow) == 4 && FragRow(-1) == UINT32_MAX, "row ids must reach 2^32 - 1");
struct FragBuffers {
    int64_t* dec[kMaxCols];      // decoded integer columns (codes for DICT)
    int64_t* str_off[kMaxCols];  // decoded string offsets [nrows + 1]
    uint8_t* str_bytes[kMaxCols];
    const DevCol* str_col[kMaxCols];  // the column's descriptor with its heap at str_bytes
    uint8_t* flags;              // [nrows]
    FragRow* rows[2];            // ping-pong row lists [nrows]
    int64_t* pay[2][2 * kMaxProbes];  // payload arrays aligned with the row lists
    unsigned long long* counts;  // [kMaxProbes + 2] list lengths
};
// Returns the number of kernels launched, or -1 on a launch error.
int run_fragmented(const DevQuery* d_q, const DevQuery& h_q, const FragBuffers& fb, hipStream_t s);

}  // namespace dpf
