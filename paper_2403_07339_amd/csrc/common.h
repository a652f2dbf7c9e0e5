// Shared declarations of the gfx950 IM-Unpack library (host + device).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

#include "../../include/imunpack.h"

namespace imu {

// ---- error plumbing ---------------------------------------------------------------------------
extern thread_local int g_last_hip_error;

#define IMU_HIP(call)                                   \
    do {                                                \
        hipError_t e__ = (call);                        \
        if (e__ != hipSuccess) {                        \
            imu::g_last_hip_error = (int)e__;           \
            return IMUNPACK_EHIP;                       \
        }                                               \
    } while (0)

#define IMU_TRY(expr)                                   \
    do {                                                \
        int rc__ = (expr);                              \
        if (rc__ != IMUNPACK_OK) return rc__;           \
    } while (0)

static inline int launch_status() {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        g_last_hip_error = (int)e;
        return IMUNPACK_EHIP;
    }
    return IMUNPACK_OK;
}

// Whether what is queued on the stream goes into a graph (or cannot be queued, because another stream's capture forbids it).
static inline bool capturing(hipStream_t st) {
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &status) == hipSuccess) return status != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return true;
}

// ---- geometry shared by planner, scatter and GEMM ----------------------------------------------
constexpr int kTile = 256;       // GEMM output tile edge in unpacked rows (both operands)
constexpr int kChunk = 64;       // physical rows the GEMM epilogue holds at a time; no source row straddles a chunk
constexpr int kChunkPairs = (kTile / kChunk) * (kTile / kChunk);  // 64 x 64 tiles in one of 256 x 256
constexpr int kEvenStep = 32;    // from level to level of an evenly laid out row of B: a column block of the matrix instruction
constexpr int kXcdCus = 32;      // CUs of an XCD
constexpr int kKPad = 128;       // every exponent group is padded to a multiple of this many columns
constexpr int kMaxGroups = 64;   // distinct diagonal entries of S the planner supports
constexpr int kMaxItems = 1024;  // products of a batch that are planned together
constexpr int kBoundBlocks = 256;  // workgroups that measure the accumulator bounds, at most
constexpr int kMaxRuns = 128;    // stretches of consecutive k-tiles that read consecutive blocks of the A store
constexpr int kProwLevel = 24;   // dimensions are at most 2^24, digit levels fewer than 64
constexpr uint32_t kNever = 0xFFFFFFFFu;  // split time of a row/column that is never split

// One set of growing row (or column) slots: what Pi (or S) needs per slot, plus the split
// bookkeeping that lets the scatter kernel follow an entry's digits.
struct SlotSet {
    int32_t *root;    // original row / phase-entry column this slot descends from
    int32_t *exp;     // number of splits between root and this slot (digit level along this axis)
    uint32_t *time;   // when this slot was split (order among all splits of the phase), kNever if not
    int32_t *child;   // slot created by that split, -1 if none
    unsigned long long *key;  // appended slots: order among the appended slots (batch, count desc, split slot)
    int32_t cap;
};

// Header kept on the device and mirrored to the host after planning.
struct PlanHeader {
    int32_t n_u, h_u, d1, d_u;       // n', h', columns after unpacking A, d'
    int32_t Mp, Np, Kp;              // physical (padded) sizes
    int32_t KA;                      // stored columns of A (a multiple of 128)
    int32_t ldA, ldB;                // bytes from one physical row to the next in the A store / in B_eu: the width
                                     // rounded up to an odd multiple of 256, so that the rows of a tile that are
                                     // read together spread over the memory channels
    int32_t mtiles, ntiles;
    int32_t lmaxA, lmaxB;            // largest number of digit levels of a row of A / B
    int32_t ngroups;
    int32_t grp_exp[kMaxGroups];     // exponent of s per group, descending
    int32_t grp_k0[kMaxGroups];      // first physical column
    int32_t grp_len[kMaxGroups];     // columns of the group (whole k-tiles)
    int32_t nruns;                   // k-tiles [run_kt0[i], run_kt0[i+1]) read blocks run_blk0[i], run_blk0[i]+1, ... of the A store
    int32_t run_kt0[kMaxRuns];
    int32_t run_blk0[kMaxRuns];
    int32_t run_grp[kMaxRuns];       // the group the run belongs to
    int32_t edgesA, edgesB;          // OB entry lists built for UnpackBoth
    int32_t nobA, nobB;              // OB entries of A / B kept for the scatter (UnpackBoth operands)
    int32_t nsparse;                 // columns that the fused GEMM takes from lists (see SparseLists) ...
    int32_t list_kt0;                // ... instead of the k-tiles of B_eu from this one on, the last run
    int32_t cols_left;               // the layout that knows lists cannot hold the columns: the general one has yet to place them
    int32_t sparse_room;             // places that the longest list of digits would have needed, if one was too short (else 0)
    int32_t overflow;                // bit set: which capacity was too small
    int32_t need[10];                // size that would have been needed, per capacity
    int32_t err;                     // IMUNPACK_ERANGE conditions found on the device
    uint32_t cols_done;              // column-layout workgroups that have finished (the last one orders the units)
    uint32_t lists_done;             // workgroups that have filled their share of the lists (the last one publishes the header)
    int32_t extras;                  // edges that the repeated columns of B_e add to B's OB entries (UnpackBoth on B)
    int32_t reusedB;                 // the second operand's unpacking was taken over from the plan before (keep-weights mode)
    int32_t chunkB;                  // no source row of B straddles that many physical rows: kTile, or kChunk for small products
    int32_t evenA;                   // 2, 4: every source row of A has that many physical rows side by side (some of them padding)
    int32_t evenB;                   // 2, 4: every source row of B has that many physical rows (some of them padding), kEvenStep apart;
                                     // 0: its levels lie one behind the other
    int32_t seq;                     // in the host's copy: which plan's header it holds
    unsigned long long bound[2];     // max over rows of sum_c s^e(c) |digit| for A_ue, B_eu
};

// What a plan in keep-weights mode remembers of the plan before it, on the device: the column unpacking of
// the first operand that the second operand's unpacking was computed for, and the header fields that unpacking left.
struct KeepState {
    int32_t valid, d1, same;
    int32_t h_u, d_u, nobB, edgesB, extras;
    int32_t pad_[8];
    PlanHeader saved;  // the header as that plan left it: the layout of the second operand and of the columns
};

enum CapIndex { CAP_ROWA = 0, CAP_ROWB = 1, CAP_C1 = 2, CAP_C2 = 3, CAP_EDGEA = 4, CAP_EDGEB = 5, CAP_OB = 6,
                CAP_LISTA = 7, CAP_LISTB = 8,  // (a caller's OB list was too short)
                CAP_SPARSE = 9 };              // places in a list of SparseLists

// Physical-row description used by scatter and by the GEMM epilogue.
struct RowLayout {
    int32_t *prow;        // [Mp]  source row of physical row | its digit level << kProwLevel, -1 = padding
    int32_t *row_phys;    // [n']  physical row of canonical slot
    int32_t *src_pstart;  // [n]   first physical row of source row i
    int32_t *src_nlev;    // [n]   number of levels of source row i
    int32_t *tile_src0;   // [tiles+1] first source row of each tile
    int32_t *chunk_src0;  // [4 tiles+1] first source row of each chunk of kChunk physical rows
    int32_t *tile_flat;   // [tiles]   1 if every source row of the tile has a single level
    int32_t *chunk_lev;   // [4 tiles] (A) how many levels every source row of the chunk has, 0 if they differ
    // weighted L1 norm  sum_c s^e(c) |digit|  per physical row, in pieces: what the fix-up pass placed
    // (cleared by the planner) and one partial sum per wave of the scatter kernel
    unsigned long long *rowsum;   // [Mp]
    unsigned long long *wavesum;  // [Mp][windows per row]
};

// Columns.  B_eu is stored in full: Kp physical columns, one GEMM k-tile per 128 of them, grouped by
// the exponent of the diagonal entry of S.  A_ue repeats column r of A_u in every column slot of the
// second unpacking that descends from r (Alg. 2 line 6 / Alg. 4 line 13); those copies are not
// stored.  The A store holds every column of A_u once, level by level (level 0 = the d original
// columns in order, level a = the columns appended by a-fold splits, ordered by original column), each
// level padded to whole blocks of 128, plus a few blocks of gathered copies for exponent groups that
// use only a small part of a level; the GEMM walks it run by run (PlanHeader::run_*).
struct ColLayout {
    int32_t *pcol_slot;   // [Kp] column slot of the second unpacking in this column of B_eu, -1 = zero column
    int32_t *col_phys;    // [d'] column of B_eu of every column slot of the second unpacking
    int32_t *colB_k;      // [Kp] original column (-1 = zero column)
    int32_t *colB_e;      // [Kp] digit level along the columns of B_e
    int32_t *col_sexp;    // [Kp] exponent of the diagonal entry of S
    int4 *unitB;          // [Kp/16] per 16-column unit: x = first original column, y >= 0 if there is one (-1:
                          // nothing to read), z bit 0: 16 consecutive original columns, bit 1: one digit level for all of
                          // them, bit 2: one weight for all of them; w = that level | exponent of S << 16
    int32_t *acol_phys;   // [d'] stored column of A that every column slot of the second unpacking reads
    int32_t *apos;        // [columns of A_u] stored column of every column slot of A's unpacking
    int32_t *colA_k;      // [KA] original column (-1 = padding)
    int32_t *colA_e;      // [KA] digit level along the columns of A
    unsigned long long *colA_w;   // [KA] sum of s^e over the column slots that read this stored column (what an
                                  // entry of it weighs in the row norm behind the accumulator bound)
    int4 *unitA;          // [KA/16] as unitB (w = level only)
    unsigned long long *unitA_w;  // [KA/16] the weight of the unit's columns if they share one
};

// Columns that UnpackBoth appends to B for a few heavy hitters hold next to nothing but zeros (on a 11008 x 4096 weight with
// 0.1 % of them 9 digits in 11008 places, and there is one for nearly every original column), yet multiplied as columns they double the
// contraction.  Those that carry digit 1 along the columns of an original column (level 0 along A, exponent 1) and few enough
// digits come last in B_eu, in a run of their own that the fused GEMM leaves out: the plan holds their digits in a list for every kSparseRows
// physical rows of B, and the GEMM multiplies a list's digits, 32 at a time, with the columns of A that they meet, which it
// reads from a transposed copy of level 0 of the A store.  Every product of two digits other than zero is still the low-bit GEMM's.
// The lists are written once, by the launch that completes the plan (lists_kernel): an unpack, which may come again, from a graph or
// beside a GEMM on another stream, leaves them alone.
// 4096 x 4096 by 11008: GEMM 343 -> 289 us; a step 452 -> 408 on resident weights, 710 -> 683 where the weights are unpacked in
// every step (planner 6 us more, the copy 5); 16 rows against resident weights that no cache holds 116 -> 84.
//
// An entry: physical row inside the kSparseRows | original column << 7 | digit << 24 (in no particular order: the sums are integers).
// The copy: column k of the store in rows 128 g .. 128 g + 127 is the line of 128 bytes at (g d + k) * 128, row p at its byte
// (p % 32) * 4 + p / 32 % 4, so that one word is what a lane of the matrix instruction needs of the four row blocks of a wave.
constexpr int kSparseRows = 32;
constexpr uint32_t kSparseLine = 0x00ffff80u;  // of an entry: its line in the copy (the column layout in LDS takes 12288 slots, so k < 2^17)
struct SparseLists {
    int32_t *cnt;       // [Np / kSparseRows] entries in a list
    uint32_t *ent;      // list x begins at entry x * cap
    int32_t cap;        // places in a list (a multiple of 32)
};

// ---- batches.  The items of a batch (products of one shape) are planned, unpacked and multiplied by the
// same launches: every device array of item i lies i * stride bytes behind that of item 0 (the headers lie
// side by side in an array of their own), and a kernel moves the pointers it was given to its item.
// (Byte-pointer arithmetic, not integers: through an integer the compiler loses that these are global
// addresses and every access becomes a flat one: 82 -> 99 us for the scatter of a 4096 x 4096 and a 11008 x 4096
// operand.)
template <class T>
__host__ __device__ __forceinline__ T *item_at(T *p, int64_t off) {
    return p ? (T *)((const char *)p + off) : p;
}
__host__ __device__ __forceinline__ void move_to_item(SlotSet &s, int64_t off) {
    s.root = item_at(s.root, off); s.exp = item_at(s.exp, off); s.time = item_at(s.time, off);
    s.child = item_at(s.child, off); s.key = item_at(s.key, off);
}
__host__ __device__ __forceinline__ void move_to_item(RowLayout &l, int64_t off) {
    l.prow = item_at(l.prow, off);
    l.row_phys = item_at(l.row_phys, off); l.src_pstart = item_at(l.src_pstart, off); l.src_nlev = item_at(l.src_nlev, off);
    l.tile_src0 = item_at(l.tile_src0, off); l.chunk_src0 = item_at(l.chunk_src0, off); l.tile_flat = item_at(l.tile_flat, off);
    l.chunk_lev = item_at(l.chunk_lev, off);
    l.rowsum = item_at(l.rowsum, off); l.wavesum = item_at(l.wavesum, off);
}
__host__ __device__ __forceinline__ void move_to_item(ColLayout &c, int64_t off) {
    c.pcol_slot = item_at(c.pcol_slot, off); c.col_phys = item_at(c.col_phys, off); c.colB_k = item_at(c.colB_k, off);
    c.colB_e = item_at(c.colB_e, off); c.col_sexp = item_at(c.col_sexp, off); c.unitB = item_at(c.unitB, off);
    c.acol_phys = item_at(c.acol_phys, off); c.apos = item_at(c.apos, off); c.colA_k = item_at(c.colA_k, off);
    c.colA_e = item_at(c.colA_e, off); c.colA_w = item_at(c.colA_w, off); c.unitA = item_at(c.unitA, off);
    c.unitA_w = item_at(c.unitA_w, off);
}

// What the quantize pass needs to know of a batch: strides in bytes from item to item of the two inputs and of everything that belongs
// to an item (integers, statistics, lists, steps on the device).  flag: if set, `status` is not used and
// what goes wrong in any item is ORed into *flag, which the caller has cleared.
struct QuantBatch {
    int nitems = 1;
    int64_t a_stride = 0, b_stride = 0, out_stride = 0;
    int32_t *flag = nullptr;
};

// ---- wave-wide reductions and scans on the vector ALU's data-parallel-primitive moves (shifts within a
// row of 16 lanes, then the last lane of a row broadcast to the following rows) instead of permutes
// through LDS.  Lanes without a source read 0, so these serve sums and maxima of non-negative values.
#if defined(__HIPCC__)
#define IMU_DPP(v, ctrl, rows, zero_fill) __builtin_amdgcn_update_dpp(0, (int)(v), (ctrl), (rows), 0xf, (zero_fill))
// Inclusive prefix sum over the 64 lanes (lane 63 holds the wave's total).
__device__ __forceinline__ int wave_inclusive_sum(int v) {
    v += IMU_DPP(v, 0x111, 0xf, true);   // row_shr:1
    v += IMU_DPP(v, 0x112, 0xf, true);   // row_shr:2
    v += IMU_DPP(v, 0x114, 0xf, true);   // row_shr:4
    v += IMU_DPP(v, 0x118, 0xf, true);   // row_shr:8
    v += IMU_DPP(v, 0x142, 0xa, false);  // row_bcast:15 into rows 1 and 3
    v += IMU_DPP(v, 0x143, 0xc, false);  // row_bcast:31 into rows 2 and 3
    return v;
}
// Sum over the wave, valid in lane 63 only.
__device__ __forceinline__ unsigned wave_sum_lane63(unsigned v) { return (unsigned)wave_inclusive_sum((int)v); }
// Largest of a non-negative value over the wave, valid in lane 63 only.
__device__ __forceinline__ int wave_max_nonneg_lane63(int v) {
    v = max(v, IMU_DPP(v, 0x111, 0xf, true));
    v = max(v, IMU_DPP(v, 0x112, 0xf, true));
    v = max(v, IMU_DPP(v, 0x114, 0xf, true));
    v = max(v, IMU_DPP(v, 0x118, 0xf, true));
    v = max(v, IMU_DPP(v, 0x142, 0xa, false));
    v = max(v, IMU_DPP(v, 0x143, 0xc, false));
    return v;
}
// The same over each half of the wave, valid in lanes 31 and 63.
__device__ __forceinline__ int half_wave_max_nonneg_last(int v) {
    v = max(v, IMU_DPP(v, 0x111, 0xf, true));
    v = max(v, IMU_DPP(v, 0x112, 0xf, true));
    v = max(v, IMU_DPP(v, 0x114, 0xf, true));
    v = max(v, IMU_DPP(v, 0x118, 0xf, true));
    v = max(v, IMU_DPP(v, 0x142, 0xa, false));
    return v;
}
// Waits until this wave's stores have arrived.  Between words stored to the host's pinned memory (system scope, not cached)
// and the word that says they are there this is all the order it takes; a release at system scope would first write back
// the L2 of the XCD, with megabytes of operands in it.
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
// An accumulator bound for the host (saturated: beyond 2^44 no path asks how far).  The word carries the low bits of the
// sequence number, so that no store has to wait for another.
__device__ __forceinline__ void tell_bound(unsigned long long *word, unsigned long long bound, int32_t seq) {
    const unsigned long long v = bound < (1ull << 44) ? bound : (1ull << 44);
    __hip_atomic_store(word, v | ((unsigned long long)(unsigned)seq << 48), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
// 6-bit floating-point digits in memory.  The matrix instruction takes, per lane, 32 consecutive columns of a
// row as one 192-bit string (column j of the fragment at bits 6j .. 6j+5).  A row stores its columns in
// groups of 64 (48 bytes): the first 128 bits of the group's two fragments (16 bytes each), then their
// last 64 bits (8 bytes each), so that a lane reads its fragment as one aligned 16-byte and one aligned
// 8-byte piece.  The two 8-byte pieces change places in the rows whose index has bit 4 set: the thirty-two
// rows that an 8-byte LDS read serves together then fall on different banks (see fp6_piece in gemm.hip).
// Returns the position, in 32-bit words from the start of the row's 96 bytes of a k-tile, of word i (0..5) of fragment
// `frag` (0, 1) of group `grp` (0, 1) in physical row `row`.
__host__ __device__ __forceinline__ int fp6_dword(int row, int grp, int frag, int i) {
    return 12 * grp + (i < 4 ? 4 * frag + i : 8 + 2 * (frag ^ ((row >> 4) & 1)) + (i - 4));
}
// Where the 96 bytes of k-tile kt of a row begin.  The caches hand 64 bytes at a time to a CU, so that 96 of a row cost 128; the rows
// 2i and 2i + 1 therefore share their bytes: row 2i of the store holds the even k-tiles of both, 192 bytes each, row 2i + 1 the odd
// ones.  A last k-tile without a partner leaves 192 zeros in row 2i + 1; a single one is two rows side by side
// all the same.  12288 stored columns, 16384 rows by 4096: GEMM 451 -> 388 us, the
// scatter that writes them 67 -> 71.
__host__ __device__ __forceinline__ int64_t fp6_ktile(int row, int kt, int64_t ld) {
    return ((row & ~1) + (kt & 1)) * ld + (kt >> 1) * 192 + (row & 1) * 96;
}
// int8 digits in memory: rows 2i and 2i + 1 of a store share their bytes, so that 64 columns of both are one line of 128 bytes: row 2i
// holds the columns [128 k, 128 k + 64) of both, row 2i + 1 the other half.  A GEMM that walks the contraction 64 columns at a time
// still fetches whole lines (64 bytes of a line at a time arrive at some 25 bytes per clock and CU, whole lines at 41).
// Where byte `col` of row `row` lies:
__host__ __device__ __forceinline__ int64_t i8_at(int row, int col, int64_t ld) {
    return ((row & ~1) + ((col >> 6) & 1)) * ld + (col >> 7) * 128 + (row & 1) * 64 + (col & 63);
}
// The digits above digit 0 of an OB entry of magnitude av at row slot R and column slot C of an operand unpacked by UnpackBoth,
// emit(row slot, column slot, digit) for those that are not zero: the remainder floor(av / s) moves to the child of whichever of R
// and C was split first (Alg. 4 lines 7-9 / 11-14).
template <class E>
__device__ __forceinline__ void digits_above(const SlotSet &rows, const SlotSet &cols, int R, int C, unsigned av, int sh, E emit) {
    unsigned rem = av;
    for (int step = 0; step < 40; ++step) {
        rem >>= sh;
        if (rem == 0) break;
        const uint32_t tr = rows.time[R], tc = cols.time[C];
        if (tr < tc) R = rows.child[R];
        else if (tc != kNever) C = cols.child[C];
        else break;  // an OB remainder nothing splits: not a complete plan
        if (R < 0 || C < 0) break;
        const int m = (int)(rem & ((1u << sh) - 1u));
        if (m != 0) emit(R, C, m);
    }
}
// Lane 63's value in every lane (a scalar register).
__device__ __forceinline__ int from_lane63(int v) { return __builtin_amdgcn_readlane(v, 63); }
#endif

}  // namespace imu

// Opaque plan object.
struct imunpack_plan {
    // problem
    int64_t n, d, h;
    int b, sA, sB;
    int s, sh;
    hipStream_t stream;
    // device arena
    char *arena;
    size_t arena_bytes;
    // capacities (grow on overflow)
    int32_t cap[10];
    // views into the arena (valid after a successful imunpack_plan)
    imu::PlanHeader *d_hdr;       // one per item
    imu::PlanHeader hdr;          // host mirror (of item 0)
    imu::PlanHeader *pin_hdr;     // pinned copies of the headers, written by the kernels that complete them
    int pin_items;                // ... how many of them fit
    // batch: the plans of `nitems` products of one shape, made by the same launches (1: a plan of its own)
    int nitems;
    int64_t item_bytes;           // from the arrays of one item in the arena to those of the next
    int64_t op_stride;            // from item to item: the integer operands, their statistics and OB lists
    void *split_ws;               // where the parts of a GEMM tile meet (gemm.hip), if a product needed it
    hipEvent_t split_done;        // recorded behind the launch that used it last
    int gemm_halves;              // whether that ran in half tiles (imunpack_diag_gemm_halves)
    int gemm_parts;               // parts of a tile in the last fused launch (0: 64 x 64 tiles; imunpack_diag_gemm_parts)
    int chunkB;                   // kChunk if the rows of B may be laid out for the small-tile GEMM (PlanHeader::chunkB: whether they are)
    int32_t seq;                  // of the last header or bounds that the host asked for (the kernel writes it with them)
    unsigned long long *pin_bounds;  // pinned, behind the headers: two words per workgroup that measured the bounds
    int bound_pending;            // the bounds of the last imunpack_unpack have not been read back yet
    int32_t bound_seq;            // ... and carry this number
    int bound_words;              // ... in that many pinned words (0: the unpack was captured into a graph, none are written)
    int guess_fusable;            // whether the fused GEMM was exact for this plan object the last time
    imu::SlotSet rowA, rowB, c1, c2;
    imu::RowLayout layA, layB;
    imu::ColLayout cols;
    imu::SparseLists sparse;          // ent == nullptr: the fused GEMM multiplies every column of B_eu
    int no_sparse;                    // plans of this shape get no lists: they have more columns than the layout of those holds
    int8_t *at;                       // the transposed copy of level 0 of the A store (with lists: room for all physical rows there may be)
    int32_t *statsA[4], *statsB[4];   // rowcnt, colcnt, rowmax, colmax actually used
    // greedy scratch
    unsigned long long *edges;        // two lists of edge_cap packed edges each
    int edge_cap;
    int32_t *rcnt, *ccnt;
    int32_t *extraRows;               // per row of B: how many of those extra edges it has
    int32_t *obcopyA, *obcopyB;       // OB entries of an UnpackBoth operand, kept for the scatter: [3][cap[CAP_EDGEx]]
    int32_t *ob, *obcnt;              // own OB entry list [3][cap[CAP_OB]] when the caller gave none, and its length
    int32_t *tmpL, *tmpCur, *tmpPA, *tmpPB, *tmpE, *tmpK, *tmpR, *tmpOff;
    int ignore_listA, ignore_listB;   // a caller's OB list overflowed: scan the operand ourselves
    int bothA, bothB;                 // slot numbering of the set needs the export-time sort
    // canonical (paper-order) numbering, built lazily by the export / test paths
    int canon_valid;
    int32_t *canon_rowphysA, *canon_rowphysB, *canon_colphys, *canon_acolphys;   // device, indexed by canonical slot
    int fusable;      // set by imunpack_unpack
    int unpacked;
    int valid;
    int keep_B;       // keep-weights mode: the second operand is the same from plan to plan
    int keep_valid;   // the arena holds a complete unpacking of the second operand and the snapshot it belongs to
    unsigned long long keep_sig;  // ... for the arena layout with this signature
    int32_t *snapRoot, *snapExp, *snapChild;  // the first operand's column slots at that time
    const int8_t *kept_Beu;  // the buffer the last imunpack_unpack wrote B_eu to, while it still matches the plan
    int kept_Beu_fp6;
    imu::KeepState *d_keep;
    int digits_req;   // IMUNPACK_DIGITS_*: what imunpack_plan_set_digits asked for (kept across re-planning)
    int fp6;          // in effect for the current plan: 6-bit floating-point digits (requested and b <= 4)
};

namespace imu {
using Plan = struct ::imunpack_plan;  // the C function imunpack_plan() hides the bare struct name

// Products that the small-tile GEMM may be the better one for (gemm.hip decides once the unpacked sizes are known: never
// above about 120 tiles of unpacked rows).
inline bool small_tiles_possible(int64_t n, int64_t h, int nitems) {
    return ((n + kTile - 1) / kTile) * ((h + kTile - 1) / kTile) * nitems <= 128;
}

// Into how many parts the tiles of the last round are cut (1: not at all): where at most half of the CUs would work on it and
// the contraction is long enough.  Cut in four, the round is not four times as fast (CUs that share L2 and power walk
// slower, and 256 KiB of sums change hands per part): 4096 x 8448 by 8448 rows, 66 k-tiles: 402 -> 381 us; 17408 rows,
// 96 k-tiles of six-bit digits: 518 -> 493; 2048 x 15104 by 2048, 118 k-tiles: 140 -> 81; 3072 x 6144 by 6400, 48: 138 -> 125;
// but 32 k-tiles: 430 -> 434, 19: 37 -> 42.  In eight parts none was faster than in four.
__host__ __device__ inline int split_parts(int64_t tiles, int64_t ktiles) {
    const int m = (int)((tiles + 7) / 8 % kXcdCus);
    if (m == 0 || m > kXcdCus / 2 || ktiles < 48) return 1;
    return kXcdCus / m < 4 ? kXcdCus / m : 4;
}

// Whether 64 x 64 tiles are the better ones for `tiles` tiles of 256 x 256, of which `pairs` chunk pairs hold anything, with
// `ktiles` k-tiles each, from what either kernel measured (nanoseconds): a 256 x 256 tile takes 14 us and 1.05 us per k-tile, 256
// of them at a time (one round of tiles in parts: 20 us and 0.52 us per k-tile); the small tiles take 0.2 us and 10 ns per
// k-tile for each sixteen of them, and no less than 0.3 us per k-tile.  (1024 x 1664 by 2048 rows, 32 tiles: 27 and 12 us;
// 2048 x 1152 by 2048, 64 tiles: 28 and 24; 3072 x 1920 by 2048, 96 tiles: 29 and 32; 3840 x 1024 by 2048, 120 tiles: 22 and 30;
// 4096 x 1920 by 2048, 128 tiles: 31 and 42; 2048 x 15104 by 2048: 81 in parts and 96; 3328 x 4608 by 768, 39 tiles: 51 and 29.)
// `single`: a product of its own, whose last round may be cut.  margin: percent by which the large tiles have to be better.
// tile_ns: what a tile takes besides its walk, kTileNs where its results go out from the registers.
constexpr int kTileNs = 14000;
__host__ __device__ inline bool small_tiles_win(int64_t tiles, int64_t pairs, int64_t ktiles, bool single, int margin, int tile_ns = kTileNs) {
    const int64_t walk = 300 * ktiles, work = pairs * (200 + 10 * ktiles) / kChunkPairs;
    const int64_t small = 6000 + (walk > work ? walk : work);
    const bool parts = single && tiles <= 256 && split_parts(tiles, ktiles) > 1;
    const int64_t large = parts ? tile_ns + 6000 + 520 * ktiles : (tiles + 255) / 256 * (tile_ns + 1050 * ktiles);
    return small * 100 < large * (100 + margin);
}

// Waits until a kernel on `st` has written `want` to a word of pinned memory (behind the data that goes with it).  The host
// polls the word: a blocking wait costs tens of microseconds of wake-up during which the GPU idles between two stages of
// the path, and a copy with an event behind it a launch and three calls.  (All pinned memory that kernels write while the host
// polls it is allocated as coherent, whatever the environment's default.)
template <class T>
int wait_word(const T *word, T want, hipStream_t st);
// The entry points' inner forms, which also serve the items of a batch (p->nitems of them).
int plan_impl(const int32_t *A, int64_t n, int64_t d, int64_t lda, const int32_t *B, int64_t h, int64_t ldb, int b,
              int strategy_A, int strategy_B, const imunpack_stats_t *stats_A, const imunpack_stats_t *stats_B,
              imunpack_plan_t **plan, int nitems, int64_t op_stride, hipStream_t st);
Plan item_view(const Plan &batch, int i);
// Device memory that the plan of one item of a batch takes (before anything overflows its first guesses).
int64_t plan_item_bytes(int64_t n, int64_t d, int64_t h, int b, int strategy_A, int strategy_B);
int unpack_impl(imunpack_plan_t *p, const int32_t *A, int64_t lda, const int32_t *B, int64_t ldb, int8_t *A_ue,
                int64_t a_stride, int8_t *B_eu, int64_t b_stride, hipStream_t st);
int quantize_pair(const float *A, int64_t n, int64_t sa_r, int64_t sa_c, float scale_A, const float *scale_A_dev,
                  int32_t *QA, int64_t ldqa, const imunpack_stats_t *stA, const float *B, int64_t h, int64_t sb_r,
                  int64_t sb_c, float scale_B, const float *scale_B_dev, int32_t *QB, int64_t ldqb,
                  const imunpack_stats_t *stB, int64_t d, int b, int32_t *status, const QuantBatch &bt, hipStream_t stream);
int gemm_impl(imunpack_plan_t *p, const int8_t *A_ue, const int8_t *B_eu, void *workspace, int64_t *C_int,
              float *C_fp, int64_t ldc, float scale_A, float scale_B, const float *scale_a_dev,
              const float *scale_b_dev, int fuse, hipStream_t stream);
// The fused launch for every item of a batch.  An item whose accumulator bound is too large for it writes
// nothing and sets refused[item] (device, cleared by the caller).
int gemm_batch(imunpack_plan_t *p, const int8_t *A_ue, int64_t a_stride, const int8_t *B_eu, int64_t b_stride, float *C_fp,
               int64_t c_stride, int64_t ldc, const float *scale_a_dev, const float *scale_b_dev, int64_t scale_stride,
               int32_t *refused, hipStream_t stream);
// The RTN steps of both operands of every item of a batch (percentile.hip); ws: two workspaces side by side.
int rtn_step_pair(const float *A, int64_t n, int64_t sa_r, int64_t sa_c, float beta_A, const float *B, int64_t h, int64_t sb_r,
                  int64_t sb_c, float beta_B, int64_t d, double p, float *steps, void *ws, const QuantBatch &bt, hipStream_t st);
// Waits for the bounds of the last imunpack_unpack and sets p->fusable.
int resolve_bound(Plan *p);
// Bytes from one physical row to the next of the A store (op 0) / of B_eu (op 1) in the digit format in
// effect.  6-bit digits: 96 bytes per k-tile of 128 columns, pairs of k-tiles (see fp6_ktile), the same rule against power-of-two
// pitches.
__host__ __device__ inline int header_pitch(const PlanHeader &h, int fp6, int op) {
    if (!fp6) return op ? h.ldB : h.ldA;
    const int tiles = (op ? h.Kp : h.KA) / kKPad, bytes = (tiles + (tiles > 1 ? tiles & 1 : 0)) * 96;
    return bytes >= 2048 ? (((bytes + 255) / 256) | 1) * 256 : bytes;
}
inline int64_t store_pitch(const Plan *p, int op) { return header_pitch(p->hdr, p->fp6, op); }
}
