// int8 MFMA GEMM over the unpacked operands (Alg. 3, ScaledMatMul) with the recombination
// (Sec. 4 "Reconstructing A": Pi applied as an index-add with power-of-two weights) and the
// dequantisation (Sec. 2, Eq. quantized_gemm) fused into the epilogue.
//
// Alg. 3 runs one GEMM per distinct diagonal entry s^e of S and adds them with weight s^e.  The
// physical column order puts the groups one after the other, highest exponent first, so a single
// pass over K evaluates  sum_e s^e C_e  by Horner's rule: the int32 accumulators are shifted left
// by (b-1) * (e_g - e_{g+1}) between group g and group g+1.  That is exact whenever the weighted
// sum fits int32, which imunpack_unpack checks for the actual operands; otherwise each group is
// launched on its own and accumulated in int64 (the un-fused path).
#include "common.h"

#include <algorithm>
#include <atomic>
#include <cstdlib>
#include <cstring>
#include <type_traits>

// first register of every aligned quad of the 256 accumulation registers
#define IMU_ACC_QUADS "0,4,8,12,16,20,24,28,32,36,40,44,48,52,56,60,64,68,72,76,80,84,88,92,96,100,104,108,112,116,120,124,128,132,136,140,144,148,152,156,160,164,168,172,176,180,184,188,192,196,200,204,208,212,216,220,224,228,232,236,240,244,248,252"

namespace imu {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f_u __attribute__((ext_vector_type(4), aligned(4)));  // 16 bytes at any float boundary
typedef long v2l_u __attribute__((ext_vector_type(2), aligned(8)));

constexpr int BM = kTile, BN = kTile, BK = 128;  // bytes (= int8 elements) of K per LDS stage: one full 128-byte line per row
constexpr int kGemmThreads = 256;                // 4 waves, 2 x 2, each 128 x 128
constexpr int kHalfBytes = BM * BK;              // 32 KiB: the A tile or the B tile of one k-tile
constexpr int kRing = 5;                         // LDS ring of half-stages: A(k) in slot 2k mod 5, B(k) in slot 2k+1 mod 5
constexpr int kGemmLds = kRing * kHalfBytes;     // all 160 KiB of the CU's LDS
// Two workgroups to a CU: tiles of 128 x 256, three stages of a piece of 64 columns each, and 2 KiB for every wave beside them.
constexpr int kDualRows = 128, kDualStages = 3, kDualStage = (kDualRows + BN) * 64, kDualSpare = 2048;
constexpr int kDualLds = kDualStages * kDualStage + 4 * kDualSpare;  // 80 KiB

struct GemmArgs {
    const int8_t *A, *B;      // the A store [Mp][ldA] and B_eu [Np][ldB] (row pitches in bytes)
    int ldA, ldB, Kp, mtiles, ntiles;
    int kt0, kt1;             // k-tile range of this launch
    // The range is cut into segments at the k-tiles where the exponent group changes (Horner step) or
    // where the walk through the A store jumps: k-tile kt of segment i reads block kt + seg_delta[i].
    int nbound;               // boundaries inside the range
    int bound_kt[kMaxGroups]; // segment i ends with this k-tile ...
    int bound_sh[kMaxGroups]; // ... after which the accumulators are shifted by this many bits (0: same group)
    int seg_delta[kMaxGroups + 1];
    // fused epilogue
    RowLayout layA, layB;
    int sh, final_shift;
    int64_t *C_int;
    float *C_fp;
    int64_t ldc;
    double scale;             // scale_A * scale_B
    const float *scale_a_dev, *scale_b_dev;  // if set: the two RTN steps are read from device memory instead
    // un-fused: C_u[p][q] (+)= acc << seg_shift
    int64_t *C_u;
    int Np;
    int seg_shift, seg_first;
    // fused launch made before the host knows the accumulator bounds: the kernel checks them itself
    // and writes nothing if the shifted group sum could leave int32
    const unsigned long long *guard;
    int guard_mul;            // s - 1
    int fold_f64;             // no int64 output wanted and every sum over digit levels is exact in binary64
    // batch (blockIdx.y is the item): everything above that the plan decides comes from the item's header;
    // an item that may not be fused writes nothing and sets refused[item]
    const PlanHeader *hdr;    // nullptr: not a batch
    int64_t a_stride, b_stride, c_stride, plan_stride, scale_stride;  // bytes from item to item
    int32_t *refused;
    // split: two words per meeting point (arrivals, how many have left their sums), and the sums of those that came first
    int32_t *meet, *sums;
    int most_parts;
    int evenB;                // PlanHeader::evenB
    int whole_rows;           // results without levels to fold leave row by row (see whole_rows_win)
    int lmaxA;                // largest number of digit levels of a row of A
    int kwaves;               // gemm_small_kernel: waves that share the contraction
    // columns of B that are taken from lists (SparseLists): they come in before k-tile sp_kt (-1: there are none), where the large tiles'
    // accumulators count in units of s, and are followed by a shift of sp_after bits (which the shift in front of that k-tile, if there is
    // a group before it, contains: the small tiles, which keep the lists' sums apart, know nothing of sp_after)
    SparseLists sparse;
    const int8_t *at;         // the transposed copy of level 0 of the A store
    int at_cols;              // ... lines of 128 bytes to a block of 128 rows
    int sp_kt, sp_after;
    // benchmark reporting: if set, workgroup 0 writes {shader clock ticks, 100 MHz wall ticks} of its K loop
    unsigned long long *clock_probe;
};

// XCD-aware tile order: workgroup ids are dealt round-robin to the 8 XCDs, each with its own L2,
// so ids that land on one XCD are given one contiguous run of tiles; inside a run the tiles walk
// bands of 4 tile-rows so that an XCD's resident workgroups share A and B panels.
template <int kBand = 4, bool DEAL = false>
__device__ __forceinline__ void place_tile(int logical, int mtiles, int ntiles, int &tm, int &tn);
template <int kBand = 4, bool DEAL = false>
__device__ __forceinline__ void tile_of(int wg, int mtiles, int ntiles, int &tm, int &tn) {
    const int total = mtiles * ntiles;
    const int xcd = wg & 7, idx = wg >> 3;
    const int per = total >> 3, rem = total & 7;
    const int logical = xcd * per + min(xcd, rem) + idx;
    place_tile<kBand, DEAL>(logical, mtiles, ntiles, tm, tn);
}
template <int kBand, bool DEAL>
__device__ __forceinline__ void place_tile(int logical, int mtiles, int ntiles, int &tm, int &tn) {
    const int band_sz = kBand * ntiles;
    const int band = logical / band_sz;
    const int first_m = band * kBand;
    const int rows_in_band = min(kBand, mtiles - first_m);
    const int in_band = logical - band * band_sz;
    tm = first_m + in_band % rows_in_band;
    tn = in_band / rows_in_band;
    if constexpr (DEAL) {
        // XCDs to a band.  They share its columns out one by one, not in stretches: the rows of B that were written last are still in the
        // last-level cache, the ones before them are not, and the XCDs that had those were a third slower per k-tile (4096 x 4352 by 11013:
        // kernel 266 -> 245 us in a step).
        const int m = 8 * kBand / max(mtiles, kBand);
        if (m > 1) {
            const int q = ntiles / m, r = ntiles - q * m;  // the first r of them have q + 1 columns
            const int k = tn < r * (q + 1) ? tn / (q + 1) : r + (q > 0 ? (tn - r * (q + 1)) / q : 0);
            tn = (tn - k * q - min(k, r)) * m + k;
        }
    }
}

// A launch of whole tiles ends in a round that leaves CUs idle (561 tiles on 256 CUs are 2.2 rounds, paid as 3).  Here the
// tiles of that round are cut along the contraction into as many equal parts as there are CUs for (up to `most`), one
// workgroup each.  All workgroups of an XCD still walk the contraction side by side, which is what lets its L2 serve them:
// dealing tiles x k-tiles out in equal stretches, every CU at a k-tile of its own, left no CU idle and was slower for all
// that (344 -> 411 us at 4096 x 8228 x 11013).
struct Piece {
    int tile, ka, kb;  // tile of the XCD's order, its k-tiles [ka, kb)
    int parts, slot;   // parts of the tile; where they meet (slot, slot + 1, ... for the sums of all but the last)
};
__device__ __forceinline__ bool piece_of(int wg, int mtiles, int ntiles, int K, int most, Piece &pc) {
    const int total = mtiles * ntiles, xcd = wg & 7, idx = wg >> 3;
    const int per = total >> 3, rem = total & 7;
    const int T = per + (xcd < rem ? 1 : 0), first = xcd * per + min(xcd, rem);
    const int whole = T / kXcdCus * kXcdCus, m = T - whole;
    pc.ka = 0;
    pc.kb = K;
    pc.parts = 1;
    pc.slot = 0;
    pc.tile = first + idx;
    if (idx < whole) return true;
    if (m == 0) return false;
    pc.parts = min(kXcdCus / m, most);
    const int t = idx - whole, part = t / m;
    if (part >= pc.parts) return false;
    pc.tile = first + whole + t % m;
    pc.slot = xcd * kXcdCus + (t % m) * pc.parts;
    pc.ka = K * part / pc.parts;
    pc.kb = K * (part + 1) / pc.parts;
    return true;
}

// One direct-to-LDS load: every lane fetches 16 bytes from gbase + voff and the wave's 1 KiB lands
// contiguously at LDS byte address lds_addr (lane l at lds_addr + 16 l).  The LDS base travels in M0.
__device__ __forceinline__ void dma16(unsigned lds_addr, unsigned voff, const int8_t *gbase) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :
                 : "s"(lds_addr), "v"(voff), "s"(gbase)
                 : "memory");
}

// (double)x by way of its bits: a conversion takes four times as long as an addition in binary64.
__device__ __forceinline__ double exact_f64(int x) { return __hiloint2double(0x43300000, x ^ (int)0x80000000) - 4503601774854144.0 /* 2^52 + 2^31 */; }
// One word at `off` bytes from the base, dropped by the hardware if that is not below the resource's size.
template <bool NT>
__device__ __forceinline__ void store_inside(float v, __amdgpu_buffer_rsrc_t to, unsigned off) {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), to, (int)off, 0, NT ? 2 : 0);
}
// The same for four, 16 bytes at any boundary; non-temporal: a wave writes a contiguous kilobyte.
__device__ __forceinline__ void store_inside4(const float (&f)[4], __amdgpu_buffer_rsrc_t to, unsigned off) {
    v4i x;
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k] = __float_as_int(f[k]);
    __builtin_amdgcn_raw_buffer_store_b128(x, to, (int)off, 0, 2);
}
// An offset that stays outside with the offset of a row added: a chunk of C ends below 2^31 bytes and no row is asked for further
// than kRowsAhead behind a chunk, so that the sum stays below 2^32 and at 2^31 or beyond.
constexpr unsigned kOutside = 0x80000000u;
constexpr int64_t kDirectPitch = 1 << 22;  // results leave by 32-bit offsets where a row of C is shorter (in elements)
constexpr int kRowsAhead = 16;
static_assert((kChunk + kRowsAhead) * kDirectPitch * (int64_t)sizeof(float) < (int64_t)kOutside, "offsets of rows");

__device__ __forceinline__ const int8_t *uniform_ptr(const int8_t *p) {
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (const int8_t *)(((uint64_t)hi << 32) | lo);
}

// c += a b on accumulation registers, by hand: with the builtin in a second place the compiler moves accumulators between the two
// register files on the way (253 registers spilled).  The operands may have been written just before (two wait states); what
// reads c next has to wait for it.  (Where the sums are ordinary registers the builtin does as well, and the compiler sees to the waits.)
__device__ __forceinline__ void mfma_in_place(const v4i &a, const v4i &b, v16i &c) {
    asm volatile("s_nop 1\n\tv_mfma_i32_32x32x32_i8 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}

// 32 S entries of a list of SparseLists as the operands of S matrix instructions, entry 32 s + 16 h + i at byte i of lane half h of
// instruction s, by way of list_lds(S) bytes of LDS that the wave has to itself: the digits of one instruction after the other in fragment order,
// behind them the entries.  (Digits put together in registers, every lane comparing sixteen rows: 20 000 cycles of the vector
// ALU for the four lists of a wave at 4096 columns of 9 digits in 11008 rows, 11 000 so; 8 000 more for what the loads of A's copy,
// from the last-level cache, leave uncovered.  More of them in flight, beside more registers held, were slower; with
// two workgroups to a CU two instructions at a time are the most that registers allow: one 20 000, two 15 000 cycles, four spill.)
constexpr int list_lds(int S) { return 1024 + 128 * S; }
template <int S>
struct ListWords {
    unsigned w[(S + 1) / 2];
    __device__ __forceinline__ void load(const uint32_t *ent, int lane) {
#pragma unroll
        for (int j = 0; j < (S + 1) / 2; ++j) w[j] = ent[64 * j + lane];
    }
    // the first `left` (at least one) are entries; digits[s]: the operand of instruction s, put together in the same place as the ones
    // before and behind it (a wave's LDS accesses are served in order)
    __device__ __forceinline__ void stage(int8_t *lds, int left, int lane, v4i (&digits)[S]) const {
        const unsigned none = (unsigned)__builtin_amdgcn_readfirstlane((int)w[0]) & kSparseLine;  // what is not there meets the first one's column
#pragma unroll
        for (int j = 0; j < (S + 1) / 2; ++j) {
            const int t = 64 * j + lane;
            if (S < 2 && t >= 32) continue;
            *reinterpret_cast<unsigned *>(lds + 1024 + 4 * t) = t < left ? w[j] : none;
        }
        asm volatile("" ::: "memory");
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const unsigned e = w[s >> 1];
            const int t = 64 * (s >> 1) + lane;
            *reinterpret_cast<v4i *>(lds + 16 * lane) = v4i{0, 0, 0, 0};
            if (lane >> 5 == (s & 1) && t < left) lds[16 * ((int)(e & (kSparseRows - 1)) + 2 * (t & 16)) + (t & 15)] = (int8_t)(e >> 24);
            asm volatile("" ::: "memory");  // (other lanes' stores: what a lane put there itself is not what it reads)
            digits[s] = *reinterpret_cast<const v4i *>(lds + 16 * lane);
        }
    }
};
// the words of A's copy that the entries of instruction s meet, one byte per block of 32 rows of A
__device__ __forceinline__ void list_columns(unsigned (&x)[16], const int8_t *entries, int s, int lhalf, const int8_t *at, unsigned row_off) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const v4i e = *reinterpret_cast<const v4i *>(entries + 128 * s + 64 * lhalf + 16 * q);
#pragma unroll
        for (int i = 0; i < 4; ++i) x[4 * q + i] = *reinterpret_cast<const unsigned *>(at + (((unsigned)e[i] & kSparseLine) | row_off));
    }
}
// f[rb]: sixteen columns in row block rb
__device__ __forceinline__ void list_rows(const unsigned (&x)[16], v4i (&f)[4]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const unsigned a = __builtin_amdgcn_perm(x[4 * q + 1], x[4 * q], 0x05010400u), b = __builtin_amdgcn_perm(x[4 * q + 1], x[4 * q], 0x07030602u);
        const unsigned c = __builtin_amdgcn_perm(x[4 * q + 3], x[4 * q + 2], 0x05010400u), d = __builtin_amdgcn_perm(x[4 * q + 3], x[4 * q + 2], 0x07030602u);
        f[0][q] = (int)__builtin_amdgcn_perm(c, a, 0x05040100u);
        f[1][q] = (int)__builtin_amdgcn_perm(c, a, 0x07060302u);
        f[2][q] = (int)__builtin_amdgcn_perm(d, b, 0x05040100u);
        f[3][q] = (int)__builtin_amdgcn_perm(d, b, 0x07060302u);
    }
}

// LDS half-stage: [256 rows][128 B] of one operand; the eight 16-byte chunks of a row are XOR-swizzled
// with bits 1..3 of the row (chunk kc of row r lives at r*128 + ((kc ^ ((r >> 1) & 7)) << 4)), which
// makes the 64-lane ds_read_b128 of an MFMA operand (32 rows x 2 chunks) conflict-free.
//
// FP6 = true: the digits are 6-bit floating-point codes (b <= 4).  A k-tile is still 128 columns, now 96
// bytes of a row, in LDS as in memory, but for the six 16-byte pieces of a row changing places two by two in
// rows whose index has bit 3 set (fp6_piece); a lane's fragment of v_mfma_f32_32x32x64_f8f6f4 is one 16-byte and one 8-byte
// read (see fp6_dword); a k-tile is two k-steps of 16 matrix instructions; the accumulators are binary32 and hold integers
// below 2^24, exactly.
//
// BATCH: the items of a batch (blockIdx.y) in one launch; what the plan decides comes from the item's header.  A
// variant of its own: read through a run-time choice, those values cost the one-product kernel its last
// registers (101 spilled; 348 -> 460 us on a 4096 x 8228 x 11013 unpacked product).
// LISTS: some columns of B are taken from lists (int8, a product of its own); a variant of its own for the registers' sake too.
//
// DUAL: two workgroups to a CU, each with a tile of 128 x 256 (a wave: 128 x 64, whose sums are ordinary vector registers: 128 of 256)
// and half of the LDS.  A workgroup with a CU to itself leaves the matrix cores idle while its first k-tiles arrive, while it takes
// columns from lists, shifts its sums and stores its results: 34 k-tiles of 4096 x 4352 by 11013 were 83 000 cycles of a tile's 190 000
// (lists 26 000, results 41 000, what loads from beyond L2 take longer than the ring covers 25 000).  Here the other workgroup goes on
// meanwhile; the two drift apart by themselves, since the older one's waves are served first.  Times stand at dual_wins.
//
// fp6_piece: rows 96 bytes apart begin at eight multiples of eight of the 64 banks, rows 8 apart at the same one; with pieces
// moved by one in every second eight rows the sixteen that a 16-byte read serves per cycle have four banks each and, with the
// swap of fp6_dword, the 32 of an 8-byte read two.  (Rows 112 bytes apart did the same with a seventh load that brought nothing.)
__device__ __forceinline__ int fp6_piece(int row, int piece) { return piece ^ ((row >> 3) & 1); }
template <int MODE, bool FP6, bool BATCH = false, bool SPLIT = false, bool LISTS = false, bool DUAL = false>  // SPLIT: parts of tiles (see piece_of); MODE 0: fused epilogue, 1: int64 segment into C_u
__device__ __forceinline__ void gemm_body(const GemmArgs &g, int8_t *smem) {
    static_assert(!DUAL || (MODE == 0 && !FP6 && !BATCH && !SPLIT), "variants with two workgroups to a CU");
    constexpr int BM = DUAL ? kDualRows : imu::BM;
    constexpr int kChunks = BM / kChunk;           // chunks of A in the tile
    constexpr int NB = DUAL ? 2 : 4;               // blocks of 32 columns of a wave (and four of 32 rows)
    constexpr int kRowB = FP6 ? 96 : BK;           // bytes of a row of the operand per k-tile
    constexpr int kPitch = kRowB;                  // bytes from row to row in LDS
    constexpr int kHalfBytes = BM * kPitch;        // the A tile or the B tile of one k-tile in LDS
    constexpr int kLoads = FP6 ? 6 : 8;            // direct-to-LDS loads per wave and half-stage
    constexpr int kWaveBytes = 64 * kPitch;        // a wave's 64 rows of a half-stage
    const int tid = threadIdx.x, lane = tid & 63;
    const PlanHeader *hdr = BATCH ? g.hdr + blockIdx.y : nullptr;
    int mtiles = g.mtiles, ntiles = g.ntiles, ldA = g.ldA, ldB = g.ldB, kt0 = g.kt0, kt1 = g.kt1, nbound = g.nbound;
    if constexpr (BATCH) {
        mtiles = hdr->mtiles; ntiles = hdr->ntiles;
        if ((int)blockIdx.x >= mtiles * ntiles) return;  // the grid covers the largest item
        ldA = header_pitch(*hdr, FP6, 0); ldB = header_pitch(*hdr, FP6, 1);
        kt0 = 0; kt1 = hdr->Kp / BK;
        nbound = hdr->nruns - 1;
    }
    // (DUAL: the branch on them stands behind the first loads; the words themselves, read under a condition, are waited for here.)
    unsigned long long bound0 = 0, bound1 = 0;
    if (MODE == 0 && (BATCH || g.guard)) {
        const unsigned long long *guard = BATCH ? hdr->bound : g.guard;
        bound0 = guard[0];
        bound1 = guard[1];
    }
    auto inexact = [&]() __attribute__((always_inline)) {
        const unsigned long long m = bound0 < bound1 ? bound0 : bound1;
        const bool bad = !(m < (1ull << 40) && m * (unsigned long long)g.guard_mul < (1ull << (FP6 ? 24 : 31))) || (BATCH && nbound >= 63);
        if (bad && g.refused && blockIdx.x == 0 && tid == 0) g.refused[blockIdx.y] = 1;
        return bad;
    };
    if (!DUAL && MODE == 0 && (BATCH || g.guard) && inexact()) return;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = DUAL ? 0 : wave >> 1, wn = DUAL ? wave : wave & 1;  // of the 128 rows and the 32 NB columns of the wave
    int tm, tn;
    Piece pc;
    const int ktiles = kt1;
    if constexpr (SPLIT) {
        if (!piece_of(blockIdx.x, mtiles, ntiles, ktiles, g.most_parts, pc)) return;
        place_tile(pc.tile, mtiles, ntiles, tm, tn);
        kt0 = __builtin_amdgcn_readfirstlane(pc.ka);
        kt1 = __builtin_amdgcn_readfirstlane(pc.kb);
        tm = __builtin_amdgcn_readfirstlane(tm);
        tn = __builtin_amdgcn_readfirstlane(tn);
    } else {
        tile_of<DUAL ? 8 : 4, DUAL>(blockIdx.x, DUAL ? mtiles * (imu::BM / BM) : mtiles, ntiles, tm, tn);
    }
    const int m0 = tm * BM, n0 = tn * BN;
    const unsigned lds0 = (unsigned)(size_t)smem;

    // ---- global -> LDS: wave w fills rows [64w, 64w+64) of the A tile and of the B tile, 8 rows x 128 B
    // (1 KiB) per load; lane l writes slot l&7 of row l>>3, so it fetches the 16-byte chunk that
    // belongs there under the swizzle: chunk kc of row r lives at r*128 + ((kc ^ ((r >> 1) & 7)) << 4),
    // which makes the 64-lane ds_read_b128 of an MFMA operand (32 rows x 2 chunks) conflict-free.
    unsigned voffA[8], voffB[8];
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {
        if (FP6) {  // slot u * 64 + lane of the wave's 64 x 6 slots: six to a row
            const int slot = u * 64 + lane;
            const int r = slot / 6, piece = fp6_piece(r, slot - 6 * r);
            const int row = 64 * wave + r;
            voffA[u] = (unsigned)fp6_ktile(row, 0, ldA) + (unsigned)(piece * 16);
            voffB[u] = (unsigned)fp6_ktile(row, 0, ldB) + (unsigned)(piece * 16);
        } else {
            const int row = 64 * wave + 8 * u + (lane >> 3);
            const int kc = (lane & 7) ^ ((row >> 1) & 7);
            voffA[u] = (unsigned)i8_at(row, kc * 16, ldA);
            voffB[u] = (unsigned)i8_at(row, kc * 16, ldB);
        }
    }
    const int8_t *gA = g.A + (int64_t)m0 * ldA, *gB = g.B + (int64_t)n0 * ldB;
    if constexpr (BATCH) {
        gA += blockIdx.y * g.a_stride;
        gB += blockIdx.y * g.b_stride;
    }
    // Loads past the end of the range are clamped to the last k-tile: they land in a free slot and
    // are never read, which keeps the count of outstanding loads the same in every iteration.
    // The loads run two k-tiles ahead of the arithmetic and so cross into the next segment earlier: they
    // keep a segment pointer of their own.  Lane i holds the end of segment i, its block offset and the shift
    // behind it, so that moving on to the next segment is two lane reads and no memory access inside the loop.
    int v_end, v_delta, v_shift = 0;
    if constexpr (BATCH) {
        const int r = min(lane, nbound), r1 = min(r + 1, nbound);
        v_end = lane < nbound ? hdr->run_kt0[r1] : kt1;
        v_delta = hdr->run_blk0[r] - hdr->run_kt0[r];
        v_shift = g.sh * (hdr->grp_exp[hdr->run_grp[r]] - hdr->grp_exp[hdr->run_grp[r1]]);
    } else {
        v_end = lane < nbound ? g.bound_kt[lane] + 1 : ktiles;
        v_delta = g.seg_delta[min(lane, nbound)];
    }
    int seg0 = 0;  // the segment of the first k-tile
    if constexpr (SPLIT)
        while (kt0 >= __builtin_amdgcn_readlane(v_end, seg0) && seg0 < nbound) ++seg0;
    int la_seg = seg0, la_end = __builtin_amdgcn_readlane(v_end, seg0), la_delta = __builtin_amdgcn_readlane(v_delta, seg0);
    auto ring = [](int slot, int k) { slot += k; return slot >= kRing ? slot - kRing : slot; };
    const int8_t *pg = nullptr;
    unsigned dl = 0;
    auto half_setup = [&](bool isA, int kt, int slot) {
        const int ktc = min(kt, kt1 - 1);
        int blk = ktc;
        if (isA) {
            // k-tiles are asked for in ascending order, one further per call: at most one segment ends
            la_seg += ktc >= la_end ? 1 : 0;
            la_end = __builtin_amdgcn_readlane(v_end, la_seg);
            la_delta = __builtin_amdgcn_readlane(v_delta, la_seg);
            blk = ktc + la_delta;
        }
        pg = uniform_ptr((isA ? gA : gB) + (FP6 ? fp6_ktile(0, blk, isA ? ldA : ldB) : (int64_t)blk * kRowB));
        dl = __builtin_amdgcn_readfirstlane(lds0 + (unsigned)(slot * kHalfBytes) + (unsigned)(wave * kWaveBytes));
    };
    auto dma_one = [&](bool isA, int u) {  // u = 0..kLoads-1: the u-th KiB of the wave's rows of the half-stage set up last
        dma16(dl + u * 1024, isA ? voffA[u] : voffB[u], pg);
    };

    // ---- LDS -> registers: operand fragments of v_mfma_i32_32x32x32_i8 (lane: row lane%32, 16 K-bytes
    // at chunk 2*ks + lane/32 of the row)
    const int lrow = lane & 31, lhalf = lane >> 5;
    const int swz = (lrow >> 1) & 7;
    const unsigned fa_base = (unsigned)((wm * 128 + lrow) * kPitch);
    const unsigned fb_base = (unsigned)((wn * 128 + lrow) * kPitch);
    unsigned kc_off[4], hi_off[2];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) kc_off[ks] = FP6 ? (unsigned)(16 * fp6_piece(lrow, 3 * ks + lhalf)) : (unsigned)(((2 * ks + lhalf) ^ swz) << 4);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) hi_off[ks] = (unsigned)(16 * fp6_piece(lrow, 3 * ks + 2) + 8 * (lhalf ^ ((lrow >> 4) & 1)));
    using FragT = std::conditional_t<FP6, v8i, v4i>;
    using AccT = std::conditional_t<FP6, v16f, v16i>;
    FragT fa[2][4], fb[2][4];
    if (FP6) {
#pragma unroll
        for (int bq = 0; bq < 8; ++bq)
#pragma unroll
            for (int r = 0; r < (int)(sizeof(FragT) / 4); ++r) {
                fa[bq >> 2][bq & 3][r] = 0;
                fb[bq >> 2][bq & 3][r] = 0;
            }
    }
    // fragment q of a k-step in the order the MFMA sequence below first needs them: a0 b0 b1 a1 b2 b3 a2 a3
    auto load_frag = [&](const int8_t *sta, const int8_t *stb, int ks, int buf, int q) {
        constexpr int isA[8] = {1, 0, 0, 1, 0, 0, 1, 1};
        constexpr int idx[8] = {0, 0, 1, 1, 2, 3, 2, 3};
        const int8_t *src = isA[q] ? sta + fa_base + idx[q] * 32 * kPitch : stb + fb_base + idx[q] * 32 * kPitch;
        FragT &dst = isA[q] ? fa[buf][idx[q]] : fb[buf][idx[q]];
        if constexpr (FP6) {
            const v4i lo = *reinterpret_cast<const v4i *>(src + kc_off[ks]);
            const v2i hi = *reinterpret_cast<const v2i *>(src + hi_off[ks & 1]);
            dst[0] = lo[0]; dst[1] = lo[1]; dst[2] = lo[2]; dst[3] = lo[3];
            dst[4] = hi[0]; dst[5] = hi[1];
        } else {
            dst = *reinterpret_cast<const v4i *>(src + kc_off[ks]);
        }
    };
    auto mma = [&](const FragT &a, const FragT &b, AccT &c) {
        if constexpr (FP6) c = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 2, 2, 0, 0, 0, 0);  // e2m3 x e2m3, no scaling
        else c = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c, 0, 0, 0);
    };

    AccT acc[4][NB];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;
    // DUAL: the contraction goes by pieces of 64 columns, three stages of 24 KiB: with k-tiles of 128 not even two would fit.  A k-tile is two pieces of 64 columns, a stage of LDS holds one: 128 rows of A, 256 of B, 64 bytes each, the four 16-byte
    // chunks of a row swizzled with bits 2 and 3 of the row.  Wave w fills rows [32 w, 32 w + 32) of A and [64 w, 64 w + 64) of B, 16
    // rows (1 KiB, eight whole lines) per load.
    unsigned voffP[6] = {};
    const int8_t *pgA = nullptr, *pgB = nullptr;
    if constexpr (DUAL) {
#pragma unroll
        for (int u = 0; u < 6; ++u) {
            const int row = (u < 2 ? 32 * wave + 16 * u : 64 * wave + 16 * (u - 2)) + (lane >> 2);
            voffP[u] = (unsigned)i8_at(row, ((lane & 3) ^ ((row >> 2) & 3)) * 16, u < 2 ? ldA : ldB);
        }
    }
    // piece kp of the contraction (asked for in ascending order) into stage `stage`
    auto piece_setup = [&](int kp, int stage) {
        const int kpc = min(kp, 2 * kt1 - 1), ktc = kpc >> 1;
        la_seg += ktc >= la_end ? 1 : 0;
        la_end = __builtin_amdgcn_readlane(v_end, la_seg);
        la_delta = __builtin_amdgcn_readlane(v_delta, la_seg);
        pgA = uniform_ptr(gA + (int64_t)(ktc + la_delta) * BK + (kpc & 1) * ldA);
        pgB = uniform_ptr(gB + (int64_t)ktc * BK + (kpc & 1) * ldB);
        dl = __builtin_amdgcn_readfirstlane(lds0 + (unsigned)(stage * kDualStage) + (unsigned)(wave * 2048));
    };
    auto dma_piece = [&](int u) {
        dma16(u < 2 ? dl + u * 1024 : dl + (unsigned)(kDualRows * 64 - 2048 * wave + 4096 * wave) + (u - 2) * 1024, voffP[u], u < 2 ? pgA : pgB);
    };
    // fragment q of a k-step: a0 b0 b1 a1 a2 a3
    auto piece_frag = [&](const int8_t *st, int ks, int buf, int q) {
        constexpr int isA[6] = {1, 0, 0, 1, 1, 1};
        constexpr int idx[6] = {0, 0, 1, 1, 2, 3};
        const int row = idx[q] * 32 + lrow + (isA[q] ? 0 : wn * 64);
        const int8_t *src = st + (isA[q] ? 0 : kDualRows * 64) + row * 64 + (((2 * ks + lhalf) ^ ((lrow >> 2) & 3)) << 4);
        if constexpr (DUAL) (isA[q] ? fa[buf][idx[q]] : fb[buf][idx[q]]) = *reinterpret_cast<const v4i *>(src);
    };
    // eight matrix instructions on the fragments in buffer `cur`, the next k-step's fragments and (if any) six loads on the way
    auto piece_step = [&](int cur, const int8_t *next, int next_ks, bool load) {
        if constexpr (DUAL)
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                if (q < 6) piece_frag(next, next_ks, cur ^ 1, q);
                mma(fa[cur][q >> 1], fb[cur][q & 1], acc[q >> 1][q & 1]);
                if (load && q < 6) dma_piece(q);
                __builtin_amdgcn_sched_barrier(0);
            }
    };
    // MFMA order: 2 x 2 sub-blocks, so that the fragments of the next k-step can trickle in
    constexpr int mi[16] = {0, 0, 1, 1, 0, 0, 1, 1, 2, 2, 3, 3, 2, 2, 3, 3};
    constexpr int mj[16] = {0, 1, 0, 1, 2, 3, 2, 3, 0, 1, 0, 1, 2, 3, 2, 3};

    // One step = 16 MFMAs on the fragments in buffer `cur`, interleaved with the 8 fragment loads of
    // the next k-step into the other buffer and with `ndma` direct-to-LDS loads (starting at block
    // `dma0`) of the half-stage set up last.
    auto step = [&](int cur, const int8_t *sta, const int8_t *stb, int next_ks, bool isA, int dma0, int ndma) {
        if constexpr (!DUAL)
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            load_frag(sta, stb, next_ks, cur ^ 1, q);
            mma(fa[cur][mi[2 * q]], fb[cur][mj[2 * q]], acc[mi[2 * q]][mj[2 * q]]);
            if (q < ndma) dma_one(isA, dma0 + q);
            mma(fa[cur][mi[2 * q + 1]], fb[cur][mj[2 * q + 1]], acc[mi[2 * q + 1]][mj[2 * q + 1]]);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    unsigned long long probe_c = 0, probe_w = 0;
    const bool probing = MODE == 0 && g.clock_probe != nullptr && blockIdx.x == 0;
    if (probing) {
        probe_c = __builtin_readcyclecounter();
        probe_w = wall_clock64();
    }
    // ---- prologue: k-tile kt0 landed, k-tile kt0+1 in flight, first fragments loaded
    int sa = 0;  // ring slot of A(kt); B(kt) is sa+1, A(kt+1) sa+2, B(kt+1) sa+3, A(kt+2) sa+4, B(kt+2) sa
    if constexpr (DUAL) {
#pragma unroll
        for (int p = 0; p < kDualStages; ++p) {
            piece_setup(2 * kt0 + p, p);
#pragma unroll
            for (int u = 0; u < 6; ++u) dma_piece(u);
        }
    } else {
        half_setup(true, kt0, 0);
#pragma unroll
        for (int u = 0; u < kLoads; ++u) dma_one(true, u);
        half_setup(false, kt0, 1);
#pragma unroll
        for (int u = 0; u < kLoads; ++u) dma_one(false, u);
        half_setup(true, kt0 + 1, 2);
#pragma unroll
        for (int u = 0; u < kLoads; ++u) dma_one(true, u);
        half_setup(false, kt0 + 1, 3);
#pragma unroll
        for (int u = 0; u < kLoads; ++u) dma_one(false, u);
    }
    // What the epilogue needs to know of the tile, a word per lane (it is read once the sums stand; by then it has long
    // arrived): 0 .. 4 first source row of each chunk, 8 .. 11 their levels, 16 / 17 first source column of the tile and of
    // the next, 18 / 19 whether no row / no column is split, 20 / 21 the steps.
    int tile_meta = 0;
    if constexpr (MODE == 0) {
        constexpr int per = kChunks;
        const int32_t *from = lane < 8    ? g.layA.chunk_src0 + tm * per + min(lane, per)
                              : lane < 16 ? g.layA.chunk_lev + tm * per + min(lane - 8, per - 1)
                              : lane < 18 ? g.layB.tile_src0 + tn + (lane - 16)
                              : lane < 19 ? g.layA.tile_flat + tm * per / (kTile / kChunk)
                                          : g.layB.tile_flat + tn;
        if constexpr (BATCH) from = item_at(from, blockIdx.y * g.plan_stride);
        if (g.scale_a_dev && lane >= 20) {
            from = reinterpret_cast<const int32_t *>(lane == 20 ? g.scale_a_dev : g.scale_b_dev);
            if constexpr (BATCH) from = item_at(from, blockIdx.y * g.scale_stride);
        }
        tile_meta = *from;
    }
    auto meta = [&](int i) __attribute__((always_inline)) {  // (read where it is needed, not kept: scalar registers are scarce)
        asm volatile("" : "+s"(i));
        return __builtin_amdgcn_readlane(tile_meta, i);
    };
    if (DUAL && inexact()) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // nothing may land in LDS behind the workgroup's end
        return;
    }
    if (DUAL) asm volatile("s_waitcnt vmcnt(13)" ::: "memory");
    else if (MODE == 0 && FP6) asm volatile("s_waitcnt vmcnt(13)" ::: "memory");
    else if (MODE == 0) asm volatile("s_waitcnt vmcnt(17)" ::: "memory");
    else if (FP6) asm volatile("s_waitcnt vmcnt(12)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if constexpr (DUAL) {
#pragma unroll
        for (int q = 0; q < 6; ++q) piece_frag(smem, 0, 0, q);
    } else {
#pragma unroll
        for (int q = 0; q < 8; ++q) load_frag(smem, smem + kHalfBytes, 0, 0, q);
    }

    // ---- main loop, one 128-byte k-tile (4 k-steps, 64 MFMAs) and one barrier per iteration.
    // Steps 1-3 stream A(kt+2) into the spare slot.  After step 3 every fragment of k-tile kt has been
    // read (lgkmcnt(0)) and this wave's parts of A(kt+1), B(kt+1) have landed (all but the 8 newest
    // loads); past the barrier that holds for all waves, so step 4 may prefetch fragments of k-tile
    // kt+1 and stream B(kt+2) into the slot of A(kt).
    int kt = kt0;
    int seg = seg0;
    // The columns that are taken from lists: the wave's four blocks of 32 physical rows of B in turn, 128 entries at a time, through what
    // the wave itself will fill of the slot of the ring that is free now (the waves are at different places here).  In half tiles two
    // blocks, 64 entries at a time, through 2 KiB that the wave has for this alone: no stage is free.
    auto lists = [&]() __attribute__((always_inline)) {
        const int8_t *at = uniform_ptr(g.at + (int64_t)(tm * (BM / 128) + wm) * g.at_cols * 128);
        const unsigned row_off = (unsigned)lrow * 4u;
        const int block0 = (n0 + wn * 32 * NB) / kSparseRows;
        constexpr int S = DUAL ? 2 : 4;  // matrix instructions at a time
        int8_t *lds = DUAL ? smem + kDualStages * kDualStage + wave * kDualSpare : smem + ring(sa, 4) * kHalfBytes + wave * kWaveBytes;
        static_assert(list_lds(S) <= kWaveBytes && list_lds(S) <= kDualSpare, "LDS of the lists");
        const int lens = min(g.sparse.cnt[block0 + min(lane, NB - 1)], g.sparse.cap);  // lane 0 .. 3: how long the lists of the wave's blocks are
        int list = block0 * g.sparse.cap;  // (no more than kSparsePlaces)
        ListWords<S> words;  // the next 32 S entries, or the first of the list behind
        words.load(g.sparse.ent + list, lane);
        auto block = [&](auto cb_c) __attribute__((always_inline)) {
            constexpr int CB = decltype(cb_c)::value;
            const int len = __builtin_amdgcn_readlane(lens, CB);
            const int next = list + g.sparse.cap;
            if (len <= 0) words.load(g.sparse.ent + next, lane);  // (there are none of this list)
            for (int t = 0; t < len; t += 32 * S) {
                v4i digits[S];
                words.stage(lds, len - t, lane, digits);
                unsigned x[S][16];
#pragma unroll
                for (int s = 0; s < S; ++s) list_columns(x[s], lds + 1024, s, lhalf, at, row_off);
                words.load(g.sparse.ent + (t + 32 * S < len ? list + t + 32 * S : next), lane);
#pragma unroll
                for (int s = 0; s < S; ++s) {
                    if (t + 32 * s >= len) break;  // uniform
                    v4i fr[4];
                    list_rows(x[s], fr);
#pragma unroll
                    for (int rb = 0; rb < 4; ++rb)
                        if constexpr (LISTS && DUAL) mma(fr[rb], digits[s], acc[rb][CB]);
                        else if constexpr (LISTS) mfma_in_place(fr[rb], digits[s], acc[rb][CB]);
                    if constexpr (DUAL) __builtin_amdgcn_sched_barrier(0);  // (the next one's rows are put together behind: 4096 x 4352 by 11013 0.7 % of a step)
                }
            }
            list = next;
        };
        block(std::integral_constant<int, 0>{});
        block(std::integral_constant<int, 1>{});
        if constexpr (!DUAL) {
            block(std::integral_constant<int, 2>{});
            block(std::integral_constant<int, 3>{});
            // What comes behind does not know of these matrix instructions: it takes the sums from here, once they stand.
            asm volatile("s_nop 15\n\ts_nop 3"
                         : "+a"(acc[0][0]), "+a"(acc[0][1]), "+a"(acc[0][NB - 2]), "+a"(acc[0][NB - 1]), "+a"(acc[1][0]), "+a"(acc[1][1]),
                           "+a"(acc[1][NB - 2]), "+a"(acc[1][NB - 1]), "+a"(acc[2][0]), "+a"(acc[2][1]), "+a"(acc[2][NB - 2]),
                           "+a"(acc[2][NB - 1]), "+a"(acc[3][0]), "+a"(acc[3][1]), "+a"(acc[3][NB - 2]), "+a"(acc[3][NB - 1]));
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the slot has been read: it may be filled
    };
    // Horner step
    auto horner = [&](const int shv) __attribute__((always_inline)) {
        // The accumulators fill the whole accumulation register file (a0..a255), so shifting every
        // one of those registers shifts every accumulator, whichever block sits where.  Written
        // out by hand: left to the compiler, this step spills three blocks to scratch memory.
        int t0, t1, t2, t3;
        if constexpr (DUAL) {  // the accumulators are ordinary registers
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < NB; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[i][j][r] = (int)((unsigned)acc[i][j][r] << shv);
        } else if constexpr (FP6) {  // binary32 accumulators: times 2^shift, exact
            asm volatile(
                "s_nop 15\n\ts_nop 7\n\t"
                ".irp n," IMU_ACC_QUADS "\n\t"
                "v_accvgpr_read_b32 %[t0], a[\\n]\n\t"
                "v_accvgpr_read_b32 %[t1], a[\\n+1]\n\t"
                "v_accvgpr_read_b32 %[t2], a[\\n+2]\n\t"
                "v_accvgpr_read_b32 %[t3], a[\\n+3]\n\t"
                "v_ldexp_f32 %[t0], %[t0], %[sh]\n\t"
                "v_ldexp_f32 %[t1], %[t1], %[sh]\n\t"
                "v_ldexp_f32 %[t2], %[t2], %[sh]\n\t"
                "v_ldexp_f32 %[t3], %[t3], %[sh]\n\t"
                "v_accvgpr_write_b32 a[\\n], %[t0]\n\t"
                "v_accvgpr_write_b32 a[\\n+1], %[t1]\n\t"
                "v_accvgpr_write_b32 a[\\n+2], %[t2]\n\t"
                "v_accvgpr_write_b32 a[\\n+3], %[t3]\n\t"
                ".endr\n\t"
                "s_nop 7"
                : [t0] "=&v"(t0), [t1] "=&v"(t1), [t2] "=&v"(t2), [t3] "=&v"(t3), "+a"(acc[0][0]), "+a"(acc[0][1]),
                  "+a"(acc[0][NB - 2]), "+a"(acc[0][NB - 1]), "+a"(acc[1][0]), "+a"(acc[1][1]), "+a"(acc[1][NB - 2]),
                  "+a"(acc[1][NB - 1]), "+a"(acc[2][0]), "+a"(acc[2][1]), "+a"(acc[2][NB - 2]), "+a"(acc[2][NB - 1]),
                  "+a"(acc[3][0]), "+a"(acc[3][1]), "+a"(acc[3][NB - 2]), "+a"(acc[3][NB - 1])
                : [sh] "s"(shv));
        } else
        asm volatile(
            "s_nop 15\n\ts_nop 7\n\t"  // the last MFMA results must have landed
            ".irp n," IMU_ACC_QUADS "\n\t"
            "v_accvgpr_read_b32 %[t0], a[\\n]\n\t"
            "v_accvgpr_read_b32 %[t1], a[\\n+1]\n\t"
            "v_accvgpr_read_b32 %[t2], a[\\n+2]\n\t"
            "v_accvgpr_read_b32 %[t3], a[\\n+3]\n\t"
            "v_lshlrev_b32 %[t0], %[sh], %[t0]\n\t"
            "v_lshlrev_b32 %[t1], %[sh], %[t1]\n\t"
            "v_lshlrev_b32 %[t2], %[sh], %[t2]\n\t"
            "v_lshlrev_b32 %[t3], %[sh], %[t3]\n\t"
            "v_accvgpr_write_b32 a[\\n], %[t0]\n\t"
            "v_accvgpr_write_b32 a[\\n+1], %[t1]\n\t"
            "v_accvgpr_write_b32 a[\\n+2], %[t2]\n\t"
            "v_accvgpr_write_b32 a[\\n+3], %[t3]\n\t"
            ".endr\n\t"
            "s_nop 7"
            : [t0] "=&v"(t0), [t1] "=&v"(t1), [t2] "=&v"(t2), [t3] "=&v"(t3), "+a"(acc[0][0]), "+a"(acc[0][1]),
              "+a"(acc[0][NB - 2]), "+a"(acc[0][NB - 1]), "+a"(acc[1][0]), "+a"(acc[1][1]), "+a"(acc[1][NB - 2]),
              "+a"(acc[1][NB - 1]), "+a"(acc[2][0]), "+a"(acc[2][1]), "+a"(acc[2][NB - 2]), "+a"(acc[2][NB - 1]),
              "+a"(acc[3][0]), "+a"(acc[3][1]), "+a"(acc[3][NB - 2]), "+a"(acc[3][NB - 1])
            : [sh] "s"(shv));
    };
    for (; seg <= nbound && (!SPLIT || kt < kt1); ++seg) {
        int shv = seg == seg0 ? 0 : BATCH ? __builtin_amdgcn_readlane(v_shift, seg - 1) : g.bound_sh[seg - 1];
        if (LISTS && seg != seg0 && kt == g.sp_kt) shv -= g.sp_after;  // (that much of it comes behind the lists)
        if (shv != 0) horner(shv);  // start of the next exponent group
        if constexpr (LISTS)
            if (kt == g.sp_kt) {  // (the first k-tile of a segment)
                lists();
                if (g.sp_after != 0) horner(g.sp_after);
            }
        int kend = BATCH ? __builtin_amdgcn_readlane(v_end, seg) : seg < nbound ? g.bound_kt[seg] + 1 : kt1;
        if constexpr (SPLIT) kend = min(kend, kt1);
        if constexpr (DUAL)
            for (; kt < kend; ++kt)
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    const int8_t *st = smem + sa * kDualStage;
                    piece_step(0, st, 1, false);
                    // the piece has been read, and this wave's parts of the next one have landed (all but the 6 newest loads): past the
                    // barrier that holds for all waves
                    asm volatile("s_waitcnt vmcnt(6) lgkmcnt(0)" ::: "memory");
                    __builtin_amdgcn_s_barrier();
                    asm volatile("" ::: "memory");
                    piece_setup(2 * kt + half + kDualStages, sa);
                    sa = sa + 1 == kDualStages ? 0 : sa + 1;
                    __builtin_amdgcn_sched_barrier(0);
                    piece_step(1, smem + sa * kDualStage, 0, true);
                }
        else
        for (; kt < kend; ++kt) {
            const int8_t *stA = smem + sa * kHalfBytes, *stB = smem + ring(sa, 1) * kHalfBytes;
            const int8_t *stA1 = smem + ring(sa, 2) * kHalfBytes, *stB1 = smem + ring(sa, 3) * kHalfBytes;
            half_setup(true, kt + 2, ring(sa, 4));
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (FP6) {  // two k-steps of 64 columns: the first streams A(kt+2), the second B(kt+2)
                step(0, stA, stB, 1, true, 0, kLoads);
                asm volatile("s_waitcnt vmcnt(6) lgkmcnt(0)" ::: "memory");
            } else {
                step(0, stA, stB, 1, true, 0, 3);
                step(1, stA, stB, 2, true, 3, 3);
                step(0, stA, stB, 3, true, 6, 2);
                asm volatile("s_waitcnt vmcnt(8) lgkmcnt(0)" ::: "memory");
            }
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            half_setup(false, kt + 2, sa);
            __builtin_amdgcn_sched_barrier(0);
            step(1, stA1, stB1, 0, false, 0, kLoads);
            sa = ring(sa, 2);
        }
    }
    if (probing && tid == 0) {
        g.clock_probe[0] = __builtin_readcyclecounter() - probe_c;
        g.clock_probe[1] = wall_clock64() - probe_w;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // drain the clamped tail loads before LDS is reused
    __syncthreads();  // all fragment reads done: the buffers may be reused by the epilogue

    // A part of a tile.  All but the last to arrive leave their sums and are done; the last adds them to its own and goes on to
    // the epilogue (it may have to wait for the end of their stores, from workgroups that are running: never for one that has
    // yet to start).  The accumulators count in units of the segment they ended in: `rest` brings a part that ends before
    // the last group to the units of that group.
    int rest = 0, partners = 0;
    const int32_t *partner = nullptr;
    if constexpr (SPLIT) {
        if (pc.parts > 1) {
            for (int x = seg - 1; x < nbound; ++x) rest += g.bound_sh[x];
            int32_t *meet = g.meet + 2 * pc.slot, *sums = g.sums + (size_t)pc.slot * (BM * BN) + 4 * tid;
            int32_t *turn = reinterpret_cast<int32_t *>(smem);
            if (tid == 0) *turn = __hip_atomic_fetch_add(meet, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            const int came = __builtin_amdgcn_readfirstlane(*turn);
            if (came < pc.parts - 1) {
                sums += (size_t)came * (BM * BN);
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        int32_t *q = sums + ((i * 4 + j) * 16) * kGemmThreads;
#pragma unroll
                        for (int r = 0; r < 16; r += 4, q += 4 * kGemmThreads) {
                            const v4i x = {(int32_t)acc[i][j][r] << rest, (int32_t)acc[i][j][r + 1] << rest, (int32_t)acc[i][j][r + 2] << rest,
                                           (int32_t)acc[i][j][r + 3] << rest};
                            // through to where every XCD reads it (and no overwriting of x in the next cycles: the compiler does not
                            // know that this is a store of four words)
                            asm volatile("global_store_dwordx4 %0, %1, off sc0 sc1\n\ts_nop 3" : : "v"(q), "v"(x) : "memory");
                        }
                    }
                stores_done();
                __syncthreads();
                if (tid == 0) __hip_atomic_fetch_add(meet + 1, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                return;
            }
            if (tid == 0) {
                while (__hip_atomic_load(meet + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < pc.parts - 1) __builtin_amdgcn_s_sleep(2);
                __hip_atomic_store(meet + 1, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // for the next launch
                __hip_atomic_store(meet, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            __syncthreads();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");  // the sums as their workgroups left them, whichever XCD those ran on
            partner = sums;
            partners = pc.parts - 1;
        }
    }

    if constexpr (MODE == 1) {
        // un-fused: the int32 partial product of this exponent group goes, shifted, into the int64
        // unpacked product C_u (physical coordinates, padded to tiles: no bounds to check)
        constexpr int FLD1 = 260;
        int32_t *buf = reinterpret_cast<int32_t *>(smem);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            __syncthreads();
            if (wm == (c >> 1)) {
#pragma unroll
                for (int ii = 0; ii < 2; ++ii)
#pragma unroll
                    for (int jj = 0; jj < 4; ++jj)
#pragma unroll
                        for (int r = 0; r < 16; ++r)
                            buf[(ii * 32 + 8 * (r >> 2) + 4 * lhalf + (r & 3)) * FLD1 + wn * 128 + jj * 32 + lrow] =
                                (int32_t)acc[(c & 1) * 2 + ii][jj][r];
            }
            __syncthreads();
            const int col4 = (tid & 63) * 4;
            for (int it = 0; it < 16; ++it) {
                const int row = (tid >> 6) + 4 * it;
                const v4i v = *reinterpret_cast<const v4i *>(buf + row * FLD1 + col4);
                int64_t *dst = g.C_u + (int64_t)(m0 + c * 64 + row) * g.Np + n0 + col4;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int64_t x = (int64_t)v[k] << g.seg_shift;
                    dst[k] = g.seg_first ? x : dst[k] + x;
                }
            }
        }
        return;
    }

    // ---- fused epilogue: C_int[i,j] = sum_{levels a of i, c of j} s^(a+c) * acc[row(i,a)][col(j,c)].  Two ways out:
    // (1) From the registers, chunk by chunk of 64 physical rows, for fp32 results where the source rows of the chunk have one,
    //     two or four levels each and the source columns too (or are split here and there: those go through strips in LDS).  A
    //     lane holds whole source rows and columns then (see rows_layout), so it folds and stores by itself, without
    //     LDS and barriers.  One wave per SIMD leaves nothing to hide latency behind, so this is bound by its instructions and
    //     by the stores of all CUs at once: 64 results a lane in some 4000 cycles (9200 through LDS with every
    //     row decided by itself); 25344 x 768 by 3072 rows 124 -> 107 us, 16384 x 3072 (six-bit) by 4096 512 -> 442 (of
    //     which three tile rows that even rows save), 8192 x 8448 by 4096 266 -> 213.
    //     Without levels to fold the stores are ordinary ones: 256 KiB a CU at once as non-temporal lines of 128 bytes take 45 000
    //     cycles instead of 34 000 (4096 x 8228 by 11013, one run: 344 and 317 us).  With levels there is a half of that or less, and
    //     the non-temporal ones leave the last-level cache to the operands: a step of 12608 x 768 by 3072 226 and 233 us.
    //     The price is code: nine pairs of levels times four blocks of rows, straight down, make this kernel 170 kB (50 with the
    //     ways through LDS alone) and spill 10 vector registers (17 six-bit, 17 and 16 in parts, 32 in parts beside lists, 10 and 26 in a batch; none in half tiles),
    //     all of them behind the walk along the contraction.
    // (2) Through LDS ([64][256] int32, rows padded to 260) for everything else: int64 results, rows of several kinds in a chunk,
    //     many split columns, results without levels of large products (whole_rows_win).  Global stores are row-contiguous, any
    //     levels can be added up (the planner keeps a source row in one chunk, a source column in one tile).
    RowLayout layA = g.layA, layB = g.layB;
    float *C_fp = g.C_fp;
    int final_shift = g.final_shift, fold_f64 = g.fold_f64, evenB = g.evenB;
    if constexpr (BATCH) {
        evenB = hdr->evenB;
        move_to_item(layA, blockIdx.y * g.plan_stride);
        move_to_item(layB, blockIdx.y * g.plan_stride);
        C_fp = item_at(C_fp, blockIdx.y * g.c_stride);
        final_shift = hdr->ngroups ? g.sh * hdr->grp_exp[hdr->ngroups - 1] : 0;
        fold_f64 = 31 + g.sh * ((hdr->lmaxA - 1) + (hdr->lmaxB - 1)) <= 52;
    }
    const int jsrc0 = meta(16), nsrcB = meta(17) - jsrc0;
    const bool flatA = meta(18) != 0, flatB = meta(19) != 0;
    const int stepB = evenB ? kEvenStep : 1;  // from level to level of a source column
    constexpr int FLD = 260;
    constexpr int kRegions = DUAL ? 1 : 2;
    int32_t *foldbuf = reinterpret_cast<int32_t *>(smem);  // kRegions of [64][FLD]
    // behind the staging buffer: per source row of the tile its first physical row (relative to the
    // tile) | levels << 16; the same per source column; the first source row of each chunk
    int32_t *rowmeta = foldbuf + kRegions * kChunk * FLD, *colmeta = rowmeta + kTile, *chunk0 = colmeta + kTile;
    // ... and the sums of split columns, a strip of the tile's physical rows for each
    constexpr int kStrips = 20, kStripPitch = BM + 4;
    int32_t *strips = chunk0 + 8;
    static_assert((kRegions * kChunk * FLD + 2 * kTile + 8 + kStrips * kStripPitch) * sizeof(int32_t) <= (DUAL ? kDualLds : kGemmLds), "LDS of the epilogue");
    // scale * 2^final_shift is exact: one multiplication in binary64, one rounding to fp32
    const double scale2 = (g.scale_a_dev ? (double)__int_as_float(meta(20)) * (double)__int_as_float(meta(21)) : g.scale) *
                          (double)(1ull << final_shift);
    // The short way out of a chunk whose source rows have one, two or four levels each: a lane holds four physical rows side
    // by side of a column, that is whole source rows, and stores their results itself.
    int direct = 0, filled = 0;  // a bit per chunk: stored from the registers (or nothing to store); holds source rows
    const bool fits = C_fp && !g.C_int && g.ldc < kDirectPitch;  // fp32 alone, and a chunk of C spans no more than 2^30 bytes
    // the split ones among the tile's 256 physical columns, and the first of each source column
    auto find_split = [&](unsigned long long (&split)[4], unsigned long long (&heads)[4]) __attribute__((always_inline)) {
        int prow[4], next[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            prow[t] = layB.prow[n0 + 64 * t + lane];
            next[t] = 64 * t + lane < BN - 1 ? layB.prow[n0 + 64 * t + lane + 1] : -1;
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const bool more = next[t] >= 0 && (next[t] >> kProwLevel) > 0, first = prow[t] >= 0 && (prow[t] >> kProwLevel) == 0;
            heads[t] = __ballot(first && more);
            split[t] = __ballot(prow[t] >= 0 && (!first || more));
        }
    };
    int nsplit = 0;
    unsigned col_off[NB];  // where the lane's columns go in a row of C
    int col_strip[NB];
#pragma unroll
    for (int t = 0; t < NB; ++t) {
        col_off[t] = kOutside;
        col_strip[t] = -1;
    }
    {
        if (fits && evenB) {  // the first level of each of the lane's columns
#pragma unroll
            for (int t = 0; t < NB; ++t) {
                const int col = evenB == 2 ? wn * (16 * NB) + (t >> 1) * 32 + lrow : wn * (8 * NB) + lrow;
                if (col < nsrcB) col_off[t] = 4u * (unsigned)col;
            }
        } else if (fits && !flatB) {
            int own[NB];
            unsigned long long split_cols[4], heads[4];
#pragma unroll
            for (int t = 0; t < NB; ++t) own[t] = layB.prow[n0 + wn * (32 * NB) + 32 * t + lrow];
            find_split(split_cols, heads);
            nsplit = __popcll(split_cols[0]) + __popcll(split_cols[1]) + __popcll(split_cols[2]) + __popcll(split_cols[3]);
            // the wave's column 32 t + lrow is bit (32 t + lrow) & 63 of word wn NB / 2 + t / 2
            unsigned long long mine[NB / 2];
            int before = 0;
            if constexpr (DUAL) {
                mine[0] = wn < 2 ? (wn ? split_cols[1] : split_cols[0]) : wn == 2 ? split_cols[2] : split_cols[3];
#pragma unroll
                for (int t = 0; t < 3; ++t) before += t < wn ? __popcll(split_cols[t]) : 0;
            } else {
                mine[0] = wn ? split_cols[2] : split_cols[0];
                mine[NB / 2 - 1] = wn ? split_cols[3] : split_cols[1];
                before = wn ? __popcll(split_cols[0]) + __popcll(split_cols[1]) : 0;
            }
#pragma unroll
            for (int t = 0; t < NB; ++t) {
                const unsigned long long m = mine[t >> 1];
                const int bit = (t & 1) * 32 + lrow;
                if ((m >> bit) & 1) col_strip[t] = before + (t >> 1 ? __popcll(mine[0]) : 0) + __popcll(m & ((1ull << bit) - 1ull));
                else if (own[t] >= 0) col_off[t] = 4u * (unsigned)((own[t] & ((1 << kProwLevel) - 1)) - jsrc0);
            }
        } else if (fits) {
#pragma unroll
            for (int t = 0; t < NB; ++t) {
                const int col = wn * (32 * NB) + 32 * t + lrow;
                if (col < nsrcB) col_off[t] = 4u * (unsigned)col;
            }
        }
#pragma unroll
        for (int c = 0; c < kChunks; ++c) {
            const bool rows = meta(c + 1) > meta(c);  // (a chunk of nothing but padding stores nothing, and no resource is made for it)
            const int lev = fits && rows ? meta(8 + c) : 0;
            // (with nothing to fold, one by one only where the stores may stay in the caches)
            const bool plain = lev == 1 && !evenB;
            const bool ok = (plain ? !g.whole_rows || nsplit > 0 : fold_f64 && (lev == 1 || lev == 2 || lev == 4) && evenB <= NB) && nsplit <= kStrips;
            direct |= (!rows || ok) << c;
            filled |= rows << c;
        }
    }
    const bool any_direct = (direct & filled) != 0, any_lds = direct != (1 << kChunks) - 1;
    if (any_lds) {
        const int isrc0 = meta(0), nsrcA = meta(kChunks) - isrc0;
        if (!flatA && tid < nsrcA)
            rowmeta[tid] = (layA.src_pstart[isrc0 + tid] - m0) | (layA.src_nlev[isrc0 + tid] << 16);
        if (!flatB && tid < nsrcB)
            colmeta[tid] = (layB.src_pstart[jsrc0 + tid] - n0) | (layB.src_nlev[jsrc0 + tid] << 16);
        if (tid <= kChunks) chunk0[tid] = tile_meta;
    }  // published by the first barrier below
    // `ns` rows of C from source row c0 on, the tile's columns.  Rows behind them begin behind the end (ldc >= nsrcB).
    auto rows_of_c = [&](int c0, int ns) __attribute__((always_inline)) {
        float *to = C_fp + (int64_t)c0 * g.ldc + jsrc0;
        return __builtin_amdgcn_make_buffer_rsrc(to, 0, (int)(((unsigned)(ns - 1) * (unsigned)g.ldc + (unsigned)nsrcB) * 4u), 0x00027000);
    };
    // The sums of 32 physical rows (I: which of the wave's four blocks of them) to where they belong.  L: physical rows of a
    // source row, M: physical columns of a source column.
    auto put = [&](auto lev_c, auto cols_c, auto block_c, auto value) __attribute__((always_inline)) {
        constexpr int L = decltype(lev_c)::value, M = decltype(cols_c)::value, G = 4 / L;  // G source rows among four physical ones
        constexpr int half = decltype(block_c)::value >> 1, ii = decltype(block_c)::value & 1;
        const int c0 = meta(2 * wm + half), ns = meta(2 * wm + half + 1) - c0;
        const unsigned pitch = (unsigned)g.ldc * 4u;
        const __amdgpu_buffer_rsrc_t rs = rows_of_c(c0, ns);
        unsigned off[NB];
#pragma unroll
        for (int j = 0; j < NB; j += M) off[j] = col_off[j] + (unsigned)(lhalf * G) * pitch;
        double w[L + M];
#pragma unroll
        for (int l = 0; l < L + M; ++l) w[l] = (double)(1ull << (g.sh * l));
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) {
            float f[G][NB];
#pragma unroll
            for (int k = 0; k < G; ++k)
#pragma unroll
                for (int j = 0; j < NB; j += M) {
                    double v = 0.0;
#pragma unroll
                    for (int m = 0; m < M; ++m) {
                        int x[L];
#pragma unroll
                        for (int l = 0; l < L; ++l) x[l] = value(j + m, 4 * rg + k * L + l);
#pragma unroll
                        for (int l = 0; l < L; l += FP6 ? 2 : 1) {
                            // (sums of six-bit digits stay below 2^24 and the weights at 8: two levels fit 32 bits)
                            const double t = exact_f64(FP6 && L > 1 ? x[l] + (x[(l + 1) % L] << g.sh) : x[l]);
                            if (m + l == 0) v = t;
                            else v += t * w[m + l];
                        }
                    }
                    f[k][j] = (float)(v * scale2);
                }
#pragma unroll
            for (int k = 0; k < G; ++k)
#pragma unroll
                for (int j = 0; j < NB; j += M)
                    store_inside<(L * M > 1)>(f[k][j], rs, off[j] + (unsigned)((ii * 32 + 8 * rg) / L + k) * pitch);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // 64 sums of a lane's partners at a time: the loads have to be many to be fast, 256 KiB a partner
    auto others = [&](int block, v4i (&other)[16]) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < 16; ++t) other[t] = v4i{0, 0, 0, 0};
        const int32_t *q = partner + block * 4 * 16 * kGemmThreads;
#pragma unroll 1
        for (int w = 0; w < partners; ++w, q += BM * BN) {
            v4i x[16];
#pragma unroll
            for (int t = 0; t < 16; ++t) x[t] = __builtin_nontemporal_load(reinterpret_cast<const v4i *>(q + t * 4 * kGemmThreads));
#pragma unroll
            for (int t = 0; t < 16; ++t) other[t] += x[t];
        }
    };
    auto store_block = [&](auto block_c) __attribute__((always_inline)) {
        constexpr int I = decltype(block_c)::value, half = I >> 1;
        if (!((direct & filled) >> (2 * wm + half) & 1)) return;
        const int my_lev = meta(8 + 2 * wm + half);
        v4i other[16];
        if (SPLIT && partner) others(I, other);
        // (read by hand, so that the compiler does not convert sixty-four sums ahead of the choice between the three)
        auto sum = [&](int jj, int r) __attribute__((always_inline)) {
            int32_t v;
            if constexpr (FP6) {
                float x;
                asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(x) : "a"(acc[I][jj][r]));
                v = (int32_t)x;
            } else if constexpr (DUAL) {
                asm volatile("v_mov_b32 %0, %1" : "=v"(v) : "v"(acc[I][jj][r]));
            } else {
                asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v) : "a"(acc[I][jj][r]));
            }
            if (SPLIT && partner) v = (v << rest) + other[jj * 4 + (r >> 2)][r & 3];
            return v;
        };
        auto with_cols = [&](auto cols_c) __attribute__((always_inline)) {
            if (my_lev == 1) put(std::integral_constant<int, 1>{}, cols_c, block_c, sum);
            else if (my_lev == 2) put(std::integral_constant<int, 2>{}, cols_c, block_c, sum);
            else if (my_lev == 4) put(std::integral_constant<int, 4>{}, cols_c, block_c, sum);
        };
        if (evenB == 0) with_cols(std::integral_constant<int, 1>{});
        else if (evenB == 2) with_cols(std::integral_constant<int, 2>{});
        else if constexpr (NB == 4) with_cols(std::integral_constant<int, 4>{});
#pragma unroll
        for (int jj = 0; jj < NB; ++jj)
            if (col_strip[jj] >= 0)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    strips[col_strip[jj] * kStripPitch + wm * 128 + I * 32 + 8 * (r >> 2) + 4 * lhalf + (r & 3)] = sum(jj, r);
    };
    if (any_direct) {
        asm volatile("s_nop 15\n\ts_nop 15");  // the last matrix instructions have landed (the compiler does not see the reads)
        store_block(std::integral_constant<int, 0>{});
        store_block(std::integral_constant<int, 1>{});
        store_block(std::integral_constant<int, 2>{});
        store_block(std::integral_constant<int, 3>{});
    }
    // two chunks per round: every wave parks 64 of its 128 rows (region wm of the staging buffer), then all threads work the
    // two chunks off
    if (any_lds)
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        __syncthreads();
#pragma unroll
        for (int ii = 0; ii < 2; ++ii) {
            v4i other[16];
            if (SPLIT && partner) others(half * 2 + ii, other);
#pragma unroll
            for (int jj = 0; jj < NB; ++jj)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    int32_t v = (int32_t)acc[half * 2 + ii][jj][r];
                    if (SPLIT && partner) v = (v << rest) + other[jj * 4 + (r >> 2)][r & 3];
                    foldbuf[(wm * kChunk + ii * 32 + 8 * (r >> 2) + 4 * lhalf + (r & 3)) * FLD + wn * (32 * NB) + jj * 32 + lrow] = v;
                }
        }
        __syncthreads();
#pragma unroll 1
        for (int reg = 0; reg < kRegions; ++reg) {
            const int c = 2 * reg + half;  // chunk of the tile: rows [64 c, 64 c + 64)
            if (direct >> c & 1) continue;
            const int32_t *fold = foldbuf + reg * kChunk * FLD;
            // source rows of this chunk: cs0 .. cs0 + ns - 1; no source row straddles a chunk
            const int cs0 = chunk0[c], ns = chunk0[c + 1] - cs0;
            const int rs0 = cs0 - chunk0[0];  // index of the chunk's first source row in rowmeta
            // A lane owns four source columns side by side, a wave works on four source rows together so that their LDS reads
            // are in flight side by side; what a row needs is uniform in the wave, the levels of the columns are masked weights.
            // (Every row and column looked at by itself: 9600 cycles a chunk, 30 000 where several columns were split.  A column
            // to a lane and every row to every wave: 20 000.)
            auto fold_chunk = [&](auto zero, auto flat_c) __attribute__((always_inline)) {
                using T = decltype(zero);
                constexpr bool F = decltype(flat_c)::value;  // source columns = physical columns
                constexpr int U = 4, RS = kGemmThreads / 64;
                static_assert((U - 1) * RS <= kRowsAhead, "rows asked for behind a chunk");
                const int j4 = lane * 4, left = nsrcB - j4;
                // fp32 alone and no quad that ends inside: one store a row, what is outside dropped by the hardware
                const bool quads = fits && (nsrcB & 3) == 0;
                const unsigned quad_off = left > 0 ? 4u * (unsigned)j4 : kOutside;
                const __amdgpu_buffer_rsrc_t rs = rows_of_c(cs0, max(ns, 1));
                int q[4], lj[4], ljmax = 1;
                if constexpr (!F) {
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const int cm = j4 + k < nsrcB ? colmeta[j4 + k] : 1 << 16;
                        q[k] = cm & 0xFFFF;
                        lj[k] = cm >> 16;
                    }
                    ljmax = from_lane63(wave_max_nonneg_lane63(max(max(lj[0], lj[1]), max(lj[2], lj[3]))));
                }
                for (int r0 = wave; r0 < ns; r0 += U * RS) {
                    int nl[U], nlmax = 1;
                    const int32_t *row[U];
                    T v[U][4];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int r = min(r0 + u * RS, ns - 1);
                        const int m = flatA ? (1 << 16) | (c * kChunk + r) : __builtin_amdgcn_readfirstlane(rowmeta[rs0 + r]);
                        row[u] = fold + ((m & 0xFFFF) - c * kChunk) * FLD;
                        nl[u] = m >> 16;
                        nlmax = max(nlmax, nl[u]);
                    }
                    {  // level 0 of all of them
                        v4i x[U];
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            if constexpr (F) x[u] = *reinterpret_cast<const v4i *>(row[u] + j4);
                            else
#pragma unroll
                                for (int k = 0; k < 4; ++k) x[u][k] = row[u][q[k]];
                        }
#pragma unroll
                        for (int u = 0; u < U; ++u)
#pragma unroll
                            for (int k = 0; k < 4; ++k) {
                                if constexpr (std::is_same<T, double>::value) v[u][k] = exact_f64(x[u][k]);
                                else v[u][k] = x[u][k];
                            }
                    }
                    for (int a = 0; a < nlmax; ++a)
                        for (int l = a == 0; l < (F ? 1 : ljmax); ++l) {
                            v4i x[U];
#pragma unroll
                            for (int u = 0; u < U; ++u) {
                                const int32_t *at = row[u] + (a < nl[u] ? a * FLD : 0);
                                if constexpr (F) x[u] = *reinterpret_cast<const v4i *>(at + j4);
                                else
#pragma unroll
                                    for (int k = 0; k < 4; ++k) x[u][k] = at[q[k] + (l < lj[k] ? l * stepB : 0)];
                            }
                            if constexpr (std::is_same<T, double>::value) {
                                const double w = (double)(1ull << (g.sh * (a + l)));
                                double wk[4];
#pragma unroll
                                for (int k = 0; k < 4; ++k) wk[k] = F || l < lj[k] ? w : 0.0;
#pragma unroll
                                for (int u = 0; u < U; ++u)
#pragma unroll
                                    for (int k = 0; k < 4; ++k) v[u][k] += exact_f64(x[u][k]) * (a < nl[u] ? wk[k] : 0.0);
                            } else {
#pragma unroll
                                for (int u = 0; u < U; ++u)
#pragma unroll
                                    for (int k = 0; k < 4; ++k)
                                        v[u][k] += (int64_t)(a < nl[u] && (F || l < lj[k]) ? x[u][k] : 0) << (g.sh * (a + l));
                            }
                        }
                    if constexpr (std::is_same<T, double>::value)
                        if (quads) {
#pragma unroll
                            for (int u = 0; u < U; ++u) {
                                const float f[4] = {(float)(v[u][0] * scale2), (float)(v[u][1] * scale2), (float)(v[u][2] * scale2), (float)(v[u][3] * scale2)};
                                store_inside4(f, rs, (unsigned)(r0 + u * RS) * (unsigned)g.ldc * 4u + quad_off);
                            }
                            continue;
                        }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        if (r0 + u * RS >= ns) break;
                        const int64_t o = (int64_t)(cs0 + r0 + u * RS) * g.ldc + jsrc0 + j4;
                        v4f_u f;
#pragma unroll
                        for (int k = 0; k < 4; ++k) f[k] = (float)((double)v[u][k] * scale2);
                        if (left >= 4) {  // 16 bytes at any boundary: a wave writes a contiguous kilobyte
                            if (C_fp) __builtin_nontemporal_store(f, reinterpret_cast<v4f_u *>(C_fp + o));
                            if constexpr (!std::is_same<T, double>::value)
                                if (g.C_int) {
                                    const v2l_u lo = {v[u][0] << final_shift, v[u][1] << final_shift}, hi = {v[u][2] << final_shift, v[u][3] << final_shift};
                                    __builtin_nontemporal_store(lo, reinterpret_cast<v2l_u *>(g.C_int + o));
                                    __builtin_nontemporal_store(hi, reinterpret_cast<v2l_u *>(g.C_int + o + 2));
                                }
                        } else {
#pragma unroll
                            for (int k = 0; k < 3; ++k)
                                if (k < left) {
                                    if (C_fp) C_fp[o + k] = f[k];
                                    if constexpr (!std::is_same<T, double>::value)
                                        if (g.C_int) g.C_int[o + k] = v[u][k] << final_shift;
                                }
                        }
                    }
                }
            };
            const bool f64 = !g.C_int && ((flatA && flatB) || fold_f64);
            if (f64 && flatB) fold_chunk(0.0, std::true_type{});
            else if (f64) fold_chunk(0.0, std::false_type{});
            else if (flatB) fold_chunk((int64_t)0, std::true_type{});
            else fold_chunk((int64_t)0, std::false_type{});
        }
    }
    // the split columns of the chunks that were stored from the registers: wave w takes chunk w, a lane a source row
    if (any_direct && nsplit > 0 && nsplit <= kStrips) {
        __syncthreads();
        if (wave >= kChunks || !((direct & filled) >> wave & 1)) return;
        const int c0 = meta(wave), L = meta(8 + wave), ns = meta(wave + 1) - c0;
        unsigned long long split_cols[4], heads[4];
        find_split(split_cols, heads);
        const int r = min(lane, ns - 1);
        const int32_t *strip = strips + wave * kChunk + r * L;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            for (unsigned long long m = heads[t]; m; m &= m - 1) {
                const int bit = __builtin_ctzll(m);
                const int src = layB.prow[n0 + 64 * t + bit] & ((1 << kProwLevel) - 1), lj = layB.src_nlev[src];
                const int32_t *s0 = strip + __popcll(split_cols[t] & ((1ull << bit) - 1ull)) * kStripPitch;
                int64_t v = 0;
                for (int l = 0; l < lj; ++l)
                    for (int a = 0; a < L; ++a) v += (int64_t)s0[l * kStripPitch + a] << (g.sh * (a + l));
                if (lane < ns) C_fp[(int64_t)(c0 + r) * g.ldc + src] = (float)((double)v * scale2);
            }
            strip += __popcll(split_cols[t]) * kStripPitch;
        }
    }
}

template <int MODE>
__global__ __launch_bounds__(kGemmThreads, 1) void gemm_i8_kernel(const GemmArgs g) {
    extern __shared__ __attribute__((aligned(1024))) int8_t smem[];
    gemm_body<MODE, false>(g, smem);
}

template <bool FP6>
__global__ __launch_bounds__(kGemmThreads, 1) void gemm_batch_kernel(const GemmArgs g) {
    extern __shared__ __attribute__((aligned(1024))) int8_t smem[];
    gemm_body<0, FP6, true>(g, smem);
}

template <bool FP6, bool LISTS>
__global__ __launch_bounds__(kGemmThreads, 1) void gemm_split_kernel(const GemmArgs g) {
    extern __shared__ __attribute__((aligned(1024))) int8_t smem[];
    gemm_body<0, FP6, false, true, LISTS>(g, smem);
}

template <bool LISTS>
__global__ __launch_bounds__(kGemmThreads, 2) void gemm_dual_kernel(const GemmArgs g) {
    extern __shared__ __attribute__((aligned(1024))) int8_t smem[];
    gemm_body<0, false, false, false, LISTS, true>(g, smem);
}

template <int MODE>
__global__ __launch_bounds__(kGemmThreads, 1) void gemm_f6_kernel(const GemmArgs g) {
    extern __shared__ __attribute__((aligned(1024))) int8_t smem[];
    gemm_body<MODE, true>(g, smem);
}

// ---- products of few tiles.  With 256 x 256 tiles a small product occupies a handful of CUs, each of which walks the whole
// contraction and then spends longer in its epilogue than in the walk.  Here a workgroup owns one 64 x 64 chunk pair of the
// layouts and its waves share the contraction: wave w of g.kwaves takes k-tiles w, w + kwaves, ... through one stage of LDS of
// its own (nothing is shared between the waves: no barrier in the loop; the stage is filled again as soon as it has been read
// into registers) and adds its 64 x 64 sums to one buffer in LDS.  Bound by the latency of a k-tile's loads; two workgroups
// per CU cover it better than two stages per wave and one workgroup (21 -> 13 us at 1000 x 1031 x 777, b = 6), and fragments
// loaded straight into registers, 64 bytes per lane and row, took twice as long (every load touches 64 lines).
// 256 x 256 x 256: 90 -> 10 us; 16 rows against 11008 x 4096 weights 83 -> 35; 1000 x 1031 x 777, b = 6: 75 -> 14.
// The planner lays rows of B out in chunks of 64 for products that it expects here (PlanHeader::chunkB).
constexpr int kSmallWaves = 4, kSmallThreads = 64 * kSmallWaves;
constexpr int kSmallPitch = 72;  // the two half-waves of an accumulator register sit four rows apart: 32 banks
constexpr int kSmallMeta = 2 * kChunk * (int)sizeof(int32_t);  // a word per source row and per source column of the chunk pair
constexpr int kSmallFold = kChunk * kSmallPitch * (int)sizeof(int32_t);
__host__ __device__ constexpr int small_stage_bytes(bool fp6) { return 2 * kChunk * (fp6 ? 96 : BK); }

template <bool FP6, bool BATCH>
__global__ __launch_bounds__(kSmallThreads, 2) void gemm_small_kernel(const GemmArgs g) {
    constexpr int kRowB = FP6 ? 96 : BK, kPitch = kRowB, kLoads = FP6 ? 6 : 8;  // as in gemm_body
    constexpr int kSteps = FP6 ? 2 : 4;                                                  // matrix instructions along a k-tile
    extern __shared__ __attribute__((aligned(1024))) int8_t smem[];
    int32_t *rowmeta = reinterpret_cast<int32_t *>(smem), *colmeta = rowmeta + kChunk;
    int8_t *stages = smem + kSmallMeta;
    int32_t *fold = reinterpret_cast<int32_t *>(stages);  // takes the place of the stages once they have been read
    const int tid = threadIdx.x, lane = tid & 63;
    const PlanHeader *hdr = BATCH ? g.hdr + blockIdx.y : nullptr;
    int mtiles = g.mtiles, ntiles = g.ntiles, ldA = g.ldA, ldB = g.ldB, kt1 = g.kt1, nbound = g.nbound;
    if constexpr (BATCH) {
        mtiles = hdr->mtiles; ntiles = hdr->ntiles;
        ldA = header_pitch(*hdr, FP6, 0); ldB = header_pitch(*hdr, FP6, 1);
        kt1 = hdr->Kp / BK;
        nbound = hdr->nruns - 1;
    }
    constexpr int kPer = kTile / kChunk;
    if (BATCH && (int)blockIdx.x >= mtiles * ntiles * kPer * kPer) return;  // the grid covers the largest item
    RowLayout layA = g.layA, layB = g.layB;
    if constexpr (BATCH) {
        move_to_item(layA, blockIdx.y * g.plan_stride);
        move_to_item(layB, blockIdx.y * g.plan_stride);
    }
    int cm, cn;
    tile_of(blockIdx.x, mtiles * kPer, ntiles * kPer, cm, cn);
    const int isrc0 = layA.chunk_src0[cm], ns = layA.chunk_src0[cm + 1] - isrc0;
    const int jsrc0 = layB.chunk_src0[cn], nc = layB.chunk_src0[cn + 1] - jsrc0;
    if (BATCH || g.guard) {
        const unsigned long long *guard = BATCH ? hdr->bound : g.guard;
        const unsigned long long b0 = guard[0], b1 = guard[1];
        const unsigned long long m = b0 < b1 ? b0 : b1;
        if (!(m < (1ull << 40) && m * (unsigned long long)g.guard_mul < (1ull << (FP6 ? 24 : 31))) || (BATCH && nbound >= 63)) {
            if (g.refused && blockIdx.x == 0 && tid == 0) g.refused[blockIdx.y] = 1;
            return;
        }
    }
    if (ns <= 0 || nc <= 0) return;  // a chunk of nothing but padding (uniform)
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m0 = cm * kChunk, n0 = cn * kChunk;

    // lane i holds the end of segment i, its block offset and the shift behind it
    int v_end, v_delta, v_shift;
    if constexpr (BATCH) {
        const int r = min(lane, nbound), r1 = min(r + 1, nbound);
        v_end = lane < nbound ? hdr->run_kt0[r1] : kt1;
        v_delta = hdr->run_blk0[r] - hdr->run_kt0[r];
        v_shift = g.sh * (hdr->grp_exp[hdr->run_grp[r]] - hdr->grp_exp[hdr->run_grp[r1]]);
    } else {
        v_end = lane < nbound ? g.bound_kt[lane] + 1 : kt1;
        v_delta = g.seg_delta[min(lane, nbound)];
        v_shift = lane < nbound ? g.bound_sh[lane] : 0;
    }
    // ---- memory -> the wave's own stage: 8 rows x 128 B per load (see gemm_body for the order inside a stage)
    const int8_t *gA = g.A + (int64_t)m0 * ldA, *gB = g.B + (int64_t)n0 * ldB;
    if constexpr (BATCH) {
        gA += blockIdx.y * g.a_stride;
        gB += blockIdx.y * g.b_stride;
    }
    unsigned voffA[kLoads], voffB[kLoads];
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {
        if (FP6) {
            const int slot = u * 64 + lane, row = slot / 6, byte = fp6_piece(row, slot - 6 * row) * 16;
            voffA[u] = (unsigned)fp6_ktile(row, 0, ldA) + (unsigned)byte;
            voffB[u] = (unsigned)fp6_ktile(row, 0, ldB) + (unsigned)byte;
        } else {
            const int row = 8 * u + (lane >> 3), byte = ((lane & 7) ^ ((row >> 1) & 7)) * 16;
            voffA[u] = (unsigned)i8_at(row, byte, ldA);
            voffB[u] = (unsigned)i8_at(row, byte, ldB);
        }
    }
    const int8_t *sa = stages + wave * small_stage_bytes(FP6), *sb = sa + kChunk * kPitch;  // the wave's stage
    const int step = g.kwaves;
    const bool busy = wave < step && wave < kt1;
    using FragT = std::conditional_t<FP6, v8i, v4i>;
    using AccT = std::conditional_t<FP6, v16f, v16i>;
    const int lrow = lane & 31, lhalf = lane >> 5;
    AccT acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;
    int seg = 0;  // follows the loads
    unsigned long long probe_c = 0, probe_w = 0;
    const bool probing = !BATCH && g.clock_probe != nullptr && blockIdx.x == 0;
    if (probing) {
        probe_c = __builtin_readcyclecounter();
        probe_w = wall_clock64();
    }
    // The wave's share of the contraction.  RA: 32-row halves of the A chunk that hold source rows (a batch of up to 32
    // decoded tokens fills one).
    auto contract = [&](auto ra_c) {
        constexpr int RA = decltype(ra_c)::value;
        constexpr int kLoadsA = RA == 2 ? kLoads : kLoads / 2;
        // starts the loads of k-tile kt; returns the Horner shift between the wave's k-tile before and this one
        auto fetch = [&](int kt) {
            int sh = 0;
            while (seg < nbound && kt >= __builtin_amdgcn_readlane(v_end, seg)) {
                sh += __builtin_amdgcn_readlane(v_shift, seg);
                ++seg;
            }
            const int blk = kt + __builtin_amdgcn_readlane(v_delta, seg);
            const int8_t *pa = uniform_ptr(gA + (FP6 ? fp6_ktile(0, blk, ldA) : (int64_t)blk * kRowB));
            const int8_t *pb = uniform_ptr(gB + (FP6 ? fp6_ktile(0, kt, ldB) : (int64_t)kt * kRowB));
            const unsigned dst = __builtin_amdgcn_readfirstlane((unsigned)(size_t)sa);
#pragma unroll
            for (int u = 0; u < kLoadsA; ++u) dma16(dst + u * 1024, voffA[u], pa);
#pragma unroll
            for (int u = 0; u < kLoads; ++u) dma16(dst + kChunk * kPitch + u * 1024, voffB[u], pb);
            return sh;
        };
        fetch(wave);  // nothing summed up yet: nothing to shift
        for (int kt = wave, sh_now = 0;; kt += step) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            FragT fa[RA][kSteps], fb[2][kSteps];
            auto load_frag = [&](const int8_t *half, int k) {
                const int8_t *row = half + lrow * kPitch;
                if constexpr (FP6) {
                    const v4i lo = *reinterpret_cast<const v4i *>(row + 16 * fp6_piece(lrow, 3 * k + lhalf));
                    const v2i hi = *reinterpret_cast<const v2i *>(row + 16 * fp6_piece(lrow, 3 * k + 2) + 8 * (lhalf ^ ((lrow >> 4) & 1)));
                    return v8i{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], 0, 0};
                } else {
                    return *reinterpret_cast<const v4i *>(row + (((2 * k + lhalf) ^ ((lrow >> 1) & 7)) << 4));
                }
            };
#pragma unroll
            for (int k = 0; k < kSteps; ++k) {
#pragma unroll
                for (int i = 0; i < RA; ++i) fa[i][k] = load_frag(sa + i * 32 * kPitch, k);
#pragma unroll
                for (int j = 0; j < 2; ++j) fb[j][k] = load_frag(sb + j * 32 * kPitch, k);
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the stage has been read: it may be filled again
            const bool more = kt + step < kt1;
            const int sh_next = more ? fetch(kt + step) : 0;
            if (sh_now != 0) {
#pragma unroll
                for (int i = 0; i < RA; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            if constexpr (FP6) acc[i][j][r] = ldexpf(acc[i][j][r], sh_now);
                            else acc[i][j][r] <<= sh_now;
                        }
            }
#pragma unroll
            for (int k = 0; k < kSteps; ++k)
#pragma unroll
                for (int i = 0; i < RA; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        if constexpr (FP6) acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fa[i][k], fb[j][k], acc[i][j], 2, 2, 0, 0, 0, 0);
                        else acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[i][k], fb[j][k], acc[i][j], 0, 0, 0);
                    }
            if (!more) break;
            sh_now = sh_next;
        }
    };
    const int lmaxA = BATCH ? hdr->lmaxA : g.lmaxA;
    const bool half_rows = ns * (lmaxA == 3 ? 4 : lmaxA) <= 32;  // uniform; the rows of a chunk start at its first (three levels may take four rows)
    if (busy) {
        if (half_rows) contract(std::integral_constant<int, 1>{});
        else contract(std::integral_constant<int, 2>{});
    }
    // The columns that are taken from lists: a wave takes 32 entries in turn, through its stage.  Sums of their own: the accumulators may
    // be counting in units of a higher group, and by `rest` they are brought to those of the lowest, which is exponent 0 here.
    AccT list_acc[2][2];
    const bool lists = !FP6 && !BATCH && g.sp_kt >= 0 && busy;
    if constexpr (!FP6 && !BATCH) {
        if (lists) {
            static_assert(list_lds(1) <= small_stage_bytes(FP6), "LDS of the lists");
            const int8_t *at = uniform_ptr(g.at + (int64_t)(cm / 2) * g.at_cols * 128);
            int8_t *lds = const_cast<int8_t *>(sa);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int r = 0; r < 16; ++r) list_acc[i][j][r] = 0;
                const int block = 2 * cn + j, len = min(g.sparse.cnt[block], g.sparse.cap);
                const uint32_t *list = g.sparse.ent + (size_t)block * g.sparse.cap;
                for (int t = wave * 32; t < len; t += step * 32) {
                    ListWords<1> words;
                    unsigned x[16];
                    words.load(list + t, lane);
                    v4i fd[1];
                    words.stage(lds, len - t, lane, fd);
                    list_columns(x, lds + 1024, 0, lhalf, at, (unsigned)lrow * 4u);
                    v4i fr[4];
                    list_rows(x, fr);
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        v4i a;
#pragma unroll
                        for (int q = 0; q < 4; ++q) a[q] = cm & 1 ? fr[2 + i][q] : fr[i][q];
                        list_acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, fd[0], list_acc[i][j], 0, 0, 0);
                    }
                }
            }
        }
    }
    if (tid < ns) rowmeta[tid] = (layA.src_pstart[isrc0 + tid] - m0) | (layA.src_nlev[isrc0 + tid] << 16);
    if (tid >= 64 && tid - 64 < nc) colmeta[tid - 64] = (layB.src_pstart[jsrc0 + tid - 64] - n0) | (layB.src_nlev[jsrc0 + tid - 64] << 16);
    __syncthreads();  // every stage has been read
    // the shifts behind the wave's last segment: then every wave counts in units of the lowest group
    int rest = 0;
    for (; seg < nbound; ++seg) rest += __builtin_amdgcn_readlane(v_shift, seg);
    auto each = [&](auto put) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            if (i == 1 && half_rows) break;
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    put(&fold[(i * 32 + 8 * (r >> 2) + 4 * lhalf + (r & 3)) * kSmallPitch + j * 32 + lrow],
                        ((int32_t)acc[i][j][r] << rest) + (lists ? (int32_t)list_acc[i][j][r] << g.sh : 0));
        }
    };
    if (wave == 0) each([](int32_t *p, int32_t x) { *p = x; });  // (wave 0 always has a k-tile)
    __syncthreads();
    if (wave != 0 && busy) each([](int32_t *p, int32_t x) { atomicAdd(p, x); });
    if (probing && tid == 0) {
        g.clock_probe[0] = __builtin_readcyclecounter() - probe_c;
        g.clock_probe[1] = wall_clock64() - probe_w;
    }
    float *C_fp = g.C_fp;
    int final_shift = g.final_shift;
    const float *scale_a_dev = g.scale_a_dev, *scale_b_dev = g.scale_b_dev;
    if constexpr (BATCH) {
        C_fp = item_at(C_fp, blockIdx.y * g.c_stride);
        final_shift = hdr->ngroups ? g.sh * hdr->grp_exp[hdr->ngroups - 1] : 0;
        scale_a_dev = item_at(scale_a_dev, blockIdx.y * g.scale_stride);
        scale_b_dev = item_at(scale_b_dev, blockIdx.y * g.scale_stride);
    }
    const double scale2 = (scale_a_dev ? (double)*scale_a_dev * (double)*scale_b_dev : g.scale) * (double)(1ull << final_shift);
    __syncthreads();
    // C_int[i,j] = sum_{levels a of i, c of j} s^(a+c) * fold[row(i,a)][col(j,c)]: a lane owns a source column, a wave works
    // on four source rows at a time so that their LDS reads are in flight together
    if (lane >= nc) return;
    const int q0 = colmeta[lane] & 0xFFFF, lj = colmeta[lane] >> 16;
    const int stepB = (BATCH ? hdr->evenB : g.evenB) ? kEvenStep : 1;  // from level to level of a source column
    constexpr int U = 4;
    for (int r0 = wave; r0 < ns; r0 += U * kSmallWaves) {
        int nl[U], nlmax = 0;
        const int32_t *row[U];
        int64_t v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int r = r0 + u * kSmallWaves;
            const int m = r < ns ? rowmeta[r] : 0;
            row[u] = fold + (m & 0xFFFF) * kSmallPitch + q0;
            nl[u] = m >> 16;  // 0 past the chunk's last source row
            nlmax = max(nlmax, nl[u]);
            v[u] = 0;
        }
        for (int a = 0; a < nlmax; ++a)
            for (int c = 0; c < lj; ++c)
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (a < nl[u]) v[u] += (int64_t)row[u][a * kSmallPitch + c * stepB] << (g.sh * (a + c));
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (nl[u]) {
                const int64_t o = (int64_t)(isrc0 + r0 + u * kSmallWaves) * g.ldc + jsrc0 + lane;
                if (C_fp) C_fp[o] = (float)((double)v[u] * scale2);
                if (g.C_int) g.C_int[o] = v[u] << final_shift;
            }
    }
}

// C_int = Pi_A C_u Pi_B^T from the int64 unpacked product, then dequantise.
__global__ __launch_bounds__(256) void recombine_kernel(const int64_t *__restrict__ C_u, int Np, RowLayout layA,
                                                        RowLayout layB, int n, int h, int sh,
                                                        int64_t *C_int, float *C_fp, int64_t ldc,
                                                        double scale_val, const float *scale_a_dev,
                                                        const float *scale_b_dev, int stepB) {
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= h) return;
    const double scale = scale_a_dev ? (double)*scale_a_dev * (double)*scale_b_dev : scale_val;
    const int q0 = layB.src_pstart[j], lj = layB.src_nlev[j];
    for (int i = blockIdx.y; i < n; i += gridDim.y) {
        const int p0 = layA.src_pstart[i], li = layA.src_nlev[i];
        int64_t acc = 0;
        for (int a = 0; a < li; ++a)
            for (int c = 0; c < lj; ++c) acc += C_u[(int64_t)(p0 + a) * Np + (q0 + c * stepB)] << (sh * (a + c));
        const int64_t o = (int64_t)i * ldc + j;
        if (C_int) C_int[o] = acc;
        if (C_fp) C_fp[o] = (float)((double)acc * scale);
    }
}

__global__ void clear_words_kernel(int32_t *p, int count) {
    for (int i = threadIdx.x; i < count; i += blockDim.x) p[i] = 0;
}

// Register-resident back-to-back int8 MFMAs (no memory traffic): what the matrix cores sustain on
// this chip, for the measured-peak line of the benchmark.  Eight independent accumulators per wave.
__global__ __launch_bounds__(256) void mfma_peak_kernel(int iters, int *sink) {
    v4i a, b;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        a[i] = (int)threadIdx.x + i;
        b[i] = (int)blockIdx.x + i;
    }
    v16i acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][r] = 0;
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, acc[i], 0, 0, 0);
    }
    int x = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) x ^= acc[i][r];
    if (x == 0x7fffffff && sink) *sink = x;  // keeps the accumulators live
}

}  // namespace imu

using namespace imu;

// device memory of the caller, see imunpack_diag_clock_probe
static std::atomic<unsigned long long *> g_clock_probe{nullptr};

static int gemm_lds_opt_in() {
    // the kernels use all 160 KiB of a CU's LDS as dynamic shared memory, above the default limit; the
    // attribute is idempotent, so two threads racing through here both set the same value
    static std::atomic<int> done{0};
    if (!done.load(std::memory_order_acquire)) {
        IMU_HIP(hipFuncSetAttribute((const void *)gemm_i8_kernel<0>, hipFuncAttributeMaxDynamicSharedMemorySize, kGemmLds));
        IMU_HIP(hipFuncSetAttribute((const void *)gemm_i8_kernel<1>, hipFuncAttributeMaxDynamicSharedMemorySize, kGemmLds));
        IMU_HIP(hipFuncSetAttribute((const void *)gemm_f6_kernel<0>, hipFuncAttributeMaxDynamicSharedMemorySize, kGemmLds));
        IMU_HIP(hipFuncSetAttribute((const void *)gemm_f6_kernel<1>, hipFuncAttributeMaxDynamicSharedMemorySize, kGemmLds));
        IMU_HIP(hipFuncSetAttribute((const void *)gemm_batch_kernel<false>, hipFuncAttributeMaxDynamicSharedMemorySize, kGemmLds));
        IMU_HIP(hipFuncSetAttribute((const void *)gemm_batch_kernel<true>, hipFuncAttributeMaxDynamicSharedMemorySize, kGemmLds));
        IMU_HIP(hipFuncSetAttribute((const void *)gemm_split_kernel<false, false>, hipFuncAttributeMaxDynamicSharedMemorySize, kGemmLds));
        IMU_HIP(hipFuncSetAttribute((const void *)gemm_split_kernel<true, false>, hipFuncAttributeMaxDynamicSharedMemorySize, kGemmLds));
        IMU_HIP(hipFuncSetAttribute((const void *)gemm_split_kernel<false, true>, hipFuncAttributeMaxDynamicSharedMemorySize, kGemmLds));
        IMU_HIP(hipFuncSetAttribute((const void *)gemm_dual_kernel<false>, hipFuncAttributeMaxDynamicSharedMemorySize, kDualLds));
        IMU_HIP(hipFuncSetAttribute((const void *)gemm_dual_kernel<true>, hipFuncAttributeMaxDynamicSharedMemorySize, kDualLds));
        constexpr int kSmallLds = kSmallMeta + kSmallWaves * small_stage_bytes(false);
        IMU_HIP(hipFuncSetAttribute((const void *)gemm_small_kernel<false, false>, hipFuncAttributeMaxDynamicSharedMemorySize, kSmallLds));
        IMU_HIP(hipFuncSetAttribute((const void *)gemm_small_kernel<true, false>, hipFuncAttributeMaxDynamicSharedMemorySize, kSmallLds));
        IMU_HIP(hipFuncSetAttribute((const void *)gemm_small_kernel<false, true>, hipFuncAttributeMaxDynamicSharedMemorySize, kSmallLds));
        IMU_HIP(hipFuncSetAttribute((const void *)gemm_small_kernel<true, true>, hipFuncAttributeMaxDynamicSharedMemorySize, kSmallLds));
        done.store(1, std::memory_order_release);
    }
    return IMUNPACK_OK;
}

static int check_shifts(const Plan *p) {
    // every weight s^(levelA + levelB + e) applied in int64 must stay below 2^62
    const int maxexp = (p->hdr.lmaxA - 1) + (p->hdr.lmaxB - 1) + (p->hdr.ngroups ? p->hdr.grp_exp[0] : 0);
    return maxexp * p->sh <= 62 ? IMUNPACK_OK : IMUNPACK_ERANGE;
}

namespace imu {
int recombine_impl(const imunpack_plan_t *p, const void *workspace, float scale_A, float scale_B,
                   const float *scale_a_dev, const float *scale_b_dev, int64_t *C_int, float *C_fp, int64_t ldc,
                   hipStream_t stream) {
    if (!p || !p->valid || !workspace || ldc < p->h) return IMUNPACK_EINVAL;
    if (!C_int && !C_fp) return IMUNPACK_OK;
    IMU_TRY(check_shifts(p));
    dim3 grid((unsigned)((p->h + 255) / 256), (unsigned)std::min<int64_t>(p->n, 65535));
    hipLaunchKernelGGL(recombine_kernel, grid, dim3(256), 0, stream,
                       (const int64_t *)workspace, p->hdr.Np, p->layA, p->layB, (int)p->n, (int)p->h, p->sh,
                       C_int, C_fp, ldc, (double)scale_A * (double)scale_B, scale_a_dev, scale_b_dev, p->hdr.evenB ? kEvenStep : 1);
    return launch_status();
}
}  // namespace imu

extern "C" int imunpack_recombine(const imunpack_plan_t *p, const void *workspace, float scale_A,
                                  float scale_B, int64_t *C_int, float *C_fp, int64_t ldc,
                                  imunpack_stream_t stream) {
    return recombine_impl(p, workspace, scale_A, scale_B, nullptr, nullptr, C_int, C_fp, ldc, (hipStream_t)stream);
}

namespace imu {
// Whether results that have no levels to fold go through LDS and out as non-temporal rows of a kilobyte.  From the registers they
// are ordinary stores (non-temporal lines of 128 bytes are slow), the faster way for the kernel (4096 x 8228 by 11013: 309 and
// 320 us, in a run of few steps 327 and 338), but they stay in the last-level cache of 256 MB, and what a step reads again, the
// operands and their integers, does not: the scatter and quantise behind that product 90 and 97 us instead of 84 and 93.  The line
// lies where the two meet, in bytes of operands, integers and results (rows by columns of A by rows of B, a step through the registers and through LDS, means of
// three turns that differ by 1 to 3 %): 235 MB 184 and 188 us (4096 x 1024 by 8192), 251 MB 184 and 187 (12608 x 768 by 3072),
// 302 MB 236 and 238 (4096 x 2048 by 7168), 319 MB 219 and 216 (8192 x 1024 by 6144), 341 MB 281 and 281 (6000 x 2048 by 6000),
// 361 MB 257 and 258 (8192 x 1024 by 7168), 403 MB 273 and 267 (8192 x 1024 by 8192), 439 MB 343 and 327 (1024 x 4096 by 11008),
// 675 MB 754 and 753, 450 and 440 with resident weights (4096 x 4096 by 11008).  Batches of several items, whose products are
// small beside that cache one by one, were not measured and stay with the registers.
static bool whole_rows_win(const Plan *p) {
    const double d = (double)p->d, rows = (double)p->n + (double)p->h;
    return 8.0 * rows * d + 4.0 * (double)p->n * (double)p->h > 320e6;
}
// The runs that the fused GEMM walks: what is taken from lists is a run of B_eu's own, the last.
static int fused_runs(const PlanHeader &h) { return h.nruns - (h.nsparse ? 1 : 0); }
// What the fused launch of one plan takes from its header.
static void fused_args(GemmArgs &g, const Plan *p) {
    const PlanHeader &h = p->hdr;
    g.ldA = (int)store_pitch(p, 0); g.ldB = (int)store_pitch(p, 1); g.Kp = h.Kp; g.mtiles = h.mtiles; g.ntiles = h.ntiles;
    g.layA = p->layA; g.layB = p->layB;
    g.sh = p->sh;
    g.Np = h.Np;
    g.lmaxA = h.lmaxA;
    g.evenB = h.evenB;
    g.whole_rows = whole_rows_win(p);
    g.guard_mul = p->s - 1;
    g.kt0 = 0; g.kt1 = h.nsparse ? h.list_kt0 : h.Kp / BK;
    g.nbound = 0;
    const int runs = fused_runs(h);
    for (int r = 0; r < runs; ++r) {
        g.seg_delta[r] = h.run_blk0[r] - h.run_kt0[r];
        if (r + 1 < runs) {
            g.bound_kt[g.nbound] = h.run_kt0[r + 1] - 1;
            g.bound_sh[g.nbound] = p->sh * (h.grp_exp[h.run_grp[r]] - h.grp_exp[h.run_grp[r + 1]]);
            ++g.nbound;
        }
    }
    g.final_shift = h.ngroups ? p->sh * h.grp_exp[h.ngroups - 1] : 0;
    g.sp_kt = -1;
    if (h.nsparse) {
        g.sparse = p->sparse;
        g.at = p->at;
        g.at_cols = (int)p->d;
        // before the first group of exponent 1 or, if no column of that exponent is stored, 0 (there always is that one)
        int r = 0;
        while (h.grp_exp[h.run_grp[r]] > 1) ++r;
        g.sp_kt = h.run_kt0[r];
        if (h.grp_exp[h.run_grp[r]] == 0) g.sp_after = p->sh;
    }
    // |accumulator| < 2^31, weights up to s^(levels of a row - 1 + levels of a column - 1)
    g.fold_f64 = 31 + p->sh * ((h.lmaxA - 1) + (h.lmaxB - 1)) <= 52;
}

// What the epilogue of a large tile takes: the longer way through LDS where levels differ from row to row (3328 x 768 in 3 and
// 5 levels by 3072 rows: 34 us a round), the more where columns are split as well (1408 x 1024 by 1800 rows of two levels 27 us,
// 250 by 6400 rows of two levels both 36).  The planner, which lays out B's rows before the levels are known, asks with kTileNs and
// a margin of 25 % instead: where splits make the large tiles dearer than that, a product between the two costs takes them all the
// same.
static int tile_ns(const PlanHeader &h) {
    if (h.lmaxB > 1 && !h.evenB) return 10000 + 4500 * h.lmaxA * h.lmaxB;
    return h.lmaxA > 1 && !h.evenA ? 12000 + 3000 * h.lmaxA : kTileNs;
}
// Where there are CUs for all half tiles (int8 digits, a product of its own, at most 128 tiles; see dual_wins) the choice is between those and the
// small ones, by least-squares fits over 895 products of 8 to 128 tiles, 1 to 64 k-tiles and one to five levels on either side (nanoseconds, rms 1.2 to
// 1.8 us and 3.3 us; what they choose takes 0.9 % more in all than the better one each time, 29 % at worst).  Half tiles: results that leave from
// the registers take the least, and where they go through LDS it is the levels of B that cost (1576 x 896 by 3072, 84 tiles, 20 us and small tiles 36;
// 459 x 256 by 2 x 3036 rows, rows of A of two and three levels, 22 and 12; 1047 x 1280 by 3 x 1257 29 and 37).  Small tiles: by the chunk
// pairs that hold anything and, for their levels, by the rounds that all of them take, two to a CU.
static bool small_tiles_beat_halves(const PlanHeader &h, int64_t tiles, int64_t pairs, int64_t ktiles) {
    const bool unevenA = h.lmaxA > 1 && !h.evenA, unevenB = h.lmaxB > 1 && !h.evenB;
    const int64_t results = unevenA && unevenB     ? 19400 + 3300 * h.lmaxB - 1800 * h.lmaxA
                            : unevenB              ? 12300 + 2900 * h.lmaxB - 900 * h.lmaxA
                            : unevenA && h.lmaxB > 1 ? 22400 - 1000 * h.lmaxA
                            : unevenA              ? 16600 - 1200 * h.lmaxA
                                                   : 10300;
    const int64_t half = std::max<int64_t>(results, 10300) + 620 * ktiles + 18 * tiles;
    const int64_t small = 8500 + 100 * ktiles + pairs * (2000 + 360 * ktiles) / 512 + (tiles * kChunkPairs + 511) / 512 * 1000 * h.lmaxB;
    return small < half;
}
// Whether the small tiles are the better ones for this plan (and B's rows are laid out for them).
static bool small_tiles(const Plan *p, int64_t tiles, int64_t pairs, int64_t ktiles) {
    if (p->hdr.chunkB != kChunk) return false;
    const bool single = p->nitems == 1;
    if (single && !p->fp6 && tiles <= 128 && split_parts(tiles, ktiles) == 1) return small_tiles_beat_halves(p->hdr, tiles, pairs, ktiles);
    return small_tiles_win(tiles, pairs, ktiles, single, 0, tile_ns(p->hdr));
}
// The chunk pairs of an unpacked product that hold source rows.
static int64_t chunk_pairs(const PlanHeader &h) {
    auto chunks = [](int rows, int lmax) { return (rows + kChunk - lmax) / (kChunk - lmax + 1); };
    return (int64_t)chunks(h.n_u, h.lmaxA) * chunks(h.h_u, h.lmaxB);
}

// The launch of the small-tile kernel: as many stages as the (longest) contraction has k-tiles for, so that short
// contractions leave LDS to more workgroups of a CU.
static int launch_small(const Plan *p, GemmArgs g, int chunks, int ktiles, bool batch, hipStream_t st) {
    g.kwaves = std::max(1, std::min(ktiles, kSmallWaves));
    const int lds = kSmallMeta + std::max(g.kwaves * small_stage_bytes(p->fp6), kSmallFold);
    const dim3 grid((unsigned)chunks, batch ? (unsigned)p->nitems : 1u), threads(kSmallThreads);
    if (batch && p->fp6) hipLaunchKernelGGL((gemm_small_kernel<true, true>), grid, threads, lds, st, g);
    else if (batch) hipLaunchKernelGGL((gemm_small_kernel<false, true>), grid, threads, lds, st, g);
    else if (p->fp6) hipLaunchKernelGGL((gemm_small_kernel<true, false>), grid, threads, lds, st, g);
    else hipLaunchKernelGGL((gemm_small_kernel<false, false>), grid, threads, lds, st, g);
    return launch_status();
}

// What the parts of a tile meet in (64 MiB): made when the plan's first product that is cut is multiplied, freed with the plan.
// Two launches that share it must not overlap.  Returns whether it can be used on this stream (never under capture).
static bool prepare_split(Plan *p, hipStream_t st) {
    if (capturing(st)) return false;
    constexpr int kMeets = 8 * kXcdCus;
    if (!p->split_ws) {
        if (hipMalloc(&p->split_ws, (size_t)kMeets * (BM * BN + 2) * sizeof(int32_t)) != hipSuccess ||
            hipEventCreateWithFlags(&p->split_done, hipEventDisableTiming) != hipSuccess) {
            (void)hipGetLastError();
            if (p->split_ws) (void)hipFree(p->split_ws);
            p->split_ws = nullptr;
            return false;
        }
        hipLaunchKernelGGL(clear_words_kernel, dim3(1), dim3(256), 0, st, (int32_t *)p->split_ws, 2 * kMeets);
    } else {  // (not by comparing stream handles: one handle may stand for a stream per thread, or be used again)
        hipError_t e = hipEventQuery(p->split_done);
        if (e == hipErrorNotReady) e = hipStreamWaitEvent(st, p->split_done, 0);
        (void)hipGetLastError();
        if (e != hipSuccess) return false;
    }
    return true;
}

// Whether half tiles, two workgroups to a CU, are the better ones (int8 digits).  While one workgroup loads its first k-tiles, takes
// columns from lists or stores its results the other one has the matrix cores, and a product that fills half the CUs with whole tiles
// fills all of them; but a half tile takes half as many operand bytes again for its operations, so over a long contraction that is
// all there is to it the whole tiles win.  Microseconds with k-tiles t (whole and half tiles, kernel alone): a full round 14 + 1.45 t and 12 +
// 1.48 t, a round of at most 256 half tiles 9 + 0.8 t.  4096 x 4352 by 11013 with lists 259 and 248 (in a step 288 and 247), 12608 x
// 896 by 3072, folded rows, 114 and 94; 5120 x 5120 by 4096 138 and 110; 2304 x 2304 by 2048 40 and 26; 10240 x 5760 by 8192 408
// and 391; but 8192 x 8320 by 4096 222 and 233, 11776 x 11392 by 8192 816 and 835, 1024 x 8448 by 11264 (176 tiles) 100 and 103.
static bool dual_wins(int64_t tiles, int64_t ktiles) {
    const int64_t halves = tiles * (BM / kDualRows), full = 12000 + 1483 * ktiles, rem = halves % 512;
    const int64_t dual = halves / 512 * full + (rem == 0 ? 0 : rem <= 256 ? 9000 + 800 * ktiles : full);
    return dual < (tiles + 255) / 256 * (kTileNs + 1450 * ktiles);
}

// Rows of B in four places each, evenly laid out, and rows of A that are too, or have one level: a whole tile folds its results in the
// registers (a lane has all four levels of a source column), a half tile, whose waves are two blocks of 32 columns wide, takes them through LDS.
// Whole and half tiles, microseconds with b = 3, rows of B of four levels: 6392 x 256 by 4 x 9904 rows 171 and 330, x 1024 286 and 398; 1500 x
// 512 by 4 x 1500 17 and 31, x 2048 31 and 44; 3000 x 1024 by 4 x 3000, rows of A of two levels 87 and 125, of four 154 and 230; over long
// contractions the walk decides: 3000 x 6016 by 4 x 3000 181 and 182, x 9088 257 and 252; 1000 x 3072 by 4 x 2000 (128 tiles) 38 and 38.  Where
// rows of A go through LDS in whole tiles too, 364 and 234 (three levels), 89 and 85 (five rows of 3000 have two), or int64 results, 148 and 88.
static bool whole_tiles_fold(const GemmArgs &g, const PlanHeader &h, int64_t tiles) {
    return h.evenB == 4 && (h.lmaxA == 1 || h.evenA) && g.fold_f64 && !g.C_int && g.ldc < kDirectPitch && g.kt1 <= (tiles <= 128 ? 24 : 48);
}

// The fused launch of one product.
static int launch_fused(Plan *p, GemmArgs &g, hipStream_t st) {
    const int tiles = g.mtiles * g.ntiles;
    p->gemm_parts = p->gemm_halves = 0;
    if (small_tiles(p, tiles, chunk_pairs(p->hdr), g.kt1)) return launch_small(p, g, tiles * kChunkPairs, g.kt1, false, st);
    // (Parts are asked for before half tiles, by what they gain over whole tiles.  Half tiles against them, microseconds in parts and in half tiles:
    // 64 tiles, 48 k-tiles 63 and 45, 118: 91 and 89; 128 tiles, 48: 75 and 54, 100: 112 and 98; 320 tiles, 48: 152 and 126, 96: 240 and 230;
    // 528 tiles, 66: 284 and 271; but 272 tiles, 128: 278 and 292.  So below about a hundred k-tiles they would be the better ones.)
    const int parts = split_parts(tiles, g.kt1);
    if (parts > 1 && prepare_split(p, st)) {
        g.meet = (int32_t *)p->split_ws;
        g.sums = g.meet + 2 * 8 * kXcdCus;
        g.most_parts = parts;
        p->gemm_parts = parts;
        const dim3 grid((unsigned)(8 * (((tiles + 7) / 8 + kXcdCus - 1) / kXcdCus * kXcdCus)));
        if (p->fp6) hipLaunchKernelGGL((gemm_split_kernel<true, false>), grid, dim3(kGemmThreads), kGemmLds, st, g);
        else if (g.sp_kt >= 0) hipLaunchKernelGGL((gemm_split_kernel<false, true>), grid, dim3(kGemmThreads), kGemmLds, st, g);
        else hipLaunchKernelGGL((gemm_split_kernel<false, false>), grid, dim3(kGemmThreads), kGemmLds, st, g);
        IMU_HIP(hipEventRecord(p->split_done, st));
        return launch_status();
    }
    p->gemm_parts = 1;
    if (!p->fp6 && (g.sp_kt >= 0 || (dual_wins(tiles, g.kt1) && !whole_tiles_fold(g, p->hdr, tiles)))) {  // (lists hold up a whole tile for some 12 us more, which its k-tiles make up for only after hundreds)
        p->gemm_halves = 1;
        const dim3 halves((unsigned)(tiles * (BM / kDualRows)));
        if (g.sp_kt >= 0) hipLaunchKernelGGL(gemm_dual_kernel<true>, halves, dim3(kGemmThreads), kDualLds, st, g);
        else hipLaunchKernelGGL(gemm_dual_kernel<false>, halves, dim3(kGemmThreads), kDualLds, st, g);
        return launch_status();
    }
    if (p->fp6) hipLaunchKernelGGL(gemm_f6_kernel<0>, dim3(tiles), dim3(kGemmThreads), kGemmLds, st, g);
    else hipLaunchKernelGGL(gemm_i8_kernel<0>, dim3(tiles), dim3(kGemmThreads), kGemmLds, st, g);
    return launch_status();
}

int gemm_impl(imunpack_plan_t *p, const int8_t *A_ue, const int8_t *B_eu, void *workspace, int64_t *C_int,
              float *C_fp, int64_t ldc, float scale_A, float scale_B, const float *scale_a_dev,
              const float *scale_b_dev, int fuse, hipStream_t st) {
    if (!p || !p->valid || !p->unpacked || !A_ue || !B_eu || (scale_a_dev == nullptr) != (scale_b_dev == nullptr))
        return IMUNPACK_EINVAL;
    const PlanHeader &h = p->hdr;
    if (h.mtiles <= 0 || h.ntiles <= 0) return IMUNPACK_OK;
    IMU_TRY(check_shifts(p));
    IMU_TRY(gemm_lds_opt_in());
    GemmArgs g;
    memset(&g, 0, sizeof(g));
    g.A = A_ue; g.B = B_eu;
    g.ldA = (int)store_pitch(p, 0); g.ldB = (int)store_pitch(p, 1); g.Kp = h.Kp; g.mtiles = h.mtiles; g.ntiles = h.ntiles;
    g.layA = p->layA; g.layB = p->layB;
    g.sh = p->sh;
    g.Np = h.Np;
    const int grid = h.mtiles * h.ntiles;
    bool fused = fuse != 0;
    const bool too_many_runs = fused_runs(h) > 63;  // more segments than the lanes of a wave can hold the tables of
    // The bounds of the last imunpack_unpack may still be on their way to the host.  If the fused
    // launch was exact for this plan object the last time, it goes out now with a guard (the kernel
    // checks the bounds on the device and writes nothing if they are too large), and only then does
    // the host wait: the GPU does not idle while the answer travels.
    if (fused && too_many_runs) {
        if (!workspace) return IMUNPACK_ERANGE;
        fused = false;
    }
    const bool speculate = fused && p->bound_pending && p->guess_fusable;
    if (!speculate) {
        IMU_TRY(resolve_bound(p));
        if (fused && !p->fusable) {
            if (!workspace) return IMUNPACK_ERANGE;
            fused = false;
        }
    }
    if (fused) {
        if ((!C_int && !C_fp) || ldc < p->h) return IMUNPACK_EINVAL;
        fused_args(g, p);
        g.guard = speculate ? p->d_hdr->bound : nullptr;
        g.C_int = C_int; g.C_fp = C_fp; g.ldc = ldc;
        g.scale = (double)scale_A * (double)scale_B;
        g.scale_a_dev = scale_a_dev; g.scale_b_dev = scale_b_dev;
        g.clock_probe = g_clock_probe.load(std::memory_order_relaxed);
        g.fold_f64 = g.fold_f64 && !C_int;
        IMU_TRY(launch_fused(p, g, st));
        if (!speculate) return IMUNPACK_OK;
        IMU_TRY(resolve_bound(p));
        if (p->fusable) return IMUNPACK_OK;
        if (!workspace) return IMUNPACK_ERANGE;  // the guarded launch wrote nothing
        g.guard = nullptr;
    }
    if (!workspace) return IMUNPACK_EINVAL;
    g.C_u = (int64_t *)workspace;
    for (int r = 0; r < h.nruns; ++r) {  // one launch per stretch of consecutive blocks of the A store
        g.kt0 = h.run_kt0[r];
        g.kt1 = r + 1 < h.nruns ? h.run_kt0[r + 1] : h.Kp / BK;
        g.nbound = 0;
        g.seg_delta[0] = h.run_blk0[r] - h.run_kt0[r];
        g.seg_shift = p->sh * h.grp_exp[h.run_grp[r]];
        g.seg_first = r == 0;
        if (p->fp6) hipLaunchKernelGGL(gemm_f6_kernel<1>, dim3(grid), dim3(kGemmThreads), kGemmLds, st, g);
        else hipLaunchKernelGGL(gemm_i8_kernel<1>, dim3(grid), dim3(kGemmThreads), kGemmLds, st, g);
    }
    IMU_TRY(launch_status());
    if (fuse != 0)  // the caller asked for final outputs: finish the job here
        return recombine_impl(p, workspace, scale_A, scale_B, scale_a_dev, scale_b_dev, C_int, C_fp, ldc, st);
    return IMUNPACK_OK;
}

int gemm_batch(imunpack_plan_t *p, const int8_t *A_ue, int64_t a_stride, const int8_t *B_eu, int64_t b_stride, float *C_fp,
               int64_t c_stride, int64_t ldc, const float *scale_a_dev, const float *scale_b_dev, int64_t scale_stride,
               int32_t *refused, hipStream_t st) {
    if (!p || !p->valid || !p->unpacked || !A_ue || !B_eu || !C_fp || ldc < p->h || !scale_a_dev || !scale_b_dev || !refused)
        return IMUNPACK_EINVAL;
    IMU_TRY(gemm_lds_opt_in());
    int grid = 0;
    int64_t tiles = 0, pairs = 0, ktiles = 0;
    for (int i = 0; i < p->nitems; ++i) {
        const PlanHeader &h = p->pin_hdr[i];
        const int maxexp = (h.lmaxA - 1) + (h.lmaxB - 1) + (h.ngroups ? h.grp_exp[0] : 0);
        if (maxexp * p->sh > 62) return IMUNPACK_ERANGE;
        grid = std::max(grid, h.mtiles * h.ntiles);
        tiles += h.mtiles * h.ntiles;
        pairs += chunk_pairs(h);
        ktiles = std::max<int64_t>(ktiles, h.Kp / BK);
    }
    GemmArgs g;
    memset(&g, 0, sizeof(g));
    g.A = A_ue; g.B = B_eu;
    g.C_fp = C_fp; g.ldc = ldc;
    g.scale_a_dev = scale_a_dev; g.scale_b_dev = scale_b_dev;
    g.refused = refused;
    if (p->nitems == 1 && fused_runs(p->pin_hdr[0]) <= 63) {  // a batch of one: the one-product kernel, its tables in the launch
        fused_args(g, p);
        g.guard = p->d_hdr->bound;
        return launch_fused(p, g, st);
    }
    g.sp_kt = -1;
    g.layA = p->layA; g.layB = p->layB;
    g.sh = p->sh;
    g.guard_mul = p->s - 1;
    g.hdr = p->d_hdr;
    g.a_stride = a_stride; g.b_stride = b_stride; g.c_stride = c_stride; g.plan_stride = p->item_bytes;
    g.scale_stride = scale_stride;
    if (small_tiles(p, tiles, pairs, ktiles)) return launch_small(p, g, grid * kChunkPairs, (int)ktiles, true, st);
    const dim3 blocks((unsigned)grid, (unsigned)p->nitems);
    if (p->fp6) hipLaunchKernelGGL(gemm_batch_kernel<true>, blocks, dim3(kGemmThreads), kGemmLds, st, g);
    else hipLaunchKernelGGL(gemm_batch_kernel<false>, blocks, dim3(kGemmThreads), kGemmLds, st, g);
    return launch_status();
}
}  // namespace imu

extern "C" int imunpack_gemm(imunpack_plan_t *p, const int8_t *A_ue, const int8_t *B_eu,
                             void *workspace, int64_t *C_int, float *C_fp, int64_t ldc, float scale_A,
                             float scale_B, int fuse, imunpack_stream_t stream) {
    return gemm_impl(p, A_ue, B_eu, workspace, C_int, C_fp, ldc, scale_A, scale_B, nullptr, nullptr, fuse, (hipStream_t)stream);
}

extern "C" int imunpack_diag_gemm_parts(const imunpack_plan_t *p) { return p ? p->gemm_parts : IMUNPACK_EINVAL; }

extern "C" int imunpack_diag_gemm_halves(const imunpack_plan_t *p) { return p ? p->gemm_halves : IMUNPACK_EINVAL; }

extern "C" int imunpack_diag_list_columns(const imunpack_plan_t *p) { return p && p->valid ? p->hdr.nsparse : IMUNPACK_EINVAL; }

extern "C" int imunpack_diag_clock_probe(uint64_t *ticks) {
    g_clock_probe.store(reinterpret_cast<unsigned long long *>(ticks), std::memory_order_relaxed);
    return IMUNPACK_OK;
}

extern "C" int imunpack_diag_mfma_peak(int workgroups, int iters, int64_t *ops, imunpack_stream_t stream) {
    if (workgroups <= 0 || workgroups > 65535 || iters <= 0 || iters > (1 << 24)) return IMUNPACK_EINVAL;
    hipLaunchKernelGGL(mfma_peak_kernel, dim3(workgroups), dim3(256), 0, (hipStream_t)stream, iters, (int *)nullptr);
    // 4 waves per workgroup, 8 MFMAs per iteration, 2 * 32 * 32 * 32 operations each
    if (ops) *ops = (int64_t)workgroups * 4 * (int64_t)iters * 8 * 65536;
    return launch_status();
}
