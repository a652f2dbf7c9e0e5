// Digit scatter (Sec. 4, Eq. (mod); Alg. 1 l.4-5, Alg. 2 l.4-6, Alg. 4 l.7-8 and 11-13): writes the
// unpacked int8 operands in the plan's physical layout, gathering from the int32 operands: B_eu in
// full, and of A_ue every column of A_u once (the copies that column unpacking of the partner asks
// for, Alg. 2 line 6 / Alg. 4 line 13, are not stored: the GEMM reads a stored column wherever a copy
// of it stands).  HBM-bound: 4 B read per source element, 1 B written per stored element.
//
// Where an entry's digits go.  A split of a row (column) keeps digit 0 of every entry of that row
// (column) in place and moves floor(v / s) to the appended row (column); a row or column is split
// at most once.  So the digits of the original entry (i, k) lie on a chain of positions: the
// remainder sitting at (R, C) moves to the child of R if R was split before C, to the child of C
// otherwise, and every other descendant position holds 0.
//   - An operand unpacked by UnpackRow or UnpackColumn splits along one axis only: position (R, C)
//     with row level eR and column level eC holds digit eR + eC of its entry.  scatter_kernel<true>
//     writes all of it.
//   - An operand unpacked by UnpackBoth holds digit 0 at the level-(0, 0) position of every entry and
//     0 elsewhere, except along the chains of its OB entries.  scatter_kernel<false> writes the
//     former, fixup_kernel then places the higher digits of the listed OB entries.
#include "common.h"

#include <type_traits>

#include <algorithm>
#include <chrono>
#include <cstddef>
#include <cstring>
#include <thread>

namespace imu {

// A wave writes kBandRows physical rows of one window of 64 output units (1024 stored columns): lane l
// owns unit l of the window.  Per row a lane reads the 16 source values of its unit (64 contiguous
// bytes when the unit copies 16 consecutive source columns, which the column layout makes the rule)
// and writes the unit's 16 bytes; the wave also leaves  sum_c w(c) |digit|  of what it wrote, its part
// of the row's weighted L1 norm.  The launch has exactly one wave per (band, window) of either
// operand, no empty workgroups, no staging and no barriers.  Short waves are what the memory system
// wants here: with two rows per wave (eight 16-byte loads per lane in flight, then out) the pass
// takes 0.10 ms on the benchmark workload, with 16 rows per wave (the unit's description decoded once
// for all of them) 0.17 ms, with 64 rows 0.42 ms; four rows at a time or one changed nothing.
constexpr int kScatterThreads = 256;
constexpr int kScatterWaves = kScatterThreads / 64;
constexpr int kBandRows = 2;  // divides kTile: the padded row counts are multiples of it
// Stores of at most 512 columns leave half of such a wave's lanes or more without a unit.  NARROW: 8, 16, 32 or 64 lanes to a band,
// as many as it has units for, and so up to eight bands to a wave (the two products of attention on 48 heads of 197 tokens,
// six-bit: 33 + 38 us with a wave to every band).
constexpr int kNarrow = 512;
__host__ __device__ inline int lg_band_lanes(int W) { return W <= 128 ? 3 : W <= 256 ? 4 : W <= 512 ? 5 : 6; }
__host__ __device__ inline int scatter_items(int rows, int W, bool narrow) {
    const int bands = rows / kBandRows;
    if (!narrow) return bands * ((W + 1023) / 1024);
    const int per = 64 >> lg_band_lanes(W);
    return (bands + per - 1) / per;
}

struct ScatterArgs {
    const int32_t *M;            // the int32 operand, row-major
    int64_t ldm;
    const int32_t *prow;         // per physical row
    const int32_t *col_k;        // per stored column: source column, -1 = none
    const int32_t *col_e;        // per stored column: digit level along this operand's column axis
    const unsigned long long *col_w;   // per stored column: weight in the row norm (nullptr: s^exponent of the unit)
    const int4 *unit;            // per 16 stored columns, see ColLayout
    const unsigned long long *unit_w;  // per unit: the weight its columns share (nullptr: s^exponent of the unit)
    int rows, W, ld, s, sh;      // physical rows, stored columns, bytes from one row of `out` to the next
    int nwin;                    // windows of 1024 stored columns
    int fp6;                     // store 6-bit floating-point codes (12 bytes per unit) instead of int8 digits
    int items;                   // waves that serve this operand
    int8_t *out;
    unsigned long long *wavesum; // [rows][nwin]: every wave leaves its part of the row norm
    // batch (blockIdx.y is the item): the sizes above differ from item to item and come from its header
    const PlanHeader *hdr;
    int op;                      // 0: A, 1: B
    int64_t m_stride, stride, out_stride;  // bytes from item to item: M, the plan's arrays, `out`
};

template <bool NARROW>
__device__ __forceinline__ void sizes_of_item(ScatterArgs &a) {
    if (!a.out) {  // nothing to do for this operand
        a.items = 0;
        return;
    }
    const PlanHeader &h = a.hdr[blockIdx.y];
    a.rows = a.op ? h.Np : h.Mp;
    a.W = a.op ? h.Kp : h.KA;
    a.ld = header_pitch(h, a.fp6, a.op);
    a.nwin = (a.W + 1023) / 1024;
    a.items = scatter_items(a.rows, a.W, NARROW);
}

typedef int v4i_u __attribute__((ext_vector_type(4), aligned(4)));  // 16 bytes at any int boundary

// Sign-magnitude digit at bit offset sft (`bits` wide) of four values, one per byte; mag += the four
// magnitudes.
__device__ __forceinline__ int digits4(const int (&x)[4], unsigned sft, int bits, unsigned &mag) {
    int dg[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int sx = x[i] >> 31;
        const unsigned av = (unsigned)((x[i] ^ sx) - sx);
        const int m = (int)__builtin_amdgcn_ubfe(av, sft, (unsigned)bits);
        mag += (unsigned)m;
        dg[i] = (m ^ sx) - sx;
    }
    return (int)(__builtin_amdgcn_perm((unsigned)dg[1], (unsigned)dg[0], 0x0c0c0400u) |
                 __builtin_amdgcn_perm((unsigned)dg[3], (unsigned)dg[2], 0x04000c0cu));
}

// Digit 0 of four values, on the four bytes at once.  With v = x mod s (the low bits of the two's
// complement), the sign-magnitude digit is v for x >= 0 and, for x < 0, 0 if v = 0 and v - s
// otherwise, which as a byte is v with the bits above the digit set.  mask4 = (s - 1) in every byte.
__device__ __forceinline__ int digit0x4(const int (&x)[4], unsigned mask4, unsigned &mag) {
    const unsigned l01 = __builtin_amdgcn_perm((unsigned)x[1], (unsigned)x[0], 0x07030400u);  // lo0 lo1 hi0 hi1
    const unsigned l23 = __builtin_amdgcn_perm((unsigned)x[3], (unsigned)x[2], 0x07030400u);
    const unsigned lo = __builtin_amdgcn_perm(l23, l01, 0x05040100u);  // the four low bytes
    const unsigned hi = __builtin_amdgcn_perm(l23, l01, 0x07060302u);  // the four high bytes (sign in bit 7)
    const unsigned v = lo & mask4;
    const unsigned nz = (v + 0x7f7f7f7fu) & 0x80808080u;              // bit 7: v != 0
    const unsigned t = hi & nz;                                        // bit 7: negative and v != 0
    const unsigned full = (t - (t >> 7)) | t;                          // 0xff in those bytes
    const unsigned r = v | (full & ~mask4);
    mag = __builtin_amdgcn_sad_u8(r ^ 0x80808080u, 0x80808080u, mag);  // sum of |int8|
    return (int)r;
}

// Four int8 digits in [-7, 7] (one per byte) -> their four e2m3 codes (one per byte): magnitudes 0..7 are
// 0, 1, 2, 1.5*2, 4, 1.25*4, 1.5*4, 1.75*4, i.e. the codes 0, 8, 16, 20, 24, 26, 28, 30; bit 5 is the sign.
__device__ __forceinline__ unsigned fp6_codes4(unsigned w) {
    const unsigned n = (w >> 7) & 0x01010101u;   // 1 in the negative bytes
    const unsigned s = (n << 8) - n;             // 0xff in the negative bytes
    const unsigned mag = (w ^ s) + n;            // |digit| per byte (no carries: every byte stays below 8)
    return __builtin_amdgcn_perm(0x1e1c1a18u, 0x14100800u, mag) | (n << 5);
}
// ... and squeezed to 24 bits, the first code lowest
__device__ __forceinline__ unsigned fp6_pack4(unsigned w) {
    const unsigned c = fp6_codes4(w);
    return (c & 0x3fu) | ((c >> 2) & 0xfc0u) | ((c >> 4) & 0x3f000u) | ((c >> 6) & 0xfc0000u);
}
typedef int v3i_u __attribute__((ext_vector_type(3), aligned(4)));
typedef int v2i_u __attribute__((ext_vector_type(2), aligned(4)));

__device__ __forceinline__ unsigned long long sat44(unsigned long long m, unsigned long long w) {
    if (m == 0) return 0;
    if (w >= (1ull << 44) || m >= (1ull << 20)) return 1ull << 44;
    const unsigned long long t = m * w;
    return t < (1ull << 44) ? t : (1ull << 44);
}

// One wave's work: band and window `item` of operand a (NARROW: the bands of group `item`).
template <bool DENSE, bool NARROW>
__device__ __forceinline__ void scatter_item(const ScatterArgs &a, int item, int lane) {
    const int nunits = a.W >> 4;
    const int lg = NARROW ? lg_band_lanes(a.W) : 6;
    const int band = NARROW ? (item << (6 - lg)) + (lane >> lg) : item / a.nwin, win = NARROW ? 0 : item - band * a.nwin;
    const int upos = NARROW ? lane & ((1 << lg) - 1) : win * 64 + lane;
    const bool there = !NARROW || band * kBandRows < a.rows;
    const bool inside = upos < nunits && there;
    const int4 ud = inside ? a.unit[upos] : make_int4(-1, -1, 7, 0);
    const int q0 = upos * 16;
    const int kfirst = ud.x, kany = ud.y;
    const bool run = (ud.z & 1) != 0, uniform = (ud.z & 2) != 0, onew = (ud.z & 4) != 0;
    const int ecu = ud.w & 0xFF;
    // what an entry of this unit weighs in the row norm: s^(exponent of S) for B_eu, the sum of those
    // over the column slots that read the stored column for A
    unsigned long long wgt = 0;
    if (inside && kany >= 0)
        wgt = a.unit_w ? a.unit_w[upos] : ((ud.w >> 16) * a.sh >= 44 ? (1ull << 44) : (1ull << ((ud.w >> 16) * a.sh)));
    const unsigned mask4 = (unsigned)(a.s - 1) * 0x01010101u;
    const int p_first = band * kBandRows;
    constexpr int RS = 2;  // rows per step
    for (int r0 = 0; r0 < kBandRows; r0 += RS) {
        int si[RS], er[RS];
        bool live[RS];
        int v[RS][4][4];
        // ---- both rows' loads first
#pragma unroll
        for (int h = 0; h < RS; ++h) {
            const int p = NARROW ? p_first + r0 + h : __builtin_amdgcn_readfirstlane(p_first + r0 + h);
            const int row = there ? a.prow[p] : -1;
            er[h] = row < 0 ? 0 : row >> kProwLevel;
            si[h] = row < 0 ? 0 : row & ((1 << kProwLevel) - 1);
            // padding row, padding unit, or (UnpackBoth operands hold digit 0 at level (0, 0) only; every
            // operand: no digit that high) a unit that holds nothing in this row
            const unsigned usft = (unsigned)(a.sh * (er[h] + ecu));
            live[h] = inside && row >= 0 && kany >= 0 && !(uniform && (DENSE ? usft >= 32u : er[h] + ecu != 0));

            if (live[h]) {
                const int32_t *src = a.M + (int64_t)si[h] * a.ldm;
                if (run) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const v4i_u x = *reinterpret_cast<const v4i_u *>(src + kfirst + 4 * j);
                        v[h][j][0] = x.x; v[h][j][1] = x.y; v[h][j][2] = x.z; v[h][j][3] = x.w;
                    }
                } else {  // gather through the column table
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int4 kk = *reinterpret_cast<const int4 *>(a.col_k + q0 + 4 * j);
                        v[h][j][0] = kk.x >= 0 ? src[kk.x] : 0;
                        v[h][j][1] = kk.y >= 0 ? src[kk.y] : 0;
                        v[h][j][2] = kk.z >= 0 ? src[kk.z] : 0;
                        v[h][j][3] = kk.w >= 0 ? src[kk.w] : 0;
                    }
                }
            }
        }
        // ---- digits, store, norm
#pragma unroll
        for (int h = 0; h < RS; ++h) {
            const int p = p_first + r0 + h;
            unsigned mag = 0;               // sum of |digit| over the unit (columns that share the weight wgt)
            unsigned long long wsum = 0;    // weighted sum, for units whose columns weigh differently
            int4 o = make_int4(0, 0, 0, 0);
            if (live[h]) {
                int pk[4];
                const unsigned usft = (unsigned)(a.sh * (er[h] + ecu));
                if (uniform) {
                    if (!DENSE || usft == 0u) {
#pragma unroll
                        for (int j = 0; j < 4; ++j) pk[j] = digit0x4(v[h][j], mask4, mag);
                    } else {
#pragma unroll
                        for (int j = 0; j < 4; ++j) pk[j] = digits4(v[h][j], usft, a.sh, mag);
                    }
                } else {  // a digit level per column
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int4 ee = *reinterpret_cast<const int4 *>(a.col_e + q0 + 4 * j);
                        const int ec[4] = {ee.x, ee.y, ee.z, ee.w};
                        pk[j] = 0;
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int level = er[h] + ec[i], x = v[h][j][i], sx = x >> 31;
                            const unsigned sft = (unsigned)(a.sh * level), av = (unsigned)((x ^ sx) - sx);
                            const int m = (DENSE ? sft < 32u : level == 0) ? (int)__builtin_amdgcn_ubfe(av, sft, (unsigned)a.sh) : 0;
                            mag += (unsigned)m;
                            pk[j] |= (((m ^ sx) - sx) & 0xFF) << (8 * i);
                        }
                    }
                }
                // A weight per column (columns of A that the partner repeats beside others that it does not): the digits are those already
                // made.  (Made once more, column by column, for the sake of the norm they kept a whole wave wherever one of its units is such:
                // 4096 x 4096 by 11008 86 -> 79 us, against resident weights 30 -> 19 and with 16 rows 12.5 -> 7, 1576 x 768 by 3072 21 -> 19.)
                if (!onew) {
                    mag = 0;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const ulonglong2 w01 = *reinterpret_cast<const ulonglong2 *>(a.col_w + q0 + 4 * j), w23 = *reinterpret_cast<const ulonglong2 *>(a.col_w + q0 + 4 * j + 2);
                        const unsigned long long w[4] = {w01.x, w01.y, w23.x, w23.y};
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int dg = (int8_t)(pk[j] >> (8 * i));
                            // (terms below 2^51, 1024 of them in a wave: no saturation before the sum is)
                            wsum += (unsigned long long)(unsigned)(dg < 0 ? -dg : dg) * min(w[i], 1ull << 44);
                        }
                    }
                }
                o = make_int4(pk[0], pk[1], pk[2], pk[3]);
            }
            if (inside) {
                if (a.fp6) {  // uniform: 16 digits -> 96 bits
                    const unsigned t0 = fp6_pack4((unsigned)o.x), t1 = fp6_pack4((unsigned)o.y), t2 = fp6_pack4((unsigned)o.z),
                                   t3 = fp6_pack4((unsigned)o.w);
                    // the unit is the lower or the upper half of a 32-column fragment (see fp6_dword in common.h)
                    const int d0 = (int)(t0 | (t1 << 24)), d1 = (int)((t1 >> 8) | (t2 << 16)), d2 = (int)((t2 >> 16) | (t3 << 8));
                    int8_t *row = a.out + fp6_ktile(p, upos >> 3, a.ld);
                    const int grp = (upos >> 2) & 1, frag = (upos >> 1) & 1;
                    if ((upos & 1) == 0) {
                        v3i_u w3;
                        w3.x = d0; w3.y = d1; w3.z = d2;
                        *reinterpret_cast<v3i_u *>(row + 4 * fp6_dword(p, grp, frag, 0)) = w3;
                    } else {
                        *reinterpret_cast<int *>(row + 4 * fp6_dword(p, grp, frag, 3)) = d0;
                        v2i_u w2;
                        w2.x = d1; w2.y = d2;
                        *reinterpret_cast<v2i_u *>(row + 4 * fp6_dword(p, grp, frag, 4)) = w2;
                    }
                    if ((p & 1) && upos >= 8 && (upos >> 3) % 2 == 0 && (upos >> 3) + 1 == a.W / kKPad) {  // the place of no k-tile
                        int *none = reinterpret_cast<int *>(a.out + (int64_t)p * a.ld + 12 * upos);  // (of this row and of the one before)
                        none[0] = none[1] = none[2] = 0;
                        none[24] = none[25] = none[26] = 0;
                    }
                } else {
                    *reinterpret_cast<int4 *>(a.out + i8_at(p, q0, a.ld)) = o;
                }
            }
            // ---- the wave's part of the row norm
            if constexpr (NARROW) {  // over the lanes of the band
                unsigned long long sum = wsum + sat44(mag, wgt);
                for (int off = 1; off < 1 << lg; off <<= 1) sum += (unsigned long long)__shfl_xor((long long)sum, off, 64);
                if (there && upos == 0) a.wavesum[p] = sum < (1ull << 44) ? sum : 1ull << 44;
                continue;
            }
            const unsigned long long nz = __ballot(mag != 0 || wsum != 0);
            unsigned long long total = 0;
            if (nz != 0) {
                const int first = __builtin_ctzll(nz);
                const unsigned wlo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)wgt, first);
                const unsigned whi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(wgt >> 32), first);
                const unsigned long long w1 = ((unsigned long long)whi << 32) | wlo;
                if (__all(wsum == 0 && (mag == 0 || wgt == w1))) {  // one weight: add the magnitudes, weigh once
                    total = sat44(wave_sum_lane63(mag), w1);  // lane 63 holds the sum
                } else {
                    total = wsum + sat44(mag, wgt);
#pragma unroll
                    for (int off = 32; off > 0; off >>= 1) total += (unsigned long long)__shfl_xor((long long)total, off, 64);
                    if (total > (1ull << 44)) total = 1ull << 44;  // every lane holds the sum
                }
            }
            if (lane == 63) a.wavesum[(int64_t)p * a.nwin + win] = total;
        }
    }
}

// Two operands in one launch when they take the same variant: waves below a0.items serve a0, the rest a1.
// (DENSE: eight waves a SIMD, 61 registers; left to itself it takes 76: 12608 x 768 by 3072 28 and 30 us.  The other kind reads less and
// computes less: held to 64 registers 4096 x 8192 by 4096 took 81 us instead of 76.)
template <bool DENSE, bool NARROW>
__global__ __launch_bounds__(kScatterThreads, DENSE ? 8 : 1) void scatter_kernel(ScatterArgs a0, ScatterArgs a1) {
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    int item = (int)blockIdx.x * kScatterWaves + wave;
    const bool second = item >= a0.items;
    const ScatterArgs &a = second ? a1 : a0;
    if (second) item -= a0.items;
    if (item >= a.items) return;  // uniform per wave; no barriers anywhere
    scatter_item<DENSE, NARROW>(a, item, (int)(threadIdx.x & 63));
}

// The same for the items of a batch, whose sizes come from their headers (a kernel of its own: the waves are too
// short to hide a further dependent read where it is not needed).
template <bool DENSE, bool NARROW>
__global__ __launch_bounds__(kScatterThreads, DENSE ? 8 : 1) void scatter_batch_kernel(ScatterArgs a0, ScatterArgs a1) {
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    int item = (int)blockIdx.x * kScatterWaves + wave;
    sizes_of_item<NARROW>(a0);
    sizes_of_item<NARROW>(a1);
    const bool second = item >= a0.items;
    ScatterArgs a = second ? a1 : a0;
    if (second) item -= a0.items;
    if (item >= a.items) return;
    const int64_t off = blockIdx.y * a.stride;
    a.M = item_at(a.M, blockIdx.y * a.m_stride);
    a.prow = item_at(a.prow, off);
    a.col_k = item_at(a.col_k, off); a.col_e = item_at(a.col_e, off); a.col_w = item_at(a.col_w, off);
    a.unit = item_at(a.unit, off); a.unit_w = item_at(a.unit_w, off);
    a.out = item_at(a.out, blockIdx.y * a.out_stride);
    a.wavesum = item_at(a.wavesum, off);
    scatter_item<DENSE, NARROW>(a, item, (int)(threadIdx.x & 63));
}

// Places the digits above digit 0 of the listed OB entries of an operand unpacked by UnpackBoth.
// (digits_above finds them.)
//   second == 0 (A): the entry's column chain lives in the column slots of A's unpacking; A_ue then
//     repeats column r of A_u in every column slot of the second unpacking that descends from r
//     (Alg. 2 line 6 / Alg. 4 line 13): the digit is stored wherever such a slot reads its column of A
//     (mostly one and the same stored column), and counts in the row norm once per such slot.
//   second == 1 (B): B_e holds a copy of column k of B in every column slot r of A's unpacking that
//     descends from k, and each copy is unpacked on its own.
struct FixupArgs {
    const int32_t *ob;          // [3][ob_cap] rows | columns | values
    int ob_cap;
    const PlanHeader *hdr;      // holds their number
    int batch;                  // blockIdx.y is the item of a batch: W comes from its header
    int64_t stride, out_stride; // bytes from item to item: the plan's arrays, `out`
    int second;
    SlotSet rows, cset;         // the operand's row slots and the column slots of its own unpacking
    const int32_t *c1_child;    // second == 1: child links among the column slots of A's unpacking
    const int32_t *c2_child;    // second == 0: child links among the column slots of the second unpacking
    const int32_t *row_phys;
    const int32_t *out_col;     // per column slot of the second unpacking: the stored column that holds it
    const int32_t *col_phys, *col_sexp;  // its column of B_eu, and per such column the exponent of S
    int W, sh;                  // bytes from one row of `out` to the next
    int fp6;                    // `out` holds 6-bit floating-point codes
    int8_t *out;
    unsigned long long *rowsum; // per physical row: what the digits placed here add to the row norm
};

// The whole norm of physical row p as far as it is known: the scatter kernel's parts plus `placed`.
__device__ __forceinline__ unsigned long long row_norm(const unsigned long long *wavesum, int wpr, int p,
                                                       unsigned long long placed) {
    unsigned long long t = placed;
    for (int w = 0; w < wpr; ++w) t += wavesum[(int64_t)p * wpr + w];
    return t < (1ull << 60) ? t : (1ull << 60);
}

// rowsum[p] += term for every lane that gets here together.  Atomics on one address are served one
// after the other, and the OB entries of a heavy row sit side by side in the list: in two rounds, the
// lanes that name the same row as the first lane still waiting are added up and share one atomic; the
// lanes left after that issue their own.
__device__ __forceinline__ void add_to_row(unsigned long long *rowsum, int p, unsigned long long term) {
    const int lane = threadIdx.x & 63;
    const int lo = (int)(unsigned)term, hi = (int)(unsigned)(term >> 32);
    unsigned long long pending = __ballot(1), sum = term;
    bool mine = true;  // this lane still has to issue its own atomic
    for (int round = 0; round < 2 && pending; ++round) {
        const int lead = __builtin_ctzll(pending);
        const int pl = __builtin_amdgcn_readlane(p, lead);
        const unsigned long long same = __ballot(mine && p == pl);
        if (same != (1ull << lead)) {  // uniform
            unsigned long long t = 0;
            for (unsigned long long m = same; m; m &= m - 1) {
                const int from = __builtin_ctzll(m);
                t += ((unsigned long long)(unsigned)__builtin_amdgcn_readlane(hi, from) << 32) |
                     (unsigned long long)(unsigned)__builtin_amdgcn_readlane(lo, from);
            }
            if (lane == lead) sum = t;
            else if (mine && p == pl) mine = false;  // carried by the leading lane
        }
        pending &= ~same;
    }
    if (mine) atomicAdd(&rowsum[p], sum);
}

// Both operands in one launch: blocks [0, blocks_a) serve fa, the next blocks_b serve fb.  What a digit
// placed here adds to its row's norm goes to rowsum; bound_kernel, launched behind this one, takes the
// largest norm (a wait for the sum inside this kernel, to keep the bound current entry by entry, was
// half its run time).
__global__ void fixup_kernel(FixupArgs fa, FixupArgs fb, int blocks_a, int blocks_b) {
    const bool first = (int)blockIdx.x < blocks_a;
    FixupArgs f = first ? fa : fb;
    const int block = first ? blockIdx.x : blockIdx.x - blocks_a;
    const int nblocks = first ? blocks_a : blocks_b;
    f.hdr += blockIdx.y;
    if (f.batch) {
        const int64_t off = blockIdx.y * f.stride;
        f.ob = item_at(f.ob, off);
        move_to_item(f.rows, off);
        move_to_item(f.cset, off);
        f.c1_child = item_at(f.c1_child, off); f.c2_child = item_at(f.c2_child, off);
        f.row_phys = item_at(f.row_phys, off); f.out_col = item_at(f.out_col, off);
        f.col_phys = item_at(f.col_phys, off); f.col_sexp = item_at(f.col_sexp, off);
        f.rowsum = item_at(f.rowsum, off);
        f.out = item_at(f.out, blockIdx.y * f.out_stride);
        f.W = header_pitch(*f.hdr, f.fp6, f.second);
    }
    const int n = min(f.second ? f.hdr->nobB : f.hdr->nobA, f.ob_cap);
    for (int t = block * blockDim.x + threadIdx.x; t < n; t += nblocks * blockDim.x) {
        const int i = f.ob[t], k = f.ob[f.ob_cap + t], v = f.ob[2 * (size_t)f.ob_cap + t];
        const unsigned av = v < 0 ? 0u - (unsigned)v : (unsigned)v;
        for (int croot = k, copies = 0; croot >= 0 && copies < 64; croot = f.second ? f.c1_child[croot] : -1, ++copies) {
            digits_above(f.rows, f.cset, i, croot, av, f.sh, [&](int R, int C, int m) {
                const int p = f.row_phys[R];
                const int8_t dg = (int8_t)(v < 0 ? -m : m);
                for (int c = C, hops = 0; c >= 0 && hops < 4096; c = f.second ? -1 : f.c2_child[c], ++hops) {
                    const int at = f.out_col[c];
                    if (f.fp6) {  // the position holds 0 (the scatter wrote it): OR the code in, 6 bits at bit 6 * column
                        const unsigned code = (fp6_codes4((unsigned)(uint8_t)dg) & 0x3fu);
                        const unsigned bit = 6u * (unsigned)(at & 31);  // inside the 32-column fragment
                        unsigned *row = reinterpret_cast<unsigned *>(f.out + fp6_ktile(p, at >> 7, f.W));
                        const int grp = (at >> 6) & 1, frag = (at >> 5) & 1, i = (int)(bit >> 5);
                        atomicOr(row + fp6_dword(p, grp, frag, i), code << (bit & 31u));
                        if ((bit & 31u) > 26u) atomicOr(row + fp6_dword(p, grp, frag, i + 1), code >> (32u - (bit & 31u)));
                    } else {
                        f.out[i8_at(p, at, f.W)] = dg;
                    }
                    const unsigned nsft = (unsigned)(f.sh * f.col_sexp[f.col_phys[c]]);
                    const unsigned long long term = nsft >= 40u ? (1ull << 44) : ((unsigned long long)m << nsft);
                    add_to_row(f.rowsum, p, term);
                }
            });
        }
    }
}

// The copy of level 0 of the A store that SparseLists describes, 128 x 128 at a time: 16 bytes a lane in, four rows by four columns a lane
// turned in registers, 16 bytes a lane (eight lanes to a line of 128 bytes) out.
struct TransposeArgs {
    const int8_t *A;   // the A store, ldA bytes from row to row
    int8_t *out;
    int ldA, d, blocks_k, blocks;  // blocks of 128 columns, blocks in all (0: nothing to do)
};
__device__ __forceinline__ void transpose_block(const TransposeArgs &t, int block, int8_t *lds /* 128 * kTrPitch */) {
    constexpr int kTrPitch = 132;
    const int g = block / t.blocks_k, k0 = (block - g * t.blocks_k) * 128, tid = threadIdx.x;
    int4 x[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)  // the stores' widths are multiples of 128
        x[u] = *reinterpret_cast<const int4 *>(t.A + i8_at(g * 128 + 32 * u + (tid >> 3), k0 + 16 * (tid & 7), t.ldA));
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        int *to = reinterpret_cast<int *>(lds + (32 * u + (tid >> 3)) * kTrPitch + 16 * (tid & 7));
        to[0] = x[u].x; to[1] = x[u].y; to[2] = x[u].z; to[3] = x[u].w;
    }
    __syncthreads();
    const int l4 = (tid & 7) * 4, kq = tid >> 3;  // rows l4 .. l4 + 3 of each block of 32, columns 4 kq .. 4 kq + 3
    unsigned o[4][4];                              // [column][row]
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        unsigned r[4];
#pragma unroll
        for (int rb = 0; rb < 4; ++rb) r[rb] = *reinterpret_cast<const unsigned *>(lds + (32 * rb + l4 + i) * kTrPitch + 4 * kq);
        const unsigned a = __builtin_amdgcn_perm(r[1], r[0], 0x05010400u), b = __builtin_amdgcn_perm(r[1], r[0], 0x07030602u);
        const unsigned c = __builtin_amdgcn_perm(r[3], r[2], 0x05010400u), e = __builtin_amdgcn_perm(r[3], r[2], 0x07030602u);
        o[0][i] = __builtin_amdgcn_perm(c, a, 0x05040100u);
        o[1][i] = __builtin_amdgcn_perm(c, a, 0x07060302u);
        o[2][i] = __builtin_amdgcn_perm(e, b, 0x05040100u);
        o[3][i] = __builtin_amdgcn_perm(e, b, 0x07060302u);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int k = k0 + 4 * kq + j;
        if (k < t.d) *reinterpret_cast<uint4 *>(t.out + ((int64_t)g * t.d + k) * 128 + 4 * l4) = make_uint4(o[j][0], o[j][1], o[j][2], o[j][3]);
    }
}

// The accumulator bounds: the largest row norm of either operand (the scatter kernel's parts per wave
// plus what the fix-up pass placed).  One update of the device's words per workgroup, and one pair of words per workgroup
// for the host.  (A step of 12608 x 768 by 3072: 248 us with the GEMM's first workgroup handing the bounds over, which the host
// could only wait for on the GEMM's stream; 235 us so.  256 x 256 x 256: 146 and 136.)
__global__ void bound_kernel(const unsigned long long *rowsum_a, const unsigned long long *wavesum_a, int rows_a,
                             unsigned long long *bound_a, const unsigned long long *rowsum_b,
                             const unsigned long long *wavesum_b, int rows_b, unsigned long long *bound_b, int wpr_a,
                             int wpr_b, const PlanHeader *hdr /* batch: the sizes come from the item's header */,
                             int64_t stride, unsigned long long *host /* nullptr: stay on the device */, int32_t seq,
                             int nscan /* workgroups behind these make the transposed copy */, TransposeArgs tr) {
    __shared__ __attribute__((aligned(16))) int8_t s_rows[128 * 132];
    if ((int)blockIdx.x >= nscan) {  // uniform
        transpose_block(tr, (int)blockIdx.x - nscan, s_rows);
        return;
    }
    unsigned long long *s_bound = reinterpret_cast<unsigned long long *>(s_rows);
    if (threadIdx.x < 2) s_bound[threadIdx.x] = 0;
    __syncthreads();
    unsigned long long ma = 0, mb = 0;
    if (hdr) {
        hdr += blockIdx.y;
        const int64_t off = blockIdx.y * stride, hoff = blockIdx.y * (int64_t)sizeof(PlanHeader);
        rowsum_a = item_at(rowsum_a, off); wavesum_a = item_at(wavesum_a, off); bound_a = item_at(bound_a, hoff);
        rowsum_b = item_at(rowsum_b, off); wavesum_b = item_at(wavesum_b, off); bound_b = item_at(bound_b, hoff);
        rows_a = hdr->Mp; rows_b = hdr->Np;
        wpr_a = (hdr->KA + 1023) / 1024; wpr_b = (hdr->Kp + 1023) / 1024;
    }
    for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < rows_a + rows_b; t += nscan * blockDim.x) {
        if (t < rows_a) ma = max(ma, row_norm(wavesum_a, wpr_a, t, rowsum_a[t]));
        else mb = max(mb, row_norm(wavesum_b, wpr_b, t - rows_a, rowsum_b[t - rows_a]));
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        ma = max(ma, (unsigned long long)__shfl_xor((long long)ma, off, 64));
        mb = max(mb, (unsigned long long)__shfl_xor((long long)mb, off, 64));
    }
    if ((threadIdx.x & 63) == 0) {
        atomicMax(&s_bound[0], ma);
        atomicMax(&s_bound[1], mb);
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        const unsigned long long m = s_bound[threadIdx.x];
        unsigned long long *bound = threadIdx.x ? bound_b : bound_a;
        // the bound only grows: a plain (possibly stale) read filters most of the updates
        if (m > __hip_atomic_load(bound, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(bound, m);
        if (host) tell_bound(host + 2 * blockIdx.x + threadIdx.x, m, seq);
    }
}

// A repeated unpack of one plan: clears what the planner left cleared for the first.
__global__ void reset_bound_kernel(PlanHeader *hdr, unsigned long long *rowsum_a, int rows_a,
                                   unsigned long long *rowsum_b, int rows_b) {
    const int t0 = blockIdx.x * blockDim.x + threadIdx.x, stride = gridDim.x * blockDim.x;
    if (t0 == 0) hdr->bound[0] = hdr->bound[1] = 0;
    for (int t = t0; t < rows_a; t += stride) rowsum_a[t] = 0;
    for (int t = t0; t < rows_b; t += stride) rowsum_b[t] = 0;
}

// canon[R][c] = phys[row_phys[R]][col_phys[c]]; ld: bytes from one physical row to the next
__global__ void canonical_kernel(const int8_t *__restrict__ phys, int ld, const int32_t *row_phys,
                                 const int32_t *col_phys, int nrows, int ncols, int8_t *__restrict__ canon, int fp6) {
    const int R = blockIdx.x;
    if (R >= nrows) return;
    for (int c = threadIdx.x; c < ncols; c += blockDim.x) {
        int8_t v;
        if (fp6) {  // e2m3 code at bit 6 * column -> the integer it stands for (digits are integers)
            const int col = col_phys[c];
            const unsigned bit = 6u * (unsigned)(col & 31);
            const int pr = row_phys[R];
            const unsigned *row = reinterpret_cast<const unsigned *>(phys + fp6_ktile(pr, col >> 7, ld));
            const int grp = (col >> 6) & 1, frag = (col >> 5) & 1, i = (int)(bit >> 5);
            unsigned long long two = row[fp6_dword(pr, grp, frag, i)];
            if ((bit & 31u) > 26u) two |= (unsigned long long)row[fp6_dword(pr, grp, frag, i + 1)] << 32;
            const unsigned code = (unsigned)(two >> (bit & 31u)) & 0x3fu;
            const unsigned e = (code >> 3) & 3u, m = code & 7u;
            const unsigned eighths = e == 0 ? m : ((8u + m) << (e - 1));   // value * 8
            const int mag = (int)(eighths >> 3);
            v = (int8_t)((code & 32u) ? -mag : mag);
        } else {
            v = phys[i8_at(row_phys[R], col_phys[c], ld)];
        }
        canon[(int64_t)R * ncols + c] = v;
    }
}

}  // namespace imu

using namespace imu;

extern "C" int imunpack_unpacked_bytes(const imunpack_plan_t *p, size_t *bytes_A, size_t *bytes_B,
                                       size_t *bytes_workspace) {
    if (!p || !p->valid) return IMUNPACK_EINVAL;
    if (bytes_A) *bytes_A = (size_t)p->hdr.Mp * (size_t)store_pitch(p, 0);
    if (bytes_B) *bytes_B = (size_t)p->hdr.Np * (size_t)store_pitch(p, 1);
    if (bytes_workspace) *bytes_workspace = (size_t)p->hdr.Mp * p->hdr.Np * sizeof(int64_t);
    return IMUNPACK_OK;
}

extern "C" int imunpack_plan_set_digits(imunpack_plan_t *p, int format) {
    if (!p || !p->valid || (format != IMUNPACK_DIGITS_INT8 && format != IMUNPACK_DIGITS_FP6)) return IMUNPACK_EINVAL;
    if (format == IMUNPACK_DIGITS_FP6 && p->b > 4) return IMUNPACK_EINVAL;
    if (p->bound_pending) IMU_TRY(resolve_bound(p));  // of an unpack in the other format
    p->digits_req = format;
    p->fp6 = format == IMUNPACK_DIGITS_FP6;
    p->kept_Beu = nullptr;
    return IMUNPACK_OK;
}

extern "C" int imunpack_plan_digits(const imunpack_plan_t *p) {
    return (p && p->valid && p->fp6) ? IMUNPACK_DIGITS_FP6 : IMUNPACK_DIGITS_INT8;
}

extern "C" int imunpack_plan_layout(const imunpack_plan_t *p, int64_t *shape) {
    if (!p || !p->valid || !shape) return IMUNPACK_EINVAL;
    const int64_t v[6] = {p->hdr.Mp, p->hdr.KA, store_pitch(p, 0), p->hdr.Np, p->hdr.Kp, store_pitch(p, 1)};
    memcpy(shape, v, sizeof(v));
    return IMUNPACK_OK;
}

// The scatter of one plan, or of every item of a batch (nitems > 1: the stores of item i lie i * a_stride and
// i * b_stride bytes behind those of item 0).  With a_stride != 0 the bounds stay on the device, where
// gemm_batch checks them.
int imu::unpack_impl(imunpack_plan_t *p, const int32_t *A, int64_t lda, const int32_t *B, int64_t ldb, int8_t *A_ue,
                     int64_t a_stride, int8_t *B_eu, int64_t b_stride, hipStream_t st) {
    if (!p || !p->valid || !A || !B || !A_ue || !B_eu || lda < p->d || ldb < p->d) return IMUNPACK_EINVAL;
    const PlanHeader &h = p->hdr;
    const bool batch = p->nitems > 1;
    const unsigned nitems = (unsigned)p->nitems;
    p->bound_pending = 0;
    p->fusable = 0;  // until the bounds say otherwise
    // keep-weights mode: the plan took the second operand's unpacking over, and the caller's buffer still holds
    // what the unpack before wrote for exactly that unpacking (same buffer, same format, row norms in place)
    const bool keepB = p->keep_B && h.reusedB && !p->unpacked && p->kept_Beu == B_eu && p->kept_Beu_fp6 == p->fp6;
    // the planner leaves the bounds and the row norms cleared, but for the norms of an unpacking it took over; a repeated
    // unpack of the same plan clears them again, and so does every replay of a graph that holds one
    auto clear = [&]() {
        hipLaunchKernelGGL(reset_bound_kernel, dim3(64), dim3(256), 0, st, p->d_hdr, p->layA.rowsum, h.Mp,
                           p->layB.rowsum, keepB ? 0 : h.Np);
    };
    const bool again = p->unpacked || (h.reusedB && !keepB);
    if (again && batch) return IMUNPACK_EINVAL;
    if (again) clear();
    FixupArgs fx[2] = {};
    int fblocks[2] = {0, 0};
    ScatterArgs sc[2];
    memset(sc, 0, sizeof(sc));
    bool launch[2] = {false, false}, dense[2] = {false, false};
    int most_rows = 0;  // physical rows of both operands, in the largest item
    int least = 1 << 30, widest = 0;  // stored columns of either operand
    for (unsigned i = 0; i < nitems; ++i) {
        const PlanHeader &hi = batch ? p->pin_hdr[i] : h;
        least = std::min(least, std::min((int)hi.Kp, (int)hi.KA));
        widest = std::max(widest, std::max((int)hi.Kp, (int)hi.KA));
    }
    const bool narrow = least <= kNarrow && widest <= 1024;
    for (int op = 0; op < 2; ++op) {
        const RowLayout &lay = op ? p->layB : p->layA;
        const bool both = (op ? p->sB : p->sA) == IMUNPACK_BOTH;
        ScatterArgs &a = sc[op];
        a.M = op ? B : A; a.ldm = op ? ldb : lda;
        a.prow = lay.prow;
        a.col_k = op ? p->cols.colB_k : p->cols.colA_k;
        a.col_e = op ? p->cols.colB_e : p->cols.colA_e;
        a.col_w = op ? nullptr : p->cols.colA_w;
        a.unit = op ? p->cols.unitB : p->cols.unitA;
        a.unit_w = op ? nullptr : p->cols.unitA_w;
        a.s = p->s; a.sh = p->sh; a.fp6 = p->fp6;
        a.op = op;
        a.hdr = batch ? p->d_hdr : nullptr;
        a.m_stride = p->op_stride; a.stride = p->item_bytes; a.out_stride = op ? b_stride : a_stride;
        a.rows = op ? h.Np : h.Mp; a.W = op ? h.Kp : h.KA; a.ld = (int)store_pitch(p, op);
        a.nwin = (a.W + 1023) / 1024;
        int nob = 0;
        for (unsigned i = 0; i < nitems; ++i) {  // the launch covers the largest item
            const PlanHeader &hi = batch ? p->pin_hdr[i] : h;
            a.items = std::max(a.items, scatter_items(op ? hi.Np : hi.Mp, op ? hi.Kp : hi.KA, narrow));
            nob = std::max(nob, (int)(op ? hi.nobB : hi.nobA));
            most_rows = std::max(most_rows, hi.Mp + hi.Np);
        }
        a.out = op ? B_eu : A_ue;
        a.wavesum = lay.wavesum;
        launch[op] = a.items > 0 && !(op == 1 && keepB);
        dense[op] = !both;
        if (both && nob > 0 && launch[op]) {
            FixupArgs &f = fx[op];
            f.ob = op ? p->obcopyB : p->obcopyA;
            f.ob_cap = p->cap[op ? CAP_EDGEB : CAP_EDGEA];
            f.hdr = p->d_hdr;
            f.batch = batch; f.stride = p->item_bytes; f.out_stride = a.out_stride;
            f.second = op;
            f.rows = op ? p->rowB : p->rowA;
            f.cset = op ? p->c2 : p->c1;
            f.c1_child = p->c1.child;
            f.c2_child = p->c2.child;
            f.row_phys = lay.row_phys;
            f.out_col = op ? p->cols.col_phys : p->cols.acol_phys;
            f.col_phys = p->cols.col_phys; f.col_sexp = p->cols.col_sexp;
            f.W = a.ld; f.sh = p->sh; f.fp6 = p->fp6;
            f.out = a.out; f.rowsum = lay.rowsum;
            fblocks[op] = (nob + 255) / 256;
        }
    }
    auto scatter = [&](const ScatterArgs &x, const ScatterArgs &y, int items, bool dns) {
        const dim3 grid((unsigned)((items + kScatterWaves - 1) / kScatterWaves), nitems);
        auto go = [&](auto dense_c, auto narrow_c) {
            constexpr bool D = decltype(dense_c)::value, N = decltype(narrow_c)::value;
            if (batch) hipLaunchKernelGGL((scatter_batch_kernel<D, N>), grid, dim3(kScatterThreads), 0, st, x, y);
            else hipLaunchKernelGGL((scatter_kernel<D, N>), grid, dim3(kScatterThreads), 0, st, x, y);
        };
        if (dns && narrow) go(std::true_type{}, std::true_type{});
        else if (dns) go(std::true_type{}, std::false_type{});
        else if (narrow) go(std::false_type{}, std::true_type{});
        else go(std::false_type{}, std::false_type{});
    };
    ScatterArgs none;
    memset(&none, 0, sizeof(none));
    if (launch[0] && launch[1] && dense[0] == dense[1]) {  // one launch: the tail of A overlaps the head of B
        scatter(sc[0], sc[1], sc[0].items + sc[1].items, dense[0]);
    } else {
        for (int op = 0; op < 2; ++op)
            if (launch[op]) scatter(sc[op], none, sc[op].items, dense[op]);
    }
    // (asked while the scatter, which does not touch the norms, is under way)
    const bool graph = a_stride == 0 && capturing(st);
    if (graph && !again) clear();
    if (most_rows > 0) {
        // after both scatters: the fix-up overwrites zeros they wrote; then the bounds from the row norms
        if (fblocks[0] + fblocks[1] > 0) {
            if (!fblocks[0]) fx[0] = fx[1];  // never dereferenced, but keep the argument well-formed
            if (!fblocks[1]) fx[1] = fx[0];
            hipLaunchKernelGGL(fixup_kernel, dim3(fblocks[0] + fblocks[1], nitems), dim3(256), 0, st, fx[0], fx[1], fblocks[0],
                               fblocks[1]);
        }
        const int nscan = std::min(kBoundBlocks, (most_rows + 255) / 256);
        // a workgroup hands what it found to the host itself, in words of its own: the host needs no stream (the caller may use
        // another for the GEMM, or destroy this one) and no event to learn the bounds, and no workgroup waits for another.  Not
        // from a graph, whose replays nobody waits for.
        p->bound_words = a_stride || graph ? 0 : 2 * nscan;
        p->bound_seq = ++p->seq;
        for (int i = 0; i < p->bound_words; ++i)  // not there yet
            __atomic_store_n(&p->pin_bounds[i], (unsigned long long)(uint16_t)~p->bound_seq << 48, __ATOMIC_RELEASE);
        TransposeArgs tr = {A_ue, p->at, sc[0].ld, (int)p->d, (int)((p->d + 127) / 128), 0};
        if (h.nsparse) tr.blocks = h.Mp / 128 * tr.blocks_k;
        hipLaunchKernelGGL(bound_kernel, dim3(nscan + tr.blocks, nitems), dim3(256), 0, st, p->layA.rowsum, p->layA.wavesum, h.Mp,
                           &p->d_hdr->bound[0], p->layB.rowsum, p->layB.wavesum, h.Np, &p->d_hdr->bound[1],
                           sc[0].nwin, sc[1].nwin, batch ? p->d_hdr : nullptr, p->item_bytes,
                           p->bound_words ? p->pin_bounds : nullptr, p->bound_seq, nscan, tr);
    }
    IMU_TRY(launch_status());
    p->unpacked = 1;
    if (a_stride) return IMUNPACK_OK;
    p->bound_pending = 1;
    p->kept_Beu = p->keep_B ? B_eu : nullptr;
    p->kept_Beu_fp6 = p->fp6;
    return IMUNPACK_OK;
}

extern "C" int imunpack_unpack(imunpack_plan_t *p, const int32_t *A, int64_t lda, const int32_t *B,
                               int64_t ldb, int8_t *A_ue, int8_t *B_eu, imunpack_stream_t stream) {
    return unpack_impl(p, A, lda, B, ldb, A_ue, 0, B_eu, 0, (hipStream_t)stream);
}

namespace imu {
int resolve_bound(Plan *p) {
    if (!p->bound_pending) return IMUNPACK_OK;
    unsigned long long bound[2] = {0, 0};
    if (p->bound_words == 0) {  // a captured unpack: nobody knows on which stream its graph ran
        IMU_HIP(hipDeviceSynchronize());
        IMU_HIP(hipMemcpy(bound, p->d_hdr->bound, sizeof(bound), hipMemcpyDeviceToHost));
    }
    long spin = 0;
    for (int i = 0; i < p->bound_words; ++i) {  // the upper sixteen bits name the unpack
        unsigned long long w;
        while ((w = __atomic_load_n(&p->pin_bounds[i], __ATOMIC_ACQUIRE)) >> 48 != (uint16_t)p->bound_seq) {
            if (++spin < (1 << 24)) continue;
            // queued behind a lot of other work; if some ten seconds do not bring it, look whether it comes at all
            if (spin < (1 << 24) + 150000) {
                std::this_thread::sleep_for(std::chrono::microseconds(20));
                continue;
            }
            IMU_HIP(hipDeviceSynchronize());
            if (__atomic_load_n(&p->pin_bounds[i], __ATOMIC_ACQUIRE) >> 48 != (uint16_t)p->bound_seq) return IMUNPACK_EHIP;
        }
        bound[i & 1] = std::max(bound[i & 1], w & ((1ull << 48) - 1));
    }
    p->hdr.bound[0] = bound[0];
    p->hdr.bound[1] = bound[1];
    p->bound_pending = 0;
    // |sum_c s^e(c) a_c b_c| <= (s - 1) * min(bound_A, bound_B): the shifted sum of all groups
    // fits int32 iff that is below 2^31.
    const unsigned long long m = p->hdr.bound[0] < p->hdr.bound[1] ? p->hdr.bound[0] : p->hdr.bound[1];
    // (6-bit floating-point digits accumulate in binary32: exact below 2^24)
    p->fusable = (m < (1ull << 40)) && (m * (unsigned long long)(p->s - 1) < (1ull << (p->fp6 ? 24 : 31)));
    p->guess_fusable = p->fusable;
    return IMUNPACK_OK;
}
}  // namespace imu

extern "C" int imunpack_plan_fusable(imunpack_plan_t *p) {
    if (!p || !p->valid || !p->unpacked) return 0;
    if (resolve_bound(p) != IMUNPACK_OK) return 0;
    return p->fusable;
}

extern "C" int imunpack_plan_bounds(imunpack_plan_t *p, uint64_t *bound) {
    if (!p || !p->valid || !p->unpacked || !bound) return IMUNPACK_EINVAL;
    IMU_TRY(resolve_bound(p));
    bound[0] = p->hdr.bound[0];
    bound[1] = p->hdr.bound[1];
    return IMUNPACK_OK;
}

namespace imu { int ensure_canonical(Plan *p); }

extern "C" int imunpack_unpack_canonical(imunpack_plan_t *p, const int8_t *A_ue, const int8_t *B_eu,
                                         int8_t *A_canon, int8_t *B_canon, imunpack_stream_t stream) {
    if (!p || !p->valid) return IMUNPACK_EINVAL;
    IMU_TRY(ensure_canonical(p));  // host-side renumbering into the paper's order (synchronises)
    hipStream_t st = (hipStream_t)stream;
    const PlanHeader &h = p->hdr;
    if (A_ue && A_canon && h.n_u > 0)
        hipLaunchKernelGGL(canonical_kernel, dim3(h.n_u), dim3(256), 0, st, A_ue, (int)store_pitch(p, 0), p->canon_rowphysA,
                           p->canon_acolphys, h.n_u, h.d_u, A_canon, p->fp6);
    if (B_eu && B_canon && h.h_u > 0)
        hipLaunchKernelGGL(canonical_kernel, dim3(h.h_u), dim3(256), 0, st, B_eu, (int)store_pitch(p, 1), p->canon_rowphysB,
                           p->canon_colphys, h.h_u, h.d_u, B_canon, p->fp6);
    return launch_status();
}
