// alpha_p(A) of Sec. 2 (the sentence after Eq. (quantized_A)): the p-th percentile of the magnitudes
// of a matrix, i.e. the smallest magnitude a such that at least p % of the entries lie in [-a, a].
// That is an order statistic: the k-th smallest |x| with k = ceil(p N / 100).
//
// The magnitude of a binary32 number, read as a 31-bit unsigned integer, orders like the magnitude
// itself, so the k-th smallest is found by a radix select over those integers.
//
// Up to kSmall entries: one workgroup holds the whole matrix in registers and selects there, one launch.
//
// More: one workgroup first selects two ranks of a random sample that enclose the wanted one (five standard
// deviations of the sample's rank and a little to either side), which leaves a window of a few per cent of the
// entries (3.6 at p = 95).  Two passes over the matrix then count the entries below the window and, per value of the
// next 11 (10) bits inside it, the entries in it (a histogram in LDS per workgroup, merged with one atomic per
// non-empty bin); a workgroup finds the bin that the pass before it narrowed the window to by itself, from the
// merged histogram.  A window of more than 2^21 values (normal entries at p = 95: every other time; heavy tails: always) takes
// a third pass of 10 bits; a window that missed (the sample was that unlucky) is left to one workgroup's own radix select over
// the whole matrix.
// The passes are bound by reading the matrix: with the window, few entries go to the histogram.  Three
// passes with a histogram of every entry, each followed by a launch that picked the bin, took 53 us each
// on 11008 x 4096 (180 MB), 3.4 TB/s, 175 us in all; now 9 us for the sample, 34 and 31 us for the passes (5.4 TB/s) and 5 us
// for the launch that closes: 79, or 108 with the third pass.  Everything stays on the stream; the caller reads *alpha when it
// needs the number.
#include "common.h"

#include <algorithm>
#include <cmath>
#include <mutex>

namespace imu {

constexpr int kSelThreads = 1024;
constexpr int kHold = 48;                          // entries a thread of the one-workgroup selection holds, at most
constexpr int64_t kSmall = kSelThreads * kHold;
constexpr int kSample = 4096;                      // entries of the sample
constexpr int kItems = 8;                          // 16-byte pieces per thread and step, loaded side by side
// Bins of the three passes: together they tell all 2^31 magnitudes apart, whatever the window (no workgroup is ever left to
// finish alone: the last bit of the window above the 99.9th percentile of 8192 x 8190 weights took it 6.8 ms).  The first pass
// needs no more than 2041: (infinity's bit pattern >> 20) + 1.
constexpr int kBins0 = 2041, kBins1 = 1024, kBins2 = 1024;
constexpr unsigned kInf = 0x7f800000u;             // above it: NaN

// What the launches of one selection leave each other: the words between the first pass's histogram and the second's.
struct SelState {
    unsigned lo, top;             // the window [lo, lo + top]
    unsigned below;               // entries below it (first pass)
    unsigned maxbits;             // largest magnitude (as its bit pattern; a NaN's is beyond infinity's)
    unsigned base1, k1;           // the second pass's window and the rank wanted inside it
    unsigned after;               // after the first pass: kFound: base1 is the answer, kMissed: the rank was outside the
                                  // window, else the second pass's bin width << 16; below them the workgroups of the third pass that are done
};
constexpr unsigned kFound = 1u << 30, kMissed = 1u << 31;
constexpr int kState0 = kBins0, kHist1 = kState0 + (int)(sizeof(SelState) / sizeof(unsigned)), kHist2 = kHist1 + kBins1;
constexpr int kSelWords = kHist2 + kBins2;
static_assert(IMUNPACK_PERCENTILE_WORKSPACE_BYTES >= kSelWords * sizeof(unsigned), "workspace");
// the first pass's bin width (as a shift) for a window of top + 1 values: the smallest that kBins0 bins cover it with
__device__ __forceinline__ unsigned sel_shift0(unsigned top) {
    unsigned s = top >= 2048u ? 32 - __clz(top) - 11 : 0;
    return (top >> s) < (unsigned)kBins0 ? s : s + 1;
}

// One matrix: nslow lines of nfast entries, entry (l, f) at X[l * sslow + f * sfast].
struct SelOperand {
    const float *X;
    int64_t sslow, sfast;
    unsigned N, nfast;
    unsigned long long magic;     // e / nfast = mulhi(e, magic) (nfast > 1)
    int kind;                     // 0: contiguous, 1: contiguous lines of a multiple of four entries, 2: any
    unsigned k;                   // rank wanted (1-based)
    unsigned m, rlo, rhi;         // sample size and the ranks in it that enclose the wanted one (0 / > m: open end)
    void *ws;
    float *out;                   // alpha, or
    float half_beta;              // > 0: the RTN step alpha / half_beta
    int32_t *status;              // set to 1 if there is a NaN ...
    int clear_status;             // ... and to 0 if not (otherwise only ever set)
    int64_t x_stride;             // bytes from item to item of a batch
};
// blockIdx.y: the items of the first matrix's batch, then those of the second's.
struct SelArgs {
    SelOperand op[2];
    int nitems;
    int64_t out_stride;           // bytes from item to item: workspace and result
};

__device__ __forceinline__ SelOperand sel_operand(const SelArgs &a) {
    const bool second = (int)blockIdx.y >= a.nitems;
    SelOperand o = second ? a.op[1] : a.op[0];
    const int64_t item = (int)blockIdx.y - (second ? a.nitems : 0);
    o.X = item_at(o.X, item * o.x_stride);
    o.ws = item_at(o.ws, item * a.out_stride);
    o.out = item_at(o.out, item * a.out_stride);
    return o;
}
__device__ __forceinline__ unsigned *sel_hist(void *ws) { return reinterpret_cast<unsigned *>(ws); }
__device__ __forceinline__ SelState *sel_state(void *ws) {
    return reinterpret_cast<SelState *>(reinterpret_cast<unsigned *>(ws) + kState0);
}
__device__ __forceinline__ unsigned sel_line(const SelOperand &o, unsigned e) {
    return o.nfast > 1 ? (unsigned)__umul64hi(e, o.magic) : e;
}
__device__ __forceinline__ float sel_entry(const SelOperand &o, unsigned e) {
    if (o.kind == 0) return o.X[e];
    const unsigned l = sel_line(o, e);
    return o.X[(int64_t)l * o.sslow + (int64_t)(e - l * o.nfast) * o.sfast];
}

// One more in a bin of a histogram in LDS.  `crowded`: lanes that name the bin of the first of them share an update, for
// matrices that are full of one value (zeros behind a ReLU, ones), of which a wave would queue up 64.  (Where values
// differ it costs 5 of 24 us, so the callers look first.)
__device__ __forceinline__ void sel_count(unsigned *hist, unsigned bin, bool crowded) {
    if (!crowded) {
        atomicAdd(&hist[bin], 1u);
        return;
    }
    const unsigned first = __builtin_amdgcn_readfirstlane(bin);
    const unsigned long long same = __ballot(bin == first);
    if (bin != first) atomicAdd(&hist[bin], 1u);
    else if ((int)(threadIdx.x & 63) == __builtin_ctzll(same)) atomicAdd(&hist[first], (unsigned)__popcll(same));
}

// Workgroup-wide: the bin of hist[0..nbins) in which the cumulative count reaches k (1-based) and the count
// before it.  Returns false (for every thread) if the total is below k or k is 0.  lds: 20 words.
__device__ __forceinline__ bool sel_pick(const unsigned *hist, int nbins, unsigned k, unsigned &bin, unsigned &before,
                                         unsigned *lds) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int b0 = 2 * (int)threadIdx.x;  // two bins per thread
    const unsigned c0 = b0 < nbins ? hist[b0] : 0u, c1 = b0 + 1 < nbins ? hist[b0 + 1] : 0u;
    const unsigned incl = (unsigned)wave_inclusive_sum((int)(c0 + c1));
    __syncthreads();  // earlier uses of lds
    if (lane == 63) lds[wave] = incl;
    if (threadIdx.x == 0) lds[16] = 0xffffffffu;
    __syncthreads();
    unsigned run = incl - (c0 + c1);
#pragma unroll
    for (int w = 0; w < kSelThreads / 64 - 1; ++w) {  // all read at once, not one behind the other
        const unsigned c = lds[w];
        if (w < wave) run += c;
    }
    if (k > run && k <= run + c0 + c1) {  // at most one thread
        const bool first = k <= run + c0;
        lds[16] = (unsigned)b0 + (first ? 0u : 1u);
        lds[17] = first ? run : run + c0;
    }
    __syncthreads();
    bin = lds[16];
    before = lds[17];
    return bin != 0xffffffffu;
}

// The result: alpha, or the RTN step of Eq. (quantized_A) formed once in binary32: beta integers cover
// [-alpha_p, alpha_p], so one step is alpha_p / (0.5 beta).  A matrix whose p-th percentile is 0 (mostly
// zeros) falls back to its largest magnitude, an all-zero (or non-finite) one to 1.
__device__ __forceinline__ void sel_result(const SelOperand &o, unsigned alpha_bits, unsigned maxbits) {
    float a = __uint_as_float(alpha_bits);
    if (o.half_beta > 0.0f) {
        if (!(a > 0.0f)) a = __uint_as_float(maxbits);
        a = (a > 0.0f && a < __uint_as_float(kInf)) ? __fdiv_rn(a, o.half_beta) : 1.0f;
    }
    *o.out = a;
}

// ---- one workgroup: the whole matrix if it is small, else the sample -------------------------------------
// HOLD entries per thread, loaded in one straight line: with a branch (on the count, on the strides) around every
// load the compiler waits for each before the next, 20 us for the 13 of a 197 x 64 matrix
// (96 of them side by side: 27 -> 12 us for the whole kernel).
template <int HOLD>
__global__ __launch_bounds__(kSelThreads) void select_small_kernel(SelArgs args) {
    __shared__ unsigned hist[2][2048];
    __shared__ unsigned lds[20], s_max, s_nan;
    const SelOperand o = sel_operand(args);
    const bool whole = o.N <= (unsigned)kSmall;
    const unsigned count = whole ? o.N : o.m;
    unsigned u[HOLD];
    unsigned umax = 0;
    auto entry = [&](int j) {
        unsigned i = min(threadIdx.x + (unsigned)(j * kSelThreads), count - 1u);
        // a random entry per sample (a multiplicative hash of its number, so that no row or column pitch can
        // line up with the choice)
        unsigned x = i * 0x9e3779b1u + 0x7f4a7c15u;
        x = (x ^ (x >> 15)) * 0x85ebca77u;
        x = (x ^ (x >> 13)) * 0xc2b2ae3du;
        return whole ? i : __umulhi(x ^ (x >> 16), o.N);
    };
    if (o.kind == 0) {
#pragma unroll
        for (int j = 0; j < HOLD; ++j) u[j] = __float_as_uint(o.X[entry(j)]);
    } else {
        const unsigned long long magic = o.nfast > 1 ? o.magic : 0ull;
        const unsigned one = o.nfast > 1 ? 0u : 0xffffffffu;  // lines of one entry: the line is the entry's number
#pragma unroll
        for (int j = 0; j < HOLD; ++j) {
            const unsigned e = entry(j), l = (unsigned)__umul64hi(e, magic) | (e & one);
            u[j] = __float_as_uint(o.X[(int64_t)l * o.sslow + (int64_t)(e - l * o.nfast) * o.sfast]);
        }
    }
#pragma unroll
    for (int j = 0; j < HOLD; ++j) {
        if (threadIdx.x + (unsigned)(j * kSelThreads) < count) {
            u[j] &= 0x7fffffffu;
            umax = max(umax, u[j]);
        } else {
            u[j] = 0xffffffffu;  // absent
        }
    }
    for (int i = threadIdx.x; i < 2 * 2048; i += kSelThreads) (&hist[0][0])[i] = 0;
    if (threadIdx.x == 0) s_max = 0;
    if (!whole) {  // a clean workspace for the passes
        unsigned *w = sel_hist(o.ws);
        for (int i = threadIdx.x; i < kSelWords; i += kSelThreads) w[i] = 0;
        if (threadIdx.x == 0 && o.status && o.clear_status) *o.status = 0;
    }
    __syncthreads();
    umax = (unsigned)wave_max_nonneg_lane63((int)umax);
    if ((threadIdx.x & 63) == 63) atomicMax(&s_max, umax);
    // digits of 11, 10 and 10 bits, most significant first; ranks r[0] (and, for the sample, r[1]).  The sample's
    // window ends need no last digit.
    unsigned r[2] = {whole ? o.k : o.rlo, whole ? o.k : o.rhi}, prefix[2] = {0, 0};
    const int passes = whole ? 3 : 2;
    bool ok[2] = {true, !whole};
    for (int pass = 0; pass < passes; ++pass) {
        const int shift = pass == 0 ? 20 : pass == 1 ? 10 : 0, nbins = pass == 0 ? 2048 : 1024;
        const unsigned bmask = (unsigned)nbins - 1u, pmask = pass == 0 ? 0u : 0xffffffffu << (shift + 10);
        // whether a quarter of the wave's first entries are the same (192 x 255, 94 % zeros: 56 -> 27 us, ones 133 -> 38)
        const bool crowded = __popcll(__ballot(u[0] == __builtin_amdgcn_readfirstlane(u[0]) && u[0] != 0xffffffffu)) >= 16;
#pragma unroll
        for (int j = 0; j < HOLD; ++j) {
            if (u[j] == 0xffffffffu) continue;
            if ((u[j] & pmask) == prefix[0]) sel_count(hist[0], (u[j] >> shift) & bmask, crowded);
            if (!whole && pass > 0 && (u[j] & pmask) == prefix[1]) sel_count(hist[1], (u[j] >> shift) & bmask, crowded);
        }
        __syncthreads();
        const unsigned p0 = prefix[0], p1 = prefix[1];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            if (q == 1 && whole) continue;
            unsigned bin, before;
            const bool got = sel_pick(hist[pass > 0 ? q : 0], nbins, r[q], bin, before, lds);
            ok[q] = ok[q] && got;
            if (ok[q]) {
                r[q] -= before;
                prefix[q] = (q ? p1 : p0) | (bin << shift);
            }
        }
        if (pass + 1 == passes) break;
        __syncthreads();
        for (int i = threadIdx.x; i < 2 * 2048; i += kSelThreads) (&hist[0][0])[i] = 0;
        __syncthreads();
    }
    if (threadIdx.x != 0) return;
    const unsigned maxbits = s_max;
    if (whole) {
        sel_result(o, prefix[0], maxbits);
        if (o.status && (o.clear_status || maxbits > kInf)) {
            if (o.clear_status) *o.status = maxbits > kInf ? 1 : 0;
            else atomicOr(o.status, 1);
        }
        return;
    }
    SelState *st = sel_state(o.ws);
    const unsigned lo = ok[0] ? min(prefix[0], kInf) : 0u, hi = ok[1] ? min(prefix[1] | 0x3ffu, kInf) : kInf;
    st->lo = lo;
    st->top = hi - lo;
}

// Calls take(bits of the magnitude) for every entry that this workgroup of `blocks` is responsible for.
typedef float v4f_a4 __attribute__((ext_vector_type(4), aligned(4)));
template <int ITEMS = kItems, class T>
__device__ __forceinline__ void sel_stream(const SelOperand &o, unsigned block, unsigned blocks, T take) {
    auto bits = [](float x) { return __float_as_uint(x) & 0x7fffffffu; };
    // a workgroup's pieces of one step lie side by side
    const unsigned long long step = (unsigned long long)blocks * (kSelThreads * ITEMS);
    const unsigned long long first = (unsigned long long)block * (kSelThreads * ITEMS) + threadIdx.x;
    if (o.kind <= 1) {
        const unsigned quads = o.N / 4;
        const unsigned qline = o.nfast / 4;
        auto run = [&](auto load) {
            for (unsigned long long q0 = first; q0 < quads; q0 += step) {
                v4f_a4 v[ITEMS];
#pragma unroll
                for (int i = 0; i < ITEMS; ++i) {
                    const unsigned long long q = q0 + (unsigned)(i * kSelThreads);
                    if (q < quads) {
                        const float *src = o.X + 4 * q;
                        if (o.kind == 1) {
                            const unsigned l = sel_line(o, (unsigned)(4 * q));
                            src = o.X + (int64_t)l * o.sslow + 4 * (int64_t)((unsigned)q - l * qline);
                        }
                        v[i] = load(reinterpret_cast<const v4f_a4 *>(src));
                    }
                }
#pragma unroll
                for (int i = 0; i < ITEMS; ++i)
                    if (q0 + (unsigned)(i * kSelThreads) < quads) {
                        take(bits(v[i][0])); take(bits(v[i][1])); take(bits(v[i][2])); take(bits(v[i][3]));
                    }
            }
        };
        // A matrix that the L2 caches cannot hold for the next pass anyway is read non-temporally (first pass over
        // 180 MB: 50 -> 35 us, 5.2 TB/s); one that they can, is not (second pass over 20 MB: 9 -> 6 us).
        if (o.N > (8u << 20)) run([](const v4f_a4 *p) { return __builtin_nontemporal_load(p); });
        else run([](const v4f_a4 *p) { return *p; });
        if (block == 0 && threadIdx.x < (o.N & 3u)) take(bits(o.X[(o.N & ~3u) + threadIdx.x]));  // contiguous only
    } else {
        for (unsigned long long e0 = first; e0 < o.N; e0 += step) {
            float v[ITEMS];
#pragma unroll
            for (int i = 0; i < ITEMS; ++i) {  // (no branch around a load: the compiler would wait for each before the next;
                // 8192 x 8190 views with odd pitches 232 -> 187 us, of every second entry 330 -> 207)
                const unsigned long long e = e0 + (unsigned)(i * kSelThreads);
                v[i] = sel_entry(o, (unsigned)min(e, (unsigned long long)o.N - 1ull));
            }
#pragma unroll
            for (int i = 0; i < ITEMS; ++i)
                if (e0 + (unsigned)(i * kSelThreads) < o.N) take(bits(v[i]));
        }
    }
}

// The rank k inside the window [base, base + top], by one workgroup on its own: a radix select of 11 bits per
// pass over the whole matrix (a window that missed).
__device__ __forceinline__ unsigned sel_alone(const SelOperand &o, unsigned base, unsigned top, unsigned k, unsigned *lh,
                                              unsigned *lds) {
    for (;;) {  // the window shrinks by eleven bits a pass
        const int shift = top >= 2048u ? 32 - __clz(top) - 11 : 0;
        for (int i = threadIdx.x; i < 2048; i += kSelThreads) lh[i] = 0;
        __syncthreads();
        sel_stream<2>(o, 0, 1, [&](unsigned u) {
            if (u - base <= top) sel_count(lh, (u - base) >> shift, true);
        });
        __syncthreads();
        unsigned bin, before;
        if (!sel_pick(lh, 2048, k, bin, before, lds)) return 0x7fffffffu;  // fewer entries than k: NaNs are not counted
        base += bin << shift;
        k -= before;
        if (shift == 0) return base;
        top = (1u << shift) - 1u;
        __syncthreads();
    }
}

// ---- a pass over the matrix (PASS 0, 1, 2) -----------------------------------------------------------------
template <int PASS>
__global__ __launch_bounds__(kSelThreads) void select_count_kernel(SelArgs args) {
    __shared__ unsigned lh[2048];
    __shared__ unsigned lds[20], s_below, s_max, s_last;
    const SelOperand o = sel_operand(args);
    if (o.N <= (unsigned)kSmall) return;  // the one-workgroup launch has done it
    SelState *st = sel_state(o.ws);
    unsigned *hist = sel_hist(o.ws) + (PASS == 0 ? 0 : PASS == 1 ? kHist1 : kHist2);
    const bool lead = blockIdx.x == 0;
    // a window with zero in it, or of next to nothing (4096 x 4095, 94 % zeros: 107 -> 66 us, ones 84 -> 33)
    const bool crowded = st->lo == 0 || st->top < 2048u;
    unsigned base = st->lo, top = st->top, shift = sel_shift0(top), k = o.k, bin, before;
    if (PASS == 1) {  // what the first pass has narrowed the window to
        const unsigned below = st->below, kw = k > below ? k - below : 0u;
        const bool got = sel_pick(sel_hist(o.ws), kBins0, kw, bin, before, lds);
        const unsigned nshift = shift > 10 ? shift - 10 : 0;
        if (lead && threadIdx.x == 0) {
            st->after = !got ? kMissed : shift == 0 ? kFound : nshift << 16;
            st->base1 = base + (bin << shift);
            st->k1 = kw - before;
        }
        if (!got || shift == 0) return;
        base += bin << shift;
        top = (1u << shift) - 1u;
        shift = nshift;
    } else if (PASS == 2) {
        const unsigned after = st->after;
        if (after & kMissed) {
            if (!lead) return;
            const unsigned a = st->maxbits > kInf ? 0x7fffffffu : sel_alone(o, 0, kInf, k, lh, lds);
            if (threadIdx.x == 0) sel_result(o, a, st->maxbits);
            return;
        }
        base = st->base1;
        shift = 0;
        if (!(after & kFound)) {
            shift = after >> 16;
            if (!sel_pick(sel_hist(o.ws) + kHist1, kBins1, st->k1, bin, before, lds)) return;  // cannot be: counted before
            base += bin << shift;
            k = st->k1 - before;
        }
        if (shift == 0) {
            if (lead && threadIdx.x == 0) sel_result(o, base, st->maxbits);
            return;
        }
        top = (1u << shift) - 1u;  // at most ten bits are left
        shift = 0;
    }
    const int nbins = PASS == 0 ? kBins0 : PASS == 1 ? kBins1 : kBins2;
    for (int i = threadIdx.x; i < nbins; i += kSelThreads) lh[i] = 0;
    if (threadIdx.x == 0) s_below = s_max = 0;
    __syncthreads();
    unsigned below = 0, umax = 0;
    sel_stream(o, blockIdx.x, gridDim.x, [&](unsigned u) {
        if (PASS == 0) {
            below += u < base ? 1u : 0u;
            umax = max(umax, u);
        }
        if (u - base <= top) sel_count(lh, (u - base) >> shift, crowded);
    });
    if (PASS == 0) {
        below = wave_sum_lane63(below);
        umax = (unsigned)wave_max_nonneg_lane63((int)umax);
        if ((threadIdx.x & 63) == 63) {
            if (below) atomicAdd(&s_below, below);
            atomicMax(&s_max, umax);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < nbins; i += kSelThreads)
        if (lh[i]) atomicAdd(&hist[i], lh[i]);
    if (PASS == 0 && threadIdx.x == 0) {
        if (s_below) atomicAdd(&st->below, s_below);
        atomicMax(&st->maxbits, s_max);
        if (s_max > kInf && o.status) atomicOr(o.status, 1);
    }
    if (PASS == 2) {  // rare: the workgroup that finishes last picks
        // (what the workgroups hand over are device-wide atomics: they only have to have arrived.  A fence to release them writes
        // back the L2 of the XCD, once per wave: 4096 x 4095 with a third
        // pass 110 us in all; so: 56, 41 without the pass)
        stores_done();
        __syncthreads();
        if (threadIdx.x == 0) s_last = (atomicAdd(&st->after, 1u) & 0xffffu) == gridDim.x - 1u;
        __syncthreads();
        if (!s_last) return;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        if (!sel_pick(hist, kBins2, k, bin, before, lds)) return;
        if (threadIdx.x == 0) sel_result(o, base + bin, st->maxbits);
    }
}

}  // namespace imu

using namespace imu;

static SelOperand sel_describe(const float *X, int64_t rows, int64_t cols, int64_t sx_r, int64_t sx_c, double p, float *out,
                               float half_beta, int32_t *status, void *ws) {
    SelOperand o = {};
    const int64_t N = rows * cols;
    double kd = std::ceil(p * (double)N / 100.0);
    if (kd < 1.0) kd = 1.0;
    if (kd > (double)N) kd = (double)N;
    // the unit-stride axis, if there is one, runs fastest
    int64_t nslow = rows, nfast = cols, sslow = sx_r, sfast = sx_c;
    if (sx_c != 1 && sx_r == 1) { nslow = cols; nfast = rows; sslow = sx_c; sfast = 1; }
    o.X = X;
    o.sslow = sslow; o.sfast = sfast;
    o.N = (unsigned)N; o.nfast = (unsigned)nfast;
    o.magic = nfast > 1 ? ~0ull / (unsigned long long)nfast + 1ull : 0ull;
    o.kind = sfast == 1 && (sslow == nfast || nslow == 1) ? 0 : sfast == 1 && nfast % 4 == 0 ? 1 : 2;
    o.k = (unsigned)kd;
    o.m = kSample;
    const double q = kd / (double)N, r = q * kSample, dr = 5.0 * std::sqrt(kSample * q * (1.0 - q)) + 4.0;
    o.rlo = r - dr < 1.0 ? 0u : (unsigned)(r - dr);
    o.rhi = (unsigned)std::ceil(r + dr);  // beyond the sample: no upper end
    o.ws = ws;
    o.out = out;
    o.half_beta = half_beta;
    o.status = status;
    o.clear_status = 1;
    return o;
}

// nops matrices (1 or 2), each the first of a batch of nitems
static int sel_launch(const SelArgs &a, int nops, hipStream_t st) {
    const unsigned y = (unsigned)(nops * a.nitems);
    unsigned most = a.op[0].N, held = 0;
    if (nops > 1) most = std::max(most, a.op[1].N);
    for (int q = 0; q < nops; ++q) held = std::max(held, a.op[q].N <= (unsigned)kSmall ? a.op[q].N : (unsigned)kSample);
    auto small = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(1, y), dim3(kSelThreads), 0, st, a); };
    if (held <= 4 * kSelThreads) small(select_small_kernel<4>);
    else if (held <= 8 * kSelThreads) small(select_small_kernel<8>);
    else if (held <= 16 * kSelThreads) small(select_small_kernel<16>);
    else if (held <= 32 * kSelThreads) small(select_small_kernel<32>);
    else small(select_small_kernel<kHold>);
    if (most > (unsigned)kSmall) {
        // one workgroup per CU at most (every workgroup merges its histogram with atomics on the same counters); a piece is one
        // entry where four cannot be loaded together
        int64_t pieces = 0;
        for (int q = 0; q < nops; ++q) pieces = std::max<int64_t>(pieces, a.op[q].kind <= 1 ? a.op[q].N / 4 : a.op[q].N);
        const unsigned blocks = (unsigned)std::min<int64_t>(256, (pieces + kSelThreads * kItems - 1) / (kSelThreads * kItems));
        hipLaunchKernelGGL(select_count_kernel<0>, dim3(blocks, y), dim3(kSelThreads), 0, st, a);
        hipLaunchKernelGGL(select_count_kernel<1>, dim3(blocks, y), dim3(kSelThreads), 0, st, a);
        hipLaunchKernelGGL(select_count_kernel<2>, dim3(blocks, y), dim3(kSelThreads), 0, st, a);
    }
    return launch_status();
}

static int run_percentile(const float *X, int64_t rows, int64_t cols, int64_t sx_r, int64_t sx_c, double p, float *out,
                          float half_beta, int32_t *status, void *ws, hipStream_t st) {
    SelArgs a = {};
    a.op[0] = sel_describe(X, rows, cols, sx_r, sx_c, p, out, half_beta, status, ws);
    a.nitems = 1;
    return sel_launch(a, 1, st);
}

extern "C" int imunpack_percentile(const float *X, int64_t rows, int64_t cols, int64_t sx_r, int64_t sx_c,
                                   double p, float *alpha, int32_t *status_flag, void *workspace,
                                   imunpack_stream_t stream) {
    if (!X || !alpha || !workspace || rows <= 0 || cols <= 0 || sx_r < 1 || sx_c < 1 || !(p > 0.0) || !(p <= 100.0))
        return IMUNPACK_EINVAL;
    if (rows > (int64_t)1 << 31 || cols > (int64_t)1 << 31 || rows * cols >= (int64_t)1 << 32) return IMUNPACK_EINVAL;
    return run_percentile(X, rows, cols, sx_r, sx_c, p, alpha, 0.0f, status_flag, workspace, (hipStream_t)stream);
}

static bool step_args_ok(const float *X, int64_t rows, int64_t cols, int64_t sx_r, int64_t sx_c, double p, float beta) {
    return X && rows > 0 && cols > 0 && sx_r >= 1 && sx_c >= 1 && p > 0.0 && p <= 100.0 && beta > 0.0f && beta < 3.0e38f &&
           rows <= (int64_t)1 << 31 && cols <= (int64_t)1 << 31 && rows * cols < (int64_t)1 << 32;
}

// The steps of both operands of every item of a batch (bt: see QuantBatch), by the same launches: steps[0] for A
// (n x d), steps[1] for B (h x d); two workspaces side by side at ws.
int imu::rtn_step_pair(const float *A, int64_t n, int64_t sa_r, int64_t sa_c, float beta_A, const float *B, int64_t h,
                       int64_t sb_r, int64_t sb_c, float beta_B, int64_t d, double p, float *steps, void *ws,
                       const QuantBatch &bt, hipStream_t st) {
    if (!step_args_ok(A, n, d, sa_r, sa_c, p, beta_A) || !step_args_ok(B, h, d, sb_r, sb_c, p, beta_B)) return IMUNPACK_EINVAL;
    SelArgs a = {};
    a.op[0] = sel_describe(A, n, d, sa_r, sa_c, p, steps, (float)(0.5 * (double)beta_A), bt.flag, ws);
    a.op[1] = sel_describe(B, h, d, sb_r, sb_c, p, steps + 1, (float)(0.5 * (double)beta_B), bt.flag,
                           static_cast<char *>(ws) + IMUNPACK_PERCENTILE_WORKSPACE_BYTES);
    a.op[0].x_stride = bt.a_stride;
    a.op[1].x_stride = bt.b_stride;
    a.op[0].clear_status = a.op[1].clear_status = 0;
    a.nitems = bt.nitems;
    a.out_stride = bt.out_stride;
    return sel_launch(a, 2, st);
}

extern "C" int imunpack_rtn_step(const float *X, int64_t rows, int64_t cols, int64_t sx_r, int64_t sx_c, double p,
                                 float beta, float *step, int32_t *status_flag, void *workspace,
                                 imunpack_stream_t stream) {
    if (!step || !workspace || !step_args_ok(X, rows, cols, sx_r, sx_c, p, beta)) return IMUNPACK_EINVAL;
    return run_percentile(X, rows, cols, sx_r, sx_c, p, step, (float)(0.5 * (double)beta), status_flag, workspace,
                          (hipStream_t)stream);
}

// ---- the same selection for callers that cannot allocate ------------------------------------------
// The counters and the selection state live in a file-scope device array instead of a caller
// workspace.  Every GPU holds its own copy of the array at its own address, which the host learns
// once per device; host code only ever uses that address, never the array's name.
static __device__ __align__(256) unsigned char scratch[IMUNPACK_PERCENTILE_WORKSPACE_BYTES];
static constexpr int kMaxDevices = 64;
static std::mutex g_scratch_lock;
static void *g_scratch_ptr[kMaxDevices];  // per device, nullptr until that device's first call

extern "C" int imunpack_percentile_static(const float *X, int64_t rows, int64_t cols, int64_t sx_r, int64_t sx_c,
                                          double p, float *alpha, int32_t *status_flag,
                                          imunpack_stream_t stream) {
    if (!X || !alpha || rows <= 0 || cols <= 0 || sx_r < 1 || sx_c < 1 || !(p > 0.0) || !(p <= 100.0))
        return IMUNPACK_EINVAL;
    // the scratch array's counters are 32 bits wide: more entries than they can count are refused
    if (rows > (int64_t)1 << 31 || cols > (int64_t)1 << 31 || rows * cols > IMUNPACK_PERCENTILE_STATIC_MAX_ENTRIES)
        return IMUNPACK_ERANGE;
    int dev = -1;
    IMU_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return IMUNPACK_EINVAL;
    void *ws = nullptr;
    {
        std::lock_guard<std::mutex> hold(g_scratch_lock);
        if (!g_scratch_ptr[dev]) {
            void *ptr = nullptr;
            IMU_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));  // the current device's copy
            if (!ptr) return IMUNPACK_EHIP;
            g_scratch_ptr[dev] = ptr;
        }
        ws = g_scratch_ptr[dev];
    }
    return run_percentile(X, rows, cols, sx_r, sx_c, p, alpha, 0.0f, status_flag, ws, (hipStream_t)stream);
}
