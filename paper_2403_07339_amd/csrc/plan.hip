// Unpack planner: decides every row / column split of Alg. 1, 2 and 4 (dispatched as in Alg. 5,
// A first, then B on the widened B_e with S_u carried over -- Sec. 4 "Combining everything")
// without touching the operands.  What it produces per unpacked row is the single non-zero of the
// matching column of Pi (source row, exponent of s); per unpacked column the exponent of the
// diagonal entry of S and the original column it copies.
//
// UnpackRow / UnpackColumn are FIFO loops whose result has a closed form: a row (column) whose
// largest magnitude has L base-s digits yields L slots, and the appended slots come level by
// level, within a level in ascending source index.  Slots are therefore assigned by one
// exclusive prefix sum per level.
//
// UnpackBoth is a greedy over OB counts.  A row split changes no other row's count and can only
// lower column counts (and vice versa), so all rows that share the current top count can be split
// as one batch, in index order, without changing the outcome of the sequential algorithm.  The
// greedy runs on the compacted list of OB entries (a tiny fraction of the operand) in a single
// persistent workgroup.
#include "common.h"

#include <type_traits>

#include <algorithm>
#include <atomic>
#include <cstddef>
#include <cstring>
#include <new>
#include <vector>

namespace imu {

constexpr int kPlanThreads = 1024;
constexpr int kPlanWaves = kPlanThreads / 64;

// ---------------------------------------------------------------------------------------------
// workgroup-wide helpers (kPlanThreads threads)
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ int block_max(int v /* >= 0 */, int *lds /* >= 40 ints */) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    v = wave_max_nonneg_lane63(v);
    if (lane == 63) lds[wave] = v;
    __syncthreads();
    int r = lds[0];
#pragma unroll
    for (int w = 1; w < kPlanWaves; ++w) r = max(r, lds[w]);
    __syncthreads();
    return r;
}

__device__ __forceinline__ int load_agent(const int32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// number of base-s digits of a magnitude (>= 1)
__device__ __forceinline__ int digit_levels(int m, int sh) {
    int L = 1;
    unsigned u = (unsigned)m >> sh;
    while (u) {
        ++L;
        u >>= sh;
    }
    return L;
}

__device__ __forceinline__ void flag_overflow(PlanHeader *hdr, int which, int need) {
    atomicOr(&hdr->overflow, 1 << which);
    atomicMax(&hdr->need[which], need);
}

// Calls emit(x, rank) for every x in [0, N) with flag(x), rank = base + the number of flagged x' < x;
// returns the number of flagged items.  Every wave owns one contiguous segment and ranks its items
// by ballot, so the whole selection costs two workgroup barriers.
template <class F, class E>
__device__ __forceinline__ int ordered_select(int N, int base, F flag, E emit, int *lds /* >= 40 ints */) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int seg = ((N + kPlanWaves - 1) / kPlanWaves + 63) & ~63;
    const int lo = wave * seg, hi = min(N, lo + seg);
    int cnt = 0;
    for (int x0 = lo; x0 < hi; x0 += 64) {
        const int x = x0 + lane;
        const bool f = x < hi && flag(x);
        cnt += __popcll(__ballot(f));
    }
    if (lane == 0) lds[wave] = cnt;
    __syncthreads();
    int run = base, total = 0;
#pragma unroll
    for (int w = 0; w < kPlanWaves; ++w) {
        const int c = lds[w];
        if (w < wave) run += c;
        total += c;
    }
    const unsigned long long below = (1ull << lane) - 1ull;
    for (int x0 = lo; x0 < hi; x0 += 64) {
        const int x = x0 + lane;
        const bool f = x < hi && flag(x);
        const unsigned long long mask = __ballot(f);
        if (f) emit(x, run + __popcll(mask & below));
        run += __popcll(mask);
    }
    __syncthreads();
    return total;
}

// Calls emit(x, prefix) for every x in [0, N), prefix = base + sum of value(x') over x' < x; returns
// the sum of all values.
template <class V, class E>
__device__ __forceinline__ int ordered_scan(int N, int base, V value, E emit, int *lds /* >= 40 ints */) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int seg = ((N + kPlanWaves - 1) / kPlanWaves + 63) & ~63;
    const int lo = wave * seg, hi = min(N, lo + seg);
    int sum = 0;
    for (int x0 = lo; x0 < hi; x0 += 64) {
        const int x = x0 + lane;
        if (x < hi) sum += value(x);
    }
    sum = wave_inclusive_sum(sum);
    if (lane == 63) lds[wave] = sum;
    __syncthreads();
    int run = base, total = 0;
#pragma unroll
    for (int w = 0; w < kPlanWaves; ++w) {
        const int c = lds[w];
        if (w < wave) run += c;
        total += c;
    }
    for (int x0 = lo; x0 < hi; x0 += 64) {
        const int x = x0 + lane;
        const int v = x < hi ? value(x) : 0;
        const int incl = wave_inclusive_sum(v);
        if (x < hi) emit(x, run + incl - v);
        run += from_lane63(incl);
    }
    __syncthreads();
    return total;
}

// ---------------------------------------------------------------------------------------------
// header / identity
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ void identity_slot(const SlotSet &set, int x) {
    set.root[x] = x;
    set.exp[x] = 0;
    set.time[x] = kNever;
    set.child[x] = -1;
}

// Clears the header and makes the first na / nb / nc slots of three sets (row slots of A and of B, column
// slots of A's unpacking) unsplit originals (a count of 0 skips a set).  The counts are known to the host,
// which has sized the sets for them.  blockIdx.y is the item of the batch, as in every planner kernel.
__global__ void setup_kernel(PlanHeader *hdr, SlotSet a, int na, SlotSet c, int nc, SlotSet b, int nb, int32_t *zeroed,
                             int nzeroed, int32_t *zeroed2, int nzeroed2, KeepState *ks, int64_t stride) {
    hdr += blockIdx.y;
    const int64_t off = blockIdx.y * stride;
    move_to_item(a, off);
    move_to_item(b, off);
    move_to_item(c, off);
    zeroed = item_at(zeroed, off);
    zeroed2 = item_at(zeroed2, off);
    if (blockIdx.x == 0) {
        static_assert(sizeof(PlanHeader) % sizeof(int32_t) == 0, "header is cleared word by word");
        for (size_t i = threadIdx.x; i < sizeof(PlanHeader) / sizeof(int32_t); i += blockDim.x)
            reinterpret_cast<int32_t *>(hdr)[i] = 0;
        __syncthreads();
        if (threadIdx.x == 0) {
            if (ks) ks->same = 0;
            if (na) hdr->n_u = na;
            if (nb) hdr->h_u = nb;
            if (nc) hdr->d1 = nc;
        }
    }
    const int step = gridDim.x * blockDim.x;
    for (int x = blockIdx.x * blockDim.x + threadIdx.x; x < na; x += step) identity_slot(a, x);
    for (int x = blockIdx.x * blockDim.x + threadIdx.x; x < nb; x += step) identity_slot(b, x);
    for (int x = blockIdx.x * blockDim.x + threadIdx.x; x < nc; x += step) identity_slot(c, x);
    for (int x = blockIdx.x * blockDim.x + threadIdx.x; x < nzeroed; x += step) zeroed[x] = 0;
    for (int x = blockIdx.x * blockDim.x + threadIdx.x; x < nzeroed2; x += step) zeroed2[x] = 0;
}

// UnpackRow on the second operand splits no column: its column slots are those that A's unpacking left.
__global__ void identity_slots_kernel(SlotSet set, PlanHeader *hdr, const int32_t *skip, int64_t stride) {
    hdr += blockIdx.y;
    move_to_item(set, blockIdx.y * stride);
    if (hdr->overflow) return;
    if (skip && *skip) return;  // keep-weights mode: this set is taken over as it stands
    const int N = hdr->d1;
    if (N > set.cap) {
        if (blockIdx.x == 0 && threadIdx.x == 0) flag_overflow(hdr, CAP_C2, N);
        return;
    }
    for (int x = blockIdx.x * blockDim.x + threadIdx.x; x < N; x += gridDim.x * blockDim.x) identity_slot(set, x);
    if (blockIdx.x == 0 && threadIdx.x == 0) hdr->d_u = N;
}

// ---------------------------------------------------------------------------------------------
// UnpackRow / UnpackColumn in closed form (Alg. 1 / Alg. 2)
// ---------------------------------------------------------------------------------------------
// Base items x = 0..N-1 with largest magnitude maxabs[via ? via[x] : x] (via: the columns that A's unpacking
// left, N read from the header); every level l >= 1 appends the items that still have a digit there, in
// ascending x.  `which` names the set.
template <int kLevelItems>
__device__ void level_major(const SlotSet &set, const int32_t *maxabs, const int32_t *via, int N, int sh, int32_t *tmpL,
                            int32_t *tmpCur, PlanHeader *hdr, int which, int *lds /* >= 40 ints */) {
    int32_t *count_out = which == CAP_ROWA ? &hdr->n_u : which == CAP_ROWB ? &hdr->h_u : which == CAP_C1 ? &hdr->d1 : &hdr->d_u;
    if (N > set.cap) {
        if (threadIdx.x == 0) flag_overflow(hdr, which, N);
        return;
    }
    // Up to kLevelItems items per thread: their levels and latest slots stay in registers (a wave owns a contiguous segment, as
    // in ordered_select), so that a level is ballots and stores.  12608 rows: 23 -> 16 us.
    if (N <= kLevelItems * kPlanThreads) {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        const int seg = ((N + kPlanWaves - 1) / kPlanWaves + 63) & ~63, x0 = wave * seg + lane;
        const int hi = min(N, (wave + 1) * seg);
        int L[kLevelItems], last[kLevelItems], lm = 1;
#pragma unroll
        for (int u = 0; u < kLevelItems; ++u) {
            const int x = x0 + 64 * u;
            last[u] = 64 * u < seg && x < hi ? (via ? via[x] : x) : -1;  // (uniform first: most operands fill a few)
        }
#pragma unroll
        for (int u = 0; u < kLevelItems; ++u) {
            if (64 * u >= seg) break;
            L[u] = last[u] >= 0 ? maxabs[last[u]] : 0;
        }
#pragma unroll
        for (int u = 0; u < kLevelItems; ++u) {
            if (64 * u >= seg) break;
            if (last[u] < 0) continue;
            const int x = x0 + 64 * u;
            last[u] = x;
            L[u] = digit_levels(L[u], sh);
            lm = max(lm, L[u]);
            set.root[x] = x;
            set.exp[x] = 0;
            if (L[u] == 1) {
                set.time[x] = kNever;
                set.child[x] = -1;
            }
        }
        const int lmax = block_max(lm, lds);
        const unsigned long long below = (1ull << lane) - 1ull;
        int base = N;
        for (int l = 1; l < lmax; ++l) {
            int cnt = 0;
#pragma unroll
            for (int u = 0; u < kLevelItems; ++u) {
                if (64 * u >= seg) break;
                cnt += __popcll(__ballot(last[u] >= 0 && L[u] > l));
            }
            if (lane == 0) lds[wave] = cnt;
            __syncthreads();
            int run = base;
#pragma unroll
            for (int w = 0; w < kPlanWaves; ++w) {
                const int c = lds[w];
                if (w < wave) run += c;
                base += c;
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < kLevelItems; ++u) {
                if (64 * u >= seg) break;
                const bool f = last[u] >= 0 && L[u] > l;
                const unsigned long long m = __ballot(f);
                const int slot = run + __popcll(m & below);
                run += __popcll(m);
                if (!f) continue;
                const int prev = last[u];
                if (slot >= set.cap) {  // the plan is made again with more room; until then the chain ends here (ob_copy walks it
                                        // before the host hears of it: no link may be left unwritten)
                    set.time[prev] = kNever;
                    set.child[prev] = -1;
                    continue;
                }
                set.root[slot] = x0 + 64 * u;
                set.exp[slot] = l;
                set.key[slot] = ((unsigned long long)l << 48) | (unsigned)prev;
                if (L[u] == l + 1) {
                    set.time[slot] = kNever;
                    set.child[slot] = -1;
                }
                set.child[prev] = slot;
                set.time[prev] = 0;  // split (only this axis splits in this phase, any finite time will do)
                last[u] = slot;
            }
        }
        if (threadIdx.x == 0) {
            *count_out = base;
            if (base > set.cap) flag_overflow(hdr, which, base);
        }
        return;
    }
    int lm = 1;
    for (int x = threadIdx.x; x < N; x += kPlanThreads) {
        const int L = digit_levels(maxabs[via ? via[x] : x], sh);
        tmpL[x] = L;
        tmpCur[x] = x;
        identity_slot(set, x);
        lm = max(lm, L);
    }
    const int lmax = block_max(lm, lds);
    int base = N;
    for (int l = 1; l < lmax; ++l) {
        base += ordered_select(
            N, base, [&](int x) { return tmpL[x] > l; },
            [&](int x, int slot) {
                if (slot >= set.cap) return;
                set.root[slot] = x;
                set.exp[slot] = l;
                set.time[slot] = kNever;
                set.child[slot] = -1;
                const int prev = tmpCur[x];
                set.key[slot] = ((unsigned long long)l << 48) | (unsigned)prev;
                set.child[prev] = slot;
                set.time[prev] = 0;  // split (only this axis splits in this phase, any finite time will do)
                tmpCur[x] = slot;
            },
            lds);
    }
    if (threadIdx.x == 0) {
        *count_out = base;
        if (base > set.cap) flag_overflow(hdr, which, base);
    }
}

__global__ __launch_bounds__(kPlanThreads) void level_major_kernel(
    SlotSet set, const int32_t *maxabs, const int32_t *via, int n_host, int sh, int32_t *tmpL, int32_t *tmpCur,
    PlanHeader *hdr, int which, const int32_t *skip, int64_t stride, int64_t stats_stride) {
    __shared__ int lds[40];
    hdr += blockIdx.y;
    {
        const int64_t off = blockIdx.y * stride;
        move_to_item(set, off);
        via = item_at(via, off);
        tmpL = item_at(tmpL, off);
        tmpCur = item_at(tmpCur, off);
        maxabs = item_at(maxabs, blockIdx.y * stats_stride);
    }
    if (hdr->overflow) return;
    if (skip && *skip) return;  // keep-weights mode: this set is taken over as it stands
    level_major<16>(set, maxabs, via, via ? hdr->d1 : n_host, sh, tmpL, tmpCur, hdr, which, lds);
}

// Both operands in one launch, where neither is unpacked by UnpackBoth.  Workgroup 0 takes the first operand and what needs
// its columns, workgroup 1, beside it, a second operand that does not: its rows, or its columns where the first operand
// leaves the columns as they are.  (One behind the other: 17 + 5 us for 12608 rows and 768 columns, 6 + 5 + 3 for 1031 columns
// and 777 rows; most of a launch this short is its start.)
struct LevelPair {
    SlotSet a, b, c1, c2;              // c1, c2: column slots of A's unpacking, of the second one
    const int32_t *max_a, *max_b;
    int strategyA, strategyB, n, d, h, sh;
    int32_t *tmpL, *tmpCur;
    PlanHeader *hdr;
    int64_t stride, stats_stride;
};
constexpr int kPairItems = 8;  // items a thread holds: more, and what chooses between the operands no longer fits the registers
__global__ __launch_bounds__(kPlanThreads) void level_major_pair_kernel(LevelPair f) {
    __shared__ int lds[40];
    PlanHeader *hdr = f.hdr + blockIdx.y;
    const int64_t off = blockIdx.y * f.stride, soff = blockIdx.y * f.stats_stride;
    move_to_item(f.a, off);
    move_to_item(f.b, off);
    move_to_item(f.c1, off);
    move_to_item(f.c2, off);
    f.max_a = item_at(f.max_a, soff);
    f.max_b = item_at(f.max_b, soff);
    f.tmpL = item_at(f.tmpL, off);
    f.tmpCur = item_at(f.tmpCur, off);
    const bool by_row = f.strategyA == IMUNPACK_ROW, b_by_row = f.strategyB == IMUNPACK_ROW;
    // workgroup 0: A, then what of B needs A's columns; workgroup 1: what does not (one call of level_major: with several the
    // compiler leaves it out of line and its arguments in scratch memory, 17 -> 52 us)
    bool second = blockIdx.x == 1;
    for (;; second = true) {
        SlotSet set = second ? (b_by_row ? f.b : f.c2) : by_row ? f.a : f.c1;
        const bool via = second && blockIdx.x == 0;
        const int N = via ? hdr->d1 : second ? (b_by_row ? f.h : f.d) : by_row ? f.n : f.d;
        level_major<kPairItems>(set, second ? f.max_b : f.max_a, via ? f.c1.root : nullptr, N, f.sh, f.tmpL, f.tmpCur, hdr,
                                second ? (b_by_row ? CAP_ROWB : CAP_C2) : by_row ? CAP_ROWA : CAP_C1, lds);
        if (second || (by_row && !b_by_row)) return;
        __syncthreads();
        if (hdr->d1 > f.c1.cap) return;  // reported: the plan is made again
        if (b_by_row) break;
    }
    // the second unpacking splits no column: its column slots are those that A's left
    const int N = hdr->d1;
    if (N > f.c2.cap) {
        if (threadIdx.x == 0) flag_overflow(hdr, CAP_C2, N);
        return;
    }
    for (int x = threadIdx.x; x < N; x += kPlanThreads) identity_slot(f.c2, x);
    if (threadIdx.x == 0) hdr->d_u = N;
}

// ---------------------------------------------------------------------------------------------
// UnpackBoth (Alg. 4): the greedy
// ---------------------------------------------------------------------------------------------
struct GreedyArgs {
    SlotSet rows, cols;
    int second;                    // second operand: starts from the column slots that unpacking A left, which are
                                   // made unsplit originals here
    const int32_t *chain_child;    // second operand: child links of the column slots of A's unpacking
    const int32_t *chain_root;     // second operand: original column of each of those slots
    const int32_t *rowcnt, *colcnt, *rowmax;  // the operand's heavy-hitter statistics
    int ob_cap;                    // entries the OB list can hold
    const int32_t *ob_count;
    int which_list;
    unsigned long long *edges;     // two lists of ecap packed edges
    int ecap;
    const int32_t *extra_rows;     // second operand: extra edges per row (repeated columns), else null
    int32_t *rcnt, *ccnt;          // live OB count per row / column slot when LDS cannot hold them
    PlanHeader *hdr;
    int64_t stride, stats_stride, list_stride;  // from item to item: the plan's arrays, the statistics, the OB list
    int whichR, whichC, whichE;
    int s, sh;
    const int32_t *skip;           // keep-weights mode: non-zero there = nothing to do
    int lds_words;                 // dynamic LDS of the launch
};

// An edge of the greedy: an OB entry's current row slot, column slot and the number of base-s digits
// it still has there (>= 2 while it is OB).  Only that number matters: a split moves floor(v / s) on.
constexpr int kEdgeSlotBits = 29;
constexpr unsigned kEdgeSlotMask = (1u << kEdgeSlotBits) - 1u;
// A packed edge is two 32-bit words, so that a pass never needs 64-bit arithmetic: the low word holds
// the row slot, the high word the column slot, and the three bits above each slot number hold the low
// and the high half of the number of digits left (2 .. 63, so a packed edge is never 0).
__device__ __forceinline__ unsigned long long pack_edge(int row, int col, int levels) {
    const unsigned lo = (unsigned)row | (((unsigned)levels & 7u) << kEdgeSlotBits);
    const unsigned hi = (unsigned)col | (((unsigned)levels >> 3) << kEdgeSlotBits);
    return (unsigned long long)lo | ((unsigned long long)hi << 32);
}

// The sequential algorithm splits, at every step, the row or column with the top OB count (rows win
// ties, then the lowest index).  Splitting a row changes no other row's count and only lowers column
// counts, so while rows are being chosen the rows come in (count descending, index ascending) order
// and every row whose count is at least the top column count at the start of the run is chosen
// before any column -- unless a split leaves OB entries in the new row (entries with three or more
// digits), whose count then competes.  Hence:
//   - if no entry has three or more digits, one batch takes all rows with count >= top column count
//     (or all columns with count > top row count);
//   - otherwise a batch takes the slots that share the top count; with the edges in LDS, where the most such entries that any
//     slot of either side holds are counted once, every slot whose count exceeds that (greedy_run: deep_row, deep_col).
// The starting counts are the operand's scan statistics.  After UnpackA the matrix B_e repeats column
// k of B once per column slot that descends from k (Alg. 2 line 6 / Alg. 4 line 13): such a slot
// starts with the count of column k, and every OB entry (j, k) adds one to row j per extra slot
// (ob_copy_kernel finds those extra edges before this kernel starts).
// A batch is one pass over the live entries: an entry in a split slot keeps digit 0 there and moves
// floor(v / s) to the new slot (Alg. 4 lines 7-9 / 11-14); if that is In-Bound the entry is finished:
// it leaves the count of the crossing slot and the list.  The entries are packed edges (row slot,
// column slot, digits left); the first list comes from ob_copy_kernel, the survivors of every pass are
// written, compacted, to the other of two lists.  The order inside a batch only decides the numbers of the appended slots; it is recorded as
// a sort key (batch, count descending, split slot) and the appended slots are renumbered on the host
// when the plan is exported.
__device__ __forceinline__ void move_to_item(GreedyArgs &g) {
    const int64_t off = blockIdx.y * g.stride, soff = blockIdx.y * g.stats_stride;
    move_to_item(g.rows, off);
    move_to_item(g.cols, off);
    g.chain_child = item_at(g.chain_child, off);
    g.chain_root = item_at(g.chain_root, off);
    g.edges = item_at(g.edges, off);
    g.extra_rows = item_at(g.extra_rows, off);
    g.rcnt = item_at(g.rcnt, off);
    g.ccnt = item_at(g.ccnt, off);
    g.rowcnt = item_at(g.rowcnt, soff);
    g.colcnt = item_at(g.colcnt, soff);
    g.rowmax = item_at(g.rowmax, soff);
    g.ob_count = item_at(g.ob_count, blockIdx.y * g.list_stride);
}

//
// If they fit the LDS that the counts leave, the edges stay there from the first batch to the last (one that is finished
// becomes 0): nothing the workgroup waits for between batches is in memory then, and its barriers need not wait for the
// stores of the new slots.  With the edges in the two lists, which every pass reads and rewrites, a batch of a small operand
// took 3 us and more, mostly round trips to memory.  (Edges in registers, 40 a thread, would reach further; the compiler
// spills them.)
struct GreedyShared {
    int top[2], T[2][4];
    int pick[kPlanWaves][256];  // per wave: the slots picked in one 256-slot step
    int found[kPlanWaves], positive[kPlanWaves];
    int lds[40];
    int count;
    alignas(16) unsigned long long split[32];  // greedy_bits
};

// What comes before the first batch: the second operand's columns become unsplit originals, the number of edges is reported.  Returns
// it, or -1 where something has no room (uniform).
__device__ __forceinline__ long long greedy_begin(const GreedyArgs &g, PlanHeader *hdr, int nc, int nob, int extras) {
    if (g.second) {
        if (nc > g.cols.cap) {
            if (threadIdx.x == 0) flag_overflow(hdr, g.whichC, nc);
            return -1;
        }
        for (int x = threadIdx.x; x < nc; x += kPlanThreads) identity_slot(g.cols, x);
    }
    if (nob > g.ob_cap) {
        if (threadIdx.x == 0) flag_overflow(hdr, g.which_list, nob);
        return -1;
    }
    const long long Etotal = (long long)nob + extras;
    if (threadIdx.x == 0) {
        *(g.second ? &hdr->edgesB : &hdr->edgesA) = (int)min(Etotal, 2147483647ll);
        *(g.second ? &hdr->nobB : &hdr->nobA) = nob;  // the OB entries kept for the scatter
    }
    if (Etotal > g.ecap) {
        if (threadIdx.x == 0) flag_overflow(hdr, g.whichE, (int)min(Etotal, 1ll << 30));
        return -1;
    }
    return Etotal;
}

// The greedy of an operand of at most 32 W rows and columns whose entries have at most three digits, on bits.  All that is left of an
// entry above digit 0 is always in the last slot of its row's and of its column's chain of splits, so the state is how often
// each original row and column has been split, and a slot's count is that of the bits of
//   (entries of two digits or more) & (other side not split)  |  (entries of three) & (other side split once)
// in its row or column of the operand (the planes move down by one when the slot is split).  A thread has the bits of one row or of
// one column in registers: a batch is some hundred instructions a wave and two
// barriers, with the batches of greedy_run, one for each turn between the sides or bound.  In it, with the edges in LDS,
// a batch takes 4 us.  24 heads, 197 x 197 gradients of a softmax, some entries of three digits: 160 us, 90 so; both operands of 256 x 256
// with 330 heavy hitters each: 23 and 23 us, 10 and 13.
// planes: 64 W W words of LDS.
template <int W, bool DEEP>  // DEEP: there are entries of three digits
__device__ __forceinline__ void greedy_bits(const GreedyArgs &g, PlanHeader *hdr, unsigned *planes, GreedyShared &sh, int nob, int extras) {
    constexpr int S = 32 * W, kSideWaves = W / 2;
    static_assert(2 * kSideWaves <= kPlanWaves && W <= 16, "a wave for every 64 slots of either side");
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int nr = g.second ? hdr->h_u : hdr->n_u, nc = hdr->d1;
    const int Etotal = (int)greedy_begin(g, hdr, nc, nob, extras);
    if (Etotal < 0) return;
    const bool is_col = wave >= kSideWaves;
    const int own_wave = wave & (kSideWaves - 1), x = own_wave * 64 + lane;  // the thread's original row or column
    constexpr int kPlanes = DEEP ? 2 : 1;
    unsigned two[W], three[W];
    auto load = [&](const unsigned *from) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < W; ++i) {
            two[i] = from[x * W + i];
            if constexpr (DEEP) three[i] = from[S * W + x * W + i];
        }
    };
    // both sides at once where LDS holds them, else one after the other
    const bool at_once = 2 * kPlanes * S * W <= g.lds_words;
    for (int side = 0; side < 2; ++side) {
        if (side && at_once) break;
        const int words = (at_once ? 2 : 1) * kPlanes * S * W;
        for (int t = threadIdx.x * 4; t < words; t += kPlanThreads * 4) *reinterpret_cast<int4 *>(planes + t) = make_int4(0, 0, 0, 0);
        __syncthreads();
        for (int e = threadIdx.x; e < Etotal; e += kPlanThreads) {
            const unsigned long long ed = g.edges[e];
            if (ed == 0ull) continue;
            const unsigned lo = (unsigned)ed, hi = (unsigned)(ed >> 32), r = lo & kEdgeSlotMask, c = hi & kEdgeSlotMask;
            const bool longer = DEEP && ((lo >> kEdgeSlotBits) | ((hi >> kEdgeSlotBits) << 3)) > 2u;
            auto set = [&](unsigned *to, unsigned own, unsigned other) __attribute__((always_inline)) {
                const unsigned at = own * W + (other >> 5), bit = 1u << (other & 31);
                atomicOr(to + at, bit);
                if (longer) atomicOr(to + S * W + at, bit);
            };
            if (at_once || side == 0) set(planes, r, c);
            if (at_once) set(planes + kPlanes * S * W, c, r);
            else if (side == 1) set(planes, c, r);
        }
        __syncthreads();
        if (wave < 2 * kSideWaves) {
            if (at_once) load(planes + (is_col ? kPlanes * S * W : 0));
            else if (is_col == (side != 0)) load(planes);
        }
        if (!at_once) __syncthreads();
    }
    const bool serves = wave < 2 * kSideWaves;  // (the other waves only keep in step)
    if (!serves)
#pragma unroll
        for (int i = 0; i < W; ++i) two[i] = three[i] = 0;
    auto sync = [] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    // the largest value of either side
    auto tops = [&](int v, int &rows, int &cols) __attribute__((always_inline)) {
        v = wave_max_nonneg_lane63(v);
        if (lane == 63 && serves) sh.found[wave] = v;
        sync();
        int m = lane < 2 * kSideWaves ? sh.found[lane] : 0;  // lanes [0, kSideWaves) the rows'
        m = max(m, IMU_DPP(m, 0x111, 0xf, true));
        m = max(m, IMU_DPP(m, 0x112, 0xf, true));
        if constexpr (kSideWaves == 8) m = max(m, IMU_DPP(m, 0x114, 0xf, true));
        rows = __builtin_amdgcn_readlane(m, kSideWaves - 1);
        cols = __builtin_amdgcn_readlane(m, 2 * kSideWaves - 1);
    };
    int deep_row = 0, deep_col = 0;  // as in greedy_run
    if constexpr (DEEP) {
        int n3 = 0;
#pragma unroll
        for (int i = 0; i < W; ++i) n3 += __popc(three[i]);
        tops(n3, deep_row, deep_col);
        sync();
    }
    // a side's slots that are not split, and those that are split once, a word per wave of the side
    auto masks = [&](bool col, int kind) __attribute__((always_inline)) { return sh.split + (col ? 16 : 0) + 8 * kind; };
    unsigned long long whole = ~0ull, once = 0ull;  // (the wave's own)
    if (lane == 0 && serves) {
        masks(is_col, 0)[own_wave] = whole;
        masks(is_col, 1)[own_wave] = once;
    }
    sync();
    const SlotSet &mine = is_col ? g.cols : g.rows;
    int slot = x, splits = 0;  // the last slot of the thread's chain
    for (int bid = 0;; ++bid) {  // (every batch splits a slot, each original twice at most)
        int cnt = 0;
        if (serves)
#pragma unroll
            for (int i = 0; i < W; i += 4) {
                const int4 a = *reinterpret_cast<const int4 *>(reinterpret_cast<const unsigned *>(masks(!is_col, 0)) + i);
                const unsigned none[4] = {(unsigned)a.x, (unsigned)a.y, (unsigned)a.z, (unsigned)a.w};
                unsigned one[4] = {0, 0, 0, 0};
                if constexpr (DEEP) {
                    const int4 c = *reinterpret_cast<const int4 *>(reinterpret_cast<const unsigned *>(masks(!is_col, 1)) + i);
                    one[0] = c.x; one[1] = c.y; one[2] = c.z; one[3] = c.w;
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) cnt += __popc(DEEP ? (two[i + k] & none[k]) | (three[i + k] & one[k]) : two[i + k] & none[k]);
            }
        int c0, c1;
        tops(cnt, c0, c1);
        if (c0 <= 0 && c1 <= 0) break;
        const bool isrow = c0 >= c1;  // rows win ties
        const int hi = isrow ? c0 : c1, least = (isrow ? deep_row : deep_col) + 1;
        const int lo = min(hi, max(isrow ? max(c1, 1) : c0 + 1, least));
        const bool turn = serves && isrow != is_col, pick = turn && cnt >= lo;
        const unsigned long long picked = __ballot(pick);
        if (turn) {
            once = (once & ~picked) | (whole & picked);
            whole &= ~picked;
            if (lane == 0) {
                masks(is_col, 0)[own_wave] = whole;
                if constexpr (DEEP) masks(is_col, 1)[own_wave] = once;
                sh.positive[own_wave] = __popcll(picked);
            }
        }
        sync();
        int nb = 0, before = 0;
#pragma unroll
        for (int w = 0; w < kSideWaves; ++w) {
            if (w == own_wave) before = nb;
            nb += sh.positive[w];
        }
        nb = __builtin_amdgcn_readfirstlane(nb);
        const int N = isrow ? nr : nc;
        if (N + nb > (isrow ? g.rows.cap : g.cols.cap)) {
            if (threadIdx.x == 0) flag_overflow(hdr, isrow ? g.whichR : g.whichC, 2 * (N + nb));
            return;
        }
        if (turn) {
            if (pick) {
                const int newX = N + before + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(picked >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)picked, 0u));
                mine.time[slot] = (uint32_t)bid;
                mine.child[slot] = newX;
                mine.root[newX] = x;
                mine.exp[newX] = ++splits;
                mine.time[newX] = kNever;
                mine.child[newX] = -1;
                mine.key[newX] = ((unsigned long long)bid << 48) | ((unsigned long long)(0xFFFFFF - cnt) << 24) | (unsigned)slot;
                slot = newX;
#pragma unroll
                for (int i = 0; i < W; ++i) {
                    two[i] = DEEP ? three[i] : 0;
                    if constexpr (DEEP) three[i] = 0;
                }
            }
        }
        if (isrow) nr += nb; else nc += nb;
    }
    if (threadIdx.x == 0) {
        *(g.second ? &hdr->h_u : &hdr->n_u) = nr;
        *(g.second ? &hdr->d_u : &hdr->d1) = nc;
    }
}
constexpr int bits_words(int slots) { return slots <= 256 ? 64 * 8 * 8 : slots <= 512 ? 64 * 16 * 16 : 0; }  // LDS of greedy_bits (0: not for so many)

template <bool LDS, bool RES, bool SHORT>  // LDS: the counts are in LDS; RES: the edges too; SHORT: fewer variants of the passes
__device__ __forceinline__ void greedy_run(const GreedyArgs &g, PlanHeader *hdr, int32_t *lds_counts, GreedyShared &sh, int nob, int extras, const int deep) {
    constexpr int UE = 4;  // edges in LDS that a thread looks at together
    auto &s_top = sh.top;
    auto &s_T = sh.T;
    auto &s_pick = sh.pick;
    auto &s_found = sh.found;
    auto &s_positive = sh.positive;
    auto &lds = sh.lds;
    int &s_count = sh.count;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const unsigned long long below = (1ull << lane) - 1ull;
    int nr = g.second ? hdr->h_u : hdr->n_u, nc = hdr->d1;
    const long long Etotal = greedy_begin(g, hdr, nc, nob, extras);
    if (Etotal < 0) return;
    // ---- the first edge list was written by ob_copy_kernel: one packed edge per OB entry, then the extra
    // edges of repeated columns (second operand only; the rows they touch start with that many more OB
    // entries)
    unsigned long long *list0 = g.edges, *list1 = g.edges + ((g.ecap + 1) & ~1);  // both 16-byte aligned
    // between the phases of a batch: what the threads hand to one another is in LDS if the edges are in registers
    auto sync = [] {
        if constexpr (RES) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        else __syncthreads();
    };
    const int rpad = (g.rows.cap + 7) & ~3, cpad = (g.cols.cap + 7) & ~3;  // int4 reads may run past the last slot
    int32_t *rc = LDS ? lds_counts : g.rcnt;
    int32_t *cc = LDS ? lds_counts + rpad : g.ccnt;
    unsigned long long *held = reinterpret_cast<unsigned long long *>(lds_counts + rpad + cpad);
    if constexpr (RES)
        for (int e = threadIdx.x; e < Etotal; e += kPlanThreads) held[e] = list0[e];
    // ---- starting counts
    auto start_counts = [&]() __attribute__((always_inline)) {
        for (int x = threadIdx.x; x < rpad; x += kPlanThreads)
            rc[x] = x < nr ? g.rowcnt[x] + (g.extra_rows ? g.extra_rows[x] : 0) : 0;
        for (int x = threadIdx.x; x < cpad; x += kPlanThreads)
            cc[x] = x < nc ? g.colcnt[g.chain_root ? g.chain_root[x] : x] : 0;
    };
    start_counts();
    if (threadIdx.x == 0) {
        s_count = 0;
        s_top[0] = s_top[1] = 0;
    }
    __syncthreads();
    // If there are entries of three or more digits: the most that any row, any column holds.  The slot that a split appends
    // starts with those of the split slot that are left (entries only lose digits), so its count never exceeds this, and
    // slots with a larger count are taken before it whatever is split in between.
    int deep_row = 0, deep_col = 0;
    if (deep) {
        for (int x = threadIdx.x; x < rpad; x += kPlanThreads) rc[x] = 0;
        for (int x = threadIdx.x; x < cpad; x += kPlanThreads) cc[x] = 0;
        __syncthreads();
        constexpr int UD = 8;
        for (int e0 = threadIdx.x; e0 < Etotal; e0 += kPlanThreads * UD) {
            unsigned long long ed[UD];
#pragma unroll
            for (int u = 0; u < UD; ++u) {
                const int e = e0 + u * kPlanThreads;
                if constexpr (RES) ed[u] = e < Etotal ? held[e] : 0ull;
                else ed[u] = e < Etotal ? list0[e] : 0ull;
            }
#pragma unroll
            for (int u = 0; u < UD; ++u) {
                const unsigned lo = (unsigned)ed[u], hi = (unsigned)(ed[u] >> 32);
                if (((lo >> kEdgeSlotBits) | ((hi >> kEdgeSlotBits) << 3)) > 2u) {
                    atomicAdd(&rc[lo & kEdgeSlotMask], 1);
                    atomicAdd(&cc[hi & kEdgeSlotMask], 1);
                }
            }
        }
        __syncthreads();
        int mr = 0, mc = 0;
        for (int x = threadIdx.x; x < nr; x += kPlanThreads) mr = max(mr, rc[x]);
        for (int x = threadIdx.x; x < nc; x += kPlanThreads) mc = max(mc, cc[x]);
        deep_row = block_max(mr, lds);
        deep_col = block_max(mc, lds);
        start_counts();
        __syncthreads();
    }
    const int nr0 = nr, nc0 = nc;  // the slots below are unsplit originals
    int E = (int)Etotal, cur = 0;  // live edges; they are in list `cur`
    int prev_kind = -1;            // 1: the batch before split rows, 0: columns
    const long long max_batches = 32ll * Etotal + 64;  // every batch retires >= one digit of one entry
    for (long long bid = 0;; ++bid) {
        if (bid > max_batches || bid >= 65535) {
            if (threadIdx.x == 0) atomicMin(&hdr->err, bid >= 65535 ? IMUNPACK_ERANGE : IMUNPACK_EHIP);
            return;
        }
        // Every wave owns one contiguous segment of the row slots and one of the column slots, four
        // slots per lane.  (1) top counts; the marks the previous batch left in split slots (negative
        // values) are cleared on the way -- a split slot never holds an OB entry again.
        const int segR = ((nr + kPlanWaves - 1) / kPlanWaves + 255) & ~255;
        const int segC = ((nc + kPlanWaves - 1) / kPlanWaves + 255) & ~255;
        int m0 = 0, m1 = 0;
        for (int x0 = wave * segR; x0 < min(nr, (wave + 1) * segR); x0 += 256) {
            const int x = x0 + lane * 4;
            if (x >= nr) continue;
            int4 c = *reinterpret_cast<const int4 *>(&rc[x]);
            if ((c.x | c.y | c.z | c.w) < 0) {
                c = make_int4(max(c.x, 0), max(c.y, 0), max(c.z, 0), max(c.w, 0));
                *reinterpret_cast<int4 *>(&rc[x]) = c;
            }
            m0 = max(max(m0, max(c.x, c.y)), max(c.z, c.w));
        }
        for (int x0 = wave * segC; x0 < min(nc, (wave + 1) * segC); x0 += 256) {
            const int x = x0 + lane * 4;
            if (x >= nc) continue;
            int4 c = *reinterpret_cast<const int4 *>(&cc[x]);
            if ((c.x | c.y | c.z | c.w) < 0) {
                c = make_int4(max(c.x, 0), max(c.y, 0), max(c.z, 0), max(c.w, 0));
                *reinterpret_cast<int4 *>(&cc[x]) = c;
            }
            m1 = max(max(m1, max(c.x, c.y)), max(c.z, c.w));
        }
        m0 = wave_max_nonneg_lane63(m0);
        m1 = wave_max_nonneg_lane63(m1);
        if (lane == 63) {
            atomicMax(&s_top[0], m0);
            atomicMax(&s_top[1], m1);
        }
        if (deep) __syncthreads();  // slots appended by an earlier batch are read from memory when they are split in turn
        else sync();
        const int c0 = s_top[0], c1 = s_top[1];  // cleared again in step 3, past the next barrier
        if (c0 <= 0 && c1 <= 0) break;
        const bool isrow = c0 >= c1;  // rows win ties (Alg. 4: "else if c0 >= c1")
        int32_t *cnt = isrow ? rc : cc, *other = isrow ? cc : rc;
        const SlotSet &mine = isrow ? g.rows : g.cols;
        const int N = isrow ? nr : nc;
        // (2) slots with lo <= count <= hi are split in this batch, numbered in index order
        const int hi = isrow ? c0 : c1;
        int lo = isrow ? max(c1, 1) : c0 + 1;
        const int least = (isrow ? deep_row : deep_col) + 1;  // appended slots hold fewer
        lo = min(hi, max(lo, least));
        // (1b) While the sequential algorithm stays on one side, the counts of that side do not change (no
        // entry has three digits) and only the top count of the other side falls, so the next batch would
        // be of the same kind with a lower bound: rows with count >= G(lo), G(lo) = top column count once
        // the rows with count >= lo are gone (columns: count >= F(lo) + 1).  Every slot down to the fixed
        // point of that recursion is split before the other side gets a turn, in (count descending, index)
        // order: one batch.  A read-only pass over the live entries evaluates G at lo, lo-1, lo-2, lo-3 at
        // once (four 8-bit counters per slot of the other side, kept in the unused upper half of that
        // side's count vector), which usually covers several steps of the recursion.  (With entries of three digits the
        // same holds down to `least`; such an entry outlives every bound.)
        // Tried only when the batch before was of the same kind: a side's first batch often is its only one.
        const bool again = prev_kind == (isrow ? 1 : 0);
        prev_kind = isrow ? 1 : 0;
        if (LDS && E > 0 && lo > max(least, 1) && again) {
            const int No = isrow ? nc : nr, No4 = (No + 3) & ~3;
            const int top_o = isrow ? c1 : c0;
            if (2 * No4 <= (isrow ? cpad : rpad) - 4 && top_o <= 255) {
                int32_t *tmp = other + No4;  // zero on entry (slots that do not exist yet) and on exit
                const unsigned long long *__restrict__ src = cur ? list1 : list0;
                if (threadIdx.x < 8) (&s_T[0][0])[threadIdx.x] = 0;
                sync();
                for (int round = 0; round < 256; ++round) {
                    int *T = s_T[round & 1];  // cleared above or during the round before
                    auto count_pass = [&](auto isrow_c, auto deep_c) __attribute__((always_inline)) {
                        constexpr bool IR = decltype(isrow_c)::value, DP = decltype(deep_c)::value;
                        auto outlives = [&](unsigned xs, unsigned os, unsigned levels, bool present) __attribute__((always_inline)) {
                            const int c = cnt[xs];  // slot 0's count is harmless for an absent entry ...
                            const int k = !present ? 0 : DP && levels > 2u ? 4 : min(4, max(0, lo - c));  // the entry outlives the bounds lo, .., lo - k + 1
                            if (k) atomicAdd(reinterpret_cast<unsigned *>(&tmp[os]), 0x01010101u >> (8 * (4 - k)));
                        };
                        if constexpr (RES) {
                            for (int e0 = threadIdx.x; e0 < E; e0 += kPlanThreads * UE) {
                                unsigned long long ed[UE];
#pragma unroll
                                for (int u = 0; u < UE; ++u) ed[u] = e0 + u * kPlanThreads < E ? held[e0 + u * kPlanThreads] : 0ull;
#pragma unroll
                                for (int u = 0; u < UE; ++u) {
                                    const unsigned wl = (unsigned)ed[u], wh = (unsigned)(ed[u] >> 32), el = wl & kEdgeSlotMask, eh = wh & kEdgeSlotMask;
                                    outlives(IR ? el : eh, IR ? eh : el, (wl >> kEdgeSlotBits) | (wh >> kEdgeSlotBits << 3), ed[u] != 0ull);
                                }
                            }
                            return;
                        }
                        constexpr int UW = 8;  // 16-byte loads (two entries each) per thread in flight
                        for (int e0 = 0; e0 < E; e0 += kPlanThreads * 2 * UW) {
                            unsigned long long ed[2 * UW];
#pragma unroll
                            for (int u = 0; u < UW; ++u) {
                                const int idx = e0 + (u * kPlanThreads + (int)threadIdx.x) * 2;
                                if (idx + 1 < E) {
                                    const ulonglong2 t = *reinterpret_cast<const ulonglong2 *>(src + idx);
                                    ed[2 * u] = t.x;
                                    ed[2 * u + 1] = t.y;
                                } else {
                                    ed[2 * u] = idx < E ? src[idx] : 0ull;
                                    ed[2 * u + 1] = 0ull;
                                }
                            }
#pragma unroll
                            for (int u = 0; u < 2 * UW; ++u) {
                                const unsigned wl = (unsigned)ed[u], wh = (unsigned)(ed[u] >> 32), el = wl & kEdgeSlotMask, eh = wh & kEdgeSlotMask;
                                outlives(IR ? el : eh, IR ? eh : el, (wl >> kEdgeSlotBits) | (wh >> kEdgeSlotBits << 3), ed[u] != 0ull);
                            }
                        }
                    };
                    if (SHORT || deep) {
                        if (isrow) count_pass(std::true_type{}, std::true_type{});
                        else count_pass(std::false_type{}, std::true_type{});
                    } else {
                        if (isrow) count_pass(std::true_type{}, std::false_type{});
                        else count_pass(std::false_type{}, std::false_type{});
                    }
                    sync();
                    int m0 = 0, m1 = 0, m2 = 0, m3 = 0;
                    if (threadIdx.x < 4) s_T[(round & 1) ^ 1][threadIdx.x] = 0;
                    for (int x = threadIdx.x * 4; x < No4; x += kPlanThreads * 4) {  // read and clear
                        const int4 v = *reinterpret_cast<const int4 *>(&tmp[x]);
                        *reinterpret_cast<int4 *>(&tmp[x]) = make_int4(0, 0, 0, 0);
                        const unsigned w4[4] = {(unsigned)v.x, (unsigned)v.y, (unsigned)v.z, (unsigned)v.w};
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            m0 = max(m0, (int)(w4[u] & 255u));
                            m1 = max(m1, (int)((w4[u] >> 8) & 255u));
                            m2 = max(m2, (int)((w4[u] >> 16) & 255u));
                            m3 = max(m3, (int)(w4[u] >> 24));
                        }
                    }
                    m0 = wave_max_nonneg_lane63(m0);
                    m1 = wave_max_nonneg_lane63(m1);
                    m2 = wave_max_nonneg_lane63(m2);
                    m3 = wave_max_nonneg_lane63(m3);
                    if (lane == 63) {
                        atomicMax(&T[0], m0);
                        atomicMax(&T[1], m1);
                        atomicMax(&T[2], m2);
                        atomicMax(&T[3], m3);
                    }
                    sync();
                    int now = lo;
                    bool stable = false;
                    for (int j = 0; j < 4; j = lo - now) {  // T[j]: the other side's top count with the bound lo - j
                        const int t = T[j];
                        const int next = max(isrow ? max(t, 1) : t + 1, least);
                        if (next >= now) {
                            stable = true;
                            break;
                        }
                        now = next;
                        if (now <= max(least, 1)) {  // nothing below that may be taken (without longer entries: every slot that holds one is)
                            stable = true;
                            break;
                        }
                    }
                    lo = now;
                    if (stable) break;
                }
                sync();  // the cleared counters and the last reads of T, before anything else touches them
            }
        }
        const int seg = isrow ? segR : segC;
        const int wlo = wave * seg, whi = min(N, wlo + seg);
        int found = 0, positive = 0;
        for (int x0 = wlo; x0 < whi; x0 += 256) {
            const int x = x0 + lane * 4;  // counts past slot N-1 (within the padding) are 0 < lo
            const int4 c = x < N ? *reinterpret_cast<const int4 *>(&cnt[x]) : make_int4(0, 0, 0, 0);
            found += __popcll(__ballot(c.x >= lo && c.x <= hi)) + __popcll(__ballot(c.y >= lo && c.y <= hi)) +
                     __popcll(__ballot(c.z >= lo && c.z <= hi)) + __popcll(__ballot(c.w >= lo && c.w <= hi));
            positive += __popcll(__ballot(c.x > 0)) + __popcll(__ballot(c.y > 0)) + __popcll(__ballot(c.z > 0)) +
                        __popcll(__ballot(c.w > 0));
        }
        if (lane == 0) {
            s_found[wave] = found;
            s_positive[wave] = positive;
        }
        sync();
        int run = 0, nb = 0, npos = 0;
#pragma unroll
        for (int w = 0; w < kPlanWaves; ++w) {
            const int c = s_found[w];
            if (w < wave) run += c;
            nb += c;
            npos += s_positive[w];
        }
        // If no entry has three or more digits and the batch takes every slot of its side that still
        // holds an OB entry, every live entry is finished by it: nothing is left to count.
        const bool finishes = !deep && nb == npos;
        if (N + nb > mine.cap || N + nb >= (1 << kEdgeSlotBits)) {
            if (threadIdx.x == 0) {
                if (N + nb >= (1 << kEdgeSlotBits)) atomicMin(&hdr->err, IMUNPACK_ERANGE);
                else flag_overflow(hdr, isrow ? g.whichR : g.whichC, 2 * (N + nb));
            }
            return;
        }
        // (3) the new slots; a split slot's count is replaced by a mark that names its new slot (only
        // the lane that owns a slot reads its count in steps 1-3).  The picked slots of a step are
        // first compacted into the wave's LDS list, so that the stores run over them densely.
        for (int x0 = wlo; x0 < whi; x0 += 256) {
            const int x = x0 + lane * 4;
            const int4 c = x < N ? *reinterpret_cast<const int4 *>(&cnt[x]) : make_int4(0, 0, 0, 0);
            const int cv[4] = {c.x, c.y, c.z, c.w};
            bool f[4];
            int before = 0, all = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                f[i] = cv[i] >= lo && cv[i] <= hi;
                const unsigned long long m = __ballot(f[i]);
                before += __popcll(m & below);
                all += __popcll(m);
            }
            if (all == 0) continue;  // uniform per wave
            int pos = before;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (f[i]) {
                    s_pick[wave][pos] = (min(cv[i], 0xFFFFFF) << 8) | (lane * 4 + i);
                    cnt[x + i] = -(run + pos + 1);
                    ++pos;
                }
            }
            for (int j = lane; j < all; j += 64) {
                const int pk = s_pick[wave][j];
                const int X = x0 + (pk & 0xFF), newX = N + run + j;
                const bool orig = X < (isrow ? nr0 : nc0);
                const int root = orig ? X : mine.root[X], ex = orig ? 0 : mine.exp[X];
                mine.time[X] = (uint32_t)bid;
                mine.child[X] = newX;
                mine.root[newX] = root;
                mine.exp[newX] = ex + 1;
                mine.time[newX] = kNever;
                mine.child[newX] = -1;
                mine.key[newX] = ((unsigned long long)bid << 48) |
                                 ((unsigned long long)(0xFFFFFF - (pk >> 8)) << 24) | (unsigned)X;
            }
            run += all;
        }
        if (threadIdx.x == 0) {
            s_count = 0;
            s_top[0] = s_top[1] = 0;
        }
        sync();
        if (finishes) {
            for (int x = threadIdx.x; x < rpad; x += kPlanThreads) rc[x] = 0;
            for (int x = threadIdx.x; x < cpad; x += kPlanThreads) cc[x] = 0;
            if (isrow) nr += nb; else nc += nb;
            break;
        }
        // (4) the pass
        if constexpr (RES) {
            auto pass = [&](auto isrow_c) __attribute__((always_inline)) {
                constexpr bool IR = decltype(isrow_c)::value;
                for (int e0 = threadIdx.x; e0 < E; e0 += kPlanThreads * UE) {
                    unsigned el[UE], eh[UE];
                    int c[UE];
#pragma unroll
                    for (int u = 0; u < UE; ++u) {
                        const unsigned long long ed = e0 + u * kPlanThreads < E ? held[e0 + u * kPlanThreads] : 0ull;
                        el[u] = (unsigned)ed;
                        eh[u] = (unsigned)(ed >> 32);
                    }
#pragma unroll
                    for (int u = 0; u < UE; ++u) c[u] = cnt[(IR ? el[u] : eh[u]) & kEdgeSlotMask];  // slot 0's is harmless for an absent edge
#pragma unroll
                    for (int u = 0; u < UE; ++u) {
                        if ((el[u] | eh[u]) == 0u || c[u] >= 0 || ~c[u] >= nb) continue;  // the mark -(k + 1) names new slot N + k
                        unsigned long long left = 0;  // finished
                        const unsigned levels = (el[u] >> kEdgeSlotBits) | ((eh[u] >> kEdgeSlotBits) << 3);
                        if (levels > 2u) {  // still OB in the new slot: move on, one digit fewer
                            const int newX = N + ~c[u];
                            atomicAdd(&cnt[newX], 1);
                            left = IR ? pack_edge(newX, (int)(eh[u] & kEdgeSlotMask), (int)levels - 1)
                                      : pack_edge((int)(el[u] & kEdgeSlotMask), newX, (int)levels - 1);
                        } else {
                            atomicSub(&other[(IR ? eh[u] : el[u]) & kEdgeSlotMask], 1);
                        }
                        held[e0 + u * kPlanThreads] = left;
                    }
                }
            };
            if (isrow) pass(std::true_type{});
            else pass(std::false_type{});
            sync();
            if (isrow) nr += nb; else nc += nb;
            continue;
        }
        // The survivors of a lane's entries are appended with one counter update per wave.
        unsigned long long *dst = cur ? list0 : list1;
        // One CU's vector ALU bounds this pass, so it is written for few instructions: the side of the batch
        // and whether entries can move on (three or more digits) are compile-time cases, the common case
        // (two digits: an entry of a split slot is simply finished) has one predicated LDS update per entry.
        auto process = [&](auto &e, auto isrow_c, auto deep_c) __attribute__((always_inline)) {  // e[u]: packed edge, 0 if absent
            constexpr bool IR = decltype(isrow_c)::value, DP = decltype(deep_c)::value;
            constexpr int UE = sizeof(e) / sizeof(unsigned long long);
            unsigned xw[UE], ow[UE];  // the word that names the slot on the batch's side, and the other one
            int c[UE];
#pragma unroll
            for (int u = 0; u < UE; ++u) {  // marks do not change during a pass; slot 0's count is harmless for absent edges
                const unsigned lo = (unsigned)e[u], hi = (unsigned)(e[u] >> 32);
                xw[u] = IR ? lo : hi;
                ow[u] = IR ? hi : lo;
                c[u] = cnt[xw[u] & kEdgeSlotMask];
            }
            int off[UE], all = 0;  // survivors are packed edge by edge: the lanes of a store write side by side
#pragma unroll
            for (int u = 0; u < UE; ++u) {
                bool live = (xw[u] | ow[u]) != 0u;
                const bool split = live && c[u] < 0 && ~c[u] < nb;  // the mark -(k + 1) names new slot N + k
                if constexpr (DP) {
                    if (split) {
                        const unsigned lo = IR ? xw[u] : ow[u], hi = IR ? ow[u] : xw[u];
                        const unsigned levels = (lo >> kEdgeSlotBits) | ((hi >> kEdgeSlotBits) << 3);
                        if (levels > 2u) {  // still OB in the new slot: move on, one digit fewer
                            const unsigned newX = (unsigned)(N + ~c[u]), lev = levels - 1u;
                            atomicAdd(&cnt[newX], 1);
                            const unsigned r = IR ? newX : (lo & kEdgeSlotMask), q = IR ? (hi & kEdgeSlotMask) : newX;
                            e[u] = pack_edge((int)r, (int)q, (int)lev);
                        } else {
                            atomicSub(&other[ow[u] & kEdgeSlotMask], 1);
                            live = false;
                        }
                    }
                } else {
                    if (split) atomicSub(&other[ow[u] & kEdgeSlotMask], 1);
                    live = live && !split;
                }
                const unsigned long long m = __ballot(live);
                const int before = (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
                off[u] = live ? all + before : -1;
                all += __popcll(m);
            }
            if (!all) return;
            int base = 0;
            if (lane == 0) base = atomicAdd(&s_count, all);
            base = __builtin_amdgcn_readfirstlane(base);
#pragma unroll
            for (int u = 0; u < UE; ++u)
                if (off[u] >= 0) dst[base + off[u]] = e[u];
        };
        auto run_pass = [&](auto isrow_c, auto deep_c) __attribute__((always_inline)) {  // the list of packed edges, two per load
            constexpr int U2 = 8;
            const unsigned long long *__restrict__ src = cur ? list1 : list0;
            auto fetch = [&](int e0, unsigned long long (&fe)[U2]) __attribute__((always_inline)) {
#pragma unroll
                for (int u = 0; u < U2; u += 2) {
                    const int idx = e0 + (u * kPlanThreads + (int)threadIdx.x * 2);
                    if (idx + 1 < E) {
                        const ulonglong2 t = *reinterpret_cast<const ulonglong2 *>(src + idx);
                        fe[u] = t.x;
                        fe[u + 1] = t.y;
                    } else {
                        fe[u] = idx < E ? src[idx] : 0ull;
                        fe[u + 1] = 0ull;
                    }
                }
            };
            unsigned long long ed[U2];
            fetch(0, ed);
            for (int e0 = 0; e0 < E; e0 += kPlanThreads * U2) {
                unsigned long long ed2[U2];
                fetch(e0 + kPlanThreads * U2, ed2);
                process(ed, isrow_c, deep_c);
#pragma unroll
                for (int u = 0; u < U2; ++u) ed[u] = ed2[u];
            }
        };
        if (deep) {
            if (isrow) run_pass(std::true_type{}, std::true_type{});
            else run_pass(std::false_type{}, std::true_type{});
        } else {
            if (isrow) run_pass(std::true_type{}, std::false_type{});
            else run_pass(std::false_type{}, std::false_type{});
        }
        __syncthreads();
        E = s_count;
        cur ^= 1;
        if (isrow) nr += nb; else nc += nb;
    }
    if (threadIdx.x == 0) {
        *(g.second ? &hdr->h_u : &hdr->n_u) = nr;
        *(g.second ? &hdr->d_u : &hdr->d1) = nc;
    }
}

// BITS: operands of few rows and columns; DEEP: three digits go by bits of 512 slots too
template <bool LDS, bool MAY_HOLD = LDS, bool BITS = false, bool DEEP = BITS>
__device__ __forceinline__ void greedy_both(const GreedyArgs &g, PlanHeader *hdr, int32_t *lds_counts) {
    __shared__ GreedyShared sh;
    const int nob = *g.ob_count, extras = g.chain_child ? load_agent(&hdr->extras) : 0;
    const int nr = g.second ? hdr->h_u : hdr->n_u;
    int deep = 0;
    for (int x = threadIdx.x; x < nr; x += kPlanThreads) deep |= g.rowmax[x] >= g.s * g.s;
    deep = __syncthreads_or(deep);
    constexpr bool SHORT = BITS || (LDS && !MAY_HOLD);
    if constexpr (BITS) {
        const int words = bits_words(max(nr, hdr->d1));
        if (words != 0 && words <= g.lds_words) {
            int longer = 0;
            if (deep) {
                for (int x = threadIdx.x; x < nr; x += kPlanThreads) longer |= g.rowmax[x] >= g.s * g.s * g.s;
                longer = __syncthreads_or(longer);
            }
            if (!longer && (DEEP || !deep || words == bits_words(256))) {
                unsigned *planes = reinterpret_cast<unsigned *>(lds_counts);
                const bool narrow = words == bits_words(256);
                if (narrow && !deep) greedy_bits<8, false>(g, hdr, planes, sh, nob, extras);
                else if (narrow) greedy_bits<8, true>(g, hdr, planes, sh, nob, extras);
                else if (!deep) greedy_bits<16, false>(g, hdr, planes, sh, nob, extras);
                else if constexpr (DEEP) greedy_bits<16, true>(g, hdr, planes, sh, nob, extras);
                return;
            }
        }
    }
    const long long E = (long long)nob + extras;
    const long long room = ((long long)g.lds_words - ((g.rows.cap + 7) & ~3) - ((g.cols.cap + 7) & ~3)) / 2;
    if (MAY_HOLD && E <= room) greedy_run<LDS, MAY_HOLD, SHORT>(g, hdr, lds_counts, sh, nob, extras, deep);
    else greedy_run<LDS, false, SHORT>(g, hdr, lds_counts, sh, nob, extras, deep);
}

// (BITS: a variant of its own, for the registers' sake)
template <bool LDS, bool BITS>
__global__ __launch_bounds__(kPlanThreads) void greedy_both_kernel(GreedyArgs g) {
    extern __shared__ __attribute__((aligned(16))) int32_t lds_counts[];
    PlanHeader *hdr = g.hdr + blockIdx.y;
    move_to_item(g);
    if (hdr->overflow) return;
    if (g.skip && *g.skip) return;
    greedy_both<LDS, LDS, BITS>(g, hdr, lds_counts);
}

// ---------------------------------------------------------------------------------------------
// physical layouts
// ---------------------------------------------------------------------------------------------
// Rows: source-major (all digit levels of a source row adjacent, level ascending), and no source
// row straddles a chunk of `chunk` physical rows: kChunk for A (four chunks per GEMM tile), so that Pi_A
// can be applied on the 64 rows the tile's epilogue holds in LDS at a time; kTile for B, whose levels
// are folded along the columns of a tile (kChunk there too if the 64 x 64 tiles of the small-tile GEMM may run).  Source row i with unpadded start P_i
// goes to chunk floor(P_i / (kChunk - (Lmax-1))): a closed form, and the rows of a chunk never exceed
// kChunk.  (Rows of A with nearly all the same number of levels: see `uniform`.)
// Bound by the latency of one workgroup's reads and stores, so rows beyond kRowSlice are shared out: every one of
// `nslices` workgroups derives the level counts and their sums for itself and writes its share of the rows.
constexpr int kRowSlice = 4096;  // source rows per workgroup, at most four workgroups (12608 rows of two levels: 34 -> 21 us)
__device__ void rows_layout(const SlotSet &rows, int nbase, const int32_t *count_dev, const RowLayout &lay,
                            int cap_phys, int cap_tiles, int32_t *tmpP_global, PlanHeader *hdr, int operand, int chunk,
                            int *lds, int32_t *fast /* 2 * nbase ints of LDS and one per chunk, or nullptr */, int slice, int nslices) {
    // the level counts and their running sums are scanned and searched over and over: in LDS when they fit
    int32_t *nlev = fast ? fast : lay.src_nlev;
    int32_t *tmpP = fast ? fast + nbase : tmpP_global;
    int32_t *chunk0 = fast ? fast + 2 * nbase : lay.chunk_src0;
    const int count = *count_dev;
    constexpr int V = 4;  // slots per thread and step, loaded side by side
    for (int i = threadIdx.x; i < nbase; i += kPlanThreads) nlev[i] = 1;
    __syncthreads();
    int lm = 1;
    for (int R0 = nbase + threadIdx.x; R0 < count; R0 += kPlanThreads * V) {
        int root[V], ex[V];
#pragma unroll
        for (int u = 0; u < V; ++u) {
            const int R = R0 + u * kPlanThreads;
            root[u] = R < count ? rows.root[R] : 0;
            ex[u] = R < count ? rows.exp[R] : 0;
        }
#pragma unroll
        for (int u = 0; u < V; ++u)
            if (ex[u] > 0) {
                atomicMax(&nlev[root[u]], ex[u] + 1);
                lm = max(lm, ex[u] + 1);
            }
    }
    const int lmax = block_max(lm, lds);
    const int base = ordered_scan(
        nbase, 0, [&](int x) { return nlev[x]; }, [&](int x, int pre) { tmpP[x] = pre; }, lds);
    // chunks of `chunk` physical rows (a divisor of kTile); source row i goes to chunk floor(P_i / Cp)
    int Cp = chunk - (lmax - 1);
    if (Cp < 1) {
        if (threadIdx.x == 0) atomicMin(&hdr->err, IMUNPACK_ERANGE);
        return;
    }
    int nchunks = nbase > 0 ? tmpP[nbase - 1] / Cp + 1 : 0;
    // Rows that (nearly) all have the same number of levels, two or four (three only where a chunk has the room): each gets two
    // or four physical rows, some of them padding, where that takes no more chunks.  Then the GEMM's epilogue stores from its
    // registers: a lane holds four physical rows of A side by side, so the levels of a row of A are neighbours; and it holds the
    // same column of every block of kEvenStep rows of B, so those of a row of B are that far apart.  Besides, nothing of a
    // chunk is lost: 4096 rows of A of four levels but 97 of three take 64 tiles instead of 67.
    int even = lmax == 1 || lmax > 4 ? 0 : lmax == 2 ? 2 : 4;
    static_assert(kEvenStep == 32 && kChunk == 64 && kTile == 256, "shifts below");
    const int step = operand ? kEvenStep : 1;  // from level to level, if so
    if (even * step > chunk) even = 0;         // (four levels of B do not fit the chunks of the small tiles)
    const int lg_chunk = chunk == kChunk ? 6 : 8, lg_even = even >> 1, lg_step = operand ? 5 : 0;
    const int most = (nbase + step - 1) / step * step;
    const bool uniform = even && (int64_t)most * even <= (int64_t)nchunks * chunk;
    if (uniform) {
        Cp = chunk;
        nchunks = (most * even + chunk - 1) / chunk;
    }
    const int total = uniform ? nbase * even : base;
    auto start = [&](int i) { return i >= nbase ? total : uniform ? i << lg_even : tmpP[i]; };
    const float per_chunk = 1.0f / (float)Cp;
    auto chunk_of = [&](int P) {  // P / Cp (a division takes some forty instructions)
        if (uniform) return P >> lg_chunk;
        if (base >= (1 << 24)) return P / Cp;
        const int q = (int)((float)P * per_chunk), r = P - q * Cp;  // off by one at most
        return q + (r >= Cp ? 1 : 0) - (r < 0 ? 1 : 0);
    };
    const int kPerTile = kTile / chunk;
    const int ntiles = (nchunks + kPerTile - 1) / kPerTile;
    const int Mp = ntiles * kTile;
    if (Mp > cap_phys || ntiles + 1 > cap_tiles || base != count) {
        if (threadIdx.x == 0) {
            if (base != count) atomicMin(&hdr->err, IMUNPACK_EHIP);  // inconsistent plan: internal error
            else flag_overflow(hdr, operand ? CAP_ROWB : CAP_ROWA, 2 * base);
        }
        return;
    }
    for (int ch = threadIdx.x; ch <= ntiles * kPerTile; ch += kPlanThreads) {
        // first i with P_i >= ch * Cp
        int lo = 0, hi = nbase;
        const int want = ch * Cp;
        if (uniform) lo = hi = min(nbase, ch << (lg_chunk - lg_even));
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (tmpP[mid] >= want) hi = mid; else lo = mid + 1;
        }
        chunk0[ch] = lo;
        if (slice == 0) {
            if (fast) lay.chunk_src0[ch] = lo;
            if (ch % kPerTile == 0) lay.tile_src0[ch / kPerTile] = lo;
        }
    }
    __syncthreads();
    if (slice == 0)
        for (int t = threadIdx.x; t < ntiles; t += kPlanThreads) {
            const int a = chunk0[t * kPerTile], e = chunk0[(t + 1) * kPerTile];
            const int slots = start(e) - start(a);
            // (rows of B in chunks: the tile's columns of C are read as one run, which gaps between the chunks break)
            lay.tile_flat[t] = (!uniform && slots == e - a && (operand == 0 || chunk == kTile || lmax == 1)) ? 1 : 0;
        }
    if (operand == 0) {  // a slice looks at the rows of its share of the chunks (all in one: 20 -> 24 us at 8880 rows of two and three levels)
        const int each = (nchunks + nslices - 1) / nslices, c0 = min(slice * each, nchunks), c1 = min(c0 + each, nchunks);
        for (int ch = c0 + threadIdx.x; ch < c1; ch += kPlanThreads) lay.chunk_lev[ch] = uniform ? even : lmax == 1 ? 1 : nlev[chunk0[ch]];
        if (!uniform && lmax > 1 && c0 < c1) {
            __syncthreads();
            for (int i = chunk0[c0] + threadIdx.x; i < chunk0[c1]; i += kPlanThreads) {
                const int ch = chunk_of(tmpP[i]);
                if (nlev[i] != nlev[chunk0[ch]]) lay.chunk_lev[ch] = 0;
            }
        }
    }
    const int threads = kPlanThreads * nslices, me = slice * kPlanThreads + threadIdx.x;
    // rows behind the last one of a chunk are padding, those of the levels that a row does not have too
    for (int p = me; p < Mp; p += threads) {
        const int ch = p >> lg_chunk, a = chunk0[ch], e = chunk0[ch + 1], at = p & (chunk - 1);
        bool none;
        if (uniform) {
            const int i = a + (at >> (lg_even + lg_step) << lg_step) + (at & (step - 1)), l = (at >> lg_step) & (even - 1);
            none = i >= e || l >= nlev[i];
        } else {
            none = at >= (a < e ? start(e) - start(a) : 0);
        }
        if (none) lay.prow[p] = -1;
        lay.rowsum[p] = 0;
    }
    if (lmax > 1) __syncthreads();  // the level counts have been looked at (where no row is split, nobody does)
    // where a source row starts takes the place of its level count (without LDS: of its own entry in the layout)
    int32_t *pstart = fast ? nlev : lay.src_pstart;
    for (int i = threadIdx.x; i < nbase; i += kPlanThreads) {
        const int P = start(i), ch = chunk_of(P);
        const int at = uniform ? (i >> lg_step << (lg_step + lg_even)) + (i & (step - 1)) : (ch << lg_chunk) + (P - start(chunk0[ch]));
        if (fast && slice == 0) {
            lay.src_nlev[i] = nlev[i];  // the GEMM epilogue reads both from memory
            lay.src_pstart[i] = at;
        }
        pstart[i] = at;
    }
    __syncthreads();
    for (int R0 = me; R0 < count; R0 += threads * V) {
        int root[V], ex[V];
#pragma unroll
        for (int u = 0; u < V; ++u) {
            const int R = R0 + u * threads;
            root[u] = R < nbase ? R : R < count ? rows.root[R] : -1;
            ex[u] = R >= nbase && R < count ? rows.exp[R] : 0;
        }
#pragma unroll
        for (int u = 0; u < V; ++u) {
            if (root[u] < 0) continue;
            const int at = pstart[root[u]] + ex[u] * (uniform ? step : 1);
            lay.prow[at] = root[u] | (ex[u] << kProwLevel);
            lay.row_phys[R0 + u * threads] = at;
        }
    }
    if (threadIdx.x == 0 && slice == 0) {
        if (operand == 0) { hdr->Mp = Mp; hdr->mtiles = ntiles; hdr->lmaxA = lmax; hdr->evenA = uniform ? even : 0; }
        else { hdr->Np = Mp; hdr->ntiles = ntiles; hdr->lmaxB = lmax; hdr->chunkB = chunk; hdr->evenB = uniform ? even : 0; }
    }
}

// Columns.  B_eu is laid out group by group (Alg. 3 runs one GEMM per distinct diagonal entry of S),
// highest exponent first, in whole k-tiles of kKPad columns.  A column slot c of the second unpacking
// descends from slot r = c2.root[c] of the first, which descends from original column k = c1.root[r];
// it holds digit level eB = c2.exp[c] of column r of B_e, its exponent is e = eA + eB with
// eA = c1.exp[r], and the column of A_ue beside it is a copy of column r of A_u.
// The A store holds A_u once: level a (the slots with eA = a) in ascending original column, padded to
// whole k-tiles; level 0 is the d original columns in place.  Inside group e the slots with eA = a
// form a subset of level a.  If that subset is (nearly) all of the level, the group walks the level's
// stored k-tiles as they are and B_eu gets a zero column where the level has a column the group has
// not ("shared": nothing of A is copied); otherwise the subset's columns are gathered, ordered by
// (original column, eA), into k-tiles of their own at the end of the group, and the columns of A they
// need are stored once more in extra blocks behind the levels ("gathered").
constexpr int kColBlocks = 8;    // workgroups that share the column layout, one exponent group at a time each
constexpr int kMaxLevelsA = 16;  // digit levels along the columns of A that the layout supports

__device__ __forceinline__ unsigned long long weight_of(int e, int sh) {  // s^e, saturating at 2^44
    const int bits = e * sh;
    return bits >= 44 ? (1ull << 44) : (1ull << bits);
}

// What the column layout knows of every group (exponent e) and every level a of A; one copy in LDS.
struct ColTables {
    int hist2[kMaxGroups * kMaxLevelsA];                   // column slots per (exponent e, level a of A)
    int kbase[kMaxGroups * kMaxLevelsA];                   // first column of B_eu of a shared (e, a), -1: gathered
    int cntA[kMaxLevelsA], lvlbase[kMaxLevelsA + 1];       // columns per level of A; first stored column
    int gk0[kMaxGroups], gext[kMaxGroups];                 // first column of a group and its extent
    int cbase[kMaxGroups], xbase[kMaxGroups], ccount[kMaxGroups];  // gathered: first column, first extra block, how many
    int kp, ka, ka_levels, bad, la;
    int lb, nsparse, list_col;                             // (of the path in LDS) columns taken from lists, the first of their run
    int unlisted;                                          // ... that could have been but hold too much
    unsigned digits;                                       // ... what those listed hold
    unsigned char tile_e[256], extra_e[256];               // group of every k-tile of B_eu / of every extra block of A
};

// Which appended columns the fused GEMM takes from lists (SparseLists), from steps with and without them on weights of scattered heavy
// hitters (columns x rows of B; us without -> with):
// * All that could be: lists beside a k-tile's worth of columns that hold more and are gathered.  (3030 of 4096 x 11008 listed and 1066
//   gathered: step of 4096 rows 526 -> 607.)  One column may hold a digit in kSparseMost rows.
// * A digit in kSparseShare rows on average.  4096 x 11008, 4096 rows of A: one in 500 510 -> 485 (resident weights 365 -> 326), in 400 514 -> 502
//   (365 -> 335), in 333 520 -> 514 (365 -> 342), in 250 528 -> 537 (370 -> 358); 1024 rows, resident: 145 -> 141, 145 -> 145, 145 -> 146.
// * At least kSparseLeast of them, and half of the original columns, for each of which their run in B_eu has a place.  Resident, one digit
//   in 1000 rows, 16 and 4096 rows of A: 1024 x 8192 59 -> 60 and 180 -> 183, 1280 62 -> 63 and 198 -> 197, 1536 66 -> 63 and 215 -> 211, 2048 68 -> 65 and
//   253 -> 234, 4096 x 11008 81 -> 77 and 401 -> 347.
// * Where B is unpacked in every step the lists and the copy of A cost the planner and the unpack some 10 us, which the GEMM has to save:
//   kSparseWork multiplications or more.  2048 x 8192, 1024, 2048 and 4096 rows: 214 -> 218, 255 -> 256, 337 -> 326; 1536 x 12288, 2048 and 4096:
//   217 -> 223, 348 -> 343; 4096 x 11008, 16, 1024, 4096: 232 -> 239, 304 -> 300, 575 -> 538.
constexpr int kSparseShare = 384, kSparseMost = 96, kSparseLeast = 1536;
constexpr int64_t kSparseWork = 1ll << 36;
constexpr int64_t kSparsePlaces = 1 << 26;   // in all lists
struct SparseArgs {
    const int32_t *colcnt;  // of B
    int h;
    int32_t *cnt;           // the lengths of the lists, cleared
};

// (the first wave)
__device__ __forceinline__ void level_bases(ColTables &t) {
    const int a = threadIdx.x, cnt = a < kMaxLevelsA ? t.cntA[a] : 0, padded = (cnt + kKPad - 1) / kKPad * kKPad;
    const int incl = wave_inclusive_sum(padded);
    const unsigned long long any = __ballot(cnt > 0);
    if (a <= kMaxLevelsA) t.lvlbase[a] = incl - padded;
    if (a == 63) {
        t.ka_levels = incl;
        t.la = any ? 64 - __builtin_clzll(any) : 1;
    }
}

// The k-tiles of every group, from hist2, cntA and the level bases: lane e of the first wave takes exponent e.  `report`:
// the workgroup that writes the run and group tables of the header.
__device__ void column_tables(ColTables &t, int cap_phys, int D, int s, int sh, PlanHeader *hdr, bool report) {
    if (threadIdx.x >= 64) return;
    const int e = threadIdx.x, la = t.la;  // (levels of A beyond it hold nothing)
    int tiles_sh = 0, ccount = 0, members = 0;
    for (int a = 0; a < kMaxLevelsA; ++a) {
        if (a >= la) {
            t.kbase[e * kMaxLevelsA + a] = -1;
            continue;
        }
        const int m = t.hist2[e * kMaxLevelsA + a];
        members += m;
        const bool shared = m > 0 && (long long)m * 8 >= (long long)t.cntA[a] * 7;
        t.kbase[e * kMaxLevelsA + a] = shared ? tiles_sh * kKPad : -1;  // relative to the group's start for now
        if (shared) tiles_sh += (t.cntA[a] + kKPad - 1) / kKPad;
        else ccount += m;
    }
    const int tiles_l = t.nsparse ? (t.cntA[0] + kKPad - 1) / kKPad : 0;  // the run that the fused GEMM leaves out
    if (e == 1) members += t.nsparse;
    const int tiles_c = (ccount + kKPad - 1) / kKPad;
    const int tiles = tiles_sh + tiles_c;
    int nrun = tiles_c > 0 ? 1 : 0;  // stretches of k-tiles that walk consecutive blocks of the A store
    for (int a = 0; a < la; ++a)
        if (t.kbase[e * kMaxLevelsA + a] >= 0) ++nrun;
    // groups come highest exponent first: sums over the lanes above this one
    int above = tiles, above_c = tiles_c, above_n = members > 0 ? 1 : 0, above_r = nrun;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int t0 = __shfl_down(above, off, 64), t1 = __shfl_down(above_c, off, 64), t2 = __shfl_down(above_n, off, 64),
                  t3 = __shfl_down(above_r, off, 64);
        if (e + off < 64) { above += t0; above_c += t1; above_n += t2; above_r += t3; }
    }
    const int k0 = (above - tiles) * kKPad, xb = above_c - tiles_c, g = above_n - (members > 0 ? 1 : 0);
    if (report) {
        int ri = above_r - nrun;
        for (int a = 0; a < kMaxLevelsA; ++a) {
            const int kb = t.kbase[e * kMaxLevelsA + a];
            if (kb < 0) continue;
            if (ri < kMaxRuns) {
                hdr->run_kt0[ri] = (k0 + kb) / kKPad;
                hdr->run_blk0[ri] = t.lvlbase[a] / kKPad;
                hdr->run_grp[ri] = g;
            }
            ++ri;
        }
        if (tiles_c > 0 && ri < kMaxRuns) {
            hdr->run_kt0[ri] = k0 / kKPad + tiles_sh;
            hdr->run_blk0[ri] = t.ka_levels / kKPad + xb;
            hdr->run_grp[ri] = g;
        }
        const int total_r = __shfl(above_r, 0, 64), dense = __shfl(above, 0, 64);
        if (e == 0) {
            hdr->nruns = total_r + (tiles_l ? 1 : 0);
            if (hdr->nruns > kMaxRuns) atomicMin(&hdr->err, IMUNPACK_ERANGE);
        }
        if (e == 1 && tiles_l && total_r < kMaxRuns) {  // behind all groups, beside level 0
            hdr->run_kt0[total_r] = dense;
            hdr->run_blk0[total_r] = 0;
            hdr->run_grp[total_r] = g;
        }
    }
    for (int a = 0; a < la; ++a)
        if (t.kbase[e * kMaxLevelsA + a] >= 0) t.kbase[e * kMaxLevelsA + a] += k0;
    t.cbase[e] = k0 + tiles_sh * kKPad;
    t.xbase[e] = xb;
    t.ccount[e] = ccount;
    t.gk0[e] = k0;
    t.gext[e] = tiles * kKPad;
    const int dense_tiles = __shfl(above, 0, 64), total_c = __shfl(above_c, 0, 64), ngroups = __shfl(above_n, 0, 64);
    const int total_tiles = dense_tiles + tiles_l;
    if (e == 0) {
        t.list_col = dense_tiles * kKPad;
        t.kp = total_tiles * kKPad;
        t.ka = t.ka_levels + total_c * kKPad;
    }
    if (members > 0) {
        const long long lim = 2147483647ll / ((long long)(s - 1) * (s - 1));
        if (e * sh > 62 || (tiles + (e == 1 ? tiles_l : 0)) * kKPad > lim) atomicMin(&hdr->err, IMUNPACK_ERANGE);
        if (report) {
            hdr->grp_exp[g] = e;
            hdr->grp_k0[g] = k0;
            hdr->grp_len[g] = tiles * kKPad;
        }
    }
    if (report && e == 0) {
        hdr->ngroups = ngroups;
        hdr->nsparse = t.nsparse;
        hdr->list_kt0 = dense_tiles;
        hdr->Kp = total_tiles * kKPad;
        hdr->KA = t.ka_levels + total_c * kKPad;
        // row pitches: wide rows get an odd multiple of 256 bytes (power-of-two strides put the rows
        // of a tile, which are read together, on the same few memory channels)
        const int wa = t.ka_levels + total_c * kKPad, wb = total_tiles * kKPad;
        hdr->ldA = wa >= 2048 ? (((wa + 255) / 256) | 1) * 256 : wa;
        hdr->ldB = wb >= 2048 ? (((wb + 255) / 256) | 1) * 256 : wb;
        if (total_tiles * kKPad > cap_phys) flag_overflow(hdr, CAP_C2, 2 * D);
    }
    for (int i = 0; i < tiles && k0 / kKPad + i < 256; ++i) t.tile_e[k0 / kKPad + i] = (unsigned char)e;
    for (int i = 0; i < tiles_c && xb + i < 256; ++i) t.extra_e[xb + i] = (unsigned char)e;
    if (e == 1)
        for (int i = 0; i < tiles_l && dense_tiles + i < 256; ++i) t.tile_e[dense_tiles + i] = 1;
}

// The same layout for unpackings whose tables fit the LDS of one workgroup (every product up to 12288 column slots):
// the general path below is a chain of phases that hand arrays to one another through memory, a microsecond or more per
// dependent read, and its workgroups end in a device-wide fence that writes back the L2 of their XCD (24 to 54 us for one
// product, 70 to 170 us for the items of a batch; this one: 14 to 37 and 14 to 16).  Here every slot stays in the registers of its thread.  A column slot is
// known by its original column k and its levels eA, eB along A and B, and no two slots share all three; so the slots are a
// bit per k in a mask per (eA, eB), every rank is a count of bits below k, and the columns of both stores are put together
// in LDS and written once, 1024 at a time by the parts in turn (every part puts all of them together; by one workgroup alone the
// layouts of 4096 x 8192 by 4096 took 40 us instead of 28, of 12288 slots 36 instead of 28).  Returns false, having written nothing but tables that are written again, if LDS is too
// small: the same in every part, so that all of them take the general path (many pairs of levels: 300 x 9000 by 300 at b = 2
// with eight levels on either side, a plan of 204 us in eight parts, 312 in one).
constexpr int kListed = 1 << 30;   // (of a slot's levels) its column is taken from lists
constexpr int kColSlotsLds = 12;  // slots per thread: as many as the registers of a 1024-thread workgroup hold
template <int kSlots, bool LISTS>
__device__ bool cols_layout_lds(const SlotSet &c1, const SlotSet &c2, const ColLayout &cols, int d, int cap_phys, int s, int sh,
                                PlanHeader *hdr, ColTables &t, int32_t *dyn, int dyn_words, int part, int parts, const SparseArgs &sp) {
    const int D = hdr->d_u, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (D > kSlots * kPlanThreads) return false;
    for (int x = tid; x < kMaxGroups * kMaxLevelsA; x += kPlanThreads) t.hist2[x] = 0;
    if (tid == 0) t.la = t.lb = t.bad = t.nsparse = t.unlisted = t.digits = 0;
    int key[kSlots], lev[kSlots];  // original column; eA | eB << 16
#pragma unroll
    for (int u = 0; u < kSlots; ++u) {
        const int c = tid + u * kPlanThreads;
        key[u] = -1;
        lev[u] = 0;
        if (u * kPlanThreads >= D) continue;  // uniform
        key[u] = c < D ? c2.root[c] : -1;
        lev[u] = c < D ? c2.exp[c] << 16 : 0;
    }
    int ma = 0, mb = 0;
#pragma unroll
    for (int u = 0; u < kSlots; ++u) {
        if (key[u] < 0) continue;
        const int r = key[u], ea = c1.exp[r];
        key[u] = c1.root[r];
        ma = max(ma, ea);
        mb = max(mb, lev[u] >> 16);
        lev[u] |= ea;
    }
    ma = wave_max_nonneg_lane63(ma);
    mb = wave_max_nonneg_lane63(mb);
    __syncthreads();
    if (lane == 63) {
        atomicMax(&t.la, ma);
        atomicMax(&t.lb, mb);
    }
    __syncthreads();
    const int LA = t.la + 1, LB = t.lb + 1, W = (d + 63) / 64;
    // what the stored columns of both operands cannot exceed, -1 if LDS and the tables may not hold them (see below for what has to)
    auto most_columns = [&](bool listed) {
        const int mine = LA * LB + (listed ? 1 : 0), appended = D - d, pads = kKPad * (LA * LB + LA + LB);
        const int kp = d + appended + appended / 7 + pads + (listed ? d : 0), ka = hdr->d1 + appended + pads;
        return LA <= kMaxLevelsA && LA + LB - 1 <= kMaxGroups && mine + LA + LB <= kMaxRuns && kp <= 256 * kKPad && appended + pads <= 256 * kKPad &&
               (long long)mine * W * 3 + kp + ka <= dyn_words ? kp + ka : -1;
    };
    if (LISTS && LB > 1) {
        const int most = sp.h / kSparseMost;
        unsigned found = 0, rest = 0, digits = 0;
#pragma unroll
        for (int u = 0; u < kSlots; ++u) {
            if (key[u] < 0 || lev[u] != 1 << 16) continue;
            const int cnt = sp.colcnt[key[u]];
            if (cnt <= most) {
                lev[u] |= kListed;
                ++found;
                digits += cnt;
            } else {
                ++rest;
            }
        }
        found = wave_sum_lane63(found);
        rest = wave_sum_lane63(rest);
        digits = wave_sum_lane63(digits);
        if (lane == 63) {
            atomicAdd(&t.nsparse, (int)found);
            atomicAdd(&t.unlisted, (int)rest);
            atomicAdd(&t.digits, digits);
        }
        __syncthreads();
        if (t.nsparse < kSparseLeast || t.nsparse * 2 < d || t.unlisted > kKPad || (unsigned long long)t.digits * kSparseShare > (unsigned long long)t.nsparse * sp.h ||
            most_columns(true) < 0) {  // uniform
#pragma unroll
            for (int u = 0; u < kSlots; ++u) lev[u] &= ~kListed;
            __syncthreads();
            if (tid == 0) t.nsparse = 0;
            __syncthreads();
        }
    }
    const int lists = LA * LB, pairs = lists + (LISTS && t.nsparse ? 1 : 0);  // the columns taken from lists have a mask of their own
    if (LA > kMaxLevelsA || LA + LB - 1 > kMaxGroups || (long long)pairs * W * 3 > dyn_words) return false;
    if (part > 0) {  // where it is certain to fit, parts that will have nothing to write need not find out
        const int most = most_columns(pairs > lists);
        if (most >= 0 && part * kPlanThreads >= most + kPlanThreads) return true;
    }
    unsigned long long *mask = reinterpret_cast<unsigned long long *>(dyn);  // [pairs][W]
    int32_t *pre = dyn + 2 * pairs * W;                                       // [pairs][W] slots of the pair below the word
    int32_t *packB = pre + pairs * W;                                         // k | eB << 24 per column of B_eu, -1: none
    auto pair_of = [=](int l) { return LISTS && l & kListed ? lists : (l & 0xffff) * LB + (l >> 16); };
    if (pairs * W * (3 + 16) <= dyn_words) {  // a byte per k first, where the stores will be put together (atomics on the
                                                // masks would queue up 32 to a word)
        unsigned char *seen = reinterpret_cast<unsigned char *>(packB);
        for (int x = tid; x < pairs * W * 16; x += kPlanThreads) packB[x] = 0;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kSlots; ++u)
            if (key[u] >= 0) seen[pair_of(lev[u]) * W * 64 + key[u]] = 1;
        __syncthreads();
        for (int x = wave; x < pairs * W; x += kPlanWaves) {
            const unsigned long long m = __ballot(seen[x * 64 + lane] != 0);
            if (lane == 0) mask[x] = m;
        }
    } else {
        for (int x = tid; x < 2 * pairs * W; x += kPlanThreads) dyn[x] = 0;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kSlots; ++u) {
            if (key[u] < 0) continue;
            const int k = key[u], pair = pair_of(lev[u]);
            atomicOr(reinterpret_cast<unsigned *>(mask) + 2 * pair * W + (k >> 5), 1u << (k & 31));
        }
    }
    __syncthreads();
    for (int pair = wave; pair < LA * LB; pair += kPlanWaves) {
        int run = 0;
        for (int w0 = 0; w0 < W; w0 += 64) {
            const int w = w0 + lane;
            const int c = w < W ? __popcll(mask[pair * W + w]) : 0;
            const int incl = wave_inclusive_sum(c);
            if (w < W) pre[pair * W + w] = run + incl - c;
            run += from_lane63(incl);
        }
        const int a = pair / LB, eb = pair - a * LB;
        if (lane == 0) {
            t.hist2[(a + eb) * kMaxLevelsA + a] = run;
            if (eb == 0) t.cntA[a] = run;
        }
    }
    if (tid >= LA && tid < kMaxLevelsA) t.cntA[tid] = 0;
    __syncthreads();
    if (tid < 64) level_bases(t);
    __syncthreads();
    column_tables(t, cap_phys, D, s, sh, hdr, part == 0);
    __syncthreads();
    const int Kp = t.kp, KA = t.ka, ka_levels = t.ka_levels;
    if (Kp > cap_phys) return true;  // reported: the plan is made again with more room
    if (Kp > 256 * kKPad || KA - ka_levels > 256 * kKPad || (long long)pairs * W * 3 + Kp + KA > dyn_words) return false;
    int32_t *packA = packB + Kp;  // k | eA << 24 per stored column of A, -1: none
    for (int x = tid; x < Kp + KA; x += kPlanThreads) packB[x] = -1;
    __syncthreads();
    auto bit = [&](int pair, int k) { return (int)(mask[pair * W + (k >> 6)] >> (k & 63)) & 1; };
    auto rank = [&](int pair, int k) {
        return pre[pair * W + (k >> 6)] + __popcll(mask[pair * W + (k >> 6)] & ((1ull << (k & 63)) - 1ull));
    };
#pragma unroll
    for (int u = 0; u < kSlots; ++u) {
        if (key[u] < 0) continue;
        const int c = tid + u * kPlanThreads, k = key[u], a = lev[u] & 0xffff, eb = lev[u] >> 16, e = a + eb;
        auto placed = [&](int q, int qa) {
            if (u % parts != part) return;  // uniform
            cols.pcol_slot[q] = c;
            cols.col_phys[c] = q;
            cols.acol_phys[c] = qa;
        };
        if (LISTS && lev[u] & kListed) {  // beside level 0 of A, which holds column k in place
            packB[t.list_col + k] = k | (1 << 24);
            placed(t.list_col + k, k);
            continue;
        }
        const int stored = t.lvlbase[a] + rank(a * LB, k);  // where level a of A holds column k
        const int kb = t.kbase[e * kMaxLevelsA + a];
        int q, qa;
        if (kb >= 0) {
            qa = stored;
            q = kb + (qa - t.lvlbase[a]);
        } else {  // gathered: behind the group's members with a lower (k, level of A)
            int pos = 0;
            for (int x = 0; x < LA && x <= e; ++x) {
                if (e - x >= LB || t.kbase[e * kMaxLevelsA + x] >= 0) continue;
                pos += rank(x * LB + e - x, k);
                if (x < a) pos += bit(x * LB + e - x, k);
            }
            q = t.cbase[e] + pos;
            qa = ka_levels + t.xbase[e] * kKPad + pos;
            packA[qa] = k | (a << 24);
        }
        packB[q] = k | (eb << 24);
        if (eb == 0) packA[stored] = k | (a << 24);
        placed(q, qa);
    }
    __syncthreads();
    // ---- out: sixteen lanes side by side hold a unit (both widths are multiples of 128); its first lane with a column
    // describes it (the first of all if none has)
    const int step = parts * kPlanThreads, firstA = (part + parts - (Kp + kPlanThreads - 1) / kPlanThreads % parts) % parts;
    auto in_unit = [&](bool f) { return (unsigned)(__ballot(f) >> (lane & 48)) & 0xffffu; };
    auto from = [&](int v, int l) { return __shfl(v, l, 64); };
    for (int q = tid + part * kPlanThreads; q < Kp; q += step) {
        const int v = packB[q], k = v == -1 ? -1 : v & 0xffffff, eb = v == -1 ? 0 : (v >> 24) & 0xff, e = t.tile_e[q / kKPad];
        cols.colB_k[q] = k;
        cols.colB_e[q] = eb;
        cols.col_sexp[q] = e;
        if (k < 0) cols.pcol_slot[q] = -1;
        const unsigned live = in_unit(k >= 0);
        const int first = (lane & 48) + (live ? __builtin_ctz(live) : 0);
        const int before = IMU_DPP(k, 0x111, 0xf, true);  // the column one to the left
        const bool run = in_unit(k >= 0 && ((lane & 15) == 0 || k == before + 1)) == 0xffffu;
        const bool uniform = in_unit(k < 0 || eb == from(eb, first)) == 0xffffu;
        if (lane == first) cols.unitB[q / 16] = make_int4(k, k, (run ? 1 : 0) | (uniform ? 2 : 0) | 4, eb | (e << 16));
    }
    for (int q = tid + firstA * kPlanThreads; q < KA; q += step) {
        const int v = packA[q], k = v == -1 ? -1 : v & 0xffffff, a = v == -1 ? 0 : (v >> 24) & 0xff;
        unsigned long long w = 0;  // what an entry of the column weighs: s^e over the slots that read it
        if (k >= 0) {
            if (q >= ka_levels) {
                w = weight_of(t.extra_e[(q - ka_levels) / kKPad], sh);
            } else {
                for (int eb = 0; eb < LB; ++eb)
                    if (t.kbase[(a + eb) * kMaxLevelsA + a] >= 0 && bit(a * LB + eb, k)) w += weight_of(a + eb, sh);
                if (LISTS && a == 0 && pairs > lists && bit(lists, k)) w += weight_of(1, sh);
            }
        }
        cols.colA_k[q] = k;
        cols.colA_e[q] = a;
        cols.colA_w[q] = w;
        const unsigned live = in_unit(k >= 0);
        const int first = (lane & 48) + (live ? __builtin_ctz(live) : 0);
        const int before = IMU_DPP(k, 0x111, 0xf, true);
        const bool run = in_unit(k >= 0 && ((lane & 15) == 0 || k == before + 1)) == 0xffffu;
        const bool uniform = in_unit(k < 0 || a == from(a, first)) == 0xffffu;
        const bool onew = in_unit(k < 0 || (unsigned)w == (unsigned)from((int)(unsigned)w, first)) == 0xffffu &&
                          in_unit(k < 0 || (unsigned)(w >> 32) == (unsigned)from((int)(unsigned)(w >> 32), first)) == 0xffffu;
        if (lane == first) {
            cols.unitA[q / 16] = make_int4(k, k, (run ? 1 : 0) | (uniform ? 2 : 0) | (onew ? 4 : 0), a);
            cols.unitA_w[q / 16] = w < (1ull << 44) ? w : (1ull << 44);
        }
    }
    return true;
}

__device__ void cols_layout(const SlotSet &c1, const SlotSet &c2, const ColLayout &cols, int d, int cap_phys,
                            int s, int sh, int32_t *tmpE, int32_t *tmpK, int32_t *tmpR, int32_t *tmpOffAll,
                            PlanHeader *hdr, int *lds, int part, int nparts, ColTables &t) {
    auto &hist2 = t.hist2;
    auto &cntA = t.cntA;
    auto &lvlbase = t.lvlbase;
    auto &kbase = t.kbase;
    auto &s_gk0 = t.gk0;
    auto &s_gext = t.gext;
    auto &s_cbase = t.cbase;
    auto &s_xbase = t.xbase;
    auto &s_ccount = t.ccount;
    const int D = hdr->d_u, D1 = hdr->d1;
    int32_t *tmpOff = tmpOffAll + (size_t)part * (d + 1);
    for (int x = threadIdx.x; x < kMaxGroups * kMaxLevelsA; x += kPlanThreads) hist2[x] = 0;
    if (threadIdx.x < kMaxLevelsA) cntA[threadIdx.x] = 0;
    if (threadIdx.x == 0) t.bad = t.nsparse = 0;  // (every column is stored here)
    __syncthreads();
    // every part computes the same per-slot values and the same tables (the stores of the parts
    // coincide); a part then lays out the groups part, part + kColBlocks, ...
    constexpr int V = 8;  // slots per thread and step, loaded side by side
    // ---- levels of A
    for (int r0 = threadIdx.x; r0 < D1; r0 += kPlanThreads * V) {
        int a[V];
#pragma unroll
        for (int u = 0; u < V; ++u) a[u] = r0 + u * kPlanThreads < D1 ? c1.exp[r0 + u * kPlanThreads] : -1;
#pragma unroll
        for (int u = 0; u < V; ++u) {
            if (a[u] < 0) continue;
            if (a[u] < kMaxLevelsA) atomicAdd(&cntA[a[u]], 1);
            else t.bad = 1;
        }
    }
    __syncthreads();
    if (threadIdx.x < 64) level_bases(t);
    __syncthreads();
    const int la = t.la;
    // ---- stored column of every column slot of A's unpacking: level 0 in place, level a >= 1 by rank
    // among the original columns whose chain reaches that level
    for (int k = threadIdx.x; k < d; k += kPlanThreads) cols.apos[k] = k;
    for (int a = 1; a < la; ++a) {
        auto slot_at = [&](int k) {
            int r = k;
            for (int i = 0; i < a && r >= 0; ++i) r = c1.child[r];
            return r;
        };
        ordered_select(
            d, lvlbase[a], [&](int k) { return slot_at(k) >= 0; },
            [&](int k, int pos) { cols.apos[slot_at(k)] = pos; }, lds);
    }
    // ---- per column slot of the second unpacking: exponent, levels, original column
    for (int c0 = threadIdx.x; c0 < D; c0 += kPlanThreads * V) {
        int r[V], eb[V], ea[V], k[V];
#pragma unroll
        for (int u = 0; u < V; ++u) {
            const int c = c0 + u * kPlanThreads;
            r[u] = c < D ? c2.root[c] : 0;
            eb[u] = c < D ? c2.exp[c] : 0;
        }
#pragma unroll
        for (int u = 0; u < V; ++u) {
            ea[u] = c1.exp[r[u]];
            k[u] = c1.root[r[u]];
        }
#pragma unroll
        for (int u = 0; u < V; ++u) {
            const int c = c0 + u * kPlanThreads;
            if (c >= D) continue;
            const int e = ea[u] + eb[u];
            tmpE[c] = e | (ea[u] << 8) | (eb[u] << 16);
            tmpK[c] = k[u];
            tmpR[c] = r[u];
            if (e < kMaxGroups && ea[u] < kMaxLevelsA && eb[u] < 256) {
                atomicAdd(&hist2[e * kMaxLevelsA + ea[u]], 1);
            } else {
                atomicMin(&hdr->err, IMUNPACK_ERANGE);
                t.bad = 1;
            }
        }
    }
    __syncthreads();
    column_tables(t, cap_phys, D, s, sh, hdr, part == 0);
    __syncthreads();
    const int Kp = t.kp, KA = t.ka, ka_levels = t.ka_levels;
    if (Kp > cap_phys || t.bad) return;
    if (nparts == 1) {  // (several workgroups add to weights that an earlier launch has cleared)
        for (int q = threadIdx.x; q < KA; q += kPlanThreads) cols.colA_w[q] = 0;
        __syncthreads();
    }
    // ---- the stored levels of A (first part)
    if (part == 0) {
        for (int q = threadIdx.x; q < ka_levels; q += kPlanThreads) {
            cols.colA_k[q] = -1;
            cols.colA_e[q] = 0;
        }
        __syncthreads();
        for (int r = threadIdx.x; r < D1; r += kPlanThreads) {
            const int q = cols.apos[r];
            cols.colA_k[q] = c1.root[r];
            cols.colA_e[q] = c1.exp[r];
        }
    }
    for (int e = kMaxGroups - 1 - part; e >= 0; e -= nparts) {  // any fixed assignment of groups to parts will do
        const int q0 = s_gk0[e], q1 = q0 + s_gext[e];
        if (q1 == q0) continue;  // uniform
        for (int q = q0 + threadIdx.x; q < q1; q += kPlanThreads) {
            cols.pcol_slot[q] = -1;
            cols.colB_k[q] = -1;
            cols.colB_e[q] = 0;
            cols.col_sexp[q] = e;
        }
        const int cbase = s_cbase[e], ccount = s_ccount[e], xcol0 = ka_levels + s_xbase[e] * kKPad;
        const int ctiles = (ccount + kKPad - 1) / kKPad;
        for (int q = threadIdx.x; q < ctiles * kKPad; q += kPlanThreads) {
            cols.colA_k[xcol0 + q] = -1;
            cols.colA_e[xcol0 + q] = 0;
            cols.colA_w[xcol0 + q] = 0;
        }
        if (ccount > 0)
            for (int k = threadIdx.x; k < d; k += kPlanThreads) tmpOff[k] = 0;
        __syncthreads();
        const unsigned long long w = weight_of(e, sh);
        // shared members go where their column of A is stored; gathered ones are counted per original column
        for (int c0 = threadIdx.x; c0 < D; c0 += kPlanThreads * V) {
            int pe[V], k[V], rr[V];
#pragma unroll
            for (int u = 0; u < V; ++u) {
                const int c = c0 + u * kPlanThreads;
                pe[u] = c < D ? tmpE[c] : -1;
                k[u] = c < D ? tmpK[c] : 0;
                rr[u] = c < D ? tmpR[c] : 0;
            }
#pragma unroll
            for (int u = 0; u < V; ++u) {
                if (pe[u] < 0 || (pe[u] & 0xFF) != e) continue;
                const int a = (pe[u] >> 8) & 0xFF, kb = kbase[e * kMaxLevelsA + a];
                if (kb < 0) {
                    atomicAdd(&tmpOff[k[u]], 1);
                    continue;
                }
                const int c = c0 + u * kPlanThreads, qa = cols.apos[rr[u]], q = kb + (qa - lvlbase[a]);
                cols.pcol_slot[q] = c;
                cols.colB_k[q] = k[u];
                cols.colB_e[q] = (pe[u] >> 16) & 0xFF;
                cols.col_phys[c] = q;
                cols.acol_phys[c] = qa;
                atomicAdd(&cols.colA_w[qa], w);
            }
        }
        if (ccount > 0) {  // uniform
            __syncthreads();
            ordered_scan(
                d, cbase, [&](int k) { return tmpOff[k]; }, [&](int k, int pre) { tmpOff[k] = pre; }, lds);
            for (int c0 = threadIdx.x; c0 < D; c0 += kPlanThreads * V) {
                int pe[V], k[V], q[V];
#pragma unroll
                for (int u = 0; u < V; ++u) {
                    const int c = c0 + u * kPlanThreads;
                    pe[u] = c < D ? tmpE[c] : -1;
                    k[u] = c < D ? tmpK[c] : 0;
                }
#pragma unroll
                for (int u = 0; u < V; ++u) {
                    if (pe[u] < 0 || (pe[u] & 0xFF) != e || kbase[e * kMaxLevelsA + ((pe[u] >> 8) & 0xFF)] >= 0) pe[u] = -1;
                    q[u] = pe[u] >= 0 ? atomicAdd(&tmpOff[k[u]], 1) : 0;
                }
#pragma unroll
                for (int u = 0; u < V; ++u) {
                    if (pe[u] < 0) continue;
                    cols.pcol_slot[q[u]] = c0 + u * kPlanThreads;
                    cols.colB_k[q[u]] = k[u];
                    cols.colB_e[q[u]] = (pe[u] >> 16) & 0xFF;
                    cols.colA_e[xcol0 + (q[u] - cbase)] = (pe[u] >> 8) & 0xFF;
                }
            }
            __syncthreads();
            // gathered columns of one group that copy the same original column: order them by their level along A
            for (int k = threadIdx.x; k < d; k += kPlanThreads) {
                const int end = tmpOff[k], beg = k ? tmpOff[k - 1] : cbase;
                for (int i = beg + 1; i < end; ++i) {
                    const int slot = cols.pcol_slot[i], ea = cols.colA_e[xcol0 + (i - cbase)], eb = cols.colB_e[i];
                    int j = i - 1;
                    while (j >= beg && cols.colA_e[xcol0 + (j - cbase)] > ea) {
                        cols.pcol_slot[j + 1] = cols.pcol_slot[j];
                        cols.colA_e[xcol0 + (j + 1 - cbase)] = cols.colA_e[xcol0 + (j - cbase)];
                        cols.colB_e[j + 1] = cols.colB_e[j];
                        --j;
                    }
                    cols.pcol_slot[j + 1] = slot;
                    cols.colA_e[xcol0 + (j + 1 - cbase)] = ea;
                    cols.colB_e[j + 1] = eb;
                }
            }
            __syncthreads();
            for (int q = cbase + threadIdx.x; q < cbase + ccount; q += kPlanThreads) {
                const int c = cols.pcol_slot[q], qa = xcol0 + (q - cbase);
                cols.col_phys[c] = q;
                cols.acol_phys[c] = qa;
                cols.colA_k[qa] = cols.colB_k[q];
                cols.colA_w[qa] = w;
            }
        }
        __syncthreads();
        // per 16-column unit of B_eu: what the scatter kernel needs to pick its path without the per-column arrays
        for (int u = q0 / 16 + threadIdx.x; u < q1 / 16; u += kPlanThreads) {
            const int qq = 16 * u;
            int kk[16], ee[16];  // all sixteen columns' words at once: one round trip instead of sixteen
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int4 a = reinterpret_cast<const int4 *>(cols.colB_k + qq)[v], b = reinterpret_cast<const int4 *>(cols.colB_e + qq)[v];
                kk[4 * v] = a.x; kk[4 * v + 1] = a.y; kk[4 * v + 2] = a.z; kk[4 * v + 3] = a.w;
                ee[4 * v] = b.x; ee[4 * v + 1] = b.y; ee[4 * v + 2] = b.z; ee[4 * v + 3] = b.w;
            }
            const int k0 = kk[0];
            int kmin = 0x7fffffff, kmax = -1, efirst = -1;
            bool run = k0 >= 0, uniform = true;
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const int k = kk[j];
                run = run && k == k0 + j;
                if (k < 0) continue;
                kmin = min(kmin, k);
                kmax = max(kmax, k);
                const int eb = ee[j];
                if (efirst < 0) efirst = eb;
                else uniform = uniform && eb == efirst;  // one level for all real columns
            }
            int4 ud;
            ud.x = kmax < 0 ? -1 : kmin;
            ud.y = kmax;
            ud.z = (run ? 1 : 0) | (uniform ? 2 : 0) | 4;
            ud.w = (max(efirst, 0) & 0xFF) | ((e & 0xFF) << 16);
            cols.unitB[u] = ud;
        }
        __syncthreads();
    }
    // The workgroup that finishes last describes the units of the A store: every part has added its
    // weights by then.
    __shared__ int s_last;
    __threadfence();
    __syncthreads();
    if (threadIdx.x == 0) s_last = atomicAdd(&hdr->cols_done, 1u) == (unsigned)(nparts - 1);
    __syncthreads();
    if (!s_last) return;
    __threadfence();  // what the other workgroups wrote before their increment is visible past this fence
    for (int u = threadIdx.x; u < KA / 16; u += kPlanThreads) {
        const int qq = 16 * u;
        int kmin = 0x7fffffff, kmax = -1, efirst = -1, kfirst = -1, jfirst = 0;
        unsigned long long wfirst = 0;
        bool run = true, uniform = true, onew = true;
        int kk[16], ee[16];  // all sixteen columns' words at once (the fence above has dropped stale cached lines)
        unsigned long long ww[16];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int4 a = reinterpret_cast<const int4 *>(cols.colA_k + qq)[v], b = reinterpret_cast<const int4 *>(cols.colA_e + qq)[v];
            kk[4 * v] = a.x; kk[4 * v + 1] = a.y; kk[4 * v + 2] = a.z; kk[4 * v + 3] = a.w;
            ee[4 * v] = b.x; ee[4 * v + 1] = b.y; ee[4 * v + 2] = b.z; ee[4 * v + 3] = b.w;
        }
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            const ulonglong2 t = reinterpret_cast<const ulonglong2 *>(cols.colA_w + qq)[v];
            ww[2 * v] = t.x;
            ww[2 * v + 1] = t.y;
        }
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int k = kk[j];
            if (k < 0) {
                run = false;
                continue;
            }
            const int ea = ee[j];
            const unsigned long long w = ww[j];
            if (efirst < 0) { efirst = ea; kfirst = k; jfirst = j; wfirst = w; }
            run = run && k == kfirst + (j - jfirst) && jfirst == 0;
            uniform = uniform && ea == efirst;
            onew = onew && w == wfirst;
            kmin = min(kmin, k);
            kmax = max(kmax, k);
        }
        int4 ud;
        ud.x = kmax < 0 ? -1 : kmin;
        ud.y = kmax;
        ud.z = (run && kmax >= 0 ? 1 : 0) | (uniform ? 2 : 0) | (onew ? 4 : 0);
        ud.w = max(efirst, 0) & 0xFF;
        cols.unitA[u] = ud;
        cols.unitA_w[u] = wfirst < (1ull << 44) ? wfirst : (1ull << 44);
    }
}

// A place in the list of `block` for every lane that gets here together: one atomic per list named, all of them in flight together (the
// entries of a block of rows sit side by side in the OB list; an atomic to each lane: 36 us for 37 000 entries).
__device__ __forceinline__ int list_place(int32_t *cnt, int block) {
    const int lane = threadIdx.x & 63;
    unsigned long long pending = __ballot(1);
    int lead = lane, before = 0, count = 0;
    while (pending) {
        const int first = __builtin_ctzll(pending);
        const unsigned long long same = __ballot(block == __builtin_amdgcn_readlane(block, first));
        if ((same >> lane) & 1) {
            lead = first;
            before = __popcll(same & ((1ull << lane) - 1ull));
            count = __popcll(same);
        }
        pending &= ~same;
    }
    int base = 0;
    if (lane == lead) base = atomicAdd(&cnt[block], count);
    return __shfl(base, lead, 64) + before;
}

// A completed header to the host: its words, then the sequence number that the host waits for.
__device__ __forceinline__ void publish_header(const PlanHeader *hdr, PlanHeader *host, int32_t seq) {
    constexpr int kWords = (int)(offsetof(PlanHeader, seq) / sizeof(int32_t));
    const int32_t *src = reinterpret_cast<const int32_t *>(hdr);
    int32_t *dst = reinterpret_cast<int32_t *>(host);
    for (int i = threadIdx.x; i < kWords; i += blockDim.x)
        __hip_atomic_store(dst + i, load_agent(src + i), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    stores_done();
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store(&host->seq, seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The digits of the columns that the fused GEMM takes from lists, into the lists: level by level like the fix-up behind the scatter, which
// writes the same digits to B_eu.  The digits of a list stand in no particular order; one that is too short is reported.  Then the header to
// the host (a launch of its own: 3 us more, which plans without lists would pay too).  Bound by the latency of an entry's dependent
// reads: 45 000 entries of 11008 x 4096 weights 9.9 us.  (Places counted row by row ahead of them, in the
// layouts' launch, and the lists filled by the fix-up: layouts 41 us instead of 27, fix-up 15 instead of 12.)
struct ListsArgs {
    const int32_t *ob;       // [3][ob_cap] the OB entries of B, kept by the plan
    int ob_cap, sh;
    SlotSet rows, cols;      // of the second unpacking
    const int32_t *row_phys, *col_phys;
    const int32_t *skip;     // keep-weights mode: set if they stand as they are
    PlanHeader *hdr;
    SparseLists lists;
    PlanHeader *host;
    int32_t seq;
};
__global__ __launch_bounds__(256) void lists_kernel(ListsArgs f) {
    PlanHeader *hdr = f.hdr;
    if (hdr->nsparse == 0 || hdr->overflow || hdr->err || (f.skip && *f.skip)) {
        if (blockIdx.x == 0) publish_header(hdr, f.host, f.seq);
        return;
    }
    const int n = min(hdr->nobB, f.ob_cap), list_col = hdr->list_kt0 * kKPad;
    for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < n; t += gridDim.x * blockDim.x) {
        const int v = f.ob[2 * (size_t)f.ob_cap + t];
        const unsigned av = v < 0 ? 0u - (unsigned)v : (unsigned)v;
        // (the copies of a column that A's unpacking repeats belong to higher levels along A, which are not listed)
        digits_above(f.rows, f.cols, f.ob[t], f.ob[f.ob_cap + t], av, f.sh, [&](int R, int C, int m) {
            const int k = f.col_phys[C] - list_col;
            if (k < 0) return;
            const int p = f.row_phys[R], block = p / kSparseRows, pos = list_place(f.lists.cnt, block);
            // (through to where every XCD reads it: once the host has the header, a stream that does not wait for this launch may)
            if (pos < f.lists.cap)
                __hip_atomic_store(&f.lists.ent[(size_t)block * f.lists.cap + pos],
                                   (uint32_t)(p % kSparseRows) | (uint32_t)k << 7 | (uint32_t)(uint8_t)(int8_t)(v < 0 ? -m : m) << 24, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            else
                atomicMax(&hdr->sparse_room, pos + 1);
        });
    }
    __shared__ unsigned s_before;
    stores_done();
    __syncthreads();
    if (threadIdx.x == 0) s_before = atomicAdd(&hdr->lists_done, 1u);
    __syncthreads();
    if (s_before == gridDim.x - 1) publish_header(hdr, f.host, f.seq);
}

__host__ __device__ inline int row_slices(int rows) {
    const int w = (rows + kRowSlice - 1) / kRowSlice;
    return w < 1 ? 1 : w > 4 ? 4 : w;
}

__global__ __launch_bounds__(256) void publish_kernel(const PlanHeader *hdr, PlanHeader *host, int32_t seq) {
    publish_header(hdr + blockIdx.y, host + blockIdx.y, seq);
}

// One to four workgroups for the rows of A, as many for the rows of B, kColBlocks for the columns (those idle that have nothing to write;
// one for each item of a batch).
// LISTS: columns of B may be taken from lists (see SparseArgs).  A variant of its own (20 -> 36 us for a product without lists in one kernel with
// them), without the general layout of the columns, which left it no registers (plans 7 to 13 us longer): the host launches the other one if it is needed.
template <bool LISTS>
__global__ __launch_bounds__(kPlanThreads) void layouts_kernel(
    SlotSet rowA, int n, RowLayout layA, int cap_physA, int32_t *tmpPA, SlotSet rowB, int h, RowLayout layB,
    int cap_physB, int32_t *tmpPB, SlotSet c1, SlotSet c2, ColLayout cols, int d, int cap_physC, int s, int sh,
    int32_t *tmpE, int32_t *tmpK, int32_t *tmpR, int32_t *tmpOff, PlanHeader *hdr, int fast_lds, const int32_t *skipB,
    int64_t stride, int chunkB, int dyn_words, SparseArgs sparse) {
    __shared__ int lds[40];
    __shared__ ColTables tables;
    extern __shared__ __attribute__((aligned(16))) int32_t fast_rows[];  // what rows_layout asks for if fast_lds; dyn_words in all
    hdr += blockIdx.y;
    {
        const int64_t off = blockIdx.y * stride;
        move_to_item(rowA, off);
        move_to_item(layA, off);
        move_to_item(rowB, off);
        move_to_item(layB, off);
        move_to_item(c1, off);
        move_to_item(c2, off);
        move_to_item(cols, off);
        tmpPA = item_at(tmpPA, off);
        tmpPB = item_at(tmpPB, off);
        tmpE = item_at(tmpE, off);
        tmpK = item_at(tmpK, off);
        tmpR = item_at(tmpR, off);
        tmpOff = item_at(tmpOff, off);
    }
    // (asked once for all waves: another workgroup of this launch may be reporting an overflow of its own just now)
    if (__syncthreads_or(load_agent(&hdr->overflow))) return;
    const int slA = fast_lds ? row_slices(n) : 1, slB = fast_lds ? row_slices(h) : 1;
    const int bx = (int)blockIdx.x;
    if (bx >= slA && skipB && *skipB) return;  // keep-weights mode: these layouts stand as they are
    // rows of A: the GEMM epilogue folds them chunk by chunk; rows of B (columns of C): tile by tile, or chunk by chunk
    // where the small-tile GEMM may be the one to run
    if (bx < slA)
        rows_layout(rowA, n, &hdr->n_u, layA, cap_physA, cap_physA / kTile + 2, tmpPA, hdr, 0, kChunk, lds, fast_lds ? fast_rows : nullptr, bx, slA);
    else if (bx < slA + slB) {
        // (chunk by chunk a few more rows of B are padding, which may cost a round of the large tiles: 2000 x 2000 x 2000 with
        // entries of three digits, un-fused: 272 tiles instead of 256, 944 us, 682 so.  Only the unpacked sizes tell: rows and k-tiles
        // without their padding, and a margin for it.  Half tiles are not counted: what they take goes by the
        // levels, and for b <= 4 the digits may still be asked for in six bits, which have none.  Counted as for products without levels they
        // brought nothing (1576 x 1537 by 6144 26.4 and 26.4 us, 2640 x 1031 by 1554 26.3 and 26.3) and took the small tiles from others: 954 x 64
        // by 2405 14 -> 32 us, 148 x 76 by 7676 14 -> 30, six-bit digits in a new plan 22 -> 40 and 19 -> 37.)
        if (chunkB == kChunk && gridDim.y == 1) {
            auto up = [](int x, int by) { return (int64_t)((x + by - 1) / by); };
            const int nu = hdr->n_u, hu = hdr->h_u;
            if (!small_tiles_win(up(nu, kTile) * up(hu, kTile), up(nu, kChunk) * up(hu, kChunk), up(hdr->d_u, kKPad), true, 25)) chunkB = kTile;
        }
        rows_layout(rowB, h, &hdr->h_u, layB, cap_physB, cap_physB / kTile + 2, tmpPB, hdr, 1, chunkB, lds, fast_lds ? fast_rows : nullptr, bx - slA, slB);
        if (LISTS && bx == slA)
            for (int x = threadIdx.x; x < cap_physB / kSparseRows; x += kPlanThreads) sparse.cnt[x] = 0;
    } else {
        const int part = bx - slA - slB, parts = (int)gridDim.x - slA - slB;
        if (!cols_layout_lds<kColSlotsLds, LISTS>(c1, c2, cols, d, cap_physC, s, sh, hdr, tables, fast_rows, dyn_words, part, parts, sparse)) {
            if (LISTS) {
                if (part == 0 && threadIdx.x == 0) hdr->cols_left = 1;
            } else {
                __syncthreads();
                cols_layout(c1, c2, cols, d, cap_physC, s, sh, tmpE, tmpK, tmpR, tmpOff, hdr, lds, part, parts, tables);
            }
        }
        if (part == 0 && threadIdx.x == 0) hdr->bound[0] = hdr->bound[1] = 0;
    }
}

// ---------------------------------------------------------------------------------------------
// strategy pricing (Sec. 4.2)
// ---------------------------------------------------------------------------------------------
// out[0] = sum_i L(rowmaxA_i), out[1] = sum_j L(rowmaxB_j), out[2] = sum_k L(colmaxA_k),
// out[3] = sum_k L(colmaxB_k), out[4] = sum_k L(colmaxA_k) * L(colmaxB_k); L = number of base-s digits.
__global__ __launch_bounds__(256) void price_kernel(const int32_t *rowmaxA, int64_t n, const int32_t *rowmaxB,
                                                    int64_t h, const int32_t *colmaxA, const int32_t *colmaxB,
                                                    int64_t d, int sh, unsigned long long *out) {
    unsigned long long acc[5] = {0, 0, 0, 0, 0};
    const int64_t stride = (int64_t)gridDim.x * blockDim.x, t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int64_t i = t0; i < n; i += stride) acc[0] += digit_levels(rowmaxA[i], sh);
    for (int64_t j = t0; j < h; j += stride) acc[1] += digit_levels(rowmaxB[j], sh);
    for (int64_t k = t0; k < d; k += stride) {
        const int la = digit_levels(colmaxA[k], sh), lb = digit_levels(colmaxB[k], sh);
        acc[2] += la;
        acc[3] += lb;
        acc[4] += (unsigned long long)la * lb;
    }
#pragma unroll
    for (int q = 0; q < 5; ++q) {
        unsigned long long v = acc[q];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
        if ((threadIdx.x & 63) == 0 && v) atomicAdd(&out[q], v);
    }
}

__global__ void clear_sums_kernel(unsigned long long *p, int count) {
    if ((int)threadIdx.x < count) p[threadIdx.x] = 0;
}

// ---------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------
int scan_i32(const int32_t *Q, int64_t rows, int64_t cols, int64_t ldq, int b, const imunpack_stats_t *st, int nitems,
             int64_t q_stride, int64_t out_stride, hipStream_t stream);

struct Carver {
    char *base;
    size_t off;
    template <typename T>
    T *take(size_t count) {
        off = (off + 255) & ~(size_t)255;
        T *p = base ? reinterpret_cast<T *>(base + off) : nullptr;
        off += count * sizeof(T);
        return p;
    }
};

static void carve_slots(Carver &cv, SlotSet &s, int cap) {
    s.root = cv.take<int32_t>(cap);
    s.exp = cv.take<int32_t>(cap);
    s.time = cv.take<uint32_t>(cap);
    s.child = cv.take<int32_t>(cap);
    s.key = cv.take<unsigned long long>(cap);
    s.cap = cap;
}

static inline int phys_cap_rows(int cap) { return (int)((int64_t)cap * kChunk / (kChunk - 8) + 2 * kTile); }
static inline int phys_cap_cols(int cap) { return cap + kMaxGroups * kKPad; }

static constexpr int kLayoutLdsMax = 140 * 1024;  // dynamic LDS the layouts kernel may use (its static tables take about 11 KiB)

static inline int list_count(const Plan *p) { return phys_cap_rows(p->cap[CAP_ROWB]) / kSparseRows; }
// Whether appended columns of B may be taken from lists: those of UnpackBoth, whose heavy hitters the plan holds one by one; a product of
// its own; digits that stay int8 (the six-bit format may be asked for once the plan is made); a product that is worth the planner's
// share (see kSparseWork), and lists that stay within 256 MiB.
static inline bool sparse_possible(const Plan *p) {
    return p->sB == IMUNPACK_BOTH && p->nitems == 1 && p->b > 4 && p->d >= kSparseLeast && 2 * p->d + 512 <= kColSlotsLds * kPlanThreads &&
           (p->keep_B || (double)p->n * (double)p->d * (double)p->h >= (double)kSparseWork) && (int64_t)list_count(p) * p->cap[CAP_SPARSE] <= kSparsePlaces;
}

// Lays every device array out in the arena for the current capacities: the headers of all items, then the
// arrays of item 0, those of item 1 (p->item_bytes further), and so on.  Returns the bytes needed.
static size_t carve(Plan *p, char *base, bool own_statsA, bool own_statsB) {
    Carver cv{base, 0};
    const int n = (int)p->n, d = (int)p->d, h = (int)p->h;
    p->d_hdr = cv.take<PlanHeader>(p->nitems);
    cv.off = (cv.off + 255) & ~(size_t)255;
    const size_t item0 = cv.off;
    carve_slots(cv, p->rowA, p->cap[CAP_ROWA]);
    carve_slots(cv, p->rowB, p->cap[CAP_ROWB]);
    carve_slots(cv, p->c1, p->cap[CAP_C1]);
    carve_slots(cv, p->c2, p->cap[CAP_C2]);
    for (int op = 0; op < 2; ++op) {
        RowLayout &l = op ? p->layB : p->layA;
        const int cap = p->cap[op ? CAP_ROWB : CAP_ROWA], nb = op ? h : n;
        const int pc = phys_cap_rows(cap);
        l.prow = cv.take<int32_t>(pc);
        l.row_phys = cv.take<int32_t>(cap);
        l.src_pstart = cv.take<int32_t>(nb + 1);
        l.src_nlev = cv.take<int32_t>(nb + 1);
        l.tile_src0 = cv.take<int32_t>(pc / kTile + 2);
        l.chunk_src0 = cv.take<int32_t>(pc / kChunk + 8);
        l.tile_flat = cv.take<int32_t>(pc / kTile + 2);
        l.chunk_lev = cv.take<int32_t>(pc / kChunk + 8);
        l.rowsum = cv.take<unsigned long long>(pc);
        l.wavesum = cv.take<unsigned long long>((size_t)pc * ((phys_cap_cols(p->cap[CAP_C2]) + 1023) / 1024));
    }
    {
        const int kc = phys_cap_cols(p->cap[CAP_C2]);
        p->cols.pcol_slot = cv.take<int32_t>(kc);
        p->cols.col_phys = cv.take<int32_t>(p->cap[CAP_C2]);
        p->cols.colB_k = cv.take<int32_t>(kc);
        p->cols.colB_e = cv.take<int32_t>(kc);
        p->cols.col_sexp = cv.take<int32_t>(kc);
        p->cols.unitB = cv.take<int4>(kc / 16 + 1);
        p->cols.acol_phys = cv.take<int32_t>(p->cap[CAP_C2]);
        p->cols.apos = cv.take<int32_t>(p->cap[CAP_C1]);
        p->cols.colA_k = cv.take<int32_t>(kc);
        p->cols.colA_e = cv.take<int32_t>(kc);
        p->cols.colA_w = cv.take<unsigned long long>(kc);
        p->cols.unitA = cv.take<int4>(kc / 16 + 1);
        p->cols.unitA_w = cv.take<unsigned long long>(kc / 16 + 1);
        p->tmpE = cv.take<int32_t>(p->cap[CAP_C2]);
        p->tmpK = cv.take<int32_t>(p->cap[CAP_C2]);
        p->tmpR = cv.take<int32_t>(p->cap[CAP_C2]);
        p->tmpOff = cv.take<int32_t>((size_t)kColBlocks * (d + 1));
    }
    p->canon_rowphysA = cv.take<int32_t>(p->cap[CAP_ROWA]);
    p->canon_rowphysB = cv.take<int32_t>(p->cap[CAP_ROWB]);
    p->canon_colphys = cv.take<int32_t>(p->cap[CAP_C2]);
    p->canon_acolphys = cv.take<int32_t>(p->cap[CAP_C2]);
    if (own_statsA) {
        p->statsA[0] = cv.take<int32_t>(n); p->statsA[1] = cv.take<int32_t>(d);
        p->statsA[2] = cv.take<int32_t>(n); p->statsA[3] = cv.take<int32_t>(d);
    }
    if (own_statsB) {
        p->statsB[0] = cv.take<int32_t>(h); p->statsB[1] = cv.take<int32_t>(d);
        p->statsB[2] = cv.take<int32_t>(h); p->statsB[3] = cv.take<int32_t>(d);
    }
    const int maxslots = std::max(std::max(p->cap[CAP_ROWA], p->cap[CAP_ROWB]), std::max(p->cap[CAP_C1], p->cap[CAP_C2]));
    p->tmpL = cv.take<int32_t>(maxslots);
    p->tmpCur = cv.take<int32_t>(maxslots);
    p->tmpPA = cv.take<int32_t>(n + 1);
    p->tmpPB = cv.take<int32_t>(h + 1);
    if (p->sA == IMUNPACK_BOTH || p->sB == IMUNPACK_BOTH) {
        const int ecap = std::max(p->sA == IMUNPACK_BOTH ? p->cap[CAP_EDGEA] : 0,
                                  p->sB == IMUNPACK_BOTH ? p->cap[CAP_EDGEB] : 0);
        p->edges = cv.take<unsigned long long>((size_t)2 * ecap + 2);
        p->obcopyA = cv.take<int32_t>(p->sA == IMUNPACK_BOTH ? (size_t)3 * p->cap[CAP_EDGEA] : 0);
        p->obcopyB = cv.take<int32_t>(p->sB == IMUNPACK_BOTH ? (size_t)3 * p->cap[CAP_EDGEB] : 0);
        p->edge_cap = ecap;
        const int rcap = std::max(p->cap[CAP_ROWA], p->cap[CAP_ROWB]), ccap = std::max(p->cap[CAP_C1], p->cap[CAP_C2]);
        p->rcnt = cv.take<int32_t>(rcap + 8);
        p->extraRows = cv.take<int32_t>(p->sB == IMUNPACK_BOTH ? (size_t)h + 1 : 0);
        p->ccnt = cv.take<int32_t>(ccap + 8);
        p->ob = cv.take<int32_t>((size_t)3 * p->cap[CAP_OB]);
        p->obcnt = cv.take<int32_t>(1);
    }
    p->sparse = SparseLists{};
    p->at = nullptr;
    if (sparse_possible(p)) {
        p->sparse.cnt = cv.take<int32_t>(list_count(p));
        p->sparse.ent = cv.take<uint32_t>((size_t)list_count(p) * p->cap[CAP_SPARSE] + 256);  // (the GEMM asks for 128 at a time, and once more behind a list)
        p->sparse.cap = p->cap[CAP_SPARSE];
        // (as many rows as the layout may have: how many it has is known only once the plan is made.  Allocated then, outside the arena, it
        // cost a new plan object of 4096 x 4096 by 11008 some 40 us)
        p->at = cv.take<int8_t>((size_t)phys_cap_rows(p->cap[CAP_ROWA]) * (size_t)d);
    }
    p->snapRoot = cv.take<int32_t>(p->cap[CAP_C1]);
    p->snapExp = cv.take<int32_t>(p->cap[CAP_C1]);
    p->snapChild = cv.take<int32_t>(p->cap[CAP_C1]);
    p->d_keep = cv.take<KeepState>(1);
    p->item_bytes = (int64_t)((cv.off - item0 + 255) & ~(size_t)255);
    return item0 + (size_t)p->nitems * (size_t)p->item_bytes + 256;
}

static inline int grid_for(int64_t items, int threads, int maxblocks = 2048) {
    int64_t b = (items + threads - 1) / threads;
    if (b < 1) b = 1;
    if (b > maxblocks) b = maxblocks;
    return (int)b;
}

// The OB entries of an UnpackBoth operand, kept for the scatter's fix-up pass: the caller's list need
// not outlive the call.  Many workgroups, ahead of the (single-workgroup) greedy.  For the second
// operand the same pass finds the edges that the repeated columns add: B_e holds a copy of column k
// of B in every column slot of A's unpacking that descends from k, so an OB entry (j, k) of B is
// also an OB entry (j, c) for every such slot c.  The pass also writes the greedy's first edge list:
// entry t of the OB list packed at position t, the edges of repeated columns behind the last entry.
__device__ __forceinline__ void ob_copy(const int32_t *ob, int ob_cap, int n, int32_t *keep, int keep_cap, const int32_t *chain_child,
                                        unsigned long long *edges, int ecap, int32_t *extras, int32_t *extra_rows, int sh, int t0,
                                        int step) {
    for (int t = t0; t < n; t += step) {
        const int j = ob[t], k = ob[ob_cap + t], v = ob[2 * (size_t)ob_cap + t];
        if (t < keep_cap) {
            keep[t] = j;
            keep[keep_cap + t] = k;
            keep[2 * (size_t)keep_cap + t] = v;
        }
        const unsigned av = v < 0 ? 0u - (unsigned)v : (unsigned)v;
        const int L = digit_levels((int)av, sh);
        if (t < ecap) edges[t] = L >= 2 ? pack_edge(j, k, L) : 0ull;  // 0: no edge
        if (!chain_child) continue;
        int c = chain_child[k];
        for (int hop = 0; c >= 0 && hop < 64; c = chain_child[c], ++hop) {
            const int pos = n + atomicAdd(extras, 1);
            if (pos < ecap) edges[pos] = pack_edge(j, c, L);
            atomicAdd(&extra_rows[j], 1);
        }
    }
}

__global__ __launch_bounds__(256) void ob_copy_kernel(const int32_t *__restrict__ ob, int ob_cap,
                                                      const int32_t *ob_count, int32_t *__restrict__ keep, int keep_cap,
                                                      const int32_t *chain_child, unsigned long long *edges, int ecap,
                                                      PlanHeader *hdr, int32_t *extra_rows, int sh, const int32_t *skip,
                                                      int64_t stride, int64_t list_stride) {
    if (skip && *skip) return;  // keep-weights mode: this operand's unpacking is taken over as it stands
    {
        const int64_t off = blockIdx.y * stride, loff = blockIdx.y * list_stride;
        ob = item_at(ob, loff);
        ob_count = item_at(ob_count, loff);
        keep = item_at(keep, off);
        chain_child = item_at(chain_child, off);
        edges = item_at(edges, off);
        extra_rows = item_at(extra_rows, off);
    }
    ob_copy(ob, ob_cap, min(*ob_count, ob_cap), keep, keep_cap, chain_child, edges, ecap, &hdr[blockIdx.y].extras, extra_rows, sh,
            blockIdx.x * blockDim.x + threadIdx.x, gridDim.x * blockDim.x);
}

// UnpackBoth on both operands of a small product: copies of the lists and greedies, one after the other, by one workgroup.  (Four
// launches otherwise, each of which waits for the one before, finds its arguments and fetches its instructions again: 256 x 256
// by 256: 31 us and four launches, 26 and one.)
constexpr int kGreedyPairSlots = 256;
constexpr int64_t kGreedyPairList = 1 << 16;  // places in either list: several workgroups copy longer ones
struct GreedyPair {
    GreedyArgs g[2];
    const int32_t *ob[2];
    int32_t *keep[2];
    int keep_cap[2];
};
__global__ __launch_bounds__(kPlanThreads) void greedy_pair_kernel(GreedyPair f) {
    extern __shared__ __attribute__((aligned(16))) int32_t lds_counts[];
    PlanHeader *hdr = f.g[0].hdr + blockIdx.y;
    for (int op = 0; op < 2; ++op) {
        if (__syncthreads_or(load_agent(&hdr->overflow))) return;
        GreedyArgs g = f.g[op];
        move_to_item(g);
        ob_copy(item_at(f.ob[op], blockIdx.y * g.list_stride), g.ob_cap, min(*g.ob_count, g.ob_cap), item_at(f.keep[op], blockIdx.y * g.stride), f.keep_cap[op],
                g.chain_child, g.edges, g.ecap, &hdr->extras, const_cast<int32_t *>(g.extra_rows), g.sh, threadIdx.x, kPlanThreads);
        __syncthreads();
        // What is not for bits of 256 slots, entries of four digits or more above all, has its edges in LDS (256 x 256 by 256, b = 5, four
        // digits, 1 % of heavy hitters: planned in 300 us with the edges in memory, in 236 so; with 5 % at b = 4 451 and 360, where two
        // launches of greedy_both_kernel and two copies by many workgroups took 336).  Three digits in a B_e of 257 to 512 columns go that way
        // too (184 and 156 us): with bits for them as well the kernel spills.
        greedy_both<true, true, true, false>(g, hdr, lds_counts);
    }
}

// ---- keep-weights mode (Sec. 4.2: weights are unpacked once, when they are loaded).  The unpacking of the
// second operand depends on the first only through the column slots of the first operand's unpacking
// (which columns of B_e are repeats, and their exponents).  If those are what they were for the plan
// before, the second operand's slots, its kept OB entries and its header fields are taken over.
// One workgroup: compares the column slots with the remembered ones and acts on the verdict.  Same slots: the
// header fields that the second operand's unpacking and the layouts of its rows and of the columns left are
// put back.  Different: its rows start afresh and the column weights are cleared for the column layout to come.
struct KeepArgs {
    const int32_t *sroot, *sexp, *schild;
    KeepState *ks;               // nullptr: not in this mode
    int host_valid;
    int h;                       // rows of B that start as unsplit originals
    int32_t *extra_rows;
    int nextra;
    int32_t *col_weights;
    int nweights;
};
__device__ bool keep_decide(const KeepArgs &k, const SlotSet &c1, PlanHeader *hdr, const SlotSet &rowB) {
    KeepState *ks = k.ks;
    const int32_t *sroot = k.sroot, *sexp = k.sexp, *schild = k.schild;
    const int h = k.h, d1 = hdr->d1;
    bool differs = !k.host_valid || !ks->valid || d1 != ks->d1 || d1 > c1.cap || load_agent(&hdr->overflow) != 0;
    if (!differs)
        for (int x = threadIdx.x; x < d1; x += kPlanThreads)
            differs = differs || c1.root[x] != sroot[x] || c1.exp[x] != sexp[x] || c1.child[x] != schild[x];
    const bool same = !__syncthreads_or(differs);
    if (threadIdx.x == 0) {
        ks->same = same;
        hdr->reusedB = same;
        if (same) {
            const PlanHeader &o = ks->saved;
            hdr->h_u = o.h_u; hdr->d_u = o.d_u; hdr->nobB = o.nobB; hdr->edgesB = o.edgesB; hdr->extras = o.extras;
            hdr->Np = o.Np; hdr->Kp = o.Kp; hdr->KA = o.KA; hdr->ldA = o.ldA; hdr->ldB = o.ldB;
            hdr->ntiles = o.ntiles; hdr->lmaxB = o.lmaxB; hdr->chunkB = o.chunkB; hdr->evenB = o.evenB; hdr->ngroups = o.ngroups; hdr->nruns = o.nruns;
            hdr->nsparse = o.nsparse; hdr->list_kt0 = o.list_kt0;
        } else if (h) {
            hdr->h_u = h;
        }
    }
    if (same) {  // the group and run tables
        constexpr size_t g0 = offsetof(PlanHeader, grp_exp) / sizeof(int32_t), g1 = offsetof(PlanHeader, nruns) / sizeof(int32_t);
        constexpr size_t r0 = offsetof(PlanHeader, run_kt0) / sizeof(int32_t), r1 = offsetof(PlanHeader, edgesA) / sizeof(int32_t);
        const int32_t *src = reinterpret_cast<const int32_t *>(&ks->saved);
        int32_t *dst = reinterpret_cast<int32_t *>(hdr);
        for (size_t i = g0 + threadIdx.x; i < g1; i += kPlanThreads) dst[i] = src[i];
        for (size_t i = r0 + threadIdx.x; i < r1; i += kPlanThreads) dst[i] = src[i];
        return true;
    }
    for (int x = threadIdx.x; x < h; x += kPlanThreads) identity_slot(rowB, x);
    for (int x = threadIdx.x; x < k.nextra; x += kPlanThreads) k.extra_rows[x] = 0;
    for (int x = threadIdx.x; x < k.nweights; x += kPlanThreads) k.col_weights[x] = 0;
    return false;
}

__global__ __launch_bounds__(kPlanThreads) void keep_decide_kernel(KeepArgs k, SlotSet c1, PlanHeader *hdr, SlotSet rowB) {
    keep_decide(k, c1, hdr, rowB);
}

// After a plan that unpacked the second operand anew: remember the column slots it was unpacked for and the
// header the plan completed.
__global__ void keep_remember_kernel(SlotSet c1, const PlanHeader *hdr, int32_t *sroot, int32_t *sexp, int32_t *schild,
                                     KeepState *ks) {
    if (ks->same) return;
    if (hdr->overflow || hdr->err || hdr->d1 > c1.cap) {
        if (blockIdx.x == 0 && threadIdx.x == 0) ks->valid = 0;
        return;
    }
    const int d1 = hdr->d1;
    for (int x = blockIdx.x * blockDim.x + threadIdx.x; x < d1; x += gridDim.x * blockDim.x) {
        sroot[x] = c1.root[x];
        sexp[x] = c1.exp[x];
        schild[x] = c1.child[x];
    }
    if (blockIdx.x == 0) {
        const int32_t *src = reinterpret_cast<const int32_t *>(hdr);
        int32_t *dst = reinterpret_cast<int32_t *>(&ks->saved);
        for (size_t i = threadIdx.x; i < sizeof(PlanHeader) / sizeof(int32_t); i += blockDim.x) dst[i] = src[i];
        if (threadIdx.x == 0) {
            ks->d1 = d1;
            ks->valid = 1;
        }
    }
}

// ---- keep-weights mode in one launch: what runs on every plan in this mode -- the first operand is unpacked, the verdict taken
// and, if the second operand's unpacking is taken over, the first operand's rows laid out.  One by one these were seven
// launches that mostly found nothing to do (16 rows against resident 11008 x 4096 weights: 42 us; 21 in one).  If the
// unpacking is not taken over, the host, which reads the verdict in the header, launches the rest.
// (The whole plan of a small product in one workgroup and launch took longer than its kernels one by one, 107 against 95 us
// at 256 x 256 x 256 and 54 against 32 at 1000 x 1031 x 777: code that runs once is bound by its instruction fetch.)
struct KeepPlan {
    PlanHeader *hdr;
    SlotSet rows, cols, rowsB;        // slots of the first operand's unpacking; row slots of the second
    RowLayout lay;
    const int32_t *rowmax, *colmax;
    GreedyArgs greedy;                // UnpackBoth
    int32_t *tmpL, *tmpCur, *tmpP;
    int n, d, h, sh, strategy, strategyB, cap_phys;
    KeepArgs keep;
    PlanHeader *host;
    int32_t seq;
};

__global__ __launch_bounds__(kPlanThreads) void keep_plan_kernel(KeepPlan f) {
    __shared__ int lds[40];
    extern __shared__ __attribute__((aligned(16))) int32_t dyn[];
    PlanHeader *hdr = f.hdr;
    for (size_t i = threadIdx.x; i < sizeof(PlanHeader) / sizeof(int32_t); i += kPlanThreads) reinterpret_cast<int32_t *>(hdr)[i] = 0;
    if (f.strategy != IMUNPACK_COL)
        for (int x = threadIdx.x; x < f.d; x += kPlanThreads) identity_slot(f.cols, x);
    if (f.strategy != IMUNPACK_ROW)
        for (int x = threadIdx.x; x < f.n; x += kPlanThreads) identity_slot(f.rows, x);
    __syncthreads();
    if (threadIdx.x == 0) {
        f.keep.ks->same = 0;
        if (f.strategy != IMUNPACK_ROW) hdr->n_u = f.n;
        if (f.strategy != IMUNPACK_COL) hdr->d1 = f.d;
        if (f.strategyB != IMUNPACK_ROW) hdr->h_u = f.h;
    }
    __syncthreads();
    if (f.strategy == IMUNPACK_BOTH) {
        greedy_both<true, false>(f.greedy, hdr, dyn);  // (the edges stay in memory: this kernel has no registers to spare)
    } else {
        const bool by_row = f.strategy == IMUNPACK_ROW;
        level_major<4>(by_row ? f.rows : f.cols, by_row ? f.rowmax : f.colmax, nullptr, by_row ? f.n : f.d, f.sh, f.tmpL, f.tmpCur, hdr,
                       by_row ? CAP_ROWA : CAP_C1, lds);
    }
    __syncthreads();
    if (keep_decide(f.keep, f.cols, hdr, f.rowsB)) {
        __syncthreads();
        rows_layout(f.rows, f.n, &hdr->n_u, f.lay, f.cap_phys, f.cap_phys / kTile + 2, f.tmpP, hdr, 0, kChunk, lds, dyn, 0, 1);
    }
    __syncthreads();
    publish_header(hdr, f.host, f.seq);
}

static constexpr int kGreedyLdsMax = 136 * 1024;  // dynamic LDS the greedy may use for the two count vectors
static constexpr int kKeepPlanCols = 16384;       // columns that keep_plan_kernel sets up and compares in one workgroup
// The larger side of an operand.
static int greedy_slots(const Plan *p, int phase) { return (int)std::max(phase == 1 ? p->n : p->h, p->d); }

// dynamic LDS of the greedy's two count vectors
static size_t greedy_lds(const Plan *p, int phase) {
    const SlotSet &rows = phase == 1 ? p->rowA : p->rowB, &cols = phase == 1 ? p->c1 : p->c2;
    return ((size_t)((rows.cap + 7) & ~3) + (size_t)((cols.cap + 7) & ~3)) * sizeof(int32_t);
}

// ob: the operand's OB entry list ([3][ob_cap], count on the device)
static GreedyArgs greedy_args(const Plan *p, int phase, int ob_cap, const int32_t *ob_count, int64_t list_stride, int which_list,
                              const int32_t *skip) {
    const bool first = phase == 1;
    GreedyArgs g;
    g.rows = first ? p->rowA : p->rowB; g.cols = first ? p->c1 : p->c2;
    g.second = !first;
    g.chain_child = first ? nullptr : p->c1.child;
    g.chain_root = first ? nullptr : p->c1.root;
    int32_t *const *stats = first ? p->statsA : p->statsB;
    g.rowcnt = stats[0]; g.colcnt = stats[1]; g.rowmax = stats[2];
    g.ob_cap = ob_cap; g.ob_count = ob_count; g.which_list = which_list;
    g.stride = p->item_bytes; g.stats_stride = p->op_stride; g.list_stride = list_stride;
    g.edges = p->edges;
    g.ecap = std::min(p->cap[first ? CAP_EDGEA : CAP_EDGEB], p->edge_cap);
    g.rcnt = p->rcnt; g.ccnt = p->ccnt;
    g.extra_rows = first ? nullptr : p->extraRows;
    g.hdr = p->d_hdr;
    g.whichR = first ? CAP_ROWA : CAP_ROWB;
    g.whichC = first ? CAP_C1 : CAP_C2;
    g.whichE = first ? CAP_EDGEA : CAP_EDGEB;
    g.s = p->s; g.sh = p->sh;
    g.skip = skip;
    // the counts, and room for edges: a workgroup per CU as long as there are CUs for the items
    const size_t counts = greedy_lds(p, phase), room = p->nitems <= 256 ? 96 * 1024 : 32 * 1024;
    g.lds_words = (int)(std::min(counts + std::min(room, (size_t)g.ecap * 8), std::max(counts, (size_t)kGreedyLdsMax)) / sizeof(int32_t));
    // ... or for the bits of a small operand (B_e may have more columns than B)
    const int slots = greedy_slots(p, phase), words = bits_words(slots);
    if (words != 0) g.lds_words = std::max(g.lds_words, first || 2 * slots <= 256 || p->nitems > 256 ? words : bits_words(512));
    return g;
}

static void launch_ob_copy(const Plan *p, const GreedyArgs &g, int phase, const int32_t *ob, hipStream_t st) {
    const bool first = phase == 1;
    const int keep_cap = p->cap[first ? CAP_EDGEA : CAP_EDGEB];  // the stride the fix-up pass reads with
    hipLaunchKernelGGL(ob_copy_kernel, dim3(grid_for(g.ob_cap, 256, 128), (unsigned)p->nitems), dim3(256), 0, st, ob, g.ob_cap, g.ob_count,
                       first ? p->obcopyA : p->obcopyB, keep_cap, g.chain_child, g.edges, g.ecap,
                       p->d_hdr, p->extraRows, p->sh, g.skip, p->item_bytes, g.list_stride);
}

static int run_greedy(Plan *p, int phase, const int32_t *ob, int ob_cap, const int32_t *ob_count, int64_t list_stride,
                      int which_list, hipStream_t st, const int32_t *skip = nullptr) {
    const GreedyArgs g = greedy_args(p, phase, ob_cap, ob_count, list_stride, which_list, skip);
    const size_t lds_bytes = greedy_lds(p, phase);
    static std::atomic<int> opted_in{0};  // the attribute is idempotent: a race sets the same value twice
    if (!opted_in.load(std::memory_order_acquire)) {
        IMU_HIP(hipFuncSetAttribute((const void *)greedy_both_kernel<true, false>, hipFuncAttributeMaxDynamicSharedMemorySize, kGreedyLdsMax));
        IMU_HIP(hipFuncSetAttribute((const void *)greedy_both_kernel<true, true>, hipFuncAttributeMaxDynamicSharedMemorySize, kGreedyLdsMax));
        opted_in.store(1, std::memory_order_release);
    }
    const unsigned items = (unsigned)p->nitems;
    launch_ob_copy(p, g, phase, ob, st);
    if (lds_bytes <= (size_t)kGreedyLdsMax && bits_words(greedy_slots(p, phase)) != 0)
        hipLaunchKernelGGL((greedy_both_kernel<true, true>), dim3(1, items), dim3(kPlanThreads), (size_t)g.lds_words * sizeof(int32_t), st, g);
    else if (lds_bytes <= (size_t)kGreedyLdsMax)
        hipLaunchKernelGGL((greedy_both_kernel<true, false>), dim3(1, items), dim3(kPlanThreads), (size_t)g.lds_words * sizeof(int32_t), st, g);
    else
        hipLaunchKernelGGL((greedy_both_kernel<false, false>), dim3(1, items), dim3(kPlanThreads), 0, st, g);
    return launch_status();
}

static void destroy_handles(Plan *p) {
    if (p->pin_hdr) (void)hipHostFree(p->pin_hdr);
    if (p->split_ws) {
        (void)hipFree(p->split_ws);
        (void)hipEventDestroy(p->split_done);
    }
}

template <class T>
int wait_word(const T *word, T want, hipStream_t st) {
    for (long spin = 1;; ++spin) {
        if (__atomic_load_n(word, __ATOMIC_ACQUIRE) == want) return IMUNPACK_OK;
        // Still nothing: look whether the stream has come to an end without it; a very long plan stops burning the core.  Not before half a
        // millisecond or so: a query of a busy stream puts a marker behind its work, whose signal wakes a thread of the runtime (every
        // 65536 spins, which took 26 or 52 us as the loop happened to be laid out, a call of 176 x 281 by 88 was one of 97 or of 76 us).  What
        // the query did of the runtime's bookkeeping on the side is left to a device synchronisation, if one follows the step at once: 256 x
        // 256 x 256 among others 143 -> 135 us, waited for by an event 147 -> 146, by such a synchronisation 158 -> 171.
        if (spin & 0xFFFFF) continue;
        hipError_t e = spin < (1 << 24) ? hipStreamQuery(st) : hipStreamSynchronize(st);
        if (e == hipErrorNotReady) {
            (void)hipGetLastError();
            continue;
        }
        if (e == hipSuccess && __atomic_load_n(word, __ATOMIC_ACQUIRE) == want) return IMUNPACK_OK;
        g_last_hip_error = (int)e;
        (void)hipGetLastError();
        return IMUNPACK_EHIP;
    }
}

template int wait_word<int32_t>(const int32_t *, int32_t, hipStream_t);

// The headers that the last launch hands over.
static int await_headers(Plan *p, hipStream_t st) {
    IMU_TRY(launch_status());
    for (int i = 0; i < p->nitems; ++i) IMU_TRY(wait_word(&p->pin_hdr[i].seq, p->seq, st));
    p->hdr = p->pin_hdr[0];
    return IMUNPACK_OK;
}

// Plans on the device and waits for the headers.
static int run_plan(Plan *p, const int32_t *A, int64_t lda, const int32_t *B, int64_t ldb,
                        const imunpack_stats_t *stA, const imunpack_stats_t *stB, bool own_statsA,
                        bool own_statsB, hipStream_t st) {
    PlanHeader *hdr = p->d_hdr;
    const int n = (int)p->n, d = (int)p->d, h = (int)p->h;
    // header cleared; the sets that start as unsplit originals with a size the host knows
    const int idA = p->sA != IMUNPACK_ROW ? n : 0, idC1 = p->sA != IMUNPACK_COL ? d : 0,
              idB = p->sB != IMUNPACK_ROW ? h : 0;
    if (idA > p->rowA.cap || idC1 > p->c1.cap || idB > p->rowB.cap) return IMUNPACK_EINVAL;
    // also cleared: the weights of the stored columns of A (the column layout adds to them)
    const int kcA = phys_cap_cols(p->cap[CAP_C2]);
    // keep-weights mode (UnpackBoth on the second operand): its rows are set up only once it is known that its
    // unpacking has to be redone
    const bool keep = p->keep_B != 0;
    const unsigned items = (unsigned)p->nitems;
    const int64_t stride = p->item_bytes, sstride = p->op_stride;
    // the row layouts keep two ints per source row and one per chunk in LDS when that fits beside the column layout's tables
    const int most_phys = std::max(phys_cap_rows(p->cap[CAP_ROWA]), phys_cap_rows(p->cap[CAP_ROWB]));
    const size_t fast_bytes = ((size_t)2 * std::max(n, h) + most_phys / kChunk + 8) * sizeof(int32_t);
    const int fast_lds = fast_bytes <= (size_t)kLayoutLdsMax ? 1 : 0;
    // the column layout: a word per column of either store, three per 64 original columns and pair of levels (sixteen pairs)
    const size_t col_bytes = ((size_t)2 * (p->cap[CAP_C2] + 2048) + (size_t)48 * ((d + 63) / 64)) * sizeof(int32_t);
    // (a batch leaves LDS to the items beside it)
    const size_t dyn_bytes = items == 1 ? (size_t)kLayoutLdsMax : std::min((size_t)kLayoutLdsMax, std::max(fast_lds ? fast_bytes : 0, col_bytes));
    static std::atomic<int> opted_in{0};  // the attributes are idempotent: a race sets the same values twice
    if (!opted_in.load(std::memory_order_acquire)) {
        IMU_HIP(hipFuncSetAttribute((const void *)layouts_kernel<false>, hipFuncAttributeMaxDynamicSharedMemorySize, kLayoutLdsMax));
        IMU_HIP(hipFuncSetAttribute((const void *)layouts_kernel<true>, hipFuncAttributeMaxDynamicSharedMemorySize, kLayoutLdsMax));
        IMU_HIP(hipFuncSetAttribute((const void *)greedy_pair_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kGreedyLdsMax));
        IMU_HIP(hipFuncSetAttribute((const void *)keep_plan_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kGreedyLdsMax));
        opted_in.store(1, std::memory_order_release);
    }
    // OB entry lists for UnpackBoth: the caller's (from the fused quantize pass) if complete, else
    // this call's own scan produces one.  The two operands are planned one after the other, so one
    // own buffer serves both.
    const bool listA = p->sA == IMUNPACK_BOTH, listB = p->sB == IMUNPACK_BOTH;
    const bool callerA = listA && stA && stA->ob && stA->ob_count && stA->ob_cap > 0 && !p->ignore_listA;
    const bool callerB = listB && stB && stB->ob && stB->ob_count && stB->ob_cap > 0 && !p->ignore_listB;
    const bool scanA = own_statsA || (listA && !callerA), scanB = own_statsB || (listB && !callerB);
    auto scan_operand = [&](const int32_t *M, int rows, int64_t ld, int32_t **own, bool own_stats, bool list) {
        if (items > 1 && own_stats) return (int)IMUNPACK_EINVAL;  // a batch brings its statistics
        imunpack_stats_t sx;
        memset(&sx, 0, sizeof(sx));
        if (own_stats) { sx.rowcnt = own[0]; sx.colcnt = own[1]; sx.rowmax = own[2]; sx.colmax = own[3]; }
        if (list) { sx.ob = p->ob; sx.ob_cap = p->cap[CAP_OB]; sx.ob_count = p->obcnt; }
        return scan_i32(M, rows, d, ld, p->b, &sx, p->nitems, sstride, stride, st);
    };
    KeepArgs keep_args = {p->snapRoot, p->snapExp, p->snapChild, keep ? p->d_keep : nullptr, p->keep_valid, idB, p->extraRows,
                          listB ? h : 0, reinterpret_cast<int32_t *>(p->cols.colA_w), 2 * kcA};
    const int32_t *skip = nullptr;
    // keep-weights mode: up to 4096 rows, which one workgroup lays out as fast as the layout kernel would
    const size_t keep_lds = std::max(((size_t)2 * n + phys_cap_rows(p->cap[CAP_ROWA]) / kChunk + 8) * sizeof(int32_t), listA ? greedy_lds(p, 1) : 0);
    // (and only if there is something to take over: otherwise it would end in a wait for a verdict that is known)
    const bool at_once = keep && p->keep_valid && items == 1 && !scanA && n <= kRowSlice && d <= kKeepPlanCols && keep_lds <= (size_t)kGreedyLdsMax;
    if (at_once) {
        KeepPlan f;
        memset((void *)&f, 0, sizeof(f));
        f.hdr = hdr;
        f.rows = p->rowA; f.cols = p->c1; f.rowsB = p->rowB;
        f.lay = p->layA;
        f.rowmax = p->statsA[2]; f.colmax = p->statsA[3];
        if (listA) {
            f.greedy = greedy_args(p, 1, (int)stA->ob_cap, stA->ob_count, sstride, CAP_LISTA, nullptr);
            f.greedy.lds_words = (int)(keep_lds / sizeof(int32_t));
            launch_ob_copy(p, f.greedy, 1, stA->ob, st);
        }
        f.tmpL = p->tmpL; f.tmpCur = p->tmpCur; f.tmpP = p->tmpPA;
        f.n = n; f.d = d; f.h = h; f.sh = p->sh; f.strategy = p->sA; f.strategyB = p->sB;
        f.cap_phys = phys_cap_rows(p->cap[CAP_ROWA]);
        f.keep = keep_args;
        f.host = p->pin_hdr; f.seq = ++p->seq;
        hipLaunchKernelGGL(keep_plan_kernel, dim3(1), dim3(kPlanThreads), keep_lds, st, f);
        IMU_TRY(await_headers(p, st));
        if (p->hdr.reusedB || p->hdr.overflow || p->hdr.err) return IMUNPACK_OK;
    }
    if (!at_once) {
        hipLaunchKernelGGL(setup_kernel, dim3(grid_for(std::max(std::max(idA, idC1), std::max(idB, kcA)), 256, 64), items),
                           dim3(256), 0, st, hdr, p->rowA, idA, p->c1, idC1, p->rowB, keep ? 0 : idB,
                           p->extraRows, (p->sB == IMUNPACK_BOTH && !keep) ? h : 0,
                           reinterpret_cast<int32_t *>(p->cols.colA_w), keep ? 0 : 2 * kcA, keep ? p->d_keep : nullptr, stride);
        if (scanA) IMU_TRY(scan_operand(A, n, lda, p->statsA, own_statsA, listA && !callerA));
    }
    // ---- phase 1: Unpack(A, B, I, b, strategy_A)
    auto closed_form = [&](const SlotSet &set, const int32_t *maxabs, const int32_t *via, int count, int which,
                           const int32_t *skip) {
        hipLaunchKernelGGL(level_major_kernel, dim3(1, items), dim3(kPlanThreads), 0, st, set, maxabs, via, count, p->sh,
                           p->tmpL, p->tmpCur, hdr, which, skip, stride, sstride);
    };
    const bool pair = !keep && !listA && !listB && !scanA && !scanB && std::max(std::max(n, h), d) <= kPairItems * kPlanThreads;
    // (A plan that has held a large product has room for its slots: the counts of so many do not fit LDS, whatever the sizes are now, and
    // the launches of run_greedy keep them in memory.)
    const bool both = !keep && callerA && callerB && !scanA && !scanB && std::max(std::max(n, h), d) <= kGreedyPairSlots &&
                      std::max(stA->ob_cap, stB->ob_cap) <= kGreedyPairList &&
                      std::max(greedy_lds(p, 1), greedy_lds(p, 2)) <= (size_t)kGreedyLdsMax;
    if (pair) {
        LevelPair f;
        f.a = p->rowA; f.b = p->rowB; f.c1 = p->c1; f.c2 = p->c2;
        f.max_a = p->statsA[p->sA == IMUNPACK_ROW ? 2 : 3]; f.max_b = p->statsB[p->sB == IMUNPACK_ROW ? 2 : 3];
        f.strategyA = p->sA; f.strategyB = p->sB;
        f.n = n; f.d = d; f.h = h; f.sh = p->sh;
        f.tmpL = p->tmpL; f.tmpCur = p->tmpCur;
        f.hdr = hdr;
        f.stride = stride; f.stats_stride = sstride;
        const bool beside = p->sB == IMUNPACK_ROW || p->sA == IMUNPACK_ROW;
        hipLaunchKernelGGL(level_major_pair_kernel, dim3(beside ? 2 : 1, items), dim3(kPlanThreads), 0, st, f);
    }
    else if (at_once) {}  // the first operand is unpacked, the second is to be unpacked anew
    else if (both) {
        GreedyPair f;
        f.g[0] = greedy_args(p, 1, (int)stA->ob_cap, stA->ob_count, sstride, CAP_LISTA, nullptr);
        f.g[1] = greedy_args(p, 2, (int)stB->ob_cap, stB->ob_count, sstride, CAP_LISTB, nullptr);
        f.ob[0] = stA->ob; f.ob[1] = stB->ob;
        f.keep[0] = p->obcopyA; f.keep[1] = p->obcopyB;
        f.keep_cap[0] = p->cap[CAP_EDGEA]; f.keep_cap[1] = p->cap[CAP_EDGEB];
        const int words = std::max(f.g[0].lds_words, f.g[1].lds_words);
        f.g[0].lds_words = f.g[1].lds_words = words;
        hipLaunchKernelGGL(greedy_pair_kernel, dim3(1, items), dim3(kPlanThreads), (size_t)words * sizeof(int32_t), st, f);
        IMU_TRY(launch_status());
    }
    else if (p->sA == IMUNPACK_ROW) closed_form(p->rowA, p->statsA[2], nullptr, n, CAP_ROWA, nullptr);
    else if (p->sA == IMUNPACK_COL) closed_form(p->c1, p->statsA[3], nullptr, d, CAP_C1, nullptr);
    else if (callerA) IMU_TRY(run_greedy(p, 1, stA->ob, (int)stA->ob_cap, stA->ob_count, sstride, CAP_LISTA, st));
    else IMU_TRY(run_greedy(p, 1, p->ob, p->cap[CAP_OB], p->obcnt, stride, CAP_OB, st));
    if (scanB) IMU_TRY(scan_operand(B, h, ldb, p->statsB, own_statsB, listB && !callerB));
    // ---- phase 2: Unpack(B_e, A_u, S_u, b, strategy_B); B_e has d1 columns
    if (keep && !at_once) {
        hipLaunchKernelGGL(keep_decide_kernel, dim3(1), dim3(kPlanThreads), 0, st, keep_args, p->c1, hdr, p->rowB);
        skip = &p->d_keep->same;
    }
    if (pair || both) {
    } else if (p->sB == IMUNPACK_ROW) {
        closed_form(p->rowB, p->statsB[2], nullptr, h, CAP_ROWB, skip);
        hipLaunchKernelGGL(identity_slots_kernel, dim3(grid_for(p->cap[CAP_C2], 256, 64), items), dim3(256), 0, st,
                           p->c2, hdr, skip, stride);
    } else if (p->sB == IMUNPACK_COL) {
        closed_form(p->c2, p->statsB[3], p->c1.root, 0, CAP_C2, skip);
    } else if (callerB) {
        IMU_TRY(run_greedy(p, 2, stB->ob, (int)stB->ob_cap, stB->ob_count, sstride, CAP_LISTB, st, skip));
    } else {
        IMU_TRY(run_greedy(p, 2, p->ob, p->cap[CAP_OB], p->obcnt, stride, CAP_OB, st, skip));
    }
    // ---- physical layouts
    const int col_blocks = items > 1 && p->cap[CAP_C2] <= kColSlotsLds * kPlanThreads ? 1 : kColBlocks;
    const int slices = fast_lds ? row_slices(n) + row_slices(h) : 2;
    const SparseArgs sparse = {p->statsB[1], h, p->sparse.cnt};
    auto lay_out = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(slices + col_blocks, items), dim3(kPlanThreads), dyn_bytes, st, p->rowA, n, p->layA,
                           phys_cap_rows(p->cap[CAP_ROWA]), p->tmpPA, p->rowB, h, p->layB,
                           phys_cap_rows(p->cap[CAP_ROWB]), p->tmpPB, p->c1, p->c2, p->cols, d,
                           phys_cap_cols(p->cap[CAP_C2]), p->s, p->sh, p->tmpE, p->tmpK, p->tmpR, p->tmpOff, hdr, fast_lds,
                           skip, stride, p->chunkB,
                           (int)(dyn_bytes / sizeof(int32_t)), sparse);
    };
    auto remember = [&]() {
        if (keep)
            hipLaunchKernelGGL(keep_remember_kernel, dim3(grid_for(p->cap[CAP_C1], 256, 16)), dim3(256), 0, st, p->c1,
                               (const PlanHeader *)hdr, p->snapRoot, p->snapExp, p->snapChild, p->d_keep);
        ++p->seq;
    };
    if (p->sparse.ent && !p->no_sparse) {
        lay_out(layouts_kernel<true>);
        remember();
        const ListsArgs f = {p->obcopyB, p->cap[CAP_EDGEB], p->sh, p->rowB, p->c2, p->layB.row_phys, p->cols.col_phys, skip, hdr, p->sparse, p->pin_hdr, p->seq};
        hipLaunchKernelGGL(lists_kernel, dim3(grid_for(p->cap[CAP_EDGEB], 256, 256)), dim3(256), 0, st, f);
        IMU_TRY(await_headers(p, st));
        if (!p->hdr.cols_left || p->hdr.overflow || p->hdr.err) return IMUNPACK_OK;
        p->no_sparse = 1;
    }
    lay_out(layouts_kernel<false>);
    remember();
    hipLaunchKernelGGL(publish_kernel, dim3(1, items), dim3(256), 0, st, (const PlanHeader *)hdr, p->pin_hdr, p->seq);
    return await_headers(p, st);
}

// First guesses of the capacities; every one of them is grown after a run that reports it too small.
static void guess_capacities(Plan *p) {
    const int64_t n = p->n, d = p->d, h = p->h;
    p->cap[CAP_ROWA] = std::max(p->cap[CAP_ROWA], (int)(p->sA == IMUNPACK_COL ? n : 2 * n + 256));
    p->cap[CAP_ROWB] = std::max(p->cap[CAP_ROWB], (int)(p->sB == IMUNPACK_COL ? h : 2 * h + 256));
    p->cap[CAP_C1] = std::max(p->cap[CAP_C1], (int)(p->sA == IMUNPACK_ROW ? d : 2 * d + 256));
    p->cap[CAP_C2] = std::max(p->cap[CAP_C2], (int)(2 * d + 512));
    p->cap[CAP_EDGEA] = std::max(p->cap[CAP_EDGEA], (int)std::min<int64_t>(n * d, std::max<int64_t>(n * d / 64, 4096)));
    p->cap[CAP_EDGEB] = std::max(p->cap[CAP_EDGEB], (int)std::min<int64_t>(2 * h * d, std::max<int64_t>(h * d / 64, 4096)));
    // (listed columns hold a digit in kSparseShare rows on average, so that a list holds d / 12; and Alg. 4 splits the longest row or column
    // first: behind a column of h / kSparseMost digits no row has more, h / 3 in all rows of a list)
    p->cap[CAP_SPARSE] = (int)std::min((h + 2) / 3, (d + 5) / 6) / kSparseRows * kSparseRows + 2 * kSparseRows;
    p->cap[CAP_OB] = std::max(p->cap[CAP_OB], (int)std::min<int64_t>(std::max(n, h) * d, std::max<int64_t>(std::max(n, h) * d / 64, 4096)));
}

int64_t plan_item_bytes(int64_t n, int64_t d, int64_t h, int b, int strategy_A, int strategy_B) {
    Plan p;
    memset((void *)&p, 0, sizeof(p));
    p.n = n; p.d = d; p.h = h; p.b = b; p.sA = strategy_A; p.sB = strategy_B;
    p.nitems = 2;  // of several
    guess_capacities(&p);
    (void)carve(&p, nullptr, false, false);
    return p.item_bytes;
}

// The plan of one product (nitems = 1), or of every product of a batch of one shape: A, B, the statistics and
// the OB lists of item i lie i * op_stride bytes behind those of item 0.
int plan_impl(const int32_t *A, int64_t n, int64_t d, int64_t lda, const int32_t *B, int64_t h, int64_t ldb, int b,
              int strategy_A, int strategy_B, const imunpack_stats_t *stats_A, const imunpack_stats_t *stats_B,
              imunpack_plan_t **plan, int nitems, int64_t op_stride, hipStream_t st) {
    if (!A || !B || !plan || n <= 0 || d <= 0 || h <= 0 || lda < d || ldb < d || b < 2 || b > 8 || nitems < 1 ||
        nitems > kMaxItems)
        return IMUNPACK_EINVAL;
    if (strategy_A < 0 || strategy_A > 2 || strategy_B < 0 || strategy_B > 2) return IMUNPACK_EINVAL;
    if (n > (1 << 24) || d > (1 << 24) || h > (1 << 24)) return IMUNPACK_EINVAL;
    Plan *p = *plan;
    if (!p) {
        p = new (std::nothrow) Plan();
        if (!p) return IMUNPACK_ENOMEM;
        memset(p, 0, sizeof(*p));
        p->guess_fusable = 1;
    }
    p->bound_pending = 0;
    const bool same = p->valid && p->nitems == nitems && p->n == n && p->d == d && p->h == h && p->b == b && p->sA == strategy_A &&
                      p->sB == strategy_B;
    p->valid = 0;
    p->unpacked = 0;
    p->n = n; p->d = d; p->h = h; p->b = b; p->sA = strategy_A; p->sB = strategy_B;
    p->s = 1 << (b - 1); p->sh = b - 1;
    p->stream = st;
    p->nitems = nitems;
    p->op_stride = op_stride;
    p->chunkB = small_tiles_possible(n, h, nitems) ? kChunk : kTile;
    if (!same) {
        guess_capacities(p);
        p->ignore_listA = p->ignore_listB = 0;
        p->no_sparse = 0;
    }
    const bool ownA = !(stats_A && stats_A->rowcnt && stats_A->colcnt && stats_A->rowmax && stats_A->colmax);
    const bool ownB = !(stats_B && stats_B->rowcnt && stats_B->colcnt && stats_B->rowmax && stats_B->colmax);
    int rc = IMUNPACK_OK;
    if (p->pin_items < nitems) {  // the pinned copy of the headers
        if (p->pin_hdr) (void)hipHostFree(p->pin_hdr);
        p->pin_hdr = nullptr;
        p->pin_items = 0;
        const size_t bytes = (size_t)nitems * sizeof(PlanHeader) + 2 * kBoundBlocks * sizeof(unsigned long long);
        if (hipHostMalloc((void **)&p->pin_hdr, bytes, hipHostMallocCoherent) != hipSuccess) {
            (void)hipGetLastError();
            p->pin_hdr = nullptr;
            rc = IMUNPACK_ENOMEM;
        } else {
            memset(p->pin_hdr, 0, bytes);
            p->pin_bounds = reinterpret_cast<unsigned long long *>(p->pin_hdr + nitems);
            p->pin_items = nitems;
        }
    }
    for (int attempt = 0; rc == IMUNPACK_OK && attempt < 24; ++attempt) {
        const size_t need = carve(p, nullptr, ownA, ownB);
        if (need > p->arena_bytes) {
            if (p->arena) {
                hipError_t e = hipFree(p->arena);
                p->arena = nullptr;
                p->arena_bytes = 0;
                if (e != hipSuccess) { g_last_hip_error = (int)e; rc = IMUNPACK_EHIP; break; }
            }
            const size_t want = need + need / 4;
            hipError_t e = hipMalloc((void **)&p->arena, want);
            if (e != hipSuccess) { (void)hipGetLastError(); p->arena = nullptr; rc = IMUNPACK_ENOMEM; break; }
            p->arena_bytes = want;
        }
        carve(p, p->arena, ownA, ownB);
        {  // what is kept of the plan before is only good for the same arrays at the same addresses
            unsigned long long sig = (unsigned long long)(uintptr_t)p->arena * 1000003ull + (unsigned long long)(uintptr_t)p->d_keep;
            const long long parts[] = {n, d, h, b, strategy_A, strategy_B, ownA, ownB, (long long)(uintptr_t)B, (long long)ldb,
                                       p->cap[CAP_SPARSE]};
            for (long long v : parts) sig = sig * 1099511628211ull + (unsigned long long)v;
            for (int c = 0; c <= CAP_OB; ++c) sig = sig * 1099511628211ull + (unsigned long long)p->cap[c];
            if (sig != p->keep_sig) p->keep_valid = 0;
            p->keep_sig = sig;
        }
        if (!ownA) { p->statsA[0] = stats_A->rowcnt; p->statsA[1] = stats_A->colcnt; p->statsA[2] = stats_A->rowmax; p->statsA[3] = stats_A->colmax; }
        if (!ownB) { p->statsB[0] = stats_B->rowcnt; p->statsB[1] = stats_B->colcnt; p->statsB[2] = stats_B->rowmax; p->statsB[3] = stats_B->colmax; }
        rc = run_plan(p, A, lda, B, ldb, stats_A, stats_B, ownA, ownB, st);
        if (rc != IMUNPACK_OK) break;
        int err = 0, overflow = 0, needed[10] = {};
        for (int i = 0; i < nitems; ++i) {
            const PlanHeader &hi = p->pin_hdr[i];
            err = std::min(err, (int)hi.err);
            overflow |= hi.overflow;
            for (int c = 0; c <= CAP_OB; ++c)
                if (hi.overflow & (1 << c)) needed[c] = std::max(needed[c], (int)hi.need[c]);
        }
        if (err) { rc = err; p->keep_valid = 0; break; }
        if (!overflow && p->hdr.nsparse && p->hdr.sparse_room > p->sparse.cap) {  // a list that was too short
            p->cap[CAP_SPARSE] = (p->hdr.sparse_room + p->hdr.sparse_room / 8 + kSparseRows) / kSparseRows * kSparseRows;
            p->keep_valid = 0;
            continue;
        }
        if (!overflow) {
            p->valid = 1;
            p->canon_valid = 0;
            p->keep_valid = p->keep_B;
            if (!p->hdr.reusedB) p->kept_Beu = nullptr;  // what an earlier unpack wrote belongs to another plan
            p->fp6 = p->digits_req == IMUNPACK_DIGITS_FP6 && b <= 4;
            p->bothA = strategy_A == IMUNPACK_BOTH;
            p->bothB = strategy_B == IMUNPACK_BOTH;
            break;
        }
        p->keep_valid = 0;
        if (overflow & (1 << CAP_LISTA)) p->ignore_listA = 1;
        if (overflow & (1 << CAP_LISTB)) p->ignore_listB = 1;
        if (needed[CAP_C2] > kColSlotsLds * kPlanThreads) p->no_sparse = 1;
        for (int c = 0; c <= CAP_OB; ++c)
            if (overflow & (1 << c)) {
                int64_t nv = std::max<int64_t>((int64_t)needed[c] + needed[c] / 8 + 256, (int64_t)p->cap[c] * 2);
                if (nv > (1ll << 30)) { rc = IMUNPACK_ENOMEM; break; }
                p->cap[c] = (int)nv;
            }
    }
    if (rc == IMUNPACK_OK && !p->valid) rc = IMUNPACK_ENOMEM;  // the attempts ran out
    if (rc != IMUNPACK_OK && !p->valid) {
        if (!*plan) {
            if (p->arena) (void)hipFree(p->arena);
            destroy_handles(p);
            delete p;
        }
        return rc;
    }
    *plan = p;
    return IMUNPACK_OK;
}

// Item i of a batch's plan as a plan of its own: a copy that borrows the arena (never destroyed).
Plan item_view(const Plan &batch, int i) {
    Plan v = batch;
    const int64_t off = (int64_t)i * batch.item_bytes;
    v.nitems = 1;
    v.d_hdr += i;
    v.hdr = batch.pin_hdr[i];
    v.pin_hdr = batch.pin_hdr + i;
    move_to_item(v.rowA, off);
    move_to_item(v.rowB, off);
    move_to_item(v.c1, off);
    move_to_item(v.c2, off);
    move_to_item(v.layA, off);
    move_to_item(v.layB, off);
    move_to_item(v.cols, off);
    v.bound_pending = 0;
    return v;
}

}  // namespace imu

using namespace imu;

extern "C" int imunpack_plan(const int32_t *A, int64_t n, int64_t d, int64_t lda, const int32_t *B,
                             int64_t h, int64_t ldb, int b, int strategy_A, int strategy_B,
                             const imunpack_stats_t *stats_A, const imunpack_stats_t *stats_B,
                             imunpack_plan_t **plan, imunpack_stream_t stream) {
    return plan_impl(A, n, d, lda, B, h, ldb, b, strategy_A, strategy_B, stats_A, stats_B, plan, 1, 0, (hipStream_t)stream);
}

extern "C" int imunpack_plan_dims(const imunpack_plan_t *p, int64_t *n_u, int64_t *d_u, int64_t *h_u,
                                  int32_t *n_groups) {
    if (!p || !p->valid) return IMUNPACK_EINVAL;
    if (n_u) *n_u = p->hdr.n_u;
    if (d_u) *d_u = p->hdr.d_u;
    if (h_u) *h_u = p->hdr.h_u;
    if (n_groups) *n_groups = p->hdr.ngroups;
    return IMUNPACK_OK;
}

extern "C" int imunpack_plan_keep_weights(imunpack_plan_t *p, int keep) {
    if (!p) return IMUNPACK_EINVAL;
    p->keep_B = keep != 0;
    if (!keep) {
        p->keep_valid = 0;
        p->kept_Beu = nullptr;
    }
    return IMUNPACK_OK;
}

extern "C" int imunpack_plan_weights_reused(const imunpack_plan_t *p) {
    return (p && p->valid && p->hdr.reusedB) ? 1 : 0;
}

namespace imu {

// Canonical (paper-order) numbering of the slots of one set.  Slots are appended in runs: a level of
// the closed-form UnpackRow / UnpackColumn, or a batch of UnpackBoth.  Inside a run the paper's
// order is (count at the split descending, index of the split slot ascending), the index being the
// canonical one.  key = run << 48 | (0xFFFFFF - count) << 24 | split slot (internal numbering).
static int canonical_order(const SlotSet &set, int nbase, int count, const std::vector<int> *base_canon,
                           hipStream_t st, std::vector<int> &canon_of, std::vector<unsigned long long> &key) {
    canon_of.assign((size_t)count, 0);
    key.clear();
    for (int x = 0; x < nbase && x < count; ++x) canon_of[x] = base_canon ? (*base_canon)[x] : x;
    const int extra = count - nbase;
    if (extra <= 0) return IMUNPACK_OK;
    key.resize((size_t)extra);
    IMU_HIP(hipMemcpyAsync(key.data(), set.key + nbase, (size_t)extra * sizeof(unsigned long long),
                           hipMemcpyDeviceToHost, st));
    IMU_HIP(hipStreamSynchronize(st));
    std::vector<int> order((size_t)extra);
    std::vector<char> assigned((size_t)count, 0);
    for (int x = 0; x < nbase && x < count; ++x) assigned[x] = 1;
    for (int t = 0; t < extra; ++t) order[t] = t;
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return (key[a] >> 48) < (key[b] >> 48); });
    int next = nbase;
    for (size_t lo = 0; lo < order.size();) {
        size_t hi = lo;
        const unsigned long long run = key[order[lo]] >> 48;
        while (hi < order.size() && (key[order[hi]] >> 48) == run) ++hi;
        auto minor = [&](int t) { return (unsigned)((key[t] >> 24) & 0xFFFFFF); };
        auto parent = [&](int t) { return (int)(key[t] & 0xFFFFFF); };
        for (size_t q = lo; q < hi; ++q) {  // the split slot must come from an earlier run
            const int par = parent(order[q]);
            if (par < 0 || par >= count || !assigned[par]) return IMUNPACK_EHIP;
        }
        std::sort(order.begin() + lo, order.begin() + hi, [&](int a, int b) {
            if (minor(a) != minor(b)) return minor(a) < minor(b);
            return canon_of[parent(a)] < canon_of[parent(b)];
        });
        for (size_t q = lo; q < hi; ++q) {
            canon_of[nbase + order[q]] = next++;
            assigned[nbase + order[q]] = 1;
        }
        lo = hi;
    }
    return IMUNPACK_OK;
}

struct CanonHost {
    std::vector<int> rowA, rowB, c1, c2;  // internal slot -> canonical slot
    std::vector<unsigned long long> keyA, keyB, key1, key2;  // sort keys of the appended slots of each set
};

static int fetch_i32(std::vector<int32_t> &dst, const int32_t *src, size_t count, hipStream_t st) {
    dst.resize(count);
    if (count) IMU_HIP(hipMemcpyAsync(dst.data(), src, count * 4, hipMemcpyDeviceToHost, st));
    return IMUNPACK_OK;
}

static int build_canonical(Plan *p, CanonHost &c) {
    hipStream_t st = p->stream;
    const PlanHeader &h = p->hdr;
    IMU_TRY(canonical_order(p->rowA, (int)p->n, h.n_u, nullptr, st, c.rowA, c.keyA));
    IMU_TRY(canonical_order(p->rowB, (int)p->h, h.h_u, nullptr, st, c.rowB, c.keyB));
    IMU_TRY(canonical_order(p->c1, (int)p->d, h.d1, nullptr, st, c.c1, c.key1));
    IMU_TRY(canonical_order(p->c2, h.d1, h.d_u, &c.c1, st, c.c2, c.key2));
    if (!p->canon_valid) {
        // physical row / column of every canonical slot, for imunpack_unpack_canonical
        std::vector<int32_t> phys, out;
        auto upload = [&](const int32_t *dev_phys, const std::vector<int> &canon, int32_t *dev_out) -> int {
            IMU_TRY(fetch_i32(phys, dev_phys, canon.size(), st));
            IMU_HIP(hipStreamSynchronize(st));
            out.assign(canon.size(), 0);
            for (size_t x = 0; x < canon.size(); ++x) out[(size_t)canon[x]] = phys[x];
            if (!out.empty()) IMU_HIP(hipMemcpy(dev_out, out.data(), out.size() * 4, hipMemcpyHostToDevice));
            return IMUNPACK_OK;
        };
        IMU_TRY(upload(p->layA.row_phys, c.rowA, p->canon_rowphysA));
        IMU_TRY(upload(p->layB.row_phys, c.rowB, p->canon_rowphysB));
        IMU_TRY(upload(p->cols.col_phys, c.c2, p->canon_colphys));
        IMU_TRY(upload(p->cols.acol_phys, c.c2, p->canon_acolphys));
        p->canon_valid = 1;
    }
    return IMUNPACK_OK;
}

int ensure_canonical(Plan *p) {
    if (p->canon_valid) return IMUNPACK_OK;
    CanonHost c;
    return build_canonical(p, c);
}

}  // namespace imu

extern "C" int imunpack_plan_export(imunpack_plan_t *p, int32_t *rowA_src, int32_t *rowA_exp,
                                    int32_t *rowB_src, int32_t *rowB_exp, int32_t *col_src,
                                    int32_t *col_exp, int32_t *col_parent, int32_t *ops, int64_t *n_ops) {
    if (!p || !p->valid) return IMUNPACK_EINVAL;
    hipStream_t st = p->stream;
    const PlanHeader &h = p->hdr;
    CanonHost c;
    IMU_TRY(build_canonical(p, c));
    std::vector<int32_t> root, ex, root1, ex1;
    auto rows_out = [&](const SlotSet &set, const std::vector<int> &canon, int32_t *o_src, int32_t *o_exp) -> int {
        if (!o_src && !o_exp) return IMUNPACK_OK;
        IMU_TRY(fetch_i32(root, set.root, canon.size(), st));
        IMU_TRY(fetch_i32(ex, set.exp, canon.size(), st));
        IMU_HIP(hipStreamSynchronize(st));
        for (size_t x = 0; x < canon.size(); ++x) {
            if (o_src) o_src[canon[x]] = root[x];
            if (o_exp) o_exp[canon[x]] = ex[x];
        }
        return IMUNPACK_OK;
    };
    IMU_TRY(rows_out(p->rowA, c.rowA, rowA_src, rowA_exp));
    IMU_TRY(rows_out(p->rowB, c.rowB, rowB_src, rowB_exp));
    if (col_src || col_exp) {
        IMU_TRY(fetch_i32(root, p->c2.root, (size_t)h.d_u, st));
        IMU_TRY(fetch_i32(ex, p->c2.exp, (size_t)h.d_u, st));
        IMU_TRY(fetch_i32(root1, p->c1.root, (size_t)h.d1, st));
        IMU_TRY(fetch_i32(ex1, p->c1.exp, (size_t)h.d1, st));
        IMU_HIP(hipStreamSynchronize(st));
        for (int x = 0; x < h.d_u; ++x) {
            const int r1 = root[x];  // column slot after unpacking A that this column descends from
            if (col_src) col_src[c.c2[x]] = root1[r1];
            if (col_exp) col_exp[c.c2[x]] = ex1[r1] + ex[x];
        }
    }
    // The appended slots in the paper's numbering are numbered in the order their splits were made, and
    // the sort key of an appended slot names the slot that was split for it (low 24 bits, internal
    // numbering) and the run it was made in (level of the closed-form UnpackRow / UnpackColumn, batch of
    // UnpackBoth; a batch holds splits of one kind only).
    const int d = (int)p->d, nA = (int)p->n, nB = (int)p->h;
    auto parent_of = [](const std::vector<unsigned long long> &key, int t) { return (int)(key[(size_t)t] & 0xFFFFFF); };
    if (col_parent) {
        for (int x = 0; x < h.d1; ++x)  // the columns the second call started from: originals and A's appended ones
            col_parent[c.c2[x]] = x < d ? -1 : c.c2[(size_t)parent_of(c.key1, x - d)];
        for (int x = h.d1; x < h.d_u; ++x) col_parent[c.c2[x]] = c.c2[(size_t)parent_of(c.key2, x - h.d1)];
    }
    const int64_t total_ops = (int64_t)(h.n_u - nA) + (h.d1 - d) + (h.h_u - nB) + (h.d_u - h.d1);
    if (n_ops) *n_ops = total_ops;
    if (ops) {
        struct Op { unsigned long long run; int kind, canon, parent; };
        int64_t at = 0;
        for (int call = 0; call < 2; ++call) {
            const std::vector<int> &rc = call ? c.rowB : c.rowA, &cc = call ? c.c2 : c.c1;
            const std::vector<unsigned long long> &rk = call ? c.keyB : c.keyA, &ck = call ? c.key2 : c.key1;
            const int rbase = call ? nB : nA, cbase = call ? h.d1 : d;
            std::vector<Op> seq;
            seq.reserve(rk.size() + ck.size());
            for (size_t t = 0; t < rk.size(); ++t)
                seq.push_back({rk[t] >> 48, 0, rc[(size_t)rbase + t], rc[(size_t)parent_of(rk, (int)t)]});
            for (size_t t = 0; t < ck.size(); ++t)
                seq.push_back({ck[t] >> 48, 1, cc[(size_t)cbase + t], cc[(size_t)parent_of(ck, (int)t)]});
            // one-axis strategies append along one axis only: creation order is the numbering; UnpackBoth
            // interleaves the axes batch by batch
            std::sort(seq.begin(), seq.end(), [](const Op &a, const Op &b) {
                if (a.run != b.run) return a.run < b.run;
                return a.canon < b.canon;
            });
            for (const Op &o : seq) {
                ops[3 * at] = call;
                ops[3 * at + 1] = o.kind;
                ops[3 * at + 2] = o.parent;
                ++at;
            }
        }
    }
    return IMUNPACK_OK;
}

extern "C" int imunpack_plan_destroy(imunpack_plan_t *p) {
    if (!p) return IMUNPACK_OK;
    int rc = IMUNPACK_OK;
    if (p->arena) {
        hipError_t e = hipFree(p->arena);
        if (e != hipSuccess) { g_last_hip_error = (int)e; rc = IMUNPACK_EHIP; }
    }
    destroy_handles(p);
    delete p;
    return rc;
}

extern "C" int imunpack_price(const imunpack_stats_t *stA, int64_t n, const imunpack_stats_t *stB, int64_t h,
                              int64_t d, int b, void *workspace, int64_t *dims_out, double *ratio_out, int *best_A,
                              int *best_B, imunpack_stream_t stream) {
    if (!stA || !stB || !stA->rowmax || !stA->colmax || !stB->rowmax || !stB->colmax || !workspace || n <= 0 ||
        h <= 0 || d <= 0 || b < 2 || b > 8 || (uintptr_t)workspace % 8)
        return IMUNPACK_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    unsigned long long *sums = static_cast<unsigned long long *>(workspace), host[5];
    static_assert(IMUNPACK_PRICE_WORKSPACE_BYTES >= sizeof(host), "workspace");
    hipLaunchKernelGGL(clear_sums_kernel, dim3(1), dim3(64), 0, st, sums, 5);
    const int64_t longest = std::max(std::max(n, h), d);
    hipLaunchKernelGGL(price_kernel, dim3(grid_for(longest, 256, 1024)), dim3(256), 0, st, stA->rowmax, n,
                       stB->rowmax, h, stA->colmax, stB->colmax, d, b - 1, sums);
    IMU_TRY(launch_status());
    IMU_HIP(hipMemcpyAsync(host, sums, sizeof(host), hipMemcpyDeviceToHost, st));
    IMU_HIP(hipStreamSynchronize(st));
    // (strategy_A, strategy_B): (ROW,ROW), (ROW,COL), (COL,ROW), (COL,COL)
    const unsigned long long dims[4][3] = {{host[0], (unsigned long long)d, host[1]},
                                            {host[0], host[3], (unsigned long long)h},
                                            {(unsigned long long)n, host[2], host[1]},
                                            {(unsigned long long)n, host[4], (unsigned long long)h}};
    double best = 0.0;
    int bi = -1;
    for (int q = 0; q < 4; ++q) {
        for (int c = 0; c < 3; ++c) {
            if (dims[q][c] > (1ull << 62)) return IMUNPACK_ERANGE;
            if (dims_out) dims_out[3 * q + c] = (int64_t)dims[q][c];
        }
        const double r = ((double)dims[q][0] / (double)n) * ((double)dims[q][1] / (double)d) *
                         ((double)dims[q][2] / (double)h);
        if (ratio_out) ratio_out[q] = r;
        if (bi < 0 || r < best) { best = r; bi = q; }
    }
    if (best_A) *best_A = (bi & 2) ? IMUNPACK_COL : IMUNPACK_ROW;
    if (best_B) *best_B = (bi & 1) ? IMUNPACK_COL : IMUNPACK_ROW;
    return IMUNPACK_OK;
}
