// Runs the planner's row layout (rows_layout.inc, the function as plan.hip has it) on the CPU: a workgroup of 1024 threads as
// coroutines that change hands at barriers only.  Between two barriers the waves of a workgroup may run in any order on the
// device, so the result has to be the same for every order: first to last, last to first and a few shuffles, with and without
// LDS, in one slice and in several.  Levels, places and what is said of every chunk are also checked against the inputs.
#define __HIP_PLATFORM_AMD__ 1
#include "common.h"

#include <ucontext.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <numeric>
#include <random>
#include <string>
#include <vector>

namespace {
constexpr int kThreads = 1024, kWaves = kThreads / 64;
struct { unsigned x; } threadIdx;

// ---- the workgroup
struct Fiber {
    ucontext_t at;
    std::vector<char> stack = std::vector<char>(64 * 1024);
    bool done = false;
};
std::vector<Fiber> fibers(kThreads);
ucontext_t scheduler;
std::function<void()> body;

void entry() {
    body();
    fibers[threadIdx.x].done = true;
}
void barrier() { const unsigned me = threadIdx.x; swapcontext(&fibers[me].at, &scheduler); }

// order: the waves in the order in which they run from one barrier to the next
void run_workgroup(const std::vector<int> &order, std::function<void()> f) {
    body = std::move(f);
    for (Fiber &x : fibers) {
        getcontext(&x.at);
        x.at.uc_stack.ss_sp = x.stack.data();
        x.at.uc_stack.ss_size = x.stack.size();
        x.at.uc_link = &scheduler;
        x.done = false;
        makecontext(&x.at, entry, 0);
    }
    for (int ended = 0; ended == 0;) {
        for (int wave : order)
            for (int lane = 0; lane < 64; ++lane) {
                threadIdx.x = (unsigned)(wave * 64 + lane);
                swapcontext(&scheduler, &fibers[threadIdx.x].at);
            }
        for (const Fiber &x : fibers) ended += x.done;
        if (ended != 0 && ended != kThreads) {
            std::printf("a barrier that %d threads do not reach\n", ended);
            std::exit(1);
        }
    }
}
}  // namespace

namespace imu {
using std::max;
using std::min;
thread_local int g_last_hip_error = 0;
constexpr int kPlanThreads = kThreads;
static void __syncthreads() { barrier(); }
static void atomicMax(int32_t *p, int32_t v) { *p = max(*p, v); }
static void atomicMin(int32_t *p, int32_t v) { *p = min(*p, v); }
static void flag_overflow(PlanHeader *hdr, int which, int) { hdr->overflow |= 1 << which; }
// the workgroup-wide helpers: the barriers of those in plan.hip, sums and maxima without the wave operations
static int scratch[kThreads];
static int block_max(int v, int *) {
    scratch[threadIdx.x] = v;
    __syncthreads();
    const int r = *std::max_element(scratch, scratch + kThreads);
    __syncthreads();
    return r;
}
template <class V, class E>
static int ordered_scan(int N, int base, V value, E emit, int *) {
    const int each = (N + kThreads - 1) / kThreads, lo = min(N, (int)threadIdx.x * each), hi = min(N, lo + each);
    int sum = 0;
    for (int x = lo; x < hi; ++x) sum += value(x);
    scratch[threadIdx.x] = sum;
    __syncthreads();
    int run = std::accumulate(scratch, scratch + threadIdx.x, base);
    const int total = std::accumulate(scratch, scratch + kThreads, 0);
    for (int x = lo; x < hi; ++x) {
        const int v = value(x);
        emit(x, run);
        run += v;
    }
    __syncthreads();
    return total;
}
#include "rows_layout.inc"
}  // namespace imu

using namespace imu;

// What a layout leaves in memory.
struct Result {
    std::vector<int32_t> prow, row_phys, src_pstart, src_nlev, tile_src0, chunk_src0, tile_flat, chunk_lev;
    PlanHeader hdr;
    bool operator==(const Result &o) const {
        return prow == o.prow && row_phys == o.row_phys && src_pstart == o.src_pstart && src_nlev == o.src_nlev && tile_src0 == o.tile_src0 &&
               chunk_src0 == o.chunk_src0 && tile_flat == o.tile_flat && chunk_lev == o.chunk_lev && memcmp(&hdr, &o.hdr, sizeof(hdr)) == 0;
    }
};

static Result lay_out(const std::vector<int> &levels, int operand, int chunk, bool fast, int nslices, const std::vector<int> &order) {
    const int n = (int)levels.size();
    std::vector<int32_t> root(n), exp(n, 0);
    std::iota(root.begin(), root.end(), 0);
    for (int l = 1; l < *std::max_element(levels.begin(), levels.end()); ++l)
        for (int i = 0; i < n; ++i)
            if (levels[i] > l) {
                root.push_back(i);
                exp.push_back(l);
            }
    const int32_t count = (int32_t)root.size();
    const int phys = (int)((int64_t)count * kChunk / (kChunk - 8) + 2 * kTile);  // as the planner sizes the arrays
    Result r;
    memset(&r.hdr, 0, sizeof(r.hdr));
    r.prow.assign(phys, -7);
    r.row_phys.assign(count, -7);
    r.src_pstart.assign(n + 1, -7);
    r.src_nlev.assign(n + 1, -7);
    r.tile_src0.assign(phys / kTile + 2, -7);
    r.chunk_src0.assign(phys / kChunk + 8, -7);
    r.tile_flat.assign(phys / kTile + 2, -7);
    r.chunk_lev.assign(phys / kChunk + 8, -7);
    std::vector<unsigned long long> rowsum(phys, 1);
    SlotSet rows = {};
    rows.root = root.data();
    rows.exp = exp.data();
    rows.cap = count;
    RowLayout lay = {};
    lay.prow = r.prow.data();
    lay.row_phys = r.row_phys.data();
    lay.src_pstart = r.src_pstart.data();
    lay.src_nlev = r.src_nlev.data();
    lay.tile_src0 = r.tile_src0.data();
    lay.chunk_src0 = r.chunk_src0.data();
    lay.tile_flat = r.tile_flat.data();
    lay.chunk_lev = r.chunk_lev.data();
    lay.rowsum = rowsum.data();
    int lds[40];
    for (int slice = 0; slice < nslices; ++slice) {
        std::vector<int32_t> dyn(2 * n + phys / kChunk + 8, -9), tmp(n, -9);
        run_workgroup(order, [&] {
            rows_layout(rows, n, &count, lay, phys, phys / kTile + 2, tmp.data(), &r.hdr, operand, chunk, lds, fast ? dyn.data() : nullptr, slice, nslices);
        });
    }
    return r;
}

// The result against the levels that went in; returns what is wrong, or nothing.
static std::string wrong(const Result &r, const std::vector<int> &levels, int operand, int chunk) {
    if (r.hdr.err || r.hdr.overflow) return "err or overflow";
    const int n = (int)levels.size(), rows = operand ? r.hdr.Np : r.hdr.Mp, even = operand ? r.hdr.evenB : r.hdr.evenA;
    const int step = even && operand ? kEvenStep : 1, chunks = rows / chunk;
    std::vector<char> taken(rows, 0);
    for (int i = 0; i < n; ++i) {
        if (r.src_nlev[i] != levels[i]) return "level count of row " + std::to_string(i);
        const int first = r.src_pstart[i], last = first + (levels[i] - 1) * step;
        if (first < 0 || last >= rows || first / chunk != last / chunk) return "place of row " + std::to_string(i);
        const int ch = first / chunk;
        if (i < r.chunk_src0[ch] || i >= r.chunk_src0[ch + 1]) return "chunk of row " + std::to_string(i);
        for (int l = 0; l < levels[i]; ++l) {
            if (r.prow[first + l * step] != (i | l << kProwLevel) || taken[first + l * step]++) return "physical row of row " + std::to_string(i);
        }
    }
    for (int p = 0; p < rows; ++p)
        if (!taken[p] && r.prow[p] != -1) return "padding row " + std::to_string(p);
    if (operand == 0)
        for (int ch = 0; ch < chunks; ++ch) {
            const int a = r.chunk_src0[ch], e = r.chunk_src0[ch + 1];
            if (a == e) continue;
            const bool alike = std::all_of(levels.begin() + a, levels.begin() + e, [&](int l) { return l == levels[a]; });
            if (r.chunk_lev[ch] != (even ? even : alike ? levels[a] : 0)) return "levels of chunk " + std::to_string(ch) + ": " + std::to_string(r.chunk_lev[ch]);
        }
    return "";
}

int main() {
    std::mt19937 rng(5);
    std::vector<std::vector<int>> orders;
    std::vector<int> waves(kWaves);
    std::iota(waves.begin(), waves.end(), 0);
    orders.push_back(waves);
    orders.emplace_back(waves.rbegin(), waves.rend());
    for (int k = 0; k < 3; ++k) {
        std::shuffle(waves.begin(), waves.end(), rng);
        orders.push_back(waves);
    }
    // most rows have `most` levels, a share of them `other` ones
    struct Case { int n, most, other; double share; };
    const Case cases[] = {{1, 1, 1, 0},      {63, 1, 1, 0},      {65, 1, 1, 0},        {1025, 1, 1, 0},     {4096, 1, 1, 0},      {12608, 1, 1, 0},
                          {300, 1, 2, 0.01}, {4096, 1, 2, 0.3},  {9424, 1, 3, 0.002},  {1000, 2, 1, 0.004}, {3003, 2, 1, 0.3},    {12608, 2, 2, 0},
                          {1025, 3, 2, 0.01}, {4096, 4, 3, 0.02}, {2890, 4, 1, 0.5},   {700, 5, 2, 0.4},    {8880, 2, 3, 0.2}};
    int failures = 0, runs = 0;
    for (const Case &c : cases) {
        std::vector<int> levels(c.n, c.most);
        for (int &l : levels)
            if (std::uniform_real_distribution<>(0, 1)(rng) < c.share) l = c.other;
        for (int form = 0; form < 3; ++form) {
            const int operand = form > 0, chunk = form == 1 ? kTile : kChunk;
            for (int slices : {0, 1, 2, 4}) {  // 0: without LDS
                Result first;
                for (size_t o = 0; o < orders.size(); ++o, ++runs) {
                    const Result r = lay_out(levels, operand, chunk, slices > 0, std::max(slices, 1), orders[o]);
                    std::string what = wrong(r, levels, operand, chunk);
                    if (o == 0) first = r;
                    else if (what.empty() && !(r == first)) what = "another result than with the waves in order";
                    if (!what.empty()) {
                        ++failures;
                        std::printf("%d rows of %d and %d levels, operand %d, chunks of %d, %d slices, order %zu: %s\n", c.n, c.most, c.other, operand,
                                    chunk, slices, o, what.c_str());
                    }
                }
            }
        }
    }
    std::printf("%d runs, %d failures\n", runs, failures);
    return failures != 0;
}
