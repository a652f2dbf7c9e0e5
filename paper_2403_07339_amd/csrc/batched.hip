// Strided-batched exact integer GEMMs: the products of a Transformer come in batches of equal shape
// (Sec. 1 "Notations": P = Q K^T and O = M V and their gradients once per sequence and head; a linear
// layer is the batch of one).  Each item runs the whole path -- the RTN step alpha_p / (0.5 beta) of
// Eq. (quantized_A) from the item's own percentile, quantize + scan of both operands, unpack plan,
// digit scatter, int8 GEMM with the recombination and the dequantisation of Eq. (quantized_gemm) in
// its epilogue.  The items of a batch share every launch (one more grid dimension; the arrays of item i lie a
// fixed distance behind those of item 0), so a batch takes the launches and the two host waits of one
// product: 24 heads of 197 tokens, forward and backward, 38.6 ms one after the other, 1.5 ms this way.
// The steps stay in device memory from the kernel that forms them to the kernels that divide and multiply by
// them; the host reads the sizes of the unpacked problems once (inside the plan call) and, at the end, whether
// an item was refused by the fused GEMM or held a NaN.
#include "common.h"

#include <algorithm>
#include <cstring>
#include <new>

namespace imu {
__global__ void clear_flags_kernel(int32_t *flags, int count) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < count; i += gridDim.x * blockDim.x) flags[i] = 0;
}

// The flags of a group to the host, the word it waits for behind them; leaves them cleared for the next group.
__global__ void tell_flags_kernel(int32_t *flags, int count, int32_t *host, int32_t *word, int32_t seq) {
    for (int i = threadIdx.x; i < count; i += blockDim.x) {
        __hip_atomic_store(host + i, flags[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        flags[i] = 0;
    }
    stores_done();
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store(word, seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
}  // namespace imu

struct imunpack_batch {
    imunpack_plan_t *plan;
    char *arena;           // flags, then per item: Q_A, Q_B, statistics, OB lists, steps, percentile workspace
    size_t arena_bytes;
    int8_t *ue;            // A stores and B_eu of all items
    size_t ue_bytes;
    void *ws;              // int64 unpacked product for items that cannot take the fused launch
    size_t ws_bytes;
    int32_t *pin_flags;    // pinned: [0] whether any item flagged NaN / Inf / overflow, [1 + i] item i was refused; last: the
                           // sequence number of the group that wrote them
    int32_t seq;
    int32_t *clean_flags;  // the device's flags as a call that went through left them: cleared
};

using namespace imu;

// Device memory of the items that go through the launches together: operands, plans and stores.
static constexpr int64_t kGroupBytes = 2ll << 30;

static int grow(void **ptr, size_t *have, size_t want) {
    if (*have >= want) return IMUNPACK_OK;
    if (*ptr) IMU_HIP(hipFree(*ptr));
    *ptr = nullptr;
    *have = 0;
    const size_t take = want + want / 4;
    if (hipMalloc(ptr, take) != hipSuccess) {
        (void)hipGetLastError();
        *ptr = nullptr;
        return IMUNPACK_ENOMEM;
    }
    *have = take;
    return IMUNPACK_OK;
}

// Gives all device memory of a context back.
static int release(imunpack_batch *c) {
    int rc = IMUNPACK_OK;
    if (c->plan) rc = imunpack_plan_destroy(c->plan);
    if (c->arena) (void)hipFree(c->arena);
    if (c->ue) (void)hipFree(c->ue);
    if (c->ws) (void)hipFree(c->ws);
    c->plan = nullptr;
    c->arena = nullptr;
    c->ue = nullptr;
    c->ws = nullptr;
    c->arena_bytes = c->ue_bytes = c->ws_bytes = 0;
    c->clean_flags = nullptr;
    return rc;
}

extern "C" int imunpack_batch_destroy(imunpack_batch_t *c) {
    if (!c) return IMUNPACK_OK;
    const int rc = release(c);
    if (c->pin_flags) (void)hipHostFree(c->pin_flags);
    delete c;
    return rc;
}

extern "C" int imunpack_gemm_batched(const float *A, int64_t sa_b, int64_t sa_r, int64_t sa_c,
                                     const float *B, int64_t sb_b, int64_t sb_r, int64_t sb_c,
                                     int64_t batch, int64_t n, int64_t d, int64_t h,
                                     double p, float beta_A, float beta_B, int b, int strategy_A, int strategy_B,
                                     float *C, int64_t sc_b, int64_t ldc, imunpack_batch_t **ctx,
                                     imunpack_stream_t stream) {
    if (!A || !B || !C || !ctx || batch < 0 || n <= 0 || d <= 0 || h <= 0 || ldc < h || sa_r < 1 || sa_c < 1 ||
        sb_r < 1 || sb_c < 1 || sa_b < 0 || sb_b < 0 || sc_b < 0 || b < 2 || b > 8 || strategy_A < 0 || strategy_A > 2 ||
        strategy_B < 0 || strategy_B > 2 || !(p > 0.0) || !(p <= 100.0) || !(beta_A > 0.0f) || !(beta_B > 0.0f))
        return IMUNPACK_EINVAL;
    if (n > (1 << 24) || d > (1 << 24) || h > (1 << 24) || n * d >= ((int64_t)1 << 32) || h * d >= ((int64_t)1 << 32))
        return IMUNPACK_EINVAL;
    if (batch == 0) return IMUNPACK_OK;
    hipStream_t st = (hipStream_t)stream;
    imunpack_batch_t *c = *ctx;
    if (!c) {
        c = new (std::nothrow) imunpack_batch();
        if (!c) return IMUNPACK_ENOMEM;
        memset(c, 0, sizeof(*c));
        if (hipHostMalloc((void **)&c->pin_flags, (2 + kMaxItems) * sizeof(int32_t), hipHostMallocCoherent) != hipSuccess) {
            (void)hipGetLastError();
            delete c;
            return IMUNPACK_ENOMEM;
        }
        memset(c->pin_flags, 0, (2 + kMaxItems) * sizeof(int32_t));
        *ctx = c;
    }
    // ---- what the shapes fix of an item: everything but its plan and its unpacked operands
    const int64_t capA = strategy_A == IMUNPACK_BOTH ? std::max<int64_t>(4096, n * d / 64) : 0;
    const int64_t capB = strategy_B == IMUNPACK_BOTH ? std::max<int64_t>(4096, h * d / 64) : 0;
    size_t off = 0;
    auto take = [&](size_t bytes) { const size_t at = off; off = (off + bytes + 255) & ~(size_t)255; return at; };
    const size_t oQa = take((size_t)n * d * 4), oQb = take((size_t)h * d * 4);
    const size_t oSa = take((size_t)2 * (n + d) * 4), oSb = take((size_t)2 * (h + d) * 4);
    const size_t oLa = take((size_t)3 * capA * 4), oLb = take((size_t)3 * capB * 4);
    const size_t oSmall = take(256);   // steps (2 floats), OB counts (2)
    const size_t oWs = take(2 * IMUNPACK_PERCENTILE_WORKSPACE_BYTES);
    const size_t item = off;
    const size_t head = (size_t)(1 + kMaxItems) * sizeof(int32_t) + 252;
    const size_t base = head & ~(size_t)255;
    // Items that go through together: all of them while their operands, their plans and what is unpacked from them (as much
    // as without a split row or column) stay small beside the memory of the GPU: a group of large products fills the chip by
    // itself.  (600 products of 1 x 65536 by 1 x 65536, some 50 MB each, nearly all of it plans and padding:
    // 37.8 GB and 19 ms when only operands were counted, 2.4 GB and 25 ms so; one at a time 0.07 GB and 554 ms.)
    auto padded = [](int64_t rows, int64_t cols) { return (rows + kTile - 1) / kTile * kTile * ((cols + kKPad - 1) / kKPad * kKPad); };
    const int64_t whole = (int64_t)item + plan_item_bytes(n, d, h, b, strategy_A, strategy_B) + padded(n, d) + padded(h, d);
    int64_t group = std::min<int64_t>(std::min<int64_t>(batch, kMaxItems), std::max<int64_t>(1, kGroupBytes / whole));
    // Items whose outputs lie on one another's outputs or operands (all but an output in the place of its own item's operand)
    // go one after the other: C_i may be A_(i+1).
    const int64_t ext_c = (n - 1) * ldc + h;
    auto crosses = [&](const float *X, int64_t rows, int64_t sr, int64_t sc, int64_t sb) {
        const int64_t ext = (rows - 1) * sr + (d - 1) * sc + 1;
        if (C + (batch - 1) * sc_b + ext_c <= X || X + (batch - 1) * sb + ext <= C) return false;
        return !(C == X && sc_b == sb && ext <= sb && ext_c <= sc_b);
    };
    const bool c_apart = sc_b >= ext_c || (sc_b >= h && ldc >= (batch - 1) * sc_b + h);  // side by side, or row by row in turn
    if (!c_apart || crosses(A, n, sa_r, sa_c, sa_b) || crosses(B, h, sb_r, sb_c, sb_b)) group = 1;
    group = (batch + (batch + group - 1) / group - 1) / ((batch + group - 1) / group);  // as many groups, of equal size

    auto run_group = [&](int64_t i0, int items, bool &bad) -> int {
        if (c->arena_bytes < base + item * (size_t)items) c->clean_flags = nullptr;  // new memory, whatever its address
        IMU_TRY(grow((void **)&c->arena, &c->arena_bytes, base + item * (size_t)items));
        int32_t *flags = (int32_t *)c->arena;
        if (c->clean_flags != flags) hipLaunchKernelGGL(clear_flags_kernel, dim3(1), dim3(256), 0, st, flags, 1 + kMaxItems);
        c->clean_flags = nullptr;
        char *first = c->arena + base;
        int32_t *Qa = (int32_t *)(first + oQa), *Qb = (int32_t *)(first + oQb);
        int32_t *sA = (int32_t *)(first + oSa), *sB = (int32_t *)(first + oSb);
        float *steps = (float *)(first + oSmall);
        int32_t *obcnt = (int32_t *)(first + oSmall) + 2;
        void *pws = first + oWs;
        imunpack_stats_t stA = {sA, sA + n, sA + n + d, sA + 2 * n + d, capA ? (int32_t *)(first + oLa) : nullptr, capA,
                                capA ? obcnt : nullptr};
        imunpack_stats_t stB = {sB, sB + h, sB + h + d, sB + 2 * h + d, capB ? (int32_t *)(first + oLb) : nullptr, capB,
                                capB ? obcnt + 1 : nullptr};
        const float *Ai = A + i0 * sa_b, *Bi = B + i0 * sb_b;
        float *Ci = C + i0 * sc_b;
        QuantBatch bt;
        bt.nitems = items;
        bt.a_stride = sa_b * 4; bt.b_stride = sb_b * 4;
        bt.out_stride = (int64_t)item;
        bt.flag = flags;
        // the steps stay on the device: percentile -> step -> division in the quantizer -> product in the epilogue
        IMU_TRY(rtn_step_pair(Ai, n, sa_r, sa_c, beta_A, Bi, h, sb_r, sb_c, beta_B, d, p, steps, pws, bt, st));
        IMU_TRY(quantize_pair(Ai, n, sa_r, sa_c, 1.0f, steps, Qa, d, &stA, Bi, h, sb_r, sb_c, 1.0f, steps + 1, Qb, d, &stB, d,
                              b, nullptr, bt, st));
        IMU_TRY(plan_impl(Qa, n, d, d, Qb, h, d, b, strategy_A, strategy_B, &stA, &stB, &c->plan, items, (int64_t)item, st));
        // digits of at most three bits: six-bit floating-point codes on the f8f6f4 matrix instruction (the
        // request stays with the context's plan object)
        if (b <= 4 && imunpack_plan_digits(c->plan) != IMUNPACK_DIGITS_FP6)
            IMU_TRY(imunpack_plan_set_digits(c->plan, IMUNPACK_DIGITS_FP6));
        size_t ba = 0, bb = 0;
        for (int i = 0; i < items; ++i) {
            const PlanHeader &hi = c->plan->pin_hdr[i];
            ba = std::max(ba, (size_t)hi.Mp * (size_t)header_pitch(hi, c->plan->fp6, 0));
            bb = std::max(bb, (size_t)hi.Np * (size_t)header_pitch(hi, c->plan->fp6, 1));
        }
        ba = (ba + 255) & ~(size_t)255;
        bb = (bb + 255) & ~(size_t)255;
        IMU_TRY(grow((void **)&c->ue, &c->ue_bytes, (ba + bb) * (size_t)items));
        int8_t *Aue = c->ue, *Beu = c->ue + ba * (size_t)items;
        IMU_TRY(unpack_impl(c->plan, Qa, d, Qb, d, Aue, (int64_t)ba, Beu, (int64_t)bb, st));
        IMU_TRY(gemm_batch(c->plan, Aue, (int64_t)ba, Beu, (int64_t)bb, Ci, sc_b * 4, ldc, steps, steps + 1, (int64_t)item,
                           flags + 1, st));
        ++c->seq;
        hipLaunchKernelGGL(tell_flags_kernel, dim3(1), dim3(256), 0, st, flags, 1 + items, c->pin_flags, c->pin_flags + 1 + kMaxItems, c->seq);
        IMU_TRY(launch_status());
        IMU_TRY(wait_word((const int32_t *)(c->pin_flags + 1 + kMaxItems), c->seq, st));
        bad = bad || c->pin_flags[0] != 0;
        bool unfused = false;
        for (int i = 0; i < items; ++i) {  // the fused launch is not exact for this item: un-fused path
            if (!c->pin_flags[1 + i]) continue;
            Plan view = item_view(*c->plan, i);
            view.fusable = 0;
            size_t bw = 0;
            IMU_TRY(imunpack_unpacked_bytes(&view, nullptr, nullptr, &bw));
            if (unfused) IMU_HIP(hipStreamSynchronize(st));  // the buffer may still be in use by an earlier item
            unfused = true;
            IMU_TRY(grow(&c->ws, &c->ws_bytes, bw));
            const float *step = (const float *)((const char *)steps + (size_t)i * item);
            IMU_TRY(gemm_impl(&view, Aue + (size_t)i * ba, Beu + (size_t)i * bb, c->ws, nullptr, Ci + i * sc_b, ldc, 1.0f, 1.0f, step,
                              step + 1, 1, st));
        }
        if (unfused) IMU_HIP(hipStreamSynchronize(st));
        c->clean_flags = flags;
        return IMUNPACK_OK;
    };
    bool bad = false;
    for (int64_t i0 = 0; i0 < batch;) {
        const int items = (int)std::min<int64_t>(group, batch - i0);
        const int rc = run_group(i0, items, bad);
        if (rc == IMUNPACK_ENOMEM && items > 1) {  // their plans or their unpacked operands grew too large: fewer at a time
            group = (items + 1) / 2;
            IMU_TRY(release(c));
            continue;
        }
        IMU_TRY(rc);
        i0 += items;
    }
    return bad ? IMUNPACK_ERANGE : IMUNPACK_OK;
}
