// Adaptive activation smoothing (Algorithm 1 step 1, Eq. 3): grid search of the exponent e
// of s = ax^e for one linear layer.  Every candidate goes through the library's own offline
// quantiser and its run-time W8A8 linear; what this file adds is the full-precision product
// the candidates are measured against, the loss reduction, and the search loop around them.
#include "f64_tile.h"

#include <cmath>
#include <limits>
#include <new>
#include <vector>

namespace haq {

namespace {

// ---- Yref = X W in binary64 ---------------------------------------------------------------
// One binary64 accumulator per output, k ascending, one fused multiply-add per term.  The
// product of a binary16 and a binary32 number is exact in binary64, so the FMA rounds exactly
// where "multiply, then add" would: the result does not depend on the tiling.
// Bound: the binary64 matrix pipe; 2048 x 4096 x 16384: 8.3 -> 5.1 ms (54 TFLOP/s).
__global__ __launch_bounds__(256, 5) void ref_gemm_f64_kernel(const __half* x, int64_t ldx, const float* w, int T, int K, int N, double* yref) {
    const int row0 = blockIdx.y * F64_B, col0 = blockIdx.x * F64_B;
    auto a = f64_operand<false>(x + row0 * ldx, ldx, T - row0, [](__half v) { return (double)h2f(v); });
    auto b = f64_operand<true>(w + col0, N, N - col0, F64Same{});
    __shared__ double lds[decltype(a)::LDS + decltype(b)::LDS];
    F64Acc acc = {};
    f64_tile_mac(acc, K, lds, a, b);
    f64_tile_each(acc, [&](double v, int i, int j) {
        if (row0 + i < T && col0 + j < N) yref[(size_t)(row0 + i) * N + col0 + j] = v;
    });
}

// ---- loss = mean (Y - Yref)^2 in binary64 ------------------------------------------------------
// Row sums run over the columns in order (one sequential chain per row, as the definition is written), so the value
// does not depend on the launch shape.  Bounds: the chain (N dependent additions) and, from one row per two lanes of
// every CU on, the read of Yref.  A work-group owns LR rows and walks over tiles of 256 columns: its first wave does
// nothing but add (lane r the values of row r, from LDS), the other four fetch two tiles ahead and leave the squared
// differences in one of two LDS buffers (2048 x 16384: 600 -> 92 us; one wave both fetched and added before).  A last
// small kernel adds the rows in order.
constexpr int LR = 8, LC = 256;
__global__ __launch_bounds__(64 + LC) void row_sq_err_kernel(const __half* y, int64_t ldy, const double* yref, int T, int N,
                                                             double* row_sum) {
    __shared__ __attribute__((aligned(16))) double sq[2][LR][LC + 2];
    const int lane = threadIdx.x, col = threadIdx.x - 64;
    const bool adds = threadIdx.x < 64;
    const int row0 = blockIdx.x * LR;
    const int ntile = (N + LC - 1) / LC;
    struct Tile {
        __half y[LR];
        double r[LR];
    };
    auto fetch = [&](int tile, Tile& f) {  // thread = one column, all rows; loads stay unconditional (clamped), masked afterwards
        const int c = min(tile * LC + col, N - 1);
#pragma unroll
        for (int r = 0; r < LR; ++r) {
            const int row = min(row0 + r, T - 1);
            f.y[r] = y[(size_t)row * ldy + c];
            f.r[r] = __builtin_nontemporal_load(yref + (size_t)row * N + c);
        }
    };
    auto stage = [&](int tile, const Tile& f) {
#pragma unroll
        for (int r = 0; r < LR; ++r) {
            const double d = (double)h2f(f.y[r]) - f.r[r];
            sq[tile & 1][r][col] = row0 + r < T && tile * LC + col < N ? d * d : 0.0;
        }
    };
    double run = 0.0;
    auto add = [&](int tile) {
        if (lane < LR) run = add_in_order(run, sq[tile & 1][lane], min(LC, N - tile * LC));
    };
    Tile f0, f1;
    if (!adds) {
        fetch(0, f0);
        if (ntile > 1) fetch(1, f1);
        stage(0, f0);
        if (ntile > 2) fetch(2, f0);
    }
    __syncthreads();
    for (int tile = 0; tile < ntile; tile += 2) {
        if (adds) {
            add(tile);
        } else if (tile + 1 < ntile) {
            stage(tile + 1, f1);
            if (tile + 3 < ntile) fetch(tile + 3, f1);
        }
        __syncthreads();
        if (tile + 1 >= ntile) break;
        if (adds) {
            add(tile + 1);
        } else if (tile + 2 < ntile) {
            stage(tile + 2, f0);
            if (tile + 4 < ntile) fetch(tile + 4, f0);
        }
        __syncthreads();
    }
    if (lane < LR && row0 + lane < T) row_sum[row0 + lane] = run;
}

__global__ __launch_bounds__(256) void total_loss_kernel(const double* row_sum, int T, int N, double* loss) {
    __shared__ double part[1024];
    double total = 0.0;
    for (int t0 = 0; t0 < T; t0 += 1024) {  // rows in order, 1024 at a time through LDS
        for (int i = threadIdx.x; i < 1024; i += 256) part[i] = t0 + i < T ? row_sum[t0 + i] : 0.0;
        __syncthreads();
        if (threadIdx.x == 0) total = add_in_order(total, part, min(1024, T - t0));
        __syncthreads();
    }
    if (threadIdx.x == 0) *loss = total / ((double)T * (double)N);
}

struct SearchWs {
    float *ax, *aw, *s_all, *sw;
    double *yref, *row_sum, *losses;
    int8_t *wq, *packed;
    __half* y;
    void* lin;
    size_t lin_bytes, bytes;
};

SearchWs carve_search(void* ws, int T, int K, int N, int n_e) {
    uint8_t* base = (uint8_t*)ws;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        void* p = base ? base + off : nullptr;
        off += (size_t)round_up((int64_t)bytes, 256);
        return p;
    };
    SearchWs w;
    w.ax = (float*)take((size_t)K * 4);
    w.aw = (float*)take((size_t)K * 4);
    w.s_all = (float*)take((size_t)n_e * K * 4);
    w.sw = (float*)take((size_t)N * 4);
    w.yref = (double*)take((size_t)T * N * 8);
    w.row_sum = (double*)take((size_t)T * 8);
    w.losses = (double*)take((size_t)n_e * 8);
    w.wq = (int8_t*)take((size_t)K * N);
    w.packed = (int8_t*)take(haq_packed_bytes(K, N));
    w.y = (__half*)take((size_t)T * N * 2);
    w.lin_bytes = haq_linear_workspace_bytes(T, K, N);
    w.lin = take(w.lin_bytes);
    w.bytes = off;
    return w;
}

}  // namespace

}  // namespace haq

using namespace haq;

extern "C" {

size_t haq_smoothing_search_workspace_bytes(int32_t T, int32_t K, int32_t N, int32_t n_e) {
    if (T <= 0 || K <= 0 || N <= 0 || n_e <= 0) return 0;
    return carve_search(nullptr, T, K, N, n_e).bytes;
}

int32_t haq_reference_matmul_f64(const void* x_fp16, int64_t ldx, const float* w, int32_t T, int32_t K, int32_t N,
                                 double* yref, void* stream) {
    if (T <= 0 || K <= 0 || N <= 0) HAQ_FAIL(HAQ_ERR_INVALID_ARG, "haq_reference_matmul_f64: T=%d K=%d N=%d", T, K, N);
    if (!x_fp16 || !w || !yref || ldx < K) HAQ_FAIL(HAQ_ERR_INVALID_ARG, "haq_reference_matmul_f64: null buffer or ldx=%lld", (long long)ldx);
    hipLaunchKernelGGL(ref_gemm_f64_kernel, dim3(cdiv(N, 64), cdiv(T, 64)), dim3(256), 0, (hipStream_t)stream,
                           (const __half*)x_fp16, ldx, w, T, K, N, yref);
    HAQ_CHECK_HIP(hipGetLastError());
    return HAQ_OK;
}

int32_t haq_quant_loss_f64(const void* y_fp16, int64_t ldy, const double* yref, int32_t T, int32_t N, double* row_scratch,
                           double* loss, void* stream) {
    if (T <= 0 || N <= 0) HAQ_FAIL(HAQ_ERR_INVALID_ARG, "haq_quant_loss_f64: T=%d N=%d", T, N);
    if (!y_fp16 || !yref || !row_scratch || !loss || ldy < N) HAQ_FAIL(HAQ_ERR_INVALID_ARG, "haq_quant_loss_f64: null buffer or ldy=%lld", (long long)ldy);
    hipStream_t st = (hipStream_t)stream;
    hipLaunchKernelGGL(row_sq_err_kernel, dim3(cdiv(T, LR)), dim3(64 + LC), 0, st, (const __half*)y_fp16, ldy, yref, T, N, row_scratch);
    hipLaunchKernelGGL(total_loss_kernel, dim3(1), dim3(256), 0, st, (const double*)row_scratch, T, N, loss);
    HAQ_CHECK_HIP(hipGetLastError());
    return HAQ_OK;
}

int32_t haq_smoothing_search(const void* x_fp16, int64_t ldx, const float* w, int32_t T, int32_t K, int32_t N,
                             const double* exponents, int32_t n_e, int32_t use_weight, double* losses, int32_t* best,
                             float* s_best, void* workspace, size_t workspace_bytes, void* stream) {
    if (T <= 0 || K <= 0 || N <= 0) HAQ_FAIL(HAQ_ERR_INVALID_ARG, "haq_smoothing_search: T=%d K=%d N=%d", T, K, N);
    if (K % 64 != 0 || K > 65535 || N % 16 != 0)
        HAQ_FAIL(HAQ_ERR_UNSUPPORTED, "haq_smoothing_search: K=%d must be a multiple of 64 (< 65536), N=%d of 16", K, N);
    if (n_e <= 0 || n_e > 256 || !exponents) HAQ_FAIL(HAQ_ERR_INVALID_ARG, "haq_smoothing_search: n_e=%d outside [1, 256] or no grid", n_e);
    for (int i = 0; i < n_e; ++i)
        if (!(exponents[i] >= 0.0 && exponents[i] <= 1.0))
            HAQ_FAIL(HAQ_ERR_INVALID_ARG, "haq_smoothing_search: exponent %d = %g outside [0, 1]", i, exponents[i]);
    if (!x_fp16 || !w || !losses || !best || !s_best) HAQ_FAIL(HAQ_ERR_INVALID_ARG, "haq_smoothing_search: null buffer");
    if (ldx < K || ldx % 8 != 0 || !aligned16(x_fp16) || !aligned16(s_best))
        HAQ_FAIL(HAQ_ERR_INVALID_ARG, "haq_smoothing_search: ldx=%lld (>= K, multiple of 8), 16-byte aligned x and s_best", (long long)ldx);
    const size_t need = carve_search(nullptr, T, K, N, n_e).bytes;
    if (!workspace || workspace_bytes < need || ((uintptr_t)workspace & 255u))
        HAQ_FAIL(HAQ_ERR_WORKSPACE, "haq_smoothing_search: workspace of %zu bytes (256-byte aligned) needed, got %zu", need, workspace_bytes);
    hipStream_t st = (hipStream_t)stream;
    SearchWs ws = carve_search(workspace, T, K, N, n_e);
    int rc;

    // channel magnitudes of the calibration activations (and of the weight rows), to the host
    HAQ_CHECK_HIP(hipMemsetAsync(ws.ax, 0, (size_t)K * 4, st));
    HAQ_CHECK_HIP(hipMemsetAsync(ws.aw, 0, (size_t)K * 4, st));
    if ((rc = haq_channel_absmax_f16(x_fp16, ldx, T, K, ws.ax, stream)) != HAQ_OK) return rc;
    if (use_weight && (rc = haq_weight_row_absmax(w, K, N, ws.aw, stream)) != HAQ_OK) return rc;
    std::vector<float> ax, aw, s_all;  // host staging; no asynchronous copy outlives this function
    try {
        ax.resize((size_t)K);
        aw.resize((size_t)K);
        s_all.resize((size_t)n_e * K);
    } catch (const std::bad_alloc&) {
        HAQ_FAIL(HAQ_ERR_HIP, "haq_smoothing_search: out of host memory");
    }
    HAQ_CHECK_HIP(hipMemcpyAsync(ax.data(), ws.ax, (size_t)K * 4, hipMemcpyDeviceToHost, st));
    HAQ_CHECK_HIP(hipMemcpyAsync(aw.data(), ws.aw, (size_t)K * 4, hipMemcpyDeviceToHost, st));
    HAQ_CHECK_HIP(hipStreamSynchronize(st));
    for (int i = 0; i < n_e; ++i)
        if ((rc = haq_smoothing_vector(ax.data(), use_weight ? aw.data() : nullptr, K, exponents[i], s_all.data() + (size_t)i * K)) != HAQ_OK)
            return rc;
    HAQ_CHECK_HIP(hipMemcpyAsync(ws.s_all, s_all.data(), s_all.size() * 4, hipMemcpyHostToDevice, st));
    HAQ_CHECK_HIP(hipStreamSynchronize(st));  // s_all is pageable host memory: the copy has landed before any return below

    if ((rc = haq_reference_matmul_f64(x_fp16, ldx, w, T, K, N, ws.yref, stream)) != HAQ_OK) return rc;
    // The column maxima of WEIGHT_NC candidates at a time, in the memory of the unpacked codes (K N bytes, K >= 4 WEIGHT_NC),
    // which this path does not need: the codes go straight into the packed layout.
    float* colmax = (float*)ws.wq;
    static_assert(4 * WEIGHT_NC <= 64, "K is a multiple of 64");
    for (int i = 0; i < n_e; ++i) {
        const float* s = ws.s_all + (size_t)i * K;
        if (i % WEIGHT_NC == 0 && (rc = launch_weight_colmax(w, s, n_e - i < WEIGHT_NC ? n_e - i : WEIGHT_NC, K, N, colmax, st)) != HAQ_OK) return rc;
        if ((rc = launch_weight_pack(w, s, K, N, colmax + (size_t)(i % WEIGHT_NC) * N, ws.packed, ws.sw, st)) != HAQ_OK) return rc;
        if ((rc = haq_w8a8_linear(x_fp16, ldx, s, ws.packed, ws.sw, T, K, N, HAQ_ACT_NONE, ws.y, N, nullptr, nullptr, nullptr,
                                  ws.lin, ws.lin_bytes, stream)) != HAQ_OK)
            return rc;
        if ((rc = haq_quant_loss_f64(ws.y, N, ws.yref, T, N, ws.row_sum, ws.losses + i, stream)) != HAQ_OK) return rc;
    }
    HAQ_CHECK_HIP(hipMemcpyAsync(losses, ws.losses, (size_t)n_e * 8, hipMemcpyDeviceToHost, st));
    HAQ_CHECK_HIP(hipStreamSynchronize(st));

    // a candidate replaces the incumbent only if its loss is strictly smaller
    int b = -1;
    double best_loss = std::numeric_limits<double>::infinity();
    for (int i = 0; i < n_e; ++i) {
        if (losses[i] < best_loss) {
            best_loss = losses[i];
            b = i;
        }
    }
    if (b < 0) HAQ_FAIL(HAQ_ERR_INVALID_ARG, "haq_smoothing_search: no candidate has a finite loss");
    *best = b;
    HAQ_CHECK_HIP(hipMemcpyAsync(s_best, ws.s_all + (size_t)b * K, (size_t)K * 4, hipMemcpyDeviceToDevice, st));
    HAQ_CHECK_HIP(hipStreamSynchronize(st));
    return HAQ_OK;
}

}  // extern "C"
