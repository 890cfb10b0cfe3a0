// Hessian-aware weight quantisation (Section III.B.2, Eq. 4-6; Algorithm 1 step 2), offline.
//
// Everything is binary64 and every accumulation is a chain of fused multiply-adds in a stated
// order (tokens ascending for the Hessian, eliminated columns ascending for the factorisation,
// quantised input channels ascending for the compensation).  Blocking only regroups which
// work-item applies a link of a chain and when; it never reorders a chain, so the bits do not
// depend on the tile sizes below.
//
//   H  = 2 Xs^T Xs + damping                       hessian_kernel, hessian_finish_kernel
//   A  = flip(H) = L L^T                           chol_panel_kernel, chol_trail_kernel
//   M  = L^-1 (lower)                              tri_inverse_block_kernel
//   U  = flip(M): upper, H^-1 = U^T U              flip_kernel
//   channels i ascending: code, error, compensate  gptq_block_kernel, gptq_update_kernel
#include <type_traits>

#include "f64_tile.h"

namespace haq {

namespace {

constexpr int PB = 64;    // Cholesky panel width, rows per block of the triangular inverse
constexpr int GB = 64;    // input channels quantised per compensation block
constexpr int GS = 256;   // input channels per rank-GS compensation of everything below them

// A lane's 64 values v against a triangular block that all lanes share: for c ascending e = f(c, v_c), then
// v_l -= e C(c, l) for l > c, with skew[c][p] = C(c, c + 1 + p).  The current value is always v[0]: the array moves down
// by one with each column (the multiply-add's destination is its neighbour's register), so that the columns are a
// loop of short code; what moves in from beyond value 63 is never used.  Written out as 64 different columns the loop
// is longer than the instruction cache, and the compiler spills vector registers.  (Scalar registers, the addresses of
// 64 rows, spill into vector lanes in the callers' prologues and in chol_panel_kernel's turns; not in these loops.)
// One wave runs alone on its SIMD: the coefficients come out of LDS in chunks of eight, three chunks ahead of their use
// (the asm keeps reads and values with their chunk: left alone, the compiler fetches everything first and spills).
template <class F>
__device__ __forceinline__ void eliminate_columns(double (&v)[64], const double (*skew)[64], F&& f) {
    typedef double v2d __attribute__((ext_vector_type(2)));
    auto sixteen = [&](auto width, int c0) __attribute__((always_inline)) {
        constexpr int W = width.value, NCH = W / 8, RING = 4;
        v2d ring[RING][4];
        auto fetch = [&](int c, int n) __attribute__((always_inline)) {  // chunk n from column c on
            const v2d* row = reinterpret_cast<const v2d*>(skew[min(c + n / NCH, 63)] + 8 * (n % NCH));
#pragma unroll
            for (int i = 0; i < 4; ++i) ring[n % RING][i] = row[i];
        };
#pragma unroll
        for (int n = 0; n < RING - 1; ++n) fetch(c0, n);
#pragma nounroll
        for (int c = c0; c < c0 + 16; c += 2) {
            double e = 0.0;
#pragma unroll
            for (int n = 0; n < 2 * NCH; ++n) {  // 2 NCH is a multiple of RING: the ring's indices are constants
                fetch(c, n + RING - 1);
                if (n % NCH == 0) e = f(c + n / NCH, v[0]);
                double* u = v + 8 * (n % NCH);
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    if (8 * (n % NCH) + i + 1 < W) u[i] = __builtin_fma(-e, ring[n % RING][i / 2][i % 2], u[i + 1]);
                asm volatile("" : "+v"(u[0]), "+v"(u[1]), "+v"(u[2]), "+v"(u[3]), "+v"(u[4]), "+v"(u[5]), "+v"(u[6]), "+v"(u[7])::"memory");
            }
        }
    };
    sixteen(std::integral_constant<int, 64>{}, 0);
    sixteen(std::integral_constant<int, 48>{}, 16);
    sixteen(std::integral_constant<int, 32>{}, 32);
    sixteen(std::integral_constant<int, 16>{}, 48);
}
// diag[c], which is the same for the whole wave, from the lane that holds it
__device__ __forceinline__ double from_lane(double v, int c) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), c), __builtin_amdgcn_readlane(__double2loint(v), c));
}

// ---- H = 2 Xs^T Xs -------------------------------------------------------------------------------
// Tiles on and below the diagonal; the product is symmetric to the bit (the factors of a multiply-add commute), so the
// other half is written from the same values.  4096 channels, 2048 tokens: 3.7 -> 1.2 ms.
struct Smoothed {  // x / s, as the layer sees it
    float s;
    __device__ double operator()(__half x) const { return (double)(h2f(x) / s); }
};
__global__ __launch_bounds__(256, 5) void hessian_kernel(const __half* x, int64_t ldx, const float* s, int T, int K, double* H) {
    const int j0 = blockIdx.y * F64_B, l0 = blockIdx.x * F64_B;
    if (l0 > j0) return;
    auto operand = [&](int c0) {
        const int c = min(c0 + (int)threadIdx.x % F64_B, K - 1);  // the one channel that a thread fetches
        return f64_operand<true>(x + c0, ldx, K - c0, Smoothed{s ? s[c] : 1.0f});
    };
    auto a = operand(j0), b = operand(l0);
    __shared__ double lds[decltype(a)::LDS + decltype(b)::LDS];
    F64Acc acc = {};
    f64_tile_mac(acc, T, lds, a, b);
    f64_tile_each(acc, [&](double v, int i, int jj) {
        const int j = j0 + i, l = l0 + jj;
        if (j >= K || l >= K) return;
        H[(size_t)j * K + l] = 2.0 * v;
        if (l0 != j0) H[(size_t)l * K + j] = 2.0 * v;
    });
}

// Dead channels get a unit diagonal; damping = percdamp * mean(diag), the diagonal summed in index order.
__global__ __launch_bounds__(256) void hessian_finish_kernel(double* H, int K, double percdamp) {
    __shared__ double part[1024];
    __shared__ double damp_s;
    double tr = 0.0;
    for (int j0 = 0; j0 < K; j0 += 1024) {
        for (int i = threadIdx.x; i < 1024; i += 256) {
            const int j = j0 + i;
            double d = 0.0;
            if (j < K) {
                d = H[(size_t)j * K + j];
                if (d == 0.0) {
                    d = 1.0;
                    H[(size_t)j * K + j] = 1.0;
                }
            }
            part[i] = d;
        }
        __syncthreads();
        if (threadIdx.x == 0) tr = add_in_order(tr, part, min(1024, K - j0));
        __syncthreads();
    }
    if (threadIdx.x == 0) damp_s = percdamp * (tr / (double)K);
    __syncthreads();
    const double damp = damp_s;
    for (int j = threadIdx.x; j < K; j += 256) H[(size_t)j * K + j] += damp;
}

// A(i, j) = H(K-1-i, K-1-j); also used to turn M into U.
__global__ void flip_kernel(const double* src, int K, double* dst) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x, i = blockIdx.y;
    if (j < K) dst[(size_t)i * K + j] = src[(size_t)(K - 1 - i) * K + (K - 1 - j)];
}

// ---- Cholesky, right-looking in panels of PB columns ------------------------------------------
// Bound: the serial chain of the panels (64 at K = 4096, 52 us each; the trailing update takes 18).
// Panel kernel: every work-group first factorises the PB x PB diagonal block (redundantly: it is one serial chain of
// PB columns, each a square root, a division and an exchange), then its first wave solves 64 rows below the block
// against it, a row per lane: x_c = v_c / L_cc; v_l -= x_c L_lc for the later columns l.  An element's links are thus
// applied for ascending c, whatever the panel width.
// The factorisation: row = lane; wave w holds columns w, w + 4, ...; the owner of a column passes it on through LDS and
// every wave divides it for itself, so that a column costs one barrier.
// Work-group 0 leaves the factorised diagonal block in `dblock` (it cannot go to A here: the other
// work-groups may still be reading the unfactorised block); the next launch moves it.
// status: first non-positive pivot + 1.
__global__ __launch_bounds__(256, 1) void chol_panel_kernel(double* A, int K, int j0, double* dblock, int* status) {
    __shared__ __attribute__((aligned(16))) double Ds[PB][PB];  // skewed: Ds[c][p] = L(c + 1 + p, c)
    __shared__ double diag[PB];
    __shared__ double col[2][PB];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int pb = min(PB, K - j0);
    double own[PB / 4];  // past the last column: the identity
#pragma unroll
    for (int m = 0; m < PB / 4; ++m) {
        const int c = 4 * m + wave;
        own[m] = A[(size_t)(j0 + min(lane, pb - 1)) * K + j0 + min(c, pb - 1)];  // loads stay unconditional: a branch each would be a wait each
    }
    const int i = j0 + pb + blockIdx.x * 64 + lane;  // row below the block (wave 0)
    double v[PB];
    if (wave == 0) {
#pragma unroll
        for (int c = 0; c < PB; ++c) v[c] = A[(size_t)(i < K ? i : j0) * K + j0 + min(c, pb - 1)];  // a row below has a full panel before it
    }
#pragma unroll
    for (int m = 0; m < PB / 4; ++m) {
        const int c = 4 * m + wave;
        own[m] = lane < pb && c <= lane ? own[m] : lane == c ? 1.0 : 0.0;
    }
    // Four columns a turn; own[0] holds the turn's columns and the array moves down by one after it.  Only the next
    // column waits for this one: the others take this column's link while the next one's root and quotient are formed.
    double l = 0.0;  // the column before the current one
    auto turns = [&](auto width, int t0, int t1) __attribute__((always_inline)) {
        constexpr int W = width.value;
        auto link = [&](int o, double v) __attribute__((always_inline)) {  // v less the link of column o with the last one; past column 63: never used
            return __builtin_fma(-l, from_lane(l, o & 63), v);
        };
#pragma nounroll
        for (int t = t0; t < t1; ++t) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int c = 4 * t + q;
                if (wave == q) col[q & 1][lane] = own[0];
                __syncthreads();
                const double d = col[q & 1][c], vc = col[q & 1][lane];
                // what the column before still owes: all but the slot that holds column c
#pragma unroll
                for (int m = 1; m < W; ++m) own[m] = link(4 * (t + m) + wave, own[m]);
                if (!(d > 0.0) && blockIdx.x == 0 && threadIdx.x == 0) atomicCAS(status, 0, j0 + c + 1);
                const double p = sqrt(d);
                l = lane == c ? p : vc / p;
                if (wave == 0) {
                    if (lane == c) diag[c] = p;
                    if (lane > c) Ds[c][lane - c - 1] = l;
                }
                if (q < 3) {
                    own[0] = wave > q ? link(4 * t + wave, own[0]) : own[0];
                } else {
                    // the next turn's columns get this link at once, the later ones (which move down) in its first column
                    own[1] = link(4 * (t + 1) + wave, own[1]);
                }
            }
#pragma unroll
            for (int m = 0; m + 1 < W; ++m) own[m] = own[m + 1];
        }
    };
    turns(std::integral_constant<int, 16>{}, 0, 8);
    turns(std::integral_constant<int, 8>{}, 8, 16);
    __syncthreads();
    if (wave != 0) return;
    if (blockIdx.x == 0) {
        for (int e = lane; e < pb * pb; e += 64) {
            const int c = e / pb, r = e % pb;
            dblock[e] = r == c ? diag[c] : r > c ? Ds[c][r - c - 1] : 0.0;
        }
    }
    if (j0 + pb >= K) return;
    double* out = A + (size_t)i * K + j0;
    const double my_diag = diag[lane];
    eliminate_columns(v, Ds, [&](int c, double vc) {
        const double xc = vc / from_lane(my_diag, c);
        if (i < K) out[c] = xc;
        return xc;
    });
}

__device__ __forceinline__ void chol_store_diag(double* A, int K, int j0, const double* dblock) {
    const int pb = min(PB, K - j0);
    for (int e = threadIdx.x; e < pb * pb; e += 256) {
        const int c = e / pb, r = e % pb;
        if (c <= r) A[(size_t)(j0 + r) * K + j0 + c] = dblock[e];
    }
}

__global__ __launch_bounds__(256) void chol_store_diag_kernel(double* A, int K, int j0, const double* dblock) { chol_store_diag(A, K, j0, dblock); }

// Trailing update after a panel: for i >= l >= j0 + PB: A_il -= L_ik L_lk, k over the panel ascending.
// Tiles that touch the lower triangle; tile (0, 0) also moves the factorised diagonal block into A.
__global__ __launch_bounds__(256, 5) void chol_trail_kernel(double* A, int K, int j0, const double* dblock) {
    if (blockIdx.x > blockIdx.y) return;
    if (blockIdx.x == 0 && blockIdx.y == 0) chol_store_diag(A, K, j0, dblock);
    const int i0 = j0 + PB + blockIdx.y * F64_B, l0 = j0 + PB + blockIdx.x * F64_B;
    auto a = f64_operand<false>(A + (size_t)i0 * K + j0, K, K - i0, F64Minus{});
    auto b = f64_operand<false>(A + (size_t)l0 * K + j0, K, K - l0, F64Same{});
    __shared__ double lds[decltype(a)::LDS + decltype(b)::LDS];
    F64Acc acc;
    f64_tile_each(acc, [&](double& v, int i, int l) { v = i0 + i < K && l0 + l < K ? A[(size_t)(i0 + i) * K + l0 + l] : 0.0; });
    f64_tile_mac(acc, PB, lds, a, b);
    f64_tile_each(acc, [&](double v, int i, int l) {
        if (i0 + i < K && l0 + l <= i0 + i) A[(size_t)(i0 + i) * K + l0 + l] = v;
    });
}

// ---- M = L^-1, blocks of PB rows ---------------------------------------------------------------
// M_jj = 1 / L_jj; M_ij = -(sum_{j <= k < i} L_ik M_kj) / L_ii, the sum a chain over k ascending, which grows in M
// itself: once a block of rows is final, its links are added to every row below (a rank-PB product), so a block finds
// its chains complete up to its own first row.  M must be zero on entry.  (The left-looking form, all links of 32 rows
// in one launch, kept 64 work-groups busy with chains of up to K links: 40 ms at K = 4096.)
// A link with M_kj = 0 (k < j) leaves the chain as it is: it starts from +0 and never holds -0.
__global__ __launch_bounds__(64, 1) void tri_inverse_block_kernel(const double* L, int K, int i0, double* M) {
    __shared__ __attribute__((aligned(16))) double Ls[PB][PB];  // the diagonal block, skewed: Ls[c][p] = L(c + 1 + p, c); past the last row: the identity
    __shared__ double diag[PB];
    const int lane = threadIdx.x, j = blockIdx.x * 64 + lane;
    const int rows = min(PB, K - i0);
    double v[PB];
#pragma unroll
    for (int r = 0; r < PB; ++r) v[r] = L[(size_t)(i0 + min(r, rows - 1)) * K + i0 + min(lane, rows - 1)];  // loads stay unconditional
#pragma unroll
    for (int r = 0; r < PB; ++r) {
        const double l = r < rows && lane <= r ? v[r] : lane == r ? 1.0 : 0.0;
        double* to = lane == r ? &diag[r] : lane < r ? &Ls[lane][r - lane - 1] : &Ls[lane][PB - 1];  // (an element that is not used)
        *to = l;
    }
#pragma unroll
    for (int r = 0; r < PB; ++r) v[r] = M[(size_t)(i0 + min(r, rows - 1)) * K + min(j, K - 1)];
#pragma unroll
    for (int r = 0; r < PB; ++r) v[r] = r < rows && j < i0 + rows ? (i0 + r == j ? 1.0 : v[r]) : 0.0;
    __syncthreads();
    double* out = M + (size_t)i0 * K + j;
    const double my_diag = diag[lane];
    eliminate_columns(v, Ls, [&](int c, double vc) {
        const double m = vc / from_lane(my_diag, c);
        if (c < rows && j < i0 + rows) out[(size_t)c * K] = m;
        return m;
    });
}

// M_ij -= L_ik M_kj for the rows i below the block [i0, i0 + PB), k over the block ascending, j < i0 + PB.
__global__ __launch_bounds__(256) void tri_inverse_update_kernel(const double* L, int K, int i0, double* M) {
    const int r0 = i0 + PB + blockIdx.y * F64_B, c0 = blockIdx.x * F64_B, cols = i0 + PB;
    auto a = f64_operand<false>(L + (size_t)r0 * K + i0, K, K - r0, F64Minus{});
    auto b = f64_operand<true>((const double*)M + (size_t)i0 * K + c0, K, cols - c0, F64Same{});
    __shared__ double lds[decltype(a)::LDS + decltype(b)::LDS];
    F64Acc acc;
    f64_tile_each(acc, [&](double& v, int i, int j) { v = r0 + i < K && c0 + j < cols ? M[(size_t)(r0 + i) * K + c0 + j] : 0.0; });
    f64_tile_mac(acc, PB, lds, a, b);
    f64_tile_each(acc, [&](double v, int i, int j) {
        if (r0 + i < K && c0 + j < cols) M[(size_t)(r0 + i) * K + c0 + j] = v;
    });
}

// ---- the quantise-and-compensate sweep ------------------------------------------------------------
__global__ void fold_weight_kernel(const float* w, const float* s, int K, int N, double* w64) {
    const int n = blockIdx.x * blockDim.x + threadIdx.x, k = blockIdx.y;
    if (n < N) w64[(size_t)k * N + n] = (double)((s ? s[k] : 1.0f) * w[(size_t)k * N + n]);
}

// Channels b0 .. b0 + GB - 1, one thread per output channel n: code, error, compensation of the
// block's later channels; the errors go to err [GB x N] for the rows below the block.
__global__ __launch_bounds__(64, 1) void gptq_block_kernel(double* w64, const double* U, const float* scale, int K, int N, int b0,
                                                           int8_t* wq, double* err) {
    __shared__ __attribute__((aligned(16))) double Us[GB][GB];  // skewed: Us[i][p] = U(i, i + 1 + p); past the block's channels: 0
    __shared__ double diag[GB];
    const int lane = threadIdx.x, n = blockIdx.x * 64 + lane, nc = min(n, N - 1);
    const int gb = min(GB, K - b0);
    double w[GB];
#pragma unroll
    for (int r = 0; r < GB; ++r) w[r] = U[(size_t)(b0 + min(r, gb - 1)) * K + b0 + min(lane, gb - 1)];  // loads stay unconditional
#pragma unroll
    for (int r = 0; r < GB; ++r) {
        const double u = r < gb && lane < gb && lane >= r ? w[r] : lane == r ? 1.0 : 0.0;
        double* to = lane == r ? &diag[r] : lane > r ? &Us[r][lane - r - 1] : &Us[r][GB - 1 - lane];  // (an element that is not used)
        *to = u;
    }
#pragma unroll
    for (int i = 0; i < GB; ++i) w[i] = w64[(size_t)(b0 + min(i, gb - 1)) * N + nc];
    __syncthreads();
    const float sc_f = scale[nc];
    const double sc = (double)sc_f;
    const double my_diag = diag[lane];
    eliminate_columns(w, Us, [&](int i, double wi) {
        double code = 0.0;
        if (sc_f != 0.0f) {
            code = __builtin_rint(wi / sc);
            code = fmin(fmax(code, -127.0), 127.0);
        }
        const double e = (wi - code * sc) / from_lane(my_diag, i);
        if (i < gb && n < N) {
            wq[(size_t)(b0 + i) * N + n] = (int8_t)code;
            err[(size_t)i * N + n] = e;
        }
        return e;
    });
}

// Rows [r_lo, r_hi): w_jn -= err_in U_ij for the n_i channels from i0 on, ascending.  Applied after every 64 channels to
// the rest of a stretch of 256 and after the stretch to everything below: w is read and written once per stretch there
// (34 GB -> 9 GB in all at 4096 x 16384, which took 25 ms; now 6.3, 44 TFLOP/s of the matrix pipe's 55).
__global__ __launch_bounds__(256, 5) void gptq_update_kernel(double* w64, const double* U, const double* err, int K, int N, int i0, int n_i,
                                                          int r_lo, int r_hi) {
    const int r0 = r_lo + blockIdx.y * F64_B, n0 = blockIdx.x * F64_B;
    auto a = f64_operand<true>(U + (size_t)i0 * K + r0, K, r_hi - r0, F64Minus{});
    auto b = f64_operand<true>(err + n0, N, N - n0, F64Same{});
    __shared__ double lds[decltype(a)::LDS + decltype(b)::LDS];
    F64Acc acc;
    f64_tile_each(acc, [&](double& v, int j, int n) { v = r0 + j < r_hi && n0 + n < N ? w64[(size_t)(r0 + j) * N + n0 + n] : 0.0; });
    f64_tile_mac(acc, n_i, lds, a, b);
    f64_tile_each(acc, [&](double v, int j, int n) {
        if (r0 + j < r_hi && n0 + n < N) w64[(size_t)(r0 + j) * N + n0 + n] = v;
    });
}

constexpr size_t STATUS_BYTES = 64 + 8192;  // the status word; the rest keeps the workspace sizes that callers have stored

struct HessWs {
    double *H, *A, *M, *w64, *err;
    int* status;
    size_t bytes;
};

HessWs carve_hess(void* ws, int K, int N) {
    uint8_t* base = (uint8_t*)ws;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        void* p = base ? base + off : nullptr;
        off += (size_t)round_up((int64_t)bytes, 256);
        return p;
    };
    HessWs w;
    w.H = (double*)take((size_t)K * K * 8);
    w.A = (double*)take((size_t)K * K * 8);
    w.M = (double*)take((size_t)K * K * 8);
    w.w64 = (double*)take((size_t)K * N * 8);
    w.err = (double*)take((size_t)GB * N * 8);
    w.status = (int*)take(STATUS_BYTES);
    w.bytes = off;
    return w;
}

}  // namespace

}  // namespace haq

using namespace haq;

extern "C" {

int32_t haq_hessian_f64(const void* x_fp16, int64_t ldx, const float* s, int32_t T, int32_t K, double percdamp, double* H,
                        void* stream) {
    if (T <= 0 || K <= 0 || !(percdamp >= 0.0)) HAQ_FAIL(HAQ_ERR_INVALID_ARG, "haq_hessian_f64: T=%d K=%d percdamp=%g", T, K, percdamp);
    if (!x_fp16 || !H || ldx < K) HAQ_FAIL(HAQ_ERR_INVALID_ARG, "haq_hessian_f64: null buffer or ldx=%lld", (long long)ldx);
    hipStream_t st = (hipStream_t)stream;
    hipLaunchKernelGGL(hessian_kernel, dim3(cdiv(K, 64), cdiv(K, 64)), dim3(256), 0, st, (const __half*)x_fp16, ldx, s, T, K, H);
    hipLaunchKernelGGL(hessian_finish_kernel, dim3(1), dim3(256), 0, st, H, K, percdamp);
    HAQ_CHECK_HIP(hipGetLastError());
    return HAQ_OK;
}

size_t haq_inverse_cholesky_workspace_bytes(int32_t K) {
    if (K <= 0) return 0;
    return 2 * (size_t)round_up((int64_t)K * K * 8, 256) + STATUS_BYTES;
}

// H may alias U: H is read once, into A, before anything else runs.
static int32_t inverse_cholesky_upper(const double* H, int K, double* U, double* A, double* M, int* status, hipStream_t st) {
    double* dblock = M;  // the factorised diagonal block on its way into A (M is filled afterwards)
    HAQ_CHECK_HIP(hipMemsetAsync(status, 0, sizeof(int), st));
    hipLaunchKernelGGL(flip_kernel, dim3(cdiv(K, 256), K), dim3(256), 0, st, H, K, A);
    for (int j0 = 0; j0 < K; j0 += PB) {
        const int below = K - j0 - PB;
        hipLaunchKernelGGL(chol_panel_kernel, dim3(below > 0 ? cdiv(below, 64) : 1), dim3(256), 0, st, A, K, j0, dblock, status);
        if (below <= 0)
            hipLaunchKernelGGL(chol_store_diag_kernel, dim3(1), dim3(256), 0, st, A, K, j0, (const double*)dblock);
        else
            hipLaunchKernelGGL(chol_trail_kernel, dim3(cdiv(below, 64), cdiv(below, 64)), dim3(256), 0, st, A, K, j0, (const double*)dblock);
    }
    HAQ_CHECK_HIP(hipMemsetAsync(M, 0, (size_t)K * K * sizeof(double), st));
    for (int i0 = 0; i0 < K; i0 += PB) {
        const int cols = i0 + PB < K ? i0 + PB : K, below = K - i0 - PB;
        hipLaunchKernelGGL(tri_inverse_block_kernel, dim3(cdiv(cols, 64)), dim3(64), 0, st, (const double*)A, K, i0, M);
        if (below <= 0) break;
        hipLaunchKernelGGL(tri_inverse_update_kernel, dim3(cdiv(cols, 64), cdiv(below, 64)), dim3(256), 0, st, (const double*)A, K, i0, M);
    }
    hipLaunchKernelGGL(flip_kernel, dim3(cdiv(K, 256), K), dim3(256), 0, st, (const double*)M, K, U);
    HAQ_CHECK_HIP(hipGetLastError());
    int host_status = 0;
    HAQ_CHECK_HIP(hipMemcpyAsync(&host_status, status, sizeof(int), hipMemcpyDeviceToHost, st));
    HAQ_CHECK_HIP(hipStreamSynchronize(st));
    if (host_status != 0)
        HAQ_FAIL(HAQ_ERR_INVALID_ARG, "the Hessian is not positive definite (pivot %d of the flipped matrix)", host_status - 1);
    return HAQ_OK;
}

int32_t haq_inverse_cholesky_upper_f64(const double* H, int32_t K, double* U, void* workspace, size_t workspace_bytes,
                                       void* stream) {
    if (K <= 0 || K > 65535 || !H || !U) HAQ_FAIL(HAQ_ERR_INVALID_ARG, "haq_inverse_cholesky_upper_f64: K=%d or null buffer", K);
    if (!workspace || workspace_bytes < haq_inverse_cholesky_workspace_bytes(K) || ((uintptr_t)workspace & 255u))
        HAQ_FAIL(HAQ_ERR_WORKSPACE, "haq_inverse_cholesky_upper_f64: workspace of %zu bytes (256-byte aligned) needed, got %zu",
                 haq_inverse_cholesky_workspace_bytes(K), workspace_bytes);
    const size_t mat = (size_t)round_up((int64_t)K * K * 8, 256);
    return inverse_cholesky_upper(H, K, U, (double*)workspace, (double*)((uint8_t*)workspace + mat),
                                  (int*)((uint8_t*)workspace + 2 * mat), (hipStream_t)stream);
}

size_t haq_hessian_quant_workspace_bytes(int32_t K, int32_t N) {
    if (K <= 0 || N <= 0) return 0;
    return carve_hess(nullptr, K, N).bytes;
}

int32_t haq_hessian_quant_weight(const void* x_fp16, int64_t ldx, int32_t T, const float* w, const float* s, int32_t K,
                                 int32_t N, double percdamp, int8_t* wq, float* w_scale, void* workspace,
                                 size_t workspace_bytes, void* stream) {
    if (T <= 0 || K <= 0 || N <= 0 || K > 65535) HAQ_FAIL(HAQ_ERR_INVALID_ARG, "haq_hessian_quant_weight: T=%d K=%d N=%d", T, K, N);
    if (!x_fp16 || !w || !wq || !w_scale || ldx < K) HAQ_FAIL(HAQ_ERR_INVALID_ARG, "haq_hessian_quant_weight: null buffer or ldx=%lld", (long long)ldx);
    const size_t need = carve_hess(nullptr, K, N).bytes;
    if (!workspace || workspace_bytes < need || ((uintptr_t)workspace & 255u))
        HAQ_FAIL(HAQ_ERR_WORKSPACE, "haq_hessian_quant_weight: workspace of %zu bytes (256-byte aligned) needed, got %zu", need, workspace_bytes);
    hipStream_t st = (hipStream_t)stream;
    HessWs ws = carve_hess(workspace, K, N);
    int rc;
    // the per-output-channel grid is the one of plain rounding
    if ((rc = launch_weight_colmax(w, s, 1, K, N, w_scale, st)) != HAQ_OK || (rc = launch_weight_scale(w_scale, N, st)) != HAQ_OK) return rc;
    if ((rc = haq_hessian_f64(x_fp16, ldx, s, T, K, percdamp, ws.H, stream)) != HAQ_OK) return rc;
    if ((rc = inverse_cholesky_upper(ws.H, K, ws.H, ws.A, ws.M, ws.status, st)) != HAQ_OK) {  // U replaces H
        // an indefinite Hessian leaves the codes of plain rounding, which belong to the scales above
        if (rc == HAQ_ERR_INVALID_ARG) (void)haq_quant_weight(w, s, K, N, wq, w_scale, stream);
        return rc;
    }
    const double* U = ws.H;
    hipLaunchKernelGGL(fold_weight_kernel, dim3(cdiv(N, 256), K), dim3(256), 0, st, w, s, K, N, ws.w64);
    // The errors of a stretch of channels are kept for one product over everything below it: in the memory of A and M,
    // which are done with, where GS channels fit there, else block by block in the block's own memory.
    const bool wide = (size_t)2 * K * K >= (size_t)GS * N;
    double* err = wide ? ws.A : ws.err;
    const int stretch = wide ? GS : GB;
    for (int s0 = 0; s0 < K; s0 += stretch) {
        const int s1 = s0 + stretch < K ? s0 + stretch : K;
        for (int b0 = s0; b0 < s1; b0 += GB) {
            hipLaunchKernelGGL(gptq_block_kernel, dim3(cdiv(N, 64)), dim3(64), 0, st, ws.w64, U, (const float*)w_scale, K, N, b0, wq,
                               err + (size_t)(b0 - s0) * N);
            if (b0 + GB < s1)
                hipLaunchKernelGGL(gptq_update_kernel, dim3(cdiv(N, 64), cdiv(s1 - b0 - GB, 64)), dim3(256), 0, st, ws.w64, U,
                                   (const double*)err + (size_t)(b0 - s0) * N, K, N, b0, GB, b0 + GB, s1);
        }
        if (s1 >= K) break;
        hipLaunchKernelGGL(gptq_update_kernel, dim3(cdiv(N, 64), cdiv(K - s1, 64)), dim3(256), 0, st, ws.w64, U, (const double*)err, K, N,
                               s0, stretch, s1, K);
    }
    HAQ_CHECK_HIP(hipGetLastError());
    return HAQ_OK;
}

size_t haq_quantize_layer_workspace_bytes(int32_t T, int32_t K, int32_t N, int32_t n_e) {
    const size_t a = haq_smoothing_search_workspace_bytes(T, K, N, n_e), b = haq_hessian_quant_workspace_bytes(K, N);
    return a > b ? a : b;
}

int32_t haq_quantize_layer(const void* x_fp16, int64_t ldx, int32_t T, const float* w, int32_t K, int32_t N,
                           const double* exponents, int32_t n_e, int32_t use_weight, double percdamp, float* s,
                           int8_t* wq, float* w_scale, double* losses, int32_t* best, void* workspace,
                           size_t workspace_bytes, void* stream) {
    if (!s || !wq || !w_scale) HAQ_FAIL(HAQ_ERR_INVALID_ARG, "haq_quantize_layer: null output");
    if (T <= 0 || K <= 0 || N <= 0 || n_e <= 0) HAQ_FAIL(HAQ_ERR_INVALID_ARG, "haq_quantize_layer: T=%d K=%d N=%d n_e=%d", T, K, N, n_e);
    if (workspace_bytes < haq_quantize_layer_workspace_bytes(T, K, N, n_e))
        HAQ_FAIL(HAQ_ERR_WORKSPACE, "haq_quantize_layer: workspace of %zu bytes needed, got %zu", haq_quantize_layer_workspace_bytes(T, K, N, n_e),
                 workspace_bytes);
    // step 1: smoothing vector by grid search; step 2: Hessian-aware quantisation of the folded weight;
    // step 3 on this device is to keep the int8 codes (the caller packs them for the MFMA kernels)
    int rc = haq_smoothing_search(x_fp16, ldx, w, T, K, N, exponents, n_e, use_weight, losses, best, s, workspace, workspace_bytes, stream);
    if (rc != HAQ_OK) return rc;
    return haq_hessian_quant_weight(x_fp16, ldx, T, w, s, K, N, percdamp, wq, w_scale, workspace, workspace_bytes, stream);
}

}  // extern "C"
