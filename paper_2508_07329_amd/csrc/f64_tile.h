// Binary64 products on the matrix cores with the order of every sum kept: C(i, j) followed by fma(a(i, k), b(k, j), C)
// for k ascending, which is what v_mfma_f64_16x16x4_f64 computes (checked bit for bit against scalar chains, subnormal
// operands and sums and both zeros included).
//
// A work-group of 4 waves (2 x 2) owns a 64 x 64 tile, a wave 32 x 32 of it; k comes through LDS in chunks of 16, the
// next chunk held in registers meanwhile.  Bound: the binary64 matrix pipe, an instruction of 1024 multiply-adds every
// 91 cycles with several waves on a SIMD (138 with one: hence a small tile, four to seven waves to a SIMD; 128 x 128
// tiles, two waves, took 424 us where four 64 x 64 ones take 400), which is 55 TFLOP/s at 2.4 GHz.  The reference product
// (4096 links a tile) reaches 54, the compensation's products, which load and store their tile for 64 to 256 links, 44.
// The 4 x 4 register tiles of the vector unit that these products used before were bound by LDS, 8 reads for 16
// multiply-adds.
#pragma once
#include "haq_common.h"

namespace haq {

typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int F64_B = 64;   // rows and columns of a tile
constexpr int F64_KC = 16;  // k per chunk
constexpr int F64_PER = F64_KC * F64_B / 256;  // elements of an operand per thread and chunk

// An operand: element (k, i) of the tile's rows i is cvt(p[k ld + i]) (KMAJOR) or cvt(p[i ld + k]), p at the tile's first
// row.  Rows past n_i re-read the last one: they end in results that nobody stores.  Nothing bounds a stride, so every
// offset that holds ld is 64-bit.  KMAJOR: a wave fetches whole rows of k, whose addresses are scalar, and the lane adds
// its i (with 64-bit offsets for each lane the compensation's products took 6.4 ms instead of 6.2 at 4096 x 16384).
template <bool KMAJOR, class T, class CVT>
struct F64Operand {
    static constexpr int LDS = KMAJOR ? F64_KC * (F64_B + 16) : F64_B * (F64_KC + 1);  // doubles; both pitches spread a fragment over the banks
    const T* p;
    int64_t ld;
    CVT cvt;
    int64_t off[KMAJOR ? 1 : F64_PER];
    double r[F64_PER];
    static __device__ __forceinline__ int at(int k, int i) { return KMAJOR ? k * (F64_B + 16) + i : i * (F64_KC + 1) + k; }
    static __device__ __forceinline__ int my_k(int n) {
        return KMAJOR ? __builtin_amdgcn_readfirstlane(threadIdx.x / F64_B) + 256 / F64_B * n : threadIdx.x % F64_KC;
    }
    static __device__ __forceinline__ int my_i(int n) { return KMAJOR ? threadIdx.x % F64_B : threadIdx.x / F64_KC + 256 / F64_KC * n; }
    __device__ __forceinline__ F64Operand(const T* p_, int64_t ld_, int n_i, CVT cvt_) : p(p_), ld(ld_), cvt(cvt_) {
#pragma unroll
        for (int n = 0; n < (KMAJOR ? 1 : F64_PER); ++n) {
            const int i = min(my_i(n), n_i - 1);
            off[n] = KMAJOR ? i : i * ld + my_k(n);
        }
    }
    __device__ __forceinline__ T element(int k0, int n) const {
        if constexpr (KMAJOR)
            return (p + (k0 + my_k(n)) * ld)[(uint32_t)off[0]];
        else
            return (p + k0)[off[n]];
    }
    __device__ __forceinline__ void fetch(int k0, int klen) {
        if (k0 + F64_KC <= klen) {
#pragma unroll
            for (int n = 0; n < F64_PER; ++n) r[n] = cvt(element(k0, n));
        } else {  // past the last k: 0, which leaves a chain that has started from +0 as it is
#pragma unroll
            for (int n = 0; n < F64_PER; ++n) r[n] = k0 + my_k(n) < klen ? cvt(element(k0, n)) : 0.0;
        }
    }
    __device__ __forceinline__ void store(double* lds) {
#pragma unroll
        for (int n = 0; n < F64_PER; ++n) lds[at(my_k(n), my_i(n))] = r[n];
    }
};
template <bool KMAJOR, class T, class CVT>
__device__ __forceinline__ F64Operand<KMAJOR, T, CVT> f64_operand(const T* p, int64_t ld, int n_i, CVT cvt) {
    return F64Operand<KMAJOR, T, CVT>(p, ld, n_i, cvt);
}

// The tile's accumulators: [mi][ni][r] is row 32 wm + 16 mi + 4 r + lane / 16, column 32 wn + 16 ni + lane % 16.
typedef v4d F64Acc[2][2];

template <class A, class B>
__device__ __forceinline__ void f64_tile_mac(F64Acc& acc, int klen, double* lds, A a, B b) {
    double* la = lds;
    double* lb = lds + A::LDS;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int ia = 32 * (wave >> 1) + (lane & 15), ib = 32 * (wave & 1) + (lane & 15), q = lane >> 4;
    a.fetch(0, klen);
    b.fetch(0, klen);
    for (int k0 = 0; k0 < klen; k0 += F64_KC) {
        __syncthreads();  // the previous chunk has been read
        a.store(la);
        b.store(lb);
        __syncthreads();
        if (k0 + F64_KC < klen) {
            a.fetch(k0 + F64_KC, klen);
            b.fetch(k0 + F64_KC, klen);
        }
#pragma unroll
        for (int kk = 0; kk < F64_KC; kk += 4) {
            double fa[2], fb[2];
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                fa[m] = la[A::at(kk + q, ia + 16 * m)];
                fb[m] = lb[B::at(kk + q, ib + 16 * m)];
            }
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int n = 0; n < 2; ++n) acc[m][n] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[m], fb[n], acc[m][n], 0, 0, 0);
        }
    }
}

// f(value, row, column) for each of the thread's elements of the tile.
template <class F>
__device__ __forceinline__ void f64_tile_each(F64Acc& acc, F&& f) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i0 = 32 * (wave >> 1) + (lane >> 4), j0 = 32 * (wave & 1) + (lane & 15);
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int ni = 0; ni < 2; ++ni) {
                double v = acc[mi][ni][r];
                f(v, i0 + 16 * mi + 4 * r, j0 + 16 * ni);
                acc[mi][ni][r] = v;
            }
}

struct F64Same {
    template <class T>
    __device__ double operator()(T v) const { return (double)v; }
};
struct F64Minus {
    __device__ double operator()(double v) const { return -v; }
};

// run + p[0] + p[1] + ... + p[n - 1], one addition after another (the values are fetched ahead of the chain).
__device__ __forceinline__ double add_in_order(double run, const double* p, int n) {
    int c = 0;
    for (; c + 16 <= n; c += 16) {
        double t[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) t[i] = p[c + i];
#pragma unroll
        for (int i = 0; i < 16; ++i) run += t[i];
    }
    for (; c < n; ++c) run += p[c];
    return run;
}

}  // namespace haq
