// W8A8 linear for short batches (at most 128 token rows, longer ones on few output channels, the down projections of expert
// groups of few rows): the weights are streamed from HBM once, straight into MFMA operand registers, as on the decode path
// of the routed expert FFN.
//
// Bound: the weight stream (K N bytes).  The tiled GEMM cannot draw it at these batches: its grid is one
// work-group per 128 or 256 channels (32 on a 4096-channel layer), with two K-steps of 16 KB in flight each.
// Here a work-group owns 16 C channels and splits K over its 8 waves (a 64-byte K-step each in turn), every wave
// holds the fragments of DEPTH K-steps, and the exact int32 partial sums are added in LDS.
// v_mfma_i32_16x16x64_i8: the weights are the first operand (16 channels x 64 k, lane = channel, 16-byte chunk), a
// block of 16 token rows the second, so a lane ends up with four consecutive channels of one row.
// Measured (weights cold, us; 128 x 128 tiles of the GEMM - this kernel):
//   rows             1          16          32          64         128
//   4096 x 16384   20.7-12.3   20.9-12.4   20.8-14.1   21.5-15.4   23.6-21.0   (13.2 at the rate of a large copy)
//   16384 x 4096   57.5-13.3   57.8-14.7   57.7-18.7   59.3-25.3   66.1-36.3   (13.2; the token rows are re-read per unit)
//   768 x 3072      7.6- 3.6    7.9- 3.7    7.9- 4.3    8.2- 4.6    8.4- 6.5
#include "group_tiles.h"
#include "haq_common.h"
#include "quant_math.h"

namespace haq {

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(1))) v4i* gptr_v4i;
__device__ __forceinline__ v4i gload16(const int8_t* p) { return *(gptr_v4i)(uintptr_t)p; }
__device__ __forceinline__ v4i gload16_stream(const int8_t* p) { return __builtin_nontemporal_load((gptr_v4i)(uintptr_t)p); }

constexpr int SK_WAVES = 8, SG_WAVES = 4;  // waves of a work-group: dense, expert groups

struct StreamTile {
    const int8_t* B;        // packed weights
    const float* sw;        // channel scales
    const int32_t* colsum;  // column sums of the weight codes (asymmetric codes)
    int row0, rows;         // first row and row count (at most 16 RB)
    int n0;                 // first channel
};

// One tile: 16 C channels x `rows` token rows, K split over the work-group's NW waves.  STREAM: no other work-group
// reads these weights.
template <int NW, int C, int RB, int DEPTH, bool ASYM, bool STREAM>
__device__ __forceinline__ void stream_tile(const GemmArgs& a, const StreamTile& t, int (*sum)[4][64]) {
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, q = lane >> 4;
    const int nk = (a.K + 63) / 64;  // a last partial K-step reads chunks past K: the weights are zero there
    const int n = nk > wave ? (nk - wave + NW - 1) / NW : 0;  // this wave's K-steps: wave, wave + NW, ...
    const size_t wstep = (size_t)4 * NW * a.Npad * 16, xstep = (size_t)4 * NW * a.R * 16;
    const int8_t* pw = t.B + ((size_t)(4 * wave + q) * a.Npad + t.n0 + l16) * 16;
    const int8_t* px = a.A + ((size_t)(4 * wave + q) * a.R + t.row0) * 16;
    int xoff[RB];  // rows past the last one re-read it (their results are dropped)
#pragma unroll
    for (int b = 0; b < RB; ++b) xoff[b] = min(16 * b + l16, t.rows - 1) * 16;

    v4i acc[C][RB];
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
        for (int b = 0; b < RB; ++b) acc[c][b] = v4i{0, 0, 0, 0};
    struct Frag {
        v4i w[C], x[RB];
    };
    auto fetch = [&](Frag& f) {
#pragma unroll
        for (int c = 0; c < C; ++c) f.w[c] = STREAM ? gload16_stream(pw + c * 256) : gload16(pw + c * 256);
#pragma unroll
        for (int b = 0; b < RB; ++b) f.x[b] = gload16(px + xoff[b]);
    };
    auto mac = [&](const Frag& f) {
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
            for (int b = 0; b < RB; ++b) acc[c][b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(f.w[c], f.x[b], acc[c][b], 0, 0, 0);
    };
    Frag fr[DEPTH];
    int fetched = 0;  // the loads stay unconditional: past this wave's last K-step they re-read it
    auto next = [&](Frag& f) {
        fetch(f);
        if (++fetched < n) {
            pw += wstep;
            px += xstep;
        }
    };
    if (n > 0) {
#pragma unroll
        for (int i = 0; i < DEPTH; ++i) next(fr[i]);
    }
    for (int i = tid; i < C * RB * 256; i += NW * 64) (&sum[0][0][0])[i] = 0;
    __syncthreads();
    if (n > 0) {
        int k = 0;
        for (; k + DEPTH < n; k += DEPTH) {
#pragma unroll
            for (int i = 0; i < DEPTH; ++i) {
                mac(fr[i]);
                next(fr[i]);
                // Expert groups: without it the loads sink below the next steps' MFMAs (two groups of 112 rows of
                // 1024 x 3584: 57.4 -> 55.6 us a layer).  The dense forms, eight waves that cover for each other, are
                // faster as the compiler places them (400 rows of 16384 x 4096: 42.6 against 44.0).
                if (NW == SG_WAVES) __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int i = 0; i < DEPTH; ++i)
            if (k + i < n) mac(fr[i]);
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
            for (int b = 0; b < RB; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r) atomicAdd(&sum[c * RB + b][r][lane], acc[c][b][r]);  // exact: the order is immaterial
    }
    __syncthreads();
    for (int i = tid; i < C * RB * 64; i += NW * 64) {
        const int cb = i >> 6, ln = i & 63;
        const int row = 16 * (cb % RB) + (ln & 15), ch = t.n0 + 16 * (cb / RB) + 4 * (ln >> 4);
        if (row >= t.rows || ch >= a.N) continue;
        const float sx = a.sx[t.row0 + row];
        const int zshift = ASYM ? 128 - a.zp[t.row0 + row] : 0;
        __half hv[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            int v = sum[cb][r][ln];
            if (ASYM) v += zshift * t.colsum[ch + r];
            if (a.acc_dbg) a.acc_dbg[(size_t)(t.row0 + row) * a.N + ch + r] = v;
            float f = dequant(v, sx, t.sw[ch + r]);
            if (a.act == HAQ_ACT_RELU) f = fmaxf(f, 0.0f);
            hv[r] = f2h(f);
        }
        *reinterpret_cast<uint2*>(a.Y + (size_t)(t.row0 + row) * a.ldy + ch) = *reinterpret_cast<const uint2*>(hv);
    }
}

// C: blocks of 16 channels per work-group; RB: blocks of 16 token rows; WPS: waves per SIMD (register budget).
template <int C, int RB, int DEPTH, int WPS, bool ASYM>
__global__ __launch_bounds__(SK_WAVES * 64, WPS) void skinny_linear_kernel(GemmArgs a) {
    __shared__ int sum[C * RB][4][64];
    const StreamTile t{a.B, a.sw, a.colsum, 0, a.M, (int)blockIdx.x * (16 * C)};
    stream_tile<SK_WAVES, C, RB, DEPTH, ASYM, true>(a, t, sum);
}

// More rows: `mt` row tiles of `tile_rows` rows share a unit of 64 channels.  Work-group ids are dealt round-robin to
// the eight XCDs; each of them (one L2) takes a contiguous range of tiles, rows fastest, so that a unit's weights cross
// the fabric once.  Bound: the fragments of a K-step, 1 KB for each block of 16 channels or rows, through a CU's load
// path (64 B a cycle) against 4 RB matrix instructions; 16384 x 4096 on 333 rows, 256 tiles of 96 x 64
// 39.2 us, 128 x 128 tiles 62.5.
template <int RB, int DEPTH, bool ASYM>
__global__ __launch_bounds__(SK_WAVES * 64, 2) void stream_linear_kernel(GemmArgs a, int mt, int tile_rows) {
    __shared__ int sum[4 * RB][4][64];
    const int total = mt * ((a.N + 63) / 64), per = (total + 7) / 8, slot = blockIdx.x / 8;
    const int id = (int)(blockIdx.x % 8) * per + slot;
    if (slot >= per || id >= total) return;
    const int row0 = (id % mt) * tile_rows;
    const StreamTile t{a.B, a.sw, a.colsum, row0, min(tile_rows, a.M - row0), (id / mt) * 64};
    stream_tile<SK_WAVES, 4, RB, DEPTH, ASYM, false>(a, t, sum);
}

// Down projections of expert groups of few rows.  Bound: the weight stream, each activated expert's once; the tiled
// kernel has one work-group per 256 channels and expert with two K-steps in flight (14336 x 4096, 8 experts of 20 rows:
// the layer 280 us, 248 here).  An expert's m rows
// are cut into ceil(m / 128) tiles of equal height; the units of 64 channels go round the XCDs, as work-group ids do, and
// the row tiles of a unit stay on one of them.  Four waves, so that a CU holds two work-groups, one streaming while the
// other adds up and stores.
template <bool ASYM>
__global__ __launch_bounds__(SG_WAVES * 64, 2) void stream_grouped_kernel(GemmArgs a) {
    __shared__ int sum[4 * 8][4][64];
    const GroupLanes g(a);
    GroupTile gt;
    if (!g.deal<128>(a, a.N / 64, gt)) return;
    const int e = g.of(g.e, gt.i), lo = g.of(g.lo, gt.i), m = g.of(g.hi, gt.i) - lo;
    const int tile_rows = ((m + gt.mt - 1) / gt.mt + 15) / 16 * 16;  // (mt - 1) tile_rows < m: no tile is empty
    const int r0 = gt.mi * tile_rows, rows = min(tile_rows, m - r0);
    const ExpertTab& x = a.tab[e];
    const StreamTile t{x.w2, x.sw2, ASYM ? a.cstab[e].cs2 : nullptr, lo + r0, rows, gt.u * 64};
    // Row tiles that share their weights read them through the caches (4096 x 14336, 8 experts of 76 rows, skewed: the layer
    // 339 -> 333 us; two of 192 rows: 161 -> 152); two and more have over 32 rows each.
    if (gt.mt > 1) {
        if (rows <= 64)
            stream_tile<SG_WAVES, 4, 4, 4, ASYM, false>(a, t, sum);
        else if (rows <= 96)
            stream_tile<SG_WAVES, 4, 6, 3, ASYM, false>(a, t, sum);
        else
            stream_tile<SG_WAVES, 4, 8, 2, ASYM, false>(a, t, sum);
    } else if (rows <= 32) {
        stream_tile<SG_WAVES, 4, 2, 6, ASYM, true>(a, t, sum);
    } else if (rows <= 64) {
        stream_tile<SG_WAVES, 4, 4, 4, ASYM, true>(a, t, sum);
    } else if (rows <= 96) {
        stream_tile<SG_WAVES, 4, 6, 3, ASYM, true>(a, t, sum);
    } else {
        stream_tile<SG_WAVES, 4, 8, 2, ASYM, true>(a, t, sum);
    }
}

// A few rows of short K: every work-group forms the codes itself, so that the layer is one launch.  WPR waves share a
// row (a chunk of 16 channels to each lane, K <= 1024 WPR), 8 / WPR rows at a time, at most two to a lane, which shares the
// reciprocals of the smoothing vector between them; the codes (16 KB, chunk-major) and the row scales stay in LDS.
// Bound: latency, of the loads, of the row maximum and of the weight stream, one after another; the first weights are
// fetched behind the rows' loads and in front of their use.  us a call on the GPU, the quantiser's launch and the linear's / this:
//   512 x 512, 16 rows 7.8 / 6.5;  768 x 3072, 1: 7.4 / 6.6, 16: 7.8 / 6.7;  1024 x 16384, 16: 10.3 / 9.1;  2048 x 8192, 8: 10.1 / 9.5
//   4096 x 4096, 4: 9.7 / 9.1;  4096 x 16384, 4: 16.6 / 16.1;  8192 x 1024, 2: 11.4 / 9.3;  8192 x 16384, 2: 26.9 / 25.6
// and the host launches once: 768 x 3072 on 16 rows, back to back, 9.8 -> 7.5.
template <int C, int WPR>
__global__ __launch_bounds__(SK_WAVES * 64, C == 1 ? 4 : 2) void fused_linear_kernel(GemmArgs a, const __half* x, int64_t ldx, const float* s) {
    constexpr int RG = SK_WAVES / WPR, ROWS = 2 * RG, DEPTH = WPR == 1 ? 2 : 4;
    __shared__ __attribute__((aligned(16))) uint4 codes[64 * WPR][ROWS];
    __shared__ float red[ROWS][WPR], scale_s[ROWS];
    __shared__ int sum[C][4][64];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nchunk = a.K / 16, c = (wave % WPR) * 64 + lane, cc = min(c, nchunk - 1), g = wave / WPR;
    uint4 raw[2][2];  // loads stay unconditional: rows and chunks past the last re-read it
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const uint4* px = reinterpret_cast<const uint4*>(x + (size_t)min(g + j * RG, a.M - 1) * ldx + cc * 16);
        raw[j][0] = px[0];
        raw[j][1] = px[1];
    }
    float4 s4[4];
    if (s) {
#pragma unroll
        for (int i = 0; i < 4; ++i) s4[i] = reinterpret_cast<const float4*>(s + cc * 16)[i];
    }
    __builtin_amdgcn_sched_barrier(0);

    const int l16 = lane & 15, q = lane >> 4, n0 = (int)blockIdx.x * (16 * C);
    const int nk = (a.K + 63) / 64, n = nk > wave ? (nk - wave + SK_WAVES - 1) / SK_WAVES : 0;  // this wave's K-steps: wave, wave + 8, ...
    const int8_t* pw = a.B + ((size_t)(4 * wave + q) * a.Npad + n0 + l16) * 16;
    const size_t wstep = (size_t)4 * SK_WAVES * a.Npad * 16;
    v4i w[DEPTH][C];
    int fetched = 0;
    auto next = [&](v4i(&f)[C]) {  // past this wave's last K-step it is fetched again
#pragma unroll
        for (int b = 0; b < C; ++b) f[b] = gload16_stream(pw + b * 256);
        if (++fetched < n) pw += wstep;
    };
    if (n > 0) {
#pragma unroll
        for (int i = 0; i < DEPTH; ++i) next(w[i]);
    }
    __builtin_amdgcn_sched_barrier(0);

    float y[2][16], sv[16], rv[16], amax[2];
    bool fast = true;
    if (s) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            sv[i] = i % 4 == 0 ? s4[i / 4].x : i % 4 == 1 ? s4[i / 4].y : i % 4 == 2 ? s4[i / 4].z : s4[i / 4].w;
            rv[i] = 1.0f / sv[i];
            fast = fast & safe_divisor(sv[i]);
        }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        Half8 h0, h1;
        *reinterpret_cast<uint4*>(&h0) = raw[j][0];
        *reinterpret_cast<uint4*>(&h1) = raw[j][1];
        amax[j] = 0.0f;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const float v = h2f(i < 8 ? h0.v[i] : h1.v[i - 8]);
            y[j][i] = !s ? v : fast ? div_by(v, sv[i], rv[i], true) : v / sv[i];
            amax[j] = fmaxf(amax[j], fabsf(y[j][i]));
        }
        amax[j] = wave_max(c < nchunk ? amax[j] : 0.0f);
        if (lane == 0) red[g + j * RG][wave % WPR] = amax[j];
    }
    for (int i = tid; i < C * 256; i += SK_WAVES * 64) (&sum[0][0][0])[i] = 0;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int row = g + j * RG;
        float m = 0.0f;
#pragma unroll
        for (int i = 0; i < WPR; ++i) m = fmaxf(m, red[row][i]);
        const float scale = m / 127.0f, rscale = 1.0f / scale;
        const bool sfast = scale >= 0x1p-100f && scale <= 0x1p100f;
        uint32_t u[4] = {0, 0, 0, 0};
        if (m != 0.0f) {
            if (fast && sfast) {
                float v[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) v[i] = div_by(y[j][i], scale, rscale, true);
#pragma unroll
                for (int i = 0; i < 4; ++i) u[i] = round_pack4(v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]);
            } else {
#pragma unroll
                for (int i = 0; i < 16; ++i) u[i / 4] |= (uint32_t)(code_of(y[j][i], scale) & 0xff) << (8 * (i % 4));
            }
        }
        if (c < nchunk) codes[c][row] = make_uint4(u[0], u[1], u[2], u[3]);
        if (c == 0) scale_s[row] = scale;
    }
    __syncthreads();

    if (n > 0) {
        v4i acc[C];
#pragma unroll
        for (int b = 0; b < C; ++b) acc[b] = v4i{0, 0, 0, 0};
        const int xr = min(l16, a.M - 1);
        auto mac = [&](const v4i(&f)[C], int k) {  // a last partial K-step reads chunks past K: the weights are zero there
            const v4i xv = *reinterpret_cast<const v4i*>(&codes[4 * (wave + SK_WAVES * k) + q][xr]);
#pragma unroll
            for (int b = 0; b < C; ++b) acc[b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(f[b], xv, acc[b], 0, 0, 0);
        };
        int k = 0;
        for (; k + DEPTH < n; k += DEPTH) {
#pragma unroll
            for (int i = 0; i < DEPTH; ++i) {
                mac(w[i], k + i);
                next(w[i]);
            }
        }
#pragma unroll
        for (int i = 0; i < DEPTH; ++i)
            if (k + i < n) mac(w[i], k + i);
#pragma unroll
        for (int b = 0; b < C; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) atomicAdd(&sum[b][r][lane], acc[b][r]);  // exact: the order is immaterial
    }
    __syncthreads();
    for (int i = tid; i < C * 64; i += SK_WAVES * 64) {
        const int b = i >> 6, ln = i & 63, row = ln & 15, ch = n0 + 16 * b + 4 * (ln >> 4);
        if (row >= a.M || ch >= a.N) continue;
        __half hv[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float f = dequant(sum[b][r][ln], scale_s[row], a.sw[ch + r]);
            if (a.act == HAQ_ACT_RELU) f = fmaxf(f, 0.0f);
            hv[r] = f2h(f);
        }
        *reinterpret_cast<uint2*>(a.Y + (size_t)row * a.ldy + ch) = *reinterpret_cast<const uint2*>(hv);
    }
}

template <int C, int RB, int DEPTH, int WPS>
int launch_one(const GemmArgs& a, bool asym, hipStream_t st) {
    const dim3 grid(cdiv(a.N, 16 * C));
    if (asym)
        hipLaunchKernelGGL((skinny_linear_kernel<C, RB, DEPTH, WPS, true>), grid, dim3(SK_WAVES * 64), 0, st, a);
    else
        hipLaunchKernelGGL((skinny_linear_kernel<C, RB, DEPTH, WPS, false>), grid, dim3(SK_WAVES * 64), 0, st, a);
    HAQ_CHECK_HIP(hipGetLastError());
    return HAQ_OK;
}

template <int RB, int DEPTH>
int launch_rows(const GemmArgs& a, bool asym, hipStream_t st) {
    const int mt = cdiv(a.M, 16 * RB), tile_rows = 16 * cdiv(cdiv(a.M, mt), 16);
    const dim3 grid((unsigned)round_up((int64_t)mt * cdiv(a.N, 64), 8));
    if (asym)
        hipLaunchKernelGGL((stream_linear_kernel<RB, DEPTH, true>), grid, dim3(SK_WAVES * 64), 0, st, a, mt, tile_rows);
    else
        hipLaunchKernelGGL((stream_linear_kernel<RB, DEPTH, false>), grid, dim3(SK_WAVES * 64), 0, st, a, mt, tile_rows);
    HAQ_CHECK_HIP(hipGetLastError());
    return HAQ_OK;
}

}  // namespace

// 64 channels per work-group share every token fragment, but only from 128 such units on do enough CUs draw
// weights: 12672 channels, 16 rows of 3168: 9.9 us against 13.2 with 16 channels, 64 rows: 13.6 against 22.9;
// 4096 channels, 16 rows of 4096: 8.3 us against 5.8, 64 rows: 12.0 against 8.0.
static int channel_blocks(int N) { return N / 64 >= 128 ? 4 : 1; }

// Up to 64 rows the weight stream decides: one round of work-groups wins; more rounds each pay the start, the sums and the
// epilogue again, while 128 x 128 tiles have work-groups enough and fetch every weight once past the caches: further rounds are
// level with them on few rows of long K only.  From 65 rows on a K-step also costs 6 or 8 row fragments, on one work-group per CU.
// Measured (weights cold, us, this kernel / 128 x 128 tiles; K x N):
//   one round:   1 row:  512 x 16384 5.6 / 7.3;  13 rows:  848 x 25600 9.2 / 9.3, 528 x 27888 8.5 / 7.9;  15: 2416 x 24528 15.0 / 15.6;  41: 672 x 14000 7.9 / 8.3
//   two rounds:  15 rows:  848 x 37168 12.3 / 12.4;  9: 1168 x 39632 13.6 / 14.9;  16: 1840 x 34112 14.9 / 19.0
//                13: 832 x 54752 15.6 / 12.7;  10: 1232 x 53408 17.4 / 16.2;  13: 1520 x 48784 17.4 / 17.9;  5: 1680 x 56592 18.8 / 19.8;  16: 1024 x 65536 19.0 / 15.3
//                20 rows:  1536 x 18784 12.8 / 11.6;  31: 2112 x 17120 14.1 / 13.9;  19: 2288 x 16464 13.5 / 14.3;  21: 4720 x 16640 21.6 / 23.6;  28: 5712 x 29600 34.4 / 30.7
//                33 rows:  1232 x 24656 15.3 / 11.2;  48: 7040 x 23680 41.0 / 34.9;   64: 2048 x 24576 17.9 / 14.8, 11264 x 24048 65 / 54
//   three:       23 rows:  1536 x 37840 19.1 / 17.2;  22: 2032 x 34256 20.0 / 20.4;  29: 2560 x 41072 22.6 / 24.6;  25: 4912 x 41584 37.7 / 42.5
//   four:        32 rows:  2048 x 65536 31.7 / 24.5;   33: 4096 x 65536 53 / 43;   64: 4096 x 65536 62 / 45
//   96 rows:  512 x 16384 9.1 / 7.7, 768 x 16384 9.9 / 8.8;  79: 1104 x 11280 9.6 / 10.2;   128: 1024 x 16384 11.1 / 10.2, 1168 x 15264 11.3 / 11.2;  117: 2448 x 11632 15.2 / 16.3
// Between one round of 16-channel units and 128 units of 64 channels two row tiles of 64 rows (launch_stream_rows) fill the
// chip (this kernel / those): 96 rows of 512 x 8192 8.1 / 7.6, 1536 x 6144 11.4 / 9.0, 4096 x 8192 16.4 / 14.2, 8192 x 8192 28.2 / 22.5.  On fewer
// channels those are too few work-groups: 128 rows of 4096 x 4096 11.2 / 13.3, 16384 x 4096 36.2 / 36.7.
bool skinny_pays(const GemmArgs& a) {
    if (a.offsets || a.M < 1 || a.M > SKINNY_MAX_ROWS) return false;
    const int n_cu = cu_count(), C = channel_blocks(a.N), RB = (a.M + 15) / 16;
    const int per_cu = RB == 1 || (C == 1 && RB <= 4) ? 2 : 1;  // work-groups that a CU holds
    const int rounds = cdiv(cdiv(a.N, 16 * C), per_cu * n_cu);
    if (RB > 4) {
        if (a.N <= 16 * n_cu) return true;
        return 2 * cdiv(a.N, 64) > n_cu && rounds == 1 && a.K >= (RB > 6 ? 1152 : 1024);
    }
    if (RB == 1 && rounds == 2) return a.K >= (a.N <= 160 * n_cu ? 896 : 1472);  // a second round that is hardly begun costs less
    return rounds == 1 || (RB == 2 && rounds <= 3 && a.K >= (rounds == 2 ? 2176 : 2048));
}

// 16 rows up to K = 1024, 8 to 2048, 4 to 4096, 2 to 8192, and a work-group for each CU at most: 3 to 23 % faster there at
// every one of 70 sizes.  A second work-group on a CU forms the codes again, on vector units that are busy with the first
// one's: that pays where the weight stream is long enough to hide it.  us on the GPU, two launches / this:
//   16-channel units:  K = 48: 7.1 / 7.8,  144: 7.2 / 8.1,  256: 7.6 / 8.1,  384: 8.3 / 8.3,  848: 8.9 / 8.7,  1392: 8.8 / 9.1,
//                      1984: 9.6 / 10.3,  2240: 9.8 / 9.8,  3472: 11.1 / 10.6,  4336: 13.1 / 10.8,  7280: 17.9 / 14.0
//                      (what is lost from 1040 to 2112 the host's second launch costs: 8 rows of 1984 x 7936 back to back 11.1 / 8.7)
//   64-channel units (past 16384 channels):  K = 16: 7.2 / 8.5,  128: 8.0 / 8.7,  288: 9.2 / 9.2,  400: 11.0 / 9.9,  992: 12.4 / 11.4,
//                      1056: 12.2 / 15.8,  1536: 13.9 / 17.5,  2400: 18.3 / 21.2,  5488: 26.2 / 28.4
bool fused_linear_fits(int M, int K, int N) {
    if (M < 1 || K > 8192 || M * (K <= 1024 ? 1 : K <= 2048 ? 2 : K <= 4096 ? 4 : 8) > 16) return false;
    const int C = channel_blocks(N), groups = cdiv(N, 16 * C), n_cu = cu_count();
    return groups <= n_cu || (groups <= 2 * n_cu && K >= 288 && (C == 1 || K <= 1024));
}

int launch_fused_linear(const GemmArgs& a, const __half* x, int64_t ldx, const float* s, hipStream_t st) {
    const int C = channel_blocks(a.N);
    const dim3 grid(cdiv(a.N, 16 * C)), block(SK_WAVES * 64);
#define HAQ_FUSED(c, wpr)                                                                            \
    if (C == c && a.K <= 1024 * wpr) {                                                               \
        hipLaunchKernelGGL((fused_linear_kernel<c, wpr>), grid, block, 0, st, a, x, ldx, s);         \
        HAQ_CHECK_HIP(hipGetLastError());                                                            \
        return HAQ_OK;                                                                               \
    }
    HAQ_FUSED(1, 1)
    HAQ_FUSED(1, 2)
    HAQ_FUSED(1, 4)
    HAQ_FUSED(1, 8)
    HAQ_FUSED(4, 1)
    HAQ_FUSED(4, 2)
    HAQ_FUSED(4, 4)
    HAQ_FUSED(4, 8)
#undef HAQ_FUSED
    return HAQ_ERR_UNSUPPORTED;
}

int launch_skinny(const GemmArgs& a, bool asym, hipStream_t st) {
    static_assert(SKINNY_MAX_ROWS == 128, "eight blocks of 16 rows");
    const int C = channel_blocks(a.N);
    const int RB = (a.M + 15) / 16;
#define HAQ_SKINNY(c, b, d, w) \
    if (C == c && RB <= b) return launch_one<c, b, d, w>(a, asym, st)
    HAQ_SKINNY(1, 1, 4, 4);
    HAQ_SKINNY(1, 2, 6, 4);
    HAQ_SKINNY(1, 4, 4, 4);
    HAQ_SKINNY(1, 6, 5, 2);
    HAQ_SKINNY(1, 8, 4, 2);
    HAQ_SKINNY(4, 1, 4, 4);
    HAQ_SKINNY(4, 2, 5, 2);
    HAQ_SKINNY(4, 4, 4, 2);
    HAQ_SKINNY(4, 6, 3, 2);
    HAQ_SKINNY(4, 8, 2, 2);
#undef HAQ_SKINNY
    return HAQ_ERR_UNSUPPORTED;
}

int launch_stream_rows(const GemmArgs& a, bool asym, int rb, hipStream_t st) {
    switch (rb) {
        case 4: return launch_rows<4, 4>(a, asym, st);
        case 6: return launch_rows<6, 3>(a, asym, st);
        default: return launch_rows<8, 2>(a, asym, st);
    }
}

int launch_stream_grouped(const GemmArgs& a, bool asym, hipStream_t st) {
    if (a.which != 1 || a.N % 64) return HAQ_ERR_UNSUPPORTED;  // the expert entry points take multiples of 64 only
    const dim3 grid((unsigned)((int64_t)(a.max_rows / 128 + a.n_sel) * round_up(a.N / 64, 8))), block(SG_WAVES * 64);
    if (asym)
        hipLaunchKernelGGL(stream_grouped_kernel<true>, grid, block, 0, st, a);
    else
        hipLaunchKernelGGL(stream_grouped_kernel<false>, grid, block, 0, st, a);
    HAQ_CHECK_HIP(hipGetLastError());
    return HAQ_OK;
}

}  // namespace haq
