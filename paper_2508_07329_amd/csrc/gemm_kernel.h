// int8 x int8 -> int32 GEMM kernel for the gfx950 matrix cores with the dequantise /
// activation epilogue (Eq. 1 evaluated at run time: Q(s^-1 X) . Q(W s), scales on the
// token and output-channel dimensions), for one matrix or for expert groups over rows
// sorted by expert.
//
// Data flow of a work-group (BM x BN output tile, WAVES_M x WAVES_N waves):
//   HBM/L2 --buffer_load ... lds (16 B/lane, no VGPR staging)--> LDS ring of STAGES K-steps
//   (64 bytes of k each) --ds_read_b128--> fragment registers, half a K-step ahead
//   --> v_mfma_i32_32x32x32_i8 (16 bytes of k per lane per operand).
// Both operands are chunk-major ([K/16][rows][16]), so a K-step of a tile is four
// contiguous row segments per operand, lands in LDS in fragment order and is read back
// without bank conflicts.  One raw s_barrier per K-step.  The product is formed
// transposed (weights as first operand) so that a lane owns four consecutive output
// channels; the epilogue dequantises, applies the activation, stages fp16 rows in LDS
// and writes 16 bytes per lane.
//
// What bounds the K loop: a matrix instruction holds its pipe for 32 cycles, and a wave issues in order, so whatever
// stands between two of them and takes longer stops the pipe.  A K-step of a 128 x 128 tile, whose matrix instructions
// take 256 cycles, took 550 on a CU of its own (128 x 256: 963 for 512; 256 x 256: 1450 for 1024), however deep the ring
// and with every load served by L2: the loads stood in a block behind the barrier, each with its scalar address
// arithmetic, and every LDS read was waited for in front of it.  With one load or one read behind a matrix instruction,
// loads whose address costs nothing but the write of m0, and reads half a K-step ahead it takes 385 (655, 1170); what is
// left over the matrix instructions, some 140 cycles for any tile, is the barrier and the instructions around it.
// Whole launches (us, weights cold): 2048 x 4096 x 16384 122 -> 115, 2048 x 16384 x 4096 126 -> 118, 4096 x 8192 x 8192
// 228 -> 213: from some 2.4 POP/s on the chip's power management slows the clock (1.6 GHz under nothing but matrix
// instructions and LDS reads).
#pragma once
#include "group_tiles.h"
#include "haq_common.h"

#include <type_traits>

namespace haq {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

// s_waitcnt immediates (gfx9 encoding): vmcnt in bits [3:0] and [15:14], lgkmcnt in [11:8]
#define HAQ_WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt(((n) & 0xF) | (((n) >> 4) << 14) | (0x7 << 4) | (0xF << 8))
#define HAQ_WAIT_LGKM0() __builtin_amdgcn_s_waitcnt(0xF | (0x3 << 14) | (0x7 << 4) | (0x0 << 8))
#define HAQ_CFENCE() asm volatile("" ::: "memory")

// Buffer resources: the address of a lane's 16 bytes is a scalar base, a lane offset and a scalar offset, 32 bits each
// but the base, and only the scalar offset changes with the K-step; a lane whose offset lies past the resource's bytes
// fetches nothing and gets zeros.  (The builtins exist on the device side only.)
#ifdef __HIP_DEVICE_COMPILE__
typedef __amdgpu_buffer_rsrc_t BufferRsrc;
__device__ __forceinline__ BufferRsrc buffer_rsrc(const int8_t* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, bytes, 0x00027000);
}
template <int AUX>
__device__ __forceinline__ void buffer_to_lds(BufferRsrc r, int8_t* to, uint32_t lane_off, uint32_t off) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)to, 16, lane_off, off, 0, AUX);
}
#else
typedef const int8_t* BufferRsrc;
__device__ __forceinline__ BufferRsrc buffer_rsrc(const int8_t* p, uint32_t) { return p; }
template <int AUX>
__device__ __forceinline__ void buffer_to_lds(BufferRsrc, int8_t*, uint32_t, uint32_t) {}
#endif

// How a launch fetches its operands.
enum {
    FETCH_PLAIN = 0,
    FETCH_WIDE = 1,   // offsets of 64 bits: operands of 4 GB and more
    FETCH_ONCE = 2,   // weights that hardly any other tile reads pass the caches by (non-temporal)
};
constexpr uint32_t PAST_END = 0xFFFF0000u;  // an offset past every resource's bytes

struct TileCoord {
    int m0;     // first (sorted) row of the tile
    int m_end;  // one past the last valid row (end of the group)
    int n0;     // first packed output channel of the tile
    int e;      // expert (0 for a single matrix)
    bool valid;
};

// Work-group id -> tile.  The hardware deals work-group ids round-robin to the 8 XCDs;
// undo that so that each XCD (one L2) owns a contiguous range of tile ids, M fastest:
// neighbouring work-groups of an XCD share weight tiles and the activation tiles stay in
// its L2.  The grid is a multiple of 8 and at least the tile count.
#ifndef HAQ_TILE_BAND
#define HAQ_TILE_BAND 8
#endif
constexpr int TILE_BAND = HAQ_TILE_BAND;

template <int BM, int BN, bool FEW>
__device__ __forceinline__ TileCoord decode_tile(const GemmArgs& a) {
    TileCoord tc;
    tc.valid = false;
    tc.e = 0;
    tc.m0 = tc.m_end = tc.n0 = 0;
    const int ntn = (a.N + BN - 1) / BN;
    if constexpr (FEW) {
        const GroupLanes g(a);
        GroupTile t;
        if (g.template deal<BM>(a, ntn, t)) {
            tc.e = g.of(g.e, t.i);
            tc.m0 = g.of(g.lo, t.i) + t.mi * BM;
            tc.m_end = g.of(g.hi, t.i);
            tc.n0 = t.u * BN;
            tc.valid = true;
        }
        return tc;  // the grid is an upper bound
    }
    int total_mt = 0;
    if (!a.offsets) {
        total_mt = (a.M + BM - 1) / BM;
    } else {
        for (int i = 0; i < a.n_sel; ++i) {
            const int e = a.sel[i];
            total_mt += (a.offsets[e + 1] - a.offsets[e] + BM - 1) / BM;
        }
    }
    const int total = total_mt * ntn;
    const int per = (total + 7) / 8;
    const int xcd = blockIdx.x % 8, slot = blockIdx.x / 8;
    if (slot >= per) return tc;
    const int id = xcd * per + slot;
    if (id >= total) return tc;
    // bands of TILE_BAND row tiles, channel tiles inside a band, rows fastest: the
    // work-groups resident on one XCD at a time then form a compact block of the tile grid
    // (a row tile's activations and a channel tile's weights are each shared by ~8 of them
    // in L2) instead of one channel tile across every row tile of every expert
    // (256-row tiles: bands of 4, the same 1024 rows; with one work-group per CU an XCD then holds 4 x 8 tiles)
    constexpr int BAND = BM >= 256 ? TILE_BAND / 2 : TILE_BAND;
    const int band = id / (BAND * ntn), rem = id % (BAND * ntn);
    const int band_rows = min(BAND, total_mt - band * BAND);
    int mi = band * BAND + rem % band_rows;
    tc.n0 = (rem / band_rows) * BN;
    if (!a.offsets) {
        tc.m0 = mi * BM;
        tc.m_end = a.M;
        tc.valid = true;
        return tc;
    }
    for (int i = 0; i < a.n_sel; ++i) {
        const int e = a.sel[i];
        const int lo = a.offsets[e], hi = a.offsets[e + 1];
        const int mt = (hi - lo + BM - 1) / BM;
        if (mi < mt) {
            tc.e = e;
            tc.m0 = lo + mi * BM;
            tc.m_end = hi;
            tc.valid = true;
            return tc;
        }
        mi -= mt;
    }
    return tc;
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int STAGES>
struct GemmShape {
    static constexpr int NW = WAVES_M * WAVES_N;
    static constexpr int THREADS = NW * 64;
    static constexpr int STAGE_BYTES = (BM + BN) * 64;
    static constexpr int SCALE_BYTES = (BM + 2 * BN) * 4;  // row scales, channel scales and (asymmetric codes) column sums of the tile
    static constexpr int LDS_BYTES = STAGES * STAGE_BYTES + SCALE_BYTES;
};

template <int BM, int BN, int WAVES_M, int WAVES_N, int STAGES, int MINB, int EPI, bool DBG, bool FEW = false, int FETCH = FETCH_PLAIN>
__global__ __launch_bounds__(WAVES_M * WAVES_N * 64, MINB) void gemm_i8_kernel(GemmArgs a) {
    using S = GemmShape<BM, BN, WAVES_M, WAVES_N, STAGES>;
    constexpr int NW = S::NW;
    constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;  // wave tile
    constexpr int MI = WM / 32, NI = WN / 32;
    constexpr int STAGE_BYTES = S::STAGE_BYTES;
    constexpr int GA = 4 * BM / 64, GB = 4 * BN / 64;  // 1 KB (64 rows x 16 B) load groups per K-step
    constexpr int LPW = (GA + GB) / NW;                // direct-to-LDS loads per wave per K-step
    static_assert(GA % NW == 0 && GB % NW == 0, "a load slot is of one operand for all waves");
    static_assert(LPW * STAGES <= 63, "s_waitcnt counts the loads of a whole ring");
    // a tile's loads cover BM rows and BN channels whatever the problem size: the packed operands are padded for that
    static_assert(NPAD % BN == 0, "a channel tile must not reach past the padded width of the packed weights");
    static_assert(BM <= 256, "packed activations carry 256 rows of padding");
    constexpr bool WIDE = FETCH == FETCH_WIDE;
    constexpr bool SWIGLU = EPI == EPI_SWIGLU || EPI == EPI_SWIGLU_ASYM;
    constexpr bool ASYM = EPI == EPI_LINEAR_ASYM || EPI == EPI_SWIGLU_ASYM;
    static_assert(!SWIGLU || NI % 2 == 0, "gate/up blocks come in pairs");
    constexpr int OUT_WN = SWIGLU ? WN / 2 : WN;  // output channels per wave tile
    // staged fp16 row pitch in bytes: 2 (mod 64) dwords, so the 8-byte pieces that the 32 rows of a half-wave
    // write land in 32 different bank pairs (a pitch of 4 (mod 64) dwords costs 6 conflict cycles per write)
    constexpr int PITCH = OUT_WN * 2 + 8;
    static_assert(32 * PITCH * NW <= STAGES * STAGE_BYTES, "epilogue staging must fit in the ring");
    extern __shared__ __attribute__((aligned(1024))) int8_t lds[];
    float* sx_s = reinterpret_cast<float*>(lds + STAGES * STAGE_BYTES);  // [BM] row scales of the tile
    float* sw_s = sx_s + BM;                                             // [BN] channel scales, packed order
    int32_t* cs_s = reinterpret_cast<int32_t*>(sw_s + BN);               // [BN] column sums of the weight codes, packed order (ASYM)

    const TileCoord tc = decode_tile<BM, BN, FEW>(a);
    if (!tc.valid) return;

    const int8_t* Bmat = a.B;
    const float* sw_a = a.sw;
    const float* sw_b = nullptr;
    const int32_t* cs_a = a.colsum;  // column sums of the weight codes (asymmetric activation codes only)
    const int32_t* cs_b = nullptr;
    if (a.offsets) {
        const ExpertTab& t = a.tab[tc.e];
        if (a.which == 0) {
            Bmat = t.w13;
            sw_a = t.sw1;
            sw_b = t.sw3;
        } else {
            Bmat = t.w2;
            sw_a = t.sw2;
        }
        if (ASYM) {
            const ColsumTab& c = a.cstab[tc.e];
            cs_a = a.which == 0 ? c.cs1 : c.cs2;
            cs_b = c.cs3;
        }
    }

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;
    const int nkt = (a.K + 63) / 64;  // a last partial k-step reads chunks past K: the weight operand is zero there

    // tile scales into LDS (consumed only by the epilogue)
    for (int i = tid; i < BM; i += S::THREADS) {
        const int row = tc.m0 + i;
        sx_s[i] = row < tc.m_end ? a.sx[row] : 0.0f;
    }
    for (int i = tid; i < BN; i += S::THREADS) {
        const int pc = tc.n0 + i;
        float v = 0.0f;
        int cs = 0;
        if (pc < a.N) {
            if (SWIGLU) {
                const int col = (pc / 64) * 32 + (pc % 32);
                v = ((pc / 32) & 1) ? sw_b[col] : sw_a[col];
                if (ASYM) cs = ((pc / 32) & 1) ? cs_b[col] : cs_a[col];
            } else {
                v = sw_a[pc];
                if (ASYM) cs = cs_a[pc];
            }
        }
        sw_s[i] = v;
        if (ASYM) cs_s[i] = cs;
    }

    // Direct-to-LDS loads: group g = wave + i*NW covers 64 rows of one 16-byte chunk.  The tile's origin in either operand
    // is the same for all lanes of the wave (the tile coordinates and the expert's matrix come out of memory and are made
    // wave-uniform explicitly).
    auto uniform_ptr = [](const int8_t* p) {
        const uint64_t v = (uint64_t)(uintptr_t)p;
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
        return (const int8_t*)(uintptr_t)(((uint64_t)hi << 32) | lo);
    };
    const int m0u = __builtin_amdgcn_readfirstlane(tc.m0), n0u = __builtin_amdgcn_readfirstlane(tc.n0);
    const int8_t* Au = uniform_ptr(a.A);
    const int8_t* Bu = uniform_ptr(Bmat);
    const int8_t* Ag = Au + (size_t)m0u * 16;
    const int8_t* Bg = Bu + (size_t)n0u * 16;
    using Off = std::conditional_t<WIDE, size_t, uint32_t>;
    uint32_t bytes_a = (uint32_t)(((size_t)nkt * 4 * a.R - m0u) * 16), bytes_b = PAST_END;  // of the buffer resources
    const Off step_a = (Off)4 * a.R * 16, step_b = (Off)4 * a.Npad * 16;
    Off off[LPW];  // of this lane's 16 bytes from the tile's origin, at K-step 0
#pragma unroll
    for (int i = 0; i < LPW; ++i) {
        const int g = wave + i * NW;
        if (i * NW < GA) {
            const int row = g % (BM / 64) * 64 + lane;
            off[i] = ((Off)(g / (BM / 64)) * a.R + row) * 16;
            if (!WIDE && m0u + row >= tc.m_end) off[i] = PAST_END;  // a row past the last one: its results are dropped
        } else {
            const int g2 = g - GA;
            off[i] = ((Off)(g2 / (BN / 64)) * a.Npad + g2 % (BN / 64) * 64 + lane) * 16;
        }
    }
    // FEW: for a group's second row tile too (cached from there on: two experts of 256 rows of 4096 x 14336 172 -> 188 us
    // a layer, eight of 10 to 183 rows 364 -> 363)
    constexpr int NT = FEW || FETCH == FETCH_ONCE ? 2 : 0;
    Off next_a = 0, next_b = 0;  // of the next K-step to request
    auto load = [&](int buf, int i) __attribute__((always_inline)) {
        int8_t* to = lds + buf * STAGE_BYTES + (wave + i * NW) * 1024;
        if constexpr (WIDE) {
            const int8_t* src = i * NW < GA ? Ag + next_a + off[i] : Bg + next_b + off[i];
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(uintptr_t)src,
                                             (__attribute__((address_space(3))) void*)to, 16, 0, 0);
        } else if (i * NW < GA) {
            buffer_to_lds<0>(buffer_rsrc(Ag, bytes_a), to, off[i], next_a);
        } else {
            buffer_to_lds<NT>(buffer_rsrc(Bg, bytes_b), to, off[i], next_b);
        }
    };
    // K-step kt has been requested.  Past the last one the loads go on, into stages that nobody reads any more, so that every
    // K-step is the same code and the same count for s_waitcnt; their resources are empty then and nothing is fetched
    // (with the last K-step requested again 2339 rows of 720 x 6464 took 24.3 us instead of 23.4).  64-bit offsets: it is.
    auto advance = [&](int kt) __attribute__((always_inline)) {
        const bool more = kt + 1 < nkt;
        next_a = more ? next_a + step_a : WIDE ? next_a : 0;  // (0: nothing is in range of an empty resource at scalar offset 0)
        next_b = more ? next_b + step_b : WIDE ? next_b : 0;
        if (!more) bytes_a = bytes_b = 0;
    };

    v16i acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;

    // fragment address inside a stage: chunk = 2*half + lane/32, row = wave base + 32*tile + lane%32
    const int frag_a = ((lane >> 5) * BM + wm * WM + (lane & 31)) * 16;
    const int frag_b = BM * 64 + ((lane >> 5) * BN + wn * WN + (lane & 31)) * 16;
    v4i fa[2][MI], fb[2][NI];  // fragments of either half (32 bytes of k) of a K-step

    // The matrix instructions on half KK of a K-step; behind them, one at a time, the LDS reads of the next half (half
    // 1 - KK of stage `rbuf`) and, spread over both halves, the loads into stage `lbuf`.
    auto half = [&](auto kk, auto reads, auto loads, int rbuf, int lbuf) __attribute__((always_inline)) {
        constexpr int KK = decltype(kk)::value, M = MI * NI, R = MI + NI;
        static_assert(M >= R, "one read behind each of the first matrix instructions");
        const int8_t* sb = lds + rbuf * STAGE_BYTES;
#pragma unroll
        for (int m = 0; m < M; ++m) {
            // channel block outermost: consecutive MFMAs keep the weight fragment and change the (fewer)
            // token fragments -- measured 2.4 % faster than the other nesting on 64 x 128 wave tiles
            const int j = m / MI, i = m % MI;
            acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fb[KK][j], fa[KK][i], acc[i][j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (decltype(reads)::value) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    if (r != m) continue;
                    if (r < NI)
                        fb[1 - KK][r] = *reinterpret_cast<const v4i*>(sb + frag_b + ((1 - KK) * 2 * BN + r * 32) * 16);
                    else
                        fa[1 - KK][r - NI] = *reinterpret_cast<const v4i*>(sb + frag_a + ((1 - KK) * 2 * BM + (r - NI) * 32) * 16);
                }
            }
            if (decltype(loads)::value) {
#pragma unroll
                for (int l = 0; l < LPW; ++l)
                    if ((2 * l + 1) * M / LPW == (1 - KK) * M + m) load(lbuf, l);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    using H0 = std::integral_constant<int, 0>;
    using H1 = std::integral_constant<int, 1>;
    using Yes = std::true_type;
    using No = std::false_type;

    // prologue: request every stage (K-steps 0..STAGES-1); K-step 0 landed -> the first half of it
#pragma unroll
    for (int s = 0; s < STAGES; ++s) {
#pragma unroll
        for (int i = 0; i < LPW; ++i) load(s, i);
        advance(s);
    }
    HAQ_WAIT_VMCNT(LPW * (STAGES - 1));
    HAQ_CFENCE();
    __builtin_amdgcn_s_barrier();
    HAQ_CFENCE();
#pragma unroll
    for (int i = 0; i < MI; ++i) fa[0][i] = *reinterpret_cast<const v4i*>(lds + frag_a + i * 32 * 16);
#pragma unroll
    for (int j = 0; j < NI; ++j) fb[0][j] = *reinterpret_cast<const v4i*>(lds + frag_b + j * 32 * 16);
    half(H0{}, Yes{}, No{}, 0, 0);

    // iteration kt: the second half of K-step kt and the first of kt+1 (registers), the LDS reads of K-step kt+1, the
    // loads of K-step kt+STAGES into the stage that K-step kt has left.
    int cur = 0;
    for (int kt = 0; kt + 1 < nkt; ++kt) {
        const int nxt = cur + 1 >= STAGES ? 0 : cur + 1;
        // K-step kt+1 has landed for this wave and its reads of K-step kt (issued with the half before) are complete;
        // after the barrier that holds for every wave, so the stage of K-step kt may be overwritten.
        HAQ_WAIT_VMCNT(LPW * (STAGES - 2));
        HAQ_WAIT_LGKM0();
        HAQ_CFENCE();
        __builtin_amdgcn_s_barrier();
        HAQ_CFENCE();
        __builtin_amdgcn_sched_barrier(0);
        half(H1{}, Yes{}, Yes{}, nxt, cur);
        half(H0{}, Yes{}, Yes{}, nxt, cur);
        advance(kt + STAGES);
        cur = nxt;
    }
    half(H1{}, No{}, No{}, 0, 0);

    // ---- epilogue.  Lane l, register r of acc[i][j] holds token row i*32 + l%32 and packed
    // channel j*32 + 8*(r/4) + 4*(l/32) + r%4 of the wave tile.
    HAQ_WAIT_VMCNT(0);  // the loads past the last K-step
    HAQ_WAIT_LGKM0();
    HAQ_CFENCE();
    __builtin_amdgcn_s_barrier();  // all reads and writes of the ring are complete: it becomes the staging area
    HAQ_CFENCE();
    int8_t* stage = lds + wave * (32 * PITCH);  // private to the wave, 32 rows at a time
    const int m_l = lane & 31, n_l = (lane >> 5) * 4;
    constexpr int LANES_PER_ROW = OUT_WN * 2 / 16;
    constexpr int ROWS_PER_IT = 64 / LANES_PER_ROW;
    const int out_n = SWIGLU ? a.N / 2 : a.N;
    const int out_n0 = SWIGLU ? (tc.n0 + wn * WN) / 2 : tc.n0 + wn * WN;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const int rloc = wm * WM + i * 32 + m_l;
        const float sx = sx_s[rloc];
        int zshift = 0;  // 128 - zero point of this lane's token row (asymmetric codes only)
        if (ASYM) zshift = (tc.m0 + rloc < tc.m_end) ? 128 - a.zp[tc.m0 + rloc] : 0;
        if (!SWIGLU) {
#pragma unroll
            for (int j = 0; j < NI; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int nloc = j * 32 + 8 * q + n_l;
                    const float4 sw = *reinterpret_cast<const float4*>(sw_s + wn * WN + nloc);
                    const float swv[4] = {sw.x, sw.y, sw.z, sw.w};
                    int csv[4] = {0, 0, 0, 0};
                    if (ASYM) {
                        const int4 c4 = *reinterpret_cast<const int4*>(cs_s + wn * WN + nloc);
                        csv[0] = c4.x, csv[1] = c4.y, csv[2] = c4.z, csv[3] = c4.w;
                    }
                    __half hv[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        int v = acc[i][j][4 * q + e];
                        if (ASYM) v += zshift * csv[e];  // channels past N hold column sum 0
                        if (DBG) {
                            const int row = tc.m0 + rloc, col = tc.n0 + wn * WN + nloc + e;
                            if (row < tc.m_end && col < a.N) a.acc_dbg[(size_t)row * a.N + col] = v;
                        }
                        float f = dequant(v, sx, swv[e]);
                        if (a.act == HAQ_ACT_RELU) f = fmaxf(f, 0.0f);
                        hv[e] = f2h(f);
                    }
                    *reinterpret_cast<uint2*>(stage + m_l * PITCH + nloc * 2) = *reinterpret_cast<const uint2*>(hv);
                }
        } else {
#pragma unroll
            for (int j = 0; j < NI; j += 2)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int nloc = j * 32 + 8 * q + n_l;  // packed channel of the gate value
                    const float4 s1 = *reinterpret_cast<const float4*>(sw_s + wn * WN + nloc);
                    const float4 s3 = *reinterpret_cast<const float4*>(sw_s + wn * WN + nloc + 32);
                    const float s1v[4] = {s1.x, s1.y, s1.z, s1.w}, s3v[4] = {s3.x, s3.y, s3.z, s3.w};
                    int c1v[4] = {0, 0, 0, 0}, c3v[4] = {0, 0, 0, 0};
                    if (ASYM) {
                        const int4 c1 = *reinterpret_cast<const int4*>(cs_s + wn * WN + nloc);
                        const int4 c3 = *reinterpret_cast<const int4*>(cs_s + wn * WN + nloc + 32);
                        c1v[0] = c1.x, c1v[1] = c1.y, c1v[2] = c1.z, c1v[3] = c1.w;
                        c3v[0] = c3.x, c3v[1] = c3.y, c3v[2] = c3.z, c3v[3] = c3.w;
                    }
                    __half hv[4];
                    const int oloc = (j / 2) * 32 + 8 * q + n_l;  // output channel inside the wave tile
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        int ag = acc[i][j][4 * q + e], au = acc[i][j + 1][4 * q + e];
                        if (ASYM) {
                            ag += zshift * c1v[e];
                            au += zshift * c3v[e];
                        }
                        const float g = dequant(ag, sx, s1v[e]);
                        const float u = dequant(au, sx, s3v[e]);
                        hv[e] = f2h(silu(g) * u);
                    }
                    *reinterpret_cast<uint2*>(stage + m_l * PITCH + oloc * 2) = *reinterpret_cast<const uint2*>(hv);
                }
        }
        // the staging area is private to the wave and LDS serves one wave's requests in order
        HAQ_CFENCE();
#pragma unroll
        for (int it = 0; it < 32 / ROWS_PER_IT; ++it) {
            const int r2 = it * ROWS_PER_IT + lane / LANES_PER_ROW;
            const int c8 = (lane % LANES_PER_ROW) * 8;
            const int orow = tc.m0 + wm * WM + i * 32 + r2, ocol = out_n0 + c8;
            const uint2 v0 = *reinterpret_cast<const uint2*>(stage + r2 * PITCH + c8 * 2);  // rows are 8-byte aligned
            const uint2 v1 = *reinterpret_cast<const uint2*>(stage + r2 * PITCH + c8 * 2 + 8);
            const uint4 v = make_uint4(v0.x, v0.y, v1.x, v1.y);
            if (orow < tc.m_end && ocol < out_n) *reinterpret_cast<uint4*>(a.Y + (size_t)orow * a.ldy + ocol) = v;
        }
        HAQ_CFENCE();
    }
}

}  // namespace haq
