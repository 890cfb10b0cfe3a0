// Launcher of the int8 MFMA GEMM kernel (gemm_kernel.h): picks the tile shape, sizes
// the grid and opts the kernel into its dynamic LDS size.
#include <mutex>

#include "gemm_kernel.h"

namespace haq {

namespace {

// 128 x 256 tiles, 4 waves (2 x 2, 64 x 128 each), 3-deep ring: 75 KB of LDS and at most
// 256 registers per lane, so two work-groups share a CU and fill each other's stalls.
// (The shape can be overridden at compile time to measure other tilings; the other shapes below are fixed.)
#ifndef HAQ_BM
#define HAQ_BM 128
#define HAQ_BN 256
#define HAQ_MINB 2
#define HAQ_STAGES 3
#endif
#ifndef HAQ_WAVES_M
#define HAQ_WAVES_M 2
#endif
#ifndef HAQ_WAVES_N
#define HAQ_WAVES_N 2
#endif
constexpr int BM = HAQ_BM, BN = HAQ_BN, WAVES_M = HAQ_WAVES_M, WAVES_N = HAQ_WAVES_N, STAGES = HAQ_STAGES, MINB = HAQ_MINB;
using Shape = GemmShape<BM, BN, WAVES_M, WAVES_N, STAGES>;

// Row tiles of `bm` rows: exact for one matrix; an upper bound, rows / bm plus one partial tile per group, otherwise.
int row_tiles(const GemmArgs& a, int bm) { return a.offsets ? a.max_rows / bm + a.n_sel : cdiv(a.M, bm); }
// Every launch takes its grid from the tile of its own kernel: at least the tile count, a multiple of 8.
dim3 tile_grid(const GemmArgs& a, int bm, int bn) { return dim3((unsigned)round_up((int64_t)row_tiles(a, bm) * cdiv(a.N, bn), 8)); }

template <int BM_, int BN_, int WM_, int WN_, int STAGES_, int MINB_, int EPI, bool DBG, bool FEW, bool WIDE>
int launch_tiles(const GemmArgs& a, dim3 grid, hipStream_t st) {
    using S = GemmShape<BM_, BN_, WM_, WN_, STAGES_>;
    static_assert(MINB_ * S::LDS_BYTES <= 160 * 1024, "the LDS of a CU");
    auto kern = gemm_i8_kernel<BM_, BN_, WM_, WN_, STAGES_, MINB_, EPI, DBG, FEW, WIDE>;
    static std::once_flag once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(once, [&] { attr_err = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, S::LDS_BYTES); });
    HAQ_CHECK_HIP(attr_err);
    hipLaunchKernelGGL(kern, grid, dim3(S::THREADS), S::LDS_BYTES, st, a);
    HAQ_CHECK_HIP(hipGetLastError());
    return HAQ_OK;
}

template <int EPI, bool DBG, bool FEW = false, bool WIDE = false>
int launch_one(const GemmArgs& a, hipStream_t st) {
    // FEW: an expert's channel tiles go round the XCDs (decode_tile), a multiple of 8 of them for each row tile
    const dim3 grid = FEW ? dim3((unsigned)((int64_t)row_tiles(a, BM) * round_up(cdiv(a.N, BN), 8))) : tile_grid(a, BM, BN);
    return launch_tiles<BM, BN, WAVES_M, WAVES_N, STAGES, MINB, EPI, DBG, FEW, WIDE>(a, grid, st);
}

// The other tile shapes.  Dense linears take the one that the estimate below finds fastest.
struct TileShape {
    int bm, bn, per_cu;  // tile, work-groups that a CU holds
    // Estimated us of a launch of T tiles on C compute units: c0 + per full round of per_cu C tiles (fix + K-steps step[per_cu-1][1])
    // + for a last round of rem tiles, k = ceil(rem / C) to a CU, (fix + K-steps step), step between step[k-1][0] (a CU alone)
    // and step[k-1][1] (every CU busy: the caches and the chip's power are shared) in proportion to rem / (k C).
    float c0, fix, step[2][2];
};
enum { T128x256, T128x128, T192x128, T192x256, T256x256, N_TILES };
// Fitted to 195 launches of each shape (129 to 4096 rows, 13 layers between 768 x 3072 and 16384 x 4096, weights cold; mean
// deviation 3 to 6 %).  The shape with the lowest estimate is on average 1.1 % slower than the fastest of these and four
// more (256 x 128, 128 x 256 alone on its CU, 192 x 128 and 128 x 128 with two and three to a CU); one shape fewer costs
// another 0.3 to 1.5 %.  Against the two thresholds on tile counts before (us, with the kernel before and now):
//   4096 x 16384:  333 rows 38.8 / 34.0,  600: 60 / 51,  777: 65 / 61,  2048: 124 / 118;   16384 x 4096:  777: 86 / 72,  1300: 120 / 87
//   8192 x 8192:  333: 48 / 41,  600: 71 / 52,  1300: 108 / 81,  4096: 228 / 213;   5120 x 13824:  256: 35.6 / 30.7,  1024: 79 / 66
//   4096 x 11008:  1024: 64 / 51;   2064 x 8208:  777: 25.2 / 24.6;   768 x 3072:  1024: 10.3 / 9.5
constexpr TileShape TILES[N_TILES] = {
    {128, 256, 2, 0.64f, 8.13f, {{0.369f, 0.461f}, {0.608f, 0.846f}}},
    {128, 128, 2, 1.95f, 4.77f, {{0.216f, 0.280f}, {0.421f, 0.502f}}},
    {192, 128, 1, 2.90f, 5.46f, {{0.242f, 0.340f}}},
    {192, 256, 1, 2.08f, 9.20f, {{0.402f, 0.563f}}},
    {256, 256, 1, 0.00f, 9.61f, {{0.452f, 0.745f}}},
};
float tile_us(const TileShape& t, int M, int N, int nk, int n_cu) {
    const int64_t tiles = (int64_t)cdiv(M, t.bm) * cdiv(N, t.bn), round = (int64_t)t.per_cu * n_cu;
    const int rem = (int)(tiles % round), k = cdiv(rem, n_cu);
    float us = t.c0 + (float)(tiles / round) * (t.fix + (float)nk * t.step[t.per_cu - 1][1]);
    if (rem) {
        const float* step = t.step[k - 1];
        us += t.fix + (float)nk * (step[0] + (step[1] - step[0]) * (float)rem / (float)(k * n_cu));
    }
    return us;
}
// More than half a 192- or 256-row tile would be empty on at most 128 rows.
int fastest_tile(int M, int N, int nk, int n_cu, float& us) {
    int best = 0;
    for (int i = 0; i < (M <= 128 ? T192x128 : N_TILES); ++i) {
        const float t = tile_us(TILES[i], M, N, nk, n_cu);
        if (i == 0 || t < us) us = t, best = i;
    }
    return best;
}

template <int EPI>
int launch_shape(const GemmArgs& a, int shape, hipStream_t st) {
    const dim3 grid = tile_grid(a, TILES[shape].bm, TILES[shape].bn);
    switch (shape) {
        case T128x128: return launch_tiles<128, 128, 2, 2, 4, 2, EPI, false, false, false>(a, grid, st);  // wave tile 64 x 64
        case T192x128: return launch_tiles<192, 128, 2, 2, 7, 1, EPI, false, false, false>(a, grid, st);  // 96 x 64
        case T192x256: return launch_tiles<192, 256, 2, 2, 5, 1, EPI, false, false, false>(a, grid, st);  // 96 x 128
        case T256x256: return launch_tiles<256, 256, 4, 2, 4, 1, EPI, false, false, false>(a, grid, st);  // 64 x 128, eight waves
        default: return launch_one<EPI, false>(a, st);
    }
}

// Operands whose offsets need more than 32 bits (4 GB): the tiled kernel computes its addresses in 64.
bool wide_operands(const GemmArgs& a) {
    const int64_t rows = a.R > a.Npad ? a.R : a.Npad;
    return rows > INT64_C(0xFFFFFFFF) / (64 * (int64_t)cdiv(a.K, 64));
}
template <bool DBG>
int launch_wide(const GemmArgs& a, int epi, hipStream_t st) {
    switch (epi) {
        case EPI_SWIGLU: return launch_one<EPI_SWIGLU, false, false, true>(a, st);
        case EPI_SWIGLU_ASYM: return launch_one<EPI_SWIGLU_ASYM, false, false, true>(a, st);
        case EPI_LINEAR_ASYM: return launch_one<EPI_LINEAR_ASYM, DBG, false, true>(a, st);
        default: return launch_one<EPI_LINEAR, DBG, false, true>(a, st);
    }
}

}  // namespace

// Row blocks of 16 per tile (4, 6 or 8) with which the streaming kernel (skinny.hip: 64-channel tiles, K split over
// the waves, operands straight into registers) beats the tiled kernel, whose fastest shape takes `tiled_us`, or 0.  A
// round of streaming tiles costs (4 + RB) / 80 us a K-step, the fragments of a step through a CU's load path, and
// 3.4 + RB / 5 us to start, add up and finish.  Measured (us, M rows, K x N, streaming against tiled):
//   16384 x 4096:  129 rows 30 / 78,  333: 37 / 78,  512: 44 / 79,  700: 70 / 82,  1024: 84 / 85
//   4096 x 4096:   129 rows 10 / 20,  333: 13 / 20,  512: 15 / 20,  700: 25 / 21 (tiled stays)
//   3072 x 768:    333 rows 9.4 / 15.3,  1024: 9.7 / 15.7;   2048 x 8192: 192 rows 10.3 / 13.1,  333: 18 / 13 (tiled)
// and where few K-steps leave the start and the end to decide (weights cold):
//   512 x 4096:    256 rows 7.6 / 8.5,  333: 9.2 / 8.6 (tiled);   768 x 3072: 400 rows 9.6 / 9.9,  512: 10.3 / 10.0 (tiled)
//   1024 x 4096:   512 rows 10.7 / 11.2
// Two bounds: a round of 128 x 128 tiles at 0.3 us a K-step, which keeps the tiled kernel on short K (its estimate counts
// the start of a launch, some 3 us, and the streaming tiles' terms do not), and the estimate, less what evens out where the
// two measure the same (700 rows of 16384 x 4096: 71 / 71).  300 rows of 8192 x 8192: 48 / 41 (tiled).
static int stream_row_blocks(const GemmArgs& a, int n_cu, float tiled_us) {
    const int nk = cdiv(a.K, 64);
    const float before = 3.0f + 0.3f * nk, now = tiled_us - 1.0f;
    float best = before < now ? before : now;
    int rb = 0;
    for (int r = 4; r <= 8; r += 2) {
        if (a.M <= 16 * r) break;  // a single row tile: skinny_pays has decided
        const int64_t tiles = (int64_t)cdiv(a.M, 16 * r) * cdiv(a.N, 64);
        const float t = (float)((tiles + n_cu - 1) / n_cu) * (3.4f + 0.2f * r + nk * (4 + r) * (1.0f / 80.0f));
        if (t < best) {
            best = t;
            rb = r;
        }
    }
    return rb;
}

int cu_count() {
    static const int n_cu = [] {
        int devid = 0, v = 0;
        if (hipGetDevice(&devid) == hipSuccess && hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, devid) == hipSuccess && v > 0) return v;
        return 256;
    }();
    return n_cu;
}

// Down projections of expert groups: rows per selected expert, on average, up to which the streaming kernel is taken.
// Units of 64 channels, one row tile each, are its work-groups, of which a CU holds two.  Measured on whole layers (us,
// weights cold, tokens spread evenly, then by 1 / rank^1.1; streaming / 128 x 128 tiles / FEW / many rows):
//   units 128 (1024 x 3584, 8 experts), 100 rows: 71 / 77 / 82 / 86, 75 / 82 / 86 / 92
//         256 (4096 x 14336, 4), 100: 171 / 184 / 216 / 214, 197 / 201 / 233 / 232;  (2048 x 8192, 8), 100: 124 / 135 / 147 / 151, 137 / 144 / 155 / 160
//         384 (3072 x 14336, 8), 100: 275 / 271 / 286 / 294, 308 / 341 / 312 / 321
//         448 (3584 x 8192, 8), 48: 165 / 161 / 180 / 174, 170 / 161 / 182 / 173;  76: 179 / 167 / 189 / 180, 187 / 182 / 199 / 192
//         512 (4096 x 14336, 8), 56: 289 / 295 / 306 / 317, 306 / 334 / 308 / 319;  76: 312 / 313 / 325 / 333, 333 / 347 / 320 / 332;
//              100: 318 / 316 / 328 / 338, 363 / 388 / 363 / 375
//         512 (2048 x 5632, 16), 64: 160 / 161 / 166 / 171, 177 / 184 / 172 / 179;  100: 169 / 166 / 172 / 176, 194 / 197 / 185 / 192
// More units than two for each CU: FEW, unless its own 128 x 256 tiles fill the chip and a second row tile starts a round:
//         768 (3072 x 8192, 16), 20: 238 / 265 / 241 / 255;  36: 266 / 277 / 253 / 268, 269 / 287 / 263 / 278
//         1024 (4096 x 7168, 16), 36: 294 / 297 / 290 / 297, 288 / 322 / 317 / 335;  56: 311 / 306 / 299 / 306, 331 / 352 / 349 / 364
static int stream_mean_rows(const GemmArgs& a, int n_cu) {
    const int units = a.n_sel * (a.N / 64);
    if (2 * units <= 3 * n_cu) return 112;
    if (units <= 2 * n_cu) return 64;
    return a.n_sel * cdiv(a.N, BN) >= n_cu ? 48 : 24;
}
static constexpr int FEW_MEAN_ROWS = 112;  // likewise for the form for few rows

int launch_gemm(const GemmArgs& a, int epi, hipStream_t st) {
    if (skinny_pays(a) && (epi == EPI_LINEAR || epi == EPI_LINEAR_ASYM)) return launch_skinny(a, epi == EPI_LINEAR_ASYM, st);
    if (row_tiles(a, BM) <= 0 || a.N <= 0) return HAQ_OK;
    if (wide_operands(a)) return a.acc_dbg ? launch_wide<true>(a, epi, st) : launch_wide<false>(a, epi, st);
    if (!a.offsets && !a.acc_dbg && (epi == EPI_LINEAR || epi == EPI_LINEAR_ASYM)) {
        const bool asym = epi == EPI_LINEAR_ASYM;
        const int n_cu = cu_count();
        float us = 0.0f;
        const int shape = fastest_tile(a.M, a.N, cdiv(a.K, 64), n_cu, us);
        if ((int64_t)cdiv(a.M, 128) * cdiv(a.N, 128) <= n_cu) {
            if (const int rb = stream_row_blocks(a, n_cu, us)) return launch_stream_rows(a, asym, rb, st);
        }
        return asym ? launch_shape<EPI_LINEAR_ASYM>(a, shape, st) : launch_shape<EPI_LINEAR>(a, shape, st);
    }
    if (a.offsets) {
        // Few rows per expert: bound by the weight stream, not by the matrix cores.  Gate/up, FEW / many rows, whole layers (us)
        // by rows per expert: 4096 x 14336, 8 experts: 18: 310 / 325, 32: 315 / 334, 75: 340 / 363, 112: 366 / 368, 150: 513 / 441;
        // 2048 x 5632, 16 experts: 37: 159 / 173, 75: 176 / 185.  (The streaming kernel there: 307, 327, 393; 169.)
        const int mean = a.max_rows / (a.n_sel > 0 ? a.n_sel : 1);
        const bool down = epi == EPI_LINEAR || epi == EPI_LINEAR_ASYM, asym = epi == EPI_LINEAR_ASYM;
        if (down && mean <= stream_mean_rows(a, cu_count())) return launch_stream_grouped(a, asym, st);
        // 128 x 128 tiles where they cover the groups in one round (a CU with two of them takes 1.4 times as long: 14336 x 4096,
        // 8 experts, 256 tiles 99 us, 288 tiles 137): at one row tile for each group while few have more, else by the upper bound
        const int row_tiles_s = mean <= 104 ? a.n_sel : mean <= FEW_MEAN_ROWS ? a.n_sel + cdiv(a.n_sel, 8) : row_tiles(a, 128);
        if (down && row_tiles_s * cdiv(a.N, 128) <= cu_count())
            return asym ? launch_shape<EPI_LINEAR_ASYM>(a, T128x128, st) : launch_shape<EPI_LINEAR>(a, T128x128, st);
        if (mean <= FEW_MEAN_ROWS) {
            switch (epi) {
                case EPI_SWIGLU: return launch_one<EPI_SWIGLU, false, true>(a, st);
                case EPI_SWIGLU_ASYM: return launch_one<EPI_SWIGLU_ASYM, false, true>(a, st);
                case EPI_LINEAR_ASYM: return launch_one<EPI_LINEAR_ASYM, false, true>(a, st);
                default: return launch_one<EPI_LINEAR, false, true>(a, st);
            }
        }
    }
    if (epi == EPI_SWIGLU) return launch_one<EPI_SWIGLU, false>(a, st);
    if (epi == EPI_SWIGLU_ASYM) return launch_one<EPI_SWIGLU_ASYM, false>(a, st);
    if (epi == EPI_LINEAR_ASYM) return a.acc_dbg ? launch_one<EPI_LINEAR_ASYM, true>(a, st) : launch_one<EPI_LINEAR_ASYM, false>(a, st);
    if (a.acc_dbg) return launch_one<EPI_LINEAR, true>(a, st);
    return launch_one<EPI_LINEAR, false>(a, st);
}

}  // namespace haq
