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

template <int EPI, bool DBG, bool FEW = false>
int launch_one(const GemmArgs& a, hipStream_t st) {
    // FEW: an expert's channel tiles go round the XCDs (decode_tile), a multiple of 8 of them for each row tile
    const dim3 grid = FEW ? dim3((unsigned)((int64_t)row_tiles(a, BM) * round_up(cdiv(a.N, BN), 8))) : tile_grid(a, BM, BN);
    auto kern = gemm_i8_kernel<BM, BN, WAVES_M, WAVES_N, STAGES, MINB, EPI, DBG, FEW>;
    static std::once_flag once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(once, [&] {
        attr_err = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, Shape::LDS_BYTES);
    });
    HAQ_CHECK_HIP(attr_err);
    hipLaunchKernelGGL(kern, grid, dim3(Shape::THREADS), Shape::LDS_BYTES, st, a);
    HAQ_CHECK_HIP(hipGetLastError());
    return HAQ_OK;
}

// 128 x 128 tiles (wave tile 64 x 64) for problems whose 128 x 256 tiling would leave half of the
// work-group slots empty: twice the tiles, 49 KB of LDS, three work-groups per CU.
#ifndef HAQ_SMALL_TILE_LIMIT
#define HAQ_SMALL_TILE_LIMIT 256
#endif
constexpr int SMALL_TILE_LIMIT = HAQ_SMALL_TILE_LIMIT;  // 128 x 256 tiles that would not even give every CU one work-group
constexpr int BN_S = 128, MINB_S = 3;
using ShapeS = GemmShape<128, BN_S, 2, 2, 3>;
template <int EPI>
int launch_small(const GemmArgs& a, hipStream_t st) {
    auto kern = gemm_i8_kernel<128, BN_S, 2, 2, 3, MINB_S, EPI, false>;
    static std::once_flag once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(once, [&] {
        attr_err = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, ShapeS::LDS_BYTES);
    });
    HAQ_CHECK_HIP(attr_err);
    hipLaunchKernelGGL(kern, tile_grid(a, 128, BN_S), dim3(ShapeS::THREADS), ShapeS::LDS_BYTES, st, a);
    HAQ_CHECK_HIP(hipGetLastError());
    return HAQ_OK;
}

// 256 x 256 tiles, 8 waves (4 x 2, the same 64 x 128 wave tile and per-wave code as the main shape), one
// work-group per CU: a third fewer direct-to-LDS bytes per matrix instruction, which is what limits the K loop.
// For dense problems with at least two full rounds of such tiles (one per CU and round); measured +3 % on
// 2048..8192 x 4096 x 16384, -8 % on a single round, and slower on ragged expert groups (more padding rows).
constexpr int LARGE_TILE_MIN = 512;
using ShapeL = GemmShape<256, 256, 4, 2, 3>;
template <int EPI>
int launch_large(const GemmArgs& a, hipStream_t st) {
    auto kern = gemm_i8_kernel<256, 256, 4, 2, 3, 1, EPI, false>;
    static std::once_flag once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(once, [&] {
        attr_err = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, ShapeL::LDS_BYTES);
    });
    HAQ_CHECK_HIP(attr_err);
    hipLaunchKernelGGL(kern, tile_grid(a, 256, 256), dim3(ShapeL::THREADS), ShapeL::LDS_BYTES, st, a);
    HAQ_CHECK_HIP(hipGetLastError());
    return HAQ_OK;
}

// 256 x 128 tiles, 8 waves (4 x 2 of 64 x 64), one work-group per CU: for dense problems that this tiling covers in
// one round with most CUs busy (fc2 of the OPT-6.7B block: 8 x 32 tiles on 256 CUs).  A quarter fewer
// direct-to-LDS bytes per matrix instruction than the 128 x 128 shape such problems would otherwise take: -2 %.
// Not for 128 rows and fewer, of which the tile would waste half: 64 rows of 512 x 32768 10.2 us instead of 10.8.
using ShapeT = GemmShape<256, 128, 4, 2, 3>;
template <int EPI>
int launch_tall(const GemmArgs& a, hipStream_t st) {
    auto kern = gemm_i8_kernel<256, 128, 4, 2, 3, 1, EPI, false>;
    static std::once_flag once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(once, [&] {
        attr_err = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, ShapeT::LDS_BYTES);
    });
    HAQ_CHECK_HIP(attr_err);
    hipLaunchKernelGGL(kern, tile_grid(a, 256, 128), dim3(ShapeT::THREADS), ShapeT::LDS_BYTES, st, a);
    HAQ_CHECK_HIP(hipGetLastError());
    return HAQ_OK;
}

}  // namespace

// Row blocks of 16 per tile (4, 6 or 8) with which the streaming kernel (skinny.hip: 64-channel tiles, K split over
// the waves, operands straight into registers) beats one round of 128 x 128 tiles, or 0.  Such a round costs a
// work-group 0.3 us for each 64-byte K-step however few of them there are (77 us at K = 16384 for 64 to 256 tiles);
// a round of streaming tiles costs (4 + RB) / 80 us a K-step, the fragments of a step through a CU's load path, and
// 3.4 + RB / 5 us to start, add up and finish.  Measured (us, M rows, K x N, streaming against tiled):
//   16384 x 4096:  129 rows 30 / 78,  333: 37 / 78,  512: 44 / 79,  700: 70 / 82,  1024: 84 / 85
//   4096 x 4096:   129 rows 10 / 20,  333: 13 / 20,  512: 15 / 20,  700: 25 / 21 (tiled stays)
//   3072 x 768:    333 rows 9.4 / 15.3,  1024: 9.7 / 15.7;   2048 x 8192: 192 rows 10.3 / 13.1,  333: 18 / 13 (tiled)
// and where few K-steps leave the start and the end to decide (weights cold):
//   512 x 4096:    256 rows 7.6 / 8.5,  333: 9.2 / 8.6 (tiled);   768 x 3072: 400 rows 9.6 / 9.9,  512: 10.3 / 10.0 (tiled)
//   1024 x 4096:   512 rows 10.7 / 11.2
static int stream_row_blocks(const GemmArgs& a, int n_cu) {
    const int nk = cdiv(a.K, 64);
    float best = 3.0f + 0.3f * nk;
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
    const int ntn = cdiv(a.N, BN);
    const int mt = row_tiles(a, BM);
    if (mt <= 0 || ntn <= 0) return HAQ_OK;
    if (!a.offsets && !a.acc_dbg && (epi == EPI_LINEAR || epi == EPI_LINEAR_ASYM)) {
        const bool asym = epi == EPI_LINEAR_ASYM;
        const int n_cu = cu_count();
        const int64_t tiles_l = (int64_t)cdiv(a.M, 256) * cdiv(a.N, 256);
        if (tiles_l >= LARGE_TILE_MIN) return asym ? launch_large<EPI_LINEAR_ASYM>(a, st) : launch_large<EPI_LINEAR>(a, st);
        const int64_t tiles_s = (int64_t)cdiv(a.M, 128) * cdiv(a.N, BN_S);
        if (tiles_s <= n_cu) {
            if (const int rb = stream_row_blocks(a, n_cu)) return launch_stream_rows(a, asym, rb, st);
        }
        const int64_t tiles_t = (int64_t)cdiv(a.M, 256) * cdiv(a.N, 128);
        if (a.M > 128 && tiles_t <= n_cu && 4 * tiles_t > 3 * n_cu) return asym ? launch_tall<EPI_LINEAR_ASYM>(a, st) : launch_tall<EPI_LINEAR>(a, st);
        if (mt * ntn <= SMALL_TILE_LIMIT) return asym ? launch_small<EPI_LINEAR_ASYM>(a, st) : launch_small<EPI_LINEAR>(a, st);
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
        if (down && row_tiles_s * cdiv(a.N, BN_S) <= cu_count()) return asym ? launch_small<EPI_LINEAR_ASYM>(a, st) : launch_small<EPI_LINEAR>(a, st);
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
