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

// Row tiles of `bm` rows: exact for one matrix; an upper bound, rows / bm plus one partial tile per group, otherwise.
int row_tiles(const GemmArgs& a, int bm) { return a.offsets ? a.max_rows / bm + a.n_sel : cdiv(a.M, bm); }
// Every launch takes its grid from the tile of its own kernel: at least the tile count, a multiple of 8.
dim3 tile_grid(const GemmArgs& a, int bm, int bn) { return dim3((unsigned)round_up((int64_t)row_tiles(a, bm) * cdiv(a.N, bn), 8)); }

template <int BM_, int BN_, int WM_, int WN_, int STAGES_, int MINB_, int EPI, bool DBG, bool FEW, int FETCH>
int launch_tiles(const GemmArgs& a, dim3 grid, hipStream_t st) {
    using S = GemmShape<BM_, BN_, WM_, WN_, STAGES_>;
    static_assert(MINB_ * S::LDS_BYTES <= 160 * 1024, "the LDS of a CU");
    auto kern = gemm_i8_kernel<BM_, BN_, WM_, WN_, STAGES_, MINB_, EPI, DBG, FEW, FETCH>;
    static std::once_flag once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(once, [&] { attr_err = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, S::LDS_BYTES); });
    HAQ_CHECK_HIP(attr_err);
    hipLaunchKernelGGL(kern, grid, dim3(S::THREADS), S::LDS_BYTES, st, a);
    HAQ_CHECK_HIP(hipGetLastError());
    return HAQ_OK;
}

template <int EPI, bool DBG, bool FEW = false, int FETCH = FETCH_PLAIN>
int launch_one(const GemmArgs& a, hipStream_t st) {
    // FEW: an expert's channel tiles go round the XCDs (decode_tile), a multiple of 8 of them for each row tile
    const dim3 grid = FEW ? dim3((unsigned)((int64_t)row_tiles(a, BM) * round_up(cdiv(a.N, BN), 8))) : tile_grid(a, BM, BN);
    return launch_tiles<BM, BN, WAVES_M, WAVES_N, STAGES, MINB, EPI, DBG, FEW, FETCH>(a, grid, st);
}

// The other tile shapes.  Dense linears take the one that the estimate below finds fastest.
struct TileShape {
    int bm, bn, per_cu;  // tile, work-groups that a CU holds
    // Estimated us of a launch of T tiles on C compute units.  A round is per_cu C tiles; one of n tiles, k = ceil(n / C) to a
    // CU, takes fix + K-steps step: fix between fix[0] and fix[1] in proportion to n / (per_cu C), step between step[k-1][0] (a
    // CU alone) and step[k-1][1] (every CU busy: the caches and the chip's power are shared) in proportion to n / (k C).  Full
    // rounds before the last one overlap (`round` of that each); the last one costs its share of a full round and, as far as
    // `tail` goes, what it takes alone.
    float fix[2], step[3][2], round, tail;
};
enum { T128x256, T128x128, T128x128x3, T192x128, T192x256, T256x128, T256x256, N_TILES };  // x3: three work-groups to a CU
// Fitted to 1313 launches of each shape (129 to 4200 rows, layers of 64 to 16384 input and 256 to 28000 output channels, 300 of
// them near whole rounds of one of the shapes; weights cold; mean deviation 3 to 5 %; `round` held to 0.85 and more, below which
// one nearly full round of long K was overestimated by 16 %).  The shape with the lowest estimate is on average 0.6 % slower than the
// fastest of these and the streaming tiles; without 256 x 128 1.2 %, without 128 x 128 thrice to a CU either 1.8 %.
// Against two thresholds on tile counts (us, with the kernel of that time and now):
//   4096 x 16384:  333 rows 41.7 / 31.3,  600: 59 / 45,  777: 64 / 53,  2048: 121 / 113;   16384 x 4096:  777: 87 / 64,  1300: 121 / 83
//   8192 x 8192:  333: 47 / 38,  600: 69 / 45,  1300: 106 / 77,  4096: 223 / 208;   5120 x 13824:  256: 35.8 / 30.0,  1024: 78 / 64
//   4096 x 11008:  1024: 62 / 46;   2064 x 8208:  777: 24.2 / 21.7;   768 x 3072:  1024: 10.3 / 9.5
// and with all seven / without 256 x 128 and 128 x 128 thrice to a CU:  879 rows of 544 x 12704 15.5 / 26.6, 418 of 864 x 10352 11.9 / 15.6
constexpr TileShape TILES[N_TILES] = {
    {128, 256, 2, {7.146f, 11.345f}, {{0.3866f, 0.4416f}, {0.4107f, 0.8608f}}, 0.850f, 0.679f},
    {128, 128, 2, {5.549f, 7.319f}, {{0.2288f, 0.2614f}, {0.3044f, 0.5239f}}, 0.850f, 0.677f},
    {128, 128, 3, {5.194f, 8.811f}, {{0.3205f, 0.3336f}, {0.2915f, 0.4967f}, {0.3656f, 0.7871f}}, 0.850f, 0.658f},
    {192, 128, 1, {6.836f, 7.551f}, {{0.2385f, 0.3419f}}, 0.850f, 0.888f},
    {192, 256, 1, {9.988f, 12.129f}, {{0.3722f, 0.5366f}}, 0.906f, 0.945f},
    {256, 128, 1, {5.942f, 6.877f}, {{0.2803f, 0.4261f}}, 0.891f, 0.907f},
    {256, 256, 1, {8.004f, 10.893f}, {{0.4526f, 0.6699f}}, 0.945f, 0.950f},
};
float tile_us(const TileShape& t, int M, int N, int nk, int n_cu) {
    const int64_t tiles = (int64_t)cdiv(M, t.bm) * cdiv(N, t.bn), round = (int64_t)t.per_cu * n_cu;
    auto one_round = [&](int n) {
        const int k = cdiv(n, n_cu);
        const float* step = t.step[k - 1];
        return t.fix[0] + (t.fix[1] - t.fix[0]) * (float)n / (float)round +
               (float)nk * (step[0] + (step[1] - step[0]) * (float)n / (float)(k * n_cu));
    };
    if (tiles <= round) return one_round((int)tiles);
    const float full_us = one_round((int)round);
    const int rem = (int)(tiles % round);
    const float share = full_us * (float)rem / (float)round;
    return (float)(tiles / round) * full_us * t.round + share + (rem ? t.tail * (one_round(rem) - share) : 0.0f);
}
// On at most 128 rows every taller tile is half empty, and the weights are read once: 128 x 128 (with FETCH_ONCE) there.
// One round of 256 x 256 tiles, one to a CU, that fills the chip stores everything at its end, and on few K-steps that is what
// counts, which the estimate does not know: 1024 rows of 512 x 16384 26.1 us against 20.2, of 768 x 16384 29.3 / 24.9; 3856 of
// 880 x 4048 22.0 / 24.4, 913 of 784 x 15088 21.1 / 24.2 (236 tiles).
int fastest_tile(int M, int N, int nk, int n_cu, float& us) {
    if (M <= 128) {
        us = tile_us(TILES[T128x128], M, N, nk, n_cu);
        return T128x128;
    }
    int best = 0;
    for (int i = 0; i < N_TILES; ++i) {
        if (i == T256x256 && nk <= 12) {
            const int64_t tiles = (int64_t)cdiv(M, 256) * cdiv(N, 256);
            if (tiles <= n_cu && 10 * tiles > 9 * n_cu) continue;
        }
        const float t = tile_us(TILES[i], M, N, nk, n_cu);
        if (i == 0 || t < us) us = t, best = i;
    }
    return best;
}

// FETCH_ONCE: 128 x 128 and 192 x 128 tiles whose weights one row tile reads, or most of whose weights.  As many weights
// pass the caches by, and the token rows stay there: 128 rows of 2048 x 32768 21.4 -> 18.0 us, of 512 x 16384 8.2 -> 7.9, 192
// rows of 4096 x 16384 29.5 -> 27.9; 8 experts of 75 rows of 14336 x 4096, the layer 308 -> 298.  With several row tiles it
// depends on who comes first (256 rows of 4096 x 16384 31.6 -> 30.5, of 2048 x 32768 32.6 -> 34.2): left as it is.
template <int EPI, int FETCH = FETCH_PLAIN>
int launch_shape(const GemmArgs& a, int shape, hipStream_t st) {
    const dim3 grid = tile_grid(a, TILES[shape].bm, TILES[shape].bn);
    switch (shape) {
        case T128x128: return launch_tiles<128, 128, 2, 2, 4, 2, EPI, false, false, FETCH>(a, grid, st);  // wave tile 64 x 64
        case T128x128x3: return launch_tiles<128, 128, 2, 2, 3, 3, EPI, false, false, FETCH_PLAIN>(a, grid, st);
        case T256x128: return launch_tiles<256, 128, 4, 2, 5, 1, EPI, false, false, FETCH_PLAIN>(a, grid, st);  // 64 x 64, eight waves
        case T192x128: return launch_tiles<192, 128, 2, 2, 7, 1, EPI, false, false, FETCH>(a, grid, st);  // 96 x 64
        case T192x256: return launch_tiles<192, 256, 2, 2, 5, 1, EPI, false, false, FETCH_PLAIN>(a, grid, st);  // 96 x 128
        case T256x256: return launch_tiles<256, 256, 4, 2, 4, 1, EPI, false, false, FETCH_PLAIN>(a, grid, st);  // 64 x 128, eight waves
        default: return launch_one<EPI, false>(a, st);
    }
}

// 128 x 128 tiles dealt over the XCDs, for the gate/up projection of very few rows.
template <int EPI>
int launch_few_narrow(const GemmArgs& a, hipStream_t st) {
    const dim3 grid((unsigned)((int64_t)row_tiles(a, 128) * round_up(cdiv(a.N, 128), 8)));
    return launch_tiles<128, 128, 2, 2, 4, 2, EPI, false, true, FETCH_PLAIN>(a, grid, st);
}

// Operands whose offsets need more than 32 bits (4 GB): the tiled kernel computes its addresses in 64.
bool wide_operands(const GemmArgs& a) {
    const int64_t rows = a.R > a.Npad ? a.R : a.Npad;
    return rows > (int64_t)PAST_END / (64 * (int64_t)cdiv(a.K, 64));
}
template <bool DBG>
int launch_wide(const GemmArgs& a, int epi, hipStream_t st) {
    switch (epi) {
        case EPI_SWIGLU: return launch_one<EPI_SWIGLU, false, false, FETCH_WIDE>(a, st);
        case EPI_SWIGLU_ASYM: return launch_one<EPI_SWIGLU_ASYM, false, false, FETCH_WIDE>(a, st);
        case EPI_LINEAR_ASYM: return launch_one<EPI_LINEAR_ASYM, DBG, false, FETCH_WIDE>(a, st);
        default: return launch_one<EPI_LINEAR, DBG, false, FETCH_WIDE>(a, st);
    }
}

}  // namespace

// Row blocks of 16 per tile (4, 6 or 8) with which the streaming kernel (skinny.hip: 64-channel tiles, K split over
// the waves, operands straight into registers) beats the tiled kernel, whose fastest shape takes `tiled_us`, or 0.  Its
// three tiles are estimated alike (fitted to the 470 to 562 launches of each with at most 256 tiles of 128 x 128 and between 0.6 and
// 1.6 times the fastest tiled shape; mean deviation 6 to 8 %): a K-step costs them a third to a half of the others', which pays
// where few of either fit and K is long.  Of 1313 sizes the estimates choose the slower kernel, by 4 to 11 %, at 10.
// Measured (us, M rows, K x N, streaming against tiled):
//   16384 x 4096:  129 rows 30 / 69,  333: 39 / 62,  600: 68 / 62 (tiled),  700: 70 / 63 (tiled);   4096 x 4096:  129: 12 / 20,  512: 18 / 22
//   3072 x 768:    1024 rows 12 / 18;   2048 x 8192:  256 rows 13.5 / 14.5,  300: 22 / 13.9 (tiled)
//   8192 x 8192:   300 rows 47 / 36 (tiled);   4352 x 10304:  170 rows 28.0 / 23.4 (tiled);   5872 x 8800:  185: 33.4 / 29.0 (tiled)
// and where few K-steps leave the start and the end to decide:
//   512 x 4096:    256 rows 7.5 / 7.8,  333: 9.1 / 7.9 (tiled);   768 x 3072: 400 rows 9.6 / 8.6 (tiled);   1024 x 4096: 512 rows 10.7 / 10.0 (tiled)
static int stream_row_blocks(const GemmArgs& a, int n_cu, float tiled_us) {
    static constexpr TileShape STREAM[3] = {
        {64, 64, 1, {5.130f, 5.486f}, {{0.1169f, 0.1422f}}, 0.701f, 0.910f},
        {96, 64, 1, {6.364f, 7.031f}, {{0.1287f, 0.1512f}}, 0.782f, 0.866f},
        {128, 64, 1, {6.776f, 7.347f}, {{0.1461f, 0.1791f}}, 0.869f, 0.792f},
    };
    float best = tiled_us;
    int rb = 0;
    for (const TileShape& t : STREAM) {
        if (a.M <= t.bm) break;  // a single row tile: skinny_pays has decided
        const float us = tile_us(t, a.M, a.N, cdiv(a.K, 64), n_cu);
        if (us <= best) {
            best = us;
            rb = t.bm / 16;
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
//   units 128 (1024 x 3584, 8 experts), 100 rows: 68 / 68 / 79 / 82, 73 / 74 / 84 / 88;  132 (704 x 11008, 12), 109: 146 / 155, 152 / 159 (first two)
//         256 (4096 x 14336, 4), 100: 176 / 178 / 212 / 219, 212 / 203 / 240 / 246;  112: 180 / 180 / 216 / 222, 218 / 210 / 247 / 253
//             (2048 x 8192, 8), 100: 127 / 128 / 149 / 155, 146 / 140 / 163 / 168;  112: 157 / 141 / 162 / 168, 148 / 139 / 162 / 168
//         384 (3072 x 14336, 8), 20: 208 / 204 / 239 / 246, 207 / 206 / 240 / 248;  76: 266 / 250 / 281 / 288, 274 / 264 / 292 / 301;
//              100: 285 / 263 / 292 / 300, 320 / 340 / 315 / 324
//         448 (3584 x 8192, 8), 36: 160 / 154 / 177 / 182, 165 / 157 / 178 / 183;  76: 180 / 169 / 187 / 192, 188 / 182 / 199 / 205
//         512 (4096 x 14336, 8), 20: 248 / 247 / 271 / 280, 251 / 249 / 274 / 282;  56: 284 / 275 / 298 / 311, 294 / 280 / 304 / 314;
//              64: 302 / 285 / 309 / 321, 321 / 347 / 317 / 333;  76: 314 / 292 / 318 / 329, 351 / 354 / 329 / 343
//         512 (2048 x 5632, 16), 20: 138 / 135 / 144 / 149, 138 / 135 / 143 / 148;  36: 146 / 144 / 154 / 160, 149 / 160 / 153 / 160;
//              64: 163 / 156 / 167 / 173, 184 / 185 / 176 / 181;  100: 174 / 165 / 176 / 182, 201 / 200 / 191 / 196
//         between 256 and 384 (first two):  336 (1344 x 4416, 16), 29: 102 / 107, 104 / 106;  294 (3136 x 7616, 6), 60: 137 / 136, 127 / 130
// One and a half to two units for each CU: one round of 128 x 128 tiles from 24 rows on, as long as few rows in all keep the
// largest group of skewed routing within one row tile (192 tokens; at 224 a draw of the 56 rows above with 130 in one group: 301 / 332),
// or within two where the round has room for another row tile (304 tokens).  More units than two for each CU: FEW, unless its own
// 128 x 256 tiles fill the chip and a second row tile starts a round:
//         768 (3072 x 8192, 16), 20: 235 / 239 / 233 / 247, 241 / 246 / 234 / 248;  36: 264 / 256 / 250 / 263, 274 / 280 / 263 / 276
//         1024 (4096 x 7168, 16), 36: 289 / 282 / 281 / 291, 290 / 301 / 314 / 325;  56: 305 / 293 / 292 / 301, 312 / 316 / 325 / 336
static int stream_mean_rows(const GemmArgs& a, int n_cu) {
    const int units = a.n_sel * (a.N / 64), ntn = cdiv(a.N, 128);
    if (units <= n_cu) return 4 * units <= 3 * n_cu ? 112 : 104;
    if (2 * units < 3 * n_cu) return 112;
    if (units <= 2 * n_cu) {
        if (a.n_sel * ntn <= n_cu && a.max_rows <= 2 * ((a.n_sel + 1) * ntn <= n_cu ? 304 : 192)) return 24;
        return 2 * units == 3 * n_cu ? 112 : 64;
    }
    return a.n_sel * cdiv(a.N, BN) >= n_cu ? 48 : 24;
}
static constexpr int FEW_MEAN_ROWS = 112;  // likewise for the form for few rows
// ... and for its 128 x 128 tiles on the gate/up projection: with two work-groups of four stages to a CU more of the weight
// stream is in flight than with 128 x 256 tiles, which fetch the token rows half as often.  Whole layers (us, 128 x 256 / 128 x 128):
//   4096 x 14336, 8 experts:  18 rows 256 / 246,  24: 258 / 250,  32: 269 / 264,  56: 288 / 298,  76: 293 / 308;   2048 x 5632, 16:  18: 137 / 136,  40: 147 / 148
// Twice the work-groups also start, store and (experts without rows) end twice as often, which few K-steps in many tiles do not
// carry: 128 x 12672, 32 experts, 4 rows 144 / 167, 512 x 9984, 32: 7 rows 156 / 176, 384 x 4032, 32: 14 rows 86 / 95, 1472 x 11648, 32:
// 1 token 76 / 91, 1024 x 3840, 32: 12 rows 116 / 122, 768 x 1536, 32: 67 / 70;  and 768 x 1216, 16 (160 tiles of 128 x 256): 47 / 44,
// 1472 x 11648, 8 (728): 109 / 110, 1792 x 6464, 12 (612), 26 rows: 123 / 118, 1408 x 4864, 16 (608): 111 / 107, 1152 x 11584, 6 (546),
// 11: 91 / 87, 1856 x 4096, 32 (1024), one token 54 / 47, 2112 x 5696, 16 (720): 134 / 135.
static bool narrow_gate_up(const GemmArgs& a, int mean, int n_cu) {
    return mean <= 32 && (a.K >= 28 * 64 || 4 * a.n_sel * cdiv(a.N, BN) <= (a.K >= 18 * 64 ? 12 : 5) * n_cu);
}

// Down projections of more than 128 rows per expert: 192 x 256 tiles (a tenth less time for the same work than 128 x 256,
// more rows of padding) by the estimates of dense launches, where they fill most of a round and no more, or one and a half
// rounds and more.  Rounds of uneven groups run into each other, which over 64 K-steps and more makes up for an estimate that is a fifth
// higher.  The tiles are counted for experts between half and one and a half times the average.  Of 320 layers 33 would be more
// than 3 % faster with the other tiles (74 with 192 x 256 from one and a half rounds on whatever K is).  Whole layers (us,
// tokens even, then by 1 / rank^1.1; 128 x 256 / 192 x 256):
//   4096 x 14336, 8 experts:  194 rows 431 / 451, 456 / 469 (no);  256: 579 / 528, 587 / 535;  512: 908 / 875, 885 / 854;  1024: 1565 / 1515, 1529 / 1493
//   2048 x 5632, 16:  300: 321 / 305, 321 / 334 (no);  512: 442 / 436, 438 / 434;   1024 x 3584, 8:  600: 149 / 152, 148 / 152 (no)
//   few K-steps in several rounds:  6016 x 704, 16: 177 rows 148 / 152, 150 / 167 (no);  5952 x 3712, 8: 437: 322 / 353, 337 / 363 (no);
//   3648 x 832, 8: 930: 166 / 182, 169 / 184 (no);  5184 x 7168, 8: 751: 791 / 762, 800 / 772
static bool tall_group_tiles(const GemmArgs& a, int n_cu) {
    const int mean = a.max_rows / a.n_sel, nk = cdiv(a.K, 64), ntn = cdiv(a.N, 256);
    auto count = [&](int bm) {
        int n = 0;
        for (int f = 2; f <= 6; ++f) n += cdiv((int64_t)mean * f, 4 * bm);
        return (int)((int64_t)n * a.n_sel * ntn / 5);
    };
    const int tall = count(192);
    const bool rounds = 2 * tall >= 3 * n_cu;
    if (!rounds && 20 * tall > 17 * n_cu) return false;
    return tile_us(TILES[T192x256], 1, tall * 256, nk, n_cu) <
           (rounds && nk >= 64 ? 1.2f : 1.0f) * tile_us(TILES[T128x256], 1, count(128) * 256, nk, n_cu);
}

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
        if (a.M <= TILES[shape].bm) return asym ? launch_shape<EPI_LINEAR_ASYM, FETCH_ONCE>(a, shape, st) : launch_shape<EPI_LINEAR, FETCH_ONCE>(a, shape, st);
        return asym ? launch_shape<EPI_LINEAR_ASYM>(a, shape, st) : launch_shape<EPI_LINEAR>(a, shape, st);
    }
    if (a.offsets) {
        // Few rows per expert: bound by the weight stream, not by the matrix cores.  Gate/up, FEW / many rows, whole layers (us)
        // by rows per expert: 4096 x 14336, 8 experts: 40: 274 / 301, 76: 293 / 317, 112: 338 / 365, 124: 449 / 421, 150: 503 / 414;
        // 2048 x 5632, 16 experts: 40: 147 / 159, 76: 160 / 171, 112: 182 / 197, 124: 204 / 206, 150: 243 / 235.
        const int mean = a.max_rows / (a.n_sel > 0 ? a.n_sel : 1);
        const bool down = epi == EPI_LINEAR || epi == EPI_LINEAR_ASYM, asym = epi == EPI_LINEAR_ASYM;
        if (down && mean <= stream_mean_rows(a, cu_count())) return launch_stream_grouped(a, asym, st);
        // 128 x 128 tiles where they cover the groups in one round (a CU with two of them takes 1.6 times as long: 1024 rows of
        // 14336 x 4096, 256 tiles 66 us, 1152 rows, 288 tiles 103): at one row tile for each group while few have more, else by the upper bound
        const int row_tiles_s = mean <= 104 ? a.n_sel : mean <= FEW_MEAN_ROWS ? a.n_sel + cdiv(a.n_sel, 8) : row_tiles(a, 128);
        if (down && row_tiles_s * cdiv(a.N, 128) <= cu_count()) {
            // several row tiles to a group: the caches keep its weights (whole layers, FETCH_ONCE / plain: 2048 x 8192, 4 experts, 300
            // rows 137 / 135, 256 rows skewed 137 / 133; 1024 x 3584, 8: 300 rows 104 / 103)
            if (mean > FEW_MEAN_ROWS) return asym ? launch_shape<EPI_LINEAR_ASYM>(a, T128x128, st) : launch_shape<EPI_LINEAR>(a, T128x128, st);
            return asym ? launch_shape<EPI_LINEAR_ASYM, FETCH_ONCE>(a, T128x128, st) : launch_shape<EPI_LINEAR, FETCH_ONCE>(a, T128x128, st);
        }
        if (!down && narrow_gate_up(a, mean, cu_count()))
            return epi == EPI_SWIGLU_ASYM ? launch_few_narrow<EPI_SWIGLU_ASYM>(a, st) : launch_few_narrow<EPI_SWIGLU>(a, st);
        if (down && mean > 128 && tall_group_tiles(a, cu_count())) return asym ? launch_shape<EPI_LINEAR_ASYM>(a, T192x256, st) : launch_shape<EPI_LINEAR>(a, T192x256, st);
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
