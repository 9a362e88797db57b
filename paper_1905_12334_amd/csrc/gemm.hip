// mp8_gemm_fp8: the FP8 compute primitive of Section 3 (arXiv 1905.12334) for gfx950 --
// two 8-bit (1,5,2) operands, FP32 accumulation on the matrix cores, and the Q node of
// Figure 1a (one rounding of the complete FP32 sum to 8 bits, RNE or stochastic) fused into
// the epilogue.  The three training GEMMs (forward, backward-data, weight-gradient) are the
// same contraction  out[r,c] = sum_j a[r,j] * b[c,j]  on differently oriented operands.
//
// This file is the host side: kernel table, choice of kernel and contraction slices, argument
// checks and launches.  The kernels live in headers of their own:
//   gemm_common.hpp   argument structs, the epilogue of a run of outputs, direct-to-LDS loads
//   gemm_mfma.hpp     the general kernel: block tile BM x BN, ring of 2-4 stages of 128 bytes of
//                     contraction, slot-scheduled MFMA loop, every operand layout, 3x3 convolutions
//   gemm_stream.hpp   several 256x256 tiles per CU: the operand stream goes on from tile to tile
//   gemm_shortk.hpp   contractions of one or two stages (all start-up and epilogue)
//   gemm_wavek.hpp    small outputs with long contractions (contraction divided among waves)
//   gemm_wave128.hpp  about one 128x128 tile per CU and a long contraction (every wave the whole tile)
//   gemm_any.hpp      row lengths, leading dimensions, contractions that are not multiples of 16
// (contractions that are not multiples of 128: half-precision forms of the general and the wave-split kernel)
//   gemm_conv.hpp     3x3 convolutions, forward and backward data: a tile's pixel rows in LDS for all taps
//   gemm_epilogue.hpp  from a tile's accumulators to its outputs
//   gemm_finish.hpp   second pass for split contractions and unfused epilogues, optionally with
//                     the master-weight update; the any-shape fallback kernel
// Split contraction, ragged column counts, FP32 results alone, and FP32 or transposed results of poorly filled tiles: the
// MFMA kernels write FP32 tiles and the second pass sums the slices in order and applies the epilogue -- the sum is
// rounded exactly once.  Everything else leaves in the kernels' own epilogues.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <type_traits>

#include "../../include/mp8.h"
#include "gemm_any.hpp"
#include "gemm_common.hpp"
#include "gemm_conv.hpp"
#include "gemm_finish.hpp"
#include "gemm_mfma.hpp"
#include "gemm_shortk.hpp"
#include "gemm_stream.hpp"
#include "gemm_wavek.hpp"
#include "gemm_wave128.hpp"
#include "gemm_qfwd.hpp"

namespace mp8 {

// ---------------------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------------------
struct TileConfig {
    int bm, bn;
    const char *name;
    void (*kernel[3])(const GemmArgs);     // indexed by EPI_*
    void (*kernel_tn[3])(const GemmArgs);  // both operands contraction-major; null if not built
    void (*kernel_bt[3])(const GemmArgs);  // only b contraction-major; null if not built
    void (*kernel_conv[3][3])(const GemmArgs);  // [mp8_op][EPI_*] 3x3 convolution; null if not built
    int max_ksteps;      // 0: any contraction length; else the most stages the kernel takes
    int lds_per_stage;   // dynamic LDS bytes per stage (kernels that load all stages at once)
};

#define MP8_TILE(BM, BN, WGM, WGN, NS, MB)                                   \
    {BM, BN, #BM "x" #BN "x128s" #NS,                                         \
     {gemm_mfma_kernel<BM, BN, WGM, WGN, NS, MB, EPI_PARTIAL>,                \
      gemm_mfma_kernel<BM, BN, WGM, WGN, NS, MB, EPI_RNE>,                    \
      gemm_mfma_kernel<BM, BN, WGM, WGN, NS, MB, EPI_FULL>},                  \
     {nullptr, nullptr, nullptr}, {nullptr, nullptr, nullptr},                \
     {{nullptr, nullptr, nullptr}, {nullptr, nullptr, nullptr}, {nullptr, nullptr, nullptr}}, 0, 0}
#define MP8_TILE_TN(BM, BN, WGM, WGN, NS, MB)                                \
    {BM, BN, #BM "x" #BN "x128s" #NS,                                         \
     {gemm_mfma_kernel<BM, BN, WGM, WGN, NS, MB, EPI_PARTIAL>,                \
      gemm_mfma_kernel<BM, BN, WGM, WGN, NS, MB, EPI_RNE>,                    \
      gemm_mfma_kernel<BM, BN, WGM, WGN, NS, MB, EPI_FULL>},                  \
     {gemm_mfma_kernel<BM, BN, WGM, WGN, NS, MB, EPI_PARTIAL, true, true>,    \
      gemm_mfma_kernel<BM, BN, WGM, WGN, NS, MB, EPI_RNE, true, true>,        \
      gemm_mfma_kernel<BM, BN, WGM, WGN, NS, MB, EPI_FULL, true, true>},      \
     {gemm_mfma_kernel<BM, BN, WGM, WGN, NS, MB, EPI_PARTIAL, false, true>,   \
      gemm_mfma_kernel<BM, BN, WGM, WGN, NS, MB, EPI_RNE, false, true>,       \
      gemm_mfma_kernel<BM, BN, WGM, WGN, NS, MB, EPI_FULL, false, true>},      \
     {{gemm_mfma_kernel<BM, BN, WGM, WGN, NS, MB, EPI_PARTIAL, false, true, 1>, \
       gemm_mfma_kernel<BM, BN, WGM, WGN, NS, MB, EPI_RNE, false, true, 1>,     \
       gemm_mfma_kernel<BM, BN, WGM, WGN, NS, MB, EPI_FULL, false, true, 1>},   \
      {gemm_mfma_kernel<BM, BN, WGM, WGN, NS, MB, EPI_PARTIAL, false, false, 2>, \
       gemm_mfma_kernel<BM, BN, WGM, WGN, NS, MB, EPI_RNE, false, false, 2>,    \
       gemm_mfma_kernel<BM, BN, WGM, WGN, NS, MB, EPI_FULL, false, false, 2>},  \
      {gemm_mfma_kernel<BM, BN, WGM, WGN, NS, MB, EPI_PARTIAL, true, true, 3>,  \
       gemm_mfma_kernel<BM, BN, WGM, WGN, NS, MB, EPI_RNE, true, true, 3>,      \
       gemm_mfma_kernel<BM, BN, WGM, WGN, NS, MB, EPI_FULL, true, true, 3>}}, 0, 0}
#define MP8_TILE_SHORTK                                                      \
    {128, 128, "128x128x128k",                                                \
     {gemm_shortk_kernel<EPI_PARTIAL>, gemm_shortk_kernel<EPI_RNE>, gemm_shortk_kernel<EPI_FULL>}, \
     {nullptr, nullptr, nullptr}, {nullptr, nullptr, nullptr},                \
     {{nullptr, nullptr, nullptr}, {nullptr, nullptr, nullptr}, {nullptr, nullptr, nullptr}}, 2, 32768}
#define MP8_WAVEK(ATN, BTN, CONV)                                            \
    {gemm_wavek_kernel<EPI_PARTIAL, ATN, BTN, CONV>, gemm_wavek_kernel<EPI_RNE, ATN, BTN, CONV>, \
     gemm_wavek_kernel<EPI_FULL, ATN, BTN, CONV>}
#define MP8_TILE_WAVEK                                                       \
    {64, 64, "64x64x128w", MP8_WAVEK(false, false, 0), MP8_WAVEK(true, true, 0),  \
     MP8_WAVEK(false, true, 0),                                                \
     {{nullptr, nullptr, nullptr}, {nullptr, nullptr, nullptr}, MP8_WAVEK(true, true, 3)}, 0, 0}
#define MP8_WAVEK32(BTN, BN)                                                 \
    {gemm_wavek_kernel<EPI_PARTIAL, false, BTN, 0, 32, BN>, gemm_wavek_kernel<EPI_RNE, false, BTN, 0, 32, BN>, \
     gemm_wavek_kernel<EPI_FULL, false, BTN, 0, 32, BN>}
#define MP8_NO_KERNELS {nullptr, nullptr, nullptr}
#define MP8_WAVE128(ATN, BTN)                                                \
    {gemm_wave128_kernel<EPI_PARTIAL, ATN, BTN>, gemm_wave128_kernel<EPI_RNE, ATN, BTN>, \
     gemm_wave128_kernel<EPI_FULL, ATN, BTN>}
#define MP8_TILE_WAVE128                                                     \
    {128, 128, "128x128x128p", MP8_WAVE128(false, false), MP8_WAVE128(true, true), MP8_WAVE128(false, true), \
     {MP8_NO_KERNELS, MP8_NO_KERNELS, MP8_NO_KERNELS}, 0, 0}
#define MP8_TILE_WAVEK32x64                                                  \
    {32, 64, "32x64x128w", MP8_WAVEK32(false, 64), MP8_NO_KERNELS, MP8_WAVEK32(true, 64), \
     {MP8_NO_KERNELS, MP8_NO_KERNELS, MP8_NO_KERNELS}, 0, 0}
#define MP8_TILE_WAVEK32x32                                                  \
    {32, 32, "32x32x128w", MP8_WAVEK32(false, 32), MP8_NO_KERNELS, MP8_NO_KERNELS, \
     {MP8_NO_KERNELS, MP8_NO_KERNELS, MP8_NO_KERNELS}, 0, 0}
static const TileConfig kTiles[] = {
    MP8_TILE_TN(256, 256, 2, 2, 2, 1), MP8_TILE(256, 128, 2, 2, 3, 1), MP8_TILE(128, 256, 2, 2, 3, 1),
    MP8_TILE_TN(128, 128, 2, 2, 2, 2), MP8_TILE_TN(128, 128, 2, 2, 4, 1), MP8_TILE(64, 128, 1, 4, 3, 2),
    MP8_TILE(128, 64, 4, 1, 3, 2),  MP8_TILE_TN(64, 64, 2, 2, 4, 2), MP8_TILE(64, 128, 1, 4, 2, 3),
    MP8_TILE(128, 64, 4, 1, 2, 3),  MP8_TILE_TN(64, 64, 2, 2, 2, 4),   MP8_TILE_SHORTK,
    MP8_TILE_WAVEK, MP8_TILE_WAVEK32x64, MP8_TILE_WAVEK32x32, MP8_TILE_WAVE128,
};
constexpr int kNumTiles = (int)(sizeof(kTiles) / sizeof(kTiles[0]));
constexpr int kCUs = 256;
constexpr int kMaxSplits = 64;

// gemm_any_kernel by operand layout (row-major, b contraction-major, both): the FP32 tiles of a split
// contraction, an unsplit one, a split one slice by slice
static void (*const kAny[3][3])(const GemmArgs) = {
    {gemm_any_kernel<EPI_PARTIAL, false, false>, gemm_any_kernel<EPI_FULL, false, false>, gemm_any_kernel<EPI_FULL, false, false, true>},
    {gemm_any_kernel<EPI_PARTIAL, false, true>, gemm_any_kernel<EPI_FULL, false, true>, gemm_any_kernel<EPI_FULL, false, true, true>},
    {gemm_any_kernel<EPI_PARTIAL, true, true>, gemm_any_kernel<EPI_FULL, true, true>, gemm_any_kernel<EPI_FULL, true, true, true>}};

// ... and in tiles of 32 rows, unsplit: [b contraction-major]
static void (*const kAny32[2])(const GemmArgs) = {gemm_any_kernel<EPI_FULL, false, false, false, 32>, gemm_any_kernel<EPI_FULL, false, true, false, 32>};

// Half-precision forms of the direct-to-LDS kernels, for contractions that are not whole stages: [64x64, 64x64
// divided among the waves, 128x128][operand layout as above][EPI_*] (they never write FP32 tiles)
#define MP8_HALF_64(ATN, BTN)                                                                                    \
    {nullptr, gemm_mfma_kernel<64, 64, 2, 2, 2, 4, EPI_RNE, ATN, BTN, 0, true>,                                  \
     gemm_mfma_kernel<64, 64, 2, 2, 2, 4, EPI_FULL, ATN, BTN, 0, true>}
#define MP8_HALF_WAVEK(ATN, BTN)                                                                                 \
    {nullptr, gemm_wavek_kernel<EPI_RNE, ATN, BTN, 0, 64, 64, true>, gemm_wavek_kernel<EPI_FULL, ATN, BTN, 0, 64, 64, true>}
#define MP8_HALF_128(ATN, BTN)                                                                                   \
    {nullptr, gemm_mfma_kernel<128, 128, 2, 2, 2, 2, EPI_RNE, ATN, BTN, 0, true>,                                \
     gemm_mfma_kernel<128, 128, 2, 2, 2, 2, EPI_FULL, ATN, BTN, 0, true>}
static void (*const kHalf[3][3][3])(const GemmArgs) = {
    {MP8_HALF_64(false, false), MP8_HALF_64(false, true), MP8_HALF_64(true, true)},
    {MP8_HALF_WAVEK(false, false), MP8_HALF_WAVEK(false, true), MP8_HALF_WAVEK(true, true)},
    {MP8_HALF_128(false, false), MP8_HALF_128(false, true), MP8_HALF_128(true, true)}};

// Kernels whose epilogue applies the master-weight update: [8-bit, half-precision products][row-major,
// contraction-major operands][state words per weight].
using UpdateKernel = void (*)(const GemmArgs, const UpdateHook);
#define MP8_WAVEK_UPDATE(KM, HALF)                                                                               \
    {gemm_wavek_update_kernel<0, KM, KM, 0, HALF>, gemm_wavek_update_kernel<1, KM, KM, 0, HALF>,                 \
     gemm_wavek_update_kernel<2, KM, KM, 0, HALF>}
#define MP8_64_UPDATE(KM, HALF)                                                                                  \
    {gemm_mfma_update_kernel<64, 64, 2, 2, 2, 4, 0, KM, KM, HALF>, gemm_mfma_update_kernel<64, 64, 2, 2, 2, 4, 1, KM, KM, HALF>, \
     gemm_mfma_update_kernel<64, 64, 2, 2, 2, HALF ? 3 : 4, 2, KM, KM, HALF>}
static const UpdateKernel kWavekUpdate[2][2][3] = {{MP8_WAVEK_UPDATE(false, false), MP8_WAVEK_UPDATE(true, false)},
                                                   {MP8_WAVEK_UPDATE(false, true), MP8_WAVEK_UPDATE(true, true)}};
static const UpdateKernel k64x64Update[2][2][3] = {{MP8_64_UPDATE(false, false), MP8_64_UPDATE(true, false)},
                                                   {MP8_64_UPDATE(false, true), MP8_64_UPDATE(true, true)}};

struct Plan {
    bool mfma;   // one of kTiles
    int tile;    // index into kTiles
    int splits;
    bool half;     // the half-precision form of that tile: unsplit, one pass
    bool in_turn;  // gemm_any_kernel: a workgroup takes all slices of its tile
    int conv_rows; // gemm_conv_kernel: output rows per tile (0: another kernel)
    int tiles_m, tiles_n;
};

static void op_dims(mp8_op op, int64_t M, int64_t N, int64_t K, int64_t &rows, int64_t &cols,
                    int64_t &kc) {
    switch (op) {
        case MP8_FWD: rows = M; cols = N; kc = K; break;
        case MP8_BWD_DATA: rows = M; cols = K; kc = N; break;
        default: rows = K; cols = N; kc = M; break;
    }
}

// Choose tile shape and number of contraction slices.  Measured on MI355X: the 256x256 tile
// is the only one that approaches the matrix-core peak (fewest LDS and L2 bytes per flop) but
// needs enough tiles to fill whole rounds of 256 CUs; 128x128 serves mid-sized outputs (two
// resident blocks per CU when the contraction is short, a deeper ring when it is long); small
// outputs take 64x64 tiles and, if even those are too few, a split contraction -- kept to a
// minimum because the second pass costs several microseconds.
enum { T256x256 = 0, T128x128s2 = 3, T128x128s4 = 4, T128x64s2 = 9, T64x64s2 = 10, T128x128k = 11, T64x64w = 12,
       T32x64w = 13, T32x32w = 14, T128x128p = 15 };
static Plan make_plan(int64_t rows, int64_t cols, int64_t kc, int tile_config, int split_k,
                      int layout = 0,      // bit 0: a contraction-major, bit 1: b
                      bool conv = false) { // a convolution: only the tiles with convolution addressing
    Plan pl{};
    pl.mfma = (kc % BK) == 0 && kc > 0;
    // contraction-major operands are fetched in 16-row chunks, by the tiles built for them
    if ((layout & 1) && (rows & 15) != 0) pl.mfma = false;
    if ((layout & 2) && (cols & 15) != 0) pl.mfma = false;
    if (layout != 0 && tile_config > 0 &&
        (layout == 3 ? kTiles[tile_config - 1].kernel_tn[0] : kTiles[tile_config - 1].kernel_bt[0]) == nullptr)
        pl.mfma = false;
    const bool tn = layout != 0;
    if (layout == 0 && tile_config > 0 && kTiles[tile_config - 1].kernel[0] == nullptr) pl.mfma = false;
    if (tile_config > 0 && kTiles[tile_config - 1].max_ksteps > 0 &&
        (tn || kc / BK > kTiles[tile_config - 1].max_ksteps))
        pl.mfma = false;
    if (!pl.mfma) {
        pl.splits = 1;
        return pl;
    }
    const int ksteps = (int)(kc / BK);
    auto count = [&](int t) {
        return ((rows + kTiles[t].bm - 1) / kTiles[t].bm) * ((cols + kTiles[t].bn - 1) / kTiles[t].bn);
    };
    int t;
    if (tile_config > 0) {
        t = tile_config - 1;
    } else {
        const int64_t n256 = count(T256x256), n128 = count(T128x128s2);
        const double fill256 = (double)n256 / (double)(((n256 + kCUs - 1) / kCUs) * kCUs);
        const int64_t n64 = count(T64x64s2);
        // 128x128 tiles.  One round (one tile per CU at most): from 64 stages on every wave takes the whole
        // tile on a quarter of the contraction, below that the four-stage ring keeps more loads in
        // flight than the two-stage one (2048 x 2048 x 4096 contraction-major 25.3 -> 23.4 us, 1536 x 2048
        // 25.3 -> 21.4; with all CUs taken it pays from 24 stages on: 19.7 both, at 16 14.5 against
        // 15.5).  Two rounds: two workgroups of the two-stage ring per CU beat both, whose second tile
        // starts when the first has ended (2304 x 2048 x 8192 47.7 us, four stages 69.0, wave-divided
        // 67.5; 4096 x 2048 x 16384 119.5 / 135.2 / 132.3).  A row-major a with both rounds nearly full is the
        // exception from 128 stages on (4096 x 2048 x 16384 124.0 us, wave-divided 121.4; x 8192 57.7 and 63.9).
        const bool one_round = !conv && n128 >= kCUs / 2 && n128 <= kCUs;
        const int ring128 = one_round && ksteps >= (n128 <= kCUs - kCUs / 8 ? 16 : 24) ? T128x128s4 : T128x128s2;
        const bool two_rounds = !conv && n128 > kCUs && n128 <= 2 * kCUs;
        const bool wave_rounds = two_rounds && layout != 3 && n128 >= 2 * kCUs - kCUs / 4 && ksteps >= 128;
        const int long128 = one_round || wave_rounds ? T128x128p : two_rounds ? T128x128s2 : T128x128s4;
        if (n256 >= 208 && fill256 >= 0.8 && ksteps >= 8) t = T256x256;
        // so few tiles that most CUs would idle and the contraction is too short to split:
        // half the rows per tile, and half the columns too if that still fits one round
        else if (layout == 0 && 4 * n64 <= kCUs && ksteps >= 16 && ksteps <= 40 && count(T32x32w) <= kCUs)
            t = T32x32w;
        else if (!(layout & 1) && 2 * n64 <= kCUs && ksteps >= 16 && ksteps <= 40 && count(T32x64w) <= kCUs)
            t = T32x64w;
        else if (n64 <= kCUs && ksteps >= 16) t = T64x64w;  // one workgroup per CU, one round
        // between half and three quarters of the CUs with a 128x128 tile, both operands contraction-major: two
        // to three 64x64 tiles per CU until the contraction is long enough to pay for an update kernel of its
        // own, which the 64x64 tiles do not need (2304 x 1024 x 4096 29.0 us, four-stage ring 20.7; 2048 x 1024,
        // where every CU has two, 20.5 and 20.6, x 6144 31.3 and 26.6)
        else if (layout == 3 && one_round && n128 < 192 && ksteps <= 64 && ksteps >= (n128 > kCUs / 2 ? 32 : 48))
            t = T128x128s4;
        else if (tn && (n128 < 16 || (n128 < 192 && ksteps <= 64))) t = T64x64s2;
        else if (tn) t = ksteps >= 64 ? long128 : ring128;
        else if (n128 >= 192 && ksteps <= 2) t = T128x128k;  // all prologue and epilogue
        else if (n128 >= 192) t = (ksteps >= 64 && n128 <= 2 * kCUs) ? long128 : ring128;
        else t = T64x64s2;
    }
    pl.tile = t;
    pl.tiles_m = (int)((rows + kTiles[t].bm - 1) / kTiles[t].bm);
    pl.tiles_n = (int)((cols + kTiles[t].bn - 1) / kTiles[t].bn);
    const int64_t nt = (int64_t)pl.tiles_m * pl.tiles_n;
    int s = 1;
    if (kTiles[t].max_ksteps > 0) {
        s = 1;  // these kernels take the whole contraction at once
    } else if (split_k == 0 && (t == T32x64w || t == T32x32w)) {
        s = 1;
    } else if (split_k == 0 && t == T64x64w) {
        // one workgroup per CU and never more workgroups than CUs (a second round would double
        // the time); at least two stages for each of the four waves.  A split costs the finishing
        // pass (about 4 us, the time of some 32 stages of one wave), so it must save more than that.
        s = (int)std::max<int64_t>(1, std::min<int64_t>(kCUs / nt, ksteps / 8));
        s = std::min(s, kMaxSplits);
        if ((int64_t)ksteps * (s - 1) <= (int64_t)40 * s) s = 1;
    } else if (split_k > 0) {
        s = split_k;
    } else if (nt < kCUs / 2) {
        // about one and a half blocks per CU; two for the smallest tiles; fewer for the 128-row
        // tiles of contraction-major operands, whose FP32 partial tiles are four times as large
        const int target = kTiles[t].bm * kTiles[t].bn <= 64 * 64 ? 512 : tn ? 160 : 384;
        s = std::max(1, (int)(target / nt));        // never more blocks than the target: the
                                                    // CUs that got one more would set the time
        s = std::min(s, std::max(1, ksteps / 8));  // at least eight stages per slice
        s = std::min(s, kMaxSplits);
    }
    s = std::max(1, std::min(s, ksteps));
    pl.splits = s;
    return pl;
}

// Outputs of more 256x256 tiles than CUs whose codes are rounded to nearest and nothing else is asked for: does
// gemm_stream_kernel, which starts once and not per tile, beat the tile that make_plan names?  Both deal whole tiles to the CUs, 256 of them or
// 512 of 128x128 at a time, and what counts is how many rounds that makes: a round of 256x256 tiles takes as long as 1.6 to 2 of 128x128,
// so two of them have to stand for four, four for seven.  128x128 tiles (contractions of two stages: their own kernel) / 256x256, us, b
// row-major, contraction-major, both operands contraction-major:
//   rounds 4 / 2   25088 x 1024 (392 tiles of 256x256) x 384 17.4 17.4 17.9 / 17.0 17.0 17.2, x 1024 32.1 32.2 32.5 / 29.0 29.5 30.0, x 2048 56.3 54.3 54.8 / 47.5 47.5 48.6
//          4 / 2   25088 x 960 (as many) x 384 17.2 18.1 18.6 / 17.2 17.5 17.4, x 1024 31.9 33.6 34.2 / 29.2 29.3 30.1
//          8 / 4   16384 x 4096 (1024) x 512 46.2 47.5 45.6 / 38.9 40.4 40.1, x 768 58.1 59.2 58.8 / 48.7 51.0 50.4
//          3 / 2   25088 x 896 (392) x 384 14.4 14.5 15.4 / 17.0 17.0 17.1, x 1024 27.6 27.3 28.1 / 29.6 29.9 30.4, x 2048 45.8 45.5 47.5 / 49.0 49.9 51.5
//          3 / 2   25088 x 832 (392) x 384 14.4 14.8 15.4 / 16.9 17.1 17.4, 65536 x 272 (512) 16.4 17.1 17.1 / 18.1 18.7 18.5, 6016 x 4096 (384) 14.9 15.0 15.6 / 16.8 17.1 17.1
//          2 / 2   100352 x 64 (392) x 384 12.2 12.0 12.2 / 18.5 18.6 18.7, 131072 x 16 (512) 13.0 13.1 13.3 / 19.0 19.4 19.2
// Below 392 tiles the two differ by less than 5 % either way.  Two stages, row-major: 25088 x 1024 x 256 12.7 / 14.5, 38400 x 1536 (rows
// that end inside a tile) 25.0 / 27.1, but 16384 x 4096 26.9 / 27.8, 16384 x 4000 27.7 / 27.0, 43504 x 2560 45.8 / 44.8.
static bool stream_pays(int64_t rows, int64_t cols, int64_t ksteps, int layout) {
    auto tiles = [&](int64_t t) { return (rows + t - 1) / t * ((cols + t - 1) / t); };
    const int64_t nt = tiles(256), rounds = (nt + kCUs - 1) / kCUs, rounds128 = (tiles(128) + 2 * kCUs - 1) / (2 * kCUs);
    const double round = (double)rounds * kCUs;
    if (nt <= kCUs || ksteps < 2 || nt < 0.765 * round || 4 * rounds128 < 7 * rounds) return false;
    return ksteps > 2 || layout != 0 || (nt > 3 * kCUs && (double)rows * (double)cols >= 0.95 * 256 * 256 * round);
}

// The plan of an aligned call.  codes_alone: it asks for codes to nearest, in rows of a multiple of 16, and nothing else.
static Plan plan_of(int64_t rows, int64_t cols, int64_t kc, int tile_config, int split_k, int layout, bool codes_alone) {
    Plan pl = make_plan(rows, cols, kc, tile_config, split_k, layout);
    if (codes_alone && pl.mfma && tile_config == 0 && split_k == 0 && pl.splits == 1 && stream_pays(rows, cols, kc / BK, layout)) {
        pl.tile = T256x256;
        pl.tiles_m = (int)((rows + 255) / 256);
        pl.tiles_n = (int)((cols + 255) / 256);
    }
    return pl;
}

// Can the direct-to-LDS kernels fetch (aligned) operands of a contraction that is not whole stages?  Row-major
// ones have to end with a whole 16-byte chunk.
static bool half_takes(int64_t rows, int64_t cols, int64_t kc, int layout) {
    return kc > 0 && kc % BK != 0 && (layout == 3 || (kc & 15) == 0) && (!(layout & 1) || (rows & 15) == 0) &&
           (!(layout & 2) || (cols & 15) == 0);
}

// The half-precision kernel that multiplies them: the tile make_plan names for whole stages, or the nearest that is
// built -- 128x128 for the large ones, 64x64 for the rest.  Not MFMA if the contraction is to be split: slices
// need a workspace, and the bits must not depend on one (gemm_any_kernel takes them in turn without).
// Against gemm_any_kernel: 12972 x 832 x 64 9.1 us (34), 2143 x 3840 x 576 13.2 (27), a training step of 6007 x 2048 x 512
// with ADAM 65.4 (82.5).
static Plan half_plan(int64_t rows, int64_t cols, int64_t kc, int layout) {
    if (!half_takes(rows, cols, kc, layout)) return Plan{};
    Plan pl = make_plan(rows, cols, (kc + BK - 1) / BK * BK, 0, 0, layout);
    if (!pl.mfma || pl.splits != 1) return Plan{};
    if (kTiles[pl.tile].bm * kTiles[pl.tile].bn > 64 * 64) pl.tile = T128x128s2;
    else if (pl.tile == T32x64w || pl.tile == T32x32w) pl.tile = T64x64w;
    else if (pl.tile != T64x64w) pl.tile = T64x64s2;
    pl.tiles_m = (int)((rows + kTiles[pl.tile].bm - 1) / kTiles[pl.tile].bm);
    pl.tiles_n = (int)((cols + kTiles[pl.tile].bn - 1) / kTiles[pl.tile].bn);
    pl.half = true;
    return pl;
}

// Can gemm_any_kernel take it?  (Lane offsets of a tile stay within 32 bits; an edge chunk is read as
// the last sixteen bytes of its row, so such rows must have sixteen.)
static bool any_kernel_takes(int64_t rows, int64_t cols, int64_t kc, int64_t lda, int64_t ldb, int layout) {
    return kc >= 16 && (!(layout & 1) || rows >= 16) && (!(layout & 2) || cols >= 16) && lda < (1 << 24) &&
           ldb < (1 << 24) && (rows + 63) / 64 * ((cols + 63) / 64) < 0x1000000;
}

// Contraction slices of gemm_any_kernel: two workgroups fit a CU, so up to 512 run at once, and a
// slice should keep two stages for each of the four waves.  The finishing pass costs about as much
// as ANY_FINISH_STAGES stages of one wave, so a split must save more than that.  (The shape alone decides,
// so that the order of additions does not depend on the workspace.)
constexpr int64_t ANY_FINISH_STAGES = 24;
static Plan any_plan(int64_t rows, int64_t cols, int64_t kc) {
    Plan pl{};
    pl.tiles_m = (int)((rows + 63) / 64);
    pl.tiles_n = (int)((cols + 63) / 64);
    const int64_t nt = (int64_t)pl.tiles_m * pl.tiles_n, ksteps = (kc + BK - 1) / BK;
    int64_t s = std::max<int64_t>(1, std::min<int64_t>({2 * kCUs / nt, ksteps / 8, (int64_t)kMaxSplits}));
    if (ksteps * (s - 1) <= ANY_FINISH_STAGES * s) s = 1;
    pl.splits = (int)s;
    return pl;
}

// Tiles of 32 rows (row-major a, unsplit): twice as many CUs share the work while half of them would idle, and up to three
// stages they also end sooner on all of them.  In 64 rows / in 32, us, b row-major and contraction-major: 256 x 1000 x 2048
// (64 tiles of 64) contraction-major 9.4 / 7.2, 1000 x 500 x 1001 (128) 7.9 7.7 / 6.6 6.2, 17 x 100 x 200 (2) 5.1 5.1 / 4.4 4.3; 600 x 1000
// (160) x 300 5.2 5.4 / 4.9 5.1, x 2000 8.3 9.9 / 8.3 11.6; 1000 x 1000 (256) x 200 5.3 5.4 / 5.0 5.2, x 380 5.3 5.5 / 5.1 5.5, x 500 5.4 5.6 /
// 5.3 5.9, x 1000 6.8 7.2 / 6.9 7.9; 1500 x 1000 (384) x 300 6.0 6.3 / 5.8 6.0, x 1500 11.4 12.5 / 11.3 13.1; 4000 x 500 (504) x 380
// 6.3 6.7 / 8.4 8.7.
static bool any_in_32_rows(const Plan &pl, int64_t kc, int layout) {
    const int64_t nt = (int64_t)pl.tiles_m * pl.tiles_n;
    return pl.splits == 1 && !(layout & 1) && (nt <= kCUs / 2 || (nt <= kCUs + kCUs / 2 && kc <= 3 * BK));
}

// The kernel that computes an unsplit weight gradient and applies the update in its epilogue, or null.  Such
// an update costs neither a launch nor a pass over the gradient codes.  Built for the 64x64 tiles, whose
// outputs are small: larger ones stream their weights and state faster in a kernel of its own.  Whole training steps
// (Q nodes, three GEMMs, update) in two launches against one, us, weights from the Infinity Cache / from memory: 256^3 SGD 15.5 against 14.8;
// ADAM 256^3 17.1 20.0 against 17.0 19.4, 1024 x 512 x 256 (32 tiles) 23.2 24.2 against 21.8 23.2, 1280 x 768 x 512 (96) 28.7 28.5 against 27.2 27.9,
// 4096 x 512 x 512 (64) 34.2 36.2 against 33.6 35.6, 640 x 1024 x 448 (112) 26.4 26.4 against 24.7 26.5 (with ADAM's
// corrections still divisions: since then one launch takes 0.3 to 0.8 less).  (Without a gradient
// to keep, ADAM on less than half of the CUs has its codes in the workspace, which such a call is asked for.)
static UpdateKernel update_kernel(const Plan &pl, int64_t cols, int layout, int states, bool keeps_codes) {
    if (!pl.mfma || pl.splits != 1 || (cols & 15) != 0 || (layout != 0 && layout != 3)) return nullptr;
    if (states == 2 && !keeps_codes && pl.tiles_m * pl.tiles_n < kCUs / 2) return nullptr;
    if (pl.tile == T64x64w) return kWavekUpdate[pl.half][layout != 0][states];
    if (pl.tile == T64x64s2) return k64x64Update[pl.half][layout != 0][states];
    return nullptr;
}

// The same for gemm_any_kernel, contraction-major operands.  Whole training steps in two launches / in one, us, weights from the Infinity Cache:
//                                          SGD              momentum         ADAM
//     12 tiles (200 x 216 x 130)       20.7 / 19.5      21.2 / 19.9      22.2 / 21.6
//     32       (300 x 104 x 1001)      23.2 / 21.8      23.5 / 22.0      24.4 / 23.8
//    256       (1000 x 1000 x 1000)    33.5 / 31.2      34.8 / 32.2      37.3 / 35.1
//    272       (129 x 1000 x 1088)     27.7 / 25.0      28.1 / 25.7      30.0 / 29.0
//    512       (256 x 1000 x 2048)     30.2 / 26.9      32.8 / 28.2      36.3 / 32.5
//    528       (129 x 1000 x 2112)     34.3 / 32.1      36.5 / 33.8      40.8 / 38.9
//    837       (64 x 1928 x 1700)      38.5 / 34.0      42.1 / 36.2      47.4 / 42.7
//   1040       (129 x 1000 x 4160)     46.3 / 42.3      50.8 / 45.3      57.4 / 54.2
//   1504       (129 x 3000 x 2002)     55.9 / 49.0      61.3 / 51.8      69.1 / 61.4
//   3995       (64 x 3000 x 5440)      87.6 / 82.4     107.2 / 91.2     127.4 / 115.2
// and the gradient with its statistics alone: 272 tiles 11.4 / 9.2, 12.0 / 9.7, 13.8 / 12.8, 512 12.1 / 9.3, 14.0 / 10.1, 16.7 / 13.5.  One launch is the
// shorter one wherever it is built, but for stochastic rounding on less than kCUs / 2 tiles whose last column is eight wide (200 x 264 x 130 21.0 / 21.1,
// 21.3 / 21.2, ADAM 22.3 / 26.1; why, is not known): that condition stands on its figures.  The others are
// those of the first kernel, whose update fetched its operands only after the contraction (a last round that was nearly empty paid for all of it, and
// the atomics of the statistics followed the updates).  They refuse calls that would gain 3 to 14 %, and are kept because which call is one kernel
// is part of what is tested.
static UpdateKernel any_update_kernel(const Plan &pl, int64_t cols, int layout, const UpdateHook &upd, bool with_stats, bool stochastic) {
    static const UpdateKernel kernels[3] = {gemm_any_update_kernel<0>, gemm_any_update_kernel<1>, gemm_any_update_kernel<2>};
    const int64_t nt = (int64_t)pl.tiles_m * pl.tiles_n, round = 2 * kCUs;
    if (pl.splits != 1 || layout != 3 || (cols & 7) != 0 || nt < 32) return nullptr;
    if (stochastic && (cols & 63) == 8 && nt < kCUs / 2) return nullptr;
    if (with_stats && nt > kCUs && nt <= round) return nullptr;
    bool pays = true;
    if (upd.states == 0) pays = nt <= round || (nt >= round + round * 3 / 4 && nt <= 2 * round);
    else if (upd.states == 1) pays = nt <= round || nt > round + round / 4 || with_stats;
    else pays = nt == round || nt >= round + round * 3 / 8 || (with_stats && nt > round + round / 4);
    return pays ? kernels[upd.states] : nullptr;
}

// Upper bound of the workspace: one FP32 tile set per contraction slice.  (The MFMA kernels
// finish their tiles themselves for an unsplit contraction with a row length that is a multiple
// of 16, unless most of a tile lies beyond the matrix (poorly_filled); otherwise they write FP32
// tiles and the finishing kernel takes over.)
static size_t plan_workspace(const Plan &pl, int64_t rows, int64_t cols) {
    if (!pl.mfma) return 0;
    return (size_t)pl.splits * (size_t)rows * (size_t)cols * sizeof(float);
}

}  // namespace mp8

extern "C" int mp8_gemm_num_tile_configs(void) { return mp8::kNumTiles; }

extern "C" int mp8_gemm_tile_config_name(int tile_config, char *buf, size_t buflen) {
    if (tile_config < 1 || tile_config > mp8::kNumTiles || !buf || buflen == 0) return -1;
    snprintf(buf, buflen, "%s", mp8::kTiles[tile_config - 1].name);
    return 0;
}

extern "C" int mp8_gemm_tile_config_lds_bytes(int tile_config, int epi) {
    if (tile_config < 1 || tile_config > mp8::kNumTiles || epi < 0 || epi > 2) return -1;
    hipFuncAttributes at;
    const mp8::TileConfig &tc = mp8::kTiles[tile_config - 1];
    const void *fn = tc.kernel[epi] ? (const void *)tc.kernel[epi] : (const void *)tc.kernel_tn[epi];
    if (fn == nullptr || hipFuncGetAttributes(&at, fn) != hipSuccess) return -1;
    return (int)at.sharedSizeBytes;
}

extern "C" size_t mp8_gemm_fp8_workspace_bytes_tuned(mp8_op op, int64_t M, int64_t N, int64_t K,
                                                     int tile_config, int split_k) {
    using namespace mp8;
    if (M <= 0 || N <= 0 || K <= 0 || (int)op < 0 || (int)op > 2) return 0;
    if (tile_config < 0 || tile_config > kNumTiles || split_k < 0) return 0;
    int64_t rows, cols, kc;
    op_dims(op, M, N, K, rows, cols, kc);
    // enough for every operand layout and alignment (and, with an incomplete stage, for the 8-bit gradient of a
    // weight gradient with an update)
    size_t need = 0;
    for (int layout : {0, 2, 3}) {
        const int64_t k = tile_config == 0 && half_takes(rows, cols, kc, layout) ? (kc + BK - 1) / BK * BK : kc;
        need = std::max(need, plan_workspace(make_plan(rows, cols, k, tile_config, split_k, layout), rows, cols));
    }
    if (tile_config == 0) {  // the slices of gemm_any_kernel side by side
        const Plan pl = any_plan(rows, cols, kc);
        if (pl.splits > 1) need = std::max(need, (size_t)pl.splits * (size_t)rows * (size_t)cols * sizeof(float));
    }
    return need;
}

extern "C" mp8_status mp8_gemm_fp8_plan(mp8_op op, int64_t M, int64_t N, int64_t K, int flags,
                                        int tile_config, int split_k, int *tile_out,
                                        int *splits_out) {
    using namespace mp8;
    if (M <= 0 || N <= 0 || K <= 0 || (int)op < 0 || (int)op > 2) return MP8_ERR_INVALID_ARG;
    if (tile_config < 0 || tile_config > kNumTiles || split_k < 0) return MP8_ERR_INVALID_ARG;
    const bool atn = (flags & MP8_FLAG_A_CONTRACTION_MAJOR) != 0, btn = (flags & MP8_FLAG_B_CONTRACTION_MAJOR) != 0;
    if (atn && !btn) return MP8_ERR_UNSUPPORTED;
    int64_t rows, cols, kc;
    op_dims(op, M, N, K, rows, cols, kc);
    const Plan pl = plan_of(rows, cols, kc, tile_config, split_k, (atn ? 1 : 0) | (btn ? 2 : 0),
                            (flags & MP8_FLAG_SATURATE) == 0 && (cols & 15) == 0);
    if (tile_out) *tile_out = pl.mfma ? pl.tile + 1 : 0;
    if (splits_out) *splits_out = pl.splits;
    return MP8_OK;
}

extern "C" size_t mp8_gemm_fp8_workspace_bytes(mp8_op op, int64_t M, int64_t N, int64_t K) {
    return mp8_gemm_fp8_workspace_bytes_tuned(op, M, N, K, 0, 0);
}

namespace mp8 {

// Outputs from which a transposed copy can be a pass of its own (see copied_from_codes).
constexpr int64_t kTransposeFrom = 1 << 23;

// Is the transposed copy made from the finished codes by a pass of its own (transpose_codes_kernel), or stored with them byte
// by byte?  With them / by the pass, us:
//   rounded by a finishing pass, whose lanes lie along the rows: 64 x 64 (contraction 16384) 8.7 / 10.4, 600 x 600 8.7 / 11.1, 512 x 512 12.6 / 13.7,
//         1000 x 1000 13.7 / 13.1, 3000 x 3000 83 / 32, 64000 x 100 32 / 24; but 200000 x 20 28.4 / 29.2, 1000 x 48 8.7 / 12.4: tiles of 128
//         columns and rows that are not there
//   256x256 tiles: codes alone leave them much faster.  To nearest 4096 x 4096 x 1024 37.3 / 29.3, 131072 x 64 x 1024 66.1 / 45.0; stochastic
//         4096 x 4096 x 1024 40.1 / 39.9, 8192 x 4096 x 1024 76.8 / 73.3
//   other aligned kernels, to nearest: 4096 x 4096 x 256 19.2 / 21.0, 8192 x 4096 x 256 32.7 / 30.0, x 128 34.3 / 30.8, in one load of the whole
//         contraction 23.7 / 28.5; 4096 x 2048 x 1024 17.8 / 18.6, x 4096 36.3 / 34.8; few columns or rows 131072 x 64 x 256 20.2 / 16.9, 256 x
//         65536 x 256 21.1 / 19.3, 262144 x 32 x 128 29.3 / 20.9; half-precision 4096 x 4096 x 144 24.2 / 25.1, 8192 x 4096 x 144 42.6 / 37.5, 4096 x 2048 x 2064 40.5 / 39.3
//   with another rounding the complete epilogue runs either way: half-precision stochastic 6000 x 6000 x 1040 100 / 106
//   gemm_any_kernel, which has one epilogue: 4096 x 4088 x 200 43.9 / 49.5, 2900 x 2900 x 500 28.6 / 35.7
static bool copied_from_codes(const Plan &pl, int64_t rows, int64_t cols, int64_t kc, bool two_pass, bool nearest_codes) {
    const int64_t n = rows * cols;
    if (two_pass) return n >= 3 << 18 && rows >= 64 && cols >= 64;
    if (!pl.mfma || n < kTransposeFrom) return false;
    const TileConfig &t = kTiles[pl.tile];
    if (!pl.half && t.bm * t.bn == 256 * 256) return true;
    if (!nearest_codes || (t.max_ksteps > 0 && kc <= BK)) return false;
    const double products = (double)n * (double)kc;
    if (pl.half) return n >= 1 << 25 || products >= 0x1p32;
    return n >= 1 << 25 || products >= (n >= 1 << 24 ? 0x1p33 : 0x1p35) || std::min(rows, cols) <= 256;
}

// Tiles so much of which lies beyond the matrix that their epilogue, which walks all of it, takes longer with an FP32 or a
// transposed result than a finishing pass over what there is (us, finishing pass / epilogue):
//   256x256   65536 rows, contraction 1024: FP32 beside the codes 48 columns 29.2 / 35.0, 80 34.8 / 35.9, 96 36.3 / 35.9; added to
//             64 35.5 / 52.1, 160 53.5 / 55.6, 320 95.9 / 102.7, 400 124.9 / 106.1; transposed 48 32.0 / 34.1, 64 37.6 / 34.5
//   128x128   16 columns: one tile per CU (32768 x 512) transposed, stochastic 9.5 / 10.9; two 65536 x 512 13.9 / 12.5, beside 13.3 / 12.1, added
//             to 14.1 / 18.2; many 262144 x 128 transposed, stochastic 26.8 / 33.5, beside 24.9 / 30.3; 32 columns: many 262144 x 128 added to
//             37.9 / 51.5, beside 34.0 / 33.7; 32768 x 2048 added to 21.3 / 24.6, x 512 11.1 / 11.2; 16 rows by 524288 x 128 added to 45.3 / 49.4
//   contractions of one or two stages, whose lanes lie along the rows: 7 by 200000 transposed 19.6 / 26.0, 16 by 524288 63 / 26, added to 39.6 / 43.5
static bool poorly_filled(const Plan &pl, int64_t rows, int64_t cols, int acc_mode, bool transposed, int64_t ksteps) {
    const TileConfig &t = kTiles[pl.tile];
    if (t.max_ksteps > 0) return (transposed && rows <= 8) || (acc_mode == 2 && rows <= 16);
    const int64_t nt = (int64_t)pl.tiles_m * pl.tiles_n;
    const double of_cols = (double)cols / ((double)pl.tiles_n * t.bn), of_tile = of_cols * (double)rows / ((double)pl.tiles_m * t.bm);
    if (t.bm * t.bn == 256 * 256) return acc_mode == 2 ? of_tile < 0.7 : of_cols < (acc_mode == 1 ? 0.375 : 0.25);
    if (t.bm * t.bn == 128 * 128) {
        if (acc_mode == 2) return of_cols <= 0.125 || (of_cols <= 0.25 && ksteps >= 16) || (nt > 2 * kCUs && of_tile <= 0.25);
        return of_cols <= 0.125 && (nt <= kCUs || nt > 2 * kCUs);
    }
    return false;
}

// More 256x256 tiles than CUs, codes to nearest: the kernel whose workgroups take several of them (null: another kernel).
static void (*stream_kernel(void (*const pick[3])(const GemmArgs), bool unit))(const GemmArgs) {
    const TileConfig &t = kTiles[T256x256];
    if (pick == t.kernel) return unit ? gemm_stream_kernel<false, false, true> : gemm_stream_kernel<false, false, false>;
    if (pick == t.kernel_bt) return unit ? gemm_stream_kernel<false, true, true> : gemm_stream_kernel<false, true, false>;
    if (pick == t.kernel_tn) return unit ? gemm_stream_kernel<true, true, true> : gemm_stream_kernel<true, true, false>;
    return nullptr;
}

// Launch the MFMA kernel chosen by `pick` (indexed by EPI_*) for plan `pl`, and the finishing
// kernel when the epilogue cannot be fused.  `ga` carries the operands; its tiling, slicing and
// epilogue fields are filled in here.
static mp8_status launch_mfma(GemmArgs ga, Epilogue ep, const Plan &pl, int64_t kc,
                              void (*const pick[3])(const GemmArgs), void *workspace,
                              size_t workspace_bytes, hipStream_t s, const UpdateHook *upd = nullptr,
                              bool validate_only = false, UpdateKernel with_update = nullptr) {
    const int64_t rows = ep.rows, cols = ep.cols;
    const int acc_mode = ep.acc_mode;
    float *acc = ep.acc;
    uint8_t *out8 = ep.out8;
    auto has_workspace = [&] {
        return workspace != nullptr && workspace_bytes >= (size_t)pl.splits * (size_t)rows * (size_t)cols * sizeof(float);
    };
    // With these outputs some tiles are finished by a second pass (poorly_filled); which ones is not the caller's concern, so
    // the 8-bit kernels ask for a workspace with all of them, as the header says.
    if (pl.mfma && !pl.half && (acc_mode == 2 || (ep.out8_t != nullptr && !(acc_mode == 1 && pl.splits == 1))) && !has_workspace())
        return MP8_ERR_WORKSPACE;
    // Fused epilogue or two passes?  An FP32 result alone is the tiles as the kernels write them; with codes the epilogues
    // do both.  (The master-weight update lives in the finishing pass or in an update kernel; the epilogues
    // of gemm_any_kernel and the half-precision forms take any row length.)
    const bool acc_alone = acc_mode == 1 && out8 == nullptr && ep.out8_t == nullptr && ep.stats == nullptr;
    const bool nearest_codes = acc_mode == 0 && out8 != nullptr && !ep.sr && !ep.sat && ep.stats == nullptr;
    const bool poor = pl.mfma && !pl.half && pl.conv_rows == 0 && ep.mask == 0 && (acc_mode != 0 || ep.out8_t != nullptr) &&
                      poorly_filled(pl, rows, cols, acc_mode, ep.out8_t != nullptr, kc / BK);
    // (of a large result codes to nearest alone, and the copy from them, are shorter still: 524288 x 16 x 128 34 us, by a finishing pass 42)
    const bool codes_first = poor && nearest_codes && rows * cols >= kTransposeFrom;
    const bool two_pass = (pl.splits > 1 && !pl.in_turn) || (upd != nullptr && with_update == nullptr) ||
                          (pl.mfma && !pl.half && ((cols & 15) != 0 || acc_alone)) || (poor && !codes_first);
    uint8_t *const copy_t = out8 != nullptr && (codes_first || copied_from_codes(pl, rows, cols, kc, two_pass, nearest_codes))
                                ? ep.out8_t : nullptr;
    if (copy_t != nullptr) ep.out8_t = nullptr;
    uint8_t *const out8_t = ep.out8_t;
    float *partial = nullptr;
    Epilogue fin = ep;  // what the finishing kernel applies
    fin.want_codes = upd != nullptr;
    if (two_pass) {
        if (pl.splits == 1 && acc_mode == 1) {
            partial = acc;  // the tile goes straight into acc; the finishing kernel reads it there
            fin.acc = nullptr;
            fin.acc_mode = 0;
        } else {
            if (!has_workspace()) return MP8_ERR_WORKSPACE;
            partial = (float *)workspace;
        }
    }
    const int64_t nblocks = (int64_t)pl.tiles_m * pl.tiles_n * (pl.in_turn ? 1 : pl.splits);
    // The FP32 result beside the codes leaves line by line, unless the grid leaves half of the CUs idle (then its stores do not matter,
    // and storing it with the codes is shorter: half-precision 64 x 64 x 64 3.7 -> 3.5 us, 512 x 512 x 528 6.1 -> 5.7, 8-bit 512 x
    // 512 x 512 4.5 -> 4.3; where it is added to, only half-precision) and, half-precision, in rows that fill no tile (65536 x 32 x 272 13.4 -> 12.6).
    ep.acc_lines = acc_mode != 0 && (cols & 15) == 0 &&
                   (pl.half ? nblocks > kCUs / 2 && std::min(rows, cols) >= (ep.sr && acc_mode == 1 ? 65 : 64) : acc_mode == 2 || nblocks > kCUs / 2);
    // What is added to by the next call as well stays in the L2s while they hold it (32 MB).  Past them / into them, us: added to, with
    // codes, 64 x 64 x 128 4.3 / 3.7, 128 x 512 x 256 5.0 / 4.2, 2048 x 2048 x 256 (16 MB) 13.8 / 12.0; 4096 x 4096 x 512 (64 MB) as fast,
    // 8192 x 8192 x 512 194 / 201.
    if (ep.acc_lines != 0 && acc_mode == 2 && rows * cols <= (int64_t)1 << 23) ep.acc_lines = 2;
    // The codes of the complete epilogue of 64x64 tiles, whose waves store them 32 bytes of a line at a time, go past the L2 where tiles of a second
    // round overlap with that, and where statistics follow them.  Past it / into it: beside an FP32 result 64 x 64 x 128 3.05 / 2.86, 512 x 512
    // x 256 3.64 / 3.50; added to 3.83 / 3.65 and 4.48 / 4.32; stochastic 1024 x 1024 (256 tiles) 1.5 % longer, 1024 x 2048 2 % shorter; with statistics
    // 3 % shorter (1024 x 512) to 6 % (1024 x 2048).
    ep.codes_plain = pl.mfma && kTiles[pl.tile].bm * kTiles[pl.tile].bn == 64 * 64 && nblocks <= kCUs && (acc_mode != 0 || ep.stats == nullptr);
    if (nblocks > 0x7FFFFFFFLL) return MP8_ERR_UNSUPPORTED;
    if (validate_only) return MP8_OK;  // every check has passed; nothing is enqueued

    ga.rows = rows;
    ga.cols = cols;
    ga.ksteps = (int)((kc + BK - 1) / BK);
    ga.tail = (int)(kc % BK);
    ga.splits = pl.splits;
    ga.tiles_m = pl.tiles_m;
    ga.tiles_n = pl.tiles_n;
    ga.div_tiles = make_fastdiv((uint32_t)(pl.tiles_m * pl.tiles_n));
    ga.div_band = make_fastdiv((uint32_t)(8 * pl.tiles_n));
    ga.div_tail = make_fastdiv((uint32_t)((pl.tiles_m & 7) ? (pl.tiles_m & 7) : 8));
    ga.div_tn = make_fastdiv((uint32_t)pl.tiles_n);
    ga.ks_per = ga.ksteps / pl.splits;
    ga.ks_extra = ga.ksteps % pl.splits;
    ga.partial = partial;
    ga.ep = ep;
    const bool complete = ep.sr || ep.sat || ep.stats != nullptr || out8 == nullptr || !pl.mfma || (cols & 15) != 0 ||
                          acc_mode != 0 || out8_t != nullptr;
    const int epi = two_pass ? EPI_PARTIAL : complete ? EPI_FULL : EPI_RNE;
    const size_t dyn_lds = pl.mfma ? (size_t)kTiles[pl.tile].lds_per_stage * (size_t)ga.ksteps : 0;
    if (with_update != nullptr && !two_pass) {
        hipLaunchKernelGGL(with_update, dim3((unsigned)nblocks), dim3(256), 0, s, ga, *upd);
        return hipGetLastError() == hipSuccess ? MP8_OK : MP8_ERR_HIP;
    }
    if (const auto stream = epi == EPI_RNE && nblocks > kCUs && ga.ksteps >= 2 ? stream_kernel(pick, ep.alpha == 1.0f) : nullptr)
        hipLaunchKernelGGL(stream, dim3(kCUs), dim3(256), 0, s, ga);
    else
        hipLaunchKernelGGL(pick[epi], dim3((unsigned)nblocks), dim3(256), dyn_lds, s, ga);
    if (hipGetLastError() != hipSuccess) return MP8_ERR_HIP;
    if (two_pass) {
        const bool only_acc = fin.acc_mode == 0 && fin.out8 == nullptr && fin.out8_t == nullptr &&
                              fin.stats == nullptr && upd == nullptr;
        if (!only_acc) {
            const int64_t items = (cols & 3) == 0 ? rows * cols / 4 : rows * cols;
            int64_t blocks = std::min<int64_t>((items + 255) / 256, 256 * 16);
            const int states = upd ? upd->states : -1;
            static void (*const finish[4][3])(const float *, int, const Epilogue, const UpdateHook) = {
                {splitk_finish_kernel<-1, 1>, splitk_finish_kernel<-1, 4>, splitk_finish_kernel<-1, 8>},
                {splitk_finish_kernel<0, 1>, splitk_finish_kernel<0, 4>, splitk_finish_kernel<0, 8>},
                {splitk_finish_kernel<1, 1>, splitk_finish_kernel<1, 4>, splitk_finish_kernel<1, 8>},
                {splitk_finish_kernel<2, 1>, splitk_finish_kernel<2, 4>, splitk_finish_kernel<2, 8>}};
            hipLaunchKernelGGL(finish[states + 1][pl.splits == 1 ? 0 : pl.splits <= 4 ? 1 : 2],
                               dim3((unsigned)blocks), dim3(256), 0, s, (const float *)partial, pl.splits, fin,
                               upd ? *upd : UpdateHook{});
            if (hipGetLastError() != hipSuccess) return MP8_ERR_HIP;
        }
    }
    if (copy_t != nullptr) {
        const int64_t tiles = (rows + 127) / 128 * ((cols + 127) / 128);
        hipLaunchKernelGGL(((rows | cols) & 15) == 0 ? transpose_codes_kernel<true> : transpose_codes_kernel<false>,
                           dim3((unsigned)std::min<int64_t>(tiles, 1 << 20)), dim3(256), 0, s, out8, copy_t, rows, cols);
        if (hipGetLastError() != hipSuccess) return MP8_ERR_HIP;
    }
    return MP8_OK;
}

}  // namespace mp8

namespace mp8 {

// mp8_gemm_fp8_tuned, optionally with the master-weight update applied to the rounded result
// (`upd`; the finishing pass or an update kernel carries it, MP8_ERR_UNSUPPORTED if the call has neither).
static mp8_status gemm_impl(mp8_op op, int64_t M, int64_t N, int64_t K, const uint8_t *a, int64_t lda,
                            const uint8_t *b, int64_t ldb, float alpha, float *acc, int acc_mode,
                            uint8_t *out8, uint8_t *out8_t, mp8_round round, int flags, uint64_t seed,
                            uint64_t offset, mp8_stats *stats, void *workspace, size_t workspace_bytes,
                            void *stream, int tile_config, int split_k, const UpdateHook *upd,
                            bool validate_only = false) {
    if ((int)op < 0 || (int)op > 2) return MP8_ERR_INVALID_ARG;
    if (M < 0 || N < 0 || K < 0) return MP8_ERR_INVALID_ARG;
    if (round != MP8_RNE && round != MP8_SR) return MP8_ERR_INVALID_ARG;
    if (acc_mode < 0 || acc_mode > 2) return MP8_ERR_INVALID_ARG;
    if (tile_config < 0 || tile_config > kNumTiles || split_k < 0) return MP8_ERR_INVALID_ARG;
    int64_t rows, cols, kc;
    op_dims(op, M, N, K, rows, cols, kc);
    if (rows == 0 || cols == 0) return MP8_OK;
    if (acc_mode != 0 && acc == nullptr) return MP8_ERR_INVALID_ARG;
    if (kc > 0 && (!a || !b)) return MP8_ERR_INVALID_ARG;
    const bool atn = (flags & MP8_FLAG_A_CONTRACTION_MAJOR) != 0;
    const bool btn = (flags & MP8_FLAG_B_CONTRACTION_MAJOR) != 0;
    if (atn && !btn) return MP8_ERR_UNSUPPORTED;  // no kernel is built for this combination
    if (kc > 0 && (lda < (atn ? rows : kc) || ldb < (btn ? cols : kc))) return MP8_ERR_INVALID_ARG;
    if (rows > (INT64_MAX / 8) / cols) return MP8_ERR_UNSUPPORTED;
    if (((uintptr_t)acc | (uintptr_t)out8 | (uintptr_t)out8_t | (uintptr_t)workspace) & 15u)
        return MP8_ERR_ALIGNMENT;

    Epilogue ep{};
    ep.alpha = alpha;
    ep.acc = acc_mode ? acc : nullptr;
    ep.acc_mode = acc_mode;
    ep.out8 = out8;
    ep.out8_t = out8_t;
    ep.sr = round == MP8_SR;
    ep.sat = (flags & MP8_FLAG_SATURATE) ? 1 : 0;
    ep.seed = seed;
    ep.offset = offset;
    ep.stats = stats;
    ep.rows = rows;
    ep.cols = cols;
    hipStream_t s = (hipStream_t)stream;

    const int layout = (atn ? 1 : 0) | (btn ? 2 : 0);
    const bool codes_alone = upd == nullptr && acc_mode == 0 && out8 != nullptr && out8_t == nullptr && stats == nullptr && !ep.sr && !ep.sat &&
                             (cols & 15) == 0;
    Plan pl = plan_of(rows, cols, kc, tile_config, split_k, layout, codes_alone);
    // the direct-to-LDS kernels want 16-byte aligned rows and 32-bit offsets inside a 256-row tile
    const bool aligned = (((uintptr_t)a | (uintptr_t)b) & 15u) == 0 && (lda & 15) == 0 &&
                         (ldb & 15) == 0 && lda < (1 << 24) && ldb < (1 << 24);
    if (pl.mfma && !aligned) {
        if (tile_config > 0) return MP8_ERR_ALIGNMENT;
        pl.mfma = false;
    }
    if (tile_config > 0 && !pl.mfma) return MP8_ERR_UNSUPPORTED;
    if (!pl.mfma && aligned) pl = half_plan(rows, cols, kc, layout);
    auto has_workspace = [&](int splits) {
        return workspace != nullptr && workspace_bytes >= (size_t)splits * (size_t)rows * (size_t)cols * sizeof(float);
    };
    if (!pl.mfma && any_kernel_takes(rows, cols, kc, lda, ldb, layout)) {
        pl = any_plan(rows, cols, kc);
        // it never needs a workspace: without one a split contraction takes its slices in turn
        pl.in_turn = pl.splits == 1 || !has_workspace(pl.splits);
        // (the update goes with the finishing pass or an unsplit call's epilogue: otherwise two launches)
        const UpdateKernel with_update =
            upd != nullptr && out8 != nullptr ? any_update_kernel(pl, cols, layout, *upd, stats != nullptr, ep.sr || upd->sr) : nullptr;
        if (upd != nullptr && pl.in_turn && with_update == nullptr) return MP8_ERR_UNSUPPORTED;
        GemmArgs ga{};
        ga.a = a;
        ga.b = b;
        ga.lda = lda;
        ga.ldb = ldb;
        void (*const *kern)(const GemmArgs) = kAny[atn ? 2 : btn ? 1 : 0];
        void (*whole)(const GemmArgs) = kern[pl.splits > 1 ? 2 : 1];
        if (any_in_32_rows(pl, kc, layout)) {  // (the same bits: the order of the additions does not depend on the tile)
            whole = kAny32[btn];
            pl.tiles_m = (int)((rows + 31) / 32);
        }
        void (*const pick[3])(const GemmArgs) = {kern[0], nullptr, whole};
        return launch_mfma(ga, ep, pl, kc, pick, workspace, workspace_bytes, s, upd, validate_only, with_update);
    }
    if (!pl.mfma || kc == 0) {
        if (upd != nullptr) return MP8_ERR_UNSUPPORTED;
        if (validate_only) return MP8_OK;
        int64_t blocks = std::min<int64_t>((rows * cols + 255) / 256, 1 << 20);
        hipLaunchKernelGGL(gemm_generic_kernel, dim3((unsigned)blocks), dim3(256), 0, s, a, lda, b,
                           ldb, kc, layout, ep);
        return hipGetLastError() == hipSuccess ? MP8_OK : MP8_ERR_HIP;
    }

    GemmArgs ga{};
    ga.a = a;
    ga.b = b;
    ga.lda = lda;
    ga.ldb = ldb;
    const UpdateKernel with_update = upd != nullptr ? update_kernel(pl, cols, layout, upd->states, out8 != nullptr) : nullptr;
    if (pl.half) {
        if (upd != nullptr && with_update == nullptr) return MP8_ERR_UNSUPPORTED;  // (two launches)
        const int form = pl.tile == T64x64s2 ? 0 : pl.tile == T64x64w ? 1 : 2;
        return launch_mfma(ga, ep, pl, kc, kHalf[form][atn ? 2 : btn ? 1 : 0], nullptr, 0, s, upd, validate_only, with_update);
    }
    const TileConfig &tc = kTiles[pl.tile];
    return launch_mfma(ga, ep, pl, kc, atn ? tc.kernel_tn : btn ? tc.kernel_bt : tc.kernel, workspace,
                       workspace_bytes, s, upd, validate_only, with_update);
}

// The checks of mp8_gemm_fp8 on these arguments without enqueuing anything: what a call made of
// several launches runs first, so that it is rejected as a whole or not at all.
static mp8_status gemm_validate(mp8_op op, int64_t M, int64_t N, int64_t K, const uint8_t *a, int64_t lda,
                                const uint8_t *b, int64_t ldb, float *acc, int acc_mode, uint8_t *out8,
                                uint8_t *out8_t, mp8_round round, int flags, void *workspace,
                                size_t workspace_bytes) {
    return gemm_impl(op, M, N, K, a, lda, b, ldb, 1.0f, acc, acc_mode, out8, out8_t, round, flags, 0, 0, nullptr,
                     workspace, workspace_bytes, nullptr, 0, 0, nullptr, true);
}

// Does the skip flag of a fused weight-gradient update live inside the statistics the same call
// accumulates into?  The finishing pass reads the flag when it starts and adds this gradient's
// Inf/NaN count when it ends, so such a flag would change under the pass that reads it; those
// calls run the weight gradient and the update as two launches instead, and the update then sees
// the final count.
static bool flag_inside_stats(const uint32_t *skip, const mp8_stats *stats) {
    if (skip == nullptr || stats == nullptr) return false;
    const uintptr_t f = (uintptr_t)skip, s0 = (uintptr_t)stats;
    return f + sizeof(uint32_t) > s0 && f < s0 + sizeof(mp8_stats);
}


// The master-weight update a finishing pass applies: plain SGD, or momentum SGD with L2
// regularisation when a velocity array is given (mp8_wgrad_adam_fp16_sr fills in ADAM's fields).
static UpdateHook make_update_hook(uint16_t *w16, uint8_t *w8_out, const uint32_t *skip, float lr,
                                   float inv_loss_scale, mp8_round w_round, uint64_t w_seed, uint64_t w_offset,
                                   float *velocity = nullptr, float momentum = 0.0f, float weight_decay = 0.0f) {
    UpdateHook upd{};
    upd.w16 = w16;
    upd.w8_out = w8_out;
    upd.skip = skip;
    upd.neg_lr = -lr;
    upd.inv_scale = inv_loss_scale;
    upd.sr = w_round == MP8_SR;
    upd.seed = w_seed;
    upd.offset = w_offset;
    upd.states = velocity != nullptr ? 1 : 0;
    upd.state0 = velocity;
    upd.mu = momentum;
    upd.wd = weight_decay;
    return upd;
}

// Where the 8-bit weight gradient goes when the update is cheaper as a launch of its own: a
// weight-gradient GEMM that runs unsplit rounds in its own epilogue, and forcing a finishing pass
// on it just to carry the update would write and re-read the whole FP32 result (measured: 1024 x
// 4096 from 16384 tokens 91 against 77 us).  Then the codes go to g8_out, or to the workspace if
// the caller keeps no gradient, and the stand-alone update kernel follows.  Null: use the
// finishing pass -- or, with own_epilogue, the GEMM kernel whose epilogue carries the update.
static uint8_t *codes_for_separate_update(int64_t M, int64_t N, int64_t K, int flags, uint8_t *g8_out,
                                          void *workspace, size_t workspace_bytes, bool own_epilogue,
                                          int states) {
    const bool atn = (flags & MP8_FLAG_A_CONTRACTION_MAJOR) != 0, btn = (flags & MP8_FLAG_B_CONTRACTION_MAJOR) != 0;
    if ((atn && !btn) || (N & 15) != 0 || K > (INT64_MAX / 8) / std::max<int64_t>(N, 1)) return nullptr;
    const Plan pl = make_plan(K, N, M, 0, 0, (atn ? 1 : 0) | (btn ? 2 : 0));
    if (!pl.mfma || pl.splits != 1) return nullptr;
    if (own_epilogue && update_kernel(pl, N, (atn ? 1 : 0) | (btn ? 2 : 0), states, g8_out != nullptr) != nullptr) return nullptr;
    if (g8_out != nullptr) return g8_out;
    return workspace != nullptr && workspace_bytes >= (size_t)(K * N) ? (uint8_t *)workspace : nullptr;
}
}  // namespace mp8

extern "C" mp8_status mp8_gemm_fp8_tuned(mp8_op op, int64_t M, int64_t N, int64_t K,
                                         const uint8_t *a, int64_t lda, const uint8_t *b,
                                         int64_t ldb, float alpha, float *acc, int acc_mode,
                                         uint8_t *out8, uint8_t *out8_t, mp8_round round,
                                         int flags, uint64_t seed, uint64_t offset,
                                         mp8_stats *stats, void *workspace,
                                         size_t workspace_bytes, void *stream, int tile_config,
                                         int split_k) {
    return mp8::gemm_impl(op, M, N, K, a, lda, b, ldb, alpha, acc, acc_mode, out8, out8_t, round, flags,
                          seed, offset, stats, workspace, workspace_bytes, stream, tile_config, split_k,
                          nullptr);
}

namespace mp8 {

// Weight gradient, its rounding, and a master-weight update of the rounded codes (Figure 1b): the
// body the three optimizer variants share.  `hook` is the rule as the finishing pass applies it,
// `update_from(codes)` launches the same rule's stand-alone kernel on codes in memory.  Three ways,
// all with the same results: the update inside the finishing pass of a split contraction, or inside the
// GEMM's own epilogue (unsplit outputs, see update_kernel and any_update_kernel), or the GEMM followed by the
// update kernel (larger ones, and a skip flag that lives inside `stats` -- see flag_inside_stats).  Whatever
// can be checked is checked before the first launch.
template <class UpdateFrom>
static mp8_status wgrad_with_update(int64_t M, int64_t N, int64_t K, const uint8_t *a, int64_t lda,
                                    const uint8_t *b, int64_t ldb, float alpha, uint8_t *g8_out,
                                    mp8_round g_round, int flags, uint64_t g_seed, uint64_t g_offset,
                                    mp8_stats *stats, const UpdateHook &hook, void *workspace,
                                    size_t workspace_bytes, void *stream, UpdateFrom update_from) {
    auto two_launches = [&](uint8_t *codes, void *ws, size_t ws_bytes) -> mp8_status {
        const mp8_status sv = gemm_validate(MP8_WGRAD, M, N, K, a, lda, b, ldb, nullptr, 0, codes, nullptr,
                                            g_round, flags, ws, ws_bytes);
        if (sv != MP8_OK) return sv;
        const mp8_status sg = mp8_gemm_fp8(MP8_WGRAD, M, N, K, a, lda, b, ldb, alpha, nullptr, 0, codes, nullptr,
                                           g_round, flags, g_seed, g_offset, stats, ws, ws_bytes, stream);
        if (sg != MP8_OK) return sg;
        return update_from(codes);
    };
    const bool late_flag = flag_inside_stats(hook.skip, stats);
    if (uint8_t *codes = codes_for_separate_update(M, N, K, flags, g8_out, workspace, workspace_bytes, !late_flag,
                                                   hook.states))
        return two_launches(codes, nullptr, 0);
    if (late_flag)
        return g8_out != nullptr ? two_launches(g8_out, workspace, workspace_bytes) : MP8_ERR_INVALID_ARG;
    const mp8_status st = gemm_impl(MP8_WGRAD, M, N, K, a, lda, b, ldb, alpha, nullptr, 0, g8_out, nullptr,
                                    g_round, flags, g_seed, g_offset, stats, workspace, workspace_bytes,
                                    stream, 0, 0, &hook);
    if (st != MP8_ERR_UNSUPPORTED) return st;
    // nothing to carry the update (unaligned operands, ...): two launches through the 8-bit gradient, which lies
    // in the workspace if the caller keeps none
    if (g8_out != nullptr) return two_launches(g8_out, workspace, workspace_bytes);
    uint8_t *codes = codes_for_separate_update(M, N, K, flags, nullptr, workspace, workspace_bytes, false, hook.states);
    const int layout = ((flags & MP8_FLAG_A_CONTRACTION_MAJOR) ? 1 : 0) | ((flags & MP8_FLAG_B_CONTRACTION_MAJOR) ? 2 : 0);
    if (half_takes(K, N, M, layout) && K <= (INT64_MAX / 8) / N && workspace != nullptr && workspace_bytes >= (size_t)(K * N))
        codes = (uint8_t *)workspace;
    return codes != nullptr ? two_launches(codes, nullptr, 0) : st;
}

}  // namespace mp8

extern "C" mp8_status mp8_wgrad_update_fp16_sr(int64_t M, int64_t N, int64_t K, const uint8_t *a,
                                               int64_t lda, const uint8_t *b, int64_t ldb, float alpha,
                                               uint8_t *g8_out, mp8_round g_round, int flags,
                                               uint64_t g_seed, uint64_t g_offset, mp8_stats *stats,
                                               uint16_t *w16, float lr, float inv_loss_scale,
                                               mp8_round w_round, uint64_t w_seed, uint64_t w_offset,
                                               const uint32_t *skip_if_nonzero, uint8_t *w8_out,
                                               void *workspace, size_t workspace_bytes, void *stream) {
    using namespace mp8;
    if (M < 0 || N < 0 || K < 0) return MP8_ERR_INVALID_ARG;
    if (w_round != MP8_RNE && w_round != MP8_SR) return MP8_ERR_INVALID_ARG;
    if (K == 0 || N == 0) return MP8_OK;
    if (!w16) return MP8_ERR_INVALID_ARG;
    if (((uintptr_t)w16 | (uintptr_t)w8_out) & 15u) return MP8_ERR_ALIGNMENT;
    const UpdateHook upd = make_update_hook(w16, w8_out, skip_if_nonzero, lr, inv_loss_scale, w_round, w_seed, w_offset);
    return wgrad_with_update(M, N, K, a, lda, b, ldb, alpha, g8_out, g_round, flags, g_seed, g_offset, stats, upd,
                             workspace, workspace_bytes, stream, [&](const uint8_t *codes) {
        return mp8_sgd_update_fp16_sr(w16, codes, K * N, lr, inv_loss_scale, w_round, w_seed, w_offset,
                                      skip_if_nonzero, w8_out, nullptr, stream);
    });
}

extern "C" mp8_status mp8_wgrad_momentum_fp16_sr(int64_t M, int64_t N, int64_t K, const uint8_t *a, int64_t lda,
                                                 const uint8_t *b, int64_t ldb, float alpha, uint8_t *g8_out,
                                                 mp8_round g_round, int flags, uint64_t g_seed,
                                                 uint64_t g_offset, mp8_stats *stats, uint16_t *w16,
                                                 float *velocity, float lr, float inv_loss_scale,
                                                 float momentum, float weight_decay, mp8_round w_round,
                                                 uint64_t w_seed, uint64_t w_offset,
                                                 const uint32_t *skip_if_nonzero, uint8_t *w8_out,
                                                 void *workspace, size_t workspace_bytes, void *stream) {
    using namespace mp8;
    if (M < 0 || N < 0 || K < 0) return MP8_ERR_INVALID_ARG;
    if (w_round != MP8_RNE && w_round != MP8_SR) return MP8_ERR_INVALID_ARG;
    if (K == 0 || N == 0) return MP8_OK;
    if (!w16 || !velocity) return MP8_ERR_INVALID_ARG;
    if (((uintptr_t)w16 | (uintptr_t)w8_out | (uintptr_t)velocity) & 15u) return MP8_ERR_ALIGNMENT;
    const UpdateHook upd = make_update_hook(w16, w8_out, skip_if_nonzero, lr, inv_loss_scale, w_round, w_seed, w_offset,
                                            velocity, momentum, weight_decay);
    return wgrad_with_update(M, N, K, a, lda, b, ldb, alpha, g8_out, g_round, flags, g_seed, g_offset, stats, upd,
                             workspace, workspace_bytes, stream, [&](const uint8_t *codes) {
        return mp8_sgd_momentum_fp16_sr(w16, velocity, codes, K * N, lr, inv_loss_scale, momentum, weight_decay,
                                        w_round, w_seed, w_offset, skip_if_nonzero, w8_out, nullptr, stream);
    });
}

extern "C" mp8_status mp8_wgrad_adam_fp16_sr(int64_t M, int64_t N, int64_t K, const uint8_t *a, int64_t lda,
                                             const uint8_t *b, int64_t ldb, float alpha, uint8_t *g8_out,
                                             mp8_round g_round, int flags, uint64_t g_seed, uint64_t g_offset,
                                             mp8_stats *stats, uint16_t *w16, float *m, float *v, float lr,
                                             float inv_loss_scale, float beta1, float beta2, float eps,
                                             float weight_decay, int64_t step, mp8_round w_round,
                                             uint64_t w_seed, uint64_t w_offset,
                                             const uint32_t *skip_if_nonzero, uint8_t *w8_out,
                                             void *workspace, size_t workspace_bytes, void *stream) {
    using namespace mp8;
    if (M < 0 || N < 0 || K < 0 || step < 1) return MP8_ERR_INVALID_ARG;
    if (w_round != MP8_RNE && w_round != MP8_SR) return MP8_ERR_INVALID_ARG;
    if (K == 0 || N == 0) return MP8_OK;
    if (!w16 || !m || !v) return MP8_ERR_INVALID_ARG;
    if (((uintptr_t)w16 | (uintptr_t)w8_out | (uintptr_t)m | (uintptr_t)v) & 15u) return MP8_ERR_ALIGNMENT;
    UpdateHook upd = make_update_hook(w16, w8_out, skip_if_nonzero, lr, inv_loss_scale, w_round, w_seed, w_offset);
    upd.states = 2;
    upd.state0 = m;
    upd.state1 = v;
    upd.wd = weight_decay;
    upd.b1 = beta1;
    upd.b2 = beta2;
    upd.omb1 = 1.0f - beta1;
    upd.omb2 = 1.0f - beta2;
    // bias corrections as in mp8_adam_fp16_sr: the powers in double, the result as FP32
    upd.ric1 = 1.0 / (double)(float)(1.0 - std::pow((double)beta1, (double)step));
    upd.ric2 = 1.0 / (double)(float)(1.0 - std::pow((double)beta2, (double)step));
    upd.eps = eps;
    return wgrad_with_update(M, N, K, a, lda, b, ldb, alpha, g8_out, g_round, flags, g_seed, g_offset, stats, upd,
                             workspace, workspace_bytes, stream, [&](const uint8_t *codes) {
        return mp8_adam_fp16_sr(w16, m, v, codes, K * N, lr, inv_loss_scale, beta1, beta2, eps, weight_decay, step,
                                w_round, w_seed, w_offset, skip_if_nonzero, w8_out, nullptr, stream);
    });
}

extern "C" mp8_status mp8_gemm_fp8(mp8_op op, int64_t M, int64_t N, int64_t K, const uint8_t *a,
                                   int64_t lda, const uint8_t *b, int64_t ldb, float alpha,
                                   float *acc, int acc_mode, uint8_t *out8, uint8_t *out8_t,
                                   mp8_round round, int flags, uint64_t seed, uint64_t offset,
                                   mp8_stats *stats, void *workspace, size_t workspace_bytes,
                                   void *stream) {
    return mp8_gemm_fp8_tuned(op, M, N, K, a, lda, b, ldb, alpha, acc, acc_mode, out8, out8_t,
                              round, flags, seed, offset, stats, workspace, workspace_bytes,
                              stream, 0, 0);
}

// ---------------------------------------------------------------------------------------
// mp8_gemm_fp8 for callers that cannot allocate: the scratch of the two-pass paths (FP32 tiles of
// the contraction slices, unfused epilogues) lives in a static device array of this library.
namespace mp8 {

constexpr size_t kStaticScratchBytes = (size_t)MP8_STATIC_SCRATCH_BYTES;
// Every GPU the library runs on holds its own copy of this array, at an address of its own, until
// the process ends.  In host code the name is only a handle for hipGetSymbolAddress: kernels get
// the device address looked up below, never the name.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
static void *g_scratch_ptr[kMaxDevices];   // device address of `scratch` per device, once looked up
static std::mutex g_scratch_mutex;

// Device address of the current device's copy of `scratch` (looked up once per device).
static mp8_status static_scratch(void **out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return MP8_ERR_HIP;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_ptr[dev] == nullptr) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) {
            (void)hipGetLastError();
            return MP8_ERR_HIP;
        }
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return MP8_OK;
}

}  // namespace mp8

extern "C" size_t mp8_static_scratch_bytes(void) { return mp8::kStaticScratchBytes; }

extern "C" mp8_status mp8_gemm_fp8_static(mp8_op op, int64_t M, int64_t N, int64_t K, const uint8_t *a,
                                          int64_t lda, const uint8_t *b, int64_t ldb, float alpha,
                                          float *acc, int acc_mode, uint8_t *out8, uint8_t *out8_t,
                                          mp8_round round, int flags, uint64_t seed, uint64_t offset,
                                          mp8_stats *stats, void *stream) {
    using namespace mp8;
    // the same bound the workspace query gives the callers of mp8_gemm_fp8
    if (M > 0 && N > 0 && K > 0 && (int)op >= 0 && (int)op <= 2) {
        int64_t rows, cols, kc;
        op_dims(op, M, N, K, rows, cols, kc);
        // (a contraction that is not whole stages runs without a workspace where this one is too small)
        if (kc % BK == 0 &&
            mp8_gemm_fp8_workspace_bytes(op, M, N, K) > kStaticScratchBytes)
            return MP8_ERR_WORKSPACE;
    }
    void *ws = nullptr;
    const mp8_status ss = static_scratch(&ws);
    if (ss != MP8_OK) return ss;
    // Nothing in the scratch has to start at zero: every FP32 tile element the finishing pass
    // reads has been written by this call's first kernel.
    return gemm_impl(op, M, N, K, a, lda, b, ldb, alpha, acc, acc_mode, out8, out8_t, round, flags, seed,
                     offset, stats, ws, kStaticScratchBytes, stream, 0, 0, nullptr);
}

// ---------------------------------------------------------------------------------------
// GEMMs that quantise their own FP32 operand

extern "C" mp8_status mp8_quantize_gemm_fwd_fp8(int64_t M, int64_t N, int64_t K, const float *x,
                                                float x_scale, mp8_round x_round, int x_flags,
                                                uint64_t x_seed, uint64_t x_offset, mp8_stats *x_stats,
                                                uint8_t *x8_out, const uint8_t *w8, int64_t ldw,
                                                float alpha, float *acc, int acc_mode, uint8_t *out8,
                                                uint8_t *out8_t, mp8_round round, int flags,
                                                uint64_t seed, uint64_t offset, mp8_stats *stats,
                                                void *workspace, size_t workspace_bytes, void *stream) {
    using namespace mp8;
    if (M < 0 || N < 0 || K < 0) return MP8_ERR_INVALID_ARG;
    if ((x_round != MP8_RNE && x_round != MP8_SR) || (round != MP8_RNE && round != MP8_SR))
        return MP8_ERR_INVALID_ARG;
    if (acc_mode < 0 || acc_mode > 2) return MP8_ERR_INVALID_ARG;
    if (M == 0) return MP8_OK;  // nothing to round, nothing to multiply
    if (acc_mode != 0 && acc == nullptr && N > 0) return MP8_ERR_INVALID_ARG;
    if (K > 0 && (!x || !x8_out)) return MP8_ERR_INVALID_ARG;
    if (N > 0 && K > 0 && (!w8 || ldw < N)) return MP8_ERR_INVALID_ARG;
    if (((uintptr_t)x | (uintptr_t)x8_out | (uintptr_t)acc | (uintptr_t)out8 | (uintptr_t)out8_t) & 15u)
        return MP8_ERR_ALIGNMENT;
    // Up to 128 columns the activations are read once.  More column tiles round them again each, which pays while it
    // costs less than the launch it saves: few tiles, short contractions, and a rounding that is cheap to repeat (GPU time, us, two
    // launches / one kernel):
    //   nearest, codes only     1 x 1024 x 128 4.3 / 3.7, 1024 x 1024 x 128 5.0 / 4.1; 1 x 4096 x 256 4.55 / 4.7, 16 x 1024 x 256 5.0 / 4.65, 256 x 256 x
    //                           256 5.2 / 4.8, 4096 x 256 x 256 5.6 / 5.0; 256 x 1024 x 512 6.2 / 6.1, 4096 x 256 x 512 7.2 / 6.5; 64 x 1024 x 512 6.1 / 6.5
    //   stochastic x            1024 x 1024 x 128 5.15 / 6.3, 256 x 256 x 256 5.45 / 8.3, 1024 x 1024 x 512 6.8 / 13.3: never
    //   saturated x             1024 x 1024 x 128 5.1 / 5.3, 256 x 256 x 256 5.3 / 7.1: never
    //   statistics of x         64 x 1024 x 128 5.4 / 5.6, 1024 x 1024 x 128 6.9 / 6.1, 256 x 256 x 256 6.5 / 8.0, 1024 x 1024 x 256 8.9 / 8.2,
    //                           4096 x 256 x 512 10.7 / 12.5 (statistics make the Q node slow, but only once)
    //   complete epilogue       stochastic 64 x 1024 x 128 5.5 / 5.2, 256 x 256 x 256 6.1 / 6.1, 1024 x 1024 x 256 6.4 / 6.3, 1024 x 1024 x 512
    //                           7.5 / 7.7, 4096 x 256 x 512 8.2 / 7.8; FP32 beside codes 1024 x 1024 x 512 8.0 / 8.0, 4096 x 256 x 512 8.7 / 8.3;
    //                           transposed 1024 x 1024 x 128 6.2 / 5.8, 1024 x 1024 x 256 6.7 / 6.8, 4096 x 256 x 512 8.5 / 8.2; saturated
    //                           64 x 1024 x 128 5.5 / 5.2, 4096 x 256 x 256 6.6 / 6.7; acc += 1024 x 1024 x 128 6.9 / 7.3: never; FP32 alone 1024 x 1024 x 128
    //                           5.4 / 5.4, 1024 x 1024 x 256 5.9 / 6.3
    const int64_t ctiles = (N + 127) / 128;
    const bool narrow = N <= 128;
    const bool plain = acc_mode == 0 && out8_t == nullptr && round == MP8_RNE && !(flags & MP8_FLAG_SATURATE) && stats == nullptr &&
                       out8 != nullptr;
    const bool qplain = x_round == MP8_RNE && !(x_flags & MP8_FLAG_SATURATE) && x_stats == nullptr;
    const bool few = K <= 4 * BK && M <= 64 * 128 && ctiles <= 128 && (M + 63) / 64 * ctiles <= 128 &&
                     M >= (K <= BK ? 1 : K <= 2 * BK ? 16 : 256);
    const bool cheap_x = qplain || (x_round == MP8_RNE && !(x_flags & MP8_FLAG_SATURATE) && M >= 1024 && K <= 2 * BK);
    const bool cheap_out = plain || (acc_mode != 2 && (K <= BK || (out8 != nullptr && !(flags & MP8_FLAG_SATURATE) &&
                                                                   M >= (out8_t != nullptr ? 8 : 4) * K)));
    const bool small = few && cheap_x && cheap_out;
    const bool fused = N >= 16 && (narrow || small) && (N & 15) == 0 && K > 0 && (K & (BK - 1)) == 0 &&
                       ((uintptr_t)w8 & 15u) == 0 && (ldw & 15) == 0 && ldw < (1 << 24) &&
                       M <= (INT64_MAX / 8) / K && (M + 63) / 64 <= 0x7FFFFFFFLL;
    // (beyond 128 columns, the checks of the two calls this one stands for: what they refuse stays refused)
    if (!narrow && N > 0 && K > 0) {
        const mp8_status sv = gemm_validate(MP8_FWD, M, N, K, x8_out, K, w8, ldw, acc, acc_mode, out8, out8_t, round,
                                            (flags & MP8_FLAG_SATURATE) | MP8_FLAG_B_CONTRACTION_MAJOR, workspace, workspace_bytes);
        if (sv != MP8_OK) return sv;
    }
    if (!fused) {
        // any other shape: the two calls this one stands for (the second one's checks first, so
        // that a rejected call has enqueued nothing)
        const int gflags = (flags & MP8_FLAG_SATURATE) | MP8_FLAG_B_CONTRACTION_MAJOR;
        if (narrow && N > 0 && K > 0) {
            const mp8_status sv = gemm_validate(MP8_FWD, M, N, K, x8_out, K, w8, ldw, acc, acc_mode, out8, out8_t,
                                                round, gflags, workspace, workspace_bytes);
            if (sv != MP8_OK) return sv;
        }
        const mp8_status sq = mp8_quantize_e5m2(x, 0, x8_out, nullptr, M, K, x_scale, x_round, x_flags,
                                                x_seed, x_offset, x_stats, stream);
        if (sq != MP8_OK) return sq;
        return mp8_gemm_fp8(MP8_FWD, M, N, K, x8_out, K, w8, ldw, alpha, acc, acc_mode, out8, out8_t,
                            round, gflags, seed, offset, stats, workspace, workspace_bytes, stream);
    }
    GemmArgs ga{};
    ga.b = w8;
    ga.ldb = ldw;
    ga.rows = M;
    ga.cols = N;
    ga.ksteps = (int)(K / BK);
    ga.splits = 1;
    Epilogue &ep = ga.ep;
    ep.alpha = alpha;
    ep.acc = acc_mode ? acc : nullptr;
    ep.acc_mode = acc_mode;
    ep.out8 = out8;
    ep.out8_t = out8_t;
    ep.sr = round == MP8_SR;
    ep.sat = (flags & MP8_FLAG_SATURATE) ? 1 : 0;
    ep.seed = seed;
    ep.offset = offset;
    ep.stats = stats;
    ep.rows = M;
    ep.cols = N;
    QuantArgs qa{};
    qa.x = x;
    qa.x8 = x8_out;
    qa.scale = x_scale;
    qa.sr = x_round == MP8_SR;
    qa.sat = (x_flags & MP8_FLAG_SATURATE) ? 1 : 0;
    qa.seed = x_seed;
    qa.offset = x_offset;
    qa.stats = x_stats;
    // 128 rows per workgroup once that still gives every other CU a workgroup
    const bool tall = narrow && (M + 127) / 128 >= 128;
    void (*kernel)(const GemmArgs, const QuantArgs);
    if (tall)
        kernel = plain ? (qplain ? gemm_qfwd_kernel<EPI_RNE, true, 128> : gemm_qfwd_kernel<EPI_RNE, false, 128>)
                       : (qplain ? gemm_qfwd_kernel<EPI_FULL, true, 128> : gemm_qfwd_kernel<EPI_FULL, false, 128>);
    else
        kernel = plain ? (qplain ? gemm_qfwd_kernel<EPI_RNE, true, 64> : gemm_qfwd_kernel<EPI_RNE, false, 64>)
                       : (qplain ? gemm_qfwd_kernel<EPI_FULL, true, 64> : gemm_qfwd_kernel<EPI_FULL, false, 64>);
    const int bm = tall ? 128 : 64;
    hipLaunchKernelGGL(kernel, dim3((unsigned)((M + bm - 1) / bm), (unsigned)ctiles), dim3(4 * bm + 256), 0,
                       (hipStream_t)stream, ga, qa);
    return hipGetLastError() == hipSuccess ? MP8_OK : MP8_ERR_HIP;
}

// ---------------------------------------------------------------------------------------
// 3x3 convolution as an implicit GEMM on zero-padded channels-last tensors
// ---------------------------------------------------------------------------------------
namespace mp8 {

struct ConvDims {
    int64_t rows, cols, kc;  // of the implicit GEMM
    int64_t lda, ldb;
};

static bool conv_dims(mp8_op op, int64_t prows, int64_t Ci, int64_t Co, ConvDims &d) {
    switch (op) {
        case MP8_FWD: d = {prows, Co, 9 * Ci, Ci, Co}; return true;
        case MP8_BWD_DATA: d = {prows, Ci, 9 * Co, Co, Co}; return true;
        case MP8_WGRAD: d = {9 * Ci, Co, prows, Ci, Co}; return true;
    }
    return false;
}

// Stages of the implicit GEMM's contraction: whole stages of 128, the last one starting 64 early
// when forward / backward data contract over an odd number of 64-channel units.
static int64_t conv_kc_stages(const ConvDims &d) { return (d.kc + BK - 1) / BK * BK; }

static Plan conv_plan(mp8_op op, const ConvDims &d, int64_t Ci, int64_t W) {
    // Forward and backward data: the kernel that keeps a tile's pixel rows in LDS, while they fit.  256 rows per tile from
    // one and a half tiles per CU on: 32 x 56 x 56 x 64 (421) 7.7 us, in tiles of 128 8.3, 17 x 33 x 33, 128 to 512 (656) 16.8 and 17.5,
    // 41 x 17 x 17, 192 to 320 (290) 13.5 and 12.6.
    // Never in slices, also where tiles are few and the contraction is long: codes alone are faster whole (forward, general
    // kernel in slices / this one: 2 x 7 x 7, 512 to 512 12.5 / 11.0, 512 to 128 11.6 / 10.9, 256 to 256 11.6 / 7.0), and slices
    // would ask for a workspace.  What is slower are complete epilogues on some 30 workgroups and less with 512 contracted
    // channels, whose latency nothing covers (2 x 7 x 7, 512 to 128: with statistics 12.0 / 12.3, an FP32 result 11.6 / 12.1,
    // added to 11.7 / 13.8, with all of it 12.6 / 15.1; 256 to 256 added to 11.8 / 9.8).
    if (op != MP8_WGRAD && 2 * (W + 3) <= kConvHalo) {
        Plan pl{};
        pl.mfma = true;
        pl.tile = T128x64s2;
        pl.conv_rows = (d.rows + 255) / 256 * (d.cols / 64) >= kCUs + kCUs / 2 ? 256 : 128;
        pl.tiles_m = (int)((d.rows + pl.conv_rows - 1) / pl.conv_rows);
        pl.tiles_n = (int)(d.cols / 64);
        pl.splits = 1;
        return pl;
    }
    // Wider images, and the weight gradient, take the general kernels:
    // the tile shapes built for contraction-major operands are the ones built for convolutions
    const int64_t kc = conv_kc_stages(d);
    Plan pl = make_plan(d.rows, d.cols, kc, 0, 0, 3, true);
    // a tile row of the weight gradient must not straddle two taps
    if (pl.mfma && op == MP8_WGRAD && (Ci % kTiles[pl.tile].bm) != 0)
        pl = make_plan(d.rows, d.cols, kc, ((Ci & 127) == 0 ? T128x128s2 : T64x64s2) + 1, 0, 3, true);
    // forward and backward data have one tile row per 128 pixels and few tile columns: the
    // 128-row tile keeps the re-reads of the weights low; it is also the tile whose kernels are
    // built for stages that span two taps (contracted channels an odd multiple of 64)
    if (pl.mfma && op != MP8_WGRAD && (kTiles[pl.tile].bm < 128 || (d.kc / 9 / 64) % 2 != 0))
        pl = make_plan(d.rows, d.cols, kc, T128x128s2 + 1, 0, 3, true);
    // ... and for 64 output columns a 128x64 tile of the same kind (tile geometry and slices as
    // for the row-major kernel of that shape)
    if (pl.mfma && op != MP8_WGRAD && (d.kc / 9 / 64) % 2 != 0 && d.cols == 64)
        pl = make_plan(d.rows, d.cols, kc, T128x64s2 + 1, 0, 0, true);
    return pl;
}

// gemm_conv_kernel: [rows per tile / 128 - 1][op][EPI_*]
#define MP8_CONV_OP(BM, BTN) \
    {gemm_conv_kernel<BM, EPI_PARTIAL, BTN>, gemm_conv_kernel<BM, EPI_RNE, BTN>, gemm_conv_kernel<BM, EPI_FULL, BTN>}
static void (*const kConv[2][2][3])(const GemmArgs) = {{MP8_CONV_OP(128, true), MP8_CONV_OP(128, false)},
                                                       {MP8_CONV_OP(256, true), MP8_CONV_OP(256, false)}};

// Forward / backward data with the contracted channel count an odd multiple of 64: [op][EPI_*]
static void (*const kConvHalves[2][3])(const GemmArgs) = {
    {gemm_mfma_kernel<128, 128, 2, 2, 2, 2, EPI_PARTIAL, false, true, 4>,
     gemm_mfma_kernel<128, 128, 2, 2, 2, 2, EPI_RNE, false, true, 4>,
     gemm_mfma_kernel<128, 128, 2, 2, 2, 2, EPI_FULL, false, true, 4>},
    {gemm_mfma_kernel<128, 128, 2, 2, 2, 2, EPI_PARTIAL, false, false, 5>,
     gemm_mfma_kernel<128, 128, 2, 2, 2, 2, EPI_RNE, false, false, 5>,
     gemm_mfma_kernel<128, 128, 2, 2, 2, 2, EPI_FULL, false, false, 5>}};
// the same for 64 output columns
static void (*const kConvHalves64[2][3])(const GemmArgs) = {
    {gemm_mfma_kernel<128, 64, 4, 1, 2, 3, EPI_PARTIAL, false, true, 4>,
     gemm_mfma_kernel<128, 64, 4, 1, 2, 3, EPI_RNE, false, true, 4>,
     gemm_mfma_kernel<128, 64, 4, 1, 2, 3, EPI_FULL, false, true, 4>},
    {gemm_mfma_kernel<128, 64, 4, 1, 2, 3, EPI_PARTIAL, false, false, 5>,
     gemm_mfma_kernel<128, 64, 4, 1, 2, 3, EPI_RNE, false, false, 5>,
     gemm_mfma_kernel<128, 64, 4, 1, 2, 3, EPI_FULL, false, false, 5>}};

}  // namespace mp8

extern "C" size_t mp8_conv3x3_fp8_workspace_bytes(mp8_op op, int64_t B, int64_t H, int64_t W,
                                                  int64_t Ci, int64_t Co, int64_t prows) {
    using namespace mp8;
    ConvDims d;
    if (B <= 0 || H <= 0 || W <= 0 || Ci <= 0 || Co <= 0 || prows <= 0) return 0;
    if (!conv_dims(op, prows, Ci, Co, d)) return 0;
    return plan_workspace(conv_plan(op, d, Ci, W), d.rows, d.cols);
}

namespace mp8 {

// mp8_conv3x3_fp8, optionally (weight gradient only) with the master-weight update applied to
// the rounded result by the finishing pass.
static mp8_status conv_impl(mp8_op op, int64_t B, int64_t H, int64_t W, int64_t Ci, int64_t Co,
                            int64_t prows, const uint8_t *a, const uint8_t *b, float alpha, float *acc,
                            int acc_mode, uint8_t *out8, mp8_round round, int flags, uint64_t seed,
                            uint64_t offset, mp8_stats *stats, void *workspace, size_t workspace_bytes,
                            void *stream, const UpdateHook *upd) {
    ConvDims d;
    if (B < 0 || H < 0 || W < 0 || Ci < 0 || Co < 0 || prows < 0) return MP8_ERR_INVALID_ARG;
    if (!conv_dims(op, prows, Ci, Co, d)) return MP8_ERR_INVALID_ARG;
    if (round != MP8_RNE && round != MP8_SR) return MP8_ERR_INVALID_ARG;
    if (acc_mode < 0 || acc_mode > 2) return MP8_ERR_INVALID_ARG;
    if (flags & ~MP8_FLAG_SATURATE) return MP8_ERR_INVALID_ARG;
    if (B == 0 || H == 0 || W == 0 || Ci == 0 || Co == 0) return MP8_OK;
    const int64_t img = (H + 2) * (W + 2);
    if (B > (int64_t)0x7FFFFFFF / img || prows < B * img || prows > 0x7FFFFFFF) return MP8_ERR_INVALID_ARG;
    if (!a || !b || (acc_mode != 0 && !acc)) return MP8_ERR_INVALID_ARG;
    // whole 64-byte halves of a stage per tap, whole tiles per tap of the weight gradient; lane
    // offsets (a tile's rows, a filter row's shift, a tap's weight slab) stay within 32 bits
    if ((Ci & 63) != 0 || (Co & 63) != 0 || Ci >= (1 << 15) || Co >= (1 << 15) || W >= (1 << 15))
        return MP8_ERR_UNSUPPORTED;
    if (op == MP8_WGRAD && (prows & 127) != 0) return MP8_ERR_UNSUPPORTED;
    if (((uintptr_t)a | (uintptr_t)b | (uintptr_t)acc | (uintptr_t)out8 | (uintptr_t)workspace) & 15u)
        return MP8_ERR_ALIGNMENT;
    const Plan pl = conv_plan(op, d, Ci, W);
    if (!pl.mfma) return MP8_ERR_UNSUPPORTED;

    Epilogue ep{};
    ep.alpha = alpha;
    ep.acc = acc_mode ? acc : nullptr;
    ep.acc_mode = acc_mode;
    ep.out8 = out8;
    ep.sr = round == MP8_SR;
    ep.sat = (flags & MP8_FLAG_SATURATE) ? 1 : 0;
    ep.seed = seed;
    ep.offset = offset;
    ep.stats = stats;
    ep.rows = d.rows;
    ep.cols = d.cols;
    if (op != MP8_WGRAD) {
        ep.mask = 1;
        ep.hh = (int)(H + 2);
        ep.valid_rows = B * img;
        ep.div_img = make_fastdiv((uint32_t)img);
        ep.div_w2 = make_fastdiv((uint32_t)(W + 2));
    }
    GemmArgs ga{};
    ga.a = a;
    ga.b = b;
    ga.lda = d.lda;
    ga.ldb = d.ldb;
    ga.cv.w2 = (int)(W + 2);
    ga.cv.units_per_tap = (int)((op == MP8_BWD_DATA ? Co : Ci) / 64);
    ga.cv.div_cpb = make_fastdiv((uint32_t)ga.cv.units_per_tap);
    ga.cv.odd_units = op != MP8_WGRAD && (d.kc % BK) != 0;
    ga.cv.b_tap_stride = Ci * Co;
    ga.cv.div_ci = make_fastdiv((uint32_t)Ci);
    if (pl.conv_rows != 0)  // (a chunk of 64 channels is a stage of its contraction)
        return launch_mfma(ga, ep, pl, (int64_t)ga.cv.units_per_tap * BK, kConv[pl.conv_rows / 128 - 1][(int)op], workspace,
                           workspace_bytes, (hipStream_t)stream, upd);
    const bool halves = op != MP8_WGRAD && (ga.cv.units_per_tap & 1) != 0;
    if (halves && pl.tile != T128x128s2 && pl.tile != T128x64s2) return MP8_ERR_UNSUPPORTED;
    return launch_mfma(ga, ep, pl, conv_kc_stages(d),
                       !halves ? kTiles[pl.tile].kernel_conv[(int)op]
                               : pl.tile == T128x64s2 ? kConvHalves64[(int)op] : kConvHalves[(int)op],
                       workspace, workspace_bytes,
                       (hipStream_t)stream, upd);
}

}  // namespace mp8

extern "C" mp8_status mp8_conv3x3_fp8(mp8_op op, int64_t B, int64_t H, int64_t W, int64_t Ci,
                                      int64_t Co, int64_t prows, const uint8_t *a,
                                      const uint8_t *b, float alpha, float *acc, int acc_mode,
                                      uint8_t *out8, mp8_round round, int flags, uint64_t seed,
                                      uint64_t offset, mp8_stats *stats, void *workspace,
                                      size_t workspace_bytes, void *stream) {
    return mp8::conv_impl(op, B, H, W, Ci, Co, prows, a, b, alpha, acc, acc_mode, out8, round, flags, seed,
                          offset, stats, workspace, workspace_bytes, stream, nullptr);
}

extern "C" mp8_status mp8_conv3x3_wgrad_update_fp16_sr(
    int64_t B, int64_t H, int64_t W, int64_t Ci, int64_t Co, int64_t prows, const uint8_t *x8,
    const uint8_t *e8, float alpha, uint8_t *g8_out, mp8_round g_round, int flags, uint64_t g_seed,
    uint64_t g_offset, mp8_stats *stats, uint16_t *w16, float lr, float inv_loss_scale,
    mp8_round w_round, uint64_t w_seed, uint64_t w_offset, const uint32_t *skip_if_nonzero,
    uint8_t *w8_out, void *workspace, size_t workspace_bytes, void *stream) {
    using namespace mp8;
    if (w_round != MP8_RNE && w_round != MP8_SR) return MP8_ERR_INVALID_ARG;
    if (B == 0 || H == 0 || W == 0 || Ci == 0 || Co == 0) return MP8_OK;
    if (!w16) return MP8_ERR_INVALID_ARG;
    if (((uintptr_t)w16 | (uintptr_t)w8_out) & 15u) return MP8_ERR_ALIGNMENT;
    if (flag_inside_stats(skip_if_nonzero, stats)) {
        // the flag is still being counted while the finishing pass would read it: two launches
        if (g8_out == nullptr) return MP8_ERR_INVALID_ARG;
        const mp8_status sg = conv_impl(MP8_WGRAD, B, H, W, Ci, Co, prows, x8, e8, alpha, nullptr, 0, g8_out, g_round,
                                        flags, g_seed, g_offset, stats, workspace, workspace_bytes, stream, nullptr);
        if (sg != MP8_OK) return sg;
        return mp8_sgd_update_fp16_sr(w16, g8_out, 9 * Ci * Co, lr, inv_loss_scale, w_round, w_seed, w_offset,
                                      skip_if_nonzero, w8_out, nullptr, stream);
    }
    UpdateHook upd = make_update_hook(w16, w8_out, skip_if_nonzero, lr, inv_loss_scale, w_round, w_seed, w_offset);
    return conv_impl(MP8_WGRAD, B, H, W, Ci, Co, prows, x8, e8, alpha, nullptr, 0, g8_out, g_round, flags,
                     g_seed, g_offset, stats, workspace, workspace_bytes, stream, &upd);
}

extern "C" mp8_status mp8_conv3x3_wgrad_momentum_fp16_sr(
    int64_t B, int64_t H, int64_t W, int64_t Ci, int64_t Co, int64_t prows, const uint8_t *x8,
    const uint8_t *e8, float alpha, uint8_t *g8_out, mp8_round g_round, int flags, uint64_t g_seed,
    uint64_t g_offset, mp8_stats *stats, uint16_t *w16, float *velocity, float lr, float inv_loss_scale,
    float momentum, float weight_decay, mp8_round w_round, uint64_t w_seed, uint64_t w_offset,
    const uint32_t *skip_if_nonzero, uint8_t *w8_out, void *workspace, size_t workspace_bytes,
    void *stream) {
    using namespace mp8;
    if (w_round != MP8_RNE && w_round != MP8_SR) return MP8_ERR_INVALID_ARG;
    if (B == 0 || H == 0 || W == 0 || Ci == 0 || Co == 0) return MP8_OK;
    if (!w16 || !velocity) return MP8_ERR_INVALID_ARG;
    if (((uintptr_t)w16 | (uintptr_t)w8_out | (uintptr_t)velocity) & 15u) return MP8_ERR_ALIGNMENT;
    if (flag_inside_stats(skip_if_nonzero, stats)) {
        if (g8_out == nullptr) return MP8_ERR_INVALID_ARG;
        const mp8_status sg = conv_impl(MP8_WGRAD, B, H, W, Ci, Co, prows, x8, e8, alpha, nullptr, 0, g8_out, g_round,
                                        flags, g_seed, g_offset, stats, workspace, workspace_bytes, stream, nullptr);
        if (sg != MP8_OK) return sg;
        return mp8_sgd_momentum_fp16_sr(w16, velocity, g8_out, 9 * Ci * Co, lr, inv_loss_scale, momentum,
                                        weight_decay, w_round, w_seed, w_offset, skip_if_nonzero, w8_out, nullptr,
                                        stream);
    }
    UpdateHook upd = make_update_hook(w16, w8_out, skip_if_nonzero, lr, inv_loss_scale, w_round, w_seed, w_offset,
                                      velocity, momentum, weight_decay);
    return conv_impl(MP8_WGRAD, B, H, W, Ci, Co, prows, x8, e8, alpha, nullptr, 0, g8_out, g_round, flags,
                     g_seed, g_offset, stats, workspace, workspace_bytes, stream, &upd);
}
