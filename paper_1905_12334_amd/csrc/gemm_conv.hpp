// Forward and backward data of the 3x3 convolution: the pixel rows a tile needs lie in LDS once, for all nine taps.
#pragma once

#include "gemm_common.hpp"
#include "gemm_epilogue.hpp"

namespace mp8 {

// On the zero-padded pixel grid a filter tap is a shift of the pixel row by up to W + 3, so a tile of BM output
// rows reads BM + 2 (W + 3) pixel rows, nine times over.  The general kernel fetches them nine times, a stage of 128
// contraction indices at a time, with a barrier and a wait per stage: a chain of latencies (32 x 56 x 56, 64 to 64
// channels, 12.6 us for 5 us of traffic).  Here the contraction is cut into chunks of 64 channels: a
// chunk is the slab of those pixel rows (64 bytes each) and the 64x64 weight blocks of all nine taps (36 KB), all of
// it in LDS at once, and the nine taps are multiplied from there.  256 threads, wave w owns rows w BM/4 .. and
// all 64 output columns.
//   BM = 128  53 KB: three workgroups on a CU cover each other's loads
//   BM = 256  60 KB, where the epilogue takes FP32 bands 68 KB: two; half the LDS reads of weights per product, for grids
//             that still give every CU one or two
// While a chunk is multiplied, the weights of the next one take the place of the filter rows that are done; the
// slab follows at its end.  (A second slab for the next chunk leaves room for two workgroups of BM = 128 only: 26 x 56 x
// 56, 256 to 64 channels 14.2 us, with it 16.7.  No refill at all: 2 x 28 x 28, 512 to 512 12.2 and 13.4.)  The plan
// takes the contraction whole (see conv_plan).
// Measured, forward / backward data, before and after: 32 x 28 x 28 x 128 9.5 / 9.2 and 8.2 / 8.0 us, 32 x 56 x 56 x 64 12.6
// / 12.7 and 7.7 / 7.6, 26 x 56 x 56, 256 to 64 27.5 / 24.9 and 14.2 / 17.0, 45 x 7 x 7, 64 to 128 7.0 / 8.0 and 4.1 / 5.1.
// BTN: forward (w [9 Cin, Cout] contraction-major); else backward data (w [tap][Cin][Cout], rows of a tap's slab).
// LDS images: 64-byte rows, chunk c of slab row r in slot c ^ ((r >> 2) & 3): the sixteen lanes that are served
// together read sixteen consecutive rows -- from any first row, as the taps want -- of one chunk, and fall into
// sixteen different 16-byte bank groups.  Contraction-major weights: the narrow image of the general kernel.
template <int BM, int EPI, bool BTN>
__global__ __launch_bounds__(256, BM == 256 ? 2 : 3) void gemm_conv_kernel(const GemmArgs p) {
    constexpr int BN = 64, MT = BM / 128, NT = 2;
    constexpr int SLAB = (BM + kConvHalo) * 64, TAP = 64 * 64;
    constexpr int EP_BYTES = EPI == EPI_RNE ? 0 : 4 * MT * 32 * (BN + 4) * 4;  // FP32 bands of the epilogue
    constexpr int LDS_BYTES = SLAB + 9 * TAP > EP_BYTES ? SLAB + 9 * TAP : EP_BYTES;
    __shared__ __attribute__((aligned(1024))) uint8_t lds[LDS_BYTES];
    const uint8_t *const taps = lds + SLAB;

    int split, tm, tn;
    map_block(p, split, tm, tn);
    split = __builtin_amdgcn_readfirstlane(split);
    tm = __builtin_amdgcn_readfirstlane(tm);
    tn = __builtin_amdgcn_readfirstlane(tn);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t row0 = (int64_t)tm * BM, col0 = (int64_t)tn * BN;
    const int first = split * p.ks_per + (split < p.ks_extra ? split : p.ks_extra);
    const int count = __builtin_amdgcn_readfirstlane(p.ks_per + (split < p.ks_extra ? 1 : 0));
    const int halo = p.cv.w2 + 1;  // slab row j is pixel row row0 - halo + j
    // Loads of the slab: sixteen rows each, load q of this wave brings rows 16 (wave + 4q) ..; lane i lands at (row
    // i/4, slot i%4).  Rows beyond the last guard row are clamped to it (they only feed rows that are not stored).
    const bool tall = 2 * halo > kConvHalo / 2;   // the last load of each wave is needed
    constexpr int A_DMA = (BM + kConvHalo) / 64;
    const int64_t last_row = p.rows - 1 + halo - (row0 - halo);
    uint32_t oa[A_DMA];
#pragma unroll
    for (int q = 0; q < A_DMA; ++q) {
        int64_t r = 16 * (wave + 4 * q) + (lane >> 2);
        r = r < last_row ? r : last_row;
        oa[q] = (uint32_t)(r * p.lda) + 16 * ((lane & 3) ^ ((lane >> 4) & 3));
    }
    // the weights of a tap: 64 rows of 64 bytes, sixteen by each wave
    const int brow = 16 * wave + (lane >> 2);
    const uint32_t ob = (uint32_t)(brow * p.ldb) + 16 * (BTN ? (lane & 3) ^ (((lane >> 4) & 1) << 1) : (lane & 3) ^ ((lane >> 4) & 3));
    const uint8_t *a_tile = uniform_ptr(p.a + (row0 - halo) * p.lda + 64 * first);
    const uint8_t *b_tile = uniform_ptr(BTN ? p.b + col0 + 64 * first * p.ldb : p.b + col0 * p.ldb + 64 * first);
    const int64_t b_chunk = BTN ? 64 * p.ldb : 64, b_tap = p.cv.b_tap_stride;
    const uint32_t lds0 = lds_address(lds) + wave * 1024;
    auto issue_slab = [&](int c) {
#pragma unroll
        for (int q = 0; q < A_DMA; ++q)
            if (q < A_DMA - 1 || tall) dma16(a_tile + 64 * c, oa[q], lds0 + q * 4096);
    };
    auto issue_taps = [&](int c, int row) {  // the three taps of a filter row
        const uint8_t *bc = b_tile + c * b_chunk;
#pragma unroll
        for (int tap = 3 * row; tap < 3 * row + 3; ++tap) dma16(bc + tap * b_tap, ob, lds0 + SLAB + tap * TAP);
    };

    f32x16 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
    const int frow = lane & 31, fkb = lane >> 5;
    // 32 codes of row r (chunks 2 fkb and the next) of an image of 64-byte rows
    auto row_fragment = [&](const uint8_t *image, int r) -> i32x8 {
        const int at = r * 64 + (((2 * fkb) ^ ((r >> 2) & 3)) << 4);
        const i32x4 h0 = *reinterpret_cast<const i32x4 *>(image + at);
        const i32x4 h1 = *reinterpret_cast<const i32x4 *>(image + (at ^ 16));
        return __builtin_shufflevector(h0, h1, 0, 1, 2, 3, 4, 5, 6, 7);
    };

    issue_slab(0);
#pragma unroll
    for (int row = 0; row < 3; ++row) issue_taps(0, row);
    for (int c = 0; c < count; ++c) {
        const bool more = c + 1 < count;
#pragma unroll
        for (int row = 0; row < 3; ++row) {
            // Wait until this filter row's weights (with the first, the slab) have landed: loads complete in the order
            // of their issue, and three of a later filter row may fly.  Behind the barrier they have for every wave, and
            // nobody reads the filter row before this one any more.  A single chunk waits once, for everything.
            __builtin_amdgcn_sched_barrier(0);
            if (row == 0) {
                if (c > 0) {
                    wait_vm_lds<63>();
                    __syncthreads();
                    issue_slab(c);
                    issue_taps(c, 2);
                    wait_vm_lds<3>();
                } else if (count > 1) {
                    wait_vm_lds<6>();
                } else {
                    wait_vm_lds<0>();
                }
                __syncthreads();
            } else if (count > 1) {
                if (row == 1 || more) wait_vm_lds<3>();
                else wait_vm_lds<0>();
                __syncthreads();
                if (more) issue_taps(c + 1, row - 1);
            }
#pragma unroll
            for (int tap = 3 * row; tap < 3 * row + 3; ++tap) {
                const int up = row * p.cv.w2 + tap - 3 * row;  // shift of the tap, counted from -halo
                const int r = wave * (BM / 4) + frow + (BTN ? up : 2 * halo - up);
                i32x8 af[MT], bf[NT];
#pragma unroll
                for (int i = 0; i < MT; ++i) af[i] = row_fragment(lds + 32 * 64 * i, r);  // (32 rows on: the same slots)
#pragma unroll
                for (int j = 0; j < NT; ++j) {
                    if constexpr (BTN) bf[j] = slab64_fragment<true>(taps + tap * TAP, 0, j, lane);
                    else bf[j] = row_fragment(taps + tap * TAP + 32 * 64 * j, frow);
                }
                mma64_tiles<false>(bf, af, acc);
            }
        }
    }
    tile_epilogue<BM, BN, 4, 1, EPI, false, LDS_BYTES>(p, acc, lds, split, row0, col0, wave, lane, [](const float *, int, StatsAcc &) {});
}

}  // namespace mp8
