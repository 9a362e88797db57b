// What the MFMA kernels do with a finished tile of 32x32 accumulators per wave: the epilogue variants (EPI_*).
#pragma once

#include "gemm_common.hpp"

namespace mp8 {

// A workgroup of 256 threads, WGM x WGN waves, with a tile of BM x BN outputs at (row0, col0); `lds` is
// free for reuse once every wave has arrived.  EPI_UPDATE: `update` finishes the one 32x32 tile of a wave that
// lies in a band of FP32 rows (its pitch, the statistics).  HALF: any row length.
template <int BM, int BN, int WGM, int WGN, int EPI, bool HALF, int LDS_BYTES, class Update>
__device__ __forceinline__ void tile_epilogue(const GemmArgs &p, const f32x16 (&acc)[BM / WGM / 32][BN / WGN / 32], uint8_t *lds,
                                              int split, int64_t row0, int64_t col0, int wave, int lane, Update update) {
    constexpr int WTM = BM / WGM, WTN = BN / WGN, MT = WTM / 32, NT = WTN / 32;
    const int wm = wave / WGN, wn = wave % WGN;
    const int frow = lane & 31, fkb = lane >> 5;
    // Epilogue.  acc[i][j][4g + e] is output row  wm*WTM + 32i + lane%32  and column
    // wn*WTN + 32j + 8g + 4*(lane/32) + e.  Each wave passes its tile through LDS one band
    // of 32 rows at a time, so that afterwards every lane owns 16 consecutive columns of one
    // row: full 16-byte stores of codes, one Philox block per eight elements.  FP32 leaves
    // before that, 16 bytes per lane, neighbouring lanes side by side (partial tiles, and acc where
    // acc_lines says so; else 64-byte runs per lane).
    constexpr int EP_LD = WTN + 4;                 // floats per band row (+4: bank spread)
    constexpr int CG = WTN / 16;                   // 16-column groups per band row
    constexpr int BANDS = MT >= 2 ? 2 : 1;         // bands staged per pass
    static_assert(EPI == EPI_RNE || 4 * BANDS * 32 * EP_LD * 4 <= LDS_BYTES, "band buffers fit in LDS");
    __syncthreads();                               // all waves are done with the operand ring
    if constexpr (EPI == EPI_RNE) {
        // RNE only: convert in registers (four codes = one register), join the two half-wave
        // column sets of every 32x32 tile with two v_permlane32_swap -- lane (row, h) then
        // holds the 16-byte piece of columns 32j + 16h .. +15 -- and collect the whole block
        // tile of codes (BM x BN bytes) in LDS, piece q of row r in slot q ^ f(r) with
        // f(r) = (r / rows per 256 bytes) mod pieces per row: conflict-free for the writes
        // (16 rows, one piece) and for the reads (consecutive pieces of a row).  Then the
        // block stores whole rows of the tile: BN / 16 consecutive lanes per row.
        constexpr int NP = BN / 16;                // pieces per tile row
        constexpr int RP = 256 / BN > 0 ? 256 / BN : 1;  // tile rows per 256 bytes of LDS
        static_assert(BM * BN <= LDS_BYTES, "code tile fits in LDS");
        auto slot = [&](int r, int q) { return r * BN + ((q ^ ((r / RP) & (NP - 1))) << 4); };
        auto tiles = [&](auto unit_alpha) {
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j) {
                    uint32_t pk[4];
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        float y[4] = {acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2],
                                      acc[i][j][4 * g + 3]};
                        if constexpr (!decltype(unit_alpha)::value) {
#pragma unroll
                            for (int e = 0; e < 4; ++e) y[e] *= p.ep.alpha;
                        }
                        pk[g] = e5m2_pack4<false>(y, 0u, 0u, false);
                    }
                    // after swap(pk[g], pk[g+2]): lower half = own columns 8g .. 8g+3 and the
                    // upper half's 8g+4 .. 8g+7; upper half = the lower half's 16+8g .. +3 and
                    // its own 16+8g+4 .. +7
                    const auto s0 = __builtin_amdgcn_permlane32_swap(pk[0], pk[2], false, false);
                    const auto s1 = __builtin_amdgcn_permlane32_swap(pk[1], pk[3], false, false);
                    u32x4 o = {s0[0], s0[1], s1[0], s1[1]};
                    *reinterpret_cast<u32x4 *>(lds + slot(wm * WTM + 32 * i + frow,
                                                          (wn * WTN + 32 * j) / 16 + fkb)) = o;
                }
        };
        if (p.ep.alpha == 1.0f) tiles(std::true_type{});
        else tiles(std::false_type{});
        __syncthreads();
        const int q = threadIdx.x % NP;
        const int64_t c = col0 + 16 * q;
#pragma unroll
        for (int k = 0; k < BM * NP / 256; ++k) {
            const int rr = k * (256 / NP) + threadIdx.x / NP;
            u32x4 o = *reinterpret_cast<const u32x4 *>(lds + slot(rr, q));
            const int64_t r = row0 + rr;
            if (r < p.rows && c < p.cols) {
                if (p.ep.mask && conv_padding_row(p.ep, r)) o = u32x4{0u, 0u, 0u, 0u};
                store_through(reinterpret_cast<u32x4 *>(p.ep.out8 + r * p.cols + c), o);
            }
        }
        return;
    }
    float *band = reinterpret_cast<float *>(lds) + wave * BANDS * 32 * EP_LD;
    StatsAcc st;
    const bool fast_cols = (p.cols & 15) == 0;
#pragma unroll
    for (int h = 0; h < MT; h += BANDS) {
#pragma unroll
        for (int bi = 0; bi < BANDS; ++bi)
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    f32x4 o = {acc[h + bi][j][4 * g], acc[h + bi][j][4 * g + 1],
                               acc[h + bi][j][4 * g + 2], acc[h + bi][j][4 * g + 3]};
                    *reinterpret_cast<f32x4 *>(band + (32 * bi + frow) * EP_LD + 32 * j + 8 * g +
                                               4 * fkb) = o;
                }
        // the bands are private to this wave: order the LDS writes before the reads
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if constexpr (EPI >= EPI_UPDATE) {
            update(band, EP_LD, st);
            break;
        }
        if constexpr (EPI == EPI_PARTIAL) {
            constexpr int F4 = WTN / 4;
            const int64_t c0 = col0 + wn * WTN, left = p.cols - c0;
            if (2 * left <= WTN) {  // lanes side by side in as many rows as fit, not most of them beyond the matrix (64 x 3 x 256 5.3 -> 4.85 us)
                const int lg = left <= 4 ? 0 : 32 - __builtin_clz((int)(left - 1) >> 2);
                const int c = 4 * (lane & ((1 << lg) - 1));
#pragma unroll 2
                for (int br = lane >> lg; br < BANDS * 32; br += 64 >> lg)
                    emit_partial4(p, split, row0 + wm * WTM + 32 * h + br, c0 + c, *reinterpret_cast<const f32x4 *>(band + br * EP_LD + c));
            } else
#pragma unroll 4
            for (int item = lane; item < BANDS * 32 * F4; item += 64) {
                const int br = item / F4, q = item - br * F4;
                emit_partial4(p, split, row0 + wm * WTM + 32 * h + br, col0 + wn * WTN + 4 * q,
                              *reinterpret_cast<const f32x4 *>(band + br * EP_LD + 4 * q));
            }
        } else {
            // The FP32 result leaves as the partial tiles do, neighbouring lanes side by side; the sums stay in the band.
            const bool acc_done = EPI == EPI_FULL && p.ep.acc_lines != 0;
            if (acc_done) {
                constexpr int F4 = WTN / 4;
                auto lines = [&](auto plain) {
#pragma unroll 4
                    for (int item = lane; item < BANDS * 32 * F4; item += 64) {
                        const int br = item / F4, q = item - br * F4;
                        const int64_t r = row0 + wm * WTM + 32 * h + br, c = col0 + wn * WTN + 4 * q;
                        if (r < p.rows && c < p.cols) {
                            f32x4 *at = reinterpret_cast<f32x4 *>(band + br * EP_LD + 4 * q);
                            f32x4 *to = reinterpret_cast<f32x4 *>(p.ep.acc + r * p.cols + c);
                            f32x4 x = *at;
                            if (decltype(plain)::value || p.ep.acc_mode == 2) {
                                const f32x4 o = *to;
                                x.x += o.x; x.y += o.y; x.z += o.z; x.w += o.w;
                                *at = x;
                            }
                            if constexpr (decltype(plain)::value) *to = x;
                            else store_through(to, x);
                        }
                    }
                };
                if (p.ep.acc_lines == 2) lines(std::true_type{});  // (added to)
                else lines(std::false_type{});
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            }
#pragma unroll 1
            for (int item = lane; item < BANDS * 32 * CG; item += 64) {
                const int br = item / CG, cg = item - br * CG;
                const int64_t r = row0 + wm * WTM + 32 * h + br;
                const int64_t c = col0 + wn * WTN + 16 * cg;
                if (r < p.rows && c < p.cols) {
                    float v[16];
                    const f32x4 *src = reinterpret_cast<const f32x4 *>(band + br * EP_LD + 16 * cg);
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        f32x4 x = src[q];
                        v[4 * q] = x.x; v[4 * q + 1] = x.y; v[4 * q + 2] = x.z; v[4 * q + 3] = x.w;
                    }
                    if (HALF && EPI == EPI_FULL && !fast_cols)
                        finish16_ragged(p.ep, r, c, p.cols - c < 16 ? (int)(p.cols - c) : 16, v, st);
                    else emit16<EPI, true>(p, r, c, v, st, acc_done);
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    if constexpr (EPI >= EPI_FULL) {
        if (p.ep.stats != nullptr) st.flush(p.ep.stats);
    }
}

}  // namespace mp8
