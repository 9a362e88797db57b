// GEMM kernel on the matrix cores for shapes that the direct-to-LDS kernels cannot take: row
// lengths, leading dimensions or base addresses that are not multiples of 16, row-major operands with a
// contraction that is not, and split contractions that are not multiples of 128.
#pragma once

#include "gemm_common.hpp"
#include "gemm_finish.hpp"

namespace mp8 {

// Direct-to-LDS loads want 16-byte aligned rows and whole chunks, which a matrix with, say, 1000
// columns does not have.  This kernel fetches its operands through registers instead: sixteen
// bytes per lane from any address (the hardware takes unaligned vector loads), zeros in place of
// what lies beyond the contraction, then a 16-byte write into the same swizzled slab images as the
// other kernels.  64x64 tile, and as in gemm_wavek_kernel the contraction is divided among the four
// waves: every wave multiplies the whole tile for every fourth stage, from a slab pair of its
// own, so that nothing in the loop waits for another wave.  The loads of a wave's next stage are
// issued as soon as its current one has left the registers (64 of them), before the multiplications.
// Two workgroups fit a CU (70 KB of LDS).  The epilogue takes any row length, so an unsplit call
// needs no second pass and no workspace.  Half-precision products (mma64).
//
// A split contraction gives the same bits however it runs: the slices depend on the shape alone.  With a
// workspace they run side by side (EPI_PARTIAL and a finishing pass), without one a workgroup takes
// the slices of its tile one after the other (SLICES) and adds them up in the same order.
//
// What bounds it: a 64x64 tile pulls 128 bytes per clock and CU at the 8-bit matrix rate and 64 at the
// half-precision one, which is what the path from L2 carries; unaligned rows cost more requests.  A CU needs about
// 0.4 us per 16 KB stage however many tiles or waves there are (eight waves per tile: 256 x 1001, contraction 2003,
// row-major 12.1 us instead of 11.1, both contraction-major 10.5 instead of 10.7; two 8-byte loads for one of 16
// 10.7 instead of 10.2 at 256 x 1000, contraction 2048).  A layer of
// 256 x 1000 x 2048, back to back: forward 10.2 us, backward data 7.1, weight gradient 7.2 (one thread per output
// element 639 each).
// EPI_UPDATE: an unsplit weight gradient applies the master-weight update itself (columns a multiple of eight:
// neighbouring lanes share random blocks), with the code of the other kernels' epilogues: no launch and no pass
// over the gradient codes.  256 x 1000 x 2048 with momentum 13.7 -> 12.6 us, its training step 40.0 -> 37.2; with the weights, the state
// and the random words fetched behind the first stage's loads instead of after the contraction 12.7 -> 10.1, 37.0 -> 34.4.
// Needs a contraction of at least 16, and 16 rows / columns of a contraction-major operand (an edge
// chunk is read as the last 16 bytes of its row and shifted into place).
template <int EPI, bool ATN, bool BTN, bool SLICES>
__device__ __forceinline__ void gemm_any(const GemmArgs &p, const UpdateHook &upd) {
    constexpr int STATES = EPI >= EPI_UPDATE ? EPI - EPI_UPDATE : 0;
    static_assert(EPI == EPI_FULL || !SLICES, "only a plain call takes its slices in turn");
    static_assert(BTN || !ATN, "a alone contraction-major is not built");
    constexpr int T = 64, SLAB = T * BK, WAVE_LDS = 2 * SLAB;
    constexpr int RED_LD = T + 4;  // floats per row of a tile parked for the reduction
    constexpr int RED_BYTES = 4 * T * RED_LD * 4;
    __shared__ __attribute__((aligned(1024))) uint8_t lds[RED_BYTES > 4 * WAVE_LDS ? RED_BYTES : 4 * WAVE_LDS];

    int split, tm, tn;
    map_block(p, split, tm, tn);
    split = __builtin_amdgcn_readfirstlane(split);
    tm = __builtin_amdgcn_readfirstlane(tm);
    tn = __builtin_amdgcn_readfirstlane(tn);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t row0 = (int64_t)tm * T, col0 = (int64_t)tn * T;
    // One operand: its tile's first row `first` of `limit`, leading dimension ld.
    //   row-major: load q brings tile rows 8q .. 8q+7, lane l sixteen contraction bytes of row
    //   8q + l/8, chunk l%8; rows beyond the matrix are clamped to its last row (never stored)
    //   contraction-major: load q brings contraction rows 16q .. 16q+15 of 64 bytes, lane l chunk l%4
    //   of row 16q + l/4 (one lane offset serves all loads: the rest of their addresses is uniform); a chunk
    //   that would leave the row is read as its last sixteen bytes and shifted down by `shift` bytes
    struct Operand {
        const uint8_t *base;
        int64_t ld, kstep;
        uint32_t off[8];
        int shift;
        bool edge;
    };
    auto operand = [&](bool km, const uint8_t *x, int64_t ld, int64_t first, int64_t limit) {
        Operand o;
        o.ld = ld;
        o.kstep = km ? BK * ld : BK;
        o.shift = 0;
        o.edge = km && first + T > limit;
        if (km) {
            o.base = uniform_ptr(x + first);
            const int64_t m = 16 * (lane & 3), last = limit - 16 - first;
            o.shift = m > last ? (int)(m - last < 15 ? m - last : 15) : 0;
            // (last is negative in a tile narrower than sixteen columns: the sum is not)
            o.off[0] = (uint32_t)((lane >> 2) * ld + (m > last ? last : m) + 16);
        } else {
            o.base = uniform_ptr(x + first * ld);
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                int64_t r = 8 * q + (lane >> 3);
                r = first + r < limit ? r : limit - 1 - first;
                o.off[q] = (uint32_t)(r * ld) + 16 * (lane & 7) + 16;
            }
        }
        o.base -= 16;  // (what is subtracted from a lane offset leaves it non-negative: they are unsigned)
        return o;
    };
    const Operand oa = operand(ATN, p.a, p.lda, row0, p.rows), ob = operand(BTN, p.b, p.ldb, col0, p.cols);

    // (address space 1: the base pointers have been through integers, and the compiler has to know
    // that they point to global memory)
    using Unaligned16 = u32x4 __attribute__((aligned(1)));
    auto load16 = [](const uint8_t *base, uint32_t off) {
        const auto *g = (const __attribute__((address_space(1))) uint8_t *)base;
        return (u32x4) * (const __attribute__((address_space(1))) Unaligned16 *)(g + off);
    };
    // x shifted down by 0 .. 15 bytes, zeros above
    auto shift_down = [](u32x4 x, int bytes) {
        uint64_t lo = ((uint64_t)x.y << 32) | x.x, hi = ((uint64_t)x.w << 32) | x.z;
        if (bytes & 8) {
            lo = hi;
            hi = 0;
        }
        const int s = 8 * (bytes & 7);
        lo = (lo >> s) | ((hi << 1) << (63 - s));
        hi >>= s;
        return u32x4{(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
    };
    auto load_stage = [&](bool km, const Operand &o, int s, u32x4 x[8]) {
        const uint8_t *k0 = o.base + (int64_t)s * o.kstep;
        const int64_t left64 = p.kc - (int64_t)s * BK;
        auto load = [&](int q) { return km ? load16(k0 + 16 * q * o.ld, o.off[0]) : load16(k0, o.off[q]); };
        if (left64 >= BK) {
#pragma unroll
            for (int q = 0; q < 8; ++q) x[q] = load(q);
        } else if (km) {  // the last, incomplete stage: contraction rows beyond it are zero
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                x[q] = u32x4{0, 0, 0, 0};
                if (16 * q + (lane >> 2) < (int)left64) x[q] = load(q);
            }
        } else {  // bytes beyond it are zero; a partial chunk is the row's last sixteen bytes, shifted down
            const int n = (int)left64 - 16 * (lane & 7), back = n < 16 ? 16 - n : 0;
#pragma unroll
            for (int q = 0; q < 8; ++q) x[q] = u32x4{0, 0, 0, 0};
            if (n > 0) {
#pragma unroll
                for (int q = 0; q < 8; ++q) x[q] = shift_down(load16(k0, o.off[q] - back), back);
            }
        }
    };
    auto store_stage = [&](bool km, const Operand &o, u32x4 x[8], uint8_t *slab) {
        if (km && o.edge) {
#pragma unroll
            for (int q = 0; q < 8; ++q) x[q] = shift_down(x[q], o.shift);
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int row = km ? 16 * q + (lane >> 2) : 8 * q + (lane >> 3);
            const int at = km ? row * 64 + (((lane & 3) ^ (((row >> 2) & 1) << 1)) << 4)
                              : row * BK + (((lane & 7) ^ ((row >> 1) & 7)) << 4);
            *reinterpret_cast<u32x4 *>(slab + at) = x[q];
        }
    };

    // what this thread updates: four groups of four weights, 16 lanes side by side in a row of the tile
    auto group = [&](int q) {
        const int item = threadIdx.x + 256 * q;
        const int64_t r = row0 + (item >> 4), c = col0 + 4 * (item & 15);
        return GroupAt{r, c, r < p.rows && c < p.cols};
    };
    UpdateOperands4 uo[4];
    GroupWords<4> words;
    uint32_t flag = 0;

    uint8_t *slab_a = lds + wave * WAVE_LDS, *slab_b = slab_a + SLAB;
    float *red = reinterpret_cast<float *>(lds);
    float v[16];
    for (int slice = SLICES ? 0 : split; slice < (SLICES ? p.splits : split + 1); ++slice) {
        const int ks_begin = slice * p.ks_per + (slice < p.ks_extra ? slice : p.ks_extra);
        const int ks_end = ks_begin + p.ks_per + (slice < p.ks_extra ? 1 : 0);
        f32x16 acc[2][2];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
        u32x4 xa[8], xb[8];
        // stage s is fetched into registers in the round before the one that multiplies it (the rounds
        // are written so that the code of each step exists once: the incomplete stage makes it long)
        const int first = ks_begin + wave;
        if constexpr (EPI >= EPI_UPDATE) {  // the weights, the state and the random words behind the first stage's loads
            if (first < ks_end) {
                load_stage(ATN, oa, first, xa);
                load_stage(BTN, ob, first, xb);
            }
            load_groups<STATES, 4>(p.ep, upd, group, uo, flag);
            draw_groups<4>(p.ep, upd, group, words);
        }
        for (int s = EPI >= EPI_UPDATE ? first + 4 : first; s < ks_end + 4; s += 4) {
            if (s > first) {
                store_stage(ATN, oa, xa, slab_a);
                store_stage(BTN, ob, xb, slab_b);
            }
            if (s < ks_end) {
                load_stage(ATN, oa, s, xa);
                load_stage(BTN, ob, s, xb);
            }
            if (s == first) continue;
            // the slabs are private to this wave: order its LDS writes before its reads
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int sub = 0; sub < 2; ++sub) {
                i32x8 af[2], bf[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) af[i] = slab64_fragment<ATN>(slab_a, sub, i, lane);
#pragma unroll
                for (int j = 0; j < 2; ++j) bf[j] = slab64_fragment<BTN>(slab_b, sub, j, lane);
                // b as the "row" matrix: a lane gets consecutive output columns
                mma64_tiles<true>(bf, af, acc);
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }

        // The four tiles meet in LDS: acc[i][j][4g + e] is row 32i + lane%32, column
        // 32j + 8g + 4*(lane/32) + e of this wave's tile; each thread then sums sixteen columns of a row.
        const int frow = lane & 31, fkb = lane >> 5;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    f32x4 o = {acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
                    *reinterpret_cast<f32x4 *>(red + (wave * T + 32 * i + frow) * RED_LD + 32 * j + 8 * g + 4 * fkb) = o;
                }
        __syncthreads();
        auto summed = [&](int row, int col) {  // four columns, in wave order
            const float *at = red + row * RED_LD + col;
            f32x4 sum = *reinterpret_cast<const f32x4 *>(at);
#pragma unroll
            for (int w = 1; w < 4; ++w) {
                const f32x4 x = *reinterpret_cast<const f32x4 *>(at + w * T * RED_LD);
                sum.x += x.x; sum.y += x.y; sum.z += x.z; sum.w += x.w;
            }
            return sum;
        };
        if constexpr (EPI >= EPI_UPDATE) {
            StatsAcc st;
            auto sum = [&](int q, float out[4]) {
                const int item = threadIdx.x + 256 * q;
                const f32x4 t = summed(item >> 4, 4 * (item & 15));
                out[0] = t.x; out[1] = t.y; out[2] = t.z; out[3] = t.w;
            };
            update_groups<STATES, 4>(p.ep, upd, flag, group, sum, st, uo, words);
            if (p.ep.stats != nullptr) st.flush(p.ep.stats);
            return;
        } else if constexpr (EPI == EPI_PARTIAL) {
#pragma unroll
            for (int k = 0; k < T * T / 1024; ++k) {
                const int item = threadIdx.x + 256 * k, rr = item >> 4, c4 = 4 * (item & 15);
                emit_partial4(p, split, row0 + rr, col0 + c4, summed(rr, c4));
            }
            return;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const f32x4 sum = summed(threadIdx.x >> 2, 16 * (threadIdx.x & 3) + 4 * q);
            if (SLICES && slice > 0) {
                v[4 * q] += sum.x; v[4 * q + 1] += sum.y; v[4 * q + 2] += sum.z; v[4 * q + 3] += sum.w;
            } else {
                v[4 * q] = sum.x; v[4 * q + 1] = sum.y; v[4 * q + 2] = sum.z; v[4 * q + 3] = sum.w;
            }
        }
        if constexpr (SLICES) __syncthreads();  // the slabs of the next slice overwrite the tiles
    }

    StatsAcc st;
    const int64_t r = row0 + (threadIdx.x >> 2), c = col0 + 16 * (threadIdx.x & 3);
    if (r < p.rows && c < p.cols) {
        if ((p.cols & 15) == 0) finish16(p.ep, r, c, v, st);
        else finish16_ragged(p.ep, r, c, p.cols - c < 16 ? (int)(p.cols - c) : 16, v, st);
    }
    if constexpr (EPI == EPI_FULL) {
        if (p.ep.stats != nullptr) st.flush(p.ep.stats);
    }
}

template <int EPI, bool ATN, bool BTN, bool SLICES = false>
__global__ __launch_bounds__(256, SLICES ? 1 : 2) void gemm_any_kernel(const GemmArgs p) {
    gemm_any<EPI, ATN, BTN, SLICES>(p, UpdateHook{});
}
template <int STATES>
__global__ __launch_bounds__(256, 2) void gemm_any_update_kernel(const GemmArgs p, const UpdateHook upd) {
    gemm_any<EPI_UPDATE + STATES, true, true, false>(p, upd);
}

}  // namespace mp8
