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
// BM = 32: tiles of 32 rows for small outputs (any_in_32_rows); the order of the additions is the same.
//
// What bounds it: with one tile per CU the chain of a wave -- a stage's loads, their way through the registers into LDS,
// conversion, multiplication -- of which the loads overlap with the rest; with two tiles per CU every instruction of that chain, and the
// path from L2, of which a 64-column piece of a contraction-major row uses half of each 128-byte line.  Back to back, us, loads that the
// multiplications wait for (a branch for the incomplete stage made the compiler wait there) / loads whose addresses every stage works
// out / now: 256 x 1000 x 2048 forward 10.4 / 8.0 / 7.4 (tiles of 32 rows but for the first), backward data 6.5 / 5.3 / 5.2, one thread
// per output element 639; 1500 x 1000 x 1500 11.8 / 12.0 / 11.3, b contraction-major 12.7 / 13.2 / 12.5, both 14.7 / 14.8 / 14.1; 500 x 2000 x 3000
// 13.4 13.1 12.1, 15.7 13.8 13.4, 16.7 15.3 14.4.  (Where only some CUs have two tiles, see `paced`.)
// EPI_UPDATE: an unsplit weight gradient applies the master-weight update itself (columns a multiple of eight:
// neighbouring lanes share random blocks), with the code of the other kernels' epilogues: no launch and no pass
// over the gradient codes: 256 x 1000 x 2048 with momentum 13.7 -> 12.6 us; with the weights, the state
// and the random words fetched behind the first stage's loads instead of after the contraction 12.7 -> 10.1, now 9.5.
// Needs a contraction of at least 16, and 16 rows / columns of a contraction-major operand (an edge
// chunk is read as the last 16 bytes of its row and shifted into place).
template <int EPI, bool ATN, bool BTN, bool SLICES, int BM = 64>
__device__ __forceinline__ void gemm_any(const GemmArgs &p, const UpdateHook &upd) {
    constexpr int STATES = EPI >= EPI_UPDATE ? EPI - EPI_UPDATE : 0;
    static_assert(EPI == EPI_FULL || !SLICES, "only a plain call takes its slices in turn");
    static_assert(BTN || !ATN, "a alone contraction-major is not built");
    static_assert(BM == 64 || (BM == 32 && !ATN && EPI == EPI_FULL && !SLICES), "the 32-row tile takes a row-major a and the whole contraction");
    constexpr int T = 64, SLAB_A = BM * BK, WAVE_LDS = SLAB_A + T * BK;
    constexpr int MI = BM / 32;    // 32x32 accumulator tiles along the rows
    constexpr int RED_LD = T + 4;  // floats per row of a tile parked for the reduction
    constexpr int RED_BYTES = 4 * BM * RED_LD * 4;
    __shared__ __attribute__((aligned(1024))) uint8_t lds[RED_BYTES > 4 * WAVE_LDS ? RED_BYTES : 4 * WAVE_LDS];

    int split, tm, tn;
    map_block(p, split, tm, tn);
    split = __builtin_amdgcn_readfirstlane(split);
    tm = __builtin_amdgcn_readfirstlane(tm);
    tn = __builtin_amdgcn_readfirstlane(tn);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t row0 = (int64_t)tm * BM, col0 = (int64_t)tn * T;
    // One operand: its tile's first row `first` of `limit`, leading dimension ld.
    //   row-major: load q brings tile rows 8q .. 8q+7, lane l sixteen contraction bytes of row
    //   8q + l/8, chunk l%8; rows beyond the matrix are clamped to its last row (never stored)
    //   contraction-major: load q brings contraction rows 16q .. 16q+15 of 64 bytes, lane l chunk l%4
    //   of row 16q + l/4 (one lane offset, off[0], serves all loads: the rest of their addresses, at[q], is uniform); a
    //   chunk that would leave the row is read as its last sixteen bytes and shifted down by `shift` bytes
    struct Operand {
        const uint8_t *base;
        int64_t ld, kstep;
        uint32_t off[8], at[8];
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
            o.base = uniform_ptr(x + first - 16 * ld);
            const int64_t m = 16 * (lane & 3), last = limit - 16 - first;
            o.shift = m > last ? (int)(m - last < 15 ? m - last : 15) : 0;
            // (last is negative in a tile narrower than sixteen columns: the sum is not)
            o.off[0] = (uint32_t)((lane >> 2) * ld + (m > last ? last : m) + 16);
#pragma unroll
            for (int q = 0; q < 8; ++q) o.at[q] = (uint32_t)((16 * q + 16) * ld);
        } else {
            o.base = uniform_ptr(x + first * ld);
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                int64_t r = 8 * q + (lane >> 3);
                r = first + r < limit ? r : limit - 1 - first;
                o.off[q] = (uint32_t)(r * ld) + 16 * (lane & 7) + 16;
            }
        }
        o.base -= 16;  // (16 bytes, and 16 contraction rows above: what is subtracted leaves off and at, which are unsigned, non-negative)
        return o;
    };
    Operand oa = operand(ATN, p.a, p.lda, row0, p.rows), ob = operand(BTN, p.b, p.ldb, col0, p.cols);

    // (address space 1: the base pointers have been through integers, and the compiler has to know
    // that they point to global memory)
    using Unaligned16 = u32x4 __attribute__((aligned(1)));
    auto load16 = [](const uint8_t *base, uint32_t off) {
        const auto *g = (const __attribute__((address_space(1))) uint8_t *)base;
        return (u32x4) * (const __attribute__((address_space(1))) Unaligned16 *)(g + off);
    };
    // x shifted down by 0 .. 15 bytes, zeros above
    auto shift_down = [](u32x4 x, int bytes) {
        const uint32_t whole = (bytes & 8) ? ~0u : 0u;  // (masks: with `?:` the compiler branches around every shift)
        const uint32_t w0 = (x.z & whole) | (x.x & ~whole), w1 = (x.w & whole) | (x.y & ~whole);
        uint64_t lo = ((uint64_t)w1 << 32) | w0, hi = ((uint64_t)(x.w & ~whole) << 32) | (x.z & ~whole);
        const int s = 8 * (bytes & 7);
        lo = (lo >> s) | ((hi << 1) << (63 - s));
        hi >>= s;
        return u32x4{(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
    };
    // A stage into registers: the same loads whether it is complete or not, so that nothing but the next round waits for them
    // (with a branch around them the compiler joined the two ways behind a wait for all loads).  The incomplete stage, the last one of
    // all, only changes where they read, in a branch of its own: complete ones go without an instruction for it.  Its partial chunk is read as the last
    // sixteen bytes of the row and its partial sixteen contraction rows as the last sixteen of all, what lies beyond it as something that
    // exists: store_stage puts them in place, and zeros behind them.
    auto left_of = [&](int s) { return p.tail != 0 && s == p.ksteps - 1 ? p.tail : BK; };
    auto load_stage = [&](bool km, Operand &o, int s, auto &x) {
        constexpr int N = sizeof(x) / sizeof(x[0]);  // loads: eight rows or sixteen contraction rows each
        const int left = left_of(s);
        if (left < BK) {
            if (km) {
#pragma unroll
                for (int q = 0; q < N; ++q)
                    if (16 * q + 16 > left) o.at[q] = (uint32_t)(left * o.ld);
            } else {
                const int chunk = 16 * (lane & 7), n = left - chunk, short0 = left < 16 ? 16 - left : 0;
                const uint32_t back = n <= 0 ? chunk + short0 : n < 16 ? 16 - n : 0;
#pragma unroll
                for (int q = 0; q < N; ++q) o.off[q] -= back;
            }
        }
        const uint8_t *k0 = o.base + (int64_t)s * o.kstep;
#pragma unroll
        for (int q = 0; q < N; ++q) {
            const uint8_t *from = km ? k0 + o.at[q] : k0;
            if (km) asm("" : "+s"(from));  // (a scalar base: left alone, the compiler adds in vector registers)
            x[q] = load16(from, o.off[km ? 0 : q]);
        }
    };
    auto store_stage = [&](bool km, const Operand &o, int s, auto &x, uint8_t *slab) {
        constexpr int N = sizeof(x) / sizeof(x[0]);
        const int left = left_of(s);
        auto put = [&](int row, u32x4 v) {
            const int at = km ? row * 64 + (((lane & 3) ^ (((row >> 2) & 1) << 1)) << 4)
                              : row * BK + (((lane & 7) ^ ((row >> 1) & 7)) << 4);
            *reinterpret_cast<u32x4 *>(slab + at) = v;
        };
        auto row = [&](int q) { return km ? 16 * q + (lane >> 2) : 8 * q + (lane >> 3); };
        if (km && o.edge) {
#pragma unroll
            for (int q = 0; q < N; ++q) x[q] = shift_down(x[q], o.shift);
        }
        if (left < BK && km) {  // (LDS operations of a wave are done in order)
#pragma unroll
            for (int q = 0; q < N; ++q) put(row(q), 16 * q + 16 <= left ? x[q] : u32x4{});
            const int r = left - 16 + (lane >> 2);
            put(r & (BK - 1), r >= 0 ? x[N - 1] : u32x4{});
            asm volatile("");  // (or the compiler joins the stores of both ways)
            return;
        }
        if (left < BK) {
            const int n = left - 16 * (lane & 7), shift = n >= 16 ? 0 : n > 0 ? 16 - n : 15;
            const uint32_t mask = n > 0 ? ~0u : 0u;
#pragma unroll
            for (int q = 0; q < N; ++q) {
                x[q] = shift_down(x[q], shift);
                x[q].x &= mask; x[q].y &= mask; x[q].z &= mask; x[q].w &= mask;
            }
        }
#pragma unroll
        for (int q = 0; q < N; ++q) put(row(q), x[q]);
    };

    // Some CUs have two workgroups and the others one: over a long contraction those run away from these, which then find nothing in the
    // L2 any more of what all of them read.  Loads that are waited for, one operand at a time, keep both operands' readers together.  Both
    // contraction-major, us, running free / so: 1100 x 1000 x 3000 23.2 / 21.9, x 9001 63 / 54, 1088 x 1024 x 17364 (aligned rows) 104 / 80,
    // 1300 x 1000 x 4099 32 / 30, 1500 x 1000 x 9001 59 / 55; 129 x 7001 x 3000 24.5 / 25.3, x 9001 63 / 64.  Shorter ones are better off without
    // (777 x 1333 x 2003 19.8 / 20.8), and so are those of more than two rounds (1500 x 1500 x 3000 33 / 37).  With a row-major a from
    // some 7000 on: 1100 x 1000 x 4099 31 / 31, x 7008 41 / 37, x 8752 52 / 45, x 16016 92 / 76, 1500 x 1000 x 10000 56 / 51, x 10001 67 / 66;
    // 777 x 1333 x 6001 44 / 45, 2000 x 1000 x 13001 86 / 90.  Both row-major: never (1100 x 1000 x 8752 44 / 44).
    const bool paced = BTN && gridDim.x > 256 && gridDim.x <= 512 && p.ks_per >= (ATN ? 24 : 56);
    auto pace = [&](bool on) {
        if (paced && on) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
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

    uint8_t *slab_a = lds + wave * WAVE_LDS, *slab_b = slab_a + SLAB_A;
    float *red = reinterpret_cast<float *>(lds);
    float v[16];
    for (int slice = SLICES ? 0 : split; slice < (SLICES ? p.splits : split + 1); ++slice) {
        const int ks_begin = slice * p.ks_per + (slice < p.ks_extra ? slice : p.ks_extra);
        const int ks_end = ks_begin + p.ks_per + (slice < p.ks_extra ? 1 : 0);
        f32x16 acc[MI][2];
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
        u32x4 xa[BM / 8], xb[8];
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
                store_stage(ATN, oa, s - 4, xa, slab_a);
                store_stage(BTN, ob, s - 4, xb, slab_b);
            }
            if (s < ks_end) {
                load_stage(ATN, oa, s, xa);
                pace(s > first);
                load_stage(BTN, ob, s, xb);
                pace(s > first);
            }
            if (s == first) continue;
            // the slabs are private to this wave: order its LDS writes before its reads
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            // A wave that multiplies goes ahead of one that fetches: two workgroups of a CU otherwise fetch and multiply in step
            // (1500 x 1000, contraction 1500 11.8 -> 11.2 us, 700 8.6 -> 8.1, 100 5.1 -> 5.0; one workgroup per CU as before).
            __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int sub = 0; sub < 2; ++sub) {
                i32x8 af[MI], bf[2];
#pragma unroll
                for (int i = 0; i < MI; ++i) af[i] = slab64_fragment<ATN>(slab_a, sub, i, lane);
#pragma unroll
                for (int j = 0; j < 2; ++j) bf[j] = slab64_fragment<BTN>(slab_b, sub, j, lane);
                // b as the "row" matrix: a lane gets consecutive output columns
                mma64_tiles<true>(bf, af, acc);
            }
            __builtin_amdgcn_s_setprio(0);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }

        // The four tiles meet in LDS: acc[i][j][4g + e] is row 32i + lane%32, column
        // 32j + 8g + 4*(lane/32) + e of this wave's tile; each thread then sums sixteen columns of a row.
        const int frow = lane & 31, fkb = lane >> 5;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    f32x4 o = {acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
                    *reinterpret_cast<f32x4 *>(red + (wave * BM + 32 * i + frow) * RED_LD + 32 * j + 8 * g + 4 * fkb) = o;
                }
        __syncthreads();
        auto summed = [&](int row, int col) {  // four columns, in wave order
            const float *at = red + row * RED_LD + col;
            f32x4 sum = *reinterpret_cast<const f32x4 *>(at);
#pragma unroll
            for (int w = 1; w < 4; ++w) {
                const f32x4 x = *reinterpret_cast<const f32x4 *>(at + w * BM * RED_LD);
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
        if (BM < 64 && (int)threadIdx.x >= BM * T / 16) break;  // (whole waves; nothing but the statistics is left for them)
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
    if (r < p.rows && c < p.cols && (int)threadIdx.x < BM * T / 16) {
        if ((p.cols & 15) == 0) finish16(p.ep, r, c, v, st);
        else finish16_ragged(p.ep, r, c, p.cols - c < 16 ? (int)(p.cols - c) : 16, v, st);
    }
    if constexpr (EPI == EPI_FULL) {
        if (p.ep.stats != nullptr) st.flush(p.ep.stats);
    }
}

template <int EPI, bool ATN, bool BTN, bool SLICES = false, int BM = 64>
__global__ __launch_bounds__(256, SLICES ? 1 : 2) void gemm_any_kernel(const GemmArgs p) {
    gemm_any<EPI, ATN, BTN, SLICES, BM>(p, UpdateHook{});
}
template <int STATES>
__global__ __launch_bounds__(256, 2) void gemm_any_update_kernel(const GemmArgs p, const UpdateHook upd) {
    gemm_any<EPI_UPDATE + STATES, true, true, false>(p, upd);
}

}  // namespace mp8
