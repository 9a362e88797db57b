// GEMM kernel for outputs of several 256x256 tiles per CU: one resident workgroup per CU, whose operand stream does not
// stop between tiles.
#pragma once

#include "gemm_common.hpp"

namespace mp8 {

// The general kernel (gemm_mfma.hpp) with a 256x256 tile has the CU to itself, and nothing overlaps with its start, its conversions
// and its stores: beside 1.4 us for each 128-byte stage it spends some 6 us per tile, all CUs in step (from the times below).  Here a
// workgroup takes tiles blockIdx.x, blockIdx.x + gridDim.x, ... (as the hardware would have dealt them out), and the ring of two
// stages goes on from one tile to the next: while the last stages of a tile are multiplied, the first two of the next one arrive.  The codes
// leave through 4 KB of LDS per wave beside the ring, 32 rows of 128 bytes at a time, without a barrier, and the
// stores drain while the next tile is multiplied.  As soon as an accumulator has been converted, the next tile's first
// half stage is multiplied into it, so the matrix cores work on during the conversions.  Codes to nearest only.
// us, one tile per workgroup / this: 16384 x 4096 x 1024 68.1 / 59.0 (floor of the products at the rate of 8192^3: 47), 8192 x 8192 x 8192 383 / 372
// (bound by power either way), 12288 x 4096 x 1024 52.5 / 44.4; against 128x128 tiles see stream_pays.
//
// Pipeline of a stage, slabs, fragments and their order: as in the general kernel, so are the bits.
// UNIT: alpha is 1.
template <bool ATN, bool BTN, bool UNIT>
__global__ __launch_bounds__(256, 1) void gemm_stream_kernel(const GemmArgs p) {
    static_assert(BTN || !ATN, "a alone contraction-major is not built");
    constexpr int T = 256, MT = 4, NT = 4, F = MT + NT, NM = MT * NT;
    constexpr int SLAB = T * BK, STAGE = 2 * SLAB;
    constexpr int DMA = T / 32, G = 2 * DMA;        // direct loads per wave and stage: one operand, both
    constexpr int STORES = 16;                      // per wave and tile
    constexpr int S_BAR = NM / 2, S_RD = S_BAR - 2; // see the general kernel
    constexpr int R0 = (2 * F + S_RD - 1) / S_RD;
    __shared__ __attribute__((aligned(1024))) uint8_t lds[2 * STAGE + 4 * 32 * 128];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int ksteps = p.ksteps;
    const uint32_t ntiles = (uint32_t)(p.tiles_m * p.tiles_n);
    const int64_t a_kstep = ATN ? (int64_t)BK * p.lda : BK, b_kstep = BTN ? (int64_t)BK * p.ldb : BK;

    // Operand fetch of one tile: uniform bases and the lanes' offsets (clamped at the edges of the matrix).
    const uint8_t *a_tile, *b_tile;
    uint32_t oa[DMA], ob[DMA];
    auto offsets = [&](bool km, int64_t first, int64_t limit, int64_t ld, uint32_t (&off)[DMA]) {
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));  // (worked out anew for each tile: kept for all of them, these values do not fit the registers)
#pragma unroll
        for (int q = 0; q < DMA; ++q) {
            if (km) {
                const int chunk = (lane & 7) ^ (((lane >> 4) & 3) << 1);
                int64_t m = 128 * (q >> 2) + 16 * chunk;
                m = first + m + 16 <= limit ? m : limit - 16 - first;
                off[q] = (uint32_t)((8 * (wave + 4 * (q & 3)) + (lane >> 3)) * ld + m);
            } else {
                int64_t r = 8 * (wave + 4 * q) + (lane >> 3);
                r = first + r < limit ? r : limit - 1 - first;
                off[q] = (uint32_t)(r * ld) + 16 * ((lane & 7) ^ ((4 * wave + (lane >> 4)) & 7));
            }
        }
    };
    auto fetch_from = [&](uint32_t tile, int64_t &row0, int64_t &col0) {
        int split, tm, tn;
        map_tile(p, ntiles, tile, split, tm, tn);
        row0 = (int64_t)__builtin_amdgcn_readfirstlane(tm) * T;
        col0 = (int64_t)__builtin_amdgcn_readfirstlane(tn) * T;
        a_tile = uniform_ptr(ATN ? p.a + row0 : p.a + row0 * p.lda);
        b_tile = uniform_ptr(BTN ? p.b + col0 : p.b + col0 * p.ldb);
        offsets(ATN, row0, p.rows, p.lda, oa);
        offsets(BTN, col0, p.cols, p.ldb, ob);
    };
    const uint32_t lds0 = lds_address(lds) + wave * 1024;
    auto issue_one = [&](int slot, const uint8_t *ak, const uint8_t *bk, int q) {
        const uint32_t to = lds0 + slot * STAGE;
        if (q < DMA) dma16(ak, oa[q < DMA ? q : 0], to + q * 4096);
        else dma16(bk, ob[q >= DMA ? q - DMA : 0], to + SLAB + (q - DMA) * 4096);
    };

    const int frow = lane & 31, fkb = lane >> 5, fsw = (frow >> 1) & 7;
    struct Frags {
        i32x4 h[F][2];
    };
    auto read_half = [&](int slot, int sub, int f, int half, Frags &fr) {
        const uint8_t *s = lds + slot * STAGE;
        const bool is_a = f < MT;
        const int first = is_a ? wm * 128 + f * 32 : wn * 128 + (f - MT) * 32;
        if (is_a ? ATN : BTN) {
            const int t = lane & 15, m = first + (frow & 16);
            i32x2 part[2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int k = 64 * sub + 32 * fkb + 8 * (2 * half + e) + (t >> 1);
                const int off = (is_a ? 0 : SLAB) + (m >> 7) * 16384 + k * 128 + ((((m & 127) >> 4) ^ (((k >> 1) & 3) << 1)) << 4) + 8 * (t & 1);
                part[e] = __builtin_amdgcn_ds_read_tr8_b64_v2i32((__attribute__((address_space(3))) i32x2 *)(s + off));
            }
            fr.h[f][half] = i32x4{part[0].x, part[0].y, part[1].x, part[1].y};
        } else {
            fr.h[f][half] = *reinterpret_cast<const i32x4 *>(s + (is_a ? 0 : SLAB) + (first + frow) * BK + (((4 * sub + 2 * fkb + half) ^ fsw) << 4));
        }
    };
    auto frag_order = [&](int n) -> int { return n == 0 ? MT : n == 1 ? 0 : n < NT + 1 ? MT + n - 1 : n - NT; };

    const f32x16 none = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    f32x16 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = none;
    auto mfma = [&](const Frags &fr, int m) {
        const int i = m / NT, j = m % NT;
        acc[i][j] = mma64<false>(__builtin_shufflevector(fr.h[MT + j][0], fr.h[MT + j][1], 0, 1, 2, 3, 4, 5, 6, 7),
                                 __builtin_shufflevector(fr.h[i][0], fr.h[i][1], 0, 1, 2, 3, 4, 5, 6, 7), acc[i][j]);
    };

    uint32_t tile = blockIdx.x;
    int64_t row0, col0, next_row0 = 0, next_col0 = 0;
    fetch_from(tile, row0, col0);
    Frags f0, f1;
#pragma unroll
    for (int st = 0; st < 2; ++st)  // (at least two stages, see the host)
#pragma unroll
        for (int q = 0; q < G; ++q) issue_one(st, a_tile + st * a_kstep, b_tile + st * b_kstep, q);
    wait_vm_lds<G>();
    __syncthreads();
#pragma unroll
    for (int n = 0; n < 2 * F; ++n) read_half(0, 0, frag_order(n / 2), n & 1, f0);

    uint8_t *mine = lds + 2 * STAGE + wave * 4096;
    int slot = 0;              // ring slot of the stage that is multiplied
    bool drained = true;       // no store of the tile before lies behind the loads that are waited for
    bool started = false;      // the first sub-step of this tile was multiplied in the epilogue of the one before
    for (;;) {
        const bool another = tile + gridDim.x < ntiles;
        for (int t = 0; t < ksteps; ++t, slot ^= 1) {
            // what this stage loads: the next but one of this tile, or one of the first two of the next tile
            if (t + 2 == ksteps && another) fetch_from(tile + gridDim.x, next_row0, next_col0);
            const int lt = t + 2 < ksteps ? t + 2 : t + 2 - ksteps;
            const bool more = t + 2 < ksteps || another, next = t + 1 < ksteps || another;
            const uint8_t *ak = a_tile + lt * a_kstep, *bk = b_tile + lt * b_kstep;
#pragma unroll
            for (int k = 0; k < 2 * NM; ++k) {
                if (k >= NM) mfma(f1, k - NM);
                else if (t > 0 || !started) mfma(f0, k);
                if (k < S_RD) {
#pragma unroll
                    for (int r = 0; r < R0; ++r)
                        if (k * R0 + r < 2 * F) read_half(slot, 1, frag_order((k * R0 + r) / 2), (k * R0 + r) & 1, f1);
                }
                if (k == S_BAR - 1) {
                    // the next stage has landed (its loads are older than the stores of the tile before)
                    __builtin_amdgcn_sched_barrier(0);
                    if (t == 0 && !drained) wait_vm_lds<STORES>();
                    else wait_vm_lds<0>();
                    __syncthreads();
                }
                if (k >= S_BAR && k - S_BAR < G && more) issue_one(slot, ak, bk, k - S_BAR);
                if (k >= NM && next) read_half(slot ^ 1, 0, frag_order((k - NM) / 2), (k - NM) & 1, f0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }

        // Epilogue, 32 rows of the wave's 128 x 128 codes at a time: acc[i][j][4g + e] is row 32i + lane%32, column 32j + 8g +
        // 4*(lane/32) + e.  Sixteen-byte pieces into the wave's own LDS (piece q of row r in slot q ^ ((r >> 1) & 7)),
        // whole 128-byte lines out; LDS operations of a wave are done in order.
        int el = lane;
        asm volatile("" : "+v"(el));  // (as above)
        const int erow = el & 31, ekb = el >> 5, line = el >> 3, piece = el & 7;
        const int64_t r0 = row0 + wm * 128 + line, c = col0 + wn * 128 + 16 * piece;
        const bool inside = row0 + T <= p.rows && col0 + T <= p.cols;
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            float top = 0.0f;  // a NaN stays: the conversion gives it another code than the library's
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                asm volatile("" : "+a"(acc[i][j]));  // (stays in the accumulators until here: copied out ahead of time it would be spilled)
                uint32_t pk[4];
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    float y[4] = {acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if constexpr (!UNIT) y[e] *= p.ep.alpha;
                        top = __builtin_elementwise_maximum(top, __builtin_fabsf(y[e]));
                    }
                    pk[g] = e5m2_pack4_raw<false>(y, 0u, 0u, false);
                }
                __builtin_amdgcn_sched_barrier(0);
                // (behind the last tile this multiplies what nobody reads)
                acc[i][j] = mma64<false>(__builtin_shufflevector(f0.h[MT + j][0], f0.h[MT + j][1], 0, 1, 2, 3, 4, 5, 6, 7),
                                             __builtin_shufflevector(f0.h[i][0], f0.h[i][1], 0, 1, 2, 3, 4, 5, 6, 7), none);
                const auto s0 = __builtin_amdgcn_permlane32_swap(pk[0], pk[2], false, false);
                const auto s1 = __builtin_amdgcn_permlane32_swap(pk[1], pk[3], false, false);
                const u32x4 o = {s0[0], s0[1], s1[0], s1[1]};
                *reinterpret_cast<u32x4 *>(mine + erow * 128 + (((2 * j + ekb) ^ ((erow >> 1) & 7)) << 4)) = o;
                __builtin_amdgcn_sched_barrier(0);
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const bool any_nan = __builtin_amdgcn_ballot_w64(top != top) != 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int rr = 8 * k + line;
                u32x4 o = *reinterpret_cast<const u32x4 *>(mine + rr * 128 + ((piece ^ ((rr >> 1) & 7)) << 4));
                if (any_nan) o = u32x4{canonical_nan_codes(o.x), canonical_nan_codes(o.y), canonical_nan_codes(o.z), canonical_nan_codes(o.w)};
                const int64_t r = r0 + 32 * i + 8 * k;
                if (inside || (r < p.rows && c < p.cols)) store_through(reinterpret_cast<u32x4 *>(p.ep.out8 + r * p.cols + c), o);
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
        if (!another) break;
        drained = !inside;
        started = true;
        tile += gridDim.x;
        row0 = next_row0;
        col0 = next_col0;
    }
}

}  // namespace mp8
