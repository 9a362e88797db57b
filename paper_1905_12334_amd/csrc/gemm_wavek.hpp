// GEMM kernel for small outputs with long contractions: the contraction is divided among the
// waves of a workgroup.
#pragma once

#include "gemm_common.hpp"
#include "gemm_finish.hpp"

namespace mp8 {

// Small output, long contraction (weight gradients, skinny layers): the contraction is divided
// among the four WAVES of a workgroup as well.  In the general kernel a 64x64 tile gives each
// wave one 32x32 MFMA per half stage behind a workgroup barrier, and every stage costs a chain
// of latencies (load, barrier, LDS read, MFMA) with nothing to overlap them.  Here every wave
// computes the whole 64x64 tile (four MFMAs per half stage, each fragment used twice) for every
// fourth stage of the workgroup's slice, from a two-stage ring of its own (2 x 16 KB) that it
// fills with its own direct loads and waits for with its own counter: no barrier inside the
// loop, and eight stage loads in flight per CU.  At the end the four FP32 tiles meet in LDS and
// are added in wave order; each thread then owns sixteen consecutive columns of one row for
// the epilogue.  Operand layouts and slab images as in the general kernel (ATN / BTN:
// contraction-major).  CONV = 3: the weight gradient of the 3x3 convolution (tap shift per tile
// row), else 0.  BM = 32 / BN = 32 (row-major operand only): half the tile rows / columns, for
// outputs with so few 64x64 tiles that most CUs would idle while the busy ones wait for their
// own loads (a CU takes 64 bytes per clock however few of them work).
// With EPI_UPDATE the master weights and the optimizer's state that a thread will need at the end are
// fetched behind the loads of its first two stages: one workgroup per CU leaves each lane 512 registers.  (4096 x 2048 x 512
// with ADAM 16.9 us, ahead of them 17.6.)
// HALF: as in the general kernel.
template <int EPI, bool ATN, bool BTN, int CONV, int BM = 64, int BN = 64, bool HALF = false>
__device__ __forceinline__ void gemm_wavek(const GemmArgs &p, const UpdateHook &upd) {
    constexpr int STATES = EPI >= EPI_UPDATE ? EPI - EPI_UPDATE : 0;
    static_assert(CONV == 0 || (CONV == 3 && ATN && BTN && !HALF), "plain or convolution weight gradient");
    static_assert(BTN || !ATN, "a alone contraction-major is not built");
    static_assert(BM == 64 || (BM == 32 && !ATN), "the 32-row tile takes a row-major a");
    static_assert(BN == 64 || (BN == 32 && !BTN), "the 32-column tile takes a row-major b");
    constexpr int MI = BM / 32, NJ = BN / 32;  // 32x32 accumulator tiles along rows and columns
    constexpr int QA = BM / 8, QB = BN / 8;    // direct loads per stage and operand (eight rows each)
    constexpr int SLAB_A = BM * BK;         // BM rows of 128 bytes, or 128 contraction rows of 64
    constexpr int SLAB = BN * BK;           // b
    constexpr int STAGE = SLAB_A + SLAB;    // a, then b
    constexpr int WAVE_LDS = 2 * STAGE;     // ring of two stages per wave
    constexpr int RED_LD = BN + 4;          // floats per row of a tile parked for the reduction
    static_assert(4 * BM * RED_LD * 4 <= 4 * WAVE_LDS, "reduction buffers fit in the rings");
    __shared__ __attribute__((aligned(1024))) uint8_t lds[4 * WAVE_LDS];

    int split, tm, tn;
    map_block(p, split, tm, tn);
    split = __builtin_amdgcn_readfirstlane(split);
    tm = __builtin_amdgcn_readfirstlane(tm);
    tn = __builtin_amdgcn_readfirstlane(tn);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t row0 = (int64_t)tm * BM, col0 = (int64_t)tn * BN;
    // what this thread updates: four groups of four weights, 16 lanes side by side in a row of the tile
    auto group = [&](int q) {
        const int item = threadIdx.x + 256 * q;
        const int64_t r = row0 + (item >> 4), c = col0 + 4 * (item & 15);
        return GroupAt{r, c, r < p.rows && c < p.cols};
    };
    static_assert(EPI < EPI_UPDATE || (BM == 64 && BN == 64), "four groups per thread");
    UpdateOperands4 uo[4];
    uint32_t flag = 0;
    const int per = p.ks_per, extra = p.ks_extra;
    const int ks_begin = split * per + (split < extra ? split : extra);
    const int ks_count = per + (split < extra ? 1 : 0);
    // this wave's stages: ks_begin + wave, + 4, + 8, ...
    const int mine = __builtin_amdgcn_readfirstlane(ks_count > wave ? (ks_count - wave + 3) >> 2 : 0);

    const int64_t a_kstep = ATN ? (int64_t)BK * p.lda : BK, b_kstep = BTN ? (int64_t)BK * p.ldb : BK;
    const uint8_t *a_origin;
    if constexpr (CONV == 3) {
        uint32_t ci0;
        const uint32_t tap = fastdiv((uint32_t)row0, p.cv.div_ci, ci0);
        const int r = (int)((tap * 11u) >> 5);
        const int shift = (r - 1) * p.cv.w2 + ((int)tap - 3 * r - 1);
        a_origin = p.a + (int64_t)shift * p.lda + ci0;
    } else {
        a_origin = ATN ? p.a + row0 : p.a + row0 * p.lda;
    }
    const uint8_t *b_origin = BTN ? p.b + col0 : p.b + col0 * p.ldb;
    // an incomplete stage goes first (stage 0, wave 0 of the first slice): the others start one later
    const bool has_tail = HALF && p.tail != 0;
    const int64_t ks0 = ks_begin + wave - (has_tail ? 1 : 0);
    const uint8_t *a_tile = uniform_ptr(a_origin + ks0 * a_kstep);
    const uint8_t *b_tile = uniform_ptr(b_origin + ks0 * b_kstep);
    // Direct loads, eight per operand and stage.  Row-major operand: load q brings tile rows
    // 8q .. 8q+7, lane i lands at (row i/8, slot i%8) and fetches chunk (i%8) ^ ((row >> 1) & 7);
    // rows beyond the matrix are clamped to its last row.  Contraction-major operand: load q
    // brings contraction rows 16q .. 16q+15 of 64 bytes, lane i lands at (row i/4, slot i%4) and
    // fetches the chunk that belongs there under the swizzle of the narrow slabs; chunks that
    // would start beyond the matrix are clamped to its last 16 rows.  (Clamped data is never
    // stored.)
    auto lane_offsets = [&](bool km, int64_t first, int64_t limit, int64_t ld, uint32_t off[8]) {
        if (km) {
            const int chunk = (lane & 3) ^ (((lane >> 4) & 1) << 1);
            int64_t m = 16 * chunk;
            m = first + m + 16 <= limit ? m : limit - 16 - first;
#pragma unroll
            for (int q = 0; q < 8; ++q) off[q] = (uint32_t)((16 * q + (lane >> 2)) * ld + m);
        } else {
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                int64_t r = 8 * q + (lane >> 3);
                const int chunk = (lane & 7) ^ ((r >> 1) & 7);
                r = first + r < limit ? r : limit - 1 - first;
                off[q] = (uint32_t)(r * ld) + chunk * 16;
            }
        }
    };
    uint32_t oa[8], ob[8];
    lane_offsets(ATN, row0, p.rows, p.lda, oa);
    lane_offsets(BTN, col0, p.cols, p.ldb, ob);
    uint8_t *ring = lds + wave * WAVE_LDS;
    const uint32_t ring0 = lds_address(ring);
    auto issue = [&](int j) {  // stage j of this wave into buffer j % 2: QA + QB loads
        const uint8_t *ak = a_tile + (int64_t)(4 * j) * a_kstep;
        const uint8_t *bk = b_tile + (int64_t)(4 * j) * b_kstep;
        const uint32_t sa = ring0 + (j & 1) * STAGE;
#pragma unroll
        for (int q = 0; q < QA; ++q) dma16(ak, oa[q], sa + q * 1024);
#pragma unroll
        for (int q = 0; q < QB; ++q) dma16(bk, ob[q], sa + SLAB_A + q * 1024);
    };

    auto issue_tail = [&]() {  // the incomplete stage into buffer 0
        const uint8_t *ak = a_origin + (int64_t)(p.ksteps - 1) * a_kstep;
        const uint8_t *bk = b_origin + (int64_t)(p.ksteps - 1) * b_kstep;
        auto inside = [&](bool km, int q) {
            if (km) return 16 * q + (lane >> 2) < p.tail;
            return 16 * ((lane & 7) ^ (((8 * q + (lane >> 3)) >> 1) & 7)) < p.tail;
        };
#pragma unroll
        for (int q = 0; q < QA; ++q) dma16_or_zero(ak, oa[q], inside(ATN, q), ring0 + q * 1024);
#pragma unroll
        for (int q = 0; q < QB; ++q) dma16_or_zero(bk, ob[q], inside(BTN, q), ring0 + SLAB_A + q * 1024);
    };

    f32x16 acc[MI][NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
    const int frow = lane & 31, fkb = lane >> 5;

    // (Issuing the fragment reads of a half stage ahead of the MFMAs of the one before it, as
    // the general kernel does, was measured and gained nothing here: the loop waits for loads.)
    if (HALF && has_tail && ks_begin + wave == 0) issue_tail();
    else if (mine > 0) issue(0);
    if (mine > 1) issue(1);
    GroupWords<4> words;
    constexpr int UL = EPI >= EPI_UPDATE ? kGroupLoads<STATES, 4> : 0;
    if constexpr (EPI >= EPI_UPDATE) {
        load_groups<STATES, 4>(p.ep, upd, group, uo, flag);
        draw_groups<4>(p.ep, upd, group, words);
    }
#pragma clang loop unroll(disable)
    for (int j = 0; j < mine; ++j) {
        // the loads of the next stage may fly, and during the first two stages those of the update, which lie behind them
        if (UL > 0 && j < 2) {
            if (j + 1 < mine) wait_vm_lds<QA + QB + UL>();
            else wait_vm_lds<UL>();
        } else if (j + 1 < mine) {
            wait_vm_lds<QA + QB>();
        } else {
            wait_vm_lds<0>();
        }
        const uint8_t *s = ring + (j & 1) * STAGE;
#pragma unroll
        for (int sub = 0; sub < 2; ++sub) {
            i32x8 af[MI];
#pragma unroll
            for (int i = 0; i < MI; ++i) af[i] = slab64_fragment<ATN>(s, sub, i, lane);
            i32x8 bf[NJ];
#pragma unroll
            for (int j = 0; j < NJ; ++j) bf[j] = slab64_fragment<BTN>(s + SLAB_A, sub, j, lane);
            // b as the "row" matrix: a lane gets consecutive output columns
            mma64_tiles<HALF>(bf, af, acc);
        }
        if (j + 2 < mine) {
            // the loads below are invisible to the compiler (it could sink the multiplications
            // and their wait below them): wait for this wave's LDS reads explicitly
            wait_vm_lds<63>();
            issue(j + 2);
        }
    }
    wait_vm_lds<0>();

    // The four tiles meet in LDS: acc[i][j][4g + e] is row 32i + lane%32, column
    // 32j + 8g + 4*(lane/32) + e of this wave's tile.
    __syncthreads();  // every wave is done with its ring
    float *red = reinterpret_cast<float *>(lds);
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                f32x4 o = {acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
                *reinterpret_cast<f32x4 *>(red + (wave * BM + 32 * i + frow) * RED_LD + 32 * j + 8 * g + 4 * fkb) = o;
            }
    __syncthreads();
    StatsAcc st;
    if constexpr (EPI >= EPI_UPDATE) {
        auto sum = [&](int q, float v[4]) {
            const int item = threadIdx.x + 256 * q;
            f32x4 t = {};
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const f32x4 x = *reinterpret_cast<const f32x4 *>(red + (w * BM + (item >> 4)) * RED_LD + 4 * (item & 15));
                if (w == 0) t = x;
                else { t.x += x.x; t.y += x.y; t.z += x.z; t.w += x.w; }
            }
            v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
        };
        update_groups<STATES, 4>(p.ep, upd, flag, group, sum, st, uo, words);
    } else if constexpr (EPI == EPI_PARTIAL) {
        constexpr int F4 = BN / 4;
#pragma unroll
        for (int k = 0; k < BM * F4 / 256; ++k) {
            const int item = threadIdx.x + 256 * k, rr = item / F4, q = item % F4;
            f32x4 t = {};
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const f32x4 x = *reinterpret_cast<const f32x4 *>(red + (w * BM + rr) * RED_LD + 4 * q);
                if (w == 0) t = x;
                else { t.x += x.x; t.y += x.y; t.z += x.z; t.w += x.w; }
            }
            emit_partial4(p, split, row0 + rr, col0 + 4 * q, t);
        }
    } else if constexpr (EPI == EPI_RNE && BM * BN == 4 * 256) {
        // Four columns per thread: sixteen would leave three of the four waves idle behind one wave's chain of LDS reads, sums and
        // conversions (128 x 2048 x 4096 4.75 -> 4.56 us, 512 x 512 x 2048 3.54 -> 3.35).  Tiles of 32x64 are no faster with
        // it, row-major 4.30 -> 4.39 (128 x 4096 x 2048), 64x64 slower, 7.64 -> 8.01 (1000 x 1024 x 4096).
        const int rr = threadIdx.x / (BN / 4), q = threadIdx.x % (BN / 4);
        f32x4 t = {};
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const f32x4 x = *reinterpret_cast<const f32x4 *>(red + (w * BM + rr) * RED_LD + 4 * q);
            if (w == 0) t = x;
            else { t.x += x.x; t.y += x.y; t.z += x.z; t.w += x.w; }
        }
        emit_nearest4(p, row0 + rr, col0 + 4 * q, t);
    } else if (BM * BN == 64 * 64 || threadIdx.x < BM * BN / 16) {  // whole waves either way
        constexpr int CG = BN / 16;
        const int rr = threadIdx.x / CG, cg = threadIdx.x % CG;
        const int64_t r = row0 + rr, c = col0 + 16 * cg;
        float v[16];
#pragma unroll
        for (int w = 0; w < 4; ++w)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f32x4 x = *reinterpret_cast<const f32x4 *>(red + (w * BM + rr) * RED_LD + 16 * cg + 4 * q);
                if (w == 0) {
                    v[4 * q] = x.x; v[4 * q + 1] = x.y; v[4 * q + 2] = x.z; v[4 * q + 3] = x.w;
                } else {
                    v[4 * q] += x.x; v[4 * q + 1] += x.y; v[4 * q + 2] += x.z; v[4 * q + 3] += x.w;
                }
            }
        if (r < p.rows && c < p.cols) {
            if (HALF && EPI == EPI_FULL && (p.cols & 15) != 0)
                finish16_ragged(p.ep, r, c, p.cols - c < 16 ? (int)(p.cols - c) : 16, v, st);
            else emit16<EPI>(p, r, c, v, st);
        }
    }
    if constexpr (EPI >= EPI_FULL) {
        if (p.ep.stats != nullptr) st.flush(p.ep.stats);
    }
}

template <int EPI, bool ATN, bool BTN, int CONV, int BM = 64, int BN = 64, bool HALF = false>
__global__ __launch_bounds__(256, 1) void gemm_wavek_kernel(const GemmArgs p) {
    gemm_wavek<EPI, ATN, BTN, CONV, BM, BN, HALF>(p, UpdateHook{});
}
template <int STATES, bool ATN, bool BTN, int CONV, bool HALF = false>
__global__ __launch_bounds__(256, 1) void gemm_wavek_update_kernel(const GemmArgs p, const UpdateHook upd) {
    gemm_wavek<EPI_UPDATE + STATES, ATN, BTN, CONV, 64, 64, HALF>(p, upd);
}

}  // namespace mp8
