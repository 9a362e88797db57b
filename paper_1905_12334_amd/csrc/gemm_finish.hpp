// Second pass of a GEMM whose epilogue is not fused (split contraction, ragged columns, poorly filled tiles
// with an FP32 or transposed result), optionally with the master-weight update of Figure 1b applied to the
// codes it has just rounded; and the any-shape fallback kernel.
#pragma once

#include "gemm_common.hpp"

namespace mp8 {

// Finish four consecutive columns from element i0 on (i0 % 4 == 0, row length a multiple of 4) with their random words.  Row
// and column, a division of 64 bits, are only worked out for what needs them.
__device__ __forceinline__ uint32_t finish4(const Epilogue &ep, int64_t i0, float v[4], Words4 rnd, StatsAcc &st) {
    if (ep.acc_mode != 0) {
        f32x4 *p = reinterpret_cast<f32x4 *>(ep.acc + i0);
        if (ep.acc_mode == 2) {
            f32x4 o = *p;
            v[0] += o.x; v[1] += o.y; v[2] += o.z; v[3] += o.w;
        }
        f32x4 n = {v[0], v[1], v[2], v[3]};
        *p = n;
    }
    if (ep.out8 == nullptr && ep.out8_t == nullptr && ep.stats == nullptr && !ep.want_codes) return 0;
    float y[4] = {v[0] * ep.alpha, v[1] * ep.alpha, v[2] * ep.alpha, v[3] * ep.alpha};
    uint32_t pk = e5m2_pack4_rt(y, rnd.r01, rnd.r23, ep.sr != 0, ep.sat != 0);
    int64_t r = 0, c = 0;
    if (ep.mask || ep.out8_t != nullptr) {
        r = i0 / ep.cols;
        c = i0 - r * ep.cols;
    }
    if (ep.mask && conv_padding_row(ep, r)) pk = 0;
    else if (ep.stats != nullptr) st.add4(y, pk);
    if (ep.out8 != nullptr) store_through(reinterpret_cast<uint32_t *>(ep.out8 + i0), pk);
    if (ep.out8_t != nullptr) {
        uint8_t *t = ep.out8_t + c * ep.rows + r;
        t[0] = (uint8_t)pk;
        t[ep.rows] = (uint8_t)(pk >> 8);
        t[2 * ep.rows] = (uint8_t)(pk >> 16);
        t[3 * ep.rows] = (uint8_t)(pk >> 24);
    }
    return pk;
}

// Optional second half of Figure 1b in the finishing pass: the 8-bit weight gradient that was
// just rounded is un-scaled and applied to the half-precision master weights, exactly as
// mp8_sgd_update_fp16_sr would do it from memory (same arithmetic, same random stream: element
// i uses halfword i % 8 of block i / 8 of the update's own Philox stream).  w16 == nullptr:
// no update.
struct UpdateHook {
    uint16_t *w16;
    uint8_t *w8_out;
    const uint32_t *skip;
    float neg_lr, inv_scale;
    int sr;
    uint64_t seed, offset;
    // optimizer state, in place: none (plain SGD), the velocity of momentum SGD (state0), or the
    // two moments of ADAM (state0, state1) -- the rules of the stand-alone update kernels
    int states;
    float *state0, *state1;
    float mu, wd;                            // momentum; L2 regularisation of either rule
    float b1, b2, omb1, omb2, eps;           // ADAM
    double ric1, ric2;
};

// The hook's update rule: f(rule) with the rule object the stand-alone update kernels use.
template <int STATES, class F>
__device__ __forceinline__ void with_rule(const UpdateHook &u, F f) {
    if constexpr (STATES == 0) f(SgdRule{u.neg_lr});
    else if constexpr (STATES == 1) f(MomentumRule{u.neg_lr, u.mu, u.wd});
    else f(AdamRule{u.neg_lr, u.b1, u.b2, u.omb1, u.omb2, u.eps, u.wd, u.ric1, u.ric2});
}

template <int STATES>
__device__ __forceinline__ void update_element(const UpdateHook &u, int64_t i, uint32_t code, uint32_t r16) {
    float st[2] = {0.0f, 0.0f};
    if constexpr (STATES >= 1) st[0] = u.state0[i];
    if constexpr (STATES == 2) st[1] = u.state1[i];
    uint32_t h = 0;
    with_rule<STATES>(u, [&](const auto &rule) {
        h = u.sr ? update_one<true>(rule, u.w16[i], code, st, u.inv_scale, r16)
                 : update_one<false>(rule, u.w16[i], code, st, u.inv_scale, 0u);
    });
    if constexpr (STATES >= 1) u.state0[i] = st[0];
    if constexpr (STATES == 2) u.state1[i] = st[1];
    u.w16[i] = (uint16_t)h;
    if (u.w8_out != nullptr) u.w8_out[i] = (uint8_t)e5m2_of_half(h);
}

// What update4 reads of elements i0 .. i0+3: fetched before the slices are summed, so that these
// loads fly together with the slice loads instead of after them.
struct UpdateOperands4 {
    u32x2 w;
    f32x4 s0, s1;
};
template <int STATES>
__device__ __forceinline__ UpdateOperands4 load_update4(const UpdateHook &u, int64_t i0) {
    UpdateOperands4 o{};
    o.w = *reinterpret_cast<const u32x2 *>(u.w16 + i0);
    if constexpr (STATES >= 1) o.s0 = *reinterpret_cast<const f32x4 *>(u.state0 + i0);
    if constexpr (STATES == 2) o.s1 = *reinterpret_cast<const f32x4 *>(u.state1 + i0);
    return o;
}

// Elements i0 .. i0+3 (i0 % 4 == 0) from their four packed gradient codes and random words.  All results go past the L2: a tile has little
// to store, all CUs do it at the same moment, at the end.  Weight gradients, us, past the L2 / state plain / state non-temporal / weights and
// codes plain: 4096 x 2048 x 512 momentum 15.8 / 16.2 / 16.1 / 16.1, ADAM 17.4 / 17.9 / 17.6 / 17.8; 2048 x 512 x 2048 9.7 / 10.3 / 10.3 / 10.3,
// 12.1 / 13.1 / 12.9 / 12.6; 1024^3 7.3 / 7.9 / 7.9 / 7.9, 9.3 / 10.0 / 9.9 / 9.7; whole training steps of these 0.3 to 0.9 shorter.
template <int STATES>
__device__ __forceinline__ void update4(const UpdateHook &u, int64_t i0, uint32_t pk, const UpdateOperands4 &in, Words4 r) {
    uint32_t w[2] = {in.w.x, in.w.y};
    float st[4][2] = {{0.0f, 0.0f}, {0.0f, 0.0f}, {0.0f, 0.0f}, {0.0f, 0.0f}};
    if constexpr (STATES >= 1) {
        const f32x4 x = in.s0;
        st[0][0] = x.x; st[1][0] = x.y; st[2][0] = x.z; st[3][0] = x.w;
    }
    if constexpr (STATES == 2) {
        const f32x4 x = in.s1;
        st[0][1] = x.x; st[1][1] = x.y; st[2][1] = x.z; st[3][1] = x.w;
    }
    with_rule<STATES>(u, [&](const auto &rule) {
        if (u.sr) update_four<true>(rule, w, pk, st, u.inv_scale, r);
        else update_four<false>(rule, w, pk, st, u.inv_scale, Words4{0u, 0u});
    });
    if constexpr (STATES >= 1) {
        const f32x4 x = {st[0][0], st[1][0], st[2][0], st[3][0]};
        store_through(reinterpret_cast<f32x4 *>(u.state0 + i0), x);
    }
    if constexpr (STATES == 2) {
        const f32x4 x = {st[0][1], st[1][1], st[2][1], st[3][1]};
        store_through(reinterpret_cast<f32x4 *>(u.state1 + i0), x);
    }
    const u32x2 o = {w[0], w[1]};
    store_through(reinterpret_cast<u32x2 *>(u.w16 + i0), o);
    if (u.w8_out != nullptr) store_through(reinterpret_cast<uint32_t *>(u.w8_out + i0), e5m2_of_halves(w));
}

// The update inside a GEMM's own epilogue.  A thread finishes Q groups of four consecutive weights; group
// q of neighbouring lanes lies side by side (runs of 128 or 256 bytes of FP32 state; sixteen consecutive
// weights per lane, as the plain epilogues have them, cost 6 us more here for 1 M weights with ADAM).  Lanes
// 2m and 2m + 1 hold the halves of one random block.  where(q): row, column (a multiple of 4), and whether
// it exists; value(q, v): the four sums.  `in`: what load_groups fetched.  The fetch goes out behind the loads of the
// first stages, in front of which it held them up (4096 x 2048 x 512 with ADAM 17.6 us, 16.9 now), as always the same kGroupLoads
// instructions, whether a group exists or not, so that hand-counted waits know them.
struct GroupAt {
    int64_t r, c;
    bool valid;
};
// The skip flag is fetched with them, into a vector register: as a scalar it would be waited for at once.
template <int STATES, int Q>
constexpr int kGroupLoads = Q * (1 + STATES) + 1;
template <int STATES, int Q, class Where>
__device__ __forceinline__ void load_groups(const Epilogue &ep, const UpdateHook &u, Where where, UpdateOperands4 (&in)[Q], uint32_t &flag) {
    uint32_t zero = 0;
    asm("" : "+v"(zero));
    asm volatile("" ::: "memory");
    flag = (u.skip != nullptr ? u.skip : reinterpret_cast<const uint32_t *>(u.w16))[zero];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const GroupAt g = where(q);
        in[q] = load_update4<STATES>(u, g.valid ? g.r * ep.cols + g.c : 0);
    }
    asm volatile("" ::: "memory");
}
// The random words of the two roundings (gradient, weight).  Drawn while the first operands are on their
// way: one workgroup has nothing else to do then, and 1 - 2 us of multiplications to do after the
// contraction otherwise.
template <int Q>
struct GroupWords {
    Words4 g[Q], w[Q];
};
template <int Q, class Where>
__device__ __forceinline__ void draw_groups(const Epilogue &ep, const UpdateHook &u, Where where, GroupWords<Q> &out) {
    static_assert(Q % 2 == 0, "random blocks are shared over pairs of groups");
    auto draw = [&](uint64_t seed, uint64_t offset, Words4(&w)[Q]) {
        const Philox rng(seed, offset);
#pragma unroll
        for (int q = 0; q < Q; q += 2) {
            const GroupAt a = where(q), b = where(q + 1);
            rng.pair_words((uint64_t)(a.r * ep.cols + a.c) >> 3, (uint64_t)(b.r * ep.cols + b.c) >> 3, w[q], w[q + 1]);
        }
    };
    out = GroupWords<Q>{};
    if (ep.sr) draw(ep.seed, ep.offset, out.g);
    if (u.sr) draw(u.seed, u.offset, out.w);
}
// A rolled loop, the register arrays shifted down by one group per turn: straight-line code for four groups
// of ADAM is 19 KB that every launch would fetch through a cold instruction cache.  The sums of all groups
// are read ahead of it: one latency of the LDS instead of Q.
template <int STATES, int Q, class Where, class Value>
__device__ __forceinline__ void update_groups(const Epilogue &ep, const UpdateHook &u, uint32_t flag, Where where, Value value,
                                              StatsAcc &st, UpdateOperands4 (&in)[Q], GroupWords<Q> &words) {
    const bool updating = u.skip == nullptr || flag == 0;
    float sums[Q][4];
#pragma unroll
    for (int q = 0; q < Q; ++q) value(q, sums[q]);
#pragma unroll 1
    for (int q = 0; q < Q; ++q) {
        const GroupAt g = where(q);
        if (g.valid) {
            const int64_t i0 = g.r * ep.cols + g.c;
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = sums[0][e] * ep.alpha;
            const uint32_t pk = e5m2_pack4_rt(v, words.g[0].r01, words.g[0].r23, ep.sr != 0, ep.sat != 0);
            if (ep.stats != nullptr) st.add4(v, pk);
            if (ep.out8 != nullptr) store_through(reinterpret_cast<uint32_t *>(ep.out8 + i0), pk);
            if (updating) update4<STATES>(u, i0, pk, in[0], words.w[0]);
        }
#pragma unroll
        for (int k = 0; k + 1 < Q; ++k) {
            in[k] = in[k + 1];
            words.g[k] = words.g[k + 1];
            words.w[k] = words.w[k + 1];
#pragma unroll
            for (int e = 0; e < 4; ++e) sums[k][e] = sums[k + 1][e];
        }
    }
}

// Sum the FP32 tiles of the contraction slices in slice order and finish: the complete sum is
// rounded once.  One thread per four columns (per element when the row length is not a
// multiple of four).  STATES: state words per weight of the update rule the hook carries (-1: no
// update, 0: plain SGD, 1: momentum, 2: ADAM).  NB: slice loads in flight; a grid of one chain of latencies per thread is
// what this pass mostly is, so everything it reads (the skip flag as well, into a vector register) is requested
// at once and without a branch, and the random words are drawn while it travels (weight gradients with update, us: 1152 x 128 over 25088
// 17.0 -> 16.6, 512 x 512 over 12800 14.0 -> 13.6).
template <int STATES, int NB>
__global__ __launch_bounds__(256) void splitk_finish_kernel(const float *__restrict__ partial,
                                                            int splits, const Epilogue ep,
                                                            const UpdateHook upd) {
    StatsAcc st;
    // an overflowed step leaves the master weights alone (the gradient codes are still written)
    uint32_t flag = 0;
    const bool may_skip = STATES >= 0 && upd.skip != nullptr;
    if constexpr (STATES >= 0) {
        uint32_t zero = 0;
        asm("" : "+v"(zero));
        flag = (may_skip ? upd.skip : reinterpret_cast<const uint32_t *>(partial))[zero];
    }
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t slice = ep.rows * ep.cols;
    if ((ep.cols & 3) == 0) {
        const int64_t total = slice >> 2;
        for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += stride) {
            const int64_t i0 = t << 2;
            UpdateOperands4 uo{};
            if constexpr (STATES >= 0) uo = load_update4<STATES>(upd, i0);
            // NB slices at a time, added in slice order.  Slices beyond the last are
            // read from the last one again and replaced by +0: the running sum starts from +0 and
            // is therefore never -0, so adding +0 leaves every bit of it as it is.
            float v[4] = {0.f, 0.f, 0.f, 0.f};
            f32x4 x[NB];
            auto load = [&](int s) {
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    const int sj = s + j < splits ? s + j : splits - 1;
                    x[j] = *reinterpret_cast<const f32x4 *>(partial + (int64_t)sj * slice + i0);
                }
            };
            auto add = [&](int s) {
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    const bool on = s + j < splits;
                    v[0] += on ? x[j].x : 0.f; v[1] += on ? x[j].y : 0.f;
                    v[2] += on ? x[j].z : 0.f; v[3] += on ? x[j].w : 0.f;
                }
            };
            load(0);
            Words4 rg{0u, 0u}, rw{0u, 0u};
            if (ep.sr) rg = Philox(ep.seed, ep.offset).half_block((uint64_t)i0);
            if (STATES >= 0 && upd.sr) rw = Philox(upd.seed, upd.offset).half_block((uint64_t)i0);
            add(0);
            for (int s = NB; s < splits; s += NB) {
                load(s);
                add(s);
            }
            const uint32_t pk = finish4(ep, i0, v, rg, st);
            if constexpr (STATES >= 0) {
                uint32_t skip = flag;
                asm volatile("" : "+v"(skip));  // (the test stays here: ahead of the loop it would wait for the flag)
                if (!(may_skip && skip != 0u)) update4<STATES>(upd, i0, pk, uo, rw);
            }
        }
    } else {
        for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < slice; i += stride) {
            float v = 0.f;
            for (int s = 0; s < splits; ++s) v += partial[(int64_t)s * slice + i];
            const int64_t r = i / ep.cols;
            const uint32_t code = finish1(ep, r, i - r * ep.cols, v, st);
            if constexpr (STATES >= 0) {
                if (!(may_skip && flag != 0u)) {
                    uint32_t r16 = 0;
                    if (upd.sr) {
                        const Philox rng(upd.seed, upd.offset);
                        r16 = philox_half(rng.block((uint64_t)i >> 3), (int)(i & 7));
                    }
                    update_element<STATES>(upd, i, code, r16);
                }
            }
        }
    }
    if (ep.stats != nullptr) st.flush(ep.stats);
}

// The transposed copy of finished codes: dst [cols, rows] from src [rows, cols].  A pass of its own over 2 bytes per
// element: a finishing pass would store it byte by byte, its lanes lying along the rows of src, each into a line of its
// own (4096 x 4096 x 2048 with it 124 us, now 37; where it pays: copied_from_codes).  Tiles of 128 x 128 through LDS; 16-byte pieces, eight lanes to a line, where both
// counts are multiples of 16 (WHOLE), else pieces of any alignment and length (at least four columns).
template <bool WHOLE>
__global__ __launch_bounds__(256) void transpose_codes_kernel(const uint8_t *__restrict__ src, uint8_t *__restrict__ dst,
                                                              int64_t rows, int64_t cols) {
    constexpr int T = 128, P = T / 4 + 1;  // LDS row pitch in dwords
    __shared__ uint32_t tile[T * P];
    const int64_t tiles_c = (cols + T - 1) / T, ntiles = ((rows + T - 1) / T) * tiles_c;
    const int tid = threadIdx.x, k = tid & 7, cg = tid >> 3;
    for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const int64_t r0 = t / tiles_c * T, c0 = t % tiles_c * T;
        if constexpr (WHOLE) {
            u32x4 x[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int64_t r = r0 + 32 * i + cg, c = c0 + 16 * k;
                x[i] = r < rows && c < cols ? *reinterpret_cast<const u32x4 *>(src + r * cols + c) : u32x4{0, 0, 0, 0};
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) tile[(32 * i + cg) * P + 4 * k + e] = x[i][e];
        } else {
            // (rows and pieces beyond the matrix are read from its last ones: at least four columns)
            const int g = tid & 31;
            const int64_t c = c0 + 4 * g, cl = c + 4 <= cols ? c : cols - 4;
            const int shift = c - cl < 4 ? 8 * (int)(c - cl) : 0;
            uint32_t x[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int64_t r = r0 + 8 * i + (tid >> 5);
                __builtin_memcpy(&x[i], src + (r < rows ? r : rows - 1) * cols + cl, 4);
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) tile[(8 * i + (tid >> 5)) * P + g] = x[i] >> shift;
        }
        __syncthreads();
        uint32_t colw[4][4];  // [column][row block of 4]
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            uint32_t rr[4], cc[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) rr[j] = tile[(16 * k + 4 * b + j) * P + cg];
            transpose4x4(rr, cc);
#pragma unroll
            for (int col = 0; col < 4; ++col) colw[col][b] = cc[col];
        }
        const int64_t orow = r0 + 16 * k;
#pragma unroll
        for (int col = 0; col < 4; ++col) {
            const int64_t oc = c0 + 4 * cg + col;
            if (orow < rows && oc < cols) {
                uint8_t *to = dst + oc * rows + orow;
                const u32x4 o = {colw[col][0], colw[col][1], colw[col][2], colw[col][3]};
                if (WHOLE) *reinterpret_cast<u32x4 *>(to) = o;
                else if (orow + 16 <= rows) __builtin_memcpy(to, &o, 16);
                else {
#pragma unroll
                    for (int e = 0; e < 15; ++e)
                        if (orow + e < rows) to[e] = (uint8_t)(colw[col][e >> 2] >> (8 * (e & 3)));
                }
            }
        }
        __syncthreads();  // the next tile overwrites this one
    }
}

// Any-shape fallback: one thread per output element, operands decoded one by one, FP32 fused
// multiply-adds in contraction order.  Used for what gemm_any_kernel cannot take: contractions shorter
// than 16, contraction-major operands with fewer than 16 rows or columns, enormous leading dimensions.
__global__ __launch_bounds__(256) void gemm_generic_kernel(const uint8_t *__restrict__ a,
                                                           int64_t lda,
                                                           const uint8_t *__restrict__ b,
                                                           int64_t ldb, int64_t kc, int tn,
                                                           const Epilogue ep) {
    const int64_t total = ep.rows * ep.cols;
    StatsAcc st;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += stride) {
        const int64_t r = t / ep.cols, c = t - r * ep.cols;
        // element (r, j) of a: a[r * lda + j], or a[j * lda + r] when a is contraction-major
        // (bit 0 of tn; bit 1 likewise for b)
        const uint8_t *ar = (tn & 1) ? a + r : a + r * lda, *bc = (tn & 2) ? b + c : b + c * ldb;
        const int64_t sa = (tn & 1) ? lda : 1, sb = (tn & 2) ? ldb : 1;
        float s = 0.f;
        for (int64_t j = 0; j < kc; ++j)
            s = __builtin_fmaf(e5m2_to_f32(ar[j * sa]), e5m2_to_f32(bc[j * sb]), s);
        finish1(ep, r, c, s, st);
    }
    if (ep.stats != nullptr) st.flush(ep.stats);
}

}  // namespace mp8
