// What the GEMM kernels share: argument structs, the epilogue of one output run (one rounding
// of the complete FP32 sum, Section 3 of arXiv 1905.12334), the workgroup -> tile map, and the
// direct-to-LDS load with its hand-tracked wait.
#pragma once

#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <type_traits>

#include "mp8_device.hpp"

namespace mp8 {

using i32x8 = int __attribute__((ext_vector_type(8)));
using i32x4 = int __attribute__((ext_vector_type(4)));
using i32x2 = int __attribute__((ext_vector_type(2)));
using f32x16 = float __attribute__((ext_vector_type(16)));

constexpr int BK = 128;  // bytes (= elements) of contraction per pipeline stage

// Division of a 31-bit number by a fixed divisor with a precomputed reciprocal:
// m = floor(2^32 / d) (all ones for d = 1) makes mulhi(x, m) the quotient or one less.
struct FastDiv {
    uint32_t d, m;
};
static inline FastDiv make_fastdiv(uint32_t d) {
    FastDiv f;
    f.d = d;
    f.m = d <= 1 ? 0xFFFFFFFFu : (uint32_t)((1ull << 32) / d);
    return f;
}
__device__ __forceinline__ uint32_t fastdiv(uint32_t x, const FastDiv &f, uint32_t &rem) {
    uint32_t q = __umulhi(x, f.m);
    rem = x - q * f.d;
    if (rem >= f.d) {
        ++q;
        rem -= f.d;
    }
    return q;
}

struct Epilogue {
    float alpha;
    float *acc;
    int acc_mode;
    // tile_epilogue (see launch_mfma): the FP32 result by a pass of its own ahead of the codes, past the L2 (1) or
    // into it (2); the codes into the L2
    int acc_lines, codes_plain;
    uint8_t *out8;
    uint8_t *out8_t;
    int sr;
    int sat;
    uint64_t seed, offset;
    mp8_stats *stats;
    int want_codes;  // the caller consumes the returned codes even if nothing is stored
    int64_t rows, cols;
    // Convolution outputs live on the zero-padded pixel grid (rows = padded pixels): rows that
    // are padding receive zero codes and stay out of the statistics.  mask = 0: no masking.
    int mask;
    int hh;              // H + 2
    int64_t valid_rows;  // B * (H+2) * (W+2); rows beyond are padding as well
    FastDiv div_img;     // by (H+2) * (W+2)
    FastDiv div_w2;      // by W + 2
};

// Is output row r a padding pixel of the convolution grid?
__device__ __forceinline__ bool conv_padding_row(const Epilogue &ep, int64_t r) {
    if (r >= ep.valid_rows) return true;
    uint32_t rem, x;
    fastdiv((uint32_t)r, ep.div_img, rem);
    const uint32_t y = fastdiv(rem, ep.div_w2, x);
    return y == 0 || y == (uint32_t)ep.hh - 1 || x == 0 || x == ep.div_w2.d - 1;
}

// What a convolution adds to the operand addressing (conv = 0: plain GEMM).
struct ConvArgs {
    int w2;               // W + 2: a tap (r, s) shifts the pixel row by (r-1)*w2 + (s-1)
    FastDiv div_cpb;      // by units_per_tap
    int units_per_tap;    // 64-byte units of the contraction per tap (contracted channels / 64)
    int odd_units;        // the contraction has an odd number of units: its last stage starts one early
    int64_t b_tap_stride; // bytes between the weight slabs of two taps
    FastDiv div_ci;       // weight gradient: by Cin (tile row -> tap, first channel)
};

// Pixel rows beyond a tile's own that gemm_conv_kernel holds: 2 (W + 3), so W <= 61.
constexpr int kConvHalo = 128;

struct GemmArgs {
    const uint8_t *a;
    const uint8_t *b;
    int64_t lda, ldb;
    int64_t rows, cols;
    int ksteps;         // contraction length / BK, rounded up (pipeline stages)
    // Contraction indices of a last, incomplete stage (0: the contraction is whole stages).  The half-precision
    // forms of the direct-to-LDS kernels multiply that stage FIRST, so that only their start-up code, and
    // nothing in their loops, knows of it: global stage 0 is the incomplete one and stage s > 0 covers
    // indices BK (s - 1) ...  What lies beyond the contraction reads as zero (see dma16_or_zero).
    int tail;
    int splits;         // number of contraction slices
    int tiles_m, tiles_n;
    // host-side precomputation for the workgroup -> (slice, tile) map, so that the kernel's
    // start-up does no integer division
    FastDiv div_tiles;  // by tiles_m * tiles_n
    FastDiv div_band;   // by 8 * tiles_n
    FastDiv div_tail;   // by the height of the last band of tile rows (tiles_m % 8, or 8)
    FastDiv div_tn;     // by tiles_n
    int ks_per, ks_extra;  // ksteps / splits and ksteps % splits
    float *partial;     // [splits, rows, cols] when splits > 1
    ConvArgs cv;
    Epilogue ep;
};

// One output element, any shape: optional FP32 accumulate / store, one rounding to 8 bits,
// optional transposed copy, statistics.  Only the finishing kernels use it (ragged shapes).
__device__ __forceinline__ uint32_t finish1(const Epilogue &ep, int64_t r, int64_t c, float v,
                                            StatsAcc &st) {
    const int64_t i = r * ep.cols + c;
    if (ep.acc_mode != 0) {
        if (ep.acc_mode == 2) v += ep.acc[i];
        ep.acc[i] = v;
    }
    if (ep.out8 == nullptr && ep.out8_t == nullptr && ep.stats == nullptr && !ep.want_codes) return 0;
    if (ep.mask && conv_padding_row(ep, r)) {
        if (ep.out8 != nullptr) ep.out8[i] = 0;
        if (ep.out8_t != nullptr) ep.out8_t[c * ep.rows + r] = 0;
        return 0;
    }
    const float y = v * ep.alpha;
    uint32_t code;
    if (ep.sr) {
        const Philox rng(ep.seed, ep.offset);
        uint32_t r16 = philox_half(rng.block((uint64_t)i >> 3), (int)(i & 7));
        code = e5m2_from_f32_bits<true>(f2u(y), r16, ep.sat != 0);
    } else {
        code = e5m2_from_f32_bits<false>(f2u(y), 0u, ep.sat != 0);
    }
    if (ep.stats != nullptr) st.add1(y, code);
    if (ep.out8 != nullptr) ep.out8[i] = (uint8_t)code;
    if (ep.out8_t != nullptr) ep.out8_t[c * ep.rows + r] = (uint8_t)code;
    return code;
}

// Finish sixteen consecutive columns c .. c+15 (c % 16 == 0) of output row r of an output
// whose row length is a multiple of 16: 16-byte accesses, two Philox blocks, hardware
// conversions.  Written to stay small: the rounding mode is a run-time flag and the rare
// conversions are out of line.
// acc_done: v has been through ep.acc already.  kAlways: statistics without a test (see StatsAcc::add4_always), which gemm_shortk_kernel
// alone is better off with (4096 x 4096 x 128 to nearest 35.8 us with it, 33.2 without; everywhere else the test is worth 2 to 6 %).
// kThrough: the codes by store_through, unless ep.codes_plain.
template <bool kAlways = false, bool kThrough = false>
__device__ __forceinline__ void finish16(const Epilogue &ep, int64_t r, int64_t c, float v[16],
                                         StatsAcc &st, bool acc_done = false) {
    const int64_t i0 = r * ep.cols + c;
    if (ep.acc_mode != 0 && !acc_done) {
        f32x4 *p = reinterpret_cast<f32x4 *>(ep.acc + i0);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (ep.acc_mode == 2) {
                f32x4 o = p[q];
                v[4 * q] += o.x; v[4 * q + 1] += o.y; v[4 * q + 2] += o.z; v[4 * q + 3] += o.w;
            }
            f32x4 n = {v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
            p[q] = n;
        }
    }
    if (ep.out8 == nullptr && ep.out8_t == nullptr && ep.stats == nullptr) return;
    const bool padding = ep.mask && conv_padding_row(ep, r);
    uint32_t rw[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (ep.sr) {
        const Philox rng(ep.seed, ep.offset);
        uint4 w0 = rng.block((uint64_t)i0 >> 3), w1 = rng.block(((uint64_t)i0 >> 3) + 1);
        rw[0] = w0.x; rw[1] = w0.y; rw[2] = w0.z; rw[3] = w0.w;
        rw[4] = w1.x; rw[5] = w1.y; rw[6] = w1.z; rw[7] = w1.w;
    }
    uint32_t pk[4];
    float y[4][4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
#pragma unroll
        for (int e = 0; e < 4; ++e) y[q][e] = v[4 * q + e] * ep.alpha;
        pk[q] = e5m2_pack4_rt(y[q], rw[2 * q], rw[2 * q + 1], ep.sr != 0, ep.sat != 0);
        if (padding) pk[q] = 0;
        else if (kAlways && ep.stats != nullptr) st.add4_always(y[q], pk[q]);
    }
    if (!kAlways && ep.stats != nullptr && !padding) st.add<4, false>(y, pk);
    if (ep.out8 != nullptr) {
        u32x4 o = {pk[0], pk[1], pk[2], pk[3]};
        if (kThrough && !ep.codes_plain) store_through(reinterpret_cast<u32x4 *>(ep.out8 + i0), o);
        else *reinterpret_cast<u32x4 *>(ep.out8 + i0) = o;
    }
    if (ep.out8_t != nullptr) {
        uint8_t *t = ep.out8_t + c * ep.rows + r;
#pragma nounroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t w = q == 0 ? pk[0] : q == 1 ? pk[1] : q == 2 ? pk[2] : pk[3];
            t[(4 * q + 0) * ep.rows] = (uint8_t)w;
            t[(4 * q + 1) * ep.rows] = (uint8_t)(w >> 8);
            t[(4 * q + 2) * ep.rows] = (uint8_t)(w >> 16);
            t[(4 * q + 3) * ep.rows] = (uint8_t)(w >> 24);
        }
    }
}

// finish16 for any row length and any c: n (1 .. 16) valid columns, addresses without alignment.
// The random words of sixteen elements that start at halfword h of a Philox block come from three
// blocks, shifted down by h halfwords.
__device__ __forceinline__ void finish16_ragged(const Epilogue &ep, int64_t r, int64_t c, int n, float v[16],
                                                StatsAcc &st) {
    const int64_t i0 = r * ep.cols + c;
    if (ep.acc_mode != 0) {
        float *p = ep.acc + i0;
#pragma unroll
        for (int e = 0; e < 16; ++e)
            if (e < n) {
                if (ep.acc_mode == 2) v[e] += p[e];
                p[e] = v[e];
            }
    }
    if (ep.out8 == nullptr && ep.out8_t == nullptr && ep.stats == nullptr) return;
    uint32_t rw[12];
#pragma unroll
    for (int j = 0; j < 12; ++j) rw[j] = 0;
    if (ep.sr) {
        const Philox rng(ep.seed, ep.offset);
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            const uint4 w = rng.block(((uint64_t)i0 >> 3) + b);
            rw[4 * b] = w.x; rw[4 * b + 1] = w.y; rw[4 * b + 2] = w.z; rw[4 * b + 3] = w.w;
        }
        const int h = (int)(i0 & 7);
        // (bit masks: with `?:` the compiler indexes the array in memory)
        const uint32_t m4 = (h & 4) ? ~0u : 0u, m2 = (h & 2) ? ~0u : 0u;
#pragma unroll
        for (int j = 0; j < 10; ++j) rw[j] = (rw[j + 2] & m4) | (rw[j] & ~m4);
#pragma unroll
        for (int j = 0; j < 9; ++j) rw[j] = (rw[j + 1] & m2) | (rw[j] & ~m2);
#pragma unroll
        for (int j = 0; j < 8; ++j) rw[j] = __builtin_amdgcn_alignbit(rw[j + 1], rw[j], (h & 1) * 16);
    }
    uint32_t pk[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float y[4] = {v[4 * q] * ep.alpha, v[4 * q + 1] * ep.alpha, v[4 * q + 2] * ep.alpha, v[4 * q + 3] * ep.alpha};
        pk[q] = e5m2_pack4_rt(y, rw[2 * q], rw[2 * q + 1], ep.sr != 0, ep.sat != 0);
        if (ep.stats != nullptr) {
            if (4 * q + 4 <= n) {
                st.add4_always(y, pk[q]);
            } else {
#pragma unroll
                for (int e = 0; e < 3; ++e)
                    if (4 * q + e < n) st.add1(y[e], (pk[q] >> (8 * e)) & 0xFFu);
            }
        }
    }
    if (ep.out8 != nullptr) {
        uint8_t *p = ep.out8 + i0;
        if (n == 16) {
            const u32x4 o = {pk[0], pk[1], pk[2], pk[3]};
            __builtin_memcpy(p, &o, 16);  // an unaligned 16-byte store
        } else {
#pragma unroll
            for (int e = 0; e < 15; ++e)
                if (e < n) p[e] = (uint8_t)(pk[e >> 2] >> (8 * (e & 3)));
        }
    }
    if (ep.out8_t != nullptr) {
        uint8_t *t = ep.out8_t + c * ep.rows + r;
#pragma unroll
        for (int e = 0; e < 16; ++e)
            if (e < n) t[e * ep.rows] = (uint8_t)(pk[e >> 2] >> (8 * (e & 3)));
    }
}

// Map workgroup bid of nb to (slice, tile row, tile column).  Consecutive ids go to
// different XCDs (round robin), so ids are first regrouped so that each XCD works on a
// contiguous range of tiles and its L2 sees operand reuse; inside the range, tiles are
// walked in bands of 8 tile-rows.
__device__ __forceinline__ void map_tile(const GemmArgs &p, uint32_t nb, uint32_t bid, int &split, int &tm, int &tn) {
    const uint32_t xcd = bid & 7, idx = bid >> 3;
    const uint32_t per = nb >> 3, rem = nb & 7;
    const uint32_t pid = xcd * per + (xcd < rem ? xcd : rem) + idx;
    uint32_t t, in;
    split = (int)fastdiv(pid, p.div_tiles, t);
    constexpr uint32_t GM = 8;
    const uint32_t g = fastdiv(t, p.div_band, in);
    const uint32_t first = g * GM;
    if ((uint32_t)p.tiles_m - first >= GM) {
        tm = (int)(first + (in & (GM - 1)));
        tn = (int)(in >> 3);
    } else {
        uint32_t r;
        tn = (int)fastdiv(in, p.div_tail, r);
        tm = (int)(first + r);
    }
}
__device__ __forceinline__ void map_block(const GemmArgs &p, int &split, int &tm, int &tn) { map_tile(p, gridDim.x, blockIdx.x, split, tm, tn); }

// EPI_UPDATE + s: EPI_FULL (without FP32 and transposed outputs), then the master-weight update of a rule
// with s state words per weight (UpdateHook in gemm_finish.hpp).
enum { EPI_PARTIAL = 0, EPI_RNE = 1, EPI_FULL = 2, EPI_UPDATE = 3 };

// EPI_PARTIAL: four consecutive columns c .. c+3 (c % 4 == 0) of row r of an FP32 tile to slice `split` of the workspace.
// To be called with neighbouring lanes side by side in a row, so that a store instruction of a wave covers whole lines:
// with sixteen columns per lane, four stores of every fourth sixteen bytes, the tiles left at 1 TB/s (512 x 2048 in
// two slices of 64x64 tiles over 4096: 17.5 us, half of it these stores).
__device__ __forceinline__ void emit_partial4(const GemmArgs &p, int split, int64_t r, int64_t c, f32x4 v) {
    if (r >= p.rows) return;
    float *dst = p.partial + ((int64_t)split * p.rows + r) * p.cols + c;
    if ((p.cols & 3) == 0) {
        if (c < p.cols) store_through(reinterpret_cast<f32x4 *>(dst), v);
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (c + e < p.cols) dst[e] = v[e];
    }
}

// EPI_RNE: the codes of such a group (the host sends only row lengths that are multiples of 16 here).
__device__ __forceinline__ void emit_nearest4(const GemmArgs &p, int64_t r, int64_t c, f32x4 v) {
    if (r >= p.rows || c >= p.cols) return;
    const float y[4] = {v.x * p.ep.alpha, v.y * p.ep.alpha, v.z * p.ep.alpha, v.w * p.ep.alpha};
    uint32_t pk = e5m2_pack4<false>(y, 0u, 0u, false);
    if (p.ep.mask && conv_padding_row(p.ep, r)) pk = 0;
    *reinterpret_cast<uint32_t *>(p.ep.out8 + r * p.cols + c) = pk;
}

// What a tile kernel does with sixteen consecutive columns c .. c+15 (c % 16 == 0) of output row
// r, per epilogue variant (described at the main kernel): the RNE-only conversion, or the complete epilogue.
template <int EPI, bool kThrough = false, bool kAlways = false>
__device__ __forceinline__ void emit16(const GemmArgs &p, int64_t r, int64_t c, float v[16], StatsAcc &st, bool acc_done = false) {
    static_assert(EPI != EPI_PARTIAL, "see emit_partial4");
    if constexpr (EPI == EPI_RNE) {
        // the host sends only row lengths that are multiples of 16 here
        uint32_t pk[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float y[4] = {v[4 * q] * p.ep.alpha, v[4 * q + 1] * p.ep.alpha,
                          v[4 * q + 2] * p.ep.alpha, v[4 * q + 3] * p.ep.alpha};
            pk[q] = e5m2_pack4<false>(y, 0u, 0u, false);
        }
        if (p.ep.mask && conv_padding_row(p.ep, r)) pk[0] = pk[1] = pk[2] = pk[3] = 0;
        u32x4 o = {pk[0], pk[1], pk[2], pk[3]};
        if constexpr (kThrough) store_through(reinterpret_cast<u32x4 *>(p.ep.out8 + r * p.cols + c), o);
        else *reinterpret_cast<u32x4 *>(p.ep.out8 + r * p.cols + c) = o;
    } else {
        finish16<kAlways, kThrough>(p.ep, r, c, v, st, acc_done);
    }
}

// Wait until at most n vector-memory operations of this wave are outstanding and all of its
// LDS operations have completed (gfx9 encoding: vmcnt in bits 3:0 and 15:14, lgkmcnt in
// bits 11:8, expcnt left at "no wait").
template <int n>
__device__ __forceinline__ void wait_vm_lds() {
    static_assert(n >= 0 && n < 64, "vmcnt is a 6-bit counter");
    __builtin_amdgcn_s_waitcnt((n & 0xF) | ((n >> 4) << 14) | (0x7 << 4) | (0x0 << 8));
}

// One direct-to-LDS load: 64 lanes x 16 bytes land at LDS byte address lds_addr + lane * 16
// (lds_addr is wave-uniform and travels in M0).  Written as inline assembly on purpose: the
// compiler then neither knows nor tracks that this is a load into LDS, and would otherwise
// put a wait for ALL outstanding loads in front of every later LDS read, which serialises
// the prefetch ring.  Completion is tracked by hand with the vector-memory counter.
__device__ __forceinline__ void dma16(const uint8_t *gbase, uint32_t lane_off, uint32_t lds_addr) {
    // global address = wave-uniform base (SGPR pair) + per-lane 32-bit offset
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :
                 : "v"(lane_off), "s"(gbase), "s"(lds_addr)
                 : "memory", "m0");
}

// The same for the incomplete stage of a contraction: a lane whose sixteen bytes lie beyond it
// fetches zero codes instead, from an array that exists for this, so that every address is valid.
static __device__ const uint8_t kZeroCodes[16] __attribute__((aligned(16))) = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
__device__ __forceinline__ void dma16_or_zero(const uint8_t *gbase, uint32_t lane_off, bool inside, uint32_t lds_addr) {
    const uint8_t *src = inside ? gbase + lane_off : kZeroCodes;
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
                 :
                 : "v"(src), "s"(lds_addr)
                 : "memory", "m0");
}

// ---------------------------------------------------------------------------------------
// Matrix products.  A fragment holds 32 codes per lane: contraction indices 32h .. 32h+31 of one row, h = lane / 32.
// ---------------------------------------------------------------------------------------
// Eight 8-bit codes as eight halves: the (1,5,2) format is the upper byte of an IEEE half, so the
// conversion is exact for every code (subnormals, Inf and NaN among them) and costs four byte permutes.
using half8 = _Float16 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ half8 halves_of(int lo, int hi) {
    const u32x4 w = {__builtin_amdgcn_perm(0u, (uint32_t)lo, 0x010C000Cu), __builtin_amdgcn_perm(0u, (uint32_t)lo, 0x030C020Cu),
                     __builtin_amdgcn_perm(0u, (uint32_t)hi, 0x010C000Cu), __builtin_amdgcn_perm(0u, (uint32_t)hi, 0x030C020Cu)};
    return __builtin_bit_cast(half8, w);
}

// acc += x . y over 64 contraction indices.  The 8-bit instruction cuts every product 13 bits below the largest of its
// group of eight.  HALF: four half-precision ones of sixteen indices (8t .. 8t+7 of both half waves) at half the
// rate, which keep 24 bits: at least as precise as FP32 multiply-adds, which is what every shape outside the 8-bit
// kernels' gets.  Error against 64 bits, rms over the rms of the sums, beside a chain of FP32 fused
// multiply-adds in contraction order: N(0,1) codes, 6007 long, 8-bit 9e-6, half 4.7e-8, chain 6.6e-8; ReLU x uniform, 2047
// long, 5e-6, 1.5e-8, 1.7e-8; uniform over the finite codes, 2047 long, 2.4e-5, 1.4e-7, 3.5e-7.
template <bool HALF>
__device__ __forceinline__ f32x16 mma64(i32x8 x, i32x8 y, f32x16 acc) {
    if constexpr (HALF) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
            acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(halves_of(x[2 * t], x[2 * t + 1]), halves_of(y[2 * t], y[2 * t + 1]), acc, 0, 0, 0);
        return acc;
    } else {
        // cbsz = blgp = 1 selects the (1,5,2) format for both operands; the scale operands are zero, i.e. the
        // unscaled instruction
        return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(x, y, acc, 1, 1, 0, 0, 0, 0);
    }
}

// The same for every pair of MI row and NJ column fragments: the half-precision form converts each of them once
// (4 % faster on 4091 x 287 x 1088 contraction-major than pair by pair).
template <bool HALF, int MI, int NJ>
__device__ __forceinline__ void mma64_tiles(const i32x8 (&x)[NJ], const i32x8 (&y)[MI], f32x16 (&acc)[MI][NJ]) {
    if constexpr (HALF) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            half8 xh[NJ], yh[MI];
#pragma unroll
            for (int j = 0; j < NJ; ++j) xh[j] = halves_of(x[j][2 * t], x[j][2 * t + 1]);
#pragma unroll
            for (int i = 0; i < MI; ++i) yh[i] = halves_of(y[i][2 * t], y[i][2 * t + 1]);
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(xh[j], yh[i], acc[i][j], 0, 0, 0);
        }
    } else {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j) acc[i][j] = mma64<false>(x[j], y[i], acc[i][j]);
    }
}

// Tell the compiler that a pointer is the same in every lane (keeps it in scalar registers).
__device__ __forceinline__ const uint8_t *uniform_ptr(const uint8_t *p) {
    const uint64_t v = (uint64_t)(uintptr_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (const uint8_t *)(uintptr_t)(((uint64_t)hi << 32) | lo);
}

// One MFMA operand of half stage `sub` from a 64-row slab: lane l supplies tile row 32 f + l%32 (f = 0,
// 1) and contraction indices 64*sub + 32*(l/32) .. +31 -- two 16-byte reads of a row-major slab (64
// rows of 128 bytes), four transposing reads of eight contraction indices each of a
// contraction-major one (128 contraction rows of 64 bytes); swizzles as in the general kernel.
template <bool TN>
__device__ __forceinline__ i32x8 slab64_fragment(const uint8_t *slab, int sub, int f, int lane) {
    const int frow = lane & 31, fkb = lane >> 5, t16 = lane & 15;
    if constexpr (TN) {
        const int mc = (f * 32 + (frow & 16)) >> 4;
        i32x2 part[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int k = 64 * sub + 32 * fkb + 8 * e + (t16 >> 1);
            const int off = k * 64 + ((mc ^ (((k >> 2) & 1) << 1)) << 4) + 8 * (t16 & 1);
            part[e] = __builtin_amdgcn_ds_read_tr8_b64_v2i32((__attribute__((address_space(3))) i32x2 *)(slab + off));
        }
        return i32x8{part[0].x, part[0].y, part[1].x, part[1].y, part[2].x, part[2].y, part[3].x, part[3].y};
    } else {
        const int row = f * 32 + frow;
        const uint8_t *rp = slab + row * BK;
        const int sw = (row >> 1) & 7;
        const i32x4 h0 = *reinterpret_cast<const i32x4 *>(rp + (((4 * sub + 2 * fkb) ^ sw) << 4));
        const i32x4 h1 = *reinterpret_cast<const i32x4 *>(rp + (((4 * sub + 2 * fkb + 1) ^ sw) << 4));
        return __builtin_shufflevector(h0, h1, 0, 1, 2, 3, 4, 5, 6, 7);
    }
}

__device__ __forceinline__ uint32_t lds_address(const void *p) {
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) uint8_t *)p;
}

}  // namespace mp8
