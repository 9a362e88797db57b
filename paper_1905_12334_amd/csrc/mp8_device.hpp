// Device-side building blocks shared by the mp8 kernels: bit-level conversions to the
// 8-bit (1,5,2) and half (1,5,10) formats with round-to-nearest-even or stochastic
// rounding (Section 3.2 of arXiv 1905.12334), the Philox4x32-10 stream used for the
// random bits, and wave-level reductions for the overflow / amax statistics that drive
// loss scaling (Section 3.1).  gfx950 only.
#pragma once

#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/mp8.h"

namespace mp8 {

constexpr int kWave = 64;

using f32x4 = float __attribute__((ext_vector_type(4)));
using u32x4 = uint32_t __attribute__((ext_vector_type(4)));
using u32x2 = uint32_t __attribute__((ext_vector_type(2)));
using half2v = _Float16 __attribute__((ext_vector_type(2)));

// Stores of a kernel's results that go through the L2 to memory as they are made (agent scope).  Eight XCDs have an L2 each;
// lines that are still dirty when a kernel ends are written back then, before the next kernel starts, which most of the time
// reads them from another XCD.  Storing only (back to back, 256 to 2048 workgroups), plain / through, us: 64 KB 2.19 / 2.02 (an empty
// kernel 2.05), 1 MB 2.29 / 2.02, 4 MB 2.60 / 2.18, 8 MB 3.23 / 2.64, 16 MB 4.89 / 3.64, 32 MB 7.1 / 5.7; with a kernel that reads them
// on another XCD 1 MB 4.16 / 3.68, 4 MB 5.74 / 5.43, 8 MB 8.30 / 7.79, 16 MB 14.6 / 13.1, 32 MB 25.7 / 26.3; as pieces of 64 bytes 4 MB 2.60 /
// 2.32.  Whole training steps: 4096 x 2048 x 512 with ADAM 51.9 -> 49.4, 16384 x 4096 x 1024 282 -> 268, 32 x 56 x 56 x 64
// convolution 45.7 -> 43.9.  It does not pay, and plain or non-temporal stores are kept, where a store of a wave covers no more
// than 32 or 64 bytes of a line that other waves complete later (the complete epilogues of 64x64 tiles on small grids, see
// Epilogue.codes_plain, and the codes that the forward GEMM writes while it reads); where the next kernel adds to what the L2s still
// hold (acc_lines); for the Q node's codes of 3.7 to 6.8 M (see launch_quantize); and for the optimizer's own streams (61 M weights with ADAM
// 212 us, 223), unlike an update in a GEMM's epilogue (see update4).
template <class T>
__device__ __forceinline__ void store_through(T *p, T v) {
    static_assert(sizeof(T) == 4 || sizeof(T) == 8 || sizeof(T) == 16, "4, 8 or 16 bytes");
    if constexpr (sizeof(T) == 16)
        __builtin_amdgcn_global_store_b128((__attribute__((address_space(1))) u32x4 *)p, __builtin_bit_cast(u32x4, v), "agent");
    else if constexpr (sizeof(T) == 8)
        __hip_atomic_store(reinterpret_cast<uint64_t *>(p), __builtin_bit_cast(uint64_t, v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else
        __hip_atomic_store(reinterpret_cast<uint32_t *>(p), __builtin_bit_cast(uint32_t, v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint32_t f2u(float f) { return __float_as_uint(f); }
__device__ __forceinline__ float u2f(uint32_t u) { return __uint_as_float(u); }

// ---------------------------------------------------------------------------------------
// Philox4x32-10.  The key schedule is wave-uniform, so it lives in scalar registers; each
// round is two 32x32->64 multiplies and two three-input xors per lane.
// ---------------------------------------------------------------------------------------
struct Words4 {  // random words of four consecutive elements: (0, 1) and (2, 3)
    uint32_t r01, r23;
};
struct Philox {
    uint32_t k0, k1, off_lo, off_hi;
    __device__ __forceinline__ Philox(uint64_t seed, uint64_t offset)
        : k0((uint32_t)seed), k1((uint32_t)(seed >> 32)), off_lo((uint32_t)offset),
          off_hi((uint32_t)(offset >> 32)) {}

    // The four output words for the group of eight elements with index / 8 == blk.
    __device__ __forceinline__ uint4 block(uint64_t blk) const {
        uint32_t c0 = (uint32_t)blk, c1 = (uint32_t)(blk >> 32), c2 = off_lo, c3 = off_hi;
        uint32_t ka = k0, kb = k1;
#pragma unroll
        for (int r = 0; r < 10; ++r) {
            uint64_t p0 = (uint64_t)0xD2511F53u * c0;
            uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
            uint32_t n0 = (uint32_t)(p1 >> 32) ^ c1 ^ ka;
            uint32_t n2 = (uint32_t)(p0 >> 32) ^ c3 ^ kb;
            c1 = (uint32_t)p1;
            c3 = (uint32_t)p0;
            c0 = n0;
            c2 = n2;
            ka += 0x9E3779B9u;
            kb += 0xBB67AE85u;
        }
        return make_uint4(c0, c1, c2, c3);
    }

    // The words of elements i .. i+3 (i % 4 == 0): half of block i / 8.
    __device__ __forceinline__ Words4 half_block(uint64_t i) const {
        const uint4 w = block(i >> 3);
        return {(i & 4) ? w.z : w.x, (i & 4) ? w.w : w.y};
    }

    // The words of elements i .. i+3 for any i.
    __device__ __forceinline__ Words4 words_at(uint64_t i) const {
        const uint4 a = block(i >> 3);
        const int h = (int)(i & 7);
        uint32_t w[6] = {a.x, a.y, a.z, a.w, 0u, 0u};
        if (h > 4) {  // they go on in the next block
            const uint4 b = block((i >> 3) + 1);
            w[4] = b.x;
            w[5] = b.y;
        }
        const uint32_t m4 = (h & 4) ? ~0u : 0u, m2 = (h & 2) ? ~0u : 0u;
#pragma unroll
        for (int j = 0; j < 4; ++j) w[j] = (w[j + 2] & m4) | (w[j] & ~m4);
#pragma unroll
        for (int j = 0; j < 3; ++j) w[j] = (w[j + 1] & m2) | (w[j] & ~m2);
        return {__builtin_amdgcn_alignbit(w[1], w[0], (h & 1) * 16), __builtin_amdgcn_alignbit(w[2], w[1], (h & 1) * 16)};
    }

    // Lanes 2m and 2m + 1 need the first and the second half of block `a`, and of block `b` (the same
    // for both lanes): the even lane computes a, the odd one b, and each hands over the other's half.
    // Every lane of the wave must be active.
    __device__ __forceinline__ void pair_words(uint64_t a, uint64_t b, Words4 &wa, Words4 &wb) const {
        const bool odd = (threadIdx.x & 1) != 0;
        const uint4 mine = block(odd ? b : a);
        // quad_perm [1,0,3,2]: the value of the other lane of the pair
        const uint32_t got0 = (uint32_t)__builtin_amdgcn_mov_dpp((int)(odd ? mine.x : mine.z), 0xB1, 0xF, 0xF, true);
        const uint32_t got1 = (uint32_t)__builtin_amdgcn_mov_dpp((int)(odd ? mine.y : mine.w), 0xB1, 0xF, 0xF, true);
        wa = {odd ? got0 : mine.x, odd ? got1 : mine.y};
        wb = {odd ? mine.z : got0, odd ? mine.w : got1};
    }
};

// Halfword h (0..7) of a Philox block: low half of word 0 first.
__device__ __forceinline__ uint32_t philox_half(const uint4 &w, int h) {
    uint32_t word = (h >> 1) == 0 ? w.x : (h >> 1) == 1 ? w.y : (h >> 1) == 2 ? w.z : w.w;
    return (h & 1) ? (word >> 16) : (word & 0xFFFFu);
}

// ---------------------------------------------------------------------------------------
// FP32 bit pattern -> 8-bit (1,5,2) code.
//   kSR = false: round to nearest even.  kSR = true: stochastic rounding on the magnitude,
//   r16 in [0, 65536): with F the top 16 bits of the discarded fraction, the magnitude code
//   is bumped by one iff F + r16 >= 65536.
//   NaN -> 0x7F (canonical).  Inf -> sign|0x7C.  Finite overflow -> sign|0x7C, or
//   sign|0x7B when `sat`.
// The magnitude code of a normal result is (a - (112 << 23)) >> 21 because the two formats
// differ only in exponent bias (127 vs 15) and mantissa width (23 vs 2).
// ---------------------------------------------------------------------------------------
template <bool kSR>
__device__ __forceinline__ uint32_t e5m2_from_f32_bits(uint32_t u, uint32_t r16, bool sat) {
    const uint32_t a = u & 0x7FFFFFFFu;
    const uint32_t sign = (u >> 24) & 0x80u;
    uint32_t mag;
    if (a >= 0x38800000u) {  // |y| >= 2^-14: normal in the 8-bit format (or overflow)
        uint32_t t = a - 0x38000000u;
        if constexpr (kSR) {
            uint32_t F = (t >> 5) & 0xFFFFu;
            mag = (t >> 21) + ((F + r16) >> 16);
        } else {
            mag = (t + 0x000FFFFFu + ((t >> 21) & 1u)) >> 21;
        }
    } else {  // subnormal result: count of 2^-16 quanta
        if constexpr (kSR) {
            // |y| = mant * 2^(e-150); in units of 2^-32 that is mant >> (118 - e), truncated
            uint32_t e = a >> 23;
            uint32_t mant = (a & 0x007FFFFFu) | (e ? 0x00800000u : 0u);
            e = e ? e : 1u;
            uint32_t sh = 118u - e;  // >= 6 here
            uint32_t v = sh < 32u ? (mant >> sh) : 0u;
            mag = (v >> 16) + (((v & 0xFFFFu) + r16) >> 16);
        } else {
            // adding 128.0f makes the FP32 adder round |y| to a multiple of ulp(128) = 2^-16
            // with its own round-to-nearest-even
            mag = f2u(u2f(a) + 128.0f) - 0x43000000u;
        }
    }
    if (a > 0x7F800000u) return 0x7Fu;
    if (a == 0x7F800000u) return sign | 0x7Cu;
    if (mag >= 0x7Cu) mag = sat ? 0x7Bu : 0x7Cu;
    return sign | mag;
}

// ---------------------------------------------------------------------------------------
// Hardware conversions.  v_cvt_pk_bf8_f32 (round to nearest even) and v_cvt_sr_bf8_f32 fed
// with r16 << 16 (it adds the top 21 bits of its random operand to the 21 discarded mantissa
// bits) produce exactly the codes of e5m2_from_f32_bits for every FP32 input that is not a
// NaN -- including ties, subnormal results and overflow to Inf; this was checked over all
// 2^32 inputs.  For a NaN input both instructions return a NaN code (0xFE for every payload and
// either sign, measured over all 2^24 NaN patterns) and leave the neighbouring bytes alone.  The
// canonical code 0x7F is put in its place afterwards on the packed word (kBranchFree: six integer
// operations per four values, no branch -- 0.1-0.3 us faster in the GEMM epilogues, whose code
// the compiler can then schedule freely), or groups that contain a NaN take the bit-level
// routine behind a test (cheaper where conversion competes with a stream of loads for issue
// slots: the forward GEMM that quantises its activations is 1.2 us slower without the branch).
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ bool any_nan4(const float y[4]) {
    return __builtin_isunordered(y[0], y[1]) | __builtin_isunordered(y[2], y[3]);
}

// Every byte of w that is a NaN code (magnitude 0x7D .. 0x7F) becomes 0x7F, sign dropped; other
// bytes stay.  No byte of m exceeds 0x7F, so the addition does not carry between bytes.
__device__ __forceinline__ uint32_t canonical_nan_codes(uint32_t w) {
    const uint32_t m = w & 0x7F7F7F7Fu;
    const uint32_t t = ((m + 0x03030303u) >> 7) & 0x01010101u;  // 1 in the bytes that hold a NaN code
    const uint32_t mask = (t << 8) - t;                          // 0xFF in those bytes (t * 255)
    return (w & ~mask) | (mask & 0x7F7F7F7Fu);
}

// Bit-level conversion of four values (groups that contain a NaN).  Out of line on
// purpose: it is rare, and keeping it out of the callers keeps their hot code small.
static inline __device__ __noinline__ uint32_t e5m2_pack4_slow(float y0, float y1, float y2, float y3,
                                                        uint32_t r01, uint32_t r23, bool sr,
                                                        bool sat) {
    const float y[4] = {y0, y1, y2, y3};
    const uint32_t r[4] = {r01 & 0xFFFFu, r01 >> 16, r23 & 0xFFFFu, r23 >> 16};
    uint32_t w = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t c = sr ? e5m2_from_f32_bits<true>(f2u(y[j]), r[j], sat)
                              : e5m2_from_f32_bits<false>(f2u(y[j]), 0u, sat);
        w |= c << (8 * j);
    }
    return w;
}


// Saturating mode on the hardware path: every finite value beyond the largest normal ends at
// +-57344 under either rounding rule (nearest-even: (57344, 61440) rounds down, the rest would
// overflow; stochastic: the bracket is [57344, 65536) and its upper end would overflow), so
// such values are replaced by +-57344 before the conversion.  Infinities stay infinities.
__device__ __forceinline__ float saturate_finite(float y) {
    const float a = __builtin_fabsf(y);
    return (a > 57344.0f && a < __builtin_inff()) ? __builtin_copysignf(57344.0f, y) : y;
}

// Four values -> four codes packed little-endian, as the instructions give them (NaN: 0xFE).  r01 / r23 hold the
// 16 random bits of elements (0: low half, 1: high half) and (2, 3); ignored for RNE.
template <bool kSR>
__device__ __forceinline__ uint32_t e5m2_pack4_raw(const float y[4], uint32_t r01, uint32_t r23, bool sat) {
    float z[4] = {y[0], y[1], y[2], y[3]};
    if (sat) {
#pragma unroll
        for (int j = 0; j < 4; ++j) z[j] = saturate_finite(z[j]);
    }
    int w = 0;
    if constexpr (kSR) {
        w = __builtin_amdgcn_cvt_sr_bf8_f32(z[0], (int)(r01 << 16), w, 0);
        w = __builtin_amdgcn_cvt_sr_bf8_f32(z[1], (int)(r01 & 0xFFFF0000u), w, 1);
        w = __builtin_amdgcn_cvt_sr_bf8_f32(z[2], (int)(r23 << 16), w, 2);
        w = __builtin_amdgcn_cvt_sr_bf8_f32(z[3], (int)(r23 & 0xFFFF0000u), w, 3);
    } else {
        w = __builtin_amdgcn_cvt_pk_bf8_f32(z[0], z[1], w, false);
        w = __builtin_amdgcn_cvt_pk_bf8_f32(z[2], z[3], w, true);
    }
    return (uint32_t)w;
}

// The same with canonical NaN codes.
template <bool kSR, bool kBranchFree = true>
__device__ __forceinline__ uint32_t e5m2_pack4(const float y[4], uint32_t r01, uint32_t r23,
                                               bool sat) {
    if constexpr (!kBranchFree) {
        if (any_nan4(y)) return e5m2_pack4_slow(y[0], y[1], y[2], y[3], r01, r23, kSR, sat);
    }
    const uint32_t w = e5m2_pack4_raw<kSR>(y, r01, r23, sat);
    if constexpr (kBranchFree) return canonical_nan_codes(w);
    return w;
}

// The same with the rounding mode chosen at run time.
template <bool kBranchFree = true>
__device__ __forceinline__ uint32_t e5m2_pack4_rt(const float y[4], uint32_t r01, uint32_t r23,
                                                  bool sr, bool sat) {
    if constexpr (!kBranchFree) {
        if (any_nan4(y)) return e5m2_pack4_slow(y[0], y[1], y[2], y[3], r01, r23, sr, sat);
    }
    float z[4] = {y[0], y[1], y[2], y[3]};
    if (sat) {
#pragma unroll
        for (int j = 0; j < 4; ++j) z[j] = saturate_finite(z[j]);
    }
    int w = 0;
    if (sr) {
        w = __builtin_amdgcn_cvt_sr_bf8_f32(z[0], (int)(r01 << 16), w, 0);
        w = __builtin_amdgcn_cvt_sr_bf8_f32(z[1], (int)(r01 & 0xFFFF0000u), w, 1);
        w = __builtin_amdgcn_cvt_sr_bf8_f32(z[2], (int)(r23 << 16), w, 2);
        w = __builtin_amdgcn_cvt_sr_bf8_f32(z[3], (int)(r23 & 0xFFFF0000u), w, 3);
    } else {
        w = __builtin_amdgcn_cvt_pk_bf8_f32(z[0], z[1], w, false);
        w = __builtin_amdgcn_cvt_pk_bf8_f32(z[2], z[3], w, true);
    }
    if constexpr (kBranchFree) return canonical_nan_codes((uint32_t)w);
    return (uint32_t)w;
}

// Exact value of an 8-bit (1,5,2) code as FP32: the code is the top byte of an IEEE half.
__device__ __forceinline__ float e5m2_to_f32(uint32_t code) {
    return __half2float(__ushort_as_half((unsigned short)(code << 8)));
}

// ---------------------------------------------------------------------------------------
// Statistics: per-thread partials, reduced across the wave with shuffles, then one atomic
// per wave and field.
// ---------------------------------------------------------------------------------------
struct StatsAcc {
    float amax = 0.0f;      // max |y| over non-NaN values
    uint32_t nan_seen = 0;  // any NaN among the values
    uint32_t nonfinite = 0, zero_codes = 0, zero_inputs = 0;
    // Of U times four values and their codes: the maximum, and a test of the values that decides whether anything is counted.
    // A code is Inf or NaN only if its value is beyond the largest normal, and a non-zero value becomes zero only below the
    // smallest subnormal; with its bits shifted left by one and one subtracted, a zero is the largest number and does
    // not look like one.  Two instructions per value and no dependence on the codes, whatever share of the values is
    // zero (behind a ReLU half of them; a test for zero codes, which was here before, met one in every wave).  With everything
    // counted without a test a Q node spent 25 instructions per four values, as many as on the rest of its work.
    // kRaw: the codes are as the conversion instructions give them, and are made canonical where there is a NaN.
    template <int U, bool kRaw>
    __device__ __forceinline__ void add(const float (*y)[4], uint32_t *packed) {
        float hi = 0.0f;
        uint32_t lo = ~0u;
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                hi = __builtin_elementwise_maximum(hi, __builtin_fabsf(y[u][j]));  // (a NaN stays)
                const uint32_t bits = (f2u(y[u][j]) << 1) - 1u;
                lo = bits < lo ? bits : lo;
            }
        amax = __builtin_fmaxf(amax, hi);  // (ignores a NaN)
        constexpr uint32_t kSmallestSubnormal = ((127u - 16u) << 24) - 1u;
        const bool flushed = lo < kSmallestSubnormal, large = !(hi <= 57344.0f);
        if (flushed | large) {
            if (flushed) {
#pragma unroll
                for (int u = 0; u < U; ++u) count_zeros(y[u], packed[u]);
            }
            if (large) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if constexpr (kRaw) packed[u] = canonical_nan_codes(packed[u]);
                    count_large(y[u], packed[u]);
                }
            }
        }
    }
    __device__ __forceinline__ void count_zeros(const float y[4], uint32_t packed) {
#pragma unroll
        for (int j = 0; j < 4; ++j) zero_inputs += (y[j] == 0.0f) ? 1u : 0u;
        zero_codes += 4u - __builtin_popcount(((packed & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) & 0x80808080u);
    }
    __device__ __forceinline__ void count_large(const float y[4], uint32_t packed) {
        nan_seen |= any_nan4(y) ? 1u : 0u;
        nonfinite += __builtin_popcount(((packed & 0x7C7C7C7Cu) + 0x04040404u) & 0x80808080u);
#pragma unroll
        for (int j = 0; j < 4; ++j) amax = __builtin_fmaxf(amax, __builtin_fabsf(y[j]));  // (ignores a NaN)
    }
    // four values before rounding and their packed (canonical) codes
    __device__ __forceinline__ void add4(const float y[4], uint32_t packed) {
        add<1, false>(reinterpret_cast<const float (*)[4]>(y), &packed);
    }
    // the same without the test, for code that gains less from it than the branches cost (finish16_ragged: 1000 x 1000 x 1000
    // stochastic, contraction-major 14.5 us with it, 13.9 without)
    __device__ __forceinline__ void add4_always(const float y[4], uint32_t packed) {
        count_zeros(y, packed);
        count_large(y, packed);
    }
    __device__ __forceinline__ void add1(float y, uint32_t code) {
        if (y != y) nan_seen = 1u;
        amax = __builtin_fmaxf(amax, __builtin_fabsf(y));
        zero_inputs += (y == 0.0f) ? 1u : 0u;
        nonfinite += ((code & 0x7Cu) == 0x7Cu) ? 1u : 0u;
        zero_codes += ((code & 0x7Fu) == 0u) ? 1u : 0u;
    }
    // The running maximum at the destination, for flush: the maximum only grows, so a block whose own does not
    // exceed a value seen there has nothing to add (an older value only makes the test more conservative).
    // To be called when the kernel starts: at its end this load would meet the other blocks' additions to the same line,
    // which then go to and fro between the caches (16384 x 1024, transposed, stochastic, 256 blocks: read at the end 31.8 us where a larger
    // maximum stands and 31.6 into a cleared slot, to which then every block adds; read early 23.2 and 23.6).
    static __device__ __forceinline__ uint32_t peek(const mp8_stats *out) {
        uint32_t seen = 0;
        if (threadIdx.x == 0) seen = __hip_atomic_load(&out->amax_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return seen;
    }
    // Reduce over the wave, then over the block's waves through LDS: one atomic per field
    // and block.  Every thread of the block must call this (it contains a barrier).
    __device__ __forceinline__ void flush(mp8_stats *out) { flush(out, peek(out)); }
    __device__ __forceinline__ void flush(mp8_stats *out, uint32_t seen) {
        __shared__ uint32_t part[3][16];
        uint32_t m = nan_seen ? 0x7FC00000u : f2u(amax);
        uint32_t nf = nonfinite, z = zero_codes - zero_inputs;
        reduce_wave(m, nf, z);
        const int wave = threadIdx.x / kWave, nwaves = (blockDim.x + kWave - 1) / kWave;
        if ((threadIdx.x & (kWave - 1)) == 0) {
            part[0][wave] = m;
            part[1][wave] = nf;
            part[2][wave] = z;
        }
        __syncthreads();
        if (wave == 0) {  // the first wave combines the (at most 16) wave results
            const int l = threadIdx.x;
            m = l < nwaves ? part[0][l] : 0u;
            nf = l < nwaves ? part[1][l] : 0u;
            z = l < nwaves ? part[2][l] : 0u;
            reduce_wave(m, nf, z);
            if (l == 0) {
                if (m > seen) atomicMax(&out->amax_bits, m);
                if (nf) atomicAdd(&out->nonfinite, nf);
                if (z) atomicAdd(&out->zeroed, z);
            }
        }
    }

    // Maximum of m and sums of nf and z over the 64 lanes, left in every lane.  Four
    // data-parallel-primitive steps combine the 16 lanes of a row (neighbour, pair, mirrored
    // half row, mirrored row); the four row results are then read as scalars.
    static __device__ __forceinline__ void reduce_wave(uint32_t &m, uint32_t &nf, uint32_t &z) {
#define MP8_DPP_STEP(ctrl)                                                                    \
    {                                                                                         \
        const uint32_t om = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, ctrl, 0xF, 0xF, true);   \
        const uint32_t onf = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)nf, ctrl, 0xF, 0xF, true); \
        const uint32_t oz = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)z, ctrl, 0xF, 0xF, true);   \
        m = om > m ? om : m;                                                                  \
        nf += onf;                                                                            \
        z += oz;                                                                              \
    }
        MP8_DPP_STEP(0xB1)   // quad_perm [1,0,3,2]
        MP8_DPP_STEP(0x4E)   // quad_perm [2,3,0,1]
        MP8_DPP_STEP(0x141)  // row_half_mirror
        MP8_DPP_STEP(0x140)  // row_mirror
#undef MP8_DPP_STEP
        uint32_t rm = 0, rnf = 0, rz = 0;
#pragma unroll
        for (int row = 0; row < 4; ++row) {
            const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)m, 16 * row);
            rm = a > rm ? a : rm;
            rnf += (uint32_t)__builtin_amdgcn_readlane((int)nf, 16 * row);
            rz += (uint32_t)__builtin_amdgcn_readlane((int)z, 16 * row);
        }
        m = rm;
        nf = rnf;
        z = rz;
    }
};

// ---------------------------------------------------------------------------------------
// The master-weight update of Figure 1b on four elements (shared by the update kernels and by the
// weight-gradient finishing pass that applies the update in place).
// ---------------------------------------------------------------------------------------
// FP32 -> half code, the same two rounding rules as for the 8-bit format, from hardware conversions.  RNE:
// v_cvt_f16_f32 for every input that is not a NaN.  SR: v_cvt_sr_f16_f32 adds the top 13 bits of its random operand
// to the 13 discarded ones, so r16 << 16 gives exactly the rule's code for every normal (or overflowing)
// result; for subnormal results it keeps fewer bits, and the integer form replaces it there: |x| in units of
// 2^-40, truncated, plus r16, over 2^16.  (A GPU test compares both with the rule over all 2^32
// inputs.)  NaN is made canonical.
// r: the element's 16 random bits in the upper half.
template <bool kSR>
__device__ __forceinline__ uint32_t f16_from_f32(float x, uint32_t r) {
    uint32_t h;
    if constexpr (kSR) {
        const half2v none = {0, 0};
        h = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_sr_f16_f32(none, x, r, false)) & 0xFFFFu;
        const float a = __builtin_fabsf(x);
        const uint32_t quanta = (uint32_t)(a * 0x1p40f);
        const uint32_t sub = ((quanta + (r >> 16)) >> 16) | ((f2u(x) >> 16) & 0x8000u);
        h = a < 0x1p-14f ? sub : h;
    } else {
        h = __half_as_ushort(__float2half_rn(x));
    }
    return (x != x) ? 0x7E00u : h;
}

__device__ __forceinline__ float half_bits_to_f32(uint32_t h) {
    return __half2float(__ushort_as_half((unsigned short)h));
}

// The 8-bit (RNE) copies of four half-precision weights: the next step's operand.
__device__ __forceinline__ uint32_t e5m2_of_halves(const uint32_t w[2]) {
    const float y[4] = {half_bits_to_f32(w[0]), half_bits_to_f32(w[0] >> 16), half_bits_to_f32(w[1]), half_bits_to_f32(w[1] >> 16)};
    return e5m2_pack4<false>(y, 0u, 0u, false);
}

// Optimizers with FP32 state in front of the same conversion.  A rule turns the un-scaled
// gradient g, the weight w and its state words into the new FP32 weight; every operation is a
// separately rounded FP32 operation in the order written (the build forbids contraction).
//
// Plain SGD: w' = w - lr * g.
struct SgdRule {
    static constexpr int kStates = 0;
    float neg_lr;
    __device__ __forceinline__ float operator()(float w, float g, float *) const { return __builtin_fmaf(neg_lr, g, w); }
};

// Momentum with the L2 regularisation gradient:   g += wd * w;  v' = mu * v + g;  w' = w - lr * v'
struct MomentumRule {
    static constexpr int kStates = 1;
    float neg_lr, mu, wd;
    __device__ __forceinline__ float operator()(float w, float g, float *st) const {
        g = __builtin_fmaf(wd, w, g);
        const float v = __builtin_fmaf(mu, st[0], g);
        st[0] = v;
        return __builtin_fmaf(neg_lr, v, w);
    }
};

// ADAM (Kingma & Ba, Algorithm 1) with the same regularisation gradient:
//   m' = b1 * m + (1 - b1) * g;  v' = b2 * v + (1 - b2) * g^2
//   w' = w - lr * (m' / c1) / (sqrt(v' / c2) + eps),   c_i = 1 - b_i^step (from the host)
// Division and square root are the correctly rounded IEEE operations (the compiler's default
// for FP32 `/` and sqrt in HIP code; the approximate intrinsics are not used).  The divisions by c_i are products with
// ric_i = 1 / c_i in double, rounded once to FP32: three instructions for some eleven, and the same result.  A quotient of two
// 24-bit numbers, c <= 1, is no midpoint of neighbouring FP32 numbers and at least 2^-49 of itself (a subnormal one 2^-25 of the
// last place) away from one, the product at most 2^-52 of itself off; infinities, NaN and signed zeros come out alike.
// (The arithmetic of ADAM is a serial tail of a GEMM's epilogue: weight gradients with update, us, 256^3 7.3 -> 6.8, 1024 x 512 x 256
// 8.6 -> 8.2, 640 x 1024 x 448 8.2 -> 7.7; two million weights alone 9.7 -> 9.0.)
struct AdamRule {
    static constexpr int kStates = 2;
    float neg_lr, b1, b2, omb1, omb2, eps, wd;
    double ric1, ric2;
    __device__ __forceinline__ float operator()(float w, float g, float *st) const {
        g = __builtin_fmaf(wd, w, g);
        const float m = __builtin_fmaf(b1, st[0], omb1 * g);
        const float v = __builtin_fmaf(b2, st[1], omb2 * (g * g));
        st[0] = m;
        st[1] = v;
        const float mhat = (float)((double)m * ric1), vhat = (float)((double)v * ric2);
        const float upd = mhat / (__builtin_sqrtf(vhat) + eps);
        return __builtin_fmaf(neg_lr, upd, w);
    }
};

// Four weights (two packed pairs of half codes) from their packed gradient codes, in place; st holds
// kStates words per element.
template <bool kSR, class Rule, int NS>
__device__ __forceinline__ void update_four(const Rule &rule, uint32_t w[2], uint32_t g8, float (&st)[4][NS], float inv_scale,
                                            Words4 r) {
    static_assert(NS >= Rule::kStates, "state words");
    const float g[4] = {__builtin_amdgcn_cvt_f32_bf8((int)g8, 0), __builtin_amdgcn_cvt_f32_bf8((int)g8, 1),
                        __builtin_amdgcn_cvt_f32_bf8((int)g8, 2), __builtin_amdgcn_cvt_f32_bf8((int)g8, 3)};
    const uint32_t rw[4] = {r.r01 << 16, r.r01 & 0xFFFF0000u, r.r23 << 16, r.r23 & 0xFFFF0000u};
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        uint32_t h[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int j = 2 * p + e;
            float wn = rule(half_bits_to_f32(w[p] >> (16 * e)), g[j] * inv_scale, st[j]);
            // The update is an FP32 operation whose FP32 result is then converted to half: keep the
            // compiler from merging the two into one mixed-precision instruction that rounds once.
            asm volatile("" : "+v"(wn));
            h[e] = f16_from_f32<kSR>(wn, rw[j]);
        }
        w[p] = h[0] | (h[1] << 16);
    }
}

// One weight from its gradient code (ragged ends); r16: its random bits.
template <bool kSR, class Rule>
__device__ __forceinline__ uint32_t update_one(const Rule &rule, uint32_t w16, uint32_t g8, float *st, float inv_scale,
                                               uint32_t r16) {
    float wn = rule(half_bits_to_f32(w16), e5m2_to_f32(g8) * inv_scale, st);
    asm volatile("" : "+v"(wn));  // as above
    return f16_from_f32<kSR>(wn, r16 << 16);
}
__device__ __forceinline__ uint32_t e5m2_of_half(uint32_t h) {
    return e5m2_from_f32_bits<false>(f2u(half_bits_to_f32(h)), 0u, false);
}

// Transpose a 4x4 byte block held as four row dwords into four column dwords
// (byte k of row j becomes byte j of column k).  v_perm_b32 picks bytes 0-3 from its second
// operand and 4-7 from its first.
__device__ __forceinline__ void transpose4x4(const uint32_t r[4], uint32_t c[4]) {
    const uint32_t t0 = __builtin_amdgcn_perm(r[1], r[0], 0x05010400u);  // r0.0 r1.0 r0.1 r1.1
    const uint32_t t1 = __builtin_amdgcn_perm(r[3], r[2], 0x05010400u);  // r2.0 r3.0 r2.1 r3.1
    const uint32_t t2 = __builtin_amdgcn_perm(r[1], r[0], 0x07030602u);  // r0.2 r1.2 r0.3 r1.3
    const uint32_t t3 = __builtin_amdgcn_perm(r[3], r[2], 0x07030602u);  // r2.2 r3.2 r2.3 r3.3
    c[0] = __builtin_amdgcn_perm(t1, t0, 0x05040100u);
    c[1] = __builtin_amdgcn_perm(t1, t0, 0x07060302u);
    c[2] = __builtin_amdgcn_perm(t3, t2, 0x05040100u);
    c[3] = __builtin_amdgcn_perm(t3, t2, 0x07060302u);
}

}  // namespace mp8
