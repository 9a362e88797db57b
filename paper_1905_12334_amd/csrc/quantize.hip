// mp8_quantize_e5m2 / mp8_sr_bits: the Q node of Figure 1a (arXiv 1905.12334, Section 3)
// as HBM-streaming kernels for gfx950.
//
// Flat kernel: a block owns a contiguous run of the tensor; its threads read it as
// wave-interleaved 16-byte loads (every load instruction of a wave covers 1 KiB of
// contiguous FP32), convert four values to one packed dword with the hardware conversion
// instructions and store dwords (256 B contiguous per wave instruction).
// Transposing kernels: a square tile; the row-major copy is written straight from registers,
// the codes also go to an LDS tile from which the threads gather 4x4 byte blocks, transpose
// them in registers and write the transposed copy in whole 128-byte lines (tiles of 128; tiles
// of 64 only for tensors so small that latency, not traffic, sets the time).
// Row and column counts that are not multiples of 4 take a variant of it with unaligned accesses.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "mp8_device.hpp"

namespace mp8 {

template <bool kF16>
__device__ __forceinline__ float load_src(const void *src, int64_t i) {
    if constexpr (kF16)
        return __half2float(reinterpret_cast<const __half *>(src)[i]);
    else
        return reinterpret_cast<const float *>(src)[i];
}

// Four consecutive source elements starting at element index i (i % 4 == 0).
template <bool kF16>
__device__ __forceinline__ void load4(const void *src, int64_t i, float v[4]) {
    if constexpr (kF16) {
        u32x2 raw = __builtin_nontemporal_load(
            reinterpret_cast<const u32x2 *>(reinterpret_cast<const __half *>(src) + i));
        const __half2 *h = reinterpret_cast<const __half2 *>(&raw);
        float2 a = __half22float2(h[0]), b = __half22float2(h[1]);
        v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y;
    } else {
        f32x4 x = __builtin_nontemporal_load(
            reinterpret_cast<const f32x4 *>(reinterpret_cast<const float *>(src) + i));
        v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
    }
}

// Scale and round four consecutive elements with their random words.
template <bool kSR, bool kStats>
__device__ __forceinline__ uint32_t round4(float v[4], float scale, bool sat, Words4 r, StatsAcc &st) {
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] *= scale;
    uint32_t pk = e5m2_pack4<kSR>(v, r.r01, r.r23, sat);
    if constexpr (kStats) st.add4(v, pk);
    return pk;
}

// The same for U groups, all of which exist.
template <int U, bool kSR, bool kStats>
__device__ __forceinline__ void round_groups(float (&v)[U][4], float scale, bool sat, const Words4 (&r)[U], StatsAcc &st, uint32_t (&pk)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[u][j] *= scale;
        if constexpr (kStats) pk[u] = e5m2_pack4_raw<kSR>(v[u], r[u].r01, r[u].r23, sat);
        else pk[u] = e5m2_pack4<kSR>(v[u], r[u].r01, r[u].r23, sat);
    }
    if constexpr (kStats) st.add<U, true>(v, pk);
}

// Random words of U groups of four elements per lane, group u starting at element index i(u)
// (a multiple of 4).  A group is half a Philox block.  With `paired`, lanes 2m and 2m + 1 hold the
// two halves of the same block for every u (all lanes of the wave are here), and each computes every
// other block for both: the generator's multiplications are what bounds a stochastic Q node (2^26
// elements 59.8 us against 51.9 us to nearest, when every lane computed every block it needs half of).
template <int U, class Index>
__device__ __forceinline__ void group_words(const Philox &rng, bool paired, Index i, Words4 w[U]) {
    if (U % 2 == 0 && paired) {
#pragma unroll
        for (int u = 0; u + 1 < U; u += 2) rng.pair_words((uint64_t)i(u) >> 3, (uint64_t)i(u + 1) >> 3, w[u], w[u + 1]);
    } else {
#pragma unroll
        for (int u = 0; u < U; ++u) w[u] = rng.half_block((uint64_t)i(u));
    }
}

template <bool kSR, bool kStats>
__device__ __forceinline__ uint32_t round1(float x, float scale, bool sat, const Philox &rng,
                                           int64_t i, StatsAcc &st) {
    float y = x * scale;
    uint32_t r16 = 0;
    if constexpr (kSR) r16 = philox_half(rng.block((uint64_t)i >> 3), (int)(i & 7));
    uint32_t c = e5m2_from_f32_bits<kSR>(f2u(y), r16, sat);
    if constexpr (kStats) st.add1(y, c);
    return c;
}

constexpr int kFlatUnroll = 4;  // 16-byte loads in flight per thread
constexpr int kStatsBlocks = 512;      // grid limit per tensor of a batch with statistics (256 threads)
// The flat variant with statistics: one workgroup of 1024 threads per CU.  Every workgroup ends with
// one to three atomics on the one mp8_stats (the maximum needs none where a larger one had been seen), which
// the memory side serialises at about 9 ns each.  512 of them: 4096 x 2048 stochastic into a cleared slot 14.2 us, 256 12.7; where a
// larger maximum stands 8.8 and 9.5.
constexpr int kFlatStatsBlocks = 256;
constexpr int64_t kFlatSmall = 256 * 1024;
constexpr int64_t kTiny = 128 * 1024, kTinyRagged = 256 * 1024;  // transposing: element by element up to here
constexpr int64_t kTileSwitch = 256;   // transposing: tiles of 128 x 128 from this many on, else of 64 x 64
// With statistics earlier, where tiles of 64 would be more workgroups than CUs; stochastic rounding, which they speed up
// more, at two per CU.  (us in tiles of 128 / of 64, where a larger maximum stands, and into a cleared slot, to which every
// workgroup adds: to nearest 512 x 1280 6.7 / 4.95 and 7.0 / 6.6, 1024 x 1024 6.8 / 5.15 and 7.4 / 7.95, 1920 x 2048 8.0 / 16.6 and 10.5 / 36;
// stochastic 1024 x 1280 8.2 / 6.0 and 9.0 / 9.2, 1280 x 1280 8.3 / 6.2 and 9.3 / 10.2.)
constexpr int64_t kTileSwitchStats = 65, kTileSwitchStatsSR = 128;
constexpr int64_t kMaxTileBlocks = 1 << 21;  // a launch has fewer than 2^32 threads; tiles beyond it by striding
constexpr int kStatsThreads = 1024;

// How the groups of four elements of a tensor are dealt to the workgroups: a contiguous run of `chunk` groups (a
// multiple of 64) for each.  Equal runs: with the grid limit of the stats variants, whole passes alone leave
// some workgroups a third pass where others have two (9.1 M elements: 15.1 us, in runs 10.6).  Tensors of more than
// a whole pass for every workgroup deal those out in turn first -- `rounds` of `round` groups, so that the
// workgroups read side by side -- and split the rest into runs (33.6 M elements: 34.2 us in long runs, 31.4).
struct FlatSplit {
    int64_t chunk;
    int64_t rounds, round, rest;  // rest: the first group behind the rounds
};

// The flat loop of one tensor for workgroup `block` (NT threads each).  In a whole pass all loads of a thread
// are in flight before the first is used, without guards; the end of a run takes two groups per thread, then
// one at a time (guarded), or, stochastic, what is left at once: with its random words a second pass takes longer than
// one of two groups, whose lanes share the generator's blocks (us, one at a time / at once: 0.6 M elements 2.56 / 2.23, 1 M 2.73 / 2.35; with statistics
// 0.6 M 3.17 / 2.91, 1.9 M 4.93 / 3.91, 6.2 M 8.39 / 7.28; half-precision sources below 0.2 M 1.92 / 1.95, with statistics
// 2.13 / 2.20; to nearest the other way round, 3.5 M with statistics 4.16 / 4.30).
template <bool kF16, bool kSR, bool kStats, int NT, bool kRounds = false, bool kPlain = false>
__device__ __forceinline__ void flat_body(const void *__restrict__ src, uint8_t *__restrict__ dst,
                                          int64_t n, float scale, int sat, uint64_t seed,
                                          uint64_t offset, mp8_stats *stats, int64_t block,
                                          const FlatSplit &split) {
    const Philox rng(seed, offset);
    StatsAcc st;
    uint32_t seen = 0;
    if constexpr (kStats) seen = StatsAcc::peek(stats);
    const int64_t n4 = n >> 2;  // groups of four elements
    uint32_t *dst4 = reinterpret_cast<uint32_t *>(dst);
    int64_t at = 0, end = 0;
    auto pass = [&](auto unroll, auto guard) {
        constexpr int U = decltype(unroll)::value;
        const int64_t base = at + threadIdx.x;
        float v[U][4];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t g = base + u * NT;
            if (!decltype(guard)::value || g < end) load4<kF16>(src, g * 4, v[u]);
        }
        Words4 w[U] = {};
        if constexpr (kSR) group_words<U>(rng, true, [&](int u) { return (base + u * NT) * 4; }, w);
        uint32_t pk[U];
        if constexpr (!decltype(guard)::value) round_groups<U, kSR, kStats>(v, scale, sat != 0, w, st, pk);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t g = base + u * NT;
            if (!decltype(guard)::value || g < end) {
                if constexpr (decltype(guard)::value) pk[u] = round4<kSR, kStats>(v[u], scale, sat != 0, w[u], st);
                // not a non-temporal store: the codes are what the next kernel (a GEMM) reads, and they are a
                // quarter of the bytes -- left in the 256 MB cache they were measured 7 % faster here and
                // 11 us per step faster for the GEMM that follows.  Past the L2, see store_through: 128 x 2048 2.25 -> 2.09 us,
                // 4096 x 2048 with statistics 6.97 -> 6.59, 16384 x 1024 12.8 -> 11.5
                if constexpr (kPlain) dst4[g] = pk[u];
                else store_through(dst4 + g, pk[u]);
            }
        }
        at += U * NT;
    };
    if constexpr (kRounds) {
        for (int64_t round = 0; round < split.rounds; ++round) {
            at = round * split.round + block * (NT * kFlatUnroll);
            pass(std::integral_constant<int, kFlatUnroll>{}, std::false_type{});
        }
    }
    at = (kRounds ? split.rest : 0) + block * split.chunk;
    end = at + split.chunk < n4 ? at + split.chunk : n4;
    while (at + kFlatUnroll * NT <= end) pass(std::integral_constant<int, kFlatUnroll>{}, std::false_type{});
    if (at + 2 * NT <= end) pass(std::integral_constant<int, 2>{}, std::false_type{});
    if constexpr (kSR) {
        if (at + NT < end) pass(std::integral_constant<int, 2>{}, std::true_type{});
        else if (at < end) pass(std::integral_constant<int, 1>{}, std::true_type{});
    } else {
        while (at < end) pass(std::integral_constant<int, 1>{}, std::true_type{});
    }
    // ragged tail (< 4 elements)
    if (block == 0 && threadIdx.x < 4) {
        const int64_t i = (n4 << 2) + threadIdx.x;
        if (i < n)
            dst[i] = (uint8_t)round1<kSR, kStats>(load_src<kF16>(src, i), scale, sat != 0, rng, i, st);
    }
    if constexpr (kStats) st.flush(stats, seen);
}

// Aligned, so that none of them (up to 15.2 KB) crosses a 64 KB page of code: where the end of one that ran between other kernels lay on
// another page than its start, whole training steps took up to 2 % longer with the same instructions (6007 x 2048 x 512 with ADAM 64.4 / 65.9 us).
template <bool kF16, bool kSR, bool kStats, int NT, bool kRounds, bool kPlain>
__global__ __launch_bounds__(NT) __attribute__((aligned(16384))) void quantize_flat_kernel(const void *__restrict__ src, uint8_t *__restrict__ dst,
                                                           int64_t n, float scale, int sat, uint64_t seed,
                                                           uint64_t offset, mp8_stats *stats, const FlatSplit split) {
    flat_body<kF16, kSR, kStats, NT, kRounds, kPlain>(src, dst, n, scale, sat, seed, offset, stats, blockIdx.x, split);
}

// Several tensors in one launch: a step that quantises activations and errors (and whatever
// else is due) pays one launch, and the short tensors' start-up and tail hide behind the long
// ones' streaming.  Workgroups [first[k], first[k+1]) belong to tensor k.
constexpr int kBatchMax = 8;
struct BatchItem {
    const void *src;
    uint8_t *dst;
    int64_t n;
    float scale;
    int f16, sr, sat;
    uint64_t seed, offset;
    mp8_stats *stats;
    FlatSplit split;
};
struct BatchArgs {
    BatchItem item[kBatchMax];
    unsigned int first[kBatchMax + 1];
    int count;
};

__global__ __launch_bounds__(256) void quantize_batch_kernel(const BatchArgs b) {
    int k = 0;
#pragma unroll
    for (int i = 1; i < kBatchMax; ++i)
        if (i < b.count && blockIdx.x >= b.first[i]) k = i;
    k = __builtin_amdgcn_readfirstlane(k);
    // a copy of the one descriptor in scalar registers (constant indices only)
    BatchItem it = b.item[0];
#pragma unroll
    for (int i = 1; i < kBatchMax; ++i)
        if (k == i) it = b.item[i];
    unsigned int lo = b.first[0];
#pragma unroll
    for (int i = 1; i < kBatchMax; ++i)
        if (k == i) lo = b.first[i];
    const int64_t block = blockIdx.x - lo;
#define MP8_B(F16, SR, ST) \
    flat_body<F16, SR, ST, 256>(it.src, it.dst, it.n, it.scale, it.sat, it.seed, it.offset, it.stats, block, it.split)
    const bool st = it.stats != nullptr;
    if (it.f16) {
        if (it.sr) { if (st) MP8_B(true, true, true); else MP8_B(true, true, false); }
        else       { if (st) MP8_B(true, false, true); else MP8_B(true, false, false); }
    } else {
        if (it.sr) { if (st) MP8_B(false, true, true); else MP8_B(false, true, false); }
        else       { if (st) MP8_B(false, false, true); else MP8_B(false, false, false); }
    }
#undef MP8_B
}

constexpr int kTile = 128;
constexpr int kPitch = kTile / 4 + 1;  // LDS row pitch in dwords

// Streaming transposing kernel for large tensors: 128x128 tiles, 256 threads, and every block
// walks over several tiles (tile = blockIdx.x + i * gridDim.x).  The sixteen 16-byte loads of
// a thread's share of the NEXT tile are issued before the block turns to the transposed
// stores of the current one, so reads, row-major stores and transposed stores overlap inside
// a block instead of running in lock-step phases across the whole chip.  Phase 1: convert,
// store the row-major copy from registers, park the codes in one of two LDS tiles (pitch 33
// dwords).  Phase 2: every thread gathers 16 rows x 4 columns, transposes 4x4 byte blocks in
// registers and writes 16-byte pieces of the transposed copy, eight lanes side by side per
// 128-byte line.  Requires cols % 4 == 0 and rows % 16 == 0.
// With statistics two such 256-thread teams, each with tiles of its own, make one workgroup: the
// workgroups end together, and their atomics on the one mp8_stats then queue up behind the last
// stores (16384 x 1024, stochastic, 256 workgroups 23.2 us, no statistics 21.4 us; 34.4 us before the running maximum
// was read early, which is most of it, and values were tested before they are counted, see StatsAcc).
template <bool kF16, bool kSR, bool kStats>
__global__ __launch_bounds__(kStats ? 512 : 256, kStats ? 1 : 2) void quantize_transpose_kernel(
    const void *__restrict__ src, uint8_t *__restrict__ dst, uint8_t *__restrict__ dst_t,
    int64_t rows, int64_t cols, float scale, int sat, uint64_t seed, uint64_t offset,
    mp8_stats *stats) {
    constexpr int TEAMS = kStats ? 2 : 1;
    __shared__ uint32_t tiles[TEAMS][2][kTile * kPitch];
    const Philox rng(seed, offset);
    StatsAcc st;
    uint32_t seen = 0;
    if constexpr (kStats) seen = StatsAcc::peek(stats);
    const int64_t tiles_c = (cols + kTile - 1) / kTile;
    const int64_t ntiles = ((rows + kTile - 1) / kTile) * tiles_c;
    const int team = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
    const int64_t teams = (int64_t)gridDim.x * TEAMS;
    const int tid = threadIdx.x & 255;
    const bool paired = (cols & 7) == 0;       // neighbouring lanes share their random blocks
    const int cq = tid & 31, tr0 = tid >> 5;   // phase 1: column group, first row (then +8)
    const int k = tid & 7, cg = tid >> 3;      // phase 2: row chunk of 16, column group
    float v[16][4];
    // Tiles that lie completely inside the tensor take code without any per-element guard:
    // with guards the compiler can no longer count outstanding loads and stores and falls
    // back to waiting for everything before each use, which serialises the stores.
    auto is_full = [&](int64_t t) {
        return (t / tiles_c + 1) * kTile <= rows && (t % tiles_c + 1) * kTile <= cols;
    };
    auto load_tile = [&](int64_t t, auto guard) {
        const int64_t r0 = (t / tiles_c) * kTile, c = (t % tiles_c) * kTile + 4 * cq;
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int64_t r = r0 + tr0 + 8 * u;
            if (!decltype(guard)::value || (r < rows && c < cols)) load4<kF16>(src, r * cols + c, v[u]);
        }
    };
    auto phase1 = [&](int64_t t, uint32_t *tile, auto guard) {
        const int64_t r0 = (t / tiles_c) * kTile, c = (t % tiles_c) * kTile + 4 * cq;
#pragma unroll
        for (int u = 0; u < 16; u += 4) {
            float (&x)[4][4] = *reinterpret_cast<float (*)[4][4]>(&v[u]);
            auto row = [&](int d) { return r0 + tr0 + 8 * (u + d); };
            Words4 w[4] = {};
            if constexpr (kSR) group_words<4>(rng, paired, [&](int d) { return row(d) * cols + c; }, w);
            uint32_t pk[4] = {0, 0, 0, 0};
            if constexpr (!decltype(guard)::value) round_groups<4, kSR, kStats>(x, scale, sat != 0, w, st, pk);
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                if (!decltype(guard)::value || (row(d) < rows && c < cols)) {
                    if constexpr (decltype(guard)::value) pk[d] = round4<kSR, kStats>(x[d], scale, sat != 0, w[d], st);
                    __builtin_nontemporal_store(pk[d], reinterpret_cast<uint32_t *>(dst + row(d) * cols + c));
                }
                tile[(tr0 + 8 * (u + d)) * kPitch + cq] = pk[d];
            }
        }
    };
    auto phase2 = [&](int64_t t, const uint32_t *tile, auto guard) {
        const int64_t r0 = (t / tiles_c) * kTile, c0 = (t % tiles_c) * kTile;
        uint32_t colw[4][4];  // [column][row block of 4]
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            uint32_t rr[4], cc[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) rr[j] = tile[(16 * k + 4 * b + j) * kPitch + cg];
            transpose4x4(rr, cc);
#pragma unroll
            for (int col = 0; col < 4; ++col) colw[col][b] = cc[col];
        }
        const int64_t orow = r0 + 16 * k;
        if (!decltype(guard)::value || orow < rows) {
#pragma unroll
            for (int col = 0; col < 4; ++col) {
                const int64_t oc = c0 + 4 * cg + col;
                if (!decltype(guard)::value || oc < cols) {
                    u32x4 o = {colw[col][0], colw[col][1], colw[col][2], colw[col][3]};
                    __builtin_nontemporal_store(o, reinterpret_cast<u32x4 *>(dst_t + oc * rows + orow));
                }
            }
        }
    };
    using Guarded = std::true_type;
    using Plain = std::false_type;
    int64_t t = (int64_t)blockIdx.x * TEAMS + team;
    if (t < ntiles) {
        if (is_full(t)) load_tile(t, Plain{}); else load_tile(t, Guarded{});
    }
    // (every team passes the barrier as often as the first one, which has the most tiles)
    int64_t lead = t - team;
    for (int buf = 0; lead < ntiles; t += teams, lead += teams, buf ^= 1) {
        uint32_t *tile = tiles[team][buf];
        const bool here = t < ntiles, full = here && is_full(t);
        if (full) phase1(t, tile, Plain{}); else if (here) phase1(t, tile, Guarded{});
        const int64_t tn = t + teams;
        if (tn < ntiles) {
            if (is_full(tn)) load_tile(tn, Plain{}); else load_tile(tn, Guarded{});
        }
        // LDS-only synchronisation (the prefetch just issued must stay in flight); one barrier
        // per tile is enough: the other LDS tile was last read before the previous barrier
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (full) phase2(t, tile, Plain{}); else if (here) phase2(t, tile, Guarded{});
    }
    if constexpr (kStats) st.flush(stats, seen);
}

// One tile per block (no tile loop): with thousands of tiles many blocks per CU are resident at
// different phases and this simple form streams best.  Same tile layout and phases as the
// kernel above.  Requires cols % 4 == 0 and rows % 16 == 0; not used with statistics (one
// atomic per field and block would be too many).
template <bool kF16, bool kSR, bool kStats>
__global__ __launch_bounds__(256) void quantize_transpose_oneshot_kernel(
    const void *__restrict__ src, uint8_t *__restrict__ dst, uint8_t *__restrict__ dst_t,
    int64_t rows, int64_t cols, float scale, int sat, uint64_t seed, uint64_t offset,
    mp8_stats *stats) {
    __shared__ uint32_t tile[kTile * kPitch];
    const Philox rng(seed, offset);
    StatsAcc st;
    uint32_t seen = 0;
    if constexpr (kStats) seen = StatsAcc::peek(stats);
    const int64_t tiles_c = (cols + kTile - 1) / kTile;
    const int64_t r0 = (int64_t)(blockIdx.x / tiles_c) * kTile;
    const int64_t c0 = (int64_t)(blockIdx.x % tiles_c) * kTile;
    // phase 1: 128 rows x 32 column groups of four; item = u * 256 + tid -> (row, group)
    const bool paired = (cols & 7) == 0;  // neighbouring lanes share their random blocks
    Words4 w[2] = {};
#pragma unroll 4
    for (int u = 0; u < 16; ++u) {
        const int item = u * 256 + threadIdx.x;
        const int tr = item >> 5, cq = item & 31;
        const int64_t r = r0 + tr, c = c0 + 4 * cq;
        if constexpr (kSR)
            if (u % 2 == 0) group_words<2>(rng, paired, [&](int d) { return (r + 8 * d) * cols + c; }, w);
        uint32_t pk = 0;
        if (r < rows && c < cols) {
            float v[4];
            const int64_t i = r * cols + c;
            load4<kF16>(src, i, v);
            pk = round4<kSR, kStats>(v, scale, sat != 0, w[u % 2], st);
            *reinterpret_cast<uint32_t *>(dst + i) = pk;
        }
        tile[tr * kPitch + cq] = pk;
    }
    __syncthreads();
    // phase 2: thread = (column group cg, row chunk k): 16 rows x 4 columns, k fastest so that
    // eight neighbouring lanes complete one 128-byte line of a transposed row
    const int k = threadIdx.x & 7, cg = threadIdx.x >> 3;
    uint32_t colw[4][4];  // [column][row block of 4]
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        uint32_t rr[4], cc[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) rr[j] = tile[(16 * k + 4 * b + j) * kPitch + cg];
        transpose4x4(rr, cc);
#pragma unroll
        for (int col = 0; col < 4; ++col) colw[col][b] = cc[col];
    }
    const int64_t orow = r0 + 16 * k;
    if (orow < rows) {
#pragma unroll
        for (int col = 0; col < 4; ++col) {
            const int64_t oc = c0 + 4 * cg + col;
            if (oc < cols) {
                u32x4 o = {colw[col][0], colw[col][1], colw[col][2], colw[col][3]};
                *reinterpret_cast<u32x4 *>(dst_t + oc * rows + orow) = o;
            }
        }
    }
    if constexpr (kStats) st.flush(stats, seen);
}

// Four consecutive elements of a row of any length and alignment: `have` (1 .. 4) of them exist.
template <bool kF16>
__device__ __forceinline__ void load4_ragged(const void *src, int64_t i, int have, float v[4]) {
    if (have == 4) {
        if constexpr (kF16) {
            __half h[4];
            __builtin_memcpy(h, reinterpret_cast<const __half *>(src) + i, 8);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = __half2float(h[e]);
        } else {
            __builtin_memcpy(v, reinterpret_cast<const float *>(src) + i, 16);
        }
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = e < have ? load_src<kF16>(src, i + e) : 1.0f;
    }
}

enum { kPlain, kPastCaches, kPastL2 };
template <int kStore>
__device__ __forceinline__ void store_dword(uint8_t *dst, uint32_t w) {
    if constexpr (kStore == kPastL2) store_through(reinterpret_cast<uint32_t *>(dst), w);
    else if constexpr (kStore == kPastCaches) __builtin_nontemporal_store(w, reinterpret_cast<uint32_t *>(dst));
    else *reinterpret_cast<uint32_t *>(dst) = w;
}

// Store the first `have` bytes of a dword at any address.
__device__ __forceinline__ void store4_ragged(uint8_t *dst, uint32_t w, int have) {
    if (have == 4) {
        __builtin_memcpy(dst, &w, 4);
    } else {
#pragma unroll
        for (int e = 0; e < 3; ++e)
            if (e < have) dst[e] = (uint8_t)(w >> (8 * e));
    }
}

// Transposing kernel, tile T x T with (T/4)^2 threads.  Phase 1: every thread converts four
// groups of four consecutive elements (a wave instruction reads whole rows of the tile), stores
// the row-major copy from registers and parks the packed codes in an LDS tile.  Phase 2: every
// thread takes one 4x4 block of bytes from LDS, transposes it in registers and stores four
// dwords of the transposed copy; T/4 neighbouring lanes complete T contiguous bytes of a
// transposed row.  Blocks stride over the tiles, which are numbered super-tile by super-tile
// (S x S tiles each, row-major inside); a thread's loads of the next tile are issued before the
// transposed stores of the current one.
//   kRaggedRows  row and column counts that are not multiples of four: any alignment, partial groups at the
//                edges; the other forms need both to be
//   kWholeLines  both are multiples of 64: whole 64-byte pieces go past the caches (2048 x 2048 6.5 us
//                against 7.5 us with plain stores), of a half-precision source past the L2 only (see store_through: 1024 x 1024
//                4.5 -> 3.6 us, 8192 x 1024 10.7 -> 7.8, 8192 x 8192 60.9 -> 58.7; of an FP32 source 512 x 512 3.5 -> 3.85)
//   kPartLines   others are put together in the caches (9844 x 924: 16.6 us against 20.5 us)
enum { kWholeLines, kPartLines, kRaggedRows };
template <int T, bool kF16, bool kSR, bool kStats, int kForm>
__global__ __launch_bounds__((T / 4) * (T / 4)) void quantize_tile_kernel(
    const void *__restrict__ src, uint8_t *__restrict__ dst, uint8_t *__restrict__ dst_t,
    int64_t rows, int64_t cols, float scale, int sat, uint64_t seed, uint64_t offset,
    mp8_stats *stats, int S) {
    constexpr int G = T / 4;       // column groups per tile row = threads per tile row
    constexpr int NT = G * G;      // threads
    constexpr int P = G + 1;       // LDS row pitch in dwords
    constexpr bool kRagged = kForm == kRaggedRows;
    constexpr int kStore = kForm != kWholeLines ? kPlain : kF16 ? kPastL2 : kPastCaches;
    __shared__ uint32_t tile[T * P];
    const Philox rng(seed, offset);
    StatsAcc st;
    uint32_t seen = 0;
    if constexpr (kStats) seen = StatsAcc::peek(stats);
    const int64_t tiles_c = (cols + T - 1) / T, tiles_r = (rows + T - 1) / T;
    const int64_t sup_c = (tiles_c + S - 1) / S, sup_r = (tiles_r + S - 1) / S;
    const int64_t ntiles = sup_c * sup_r * S * S;
    const int tid = threadIdx.x;
    const int k = tid % G, cg = tid / G;  // phase 2: rows 4k..4k+3, columns 4cg..4cg+3
    // first row and column of tile t; a super-tile at the edge also numbers tiles that do not exist
    auto origin = [&](int64_t t, int64_t &r0, int64_t &c0) {
        const int64_t sup = t / (S * S), in = t % (S * S);
        r0 = ((sup / sup_c) * S + in / S) * T;
        c0 = ((sup % sup_c) * S + in % S) * T;
        return r0 < rows && c0 < cols;
    };
    auto next = [&](int64_t t, int64_t &r0, int64_t &c0) {  // the first tile from t on that exists
        while (t < ntiles && !origin(t, r0, c0)) t += gridDim.x;
        return t;
    };
    float v[4][4];
    auto load_tile = [&](int64_t r0, int64_t c0) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int item = u * NT + tid;
            const int64_t r = r0 + item / G, c = c0 + 4 * (item % G);
            if (r < rows && c < cols) {
                if constexpr (kRagged) load4_ragged<kF16>(src, r * cols + c, cols - c < 4 ? (int)(cols - c) : 4, v[u]);
                else load4<kF16>(src, r * cols + c, v[u]);
            }
        }
    };
    int64_t r0 = 0, c0 = 0;
    int64_t t = next(blockIdx.x, r0, c0);
    if (t < ntiles) load_tile(r0, c0);
    while (t < ntiles) {
        Words4 w[4] = {};
        if constexpr (kSR) {
            auto index = [&](int u) { return (r0 + (u * NT + tid) / G) * cols + c0 + 4 * (tid % G); };
            if constexpr (kRagged) {
#pragma unroll
                for (int u = 0; u < 4; ++u) w[u] = rng.words_at((uint64_t)index(u));
            } else {
                group_words<4>(rng, (cols & 7) == 0, index, w);
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int item = u * NT + tid;
            const int tr = item / G, cq = item % G;
            const int64_t r = r0 + tr, c = c0 + 4 * cq;
            uint32_t pk = 0;
            if (r < rows && c < cols) {
                const int64_t i = r * cols + c;
                if constexpr (kRagged) {
                    const int have = cols - c < 4 ? (int)(cols - c) : 4;
                    if (have == 4) {
                        pk = round4<kSR, kStats>(v[u], scale, sat != 0, w[u], st);
                    } else {
                        pk = round4<kSR, false>(v[u], scale, sat != 0, w[u], st);
                        if constexpr (kStats) {
#pragma unroll
                            for (int e = 0; e < 3; ++e)
                                if (e < have) st.add1(v[u][e], (pk >> (8 * e)) & 0xFFu);
                        }
                    }
                    store4_ragged(dst + i, pk, have);
                } else {
                    pk = round4<kSR, kStats>(v[u], scale, sat != 0, w[u], st);
                    store_dword<kStore>(dst + i, pk);
                }
            }
            tile[tr * P + cq] = pk;
        }
        int64_t rn = 0, cn = 0;
        const int64_t tn = next(t + gridDim.x, rn, cn);
        if (tn < ntiles) load_tile(rn, cn);
        // LDS-only synchronisation: the loads just issued stay in flight
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        uint32_t rr[4], cc[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) rr[j] = tile[(4 * k + j) * P + cg];
        transpose4x4(rr, cc);
        const int64_t orow = r0 + 4 * k;
        if (orow < rows) {
#pragma unroll
            for (int col = 0; col < 4; ++col) {
                const int64_t oc = c0 + 4 * cg + col;
                if (oc < cols) {
                    uint8_t *to = dst_t + oc * rows + orow;
                    if constexpr (kRagged) store4_ragged(to, cc[col], rows - orow < 4 ? (int)(rows - orow) : 4);
                    else store_dword<kStore>(to, cc[col]);
                }
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");  // the tile is rewritten by the next iteration
        t = tn;
        r0 = rn;
        c0 = cn;
    }
    if constexpr (kStats) st.flush(stats, seen);
}

// Any shape: one element per thread and iteration.  For tensors so small that the shortest chain of
// latencies wins (1001 x 77: 2.6 us, 4.6 us in tiles).
template <bool kF16, bool kSR, bool kStats>
__global__ __launch_bounds__(256) void quantize_generic_kernel(
    const void *__restrict__ src, uint8_t *__restrict__ dst, uint8_t *__restrict__ dst_t,
    int64_t rows, int64_t cols, float scale, int sat, uint64_t seed, uint64_t offset,
    mp8_stats *stats) {
    const Philox rng(seed, offset);
    StatsAcc st;
    uint32_t seen = 0;
    if constexpr (kStats) seen = StatsAcc::peek(stats);
    const int64_t n = rows * cols;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const uint32_t c = round1<kSR, kStats>(load_src<kF16>(src, i), scale, sat != 0, rng, i, st);
        dst[i] = (uint8_t)c;
        if (dst_t != nullptr) {
            const int64_t r = i / cols;
            dst_t[(i - r * cols) * rows + r] = (uint8_t)c;
        }
    }
    if constexpr (kStats) st.flush(stats, seen);
}

__global__ __launch_bounds__(256) void sr_bits_kernel(uint16_t *out, int64_t n, uint64_t seed,
                                                      uint64_t offset) {
    const Philox rng(seed, offset);
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
        out[i] = (uint16_t)philox_half(rng.block((uint64_t)i >> 3), (int)(i & 7));
}

template <bool kF16, bool kSR, bool kStats>
static hipError_t launch_quantize(const void *src, uint8_t *dst, uint8_t *dst_t, int64_t rows,
                                  int64_t cols, float scale, int sat, uint64_t seed,
                                  uint64_t offset, mp8_stats *stats, hipStream_t s) {
    const int64_t n = rows * cols;
    if (dst_t == nullptr) {
        const int64_t n4 = n >> 2;
        // Codes that replace those a GEMM has just read: stores past the L2 clear the lines that the other XCDs still hold, and from about 4 MB on
        // that takes longer than writing dirty lines back does (Q node and forward GEMM into one buffer, us, past / into the L2: 1835 x 256
        // x 2048, 3.8 MB, 11.8 / 11.2, 2165 16.2 / 13.8, 2555 17.4 / 14.9, 3015 18.1 / 16.3, 3558, 7.3 MB, 17.2 / 17.6; 3110 x 144 x 1024, 3.2 MB, 10.0 / 9.9,
        // 3670 10.7 / 11.3, 5111 15.4 / 13.0, 9909 18.4 / 19.2; training steps 3379 x 128 x 1728 with momentum 45.7 / 41.6, 3123 x 384 x 1600 46.5 / 43.4;
        // the node alone 4.58 / 4.57 at 5.2 M).  Half-precision sources leave less to hide the write-back behind (alone 4.1 M 2.59 / 2.91, 6.4 M 3.01 / 3.81).
        // With statistics the node itself would gain from 4.2 to 8.0 M (6.0 M 6.97 / 6.39), but the GEMMs behind it lose more (training
        // steps 15390 x 512 x 128 33.9 / 35.5, 3759 x 1792 x 128 39.2 / 41.1, 100 of them 1 % longer).  Stochastic ones gain nothing.
        constexpr bool kPlain = !kF16 && !kSR && !kStats;
        const bool plain = n > (7 << 19) && n <= (13 << 19);
        auto launch = [&](auto threads, auto in_rounds, int64_t blocks, const FlatSplit &split) {
            constexpr int NT = decltype(threads)::value;
            hipLaunchKernelGGL((kPlain && plain ? quantize_flat_kernel<kF16, kSR, kStats, NT, decltype(in_rounds)::value, kPlain>
                                                : quantize_flat_kernel<kF16, kSR, kStats, NT, decltype(in_rounds)::value, false>),
                               dim3((unsigned)blocks), dim3(NT), 0, s, src, dst, n, scale, sat, seed, offset, stats, split);
        };
        auto runs = [&](auto threads, int64_t chunk) {
            launch(threads, std::false_type{}, std::max<int64_t>(1, (n4 + chunk - 1) / chunk), FlatSplit{chunk, 0, 0, 0});
        };
        if constexpr (kStats) {
            // At most one workgroup per CU, of 256 threads while a run is no longer than two groups for each.  Every
            // workgroup adds its atomics to the end of the chain, if it has anything to add: fewer and longer runs
            // would help where values are flushed to zero all over the tensor (to nearest 524288 elements: 256 runs
            // 5.7 us, 128 4.6, 64 4.1) and cost where they are not, as after loss scaling (3.2, 3.4, 3.7).
            constexpr int64_t round = (int64_t)kFlatStatsBlocks * kStatsThreads * kFlatUnroll;
            const int64_t rounds = n4 / round;
            const int64_t chunk = std::max<int64_t>(256, ((n4 - rounds * round + kFlatStatsBlocks - 1) / kFlatStatsBlocks + 63) / 64 * 64);
            if (rounds > 0) launch(std::integral_constant<int, kStatsThreads>{}, std::true_type{}, kFlatStatsBlocks,
                                   FlatSplit{chunk, rounds, round, rounds * round});
            else if (chunk <= 512) runs(std::integral_constant<int, 256>{}, chunk);
            else runs(std::integral_constant<int, kStatsThreads>{}, chunk);
        } else {
            // one pass per workgroup; tensors of less than kFlatSmall groups take one group per thread, so
            // that they occupy every CU
            const int64_t per = n4 <= kFlatSmall ? 256 : 256 * kFlatUnroll;
            runs(std::integral_constant<int, 256>{}, std::max(per, ((n4 >> 22) + 63) / 64 * 64));
        }
    } else {
        const bool ragged = ((rows | cols) & 3) != 0;
        const int64_t tr128 = (rows + 127) / 128, tc128 = (cols + 127) / 128;
        const int64_t nt = tr128 * tc128;
        const bool wide = tr128 >= 64 && tc128 >= 64;
        auto tiles = [&](auto edge, int S, int64_t limit) {
            constexpr int T = decltype(edge)::value;
            const int64_t tr = (rows + T - 1) / T, tc = (cols + T - 1) / T;
            const int64_t blocks = std::min<int64_t>(((tr + S - 1) / S) * ((tc + S - 1) / S) * S * S, limit);
            hipLaunchKernelGGL((ragged ? quantize_tile_kernel<T, kF16, kSR, kStats, kRaggedRows>
                                : ((rows | cols) & 63) == 0 ? quantize_tile_kernel<T, kF16, kSR, kStats, kWholeLines>
                                                            : quantize_tile_kernel<T, kF16, kSR, kStats, kPartLines>),
                               dim3((unsigned)blocks), dim3((T / 4) * (T / 4)), 0, s, src, dst, dst_t, rows, cols, scale, sat,
                               seed, offset, stats, S);
        };
        // Rows or columns so short that most of a tile would be padding go element by element: 10^6 x 1 5.5 us
        // (251 us in tiles of 128), 300000 x 8 10.8 us (41), 200000 x 17 14.5 us (59), 150001 x 31 19.4 us
        // (44); with statistics 13 us (241), 25 (54), 42 (73), 52 (59).  Tiles win from 16 columns on where they
        // need no guards (200000 x 16 14.3 and 14.2 us) and from 16 rows on (31 x 150001 17.7 us, 30.7).
        const bool narrow = cols < (ragged ? 32 : 16) || rows < 16;
        const bool tiny = n <= (ragged ? kTinyRagged : kTiny);
        if (narrow || tiny) {
            // (A grid that strides.  With statistics fewer workgroups: 256 x 512 in 512 of them 3.1 us, and 8.8 if each
            // counts flushed values; in 256 3.6 and 6.2, in tiles of 64 4.6 and 4.8.  Guarded tiles cost more:
            // 511 x 513 in 1024 workgroups 3.9, in tiles 5.3.)
            const int64_t limit = !kStats ? 256 * 32 : !tiny ? kStatsBlocks : ragged ? 1024 : kFlatStatsBlocks;
            hipLaunchKernelGGL((quantize_generic_kernel<kF16, kSR, kStats>), dim3((unsigned)std::min((n + 255) / 256, limit)),
                               dim3(256), 0, s, src, dst, dst_t, rows, cols, scale, sat, seed, offset, stats);
        } else if (!kStats && std::min(rows, cols) <= 64) {
            // one tile of 64 across: 100000 x 40 10.0 us (22 in tiles of 128), 100001 x 63 16.8 us (35)
            tiles(std::integral_constant<int, 64>{}, 1, kMaxTileBlocks);
        } else if (!ragged && !kStats && !wide && (rows & 15) == 0 && nt >= 6144) {
            // several rounds of blocks: plain one-tile blocks, many per CU
            hipLaunchKernelGGL((quantize_transpose_oneshot_kernel<kF16, kSR, kStats>),
                               dim3((unsigned)nt), dim3(256), 0, s, src, dst, dst_t, rows, cols,
                               scale, sat, seed, offset, stats);
        } else if (!ragged && !wide && (rows & 15) == 0 && nt >= 1024) {
            // a few tiles per CU: about two persistent teams of 256 threads per CU, the same number of
            // tiles each, prefetching across tiles
            const int64_t per = (nt + 511) / 512, teams = (nt + per - 1) / per;
            const int64_t blocks = kStats ? (teams + 1) / 2 : teams;
            hipLaunchKernelGGL((quantize_transpose_kernel<kF16, kSR, kStats>),
                               dim3((unsigned)blocks), dim3(kStats ? 512 : 256), 0, s, src, dst, dst_t, rows, cols,
                               scale, sat, seed, offset, stats);
        } else if (nt >= (!kStats ? kTileSwitch : kSR ? kTileSwitchStatsSR : kTileSwitchStats)) {
            // 1024-thread blocks, all loads of a tile in flight; for a matrix that is wide in
            // both directions, super-tiles of 4x4 keep the lines written by concurrently
            // running blocks close together in both copies.  With statistics one block per CU:
            // every block ends in atomics on one address, and blocks that end together wait
            // for each other there
            tiles(std::integral_constant<int, 128>{}, wide ? 4 : 1, kStats ? kFlatStatsBlocks : kMaxTileBlocks);
        } else {
            // few tiles: smaller ones shorten the latency chain of the single round of blocks
            tiles(std::integral_constant<int, 64>{}, 1, kMaxTileBlocks);
        }
    }
    return hipGetLastError();
}

}  // namespace mp8

extern "C" mp8_status mp8_quantize_e5m2(const void *src, int src_is_f16, uint8_t *dst,
                                        uint8_t *dst_t, int64_t rows, int64_t cols, float scale,
                                        mp8_round round, int flags, uint64_t seed,
                                        uint64_t offset, mp8_stats *stats, void *stream) {
    using namespace mp8;
    if (rows < 0 || cols < 0) return MP8_ERR_INVALID_ARG;
    if (round != MP8_RNE && round != MP8_SR) return MP8_ERR_INVALID_ARG;
    if (rows == 0 || cols == 0) return MP8_OK;
    if (!src || !dst) return MP8_ERR_INVALID_ARG;
    if (rows > (INT64_MAX / cols)) return MP8_ERR_UNSUPPORTED;
    if (dst_t && ((rows + kTile - 1) / kTile) * ((cols + kTile - 1) / kTile) > 0x7FFFFFFFLL)
        return MP8_ERR_UNSUPPORTED;
    if (((uintptr_t)src | (uintptr_t)dst | (uintptr_t)dst_t) & 15u) return MP8_ERR_ALIGNMENT;
    hipStream_t s = (hipStream_t)stream;
    const int sat = (flags & MP8_FLAG_SATURATE) ? 1 : 0;
    hipError_t e;
#define MP8_Q(F16, SR, ST) \
    e = launch_quantize<F16, SR, ST>(src, dst, dst_t, rows, cols, scale, sat, seed, offset, stats, s)
    const bool f16 = src_is_f16 != 0, sr = round == MP8_SR, st = stats != nullptr;
    if (f16) {
        if (sr) { if (st) MP8_Q(true, true, true); else MP8_Q(true, true, false); }
        else    { if (st) MP8_Q(true, false, true); else MP8_Q(true, false, false); }
    } else {
        if (sr) { if (st) MP8_Q(false, true, true); else MP8_Q(false, true, false); }
        else    { if (st) MP8_Q(false, false, true); else MP8_Q(false, false, false); }
    }
#undef MP8_Q
    return e == hipSuccess ? MP8_OK : MP8_ERR_HIP;
}

extern "C" mp8_status mp8_quantize_e5m2_batch(const mp8_quantize_item *items, int count,
                                              void *stream) {
    using namespace mp8;
    if (count < 0 || count > kBatchMax || (count > 0 && !items)) return MP8_ERR_INVALID_ARG;
    // validate everything first: on error nothing is enqueued
    for (int i = 0; i < count; ++i) {
        const mp8_quantize_item &q = items[i];
        if (q.n < 0 || (q.round != MP8_RNE && q.round != MP8_SR)) return MP8_ERR_INVALID_ARG;
        if (q.n > 0 && (!q.src || !q.dst)) return MP8_ERR_INVALID_ARG;
        if (((uintptr_t)q.src | (uintptr_t)q.dst) & 15u) return MP8_ERR_ALIGNMENT;
    }
    // Workgroups per tensor: one per 4096 elements (256 threads x 4 loads of 4 elements);
    // tensors with statistics at most kStatsBlocks, because every workgroup ends in atomics on
    // the one mp8_stats.  Tensors whose workgroups loop longest go first, so that they run
    // beside the others instead of after them.
    int order[kBatchMax];
    int64_t nblk[kBatchMax], iters[kBatchMax];
    int m = 0;
    for (int i = 0; i < count; ++i) {
        if (items[i].n == 0) continue;
        const int64_t want = ((items[i].n >> 2) + 256 * kFlatUnroll - 1) / (256 * kFlatUnroll);
        int64_t nb = std::max<int64_t>(want, 1);
        nb = std::min<int64_t>(nb, items[i].stats ? kStatsBlocks : (1 << 20));
        nblk[i] = nb;
        iters[i] = (want + nb - 1) / nb;
        order[m++] = i;
    }
    if (m == 0) return MP8_OK;
    std::stable_sort(order, order + m, [&](int x, int y) { return iters[x] > iters[y]; });
    BatchArgs args{};
    int64_t total = 0;
    for (int j = 0; j < m; ++j) {
        const mp8_quantize_item &q = items[order[j]];
        BatchItem &it = args.item[j];
        it.src = q.src;
        it.dst = q.dst;
        it.n = q.n;
        it.scale = q.scale;
        it.f16 = q.src_is_f16 != 0;
        it.sr = q.round == MP8_SR;
        it.sat = (q.flags & MP8_FLAG_SATURATE) ? 1 : 0;
        it.seed = q.seed;
        it.offset = q.offset;
        it.stats = q.stats;
        it.split.chunk = std::max<int64_t>(256, (((q.n >> 2) + nblk[order[j]] - 1) / nblk[order[j]] + 63) / 64 * 64);
        args.first[j] = (unsigned int)total;
        total += nblk[order[j]];
    }
    for (int j = m; j <= kBatchMax; ++j) args.first[j] = (unsigned int)total;
    args.count = m;
    if (total > 0x7FFFFFFFLL) return MP8_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(quantize_batch_kernel, dim3((unsigned)total), dim3(256), 0, (hipStream_t)stream, args);
    return hipGetLastError() == hipSuccess ? MP8_OK : MP8_ERR_HIP;
}

extern "C" mp8_status mp8_sr_bits(uint16_t *out, int64_t n, uint64_t seed, uint64_t offset,
                                  void *stream) {
    if (n < 0) return MP8_ERR_INVALID_ARG;
    if (n == 0) return MP8_OK;
    if (!out) return MP8_ERR_INVALID_ARG;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(mp8::sr_bits_kernel, dim3((unsigned)blocks), dim3(256), 0,
                       (hipStream_t)stream, out, n, seed, offset);
    return hipGetLastError() == hipSuccess ? MP8_OK : MP8_ERR_HIP;
}

// ---------------------------------------------------------------------------------------
// Measuring stick for the streaming kernels: a kernel that only moves bytes, in the access
// pattern of the flat quantize and update kernels (wave-interleaved 16-byte non-temporal loads,
// four in flight per thread) and with their read:write ratio.  What it reaches is what the
// memory system gives a kernel of this shape; the quantize and update kernels are held against it.
namespace mp8 {

// kReadsPerWrite = 4: 16 bytes read per 4 bytes written (the Q node's 4:1; the plain update's
// 3:2 sits between the two); 1: a plain copy (the optimizers with FP32 state, about 1:1).
template <int kReadsPerWrite>
__global__ __launch_bounds__(256) void stream_probe_kernel(const u32x4 *__restrict__ src, void *__restrict__ dst,
                                                           int64_t n16) {
    const int64_t stride = (int64_t)gridDim.x * 256 * kFlatUnroll;
    for (int64_t base = (int64_t)blockIdx.x * 256 * kFlatUnroll + threadIdx.x; base < n16; base += stride) {
        u32x4 v[kFlatUnroll];
#pragma unroll
        for (int u = 0; u < kFlatUnroll; ++u) {
            const int64_t g = base + u * 256;
            if (g < n16) v[u] = __builtin_nontemporal_load(src + g);
        }
#pragma unroll
        for (int u = 0; u < kFlatUnroll; ++u) {
            const int64_t g = base + u * 256;
            if (g < n16) {
                if constexpr (kReadsPerWrite == 4)
                    __builtin_nontemporal_store(v[u].x ^ v[u].y ^ v[u].z ^ v[u].w, reinterpret_cast<uint32_t *>(dst) + g);
                else
                    __builtin_nontemporal_store(v[u], reinterpret_cast<u32x4 *>(dst) + g);
            }
        }
    }
}

}  // namespace mp8

extern "C" mp8_status mp8_stream_probe(const void *src, void *dst, int64_t read_bytes, int reads_per_write,
                                       void *stream) {
    if (read_bytes < 0 || (reads_per_write != 1 && reads_per_write != 4)) return MP8_ERR_INVALID_ARG;
    if (read_bytes == 0) return MP8_OK;
    if (!src || !dst) return MP8_ERR_INVALID_ARG;
    if ((((uintptr_t)src | (uintptr_t)dst) & 15u) || (read_bytes & 15)) return MP8_ERR_ALIGNMENT;
    const int64_t n16 = read_bytes >> 4, per_block = 256 * mp8::kFlatUnroll;
    int64_t blocks = (n16 + per_block - 1) / per_block;
    if (blocks > (1 << 22)) blocks = 1 << 22;
    if (reads_per_write == 4)
        hipLaunchKernelGGL(mp8::stream_probe_kernel<4>, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream,
                           (const mp8::u32x4 *)src, dst, n16);
    else
        hipLaunchKernelGGL(mp8::stream_probe_kernel<1>, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream,
                           (const mp8::u32x4 *)src, dst, n16);
    return hipGetLastError() == hipSuccess ? MP8_OK : MP8_ERR_HIP;
}
