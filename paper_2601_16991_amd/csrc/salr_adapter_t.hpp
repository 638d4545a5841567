// T = X * A_cat (Sec. 3.2, first concatenated GEMM) for the large-batch paths: one workgroup's work.
#pragma once

#include "salr_device.hpp"
#include "salr_internal.hpp"
#include "salr_linear_common.hpp"

namespace salr {

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));   // (kept in registers; HIP's uint4 in an array is not)
typedef short i16x4 __attribute__((ext_vector_type(4)));

// Four rows of a column from a row-major bf16 tile in LDS (gfx950's transposing read): every 16 lanes read four rows of 16
// elements, lane i the quarter i % 4 of row i / 4 at `p`, and lane i receives column i of those rows.
__device__ __forceinline__ uint2 lds_read_tr4(const uint16_t* p) {
    return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                         (__attribute__((address_space(3))) i16x4*)(uintptr_t)(__attribute__((address_space(3))) const void*)p));
}

constexpr int kTaPitch = 40;   // bf16 per row of an A tile [32 k][32 ranks]: 80 bytes, 16-byte aligned, rows spread over the banks
constexpr int kTxPitch = 72;   // bf16 per row of an X tile [rows][64 k]: 144 bytes, the 16 rows of an operand on different banks

// How the small factor lies: kFactorVec, [K, R] with R % 8 == 0 (rows of whole 16-byte vectors); kFactorAny, [K, R] with any R
// (element loads); kFactorRanks, [R, K] (B_cat in the backward pass).
enum FactorLayout { kFactorVec, kFactorAny, kFactorRanks };

// T's sum over K is cut into so many interleaved slices, every sixteenth step of 64 columns each, whatever the number of waves that
// share them: the slices are fp32 sums of their own, added up in order, so a call's T has the same bits in every launch that
// computes it.  (Four slices on the four waves of a decode launch moved dA and dB of 2048 x 4096 x 4096 by 1.6e-4.)
// A wave of fewer than sixteen takes several slices.  With 16 rows it keeps their sums side by side, its steps in the order of the columns;
// with 32 rows, whose four sums would take the registers of two more workgroups on a CU, it finishes one slice after the other.
constexpr int kAdapterSlices = 16;
constexpr bool adapter_t_one_by_one(int kMT, int kWaves) { return kMT > 1 && kWaves < kAdapterSlices; }

template <int kMT, int kWaves, FactorLayout kFactor = kFactorVec>
constexpr int adapter_t_lds_bytes() {
    constexpr int factor = kFactor == kFactorRanks ? 32 * kTxPitch : 32 * kTaPitch;
    constexpr int tiles = kWaves * (factor + 16 * kMT * kTxPitch) * 2, sums = kWaves * kMT * 2 * 256 * 4;
    return tiles > sums ? tiles : sums;
}

// Rows 16 kMT rb .. of T, ranks 32 rg .. 32 rg + 31 (columns past R as zeros), bf16 [M, Rpad].  The waves split K among
// themselves, kAdapterSlices / kWaves slices each, which are summed through LDS, so that the result needs no partial sums in
// memory and no second launch.  X is fetched as whole 128-byte lines (16 rows x 64 bytes per request, the MFMA operand as it
// is, asks the L2 twice for every line, and with rows a multiple of 4 KB apart all from one channel) and turned into operands
// through LDS; A_cat's rows go there as they lie and come back transposed.  kDepth steps in flight per wave.
// A factor laid out as [R, K] is fetched and turned into operands as X is.  t_t (unless null) receives T transposed, [Rpad, M].
// `lds`: adapter_t_lds_bytes<kMT, kWaves, kFactor>().
template <int kMT, int kWaves, int kDepth, FactorLayout kFactor = kFactorVec>
__device__ __forceinline__ void adapter_t_block(const uint16_t* __restrict__ x, int64_t M, int64_t K, const uint16_t* __restrict__ a_cat,
                                                int R, int Rpad, uint16_t* __restrict__ t, int64_t rb, int rg, uint16_t* lds,
                                                uint16_t* __restrict__ t_t = nullptr) {
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i16 = lane & 15, g = lane >> 4;
    const int64_t steps = (K + 63) >> 6;
    const int64_t m0 = rb * 16 * kMT;
    constexpr int kFactorElems = kFactor == kFactorRanks ? 32 * kTxPitch : 32 * kTaPitch;
    uint16_t* a_tile = lds + wave * (kFactorElems + 16 * kMT * kTxPitch);
    uint16_t* x_tile = a_tile + kFactorElems;
    // X loader: lane l fetches segment l % 8 (16 bytes) of row l / 8 of every eight rows
    const int xseg = lane & 7;
    const uint16_t* xrow[2 * kMT];
#pragma unroll
    for (int i = 0; i < 2 * kMT; ++i) {
        const int64_t m = m0 + 8 * i + (lane >> 3);
        xrow[i] = x + (m < M ? m : M - 1) * K + 8 * xseg;
    }
    // A loader: lane l fetches eight ranks from 32 rg + 8 (l % 4) of row l / 4 of every sixteen
    const int arow = lane >> 2, acol = 32 * rg + 8 * (lane & 3);
    auto load_a = [&](int64_t k) -> u32x4_t {
        if constexpr (kFactor == kFactorVec) {
            return *reinterpret_cast<const u32x4_t*>(a_cat + k * R + (acol < R ? acol : R - 8));
        } else {   // ranks past R: any value, their columns are stored as zeros
            uint32_t e[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) e[j] = a_cat[k * R + (acol + j < R ? acol + j : R - 1)];
            return u32x4_t{e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16)};
        }
    };
    const uint16_t* frow[4];   // kFactorRanks: loaded like X, ranks past R as the last one
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = 32 * rg + 8 * i + (lane >> 3);
        frow[i] = a_cat + (int64_t)(r < R ? r : R - 1) * K + 8 * xseg;
    }
    constexpr int kOwn = kAdapterSlices / kWaves;   // slices of a wave: wave, wave + kWaves, ..
    static_assert(kOwn * kWaves == kAdapterSlices, "whole slices to a wave");
    constexpr bool kOneByOne = adapter_t_one_by_one(kMT, kWaves);
    constexpr int kHeld = kOneByOne ? 1 : kOwn;     // sums held at a time
    f32x4 acc[kHeld][kMT][2];
    auto clear = [&]() {
#pragma unroll
        for (int o = 0; o < kHeld; ++o)
#pragma unroll
            for (int i = 0; i < kMT; ++i) acc[o][i][0] = acc[o][i][1] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    clear();
    u32x4_t xq[kDepth][2 * kMT], aq[kDepth][4];
    auto request = [&](int d, int64_t s) {
        const int64_t k = (s < steps ? s : steps - 1) << 6;   // past the end: the last step again, not used
        const int64_t half = k + 64 > K ? 32 : 0;             // the last step has 32 columns when K % 64 is 32: its first half twice
#pragma unroll
        for (int i = 0; i < 2 * kMT; ++i) xq[d][i] = *reinterpret_cast<const u32x4_t*>(xrow[i] + k - (xseg >= 4 ? half : 0));
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if constexpr (kFactor == kFactorRanks) aq[d][i] = *reinterpret_cast<const u32x4_t*>(frow[i] + k - (xseg >= 4 ? half : 0));
            else aq[d][i] = load_a(k + arow + 16 * i - (i >= 2 ? half : 0));
        }
    };
    auto multiply = [&](int o, int d, int64_t s) {
#pragma unroll
        for (int i = 0; i < 2 * kMT; ++i) *reinterpret_cast<u32x4_t*>(x_tile + (8 * i + (lane >> 3)) * kTxPitch + 8 * xseg) = xq[d][i];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if constexpr (kFactor == kFactorRanks) *reinterpret_cast<u32x4_t*>(a_tile + (8 * i + (lane >> 3)) * kTxPitch + 8 * xseg) = aq[d][i];
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {   // 32 columns each
            if (h == 0 || (s << 6) + 32 < K) {   // wave-uniform
                if constexpr (kFactor != kFactorRanks) {
                    *reinterpret_cast<u32x4_t*>(a_tile + arow * kTaPitch + 8 * (lane & 3)) = aq[d][2 * h];
                    *reinterpret_cast<u32x4_t*>(a_tile + (arow + 16) * kTaPitch + 8 * (lane & 3)) = aq[d][2 * h + 1];
                }
                __builtin_amdgcn_wave_barrier();   // LDS executes a wave's accesses in order
                const uint16_t* col = a_tile + (8 * g + (i16 >> 2)) * kTaPitch + 4 * (i16 & 3);
                bf16x8 xf[kMT];
#pragma unroll
                for (int i = 0; i < kMT; ++i)
                    xf[i] = *reinterpret_cast<const bf16x8*>(x_tile + (16 * i + i16) * kTxPitch + 32 * h + 8 * g);
#pragma unroll
                for (int rt = 0; rt < 2; ++rt) {
                    uint4 bq;
                    if constexpr (kFactor == kFactorRanks) {
                        bq = *reinterpret_cast<const uint4*>(a_tile + (16 * rt + i16) * kTxPitch + 32 * h + 8 * g);
                    } else {
                        const uint2 lo = lds_read_tr4(col + 16 * rt), hi = lds_read_tr4(col + 4 * kTaPitch + 16 * rt);
                        bq = make_uint4(lo.x, lo.y, hi.x, hi.y);
                    }
                    const bf16x8 b = as_bf16x8(bq);
#pragma unroll
                    for (int i = 0; i < kMT; ++i) acc[o][i][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf[i], b, acc[o][i][rt], 0, 0, 0);
                }
                __builtin_amdgcn_wave_barrier();
            }
        }
    };
    // Accumulator layout: lane holds T[16 i + 4 g + e][16 rt + i16].  A slice of each wave at a time goes through LDS, which the tiles leave
    // to them, and they are added in order.
    float* red = reinterpret_cast<float*>(lds);
    constexpr int kSums = kMT * 512 / (64 * kWaves) > 0 ? kMT * 512 / (64 * kWaves) : 1;   // of a thread
    float sum[kSums];
#pragma unroll
    for (int j = 0; j < kSums; ++j) sum[j] = 0.f;
    auto add_up = [&](int o) {
        __syncthreads();   // the tiles, or the slices before, have been read
#pragma unroll
        for (int i = 0; i < kMT; ++i)
#pragma unroll
            for (int rt = 0; rt < 2; ++rt)
#pragma unroll
                for (int e = 0; e < 4; ++e) red[(wave * kMT * 2 + i * 2 + rt) * 256 + e * 64 + lane] = acc[o][i][rt][e];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kSums; ++j) {
            const int idx = tid + 64 * kWaves * j;
            if (idx < kMT * 512)
#pragma unroll
                for (int w = 0; w < kWaves; ++w) sum[j] += red[w * kMT * 512 + idx];
        }
    };
    if constexpr (kOneByOne) {   // a ring over the steps of all the wave's slices, in the order of the slices
        static_assert(kFactor != kFactorAny);
        int asked = 0;                      // slice and step of the next request; past the last: steps
        int64_t ask = wave;
        auto advance = [&]() {
            ask += kAdapterSlices;
            if (ask >= steps) {             // wave-uniform
                ++asked;
                ask = asked < kOwn ? wave + kWaves * asked : steps;   // (a slice without steps: so are the ones behind it)
            }
        };
#pragma unroll
        for (int d = 0; d < kDepth; ++d) {
            request(d, ask);
            advance();
        }
        int turn = 0;
#pragma unroll 1
        for (int o = 0; o < kOwn; ++o) {
#pragma unroll 1
            for (int64_t s = wave + kWaves * o; s < steps; s += kAdapterSlices) {
#pragma unroll
                for (int d = 0; d < kDepth; ++d)
                    if (turn == d) {        // wave-uniform
                        multiply(0, d, s);
                        request(d, ask);
                    }
                advance();
                turn = turn + 1 == kDepth ? 0 : turn + 1;
            }
            add_up(0);
            clear();
            __syncthreads();   // the sums have been read
        }
    } else {
        constexpr int kRound = kDepth > kOwn ? kDepth : kOwn;   // steps after which slice and registers are the same again
        static_assert(kRound % kDepth == 0 && kRound % kOwn == 0, "a round is whole turns of both");
        if constexpr (kFactor == kFactorAny) {   // element loads are packed, and so waited for, where they are asked for: kDepth steps at once
            for (int64_t s0 = wave; s0 < steps; s0 += kWaves * kRound) {
#pragma unroll
                for (int j = 0; j < kRound; j += kDepth) {
#pragma unroll
                    for (int d = 0; d < kDepth; ++d) request(d, s0 + kWaves * (j + d));
#pragma unroll
                    for (int d = 0; d < kDepth; ++d)
                        if (s0 + kWaves * (j + d) < steps) multiply((j + d) % kOwn, d, s0 + kWaves * (j + d));   // wave-uniform
                }
            }
        } else {   // a ring: a step is requested again as soon as its registers are free, kDepth steps ahead
#pragma unroll
            for (int d = 0; d < kDepth; ++d) request(d, wave + kWaves * d);
            for (int64_t s0 = wave; s0 < steps; s0 += kWaves * kRound) {
#pragma unroll
                for (int j = 0; j < kRound; ++j) {
                    const int64_t s = s0 + kWaves * j;
                    if (s < steps) multiply(j % kOwn, j % kDepth, s);   // wave-uniform
                    request(j % kDepth, s + kWaves * kDepth);
                }
            }
        }
#pragma unroll
        for (int o = 0; o < kOwn; ++o) add_up(o);
    }
#pragma unroll
    for (int j = 0; j < kSums; ++j) {
        const int idx = tid + 64 * kWaves * j;
        const int l = idx & 63, e = (idx >> 6) & 3, rt = (idx >> 8) & 1, i = idx >> 9;
        const int64_t m = m0 + 16 * i + 4 * (l >> 4) + e;
        const int r = 32 * rg + 16 * rt + (l & 15);
        if (idx < kMT * 512 && m < M) {
            const uint16_t v = r < R ? f32_to_bf16_rne(sum[j]) : (uint16_t)0;
            t[m * Rpad + r] = v;
            if (t_t != nullptr) t_t[(int64_t)r * M + m] = v;
        }
    }
}

// Workgroup `block` of T = X * A_cat (R % 8 == 0) beside a pass over the weight, by workgroups of kWaves waves: 16 rows of X and 32 ranks
// each, or 32 rows where kWide, there are kAdapterWideM and more, and blocks of 16 rows would be more than one a CU.  (16 / 32 rows, us a
// call: 256 blocks 1024 x 8192 x 1024 rank 128 52.4 / 55.2, 4096 x 4096 x 512 rank 32 41.6 / 45.9; 512 blocks 2048 x 4096 x 512 rank 128
// 40.9 / 39.4, 1024 x 8192 x 1024 rank 256 64.2 / 58.9; 1024 blocks 4096 x 8192 x 512 rank 128 104 / 89.)
template <bool kWide>
__host__ __device__ inline bool adapter_t_wide(int64_t M, int Rpad) {
    return kWide && M >= kAdapterWideM && (M + 15) / 16 * (Rpad >> 5) > 256;
}
template <bool kWide>
inline int adapter_t_blocks(int64_t M, int Rpad) {
    const int rows = adapter_t_wide<kWide>(M, Rpad) ? 32 : 16;
    return (int)((M + rows - 1) / rows) * (Rpad / 32);
}
template <int kWaves, bool kWide>
__device__ __forceinline__ void adapter_t_block_of(const uint16_t* __restrict__ x, int64_t M, int64_t K, const uint16_t* __restrict__ a_cat, int R,
                                                   int Rpad, uint16_t* __restrict__ t, int block, uint16_t* lds) {
    const int groups = Rpad >> 5;
    if (adapter_t_wide<kWide>(M, Rpad)) adapter_t_block<2, kWaves, 2>(x, M, K, a_cat, R, Rpad, t, block / groups, block % groups, lds);
    else adapter_t_block<1, kWaves, 2>(x, M, K, a_cat, R, Rpad, t, block / groups, block % groups, lds);
}

}  // namespace salr
