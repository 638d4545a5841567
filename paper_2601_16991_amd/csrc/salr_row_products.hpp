// The adapter gradients of the backward pass.
#pragma once

#include "salr_adapter_t.hpp"
#include "salr_device.hpp"
#include "salr_handover.hpp"
#include "salr_internal.hpp"
#include "salr_linear_common.hpp"

namespace salr {

// Products that contract over the ROWS of a large row-major matrix (the adapter gradients of the backward pass,
// dA = X^T T' and dB^T = dY^T T, in one launch): partial[z][c][r] = sum over the rows m of slice z of in[m][c] * s_t[r][m],
// with in [M, C] bf16 and the small factor given transposed, s_t [Rpad, M].  The large matrix is read once, row-wise and
// coalesced, and transposed on the way into the MFMA operand: no transposed copy of it in memory.
//   workgroup (b, z): columns 64 b .. 64 b + 63 (wave w the 16 columns 16 w ..), row slice z (whole steps of 32 rows);
//   kTnBatch steps at a time the 256 threads copy tiles [32 rows x 64 columns] into one half of the LDS buffers, the requests
//   of the next batch in flight while this one is multiplied (a step is 4 KB, and what bounds the kernel is requests in
//   flight: with one step ahead 2048 rows x 4096 columns took 8.2 us, 2 TB/s); the LDS' transposing read hands lane (i, g)
//   in[8 g .. 8 g + 7][16 w + i] as the A operand of 16x16x32 bf16 MFMAs, the B operand s_t[16 rt + i][8 g ..] is a plain
//   16-byte load; kRT rank tiles per pass over the slice.  Padding columns of Rpad come out as zeros (s_t is zero there).
// M % 32 == 0, C % 8 == 0.
// kSameLaunch: the slices of a block meet at p.words (salr_handover.hpp) and the last sums them, in order, in a launch that has something else
// to do meanwhile; else a launch behind this one does.
// A product's pointers are picked from arguments that are all there, not by index, which is a second trip to memory for them.  With that trip and
// with a branch on p.words at every store, a step whose gradients are launches of their own took 0.8 to 1.0 us more: 160 x 1024 x 2048, rank 128:
// 33.3 us, 32.3 so.
constexpr int kTnPitch = 64 + 8;   // bf16 elements per tile row
constexpr int kTnBatch = 4;
constexpr int kTnLdsBytes = 2 * kTnBatch * 32 * kTnPitch * 2;

// The sums over the slices of 32 matrix columns: read along the ranks, as they lie, and through LDS into out[0] [C0, R] and out[1]
// [R, C1] (read in the order of the outputs, dB's sums came one 128-byte line per value: 7.4 us a gradient on 4096 columns of
// rank 32, 16 slices).  sums: kRpCols * kRpPitch floats.
constexpr int kRpCols = 32, kRpPitch = kMaxRankPadded + 1;
static_assert(kRpCols * kRpPitch * 4 <= kTnLdsBytes);

template <bool kSameLaunch>
__device__ __forceinline__ void row_products_sum(const RowProducts& p, int job, int64_t c0, float* sums) {
    const int64_t C = job == 0 ? p.C[0] : p.C[1];
    const float* partial = p.partial + (job == 0 ? 0 : (int64_t)p.ksplit * p.C[0] * p.Rpad);
    const int cols = C - c0 < kRpCols ? (int)(C - c0) : kRpCols;
    const int Rpad = p.Rpad, ksplit = p.ksplit, R = p.R, quads = Rpad >> 2;
    for (int i = threadIdx.x; i < cols * quads; i += 256) {
        const float* from = partial + c0 * Rpad + 4 * i;
        f32x4 s = {0.f, 0.f, 0.f, 0.f};
        for (int z0 = 0; z0 < ksplit; z0 += 8) {
            f32x4 q[8];
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (z0 + j < ksplit) {
                    const float* at = from + (int64_t)(z0 + j) * C * Rpad;
                    if constexpr (kSameLaunch) q[j] = __builtin_bit_cast(f32x4, shared_load4(at));
                    else q[j] = *reinterpret_cast<const f32x4*>(at);
                }
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (z0 + j < ksplit) s += q[j];
        }
        float* to = sums + (i / quads) * kRpPitch + 4 * (i % quads);
        to[0] = s[0]; to[1] = s[1]; to[2] = s[2]; to[3] = s[3];
    }
    __syncthreads();
    if (job == 0) {
        for (int i = threadIdx.x; i < cols * R; i += 256) p.out[0][c0 * R + i] = f32_to_bf16_rne(sums[i / R * kRpPitch + i % R]);
    } else {
        for (int i = threadIdx.x; i < kRpCols * R; i += 256) {
            const int c = i % kRpCols, r = i / kRpCols;
            if (c < cols) p.out[1][r * C + c0 + c] = f32_to_bf16_rne(sums[c * kRpPitch + r]);
        }
    }
}

// lds: kTnLdsBytes
template <int kRT, bool kSameLaunch>
__device__ __forceinline__ void tall_tn_block(const RowProducts& p, int block, int z, uint16_t* lds) {
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i16 = lane & 15, g = lane >> 4;
    const int blocks0 = row_product_blocks(p.C[0]), job = block < blocks0 ? 0 : 1;   // the same for the whole workgroup
    const uint16_t* in = job == 0 ? p.in[0] : p.in[1];
    const uint16_t* s_t = job == 0 ? p.s_t[0] : p.s_t[1];
    const int64_t M = p.M, C = job == 0 ? p.C[0] : p.C[1];
    const int Rpad = p.Rpad, ksplit = p.ksplit;
    float* partial = p.partial + (job == 0 ? 0 : (int64_t)ksplit * p.C[0] * Rpad);
    const int64_t c0 = (int64_t)(block - (job == 0 ? 0 : blocks0)) * 64;
    uint16_t (*tile)[kTnBatch][32 * kTnPitch] = reinterpret_cast<uint16_t (*)[kTnBatch][32 * kTnPitch]>(lds);
    const int64_t steps = M >> 5;
    const int64_t s_begin = steps * z / ksplit, s_end = steps * (z + 1) / ksplit;   // never empty: ksplit <= steps
    // this thread's 16 bytes of a tile: row tid / 8, columns 8 (tid % 8) ..; past C a vector of other columns (never stored)
    const int trow = tid >> 3, tvec = tid & 7;
    const int64_t cv = c0 + 8 * tvec + 8 <= C ? c0 + 8 * tvec : C - 8;
    auto load_tile = [&](int64_t s) -> uint4 {   // past the slice: its last step again, not used
        return *reinterpret_cast<const uint4*>(in + (((s < s_end ? s : s_end - 1) << 5) + trow) * C + cv);
    };
    for (int rb = 0; rb < Rpad; rb += 16 * kRT) {
        f32x4 acc[kRT];
#pragma unroll
        for (int rt = 0; rt < kRT; ++rt) acc[rt] = f32x4{0.f, 0.f, 0.f, 0.f};
        const uint16_t* srow[kRT];
#pragma unroll
        for (int rt = 0; rt < kRT; ++rt) {
            const int r = rb + 16 * rt + i16;
            srow[rt] = s_t + (int64_t)(r < Rpad ? r : Rpad - 1) * M + 8 * g;
        }
        uint4 next[kTnBatch];
#pragma unroll
        for (int d = 0; d < kTnBatch; ++d) next[d] = load_tile(s_begin + d);
        int buf = 0;
        for (int64_t s = s_begin; s < s_end; s += kTnBatch) {
            uint4 bq[kTnBatch][kRT];
#pragma unroll
            for (int d = 0; d < kTnBatch; ++d) {
                const int64_t sc = s + d < s_end ? s + d : s_end - 1;
#pragma unroll
                for (int rt = 0; rt < kRT; ++rt) bq[d][rt] = *reinterpret_cast<const uint4*>(srow[rt] + (sc << 5));
            }
#pragma unroll
            for (int d = 0; d < kTnBatch; ++d) *reinterpret_cast<uint4*>(&tile[buf][d][trow * kTnPitch + 8 * tvec]) = next[d];
            if (s + kTnBatch < s_end) {
#pragma unroll
                for (int d = 0; d < kTnBatch; ++d) next[d] = load_tile(s + kTnBatch + d);
            }
            __syncthreads();   // the tiles are complete; the buffers written two batches ago have been read by everyone
#pragma unroll
            for (int d = 0; d < kTnBatch; ++d) {
                if (s + d < s_end) {   // the same for the whole workgroup
                    const uint16_t* col = &tile[buf][d][(8 * g + (i16 >> 2)) * kTnPitch + 16 * wave + 4 * (i16 & 3)];
                    const uint2 lo = lds_read_tr4(col), hi = lds_read_tr4(col + 4 * kTnPitch);
                    const bf16x8 aq = as_bf16x8(make_uint4(lo.x, lo.y, hi.x, hi.y));
#pragma unroll
                    for (int rt = 0; rt < kRT; ++rt) acc[rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aq, as_bf16x8(bq[d][rt]), acc[rt], 0, 0, 0);
                }
            }
            buf ^= 1;
        }
        __syncthreads();   // before the next pass writes buffer 0 again
        // accumulator layout of the 16x16 MFMA: lane holds column lane % 16 (rank), rows 4 (lane / 16) + e (matrix column)
#pragma unroll
        for (int rt = 0; rt < kRT; ++rt) {
            const int r = rb + 16 * rt + i16;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int64_t c = c0 + 16 * wave + 4 * g + e;
                if (c < C && r < Rpad) {
                    float* to = partial + ((int64_t)z * C + c) * Rpad + r;
                    if constexpr (kSameLaunch) __hip_atomic_store(to, acc[rt][e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    else *to = acc[rt][e];
                }
            }
        }
    }
    if constexpr (kSameLaunch) {
        stores_done();
        __syncthreads();   // (every wave's; the tiles have been read, too)
        int* last = reinterpret_cast<int*>(lds);
        if (tid == 0) *last = knockout(p.words + (int64_t)block * ksplit, z, ksplit, p.tag);
        __syncthreads();
        const bool mine = *last != 0;   // the same for the whole workgroup
        __syncthreads();
        if (!mine) return;
        for (int64_t c = c0; c < c0 + 64 && c < C; c += kRpCols) {
            row_products_sum<true>(p, job, c, reinterpret_cast<float*>(lds));
            __syncthreads();
        }
    }
}

}  // namespace salr
