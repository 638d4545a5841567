// First adapter stage of the large-batch paths (paper Sec. 3.2): T = X * A_cat, plus the small passes around it
// (transposed copy of A_cat, fixed-order sum of split-K partials, also used by the dense stage).
#include "salr_adapter_t.hpp"
#include "salr_device.hpp"
#include "salr_internal.hpp"
#include "salr_linear_common.hpp"
#include "salr_row_products.hpp"

namespace salr {

// ---------------------------------------------------------------------------------------------------
// T = X * A_cat for the large-batch paths (Sec. 3.2, first concatenated GEMM), bf16 output [M, Rpad].
// A_cat arrives transposed and zero padded, a_t [Rpad, K] (written by the transposing pre-pass), so that
// both MFMA operands are plain 16-byte loads along k.  The product is a stream over X (it is read once, nothing
// else is large), so the grid is made wide: workgroup (b, z) = 64 kMB rows of X times slice z of K, wave w owns
// 16 kMB of the rows (each a_t operand it loads is used for kMB row blocks: at kMB = 1 the a_t requests are kRT
// times the X requests and their L2 traffic, not X, sets the pace), the four waves walk the slice in step.
// kRT rank tiles of 16 columns per pass over the slice (all of them in one pass up to rank 128); 16x16x32 bf16
// MFMAs; with more than one slice the fp32 partial results go to partial[z] and splitk_reduce_kernel adds
// them in a fixed order.  Padding columns (from `ranks` on) are stored as zeros, which their products with an infinite entry of X
// are not.  keep_fp32: the caller wants the fp32 sums
// (the subspace iteration of the residual adapter), so even a single slice goes to partial[0].
// ---------------------------------------------------------------------------------------------------
template <int kMB, int kRT, int kDepth>
__global__ __launch_bounds__(256) void adapter_t_kernel(const uint16_t* __restrict__ x, int64_t M, int64_t K,
                                                        const uint16_t* __restrict__ a_t, int Rpad, int ranks, int ksplit,
                                                        uint16_t* __restrict__ t, float* __restrict__ partial,
                                                        int keep_fp32) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i16 = lane & 15, g = lane >> 4;
    const int64_t m0 = ((int64_t)blockIdx.x * 4 + wave) * 16 * kMB;
    if (m0 >= M) return;   // wave-uniform; the kernel has no barrier
    const int z = blockIdx.y;
    const int64_t units = K >> 5;
    const int64_t per_slice = (units + ksplit - 1) / ksplit;
    const int64_t u_begin = z * per_slice < units ? z * per_slice : units;
    const int64_t u_end = (z + 1) * per_slice < units ? (z + 1) * per_slice : units;
    const int64_t len = u_end - u_begin;
    const uint16_t* xrow[kMB];
#pragma unroll
    for (int mb = 0; mb < kMB; ++mb) {
        const int64_t mrow = m0 + 16 * mb + i16;
        xrow[mb] = x + (mrow < M ? mrow : M - 1) * K + 8 * g;
    }
    for (int rb = 0; rb < Rpad; rb += 16 * kRT) {
        // a pass starts inside the Rpad columns (loop bound); tiles of it that lie past them are clamped, not stored
        const uint16_t* arow[kRT];
#pragma unroll
        for (int rt = 0; rt < kRT; ++rt) {
            const int r = rb + 16 * rt + i16;
            arow[rt] = a_t + (int64_t)(r < Rpad ? r : Rpad - 1) * K + 8 * g;
        }
        f32x4 acc[kMB][kRT];
#pragma unroll
        for (int mb = 0; mb < kMB; ++mb)
#pragma unroll
            for (int rt = 0; rt < kRT; ++rt) acc[mb][rt] = f32x4{0.f, 0.f, 0.f, 0.f};
        // kDepth k-steps per trip with every load issued before the first MFMA: the kernel lives on loads in flight
        for (int64_t i0 = 0; i0 < len; i0 += kDepth) {
            uint4 aq[kDepth][kMB], bq[kDepth][kRT];
#pragma unroll
            for (int d = 0; d < kDepth; ++d) {
                const int64_t i = i0 + d < len ? i0 + d : len - 1;   // past the end: reload the last step, not used
                const int64_t k0 = (u_begin + i) << 5;
#pragma unroll
                for (int mb = 0; mb < kMB; ++mb) aq[d][mb] = *reinterpret_cast<const uint4*>(xrow[mb] + k0);
#pragma unroll
                for (int rt = 0; rt < kRT; ++rt) bq[d][rt] = *reinterpret_cast<const uint4*>(arow[rt] + k0);
            }
#pragma unroll
            for (int d = 0; d < kDepth; ++d) {
                if (i0 + d < len) {   // wave-uniform
#pragma unroll
                    for (int mb = 0; mb < kMB; ++mb)
#pragma unroll
                        for (int rt = 0; rt < kRT; ++rt)
                            acc[mb][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(aq[d][mb]), as_bf16x8(bq[d][rt]),
                                                                                  acc[mb][rt], 0, 0, 0);
                }
            }
        }
        // accumulator layout of the 16x16 MFMA: lane holds column lane % 16, rows 4 (lane / 16) + e
#pragma unroll
        for (int mb = 0; mb < kMB; ++mb)
#pragma unroll
            for (int rt = 0; rt < kRT; ++rt) {
                const int r = rb + 16 * rt + i16;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int64_t m = m0 + 16 * mb + 4 * g + e;
                    const float v = r < ranks ? acc[mb][rt][e] : 0.f;
                    if (m < M && r < Rpad) {
                        if (ksplit == 1 && !keep_fp32) t[m * Rpad + r] = f32_to_bf16_rne(v);
                        else partial[((int64_t)z * M + m) * Rpad + r] = v;
                    }
                }
            }
    }
}

// out = bf16(sum over z of partial[z]), four elements per thread, in a fixed order; slices are
// whole float4 apart (splitk_slice).  kZ threads share an
// output, thread q taking z = q, q + kZ, ..; each has up to eight requests in flight (one after the other, 56 slices of a
// [256, 32] sum took 15.9 us).  kCount: the number of slices where it is known (0: ksplit), so that no request is conditional.
// kPadded: out has rows of `cols` (a multiple of four), of which those from `valid` on are padding and stored as zeros.
template <int kZ, int kCount = 0, bool kPadded = false>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float* __restrict__ partial, int64_t count, int ksplit,
                                                            uint16_t* __restrict__ out, int cols, int valid) {
    constexpr int kOut = 256 / kZ;   // outputs (of four elements) per workgroup
    __shared__ float4 sums[kZ > 1 ? 256 : 1];
    const int64_t slice = splitk_slice(count);
    const int c = threadIdx.x % kOut, q = threadIdx.x / kOut;
    const int64_t i = ((int64_t)blockIdx.x * kOut + c) * 4;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    if (i < count) {
        if constexpr (kCount > 0) {
            float4 p[kCount];
#pragma unroll
            for (int z = 0; z < kCount; ++z) p[z] = *reinterpret_cast<const float4*>(partial + z * slice + i);
#pragma unroll
            for (int z = 0; z < kCount; ++z) { s.x += p[z].x; s.y += p[z].y; s.z += p[z].z; s.w += p[z].w; }
        } else {
            for (int z0 = q; z0 < ksplit; z0 += 8 * kZ) {
                float4 p[8];
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (z0 + kZ * j < ksplit) p[j] = *reinterpret_cast<const float4*>(partial + (int64_t)(z0 + kZ * j) * slice + i);
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (z0 + kZ * j < ksplit) { s.x += p[j].x; s.y += p[j].y; s.z += p[j].z; s.w += p[j].w; }
            }
        }
    }
    if constexpr (kZ > 1) {
        sums[threadIdx.x] = s;
        __syncthreads();
        if (q > 0) return;
#pragma unroll
        for (int j = 1; j < kZ; ++j) {
            const float4 p = sums[j * kOut + c];
            s.x += p.x; s.y += p.y; s.z += p.z; s.w += p.w;
        }
    }
    if (i >= count) return;
    if constexpr (kPadded) {
        const int c0 = (int)(i % cols);
        s = make_float4(c0 < valid ? s.x : 0.f, c0 + 1 < valid ? s.y : 0.f, c0 + 2 < valid ? s.z : 0.f, c0 + 3 < valid ? s.w : 0.f);
    }
    if (i + 4 > count) {   // the last outputs of a count that is no multiple of four
        const float e[3] = {s.x, s.y, s.z};
        for (int j = 0; i + j < count; ++j) out[i + j] = f32_to_bf16_rne(e[j]);
        return;
    }
    uint2 o;
    o.x = (uint32_t)f32_to_bf16_rne(s.x) | ((uint32_t)f32_to_bf16_rne(s.y) << 16);
    o.y = (uint32_t)f32_to_bf16_rne(s.z) | ((uint32_t)f32_to_bf16_rne(s.w) << 16);
    *reinterpret_cast<uint2*>(out + i) = o;
}

void launch_splitk_reduce(const float* partial, int64_t count, int ksplit, uint16_t* out, hipStream_t stream, int cols, int valid) {
#define SALR_SUM(OUT, ...) \
    hipLaunchKernelGGL((splitk_reduce_kernel<__VA_ARGS__>), dim3((unsigned)((count + 4 * (OUT)-1) / (4 * (OUT)))), dim3(256), 0, stream, \
                       partial, count, ksplit, out, cols, valid)
    if (valid < cols) {
        if (ksplit > 8) SALR_SUM(64, 4, 0, true);
        else SALR_SUM(256, 1, 0, true);
    } else if (ksplit > 8) SALR_SUM(64, 4);
    else if (ksplit == 2) SALR_SUM(256, 1, 2);   // the splits of the layers' kernels are powers of two
    else if (ksplit == 4) SALR_SUM(256, 1, 4);
    else if (ksplit == 8) SALR_SUM(256, 1, 8);
    else SALR_SUM(256, 1);
#undef SALR_SUM
}

// a_t[r][k] = A_cat[k][r] for r < R, 0 for R <= r < Rpad: one thread per k and block of 8 ranks.
__global__ __launch_bounds__(256) void adapter_transpose_kernel(const uint16_t* __restrict__ a_cat, int64_t K, int R,
                                                                 int Rpad, uint16_t* __restrict__ a_t) {
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k >= K) return;
    const int r0 = 8 * blockIdx.y;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int r = r0 + j;
        a_t[(int64_t)r * K + k] = r < R ? a_cat[k * R + r] : (uint16_t)0;
    }
}

void launch_adapter_transpose(const uint16_t* a_cat, int64_t K, int R, int Rpad, uint16_t* a_t, hipStream_t stream) {
    hipLaunchKernelGGL(adapter_transpose_kernel, dim3((unsigned)((K + 255) / 256), Rpad / 8), dim3(256), 0, stream, a_cat, K, R,
                       Rpad, a_t);
}

template <int kRT>
__global__ __launch_bounds__(256, kRT <= 2 ? 4 : 2) void tall_tn_kernel(RowProducts p) {
    __shared__ __attribute__((aligned(16))) uint16_t lds[kTnLdsBytes / 2];
    tall_tn_block<kRT, false>(p, (int)blockIdx.x, (int)blockIdx.y, lds);
}

__global__ __launch_bounds__(256) void row_products_reduce_kernel(RowProducts p) {
    __shared__ __attribute__((aligned(16))) float sums[kRpCols * kRpPitch];
    const int blocks0 = (int)((p.C[0] + kRpCols - 1) / kRpCols), job = (int)blockIdx.x < blocks0 ? 0 : 1;
    row_products_sum<false>(p, job, (int64_t)((int)blockIdx.x - (job == 0 ? 0 : blocks0)) * kRpCols, sums);
}

void launch_row_products(const RowProducts& p, hipStream_t stream) {
    const dim3 grid((unsigned)(row_product_blocks(p.C[0]) + row_product_blocks(p.C[1])), (unsigned)p.ksplit);
    if (p.Rpad % 64 == 0) hipLaunchKernelGGL(tall_tn_kernel<4>, grid, dim3(256), 0, stream, p);
    else hipLaunchKernelGGL(tall_tn_kernel<2>, grid, dim3(256), 0, stream, p);
    hipLaunchKernelGGL(row_products_reduce_kernel, dim3((unsigned)((p.C[0] + kRpCols - 1) / kRpCols + (p.C[1] + kRpCols - 1) / kRpCols)), dim3(256),
                       0, stream, p);
}

// T' = dY B_cat^T and T = X A_cat of the backward pass in one launch (salr_adapter_t.hpp), sixteen waves per 16 or 32 rows and 32
// ranks: the first blocks_dy workgroups take T'.  Bound by the L2: the small factor is read once per block of rows.  2048 x 4096 and
// 2048 x 4096 at rank 32: 12.1 us; padded and transposed copies of the factors, two split-K products, their sums and the
// transposes of the results took 43 us in eight launches.
template <int kMT, int kDepth, FactorLayout kFactor>
__global__ __launch_bounds__(1024) void backward_t_kernel(LowRankJob dy_b, LowRankJob x_a, int64_t M, int R, int Rpad, int blocks_dy) {
    constexpr int kBytes = adapter_t_lds_bytes<kMT, 16, kFactorRanks>(), kBytesA = adapter_t_lds_bytes<kMT, 16, kFactor>();
    __shared__ __attribute__((aligned(16))) uint16_t lds[(kBytes > kBytesA ? kBytes : kBytesA) / 2];
    const int groups = Rpad >> 5;
    if ((int)blockIdx.x < blocks_dy) {   // the same for the whole workgroup
        adapter_t_block<kMT, 16, kDepth, kFactorRanks>(dy_b.in, M, dy_b.C, dy_b.factor, R, Rpad, dy_b.t, blockIdx.x / groups,
                                                       (int)blockIdx.x % groups, lds, dy_b.t_t);
    } else {
        const int id = (int)blockIdx.x - blocks_dy;
        adapter_t_block<kMT, 16, kDepth, kFactor>(x_a.in, M, x_a.C, x_a.factor, R, Rpad, x_a.t, id / groups, id % groups, lds, x_a.t_t);
    }
}

void launch_backward_t(const LowRankJob& dy_b, const LowRankJob& x_a, int64_t M, int R, hipStream_t stream) {
    const int Rpad = (int)adapter_rank_padded(R), groups = Rpad / 32;
    const int jobs = (dy_b.in != nullptr ? 1 : 0) + (x_a.in != nullptr ? 1 : 0);
    const int tiles = adapter_t_row_tiles(M);
    const int64_t blocks = (M + 16 * tiles - 1) / (16 * tiles) * groups;
    const int blocks_dy = dy_b.in != nullptr ? (int)blocks : 0;
    const dim3 grid((unsigned)(blocks * jobs));
#define SALR_BT(MT, DEPTH, F) \
    hipLaunchKernelGGL((backward_t_kernel<MT, DEPTH, F>), grid, dim3(1024), 0, stream, dy_b, x_a, M, R, Rpad, blocks_dy)
    if (R % 8 == 0) {
        if (tiles == 2) SALR_BT(2, 2, kFactorVec);
        else SALR_BT(1, 3, kFactorVec);
    } else {
        if (tiles == 2) SALR_BT(2, 1, kFactorAny);
        else SALR_BT(1, 2, kFactorAny);
    }
#undef SALR_BT
}

template <int kMB, int kDepth>
static void launch_tall_product_rt(int rank_tiles, dim3 grid, hipStream_t stream, const uint16_t* x, int64_t M, int64_t K,
                                   const uint16_t* a_t, int Rpad, int ranks, int ksplit, uint16_t* t, float* partial, int keep) {
    switch (rank_tiles) {
#define SALR_CASE(RT)                                                                                                   \
    case RT:                                                                                                            \
        hipLaunchKernelGGL((adapter_t_kernel<kMB, RT, kDepth>), grid, dim3(256), 0, stream, x, M, K, a_t, Rpad, ranks, ksplit, t, \
                           partial, keep);                                                                              \
        break;
        SALR_CASE(2) SALR_CASE(3) SALR_CASE(4) SALR_CASE(5) SALR_CASE(6) SALR_CASE(7) SALR_CASE(8)
#undef SALR_CASE
        default: break;
    }
}

void launch_tall_product(const uint16_t* x, int64_t M, int64_t K, const uint16_t* a_t, int Rpad, int ranks, int ksplit, uint16_t* t,
                         float* partial, bool keep_fp32, hipStream_t stream) {
    const int rows = adapter_rows_per_block(M);
    const dim3 grid((unsigned)((M + rows - 1) / rows), (unsigned)ksplit);
    // rank tiles of 16 columns per pass over the slice: as few passes as eight tiles at a time allow, evenly filled
    const int tiles = Rpad / 16, passes = (tiles + 7) / 8;
    const int rank_tiles = (tiles + passes - 1) / passes;
    const int keep = keep_fp32 ? 1 : 0;
    if (rows == 256) launch_tall_product_rt<4, 2>(rank_tiles, grid, stream, x, M, K, a_t, Rpad, ranks, ksplit, t, partial, keep);
    else launch_tall_product_rt<1, 4>(rank_tiles, grid, stream, x, M, K, a_t, Rpad, ranks, ksplit, t, partial, keep);
}

void launch_adapter_t(const LinearArgs& a, hipStream_t stream) {
    const int R = (int)a.R, Rpad = (int)adapter_rank_padded(a.R);
    char* base = reinterpret_cast<char*>(a.t);
    uint16_t* a_t = reinterpret_cast<uint16_t*>(base + adapter_t_bytes(a.M, a.R));
    float* partial = reinterpret_cast<float*>(base + adapter_t_bytes(a.M, a.R) + adapter_at_bytes(a.K, a.R));
    if (adapter_uses_prekernel(a.M)) {   // two launches: split-K partials from A_cat as it is, then their sum
        launch_adapter_partial_to(a, partial, stream);
        launch_splitk_reduce(partial, a.M * Rpad, kStreamTSlices, a.t, stream);
        return;
    }
    // One launch and no partial sums where X is read once (ranks up to 32).  2:4 calls: 4096 x 2048 x 8192 135.8 -> 127.4 us,
    // 1500 x 8192 x 8192 178.4 -> 175.3; at rank 64 it reads X twice and 4096 x 4096 x 8192 goes 235 -> 237.5; at 1024 rows and
    // below the two launches above are level with it.
    if (Rpad == 32 && !adapter_t_own_product(a.M, a.K, a.R)) {
        launch_adapter_t_direct(a.x, a.M, a.K, a.a_cat, R, Rpad, a.t, stream);
        return;
    }
    launch_adapter_transpose(a.a_cat, a.K, R, Rpad, a_t, stream);
    const int ksplit = adapter_ksplit(a.M, a.K);
    launch_tall_product(a.x, a.M, a.K, a_t, Rpad, R, ksplit, a.t, partial, false, stream);
    if (ksplit > 1) launch_splitk_reduce(partial, a.M * Rpad, ksplit, a.t, stream);
}

}  // namespace salr
