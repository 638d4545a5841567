// First adapter stage of the large-batch paths (paper Sec. 3.2): T = X * A_cat, plus the small passes around it
// (transposed copy of A_cat, fixed-order sum of split-K partials, also used by the dense stage).
#include "salr_adapter_t.hpp"
#include "salr_device.hpp"
#include "salr_internal.hpp"
#include "salr_linear_common.hpp"

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

// ---------------------------------------------------------------------------------------------------
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
// ---------------------------------------------------------------------------------------------------
constexpr int kTnPitch = 64 + 8;   // bf16 elements per tile row
constexpr int kTnBatch = 4;

template <int kRT>
__global__ __launch_bounds__(256, kRT <= 2 ? 4 : 2) void tall_tn_kernel(const uint16_t* __restrict__ in0, const uint16_t* __restrict__ s_t0, int64_t C0,
                                                      const uint16_t* __restrict__ in1, const uint16_t* __restrict__ s_t1, int64_t C1,
                                                      int64_t M, int Rpad, int ksplit, float* __restrict__ partial0) {
    __shared__ __attribute__((aligned(16))) uint16_t tile[2][kTnBatch][32 * kTnPitch];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i16 = lane & 15, g = lane >> 4;
    const int blocks0 = (int)((C0 + 63) / 64);
    const bool first = (int)blockIdx.x < blocks0;   // the same for the whole workgroup
    const uint16_t* in = first ? in0 : in1;
    const uint16_t* s_t = first ? s_t0 : s_t1;
    const int64_t C = first ? C0 : C1;
    float* partial = partial0 + (first ? 0 : (int64_t)ksplit * C0 * Rpad);
    const int64_t c0 = (int64_t)((int)blockIdx.x - (first ? 0 : blocks0)) * 64;
    const int z = blockIdx.y;
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
                if (c < C && r < Rpad) partial[((int64_t)z * C + c) * Rpad + r] = acc[rt][e];
            }
        }
    }
}

// The sums over the slices of tall_tn_kernel, 32 matrix columns per workgroup: read along the ranks, as they lie, and through LDS
// into out0 [C0, R] and out1 [R, C1] (read in the order of the outputs, dB's sums came one 128-byte line per value: 7.4 us a
// gradient on 4096 columns of rank 32, 16 slices).
constexpr int kRpCols = 32;

__global__ __launch_bounds__(256) void row_products_reduce_kernel(const float* __restrict__ partial0, int64_t C0, int64_t C1, int Rpad,
                                                                  int ksplit, int R, uint16_t* __restrict__ out0,
                                                                  uint16_t* __restrict__ out1) {
    __shared__ float sums[kRpCols][kMaxRankPadded + 1];
    const int blocks0 = (int)((C0 + kRpCols - 1) / kRpCols);
    const bool first = (int)blockIdx.x < blocks0;   // the same for the whole workgroup
    const int64_t C = first ? C0 : C1;
    const float* partial = partial0 + (first ? 0 : (int64_t)ksplit * C0 * Rpad);
    const int64_t c0 = (int64_t)((int)blockIdx.x - (first ? 0 : blocks0)) * kRpCols;
    const int cols = C - c0 < kRpCols ? (int)(C - c0) : kRpCols;
    const int quads = Rpad >> 2;
    for (int i = threadIdx.x; i < cols * quads; i += 256) {
        const float* p = partial + c0 * Rpad + 4 * i;
        float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int z0 = 0; z0 < ksplit; z0 += 8) {
            float4 q[8];
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (z0 + j < ksplit) q[j] = *reinterpret_cast<const float4*>(p + (int64_t)(z0 + j) * C * Rpad);
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (z0 + j < ksplit) { s.x += q[j].x; s.y += q[j].y; s.z += q[j].z; s.w += q[j].w; }
        }
        float* to = &sums[i / quads][4 * (i % quads)];
        to[0] = s.x; to[1] = s.y; to[2] = s.z; to[3] = s.w;
    }
    __syncthreads();
    if (first) {
        for (int i = threadIdx.x; i < cols * R; i += 256) out0[c0 * R + i] = f32_to_bf16_rne(sums[i / R][i % R]);
    } else {
        for (int i = threadIdx.x; i < kRpCols * R; i += 256) {
            const int c = i % kRpCols, r = i / kRpCols;
            if (c < cols) out1[r * C + c0 + c] = f32_to_bf16_rne(sums[c][r]);
        }
    }
}

void launch_row_products(const RowProductJob& da, const RowProductJob& db, int64_t M, int R, int ksplit, float* partial,
                         hipStream_t stream) {
    const int Rpad = (int)adapter_rank_padded(R);
    const int64_t C0 = da.out != nullptr ? da.C : 0, C1 = db.out != nullptr ? db.C : 0;
    const dim3 grid((unsigned)((C0 + 63) / 64 + (C1 + 63) / 64), (unsigned)ksplit);
#define SALR_TN(RT) \
    hipLaunchKernelGGL(tall_tn_kernel<RT>, grid, dim3(256), 0, stream, da.in, da.s_t, C0, db.in, db.s_t, C1, M, Rpad, ksplit, partial)
    if (Rpad % 64 == 0) SALR_TN(4);
    else SALR_TN(2);
#undef SALR_TN
    hipLaunchKernelGGL(row_products_reduce_kernel, dim3((unsigned)((C0 + kRpCols - 1) / kRpCols + (C1 + kRpCols - 1) / kRpCols)), dim3(256), 0,
                       stream, partial, C0, C1, Rpad, ksplit, R, da.out, db.out);
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
