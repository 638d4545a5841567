// Host-side declarations shared between the C boundary and the kernel files.
#pragma once

#include <hip/hip_runtime.h>
#ifdef __HIPCC__
#include <hip/hip_ext.h>   // (SALR_LAUNCH; not for a host compiler)
#endif
#include <stddef.h>
#include <stdint.h>

namespace salr {

hipError_t launch_encode(const uint16_t* w, int64_t rows, int64_t cols, uint32_t* bitmap, uint16_t* values,
                         int64_t capacity, uint32_t* row_offsets, hipStream_t stream);

// The two halves of it, for a caller that sizes `values` in between: bitmap and row offsets (the total also to *nnz_host,
// pinned host memory, unless null), then the packed values.
hipError_t launch_encode_index(const uint16_t* w, int64_t rows, int64_t cols, uint32_t* bitmap, uint32_t* row_offsets,
                               uint32_t* nnz_host, hipStream_t stream);
hipError_t launch_encode_values(const uint16_t* w, int64_t rows, int64_t cols, const uint32_t* bitmap, const uint32_t* row_offsets,
                                uint16_t* values, int64_t capacity, hipStream_t stream);

hipError_t launch_decode(const uint32_t* bitmap, const uint16_t* values, const uint32_t* row_offsets, int64_t rows,
                         int64_t cols, uint16_t* out, hipStream_t stream);

hipError_t launch_mask_rows(const uint16_t* w, int64_t rows, int64_t cols, int64_t keep, uint16_t* out,
                            hipStream_t stream);

hipError_t launch_mask_nm(const uint16_t* w, int64_t rows, int64_t cols, int n_keep, int m_group, uint16_t* out,
                          hipStream_t stream);

hipError_t launch_residual(const uint16_t* w, const uint16_t* w_hat, int64_t rows, int64_t cols, uint16_t* e,
                           hipStream_t stream);

// Host arrays of n device pointers / ranks; R = sum of the ranks.
constexpr int kConcatBatch = 16;
hipError_t launch_concat(const uint16_t* const* a_list, const uint16_t* const* b_list, const int64_t* ranks, int64_t n,
                         int64_t K, int64_t N, int64_t R, uint16_t* a_cat, uint16_t* b_cat, hipStream_t stream);

// Residual adapter: rank-r factors of E [N, K] by subspace iteration with l = r + oversample columns (l <= 128)
constexpr int64_t kSvdMaxColumns = 128;
size_t residual_adapter_workspace_bytes(int64_t N, int64_t K, int64_t l);
hipError_t launch_residual_adapter(const uint16_t* e, int64_t N, int64_t K, int64_t r, int64_t l, int64_t iterations,
                                   const float* omega, uint16_t* a_res, uint16_t* b_res, float* sigma, void* workspace,
                                   hipStream_t stream);

// Columns of the bf16 workspace matrix T = X * A_cat: R rounded up to the MFMA k-step.
inline int64_t adapter_rank_padded(int64_t R) { return (R + 31) / 32 * 32; }

struct LinearArgs {
    const uint16_t* x;
    int64_t M, K, N;
    const uint32_t* bitmap;
    const uint16_t* values;
    const uint32_t* row_offsets;
    const uint16_t* a_cat;
    const uint16_t* b_cat;
    int64_t R;
    uint16_t* y;
    uint16_t* t;  // workspace (see linear_workspace_bytes)
    bool lean = false;  // large batches: no room for a decoded copy of the weight, take the fused kernel
    size_t room = 0;    // bytes of the workspace (large batches: see linear_takes_frag)
    const uint32_t* slice_table = nullptr;  // optional: the layer's slice table (see kSliceTableSlices)
    bool build_table = false;  // slice_table points into the workspace and the adapter pre-kernel fills it in this call
    // QSALR on the large-batch path: `values` is null and the decode stage reads these (nnz values, 4-bit codes)
    const uint8_t* codes = nullptr;
    const uint16_t* scales = nullptr;
    int64_t nnz = 0;
};

// Slice table of a layer (a derived, kernel-private index; the three arrays of the format stay what is checked): for
// row n and slice w of the small-batch kernel's 8 wave slices (chunks [C w / 8, C (w + 1) / 8) of the row's
// C = ceil(K / 128) chunks of 128 columns) two uint32: the index in `values` of the slice's first value, and the most
// nonzeros any one chunk of the slice holds.
constexpr int kSliceTableSlices = 8;
inline size_t slice_table_bytes(int64_t N) { return (size_t)N * kSliceTableSlices * 2 * sizeof(uint32_t); }
hipError_t launch_build_slice_table(const uint32_t* bitmap, const uint32_t* row_offsets, int64_t N, int64_t K, uint32_t* table,
                                    hipStream_t stream);

// Optional events recorded around the fused kernel's launch (measurement hook of the boundary).
struct TimingEvents {
    hipEvent_t start = nullptr;
    hipEvent_t stop = nullptr;
};
extern thread_local TimingEvents g_timing_events;

// Launch `kernel`; when both events are set they receive the kernel's own begin/end timestamps.
#define SALR_LAUNCH(kernel, grid, block, stream, ev, ...)                                                    \
    do {                                                                                                      \
        if ((ev).start != nullptr && (ev).stop != nullptr)                                                    \
            hipExtLaunchKernelGGL(kernel, grid, block, 0, stream, (ev).start, (ev).stop, 0, __VA_ARGS__);     \
        else                                                                                                  \
            hipLaunchKernelGGL(kernel, grid, block, 0, stream, __VA_ARGS__);                                  \
    } while (0)

// Small-batch path: M <= kStreamMaxM; T = X * A_cat arrives as kStreamTSlices split-K partials (fp32).
constexpr int64_t kStreamMaxM = 64;
constexpr int kStreamTSlices = 16;
constexpr int kRowtileTSlices = 4;   // at most, see rowtile_plan
constexpr int kMaxRankPadded = 256;  // R <= 256: pitch of the T tile the streaming kernels keep in LDS

// Large-batch path: M > kStreamMaxM decodes the weight once into scratch memory in MFMA operand order, then runs a dense
// MFMA GEMM on it (salr_gemm.hip; k-steps of 64, the 256 rows of a tile of X lie within 2 GB).  Wherever the call's workspace has room
// for it: 300 x 2720 x 2731 39 us against 111 on the generic kernel, 2048 x 4096 x 14336 249 against 284 on the next one.
constexpr int64_t kFragMaxColumns = 1 << 22;
inline bool uses_frag(int64_t M, int64_t K) { return M > kStreamMaxM && K >= 32 && K % 32 == 0 && K <= kFragMaxColumns; }
// The same in two stages with a row-major copy (salr_linear_twostage.hip), K % 64 == 0: what salr_linear_workspace_bytes sizes a
// workspace for.  It needs less room (no rank blocks beside the weight), and is what a call with that much and no more
// gets where the rank blocks do not fit; half as fast again as the kernel without a decoded copy.
inline bool uses_twostage(int64_t M, int64_t K) { return M > kStreamMaxM && K >= 64 && K % 64 == 0; }
// Decoded weight in operand order (salr_gemm.hip): 1 KB blocks of 16 rows x 32 columns, an even number along the columns,
// and the rank blocks of B_cat (likewise) behind them.
inline size_t frag_weight_bytes(int64_t K, int64_t N, int64_t R) {
    return (size_t)((N + 15) / 16) * (size_t)((K + 63) / 64 + (R + 63) / 64) * 2048;
}

// A 2:4-masked weight in sparse operand order (pack_2of4_kernel): pairs of k-steps of 16 rows x 128 columns, 2048 bytes of values
// and 256 of positions, then the rank blocks of B_cat.
constexpr int64_t kSparsePairElems = 1152;
constexpr int64_t kSparseOrderMinM = 1536;   // see launch_gemm_2of4
#ifdef __HIPCC__
__host__ __device__
#endif
inline int64_t sparse_frag_elems(int64_t K, int64_t Rpad) { return (K / 64 + 1) / 2 * kSparsePairElems + Rpad / 32 * 512; }
inline size_t sparse_weight_bytes(int64_t K, int64_t N, int64_t R) {
    return (size_t)((N + 15) / 16) * (size_t)sparse_frag_elems(K, adapter_rank_padded(R)) * 2;
}

inline size_t round_up_256(size_t b) { return (b + 255) / 256 * 256; }

// Workspace layout of the large-batch paths (M > kStreamMaxM): T [M, Rpad] bf16, the transposed padded adapter
// a_t [Rpad, K] bf16, the split-K partials of T, then (two-stage path only) the decoded weight [N, K] bf16 and the
// split-K partials of Y; each 256-byte aligned.
inline size_t adapter_t_bytes(int64_t M, int64_t R) {
    return R > 0 ? round_up_256((size_t)M * (size_t)adapter_rank_padded(R) * sizeof(uint16_t)) : 0;
}
inline size_t adapter_at_bytes(int64_t K, int64_t R) {
    return R > 0 ? round_up_256((size_t)K * (size_t)adapter_rank_padded(R) * sizeof(uint16_t)) : 0;
}
// A_cat^T in operand order (whole k-steps of 64)
inline size_t adapter_frag_bytes(int64_t K, int64_t R) {
    return R > 0 ? round_up_256((size_t)((K + 63) / 64 * 64) * (size_t)adapter_rank_padded(R) * sizeof(uint16_t)) : 0;
}
// Rows of X per block of the large-batch T (salr_adapter_t.hpp), in tiles of 16: two where the blocks are many anyway (each
// reads its ranks' part of A_cat once).
constexpr int64_t kAdapterWideM = 1024;
inline int adapter_t_row_tiles(int64_t M) { return M >= kAdapterWideM ? 2 : 1; }
// T = X * A_cat of the large-batch paths: one launch that reads X once per 32 ranks and A_cat once per block of rows
// (launch_adapter_t_direct), or a split-K product on the MFMA stage's kernel, which reads X once but costs a summing pass and
// A_cat in operand order.  The latter where the former is more than about fifteen microseconds of traffic (70B down_proj at
// 4096 tokens: 85 us; the transposing pass, tall product and sum before it 129) or a long chain of steps (300 tokens: 8.8 us at
// K = 4096, 20.6 at 14336; the product and its sum 14), and where A_cat's rows are no whole 16-byte vectors.
inline bool adapter_t_own_product(int64_t M, int64_t K, int64_t R) {
    if (R % 8 != 0 || K > 8192) return true;
    const double groups = (double)((R + 31) / 32), rows = 16.0 * adapter_t_row_tiles(M);
    return groups * ((double)M * K * 2 + M / rows * 64.0 * K) > 64e6;
}
// Where a pass over the weight runs first anyway (large batches), T is computed by workgroups of that launch: a chain of steps on a few
// CUs beside a pass that fills the memory system.  Longer rows take the product above (us a call, beside / product: 300 x 8192 x 600 at
// rank 64 75.0 / 84.7, 657 x 4736 x 768 at rank 128 37.1 / 51.3, 4096 x 8192 x 8192 at rank 64 465 / 472; 1024 x 14336 x 4096 180 / 170,
// 200 x 28672 x 1024 97 / 77).
inline bool adapter_t_in_pass(int64_t K, int64_t R) { return R > 0 && R % 8 == 0 && K <= 8192; }
// Each 32 ranks read X again, so many tokens at many ranks take the product, which reads it once (beside / product, N = 640: 2048 x 4096
// rank 256 58.4 / 76.1, 4096 x 8192 rank 64 87.0 / 88.6, 3072 x 6144 rank 192 84.9 / 93.4; 4096 x 6144 rank 160 98.4 / 93.9,
// 4096 x 8192 rank 160 124 / 108, rank 256 149 / 112; N = 4096: 302 / 273).  The pass over a 2:4-masked weight keeps it: 4096 x 8192 x 3072
// rank 256 253 / 276 against the transposing launches that path has otherwise.
inline bool adapter_t_beside(int64_t M, int64_t K, int64_t R) {
    return adapter_t_in_pass(K, R) && (R + 31) / 32 * M * K <= 120000000;
}
inline int adapter_t_product_ksplit(int64_t M, int64_t K, int64_t Rpad) {
    const int64_t wgs = (M + 255) / 256 * ((Rpad + 127) / 128), steps = (K + 63) / 64;
    int64_t ks = (256 + wgs - 1) / wgs;
    if (ks > steps / 4) ks = steps / 4;
    return (int)(ks < 1 ? 1 : ks > 64 ? 64 : ks);
}
// T = X * A_cat splits K over workgroups (fp32 partials [ksplit, M, Rpad], added up in a fixed order).
inline int adapter_rows_per_block(int64_t M) { return M >= 4096 ? 256 : 64; }
inline int adapter_ksplit(int64_t M, int64_t K) {
    const int64_t rows = adapter_rows_per_block(M);
    const int64_t blocks = (M + rows - 1) / rows, units = K / 32;
    int s = 1;
    while (s < 64 && blocks * s * 2 <= 1024 && units / (s * 2) >= 8) s *= 2;
    return s;
}
// Up to kAdapterSmallM rows the small-batch pre-kernel computes T (one launch of many short workgroups reading A_cat as it
// is, kStreamTSlices fp32 partials) and the reducing pass sums them; above, the transposing pass + tall product + sum.
constexpr int64_t kAdapterSmallM = 1024;
inline bool adapter_uses_prekernel(int64_t M) { return M <= kAdapterSmallM; }
inline size_t adapter_partial_bytes(int64_t M, int64_t K, int64_t R) {
    if (R > 0 && adapter_uses_prekernel(M))
        return round_up_256((size_t)kStreamTSlices * (size_t)M * (size_t)adapter_rank_padded(R) * sizeof(float));
    const int s = adapter_ksplit(M, K);
    return (R > 0 && s > 1) ? round_up_256((size_t)s * (size_t)M * (size_t)adapter_rank_padded(R) * sizeof(float)) : 0;
}
inline size_t twostage_dense_offset(int64_t M, int64_t K, int64_t R) {
    return adapter_t_bytes(M, R) + adapter_at_bytes(K, R) + adapter_partial_bytes(M, K, R);
}
inline size_t frag_weight_offset(int64_t M, int64_t K, int64_t R) {   // T first, then what a product of its own needs (launch_linear_frag)
    size_t b = adapter_t_bytes(M, R);
    if (R > 0 && !adapter_t_beside(M, K, R)) {
        const int64_t Rpad = adapter_rank_padded(R);
        b += adapter_frag_bytes(K, R) + round_up_256((size_t)adapter_t_product_ksplit(M, K, Rpad) * (size_t)M * (size_t)Rpad * sizeof(float));
    }
    return b;
}

// Split of K over workgroups in the dense stage of the two-stage path: used when the 256 x 128 output tiles are
// too few for the 256 CUs.  Needs N % 4 == 0 (vector stores of the reducing pass) and an even split of the 64-wide
// k-steps; the fp32 partial tiles [ksplit, M, N] follow the dense weight in the workspace.
inline int dense_ksplit(int64_t M, int64_t K, int64_t N) {
    const int64_t tiles = ((M + 255) / 256) * ((N + 127) / 128);
    const int64_t steps = K / 64;
    if (tiles >= 128 || N % 4 != 0) return 1;
    int s = 1;
    while (s < 8 && tiles * s * 2 <= 256 && steps % (s * 2) == 0 && steps / (s * 2) >= 4) s *= 2;
    return s;
}

// fp32 elements from one slice of a split contraction's partial sums to the next
#ifdef __HIPCC__
__host__ __device__
#endif
inline int64_t splitk_slice(int64_t count) { return (count + 3) / 4 * 4; }

// Output tile of the large-batch MFMA stage and its split of the contraction over workgroups (fp32 partial outputs
// [ksplit, M, N], summed by splitk_reduce_kernel).  Kt = columns of X plus padded ranks.  The choice minimises a model of the
// stage's time in microseconds.  A tile has the time of a k-step on a CU that is full of its workgroups (per workgroup: what
// the matrix cores sustain on data at this chip's power), the time of one that is alone (latency, or the same where a CU
// holds one), and what a workgroup spends outside its loop (first tiles, results; half of it hidden behind the loop of a
// neighbour on the CU).  A split adds the partial sums' way through memory and one launch.  Against all tiles and splits on 126
// points (21 layers from 512 to 28672 wide, 130 to 4096 tokens; profiles/linear_large_batch_tile_sweep.txt) the choice is the best
// at 68 and within 1 % at 79; its stage takes 3.7 % more on average.  The misses: splits of layers of a few million entries at 300
// to 512 tokens (up to 5 us of stage, -1.5 to +2.3 us of the call), and weights of 235 million entries at 130 and 300 tokens,
// where it takes rows of 64 or 128 and tiles of 256 are faster (30 to 61 us of a call of 347 to 440).  partial_room: bytes there
// are for the partial outputs.
struct GemmPlan {
    int mt, nt, ksplit;
};
inline size_t gemm_partial_bytes(int64_t M, int64_t N, int ksplit) {
    return ksplit > 1 ? round_up_256((size_t)ksplit * (size_t)splitk_slice(M * N) * sizeof(float)) : 0;
}
inline GemmPlan gemm_plan(int64_t M, int64_t Kt, int64_t N, size_t partial_room = SIZE_MAX) {
    struct Tile {
        int mt, nt, per_cu;
        double step, alone, outside;
    };
    constexpr Tile kTiles[7] = {{256, 256, 1, 1.45, 1.45, 13.8},  {256, 224, 1, 1.32, 1.32, 13.0}, {128, 256, 2, 0.80, 0.81, 7.6},
                                {128, 128, 2, 0.42, 0.53, 4.6},   {64, 256, 3, 0.45, 0.50, 5.1},   {64, 128, 4, 0.30, 0.44, 3.0},
                                {64, 64, 4, 0.17, 0.41, 2.5}};
    const int64_t steps = (Kt + 63) / 64;   // (one more when both parts end in half a step: of no account here)
    GemmPlan best{64, 64, 1};
    double best_cost = 1e300;
    for (const Tile& t : kTiles) {
        const int64_t tiles = ((M + t.mt - 1) / t.mt) * ((N + t.nt - 1) / t.nt);
        const double outside = t.outside * (N % 8 != 0 ? 1.65 : 1.0);   // results that leave in pieces
        for (int ks = 1; ks <= 16 && (ks == 1 || (steps / ks >= 3 && gemm_partial_bytes(M, N, ks) <= partial_room)); ks *= 2) {
            const int64_t on_cu = (tiles * ks + 255) / 256, rounds = (on_cu + t.per_cu - 1) / t.per_cu;
            const double full = (double)on_cu * t.step, lone = (double)rounds * t.alone;
            double cost = (full > lone ? full : lone) * (double)((steps + ks - 1) / ks);
            cost += (t.per_cu == 1 ? (double)rounds : 1.0 + (double)(on_cu - 1) * 0.46) * outside;
            if (ks > 1) cost += 1.8 + (double)M * (double)N * (8 * ks + 2) * 0.08e-6;
            if (cost < best_cost) {
                best_cost = cost;
                best = {t.mt, t.nt, ks};
            }
        }
    }
    return best;
}

// Row-tiled streaming path (one pass over the compressed weight, X shared by the 128 rows of a workgroup) on the size that
// salr_linear_workspace_bytes tells: batches of 33 to 128 tokens, and of 9 to 32 on layers of 8192 rows and more, whose rows come in
// whole 128-column chunks.  rowtile_ksplit is the split of K that this size has room for, fp32 partial outputs [ksplit, M, N] behind T;
// the 2:4 kernel, of which two workgroups share a CU, splits so.  The row-tiled kernel has one workgroup a CU and its own plan
// (rowtile_plan) within the same bytes; its other shapes and what they need are rowtile_wide's.
constexpr int64_t kRowtileMaxM = 128;
constexpr int kRowtileMaxSplit = 32;
constexpr int64_t kRowtileMaxColumns = 1 << 22;   // 32-bit offsets into X and a wave's rows of the weight
inline int rowtile_ksplit(int64_t M, int64_t K, int64_t N) {
    const int64_t tiles = (N + 127) / 128, chunks = K / 128;
    if (N % 4 != 0) return 1;   // the reducing pass stores four outputs per thread
    // (2:4 kernel:) up to 64 tokens two workgroups share a CU and hide each other's barriers, above that one fills it
    const int64_t enough = M <= 64 ? 448 : 224;
    int s = 1;
    while (s < 16 && tiles * s < enough && chunks / (s * 2) >= 4) s *= 2;
    return s;
}
inline bool rowtile_possible(int64_t M, int64_t K) { return M <= kRowtileMaxM && K >= 128 && K % 128 == 0; }
inline bool uses_rowtile(int64_t M, int64_t K, int64_t N) {
    if (!rowtile_possible(M, K) || K > kRowtileMaxColumns) return false;   // (longer rows: the paths with 64-bit offsets)
    if (N % 4 != 0 && N < 64 * 128) return false;   // K cannot be split and the row tiles are few
    return M > 32 || (M > 8 && N >= 8192);
}
// T of the row-tiled path: the split-K partials of the small-batch pre-kernel
inline size_t rowtile_t_bytes(int64_t M, int64_t K, int64_t R) {
    if (R <= 0) return 0;
    return round_up_256((size_t)kStreamTSlices * (size_t)M * (size_t)adapter_rank_padded(R) * sizeof(float));
}
// T as the launch of the row-tiled kernel itself leaves it, ahead of the partial outputs
inline size_t rowtile_t_out_bytes(int64_t M, int64_t R) {
    return R > 0 ? round_up_256((size_t)kRowtileTSlices * (size_t)M * (size_t)adapter_rank_padded(R) * sizeof(float)) : 0;
}
// fp32 partial outputs of one slice, rows of whole vectors of four
inline int64_t rowtile_pitch(int64_t N) { return (N + 3) / 4 * 4; }
inline size_t rowtile_partial_bytes(int64_t M, int64_t N) { return (size_t)M * (size_t)rowtile_pitch(N) * sizeof(float); }
// How the row-tiled kernel cuts its work: K over `ksplit` workgroups per 128 rows, and X A_cat over `t_slices` workgroups per 16
// tokens and 16 ranks of the same launch.  The least of a model of the call's time in microseconds: the launch and the start of a
// slice, rounds of 256 workgroups, one per CU, the chunks of a slice, the popcounts of the bitmap left of it, and the summing
// launch, which there is when K is split or there are adapters.  A step of T's sum, four of 32 columns for each of eight waves, is 1.7 us above 32 ranks, whose rows of
// A_cat a workgroup reads in 32 bytes each: long rows get several slices of T rather than one more of the weight (16 x 19840 x 3200 rank 64: one slice of
// T and ten of the weight 52.4 us, two and nine 36.3, the small-batch kernel 43.5).  Up to 32 ranks 1.2: with 1.7 16 of 598 calls of 17 to 64 tokens
// lose more than 3 % (64 x 6176 x 2432 rank 16 18.3 -> 20.8) and 4 gain as much; above 32 4 and 40 of 574.  Its other figures are those of up to 16, 32, 64 and 128 tokens
// on 4096 x 14336 (2 slices: 22.4, 24.9, 29.9 and 40 us; 4: 26.7, 29.0, 36.1; 1: 35.1, 38.5, 46.0, 59) and 14336 x 4096.
// partial: fp32 partial outputs in the workspace.  Without room for one slice's (`room` bytes) T comes from a launch in front and
// the only slice adds the adapters itself.
struct RowtilePlan {
    int ksplit = 1, t_slices = 1;
    int parts = 1;           // of a slice, one beside the other in a workgroup of 128 / parts rows
    bool partial = false;    // fp32 partial outputs
    bool one_launch = false; // the adapters are added in the launch itself, from T as its first workgroups leave it
    double cost = 1e300;   // microseconds by that model
    int64_t chunks = 0;    // that a CU goes through, one workgroup after the other
};
// Parts of K in a workgroup (1, 2, 4: 128, 64, 32 rows) instead of slices over workgroups, where that many row tiles and T's workgroups are one
// round: no partial outputs and no launch that sums them, but every workgroup copies all of X to LDS, in shorter panels with as many more
// barriers (part_step: what that adds to a chunk), and from 33 tokens on four parts' panels would hold half a unit.  Below kOneLaunchTiles row tiles
// too few CUs take part, whatever the model says.  us a call, slices / parts (how many; layers of 256 MB together, one after the other, rank 32):
// 16 x 4096 x 14336 20.8 / 19.9 (2), 32 tokens 23.8 / 22.6 (2), 8 x 2048 x 14336 14.4 / 12.3 (2), 16 x 4096 x 7168 15.6 / 13.9 (4), 64 x 4096 x 28672
// 47.6 / 43.2 (1), 64 x 2048 x 14336 20.3 / 17.6 (2), 16 x 8192 x 28672 rank 64 60.7 / 58.1 (1); left with slices, before their starts were made
// cheaper: 64 x 8192 x 14336 51.0 / 54.0 (2), 16 x 3072 x 8192 14.4 / 15.3 (2), 24 x 8192 x 7168 26.3 / 29.2 (4).  Of 220 random calls of 1 to 128 tokens on
// layers 512 to 16384 columns by 3000 to 28672 rows the rule makes 4 slower by more than 2 %, at most by 6, the geometric mean 1.035.
constexpr int64_t kOneLaunchTiles = 130;
inline double part_step(int64_t M, int q) {
    if (q == 1) return 0.0;
    if (M <= 16) return q == 2 ? 0.10 : 0.24;
    if (M <= 32) return q == 2 ? 0.12 : 0.40;
    return M <= 64 ? 0.42 : 0.55;
}
inline RowtilePlan rowtile_plan(int64_t M, int64_t K, int64_t N, int64_t R, size_t room, bool slices_only = false) {
    const int64_t tiles = (N + 127) / 128, chunks = (K + 127) / 128, t_units = R > 0 ? adapter_rank_padded(R) / 16 * ((M + 15) / 16) : 0;
    const double step = M <= 16 ? 0.70 : M <= 32 ? 0.85 : M <= 64 ? 1.05 : 1.50;
    const size_t t_bytes = rowtile_t_out_bytes(M, R), one = rowtile_partial_bytes(M, N);
    const int64_t most = chunks < kRowtileMaxSplit ? chunks : kRowtileMaxSplit;
    RowtilePlan best;
    for (int ts = R > 0 ? kRowtileTSlices : 1; ts >= 1; ts /= 2)
        for (int64_t filled = 1; filled <= 4; ++filled) {   // the finest split that fits so many rounds
            int64_t ks = (256 * filled - t_units * ts) / tiles;
            ks = ks < 1 ? 1 : ks > most ? most : ks;
            if (t_bytes + ks * one > room) ks = room > t_bytes ? (int64_t)((room - t_bytes) / one) : 0;
            if (ks < 1) {
                if (R > 0) continue;
                ks = 1;
            }
            const int64_t per_slice = (chunks + ks - 1) / ks;
            ks = (chunks + per_slice - 1) / per_slice;   // (no more slices than that length needs)
            const bool partial = ks > 1 || R > 0;
            const int64_t rounds = (tiles * ks + t_units * ts + 255) / 256;
            double main = 5.0 + (double)(rounds * per_slice) * step + (double)(rounds - 1) * 2.5 +
                          0.07 * (double)(chunks - chunks / ks);
            const double t = R > 0 ? 3.0 + (double)((K / 32 + 32 * ts - 1) / (32 * ts)) * (R > 32 ? 1.7 : 1.2) : 0.0;   // eight waves, four steps at a time
            if (main < t) main = t;
            const double cost = main + (partial ? 3.7 + (double)ks * (double)M * (double)N * 2e-6 : 0.0);
            if (cost < best.cost) {
                best.cost = cost;
                best.ksplit = (int)ks;
                best.parts = 1;
                best.one_launch = false;
                best.t_slices = ts;
                best.partial = partial;
                best.chunks = rounds * per_slice;
            }
            // One slice, the parts of a workgroup added up in LDS, T handed over inside the launch.
            for (int q = R > 0 ? 1 : 2; !slices_only && filled == 1 && q <= (M <= 32 ? 4 : 2); q *= 2) {
                const int64_t row_tiles = (N * q + 127) / 128, per_part = (chunks + q - 1) / q;
                if (row_tiles < kOneLaunchTiles || row_tiles + t_units * ts > 256 || chunks < 4 * q || t_bytes + one > room) continue;
                double alone = 5.0 + (double)per_part * (step + part_step(M, q)) + 0.07 * (double)(chunks - chunks / q);
                if (R > 0) {   // T's workgroups meet in a knockout, the last sums its slices and hands it out
                    double handed = t + 5.5 + 0.35e-3 * (double)(M * adapter_rank_padded(R));
                    for (int64_t blocks = t_units * ts; blocks > 8; blocks = (blocks + 1) / 2) handed += 0.5;
                    if (alone < handed) alone = handed;
                }
                alone += 1.5;
                if (alone < best.cost) {
                    best.cost = alone;
                    best.ksplit = 1;
                    best.parts = q;
                    best.t_slices = ts;
                    best.partial = best.one_launch = R > 0;
                    best.chunks = per_part;
                }
            }
            if (R == 0 && filled == 1 && best.ksplit > 1) {   // one slice writes y itself (whole rows measured 0.84 us a chunk)
                const double alone = 5.0 + (double)((tiles + 255) / 256 * chunks) * step * 1.2 + (double)((tiles + 255) / 256 - 1) * 2.5;
                if (alone < best.cost) {
                    best = RowtilePlan();
                    best.cost = alone;
                    best.chunks = (tiles + 255) / 256 * chunks;
                }
            }
        }
    // One slice, T from a launch in front (4.4 us): where there is no room for partial outputs, and on layers that the told size has no room to split
    // where short rows make the partial outputs cost more than they save (128 x 2048 x 25851 rank 256 81.5 us with three slices, 68.3 so).
    const double t_first = 9.4 + (double)((tiles + 255) / 256 * chunks) * step + (double)((tiles + 255) / 256 - 1) * 2.5;
    if (best.cost == 1e300 || (R > 0 && N % 4 != 0 && uses_rowtile(M, K, N) && t_first < best.cost)) {
        best = RowtilePlan();
        best.chunks = (tiles + 255) / 256 * chunks;
        best.cost = t_first;
    }
    return best;
}
// What a call whose row-tiled launch adds the adapters itself (RowtilePlan::one_launch) has behind its one slice of partial outputs: T,
// and the words of salr_handover.hpp.  Without room for it the summing launch does that.
inline size_t rowtile_pair_bytes(int64_t M, int64_t N, int64_t R, const RowtilePlan& p) {
    if (!p.one_launch) return 0;
    const int64_t Rpad = adapter_rank_padded(R), pairs = (N + 127) / 128 * 8, t_blocks = p.t_slices * (Rpad / 16) * ((M + 15) / 16);
    return round_up_256((size_t)M * (size_t)Rpad * sizeof(uint16_t)) + (size_t)(pairs + t_blocks) * sizeof(uint64_t);
}
uint64_t next_handover_tag();   // 64 bits that no other call of the process has
// The words are exchanged 64 bits at a time, which an address that is no multiple of 8 does not allow.  A call whose workspace starts inside a
// vector, against what it is told to bring, has its launches in front and behind.
inline bool handover_aligned(const void* workspace) { return (uintptr_t)workspace % 16 == 0; }
int handover_polls();           // looks before a workgroup does without what it waits for (salr_set_handover_polls)

// T handed over inside a small-batch kernel's launch (salr_shared_t.hpp): one word per slice of T, 32 ranks and workgroup behind the sums.
struct SharedT {
    uint64_t* words = nullptr;
    uint64_t tag = 0;
    int polls = 0;
    int extra = 0;   // leading workgroups that form T and nothing else
};
constexpr int64_t kSharedMaxRank = 128, kSharedMaxColumns = 8192;
inline int64_t shared_t_blocks(int64_t R) { return kStreamTSlices * (adapter_rank_padded(R) / 32); }
inline size_t shared_t_sums_bytes(int64_t M, int64_t R) {
    return round_up_256((size_t)kStreamTSlices * (size_t)M * (size_t)adapter_rank_padded(R) * sizeof(float));
}
inline size_t shared_t_bytes(int64_t M, int64_t N, int64_t R) {
    return shared_t_sums_bytes(M, R) + (size_t)shared_t_blocks(R) * (size_t)((N + 15) / 16) * sizeof(uint64_t);
}
// Up to 16 tokens on fewer row groups than two a CU (the kernels' variant of one workgroup a CU), A_cat in rows of whole vectors, and as
// many workgroups as T has slices (SharedT::extra: of their own, where they all are one round).  us a call, T from a launch in front / so:
// 4096 x 4096 rank 32 one token 13.2 / 11.1 (4-bit values 13.8 / 11.6), 16 tokens 15.0 / 12.8 (4-bit 15.7 / 13.8; rank 64 15.8 / 13.9);
// 16 x 2048 x 4096 10.5 / 8.8; own workgroups: 8 x 4096 x 1024 11.4 / 8.6, 16 x 4096 x 2048 rank 128 15.0 / 12.5 (14.9 where half of the
// workgroups form T beside their own work).  2:4 masks, layers of 96 MB together, rank 32: 4096 x 4096 16 tokens 13.3 / 11.1, one 11.0 / 9.0,
// 4096 x 1024 13.1 / 9.4 and 10.3 / 6.6, 3072 x 5000 19.3 / 16.9 and 13.8 / 11.4.
inline bool shares_t(int64_t M, int64_t K, int64_t N, int64_t R) {
    return R > 0 && R % 8 == 0 && R <= kSharedMaxRank && M <= 16 && K % 128 == 0 && K <= kSharedMaxColumns && (N + 15) / 16 < 2 * 256 &&
           ((N + 15) / 16 >= shared_t_blocks(R) || (N + 15) / 16 + shared_t_blocks(R) <= 256);
}
inline SharedT shared_t_of(const LinearArgs& a, size_t room) {
    SharedT p;
    if (!shares_t(a.M, a.K, a.N, a.R) || room < shared_t_bytes(a.M, a.N, a.R) || (uintptr_t)a.a_cat % 16 != 0 || !handover_aligned(a.t)) return p;
    p.words = reinterpret_cast<uint64_t*>(reinterpret_cast<char*>(a.t) + shared_t_sums_bytes(a.M, a.R));
    p.tag = next_handover_tag();
    p.polls = handover_polls();
    if ((a.N + 15) / 16 + shared_t_blocks(a.R) <= 256) p.extra = (int)shared_t_blocks(a.R);
    return p;
}
inline size_t rowtile_workspace_bytes(int64_t M, int64_t K, int64_t N, int64_t R) {
    const int ks = rowtile_ksplit(M, K, N);
    return rowtile_t_bytes(M, K, R) + (ks > 1 ? round_up_256((size_t)ks * (size_t)M * (size_t)N * sizeof(float)) : 0);
}

// The linear on 2:4-masked weights (sparse matrix-core instructions, no decode stage): tiles of 128 rows, rowtile_ksplit and its
// workspace; other shapes go through launch_linear.
inline bool uses_2of4_kernel(int64_t M, int64_t K, int64_t N) {
    return rowtile_possible(M, K) && !(N % 4 != 0 && N < 64 * 128);
}
// The barrier-free one of its kernels: up to 16 tokens it is ahead where the call is short (layers of up to 2^25 elements: no reducing launch, no
// split of K) and, on any layer, up to 4 tokens (little X to pull through the L2 per workgroup); measured on the Llama-3 shapes.
inline bool uses_2of4_stream(int64_t M, int64_t K, int64_t N) {
    return uses_2of4_kernel(M, K, N) && M <= 16 && (M <= 4 || N * K <= (int64_t(1) << 25));
}
// above 128 tokens: a tiled GEMM on the sparse MFMA (k-steps of 64 columns, four outputs per store); its workspace is
// the T part of the large-batch layout, which the general call's workspace contains
// Taken where its tiles fill the chip without crowding it (measured on the Llama-3 shapes: 14 to 32 % ahead of the
// decode + dense GEMM path there): >= 192 tiles of 256 x 256 (one workgroup per CU); on layers of >= 8192 rows from
// 128 tiles of 128 x 128 on; on smaller layers with 192 to 320 of them (about one workgroup per CU: with two the
// 128 x 128 tiles, which read more LDS per flop, are level with the other path, and below 192 the chip is not full).
constexpr int64_t kGemm2of4BigTilesMin = 192;
inline bool uses_2of4_gemm(int64_t M, int64_t K, int64_t N) {
    if (!(M > kRowtileMaxM && K >= 64 && K % 64 == 0 && N % 4 == 0)) return false;
    const int64_t big = ((M + 255) / 256) * ((N + 255) / 256), small = ((M + 127) / 128) * ((N + 127) / 128);
    if (big >= kGemm2of4BigTilesMin) return true;
    return N >= 8192 ? small >= 128 : (small >= 192 && small <= 320);
}
hipError_t launch_check_2of4(const uint32_t* bitmap, int64_t rows, int64_t cols, uint32_t* flag, hipStream_t stream);

// decode-sized batches (M <= 16, K % 128 == 0, 12288 <= K <= 32768): the streaming kernel that reads every bitmap word once
bool linear_slice_takes(int64_t M, int64_t K, int64_t N);
// Shapes that launch_linear sends down the two-stage path when the workspace has room for the decoded copy
inline bool linear_takes_twostage(int64_t M, int64_t K, int64_t N) {
    return M > kStreamMaxM && !uses_rowtile(M, K, N) && uses_twostage(M, K);
}
// Where the told size has room for a slice table behind the rest of the workspace.  A call without a table of the caller's builds
// one there where the small-batch streaming kernel runs on rows of whole chunks behind a launch for T (R > 0), which builds it on the
// side.  (The long-row kernel reads a caller's table but gains less from it than reading the bitmap a second time costs: 70B
// down_proj M = 1, kernel + launch for T 87.3 us without, 89.3 us with.)  The row-tiled kernel reads the bitmap left of its slices
// itself; its calls have these bytes so that the size a caller was told stays what it was, as room for partial outputs.
inline bool reserves_slice_table(int64_t M, int64_t K, int64_t N, int64_t R) {
    if (R <= 0 || M <= 0 || N <= 0 || K < 128 || K % 128 != 0) return false;
    if (uses_rowtile(M, K, N)) return kSliceTableSlices % rowtile_ksplit(M, K, N) == 0;
    if (linear_slice_takes(M, K, N)) return false;
    return M <= kStreamMaxM;
}
inline size_t linear_workspace_bytes_without_table(int64_t M, int64_t K, int64_t N, int64_t R);
// Workspace the linear needs: the small-batch path keeps fp32 split-K partials of T; the others see above.
inline size_t linear_workspace_bytes(int64_t M, int64_t K, int64_t N, int64_t R) {
    const size_t b = linear_workspace_bytes_without_table(M, K, N, R);
    return reserves_slice_table(M, K, N, R) ? b + round_up_256(slice_table_bytes(N)) : b;
}
inline size_t linear_workspace_bytes_without_table(int64_t M, int64_t K, int64_t N, int64_t R) {
    if (M <= 0 || N <= 0) return 0;
    if (uses_rowtile(M, K, N)) return rowtile_workspace_bytes(M, K, N, R);
    if (M <= kStreamMaxM)
        return R > 0 ? round_up_256((size_t)kStreamTSlices * (size_t)M * (size_t)adapter_rank_padded(R) * sizeof(float)) : 0;
    size_t b = twostage_dense_offset(M, K, R);
    if (uses_twostage(M, K)) {
        b += round_up_256((size_t)N * (size_t)K * sizeof(uint16_t));
        const int ks = dense_ksplit(M, K, N);
        if (ks > 1) b += round_up_256((size_t)ks * (size_t)M * (size_t)N * sizeof(float));
    }
    return b;
}

// Times of a call of up to 64 tokens in the small-batch kernels (the long-row kernel where it takes the shape) and in the row-tiled one,
// microseconds, the weight coming from memory.  Small-batch: T's launch in front, then rounds of workgroups of 16 rows, one per CU (up to
// 16 tokens from 512 workgroups on two beside each other, which share its time), each as long as the chunks of the longest of its eight
// slices.  Row-tiled: the plan's own cost, corrected for what the ranks cost the summing launch and for its chunks.
struct SmallBatchPrices {
    double call, t, t_rank;          // launch; T, and its 32 ranks of 16 tokens
    double round, chunk[3], token;   // a round, a chunk up to 16, 32 and 64 tokens, and what 16 tokens add to it
    double bank;                     // that, where rows of X are a multiple of 4 KB apart
    double pairs, ragged;            // factors of a chunk: two workgroups on a CU; rows of X and bitmap that are no whole chunks, up to 32 tokens
    double long_call, long_chunk;    // the long-row kernel
    double tiled, tiled_rank, tiled_chunk[3];
    double tiled_full;               // what a chunk costs more whose 4-bit values outgrow the vectors that are asked for first
    double density, pair_round;      // what a chunk costs more from 0 to 100 % nonzeros (0 at 50 %), and a round of two workgroups on a CU
    double later_round;              // what a round after the first costs more, from 17 tokens on
};
// Fitted, with rowtile_plan's model as it is, on 3571 calls of 1 to 64 tokens on layers 128 to 28672 wide, rank 0 to 128, 30 to 70 % zeros,
// with and without a table, timed in both kernels: with these prices 30 calls are more than 3 % slower than before the row-tiled kernel
// took any of them, at most by 1.21 (with thresholds on K, N and R: 172, at most by 1.92).  later_round from 14.1 us of 32 x 1024 x 7680 rank 16
// (10.9 row-tiled) against 9.3 in one round (1024 x 3500).
constexpr SmallBatchPrices kPrices = {0.82, 2.71, 0.39, 1.45, {1.29, 1.53, 2.39}, 0.44, 1.69, 1.9, 1.26, 3.4, 0.76, -0.71, 0.54, {-0.11, -0.27, -0.13}, 0.0, 0.0, 0.0, 1.0};
// The same on 4-bit values of 17 to 64 tokens: of 15678 calls on full layers and thin ones 22 are more than 3 % slower than in the
// small-batch kernel, at most by 1.11 (thresholds: 80 of 1281, by 2.02).
constexpr SmallBatchPrices kPricesOfCodes = {0.53, 2.31, 0.5, 2.7, {2.04, 2.07, 2.77}, 0.28, 1.62, 1.3, 1.0, 0.0, 1.0, -0.55, 1.02, {0.41, 0.09, 0.34}, 0.0, 0.0, 0.0, 0.0};
// And of up to 16, where the share of nonzeros decides: a row-tiled lane asks for two vectors of 32 codes at once, four cover a
// row's piece of 128 columns if its values and its place in the first vector come to 128 at most: nearly always at 70 % nonzeros, hardly ever
// at 80 %.  Two of the small-batch kernel's workgroups share a CU, and what counts is how many of them one CU gets (12 tokens, 80 %, us a
// call, it / row-tiled: 8192 x 12115, three a CU, 53.5 / 59.5; 9600 x 12912, four a CU, 81.9 / 72.1).  Of 15555 calls at 30 to 100 % 64 are more than 3 % slower than in the small-batch
// kernel, at most by 1.16; without these terms 178, by 1.19 (1 x 8192 x 20000 at 80 % 82.4 us instead of 73.6).
constexpr SmallBatchPrices kPricesOfFewCodes = {0.53, 2.31, 0.5, 2.7, {1.97, 0.0, 0.0}, 0.42, 1.62, 1.41, 1.0, 0.0, 1.0, -3.44, 0.86, {0.46, 0.0, 0.0}, 0.43, 0.55, 0.52, 0.0};

inline double small_batch_price(const SmallBatchPrices& c, bool codes, int64_t M, int64_t K, int64_t N, int64_t R, double nonzeros = 0.5) {
    const int64_t groups = (N + 15) / 16, chunks = ((K + 127) / 128 + 7) / 8, m_tiles = (M + 15) / 16;
    const bool pairs = M <= 16 && groups >= 512, long_rows = !codes && linear_slice_takes(M, K, N);
    double chunk = c.chunk[M <= 16 ? 0 : M <= 32 ? 1 : 2] + c.token * (double)M / 16.0 * (K % 2048 == 0 ? c.bank : 1.0);
    if (pairs) chunk *= c.pairs;
    if (K % 128 != 0 && M <= 32) chunk *= c.ragged;
    if (long_rows) chunk *= c.long_chunk;
    chunk += c.density * (nonzeros - 0.5);
    // (pairs: half of what the last round leaves idle is won back; of 4-bit values what an odd workgroup on a CU leaves)
    const double per_cu = (double)((groups + 255) / 256);
    const double rounds = !pairs ? per_cu : codes ? 0.5 * per_cu : 0.5 * ((double)((groups + 511) / 512) + (double)groups / 512.0);
    const double t = R > 0 ? c.t + c.t_rank * (double)(m_tiles * ((R + 31) / 32)) : 0.0;
    const double later = M > 16 ? c.later_round * (rounds - 1.0) : 0.0;
    return c.call + (long_rows ? c.long_call : 0.0) + t + later + rounds * (c.round + (pairs ? c.pair_round : 0.0) + chunk * (double)chunks);
}
// p: a plan of slices over workgroups, which the prices were fitted on.  (Where parts in one launch are faster still, so is the call.  Likewise
// small_batch_price has T's launch in front in it, which calls of shares_t are without: of those only 4-bit values of up to 16 tokens on rows of up
// to 4096 columns ask for prices.)
inline double rowtile_price(const SmallBatchPrices& c, const RowtilePlan& p, int64_t M, int64_t R, double nonzeros = 0.5) {
    const double full = nonzeros <= 0.7 ? 0.0 : nonzeros >= 0.8 ? 1.0 : (nonzeros - 0.7) * 10.0;   // share of the chunks that pay tiled_full
    return p.cost + c.tiled + c.tiled_rank * (double)((R + 31) / 32) +
           (c.tiled_chunk[M <= 16 ? 0 : M <= 32 ? 1 : 2] + c.tiled_full * full) * (double)p.chunks;
}
// The same kernel beyond those shapes (any K that is a multiple of 32, any N, fewer tokens), where the call's workspace has room for
// its partial outputs (salr_linear_workspace_bytes_fastest) and it has the lower price; from 65 tokens on wherever it can (99 x 7648 x
// 12288 140 us on the decoding path, 59 here).  Layers of a few microseconds stay with the small-batch kernel, which wants no launch to
// sum up, whatever the models say of them (us a call, it / this kernel: 1 x 4096 x 4096 12.1 / 14.6, 13 x 1536 x 3072 6.2 / 9.2; larger
// ones: 2 x 2560 x 26583 27.6 / 23.8, 3 x 7616 x 1792 22.6 / 15.3, 16 x 7168 x 6932 36.6 / 25.9, 59 x 3008 x 16384 79.7 / 34.3).
inline bool rowtile_can(int64_t M, int64_t K, int64_t N) {
    if (M > kRowtileMaxM || K < 128 || K % 32 != 0 || K > kRowtileMaxColumns || N < 128) return false;
    return !(M <= 8 && K > 24576 && N > 4096);   // 1 x 28672 x 8192: 83.5 in the long-row kernel, 92 here (three slices on 192 CUs)
}
inline bool rowtile_wide(int64_t M, int64_t K, int64_t N, int64_t R) {
    if (!rowtile_can(M, K, N)) return false;
    if (M > kStreamMaxM) return true;
    if (M <= 16 && !(N * K >= (18 << 20) || N >= 16384 || K >= 5376)) return false;
    // Up to 16 tokens with adapters no prices are asked.  While the small-batch kernel had a launch for T in front everywhere it was ahead by more
    // than 3 % in 211 of 9119 calls without a table, and a caller's table gains this kernel more (1 x 14336 x 4096 27.1 us without, 22.5 with).  Where
    // it forms T in its own launch (shares_t) either is ahead by up to a tenth (us a call, it / this one: 8 x 5120 x 4096 12.3 / 13.2, 8 x 6144 x 4096
    // 13.3 / 14.8, 8 x 8064 x 3000 14.3 / 15.5, 16 x 5376 x 2048 rank 128 14.2 / 15.8; 16 x 5120 x 4096 13.5 / 14.0; 16 x 8192 x 1024 15.9 / 13.8,
    // 16 x 8192 x 2048 16.1 / 14.7, 16 x 8064 x 3000 rank 128 19.9 / 18.6), and with more row groups than CUs this one is: 8 x 4608 x 5120 20.0 / 13.0,
    // 16 x 7168 x 7168 33.8 / 21.8.
    if (M <= 16 && R > 0) return true;
    if (M > 16 && M <= 32 && !(K >= 1024 || N >= 8192)) return false;
    return rowtile_price(kPrices, rowtile_plan(M, K, N, R, SIZE_MAX, true), M, R) < small_batch_price(kPrices, false, M, K, N, R);
}
// Whether the told size is all that the kernel ever uses: where that one has always had it with a split of K, so that the split, and
// with it every bit of the result, does not depend on what a caller brings beyond it.  (N % 4 != 0: the told size has no room for
// a split, the fastest one has: 64 x 4096 x 14335 at rank 32 52.3 us without, 33.3 with (14336: 31.7), 16 x 8192 x 8193 61.8 / 32.6;
// 4-bit values, 37 x 17536 x 10315: 273 / 106, the small-batch kernel 170.)
inline bool rowtile_on_told_size(int64_t M, int64_t K, int64_t N) { return uses_rowtile(M, K, N) && N % 4 == 0; }
inline RowtilePlan rowtile_plan_of(int64_t M, int64_t K, int64_t N, int64_t R, bool slices_only = false) {
    return rowtile_plan(M, K, N, R, rowtile_on_told_size(M, K, N) ? linear_workspace_bytes(M, K, N, R) : SIZE_MAX, slices_only);
}
inline size_t rowtile_plan_bytes(int64_t M, int64_t K, int64_t N, int64_t R, const RowtilePlan& p) {
    return p.partial ? round_up_256(rowtile_t_out_bytes(M, R) + (size_t)p.ksplit * rowtile_partial_bytes(M, N)) : rowtile_t_bytes(M, K, R);
}
// With this much a call of rowtile_wide's shapes goes through the kernel: what its slices need, parts in one launch or not.
inline size_t rowtile_bytes(int64_t M, int64_t K, int64_t N, int64_t R) {
    const size_t slices = rowtile_plan_bytes(M, K, N, R, rowtile_plan_of(M, K, N, R, true)), b = rowtile_plan_bytes(M, K, N, R, rowtile_plan_of(M, K, N, R));
    return slices > b ? slices : b;
}
inline size_t rowtile_bytes_fastest(int64_t M, int64_t K, int64_t N, int64_t R) {   // with room for T to be handed over
    const RowtilePlan p = rowtile_plan_of(M, K, N, R);
    const size_t least = rowtile_bytes(M, K, N, R), b = rowtile_plan_bytes(M, K, N, R, p) + rowtile_pair_bytes(M, N, R, p);
    return b > least ? b : least;
}
// The plan of a call that brings `room` bytes: the one above, or the one that fits the told size.
inline RowtilePlan rowtile_plan_in(int64_t M, int64_t K, int64_t N, int64_t R, size_t room) {
    if (rowtile_on_told_size(M, K, N) || room >= rowtile_bytes(M, K, N, R)) return rowtile_plan_of(M, K, N, R);
    return rowtile_plan(M, K, N, R, linear_workspace_bytes(M, K, N, R));
}
// Whether its launch hands T over and adds the adapters itself: where the plan has it so, with room for the words behind the rest.
inline bool rowtile_hands_over(int64_t M, int64_t K, int64_t N, int64_t R, const RowtilePlan& p, size_t room) {
    return p.one_launch && room >= rowtile_plan_bytes(M, K, N, R, p) + rowtile_pair_bytes(M, N, R, p);
}
inline bool linear_takes_rowtile(int64_t M, int64_t K, int64_t N, int64_t R, size_t room) {
    return uses_rowtile(M, K, N) || (rowtile_wide(M, K, N, R) && room >= rowtile_bytes(M, K, N, R));
}

// QSALR calls of up to 128 tokens that take the row-tiled kernel on the codes, with room for its partial outputs.  More than 64
// tokens have no other kernel that reads codes; fewer take the small-batch kernel on layers of a few microseconds and the lower price on
// others (us a call, that kernel / this one: 33 x 896 x 1260 10.5 / 19.9, 1 x 8192 x 8192 32 / 41, 16 x 2048 x 8192 14.6 / 16.5; 16 x 4096 x
// 14336 36.4 / 30.7, 1 x 13824 x 5120 61 / 36, 17 x 5696 x 4549 64 / 23).  Rows that are no whole chunks have this kernel or none.
inline bool qsalr_takes_rowtile(int64_t M, int64_t K, int64_t N, int64_t R, int64_t nnz) {
    if (nnz <= 0 || K <= 0 || !(uses_rowtile(M, K, N) || rowtile_can(M, K, N))) return false;
    if (M > kStreamMaxM) return true;
    const bool large = M > 32 || (M > 16 ? K >= 1024 || N >= 8192 : N * K >= (18 << 20) || N >= 16384 || K >= (R > 0 ? 5376 : 8192));
    if (!large || K % 128 != 0) return large;
    const SmallBatchPrices& prices = M <= 16 ? kPricesOfFewCodes : kPricesOfCodes;
    const double nonzeros = (double)nnz / ((double)N * (double)K);
    return rowtile_price(prices, rowtile_plan_of(M, K, N, R, true), M, R, nonzeros) <
           small_batch_price(prices, true, M, K, N, R, nonzeros);
}

// The operand-order path's workspace: T, what a product of its own needs for it, the weight, then the partial outputs of a split
// contraction as far as there is room (gemm_plan).
inline size_t frag_base_bytes(int64_t M, int64_t K, int64_t N, int64_t R) {
    return round_up_256(frag_weight_offset(M, K, R) + frag_weight_bytes(K, N, R));
}
inline bool linear_takes_frag(int64_t M, int64_t K, int64_t N, int64_t R, size_t room) {
    return M > kStreamMaxM && !uses_rowtile(M, K, N) && uses_frag(M, K) && room >= frag_base_bytes(M, K, N, R);
}
// Workspace with which the layer is fastest (salr_linear_workspace_bytes_fastest).
inline size_t linear_workspace_bytes_fastest(int64_t M, int64_t K, int64_t N, int64_t R) {
    const size_t told = linear_workspace_bytes(M, K, N, R);
    if (N <= 0 || rowtile_on_told_size(M, K, N)) return told;
    if (uses_rowtile(M, K, N) || rowtile_wide(M, K, N, R)) {
        const size_t b = rowtile_bytes_fastest(M, K, N, R);
        return b > told ? b : told;
    }
    if (M <= kStreamMaxM || !uses_frag(M, K)) return told;
    const size_t b = frag_base_bytes(M, K, N, R) + gemm_partial_bytes(M, N, gemm_plan(M, K + adapter_rank_padded(R), N).ksplit);
    return b > told ? b : told;
}

// The least the layer runs with: where the preferred path decodes the weight into the workspace (large batches), the
// fused kernel needs the adapter part only.
inline size_t linear_workspace_bytes_lean(int64_t M, int64_t K, int64_t N, int64_t R) {
    if (M <= 0 || N <= 0) return 0;
    if (!uses_rowtile(M, K, N) && M > kStreamMaxM && uses_twostage(M, K)) return twostage_dense_offset(M, K, R);
    return linear_workspace_bytes(M, K, N, R);
}

// Backward pass of the layer: dx [M, K], da [K, R], db [R, N]; any of them may be null (not computed)
size_t linear_backward_workspace_bytes(int64_t M, int64_t K, int64_t N, int64_t R, bool want_dx, bool want_dadb);
hipError_t launch_linear_backward(const uint16_t* x, const uint16_t* dy, int64_t M, int64_t K, int64_t N,
                                  const uint32_t* bitmap, const uint16_t* values, const uint32_t* row_offsets,
                                  const uint16_t* a_cat, const uint16_t* b_cat, int64_t R, uint16_t* dx, uint16_t* da,
                                  uint16_t* db, void* workspace, hipStream_t stream);

// QSALR: the packed values as 4-bit NormalFloat codes, one bf16 scale per 64 values
hipError_t launch_nf4_quantize(const uint16_t* values, int64_t count, uint8_t* codes, uint16_t* scales, hipStream_t stream);
hipError_t launch_nf4_dequantize(const uint8_t* codes, const uint16_t* scales, int64_t count, uint16_t* out, hipStream_t stream);
// bytes of the dequantised packed values at the start of the QSALR layer's workspace (16-byte vectors, 256-byte aligned)
inline size_t qsalr_values_bytes(int64_t nnz) { return round_up_256((size_t)((nnz + 7) / 8 * 8) * sizeof(uint16_t)); }
// QSALR at small batches (M <= 64, K a multiple of 128, nnz > 0): the streaming kernel that reads the 4-bit codes itself.
// Its workspace: the split-K partials of T (with adapters), then the call's slice table; args.t and args.slice_table
// point at the two, args.values is not used.
bool linear_nf4_takes(int64_t M, int64_t K, int64_t N, int64_t nnz);
size_t linear_nf4_table_offset(int64_t M, int64_t R);
size_t linear_nf4_workspace_bytes(int64_t M, int64_t N, int64_t R);
hipError_t launch_linear_nf4(const LinearArgs& args, const uint8_t* codes, const uint16_t* scales, int64_t nnz,
                             hipStream_t stream, const TimingEvents& ev);

// QSALR: decode from the 4-bit codes (the row-per-workgroup decode kernel's limits: cols % 8 == 0, 16-byte aligned out)
bool decode_nf4_takes(int64_t rows, int64_t cols, int64_t nnz, const void* codes, const void* out);
hipError_t launch_decode_nf4(const uint32_t* bitmap, const uint8_t* codes, const uint16_t* scales, int64_t nnz,
                             const uint32_t* row_offsets, int64_t rows, int64_t cols, uint16_t* out, hipStream_t stream);
hipError_t launch_linear(const LinearArgs& args, hipStream_t stream);
// count bf16 zeros (+0.0) at out
hipError_t launch_fill_zero(uint16_t* out, int64_t count, hipStream_t stream);
hipError_t launch_linear_stream(const LinearArgs& args, hipStream_t stream, const TimingEvents& ev);
hipError_t launch_linear_slice(const LinearArgs& args, hipStream_t stream, const TimingEvents& ev);
hipError_t launch_linear_frag(const LinearArgs& args, hipStream_t stream, const TimingEvents& ev);
hipError_t launch_linear_twostage(const LinearArgs& args, hipStream_t stream, const TimingEvents& ev);
// the same shapes without a decoded copy of the weight: decode stage and MFMA stage in one kernel (K % 64 == 0)
hipError_t launch_linear_tiled(const LinearArgs& args, hipStream_t stream, const TimingEvents& ev);
hipError_t launch_linear_rowtile(const LinearArgs& args, hipStream_t stream, const TimingEvents& ev);
hipError_t launch_linear_2of4(const LinearArgs& args, hipStream_t stream, const TimingEvents& ev);
void launch_sparse_gemm(const LinearArgs& args, uint16_t* wf, bool narrow, bool with_t, const TimingEvents& ev, hipStream_t stream);
hipError_t launch_gemm_2of4(const LinearArgs& args, hipStream_t stream, const TimingEvents& ev);
// split-K partials of T = X * A_cat (small batches): fp32 [kStreamTSlices, M, Rpad] at the start of the workspace
void launch_adapter_partial(const LinearArgs& args, hipStream_t stream);
// the same into `partial` [kStreamTSlices, M, Rpad] (no slice table)
void launch_adapter_partial_to(const LinearArgs& args, float* partial, hipStream_t stream);
// T = X * A_cat in bf16 [M, Rpad] in one launch (see adapter_t_own_product)
void launch_adapter_t_direct(const uint16_t* x, int64_t M, int64_t K, const uint16_t* a_cat, int R, int Rpad, uint16_t* t,
                             hipStream_t stream);
// T = X * A_cat in bf16 [M, Rpad] at the start of the workspace (every path with M > kStreamMaxM)
void launch_adapter_t(const LinearArgs& args, hipStream_t stream);
// The two low-rank intermediates of the backward pass, bf16: job 0 is T' = in [M, C] * factor [R, C]^T, job 1 is T = in [M, C] *
// factor [C, R]; each [M, Rpad] in t and, unless null, transposed [Rpad, M] in t_t.  A job whose `in` is null is left out.
// C % 32 == 0.
struct LowRankJob {
    const uint16_t* in;
    const uint16_t* factor;
    int64_t C;
    uint16_t* t;
    uint16_t* t_t;
};
void launch_backward_t(const LowRankJob& dy_b, const LowRankJob& x_a, int64_t M, int R, hipStream_t stream);
// the transpose of the weight in operand order, the rank blocks of A_cat [cols, R] (null with R == 0) behind it:
// frag_weight_bytes(rows, cols, R) bytes (rows % 64 == 0, cols % 32 == 0); the two jobs (see launch_backward_t; R % 8 == 0) in the same launch
hipError_t launch_decode_transposed_frags(const uint32_t* bitmap, const uint16_t* values, const uint32_t* row_offsets, int64_t rows,
                                          int64_t cols, const uint16_t* a_cat, int R, uint16_t* wf, const LowRankJob& dy_b,
                                          const LowRankJob& x_a, int64_t M, hipStream_t stream);
// Products that contract over the rows of in [M, C] (M % 32 == 0) against s_t [Rpad, M]: the adapter gradients, bf16, job 0 to
// out [C, R], job 1 to out [R, C].  A job that is not wanted has C = 0.  partial: room for ksplit fp32 slices
// [C, Rpad] of each job; tn_ksplit picks the split of M (about four workgroups per CU over both jobs, at least two
// steps of 32 rows each).  words: ksplit per 64 columns of each job, for slices that are summed in the launch that forms them, or null.
struct RowProducts {
    const uint16_t* in[2];
    const uint16_t* s_t[2];
    int64_t C[2];
    uint16_t* out[2];
    int64_t M;
    int R, Rpad, ksplit;
    float* partial;
    uint64_t* words;
    uint64_t tag;
};
constexpr int row_product_blocks(int64_t C) { return (int)((C + 63) / 64); }   // of columns
// Slices of the rows at most where the gradients are beside the stage: whoever sums them reads them all.  (With the 32 of a launch of their
// own 2272 x 1216 x 640 at rank 32 went 33 -> 41 us; with eight 29.)
constexpr int kBesideSlices = 8;
// Whether they are: on tiles of the stage g of which two fit a CU, where the stage is long enough to hide them, by what they read at 3 TB/s and what
// the stage multiplies at 1100 TFLOP/s, and up to 96 ranks.  Above 64 their workgroups go through their rows three times; where they then take
// longer than the stage and it fills half of the chip's places or more, but not all at once, those that find no place with it start behind it, and two
// launches are as fast or faster: 768 x 3072 x 768 at rank 96 45.4 us beside, 40.8 so, 768 x 2048 x 2048 54.0 and 48.9 (against 1024 x 2048 x 2048,
// where all find a place at once, 43.5 and 58.9).  Of 230 steps (128 to 3000 tokens, ranks 24 to 96) ten are 1 to 2 % slower beside the stage than
// in two launches, the geometric mean 1.12 faster; at rank 128 0.86 (448 x 5248 x 640) to 1.10 (608 x 2688 x 13440).
inline bool gradients_beside(int64_t M, int64_t K, int64_t N, const GemmPlan& g, const RowProducts& p) {
    const double gradients = (double)M * (double)(p.C[0] + p.C[1]) * 2.0 * (p.Rpad / 32) / 3e6, stage = 2.0 * (double)M * (double)N * (double)K / 1.1e9;
    if (g.mt > 128 || p.Rpad > 96 || (gradients >= 20.0 && gradients >= 0.85 * stage)) return false;
    if (p.Rpad <= 64 || gradients < stage) return true;
    const int64_t places = 256 * (g.mt * g.nt <= 64 * 64 ? 4 : g.mt * g.nt <= 128 * 128 ? 3 : 2);
    const int64_t of_stage = (M + g.mt - 1) / g.mt * ((N + g.nt - 1) / g.nt) * g.ksplit;
    const int64_t theirs = (row_product_blocks(p.C[0]) + row_product_blocks(p.C[1])) * (int64_t)(p.ksplit < kBesideSlices ? p.ksplit : kBesideSlices);
    return 2 * of_stage < places || of_stage > places || of_stage + theirs <= places;
}
inline int tn_ksplit(int64_t C0, int64_t M, int64_t C1 = 0) {
    const int64_t blocks = (C0 + 63) / 64 + (C1 + 63) / 64, steps = M / 32;
    int s = 1;
    while (s < 64 && blocks * s * 2 <= 1024 && steps / (s * 2) >= 2) s *= 2;
    return s;
}
void launch_row_products(const RowProducts& products, hipStream_t stream);   // words == nullptr
// x [M, K] bf16 times the transpose of a_t [Rpad, K] bf16 (Rpad % 32 == 0, K % 32 == 0), K split over `ksplit`
// slices: bf16 t [M, Rpad] (one slice, !keep_fp32) or fp32 partial [ksplit, M, Rpad]; columns from `ranks` on as zeros
void launch_tall_product(const uint16_t* x, int64_t M, int64_t K, const uint16_t* a_t, int Rpad, int ranks, int ksplit, uint16_t* t,
                         float* partial, bool keep_fp32, hipStream_t stream);
// a_t [Rpad, K] = A_cat [K, R]^T, rows R .. Rpad - 1 zero
void launch_adapter_transpose(const uint16_t* a_cat, int64_t K, int R, int Rpad, uint16_t* a_t, hipStream_t stream);
// out [C, R] = in [R, C]^T (bf16); R <= 65535 * 32
void launch_transpose_bf16(const uint16_t* in, int64_t R, int64_t C, uint16_t* out, hipStream_t stream);
// y [M, N] = x [M, K] * W^T (+ t [M, Rpad] * B_cat) with W and B_cat in operand order (salr_gemm.hip).  beside (or null; words set): products
// to be formed in the same launch where two of its workgroups fit a CU; whether they were.
bool launch_frag_gemm(const uint16_t* x, int64_t M, int64_t K, int64_t N, const uint16_t* wf, const uint16_t* t, int Rpad,
                      uint16_t* y, float* partial, size_t partial_room, const TimingEvents& ev, hipStream_t stream, const RowProducts* beside);
// y [M, N] = x [M, K] * wd [N, K]^T (+ t [M, Rpad] * b_cat [R, N], pitch N, when R > 0): the dense MFMA stage with its
// tile choice; K % 64 == 0; partial holds dense_ksplit(M, K, N) fp32 copies of y when that is > 1
void launch_dense_stage(const uint16_t* x, int64_t M, int64_t K, int64_t N, const uint16_t* wd, const uint16_t* t,
                        const uint16_t* b_cat, int R, int Rpad, uint16_t* y, float* partial, const TimingEvents& ev,
                        hipStream_t stream);
// out[i] = bf16(sum over z < ksplit of partial[z * splitk_slice(count) + i]); with valid < cols the columns from `valid` on of out's
// rows of `cols` are zeros instead
void launch_splitk_reduce(const float* partial, int64_t count, int ksplit, uint16_t* out, hipStream_t stream, int cols = 0, int valid = 0);

}  // namespace salr
