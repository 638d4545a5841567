// Small device helpers shared by the linear-layer kernels.
#pragma once

#include "salr_device.hpp"

namespace salr {

// fp32 -> bf16, round to nearest even; NaN stays a quiet NaN.
__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (uint16_t)((u >> 16) | 0x0040u);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float bf16_bits_to_f32(uint32_t b) { return __uint_as_float(b << 16); }

__device__ __forceinline__ bf16x8 as_bf16x8(const uint4& q) { return __builtin_bit_cast(bf16x8, q); }

// Eight ranks of B_cat from rank r0 on, as an MFMA operand, without those that fill the padded ones: they are read from the last rank and meet
// zeros of T, but an infinite entry would make NaN of that.  At the operand's use and only where R is no multiple of 32, which is the same for
// the whole launch: where the loads are packed it made the small-batch kernels wait for them (4096 x 4096, 16 tokens, 4 to 13 % of a call).
// Behind a loop over rank steps, not in it: the next step's requests would wait for the test.  So it costs ranks such as 16 or 61 up to 0.1 us a call
// (16 x 4096 x 4096, R 16: 12.75 / 12.83; 12 x 8448 x 2048, R 61: 17.3 / 17.4) and multiples of 32 nothing.
__device__ __forceinline__ uint4 ranks_below(uint4 b, int r0, int R) {
    if (R % 32 != 0) {
        asm volatile("" : "+v"(r0));   // (here: what follows is not worked out ahead and kept through a stream)
        const int n = R - r0;
        b.x = n > 1 ? b.x : n > 0 ? b.x & 0xFFFFu : 0u;
        b.y = n > 3 ? b.y : n > 2 ? b.y & 0xFFFFu : 0u;
        b.z = n > 5 ? b.z : n > 4 ? b.z & 0xFFFFu : 0u;
        b.w = n > 7 ? b.w : n > 6 ? b.w & 0xFFFFu : 0u;
    }
    return b;
}

// One block of 256 threads builds the slice-table entries of 32 rows (see kSliceTableSlices in salr_internal.hpp):
// eight lanes per row, one per slice; a lane walks the chunks of its slice (16 bytes = 128 columns a load, four loads
// in flight), then an exclusive scan over the row's eight lanes turns slice counts into value indices.  Used by
// salr_build_slice_table and, for calls without a table of the caller's, by extra blocks of the small-batch adapter
// pre-kernel.  (Two other shapes were measured and were slower inside the pre-kernel: a wave per row with wave scans,
// and the rows staged through LDS.)
constexpr int kSliceTableRowsPerBlock = 32;

__device__ __forceinline__ void slice_table_block(const uint32_t* __restrict__ bitmap, const uint32_t* __restrict__ row_offsets,
                                                  int64_t N, int64_t K, uint32_t* __restrict__ table, int64_t block,
                                                  int tid) {
    constexpr int kSlices = 8;
    const int64_t n = block * kSliceTableRowsPerBlock + (tid >> 3);
    const int w = tid & 7;
    const int64_t wpr = K >> 5;
    const int64_t chunks = (wpr + 3) / 4;
    const int64_t c_begin = chunks * w / kSlices, c_end = chunks * (w + 1) / kSlices;
    uint32_t count = 0, longest = 0;
    if (n < N) {
        const uint32_t* brow = bitmap + n * wpr;
        if ((wpr & 3) == 0) {
#pragma unroll 4
            for (int64_t c = c_begin; c < c_end; ++c) {
                const uint4 q = *reinterpret_cast<const uint4*>(brow + 4 * c);
                const uint32_t len = __popc(q.x) + __popc(q.y) + __popc(q.z) + __popc(q.w);
                count += len;
                longest = len > longest ? len : longest;
            }
        } else {
            for (int64_t c = c_begin; c < c_end; ++c) {
                uint32_t len = 0;
                for (int64_t q = 4 * c; q < 4 * c + 4 && q < wpr; ++q) len += __popc(brow[q]);
                count += len;
                longest = len > longest ? len : longest;
            }
        }
    }
    uint32_t incl = count;   // the lanes of a row are consecutive
#pragma unroll
    for (int o = 1; o < kSlices; o <<= 1) {
        const uint32_t up = __shfl_up(incl, o, kSlices);
        if (w >= o) incl += up;
    }
    if (n < N) {
        uint2 e;
        e.x = row_offsets[n] + (incl - count);
        e.y = longest;
        *reinterpret_cast<uint2*>(table + (n * kSlices + w) * 2) = e;
    }
}

// per nibble with two set bits at p0 < p1: p0 | p1 << 2 (the index field of the sparse MFMA)
__device__ __forceinline__ uint32_t index_codes_2of4(uint32_t w) {
    const uint32_t ones = 0x11111111u;
    const uint32_t b0 = w & ones, b1 = (w >> 1) & ones, b2 = (w >> 2) & ones, b3 = (w >> 3) & ones;
    const uint32_t n0 = b0 ^ ones, n1 = b1 ^ ones, n2 = b2 ^ ones;
    return (n0 & b1) | ((n0 & n1) << 1) | ((b3 | n2) << 2) | ((b3 | b2) << 3);
}

}  // namespace salr
