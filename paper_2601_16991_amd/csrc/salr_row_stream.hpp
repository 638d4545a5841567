// The weight stream of the small-batch kernels: sixteen rows of What per wave, expanded by the nibble rule of Sec. 3.3 straight
// into an operand of the 16x16x32 MFMA (lane (n = lane % 16, g = lane / 16): eight columns of row n per instruction).
//
// The units of work are pairs of halves of equal width (two chunks of 128 columns, or the two halves of one).  Lanes of even g expand
// half 0 of their row, those of odd g half 1; the order of the contraction is free, so X is read to match.  A half's packed values
// of a row are one contiguous piece, requested by its two lanes with 16-byte loads and parked in LDS with dword d at
// 128 d + 64 half + 4 row: the thirty-two lanes that LDS serves together are sixteen rows of either half, so every lane reads from a
// bank of its own wherever its cursor is.  (With the piece in one run of LDS the random cursors met 96 cycles of bank conflicts
// per chunk and wave, of 207.)
//   addresses   raw buffers that start at the wave's first row: 32-bit offsets; rows, vectors and words past the end read as zeros
//               and need no clamping.
//   bitmap      one request per four chunks, 64 bytes a row, handed to the lanes that need them by row swaps in registers.
//   cursors     twice the element index is the byte shift that aligns an odd cursor as it is (v_alignbyte takes its low two bits).
//   LDS reads   those of byte mask s + 1 are in flight while byte mask s is permuted and multiplied; the compiler's own order waits
//               for each in turn (25 dependent LDS round trips per chunk, 155 vector instructions; now 4 and 115).
#pragma once

#include "salr_device.hpp"
#include "salr_linear_common.hpp"

namespace salr {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

#define SALR_LDS __attribute__((address_space(3)))

// ---- raw buffers: `bytes` from p on are readable, loads past them give zeros
typedef __amdgpu_buffer_rsrc_t Buffer;
constexpr uint32_t kPastBuffer = 0xF0000000u;   // an offset past every buffer, and so is what a few hundred bytes on from it
constexpr uint64_t kBufferMax = 0xEFFFFF00u;

__device__ __forceinline__ Buffer make_buffer(const void* p, uint64_t bytes) {
    const uint32_t n = (uint32_t)(bytes < kBufferMax ? bytes : kBufferMax);
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)n, 0x00020000);
}
__device__ __forceinline__ u32x4 buffer_load4(Buffer b, uint32_t lane_offset, uint32_t offset = 0) {
    return __builtin_amdgcn_raw_buffer_load_b128(b, (int)lane_offset, (int)offset, 0);
}

// ---- LDS by byte address
__device__ __forceinline__ uint32_t lds_address(const void* p) {
    return (uint32_t)(uintptr_t)(SALR_LDS const char*)p;
}
template <typename T>
__device__ __forceinline__ T lds_read(uint32_t address) {
    return *(SALR_LDS const T*)(uintptr_t)address;
}
template <typename T>
__device__ __forceinline__ void lds_write(uint32_t address, const T& v) {
    *(SALR_LDS T*)(uintptr_t)address = v;
}

constexpr int kChunkColumns = 128;
// LDS of a wave's parked values: dword d of a row's piece of half h at 128 d + 64 h + 4 row (a window's third dword may lie past
// the piece).
constexpr int slot_bytes(int vectors) { return (4 * vectors + 2) * 128; }

__device__ __forceinline__ uint32_t popc4(u32x4 q, uint32_t start = 0) {
    return __popc(q.w) + (__popc(q.z) + (__popc(q.y) + (__popc(q.x) + start)));
}

// What a lane reads from LDS to expand one byte mask: two windows of three dwords and the permute selectors.
struct ByteWindow {
    uint32_t d[6];
    u32x2 sel_lo, sel_hi;
    uint32_t at_lo, at_hi;   // twice the nibbles' first element (the low bits are the byte shift that aligns it)
};

// The byte of `word` at bit `shift` (below = the bits under it); `count` = element of the piece at which the word's values start,
// slot = LDS address of the lane's column of dwords, lut = LDS address of the selector table.
__device__ __forceinline__ ByteWindow read_byte_window(uint32_t word, uint32_t below, uint32_t shift, uint32_t count, uint32_t slot,
                                                       uint32_t lut) {
    ByteWindow w;
    const uint32_t e = __popc(word & below) + count;
    const uint32_t lo = __builtin_amdgcn_ubfe(word, shift, 4), hi = __builtin_amdgcn_ubfe(word, shift + 4, 4);
    const uint32_t f = __popc(lo) + e;
    const uint32_t a = slot + 128 * (e >> 1), b = slot + 128 * (f >> 1);
    w.at_lo = 2 * e;
    w.at_hi = 2 * f;
    w.d[0] = lds_read<uint32_t>(a);
    w.d[1] = lds_read<uint32_t>(a + 128);
    w.d[2] = lds_read<uint32_t>(a + 256);
    w.d[3] = lds_read<uint32_t>(b);
    w.d[4] = lds_read<uint32_t>(b + 128);
    w.d[5] = lds_read<uint32_t>(b + 256);
    w.sel_lo = lds_read<u32x2>(lut + 8 * lo);
    w.sel_hi = lds_read<u32x2>(lut + 8 * hi);
    return w;
}

__device__ __forceinline__ bf16x8 expand_window(const ByteWindow& w) {
    const uint32_t l0 = __builtin_amdgcn_alignbyte(w.d[1], w.d[0], w.at_lo), l1 = __builtin_amdgcn_alignbyte(w.d[2], w.d[1], w.at_lo);
    const uint32_t h0 = __builtin_amdgcn_alignbyte(w.d[4], w.d[3], w.at_hi), h1 = __builtin_amdgcn_alignbyte(w.d[5], w.d[4], w.at_hi);
    u32x4 o;
    o.x = __builtin_amdgcn_perm(l1, l0, w.sel_lo.x);
    o.y = __builtin_amdgcn_perm(l1, l0, w.sel_lo.y);
    o.z = __builtin_amdgcn_perm(h1, h0, w.sel_hi.x);
    o.w = __builtin_amdgcn_perm(h1, h0, w.sel_hi.y);
    return __builtin_bit_cast(bf16x8, o);
}

// Groups of sixteen lanes 0 .. 3 of two registers: a = [a0 b0 a2 b2], b = [a1 b1 a3 b3].
__device__ __forceinline__ void swap_odd_even_groups(uint32_t& a, uint32_t& b) {
    const auto p = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    a = p[0];
    b = p[1];
}
// x = [x0 x1 x2 x3]: lo = [x0 x1 x0 x1], hi = [x2 x3 x2 x3]
__device__ __forceinline__ void spread_halves(uint32_t x, uint32_t& lo, uint32_t& hi) {
    const auto p = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    lo = p[0];
    hi = p[1];
}

// Sixteen rows' bitmap words of four chunks, chunk g with lane (n, g), to all four lanes of the row: w[chunk][word].
__device__ __forceinline__ void spread_chunks(u32x4 q, u32x4 (&w)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        uint32_t a, b;
        spread_halves(q[i], a, b);   // [x0 x1 x0 x1], [x2 x3 x2 x3]
        uint32_t a1 = a, b1 = b;
        swap_odd_even_groups(a, a1);
        swap_odd_even_groups(b, b1);
        w[0][i] = a;
        w[1][i] = a1;
        w[2][i] = b;
        w[3][i] = b1;
    }
}

}  // namespace salr
