// Bitmap encoder and standalone decoder (paper Sec. 3.3, "Mapping Sparse Weights").
//
// Encoding is three launches on the caller's stream:
//   1. encode_count_kernel   one workgroup per row: bitmap words + the row's nonzero count
//   2. row_scan_kernel       one workgroup: counts -> row_offsets (exclusive prefix, in place)
//   3. encode_compact_rows_kernel (encode_compact_kernel where rows do not allow 16-byte loads)
//                            one workgroup per row: order-preserving compaction of the nonzeros
// Decoding is one launch, one workgroup per row.  Where short rows are many, launches that go by rows give each a wave instead
// (kWaveRow).  All of it is integer/bit work; the traffic is the
// dense matrix (2 B/element) against bitmap + values (1/8 + 2(1-p) B/element).
#include "salr_device.hpp"
#include "salr_internal.hpp"
#include "salr_adapter_t.hpp"
#include "salr_linear_common.hpp"
#include "salr_nf4.hpp"

namespace salr {

constexpr int kCodecThreads = 256;             // 4 waves
constexpr int kChunkValuesMax = kCodecThreads * kUnit;  // packed values one step can own

constexpr int kDecWaves = kCodecThreads / kWave;

// Rows of up to 4096 columns (eight groups of 512), where they are many, go a wave each: a workgroup per row is mostly the start of it
// then, with waves that have no group and barriers for the rest.  Workgroup / wave per row, us to encode and to decode: 26496 x 1408
// 63 + 31 / 52 + 19, 12788 x 512 31.6 + 12.2 / 27.0 + 5.9, 3000 x 768 19.3 + 5.1 / 18.7 + 4.2, 8842 x 3072 42.2 + 17.0 / 41.6 + 15.3,
// 20000 x 4096 81.4 + 40.3 / 78.2 + 39.7; 4324 x 7040 43.9 + 17.3 / 44.9 + 16.9, 600 x 3072 17.6 + 4.3 / 19.7 + 4.7.
static bool wave_per_row(int64_t rows, int64_t cols) { return cols <= 4096 && rows > 2048; }

// kWaveRow: a wave per row.
template <bool kVec, bool kWaveRow>
__global__ __launch_bounds__(kCodecThreads) void encode_count_kernel(const uint16_t* __restrict__ w, int64_t rows,
                                                                     int64_t cols, int64_t wpr,
                                                                     uint32_t* __restrict__ bitmap,
                                                                     uint32_t* __restrict__ row_offsets) {
    __shared__ uint32_t scratch[kDecWaves];
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int64_t n = kWaveRow ? (int64_t)blockIdx.x * kDecWaves + wave : (int64_t)blockIdx.x;
    if (n >= rows) return;   // only with kWaveRow: nothing below synchronises across waves then
    const uint16_t* row = w + n * cols;
    const int64_t units = wpr * 4;  // whole words: pad bytes are produced as zeros
    uint32_t count = 0;
    for (int64_t base = 0; base < units; base += kWaveRow ? kWave : kCodecThreads) {
        const int64_t u = base + (kWaveRow ? lane : (int)threadIdx.x);
        const uint32_t m = nonzero_mask8(load_unit<kVec>(row, cols, u));
        count += __popc(m);
        // four neighbouring lanes hold the four bytes of one word, the first of them collects it (quad_perm 1, 2, 3)
        const uint32_t b1 = __builtin_amdgcn_update_dpp(0u, m, 0x01, 0xf, 0xf, false);
        const uint32_t b2 = __builtin_amdgcn_update_dpp(0u, m, 0x02, 0xf, 0xf, false);
        const uint32_t b3 = __builtin_amdgcn_update_dpp(0u, m, 0x03, 0xf, 0xf, false);
        if ((lane & 3) == 0 && u < units) bitmap[n * wpr + (u >> 2)] = m | (b1 << 8) | (b2 << 16) | (b3 << 24);
    }
    count = last_lane(wave_inclusive_scan(count));
    // the scan over the rows turns counts into offsets in place
    if constexpr (kWaveRow) {
        if (lane == 0) row_offsets[n + 1] = count;
    } else {
        if (lane == 0) scratch[wave] = count;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t s = 0;
            for (int i = 0; i < kDecWaves; ++i) s += scratch[i];
            row_offsets[n + 1] = s;
        }
    }
}

constexpr int kScanThreads = 1024;

// row_offsets[1..rows] holds per-row counts on entry and inclusive prefix sums on exit; [0] = 0.  *nnz_host (pinned host memory,
// may be null) gets the total as well.  One workgroup, bound by the latency of its
// rounds: a wave takes 256 * kVectors consecutive rows a round, all its loads (1 KB each) in flight (with eight consecutive rows a
// thread, 26496 rows took 25.8 us and 4096 5.7; now 6.5 and 4.1).
template <int kVectors>
__global__ __launch_bounds__(kScanThreads) void row_scan_kernel(uint32_t* __restrict__ row_offsets, int64_t rows,
                                                                uint32_t* __restrict__ nnz_host) {
    __shared__ uint32_t wave_sums[2][kScanThreads / kWave];
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4), aligned(4)));
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    uint32_t* counts = row_offsets + 1;
    uint32_t carry = 0;
    int parity = 0;
    for (int64_t base = 0; base < rows; base += kScanThreads * 4 * kVectors) {
        const int64_t r0 = base + (int64_t)wave * (kWave * 4 * kVectors) + 4 * lane;
        u32x4 v[kVectors];
#pragma unroll
        for (int j = 0; j < kVectors; ++j) {
            const int64_t r = r0 + j * (4 * kWave);
            if (r + 4 <= rows) {
                v[j] = *reinterpret_cast<const u32x4*>(counts + r);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) v[j][i] = r + i < rows ? counts[r + i] : 0u;
            }
        }
        uint32_t sum = 0;   // of the wave's vectors so far
#pragma unroll
        for (int j = 0; j < kVectors; ++j) {
            v[j][1] += v[j][0];
            v[j][2] += v[j][1];
            v[j][3] += v[j][2];
            const uint32_t incl = wave_inclusive_scan(v[j][3]);
            const uint32_t before = sum + incl - v[j][3];
            sum += __shfl(incl, kWave - 1, kWave);
#pragma unroll
            for (int i = 0; i < 4; ++i) v[j][i] += before;
        }
        if (lane == 0) wave_sums[parity][wave] = sum;
        __syncthreads();
        uint32_t before = carry;
#pragma unroll
        for (int i = 0; i < kScanThreads / kWave; ++i) {
            const uint32_t s = wave_sums[parity][i];
            before += i < wave ? s : 0u;
            carry += s;
        }
        parity ^= 1;   // the other half was read before this turn's barrier
#pragma unroll
        for (int j = 0; j < kVectors; ++j) {
            const int64_t r = r0 + j * (4 * kWave);
#pragma unroll
            for (int i = 0; i < 4; ++i) v[j][i] += before;
            if (r + 4 <= rows) {
                *reinterpret_cast<u32x4*>(counts + r) = v[j];
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (r + i < rows) counts[r + i] = v[j][i];
            }
        }
    }
    if (threadIdx.x == 0) {
        row_offsets[0] = 0;
        if (nnz_host != nullptr) *nnz_host = carry;
    }
}

template <bool kVec>
__global__ __launch_bounds__(kCodecThreads) void encode_compact_kernel(const uint16_t* __restrict__ w,
                                                                       int64_t cols,
                                                                       const uint32_t* __restrict__ row_offsets,
                                                                       uint16_t* __restrict__ values,
                                                                       int64_t capacity) {
    __shared__ uint32_t scratch[kCodecThreads / kWave];
    const int64_t n = blockIdx.x;
    const uint16_t* row = w + n * cols;
    const int64_t units = (cols + kUnit - 1) / kUnit;
    int64_t cursor = row_offsets[n];
    for (int64_t base = 0; base < units; base += kCodecThreads) {
        const int64_t u = base + threadIdx.x;
        const uint4 q = load_unit<kVec>(row, cols, u);
        const uint32_t m = nonzero_mask8(q);
        uint32_t total;
        const uint32_t excl = block_exclusive_scan<kCodecThreads>(__popc(m), scratch, total);
        int64_t idx = cursor + excl;
#pragma unroll
        for (int j = 0; j < kUnit; ++j) {
            if ((m >> j) & 1u) {
                if (idx < capacity) values[idx] = (uint16_t)unit_elem(q, j);
                ++idx;
            }
        }
        cursor += total;
    }
}

constexpr int kDecMaxGroups = 1024;   // rows up to 524288 columns

// prefix[g] = nonzeros of a bitmap row before group g of 16 words (512 columns), prefix[groups] = all of them; the whole
// workgroup calls it and it ends with a barrier.
__device__ __forceinline__ void group_prefix(const uint32_t* brow, int64_t wpr, int groups, uint32_t* prefix) {
    const int lane = lane_id();
    for (int g = threadIdx.x >> 4; g < groups; g += kCodecThreads / 16) {
        const int64_t w = 16 * (int64_t)g + (lane & 15);
        uint32_t c = w < wpr ? __popc(brow[w]) : 0u;
#pragma unroll
        for (int d = 8; d > 0; d >>= 1) c += __shfl_xor(c, d, kWave);
        if ((lane & 15) == 0) prefix[g + 1] = c;
    }
    __syncthreads();
    if (threadIdx.x < kWave) {
        uint32_t carry = 0;
        for (int base = 0; base < groups; base += kWave) {
            const int g = base + lane;
            const uint32_t c = g < groups ? prefix[g + 1] : 0u;
            const uint32_t incl = wave_inclusive_scan(c);
            if (g < groups) prefix[g + 1] = carry + incl;
            carry += __shfl(incl, kWave - 1, kWave);
        }
        if (lane == 0) prefix[0] = 0;
    }
    __syncthreads();
}

// Compaction of rows that allow 16-byte loads, one workgroup per row.  The bitmap is written by then, so the waves need
// nothing from each other: a first pass popcounts the bitmap row into start offsets per group of 512 columns (the only
// block barriers), then every wave takes groups on its own -- one 16-byte load per lane (the next group's in flight), a
// wave scan of the byte popcounts, the nonzeros dropped into the wave's LDS slot at their place in the output's 16-byte
// vectors, whole vectors stored as such, the ragged ends of the piece as single values.  Bound by memory: 4096 x 14336 at
// 50 %, 176 MB: 43.6 us with a block scan per 2048 columns and a two-byte store per value, now 36.
// kWaveRow: short rows, a wave per row that takes its groups in order, each where the one before ends; no pass over the bitmap, no barrier.
template <bool kWaveRow>
__global__ __launch_bounds__(kCodecThreads) void encode_compact_rows_kernel(const uint16_t* __restrict__ w, int64_t rows, int64_t cols, int64_t wpr,
                                                                            const uint32_t* __restrict__ bitmap,
                                                                            const uint32_t* __restrict__ row_offsets,
                                                                            uint16_t* __restrict__ values, int64_t capacity) {
    __shared__ uint32_t prefix[kWaveRow ? 1 : kDecMaxGroups + 1];
    __shared__ __attribute__((aligned(16))) uint16_t slot[kDecWaves][65 * 8];
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int64_t n = kWaveRow ? (int64_t)blockIdx.x * kDecWaves + wave : (int64_t)blockIdx.x;
    if (n >= rows) return;   // only with kWaveRow: nothing below synchronises across waves then
    constexpr int kStep = kWaveRow ? 1 : kDecWaves;
    const uint32_t* brow = bitmap + n * wpr;
    const int groups = (int)((wpr + 15) / 16);
    const uint16_t* row = w + n * cols;
    const int64_t units = cols / kUnit;
    const uint8_t* mask_bytes = reinterpret_cast<const uint8_t*>(brow);
    // units past the row end repeat its last one and count as empty
    auto load_group = [&](int g, uint32_t& m) -> uint4 {
        const int64_t u = 64 * (int64_t)g + lane, uc = u < units ? u : units - 1;
        const uint32_t b = mask_bytes[uc];
        m = u < units ? b : 0u;
        return *reinterpret_cast<const uint4*>(row + uc * kUnit);
    };
    uint32_t m;
    uint4 q = load_group(kWaveRow ? 0 : wave, m);
    if constexpr (!kWaveRow) group_prefix(brow, wpr, groups, prefix);
    uint32_t row_start = row_offsets[n];
    uint16_t* my_slot = slot[wave];
    const uint32_t cap = capacity < 0xFFFFFFFFLL ? (uint32_t)capacity : 0xFFFFFFFFu;
    for (int g = kWaveRow ? 0 : wave; g < groups; g += kStep) {
        uint32_t m_next;
        const uint4 next = load_group(g + kStep, m_next);
        const uint32_t incl = wave_inclusive_scan(__popc(m));
        const uint32_t cursor = kWaveRow ? row_start : row_start + prefix[g], total = last_lane(incl);
        if constexpr (kWaveRow) row_start += total;
        const uint32_t first = cursor & 7u;   // position of the piece's first value in its first output vector
        uint32_t at = first + incl - __popc(m);
#pragma unroll
        for (int j = 0; j < kUnit; ++j) {
            if ((m >> j) & 1u) my_slot[at] = (uint16_t)unit_elem(q, j);
            at += (m >> j) & 1u;
        }
        __builtin_amdgcn_wave_barrier();   // LDS executes a wave's accesses in order
        const uint32_t base = cursor - first, end = first + total;   // output index of slot 0; the piece is slots [first, end)
        for (uint32_t v = lane; 8 * v < end; v += kWave) {           // at most two trips
            const uint32_t lo = 8 * v < first ? first : 8 * v, hi = 8 * v + 8 < end ? 8 * v + 8 : end;
            if (hi - lo == 8u && base + hi <= cap) {
                *reinterpret_cast<uint4*>(values + base + lo) = *reinterpret_cast<const uint4*>(my_slot + lo);
            } else {
                for (uint32_t i = lo; i < hi; ++i)
                    if (base + i < cap) values[base + i] = my_slot[i];
            }
        }
        __builtin_amdgcn_wave_barrier();
        q = next;
        m = m_next;
    }
}

// Standalone decoder: per step the workgroup owns 2048 columns of its row; the packed values of the
// step are one contiguous piece of `values`, copied to LDS with aligned dword loads and expanded there.
template <bool kVec>
__global__ __launch_bounds__(kCodecThreads) void decode_kernel(const uint32_t* __restrict__ bitmap,
                                                               const uint16_t* __restrict__ values,
                                                               const uint32_t* __restrict__ row_offsets,
                                                               int64_t rows, int64_t cols, int64_t wpr,
                                                               uint16_t* __restrict__ out) {
    __shared__ uint32_t stage[kChunkValuesMax / 2 + 8];
    __shared__ uint32_t lut[kNibbleLutWords];
    __shared__ uint32_t scratch[kCodecThreads / kWave];
    nibble_lut_init(lut);
    __syncthreads();
    const int64_t n = blockIdx.x;
    const uint8_t* mask_bytes = reinterpret_cast<const uint8_t*>(bitmap + n * wpr);
    const uint32_t* values32 = reinterpret_cast<const uint32_t*>(values);
    uint16_t* row_out = out + n * cols;
    const int64_t units = (cols + kUnit - 1) / kUnit;
    const int64_t nnz = row_offsets[rows];
    int64_t g = row_offsets[n];  // element index in `values` of the next unread value of this row
    for (int64_t base = 0; base < units; base += kCodecThreads) {
        const int64_t u = base + threadIdx.x;
        const uint32_t m = (u < units) ? mask_bytes[u] : 0u;
        uint32_t total;
        const uint32_t excl = block_exclusive_scan<kCodecThreads>(__popc(m), scratch, total);
        const uint32_t parity = (uint32_t)(g & 1);
        const int64_t gdw = g >> 1;
        const uint32_t ndw = (parity + total + 1) >> 1;
        for (uint32_t j = threadIdx.x; j < ndw; j += kCodecThreads) {
            const int64_t e = 2 * (gdw + j);
            uint32_t d;
            if (e + 1 < nnz) d = values32[gdw + j];
            else d = (e < nnz) ? (uint32_t)values[e] : 0u;  // last, half-filled dword of the array
            stage[j] = d;
        }
        __syncthreads();
        if (u < units) {
            const uint4 q = expand_byte(stage, lut, parity + excl, m);
            const int64_t k0 = u * kUnit;
            if constexpr (kVec) {
                *reinterpret_cast<uint4*>(row_out + k0) = q;
            } else {
#pragma unroll
                for (int j = 0; j < kUnit; ++j)
                    if (k0 + j < cols) row_out[k0 + j] = (uint16_t)unit_elem(q, j);
            }
        }
        g += total;
        // the next step's block scan synchronises before `stage` is overwritten
    }
}

// Decoder for rows whose output can be written with 16-byte stores.  One workgroup per row, but the waves
// work on their own: a row is cut into groups of 512 columns (one byte mask per lane), a first pass popcounts
// the bitmap row into per-group start offsets (the only block barriers), then every wave takes groups on its
// own -- wave scan of the byte popcounts, the group's values (one contiguous piece, at most 65 aligned 16-byte
// vectors) copied into the wave's LDS slot, nibble expansion, one 16-byte store per lane -- with the loads of
// its next group already in flight.
// kNf4 (QSALR, paper Sec. 4): `values` are the 4-bit codes, eight to a dword where the bf16 kernel has a 16-byte vector of
// eight values; a lane dequantises its dword (all eight codes lie in one scale block of 64) on the way into the slot,
// and everything after that is the same.  scale_last: index of the last scale.
// kWaveRow: short rows, a wave per row (see encode_compact_rows_kernel).
template <bool kNf4, bool kWaveRow>
__global__ __launch_bounds__(kCodecThreads) void decode_rows_kernel(const uint32_t* __restrict__ bitmap,
                                                                    const uint16_t* __restrict__ values,
                                                                    const uint32_t* __restrict__ row_offsets, int64_t rows, int64_t cols,
                                                                    int64_t wpr, uint16_t* __restrict__ out,
                                                                    const uint16_t* __restrict__ scales, uint32_t scale_last) {
    __shared__ uint32_t prefix[kWaveRow ? 1 : kDecMaxGroups + 1];
    __shared__ float levels_all[kWaveRow ? kDecWaves : 1][16];
    __shared__ __attribute__((aligned(16))) uint32_t slot[kDecWaves][65 * 4 + 8];
    __shared__ uint32_t lut_all[kWaveRow ? kDecWaves : 1][kNibbleLutWords];
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    uint32_t* lut = lut_all[kWaveRow ? wave : 0];
    float* levels = levels_all[kWaveRow ? wave : 0];
    if (kNf4 && (kWaveRow ? lane : (int)threadIdx.x) < 16) levels[lane] = kNf4Levels[lane];
    if constexpr (kWaveRow) {   // tables of its own for each wave
        if (lane < 16) {
            uint32_t a, b;
            nibble_lut_entry(lane, a, b);
            lut[2 * lane] = a;
            lut[2 * lane + 1] = b;
        }
        __builtin_amdgcn_wave_barrier();   // LDS executes a wave's accesses in order
    } else {
        nibble_lut_init(lut);
    }
    const int64_t n = kWaveRow ? (int64_t)blockIdx.x * kDecWaves + wave : (int64_t)blockIdx.x;
    if (n >= rows) return;   // only with kWaveRow: nothing below synchronises across waves then
    const uint32_t* brow = bitmap + n * wpr;
    const int groups = (int)((wpr + 15) / 16);
    if constexpr (!kWaveRow) group_prefix(brow, wpr, groups, prefix);   // ---- pass 1
    // ---- pass 2
    const uint8_t* mask_bytes = reinterpret_cast<const uint8_t*>(brow);
    const uint4* values128 = reinterpret_cast<const uint4*>(values);
    const uint32_t* codes32 = reinterpret_cast<const uint32_t*>(values);
    // vector j of the packed values as requested (16 bytes of bf16; or dword j of the codes in .x and its scale in .y)
    // and as it goes into the slot (the codes dequantised: only then does the wave wait for the request)
    auto fetch = [&](uint32_t j) -> uint4 {
        if constexpr (kNf4) {
            const uint32_t blk = j >> 3;
            return make_uint4(codes32[j], scales[blk < scale_last ? blk : scale_last], 0u, 0u);
        } else {
            return values128[j];
        }
    };
    auto ready = [&](const uint4& q) -> uint4 {
        if constexpr (kNf4) return nf4_decode8(q.x, bf16_bits_to_f32(q.y), levels);
        else return q;
    };
    uint16_t* row_out = out + n * cols;
    const int64_t units = (cols + kUnit - 1) / kUnit;
    uint32_t row_start = row_offsets[n];
    uint32_t* my_slot = slot[wave];
    auto load_mask = [&](int g) -> uint32_t {
        const int64_t u = 64 * (int64_t)g + lane;
        return (g < groups && u < units) ? mask_bytes[u] : 0u;
    };
    uint32_t ahead = kWaveRow ? load_mask(0) : 0u;   // the mask of the group whose values are asked for next
    auto group_loads = [&](int g, uint32_t& m, uint4& v, uint32_t& off, uint32_t& nv, uint32_t& vbase) {
        uint32_t cursor, total;
        if constexpr (kWaveRow) {
            m = ahead;
            ahead = load_mask(g + 1);
            cursor = row_start;
            total = last_lane(wave_inclusive_scan(__popc(m)));
            row_start += total;
        } else {
            m = load_mask(g);
            const uint32_t gi = g < groups ? g : groups - 1;
            cursor = row_start + prefix[gi];
            total = g < groups ? prefix[gi + 1] - prefix[gi] : 0u;
        }
        off = cursor & 7u;
        nv = total ? (off + total + 7u) >> 3 : 0u;
        // lanes past the piece repeat its last vector (clamped, not predicated); an empty piece loads nothing new
        const uint32_t li = nv ? ((uint32_t)lane < nv ? lane : nv - 1u) : 0u;
        vbase = cursor >> 3;
        v = nv ? fetch(vbase + li) : make_uint4(0, 0, 0, 0);
    };
    uint32_t m, off, nv, vbase;
    uint4 v;
    constexpr int kStep = kWaveRow ? 1 : kDecWaves;
    group_loads(kWaveRow ? 0 : wave, m, v, off, nv, vbase);
    for (int g = kWaveRow ? 0 : wave; g < groups; g += kStep) {
        uint32_t m2, off2, nv2, vbase2;
        uint4 v2;
        group_loads(g + kStep, m2, v2, off2, nv2, vbase2);   // next group of this wave, in flight while this one expands
        const uint32_t incl = wave_inclusive_scan(__popc(m));
        if ((uint32_t)lane < nv) reinterpret_cast<uint4*>(my_slot)[lane] = ready(v);
        // a full group that starts off a vector boundary spans 65 vectors: the last one is fetched on the spot
        if (__builtin_amdgcn_readfirstlane(nv) > 64u && lane == 0) reinterpret_cast<uint4*>(my_slot)[64] = ready(fetch(vbase + 64));
        __builtin_amdgcn_wave_barrier();
        const uint4 q = expand_byte(my_slot, lut, off + incl - __popc(m), m);
        __builtin_amdgcn_wave_barrier();
        const int64_t u = 64 * (int64_t)g + lane;
        if (u < units) *reinterpret_cast<uint4*>(row_out + u * kUnit) = q;
        m = m2; v = v2; off = off2; nv = nv2; vbase = vbase2;
    }
}

template <bool kNf4>
static void launch_decode_rows(const uint32_t* bitmap, const uint16_t* values, const uint32_t* row_offsets, int64_t rows, int64_t cols,
                               uint16_t* out, const uint16_t* scales, uint32_t scale_last, hipStream_t stream) {
    const int64_t wpr = (cols + 31) / 32;
    const bool wave_row = wave_per_row(rows, cols);
    const dim3 grid((unsigned)(wave_row ? (rows + kDecWaves - 1) / kDecWaves : rows)), block(kCodecThreads);
    if (wave_row) hipLaunchKernelGGL((decode_rows_kernel<kNf4, true>), grid, block, 0, stream, bitmap, values, row_offsets, rows, cols, wpr, out, scales, scale_last);
    else hipLaunchKernelGGL((decode_rows_kernel<kNf4, false>), grid, block, 0, stream, bitmap, values, row_offsets, rows, cols, wpr, out, scales, scale_last);
}

static bool vec_ok(const void* p, int64_t cols);

// QSALR: decode from the 4-bit codes straight into the dense matrix (no bf16 copy of the values in between)
bool decode_nf4_takes(int64_t rows, int64_t cols, int64_t nnz, const void* codes, const void* out) {
    const int64_t wpr = (cols + 31) / 32;
    return rows > 0 && cols > 0 && nnz > 0 && vec_ok(out, cols) && (wpr + 15) / 16 <= kDecMaxGroups &&
           (reinterpret_cast<uintptr_t>(codes) & 3u) == 0;
}

hipError_t launch_decode_nf4(const uint32_t* bitmap, const uint8_t* codes, const uint16_t* scales, int64_t nnz,
                             const uint32_t* row_offsets, int64_t rows, int64_t cols, uint16_t* out, hipStream_t stream) {
    launch_decode_rows<true>(bitmap, reinterpret_cast<const uint16_t*>(codes), row_offsets, rows, cols, out, scales,
                             (uint32_t)((nnz + kNf4Block - 1) / kNf4Block - 1), stream);
    return hipGetLastError();
}

static bool vec_ok(const void* p, int64_t cols) {
    return (cols % kUnit == 0) && ((reinterpret_cast<uintptr_t>(p) & 15u) == 0);
}

hipError_t launch_encode_index(const uint16_t* w, int64_t rows, int64_t cols, uint32_t* bitmap, uint32_t* row_offsets,
                               uint32_t* nnz_host, hipStream_t stream) {
    const int64_t wpr = (cols + 31) / 32;
    if (rows > 0) {
        const bool wave_row = wave_per_row(rows, cols);
        const dim3 grid((unsigned)(wave_row ? (rows + kDecWaves - 1) / kDecWaves : rows)), block(kCodecThreads);
        auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, 0, stream, w, rows, cols, wpr, bitmap, row_offsets); };
        if (vec_ok(w, cols)) wave_row ? go(encode_count_kernel<true, true>) : go(encode_count_kernel<true, false>);
        else wave_row ? go(encode_count_kernel<false, true>) : go(encode_count_kernel<false, false>);
    }
    // one vector a wave as far as that is one round (4096 rows 4.1 us), else eight (6016 rows 6.6, 26496 rows 6.5)
    if (rows <= 4 * kScanThreads) hipLaunchKernelGGL((row_scan_kernel<1>), dim3(1), dim3(kScanThreads), 0, stream, row_offsets, rows, nnz_host);
    else hipLaunchKernelGGL((row_scan_kernel<8>), dim3(1), dim3(kScanThreads), 0, stream, row_offsets, rows, nnz_host);
    return hipGetLastError();
}

hipError_t launch_encode_values(const uint16_t* w, int64_t rows, int64_t cols, const uint32_t* bitmap, const uint32_t* row_offsets,
                                uint16_t* values, int64_t capacity, hipStream_t stream) {
    if (values == nullptr || rows == 0 || cols == 0) return hipSuccess;
    const int64_t wpr = (cols + 31) / 32;
    if (vec_ok(w, cols) && vec_ok(values, kUnit) && (wpr + 15) / 16 <= kDecMaxGroups) {
        if (wave_per_row(rows, cols))
            hipLaunchKernelGGL(encode_compact_rows_kernel<true>, dim3((unsigned)((rows + kDecWaves - 1) / kDecWaves)), dim3(kCodecThreads), 0, stream, w, rows, cols, wpr, bitmap, row_offsets, values, capacity);
        else
            hipLaunchKernelGGL(encode_compact_rows_kernel<false>, dim3((unsigned)rows), dim3(kCodecThreads), 0, stream, w, rows, cols, wpr, bitmap, row_offsets, values, capacity);
    } else if (vec_ok(w, cols))
        hipLaunchKernelGGL(encode_compact_kernel<true>, dim3((unsigned)rows), dim3(kCodecThreads), 0, stream, w, cols, row_offsets, values, capacity);
    else
        hipLaunchKernelGGL(encode_compact_kernel<false>, dim3((unsigned)rows), dim3(kCodecThreads), 0, stream, w, cols, row_offsets, values, capacity);
    return hipGetLastError();
}

hipError_t launch_encode(const uint16_t* w, int64_t rows, int64_t cols, uint32_t* bitmap, uint16_t* values,
                         int64_t capacity, uint32_t* row_offsets, hipStream_t stream) {
    const hipError_t e = launch_encode_index(w, rows, cols, bitmap, row_offsets, nullptr, stream);
    return e != hipSuccess ? e : launch_encode_values(w, rows, cols, bitmap, row_offsets, values, capacity, stream);
}

hipError_t launch_decode(const uint32_t* bitmap, const uint16_t* values, const uint32_t* row_offsets, int64_t rows,
                         int64_t cols, uint16_t* out, hipStream_t stream) {
    if (rows == 0 || cols == 0) return hipSuccess;
    const int64_t wpr = (cols + 31) / 32;
    if (vec_ok(out, cols) && (wpr + 15) / 16 <= kDecMaxGroups && (reinterpret_cast<uintptr_t>(values) & 15u) == 0)
        launch_decode_rows<false>(bitmap, values, row_offsets, rows, cols, out, nullptr, 0u, stream);
    else if (vec_ok(out, cols))
        hipLaunchKernelGGL(decode_kernel<true>, dim3((unsigned)rows), dim3(kCodecThreads), 0, stream, bitmap, values, row_offsets, rows, cols, wpr, out);
    else
        hipLaunchKernelGGL(decode_kernel<false>, dim3((unsigned)rows), dim3(kCodecThreads), 0, stream, bitmap, values, row_offsets, rows, cols, wpr, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------------
// Decode of the TRANSPOSED weight (the backward pass contracts over the weight's rows) into MFMA operand order, block (f, nb) =
// columns 16 f .. 16 f + 15 x rows 32 nb .. + 31 as described in salr_gemm.hip, with the rank blocks of A_cat behind those of
// the weight: the reconstruction rule of Sec. 3.3 as in the kernels above, the transposition done in LDS on the way out, so
// that the dense matrix crosses memory once.  cols % 32 == 0, rows % 64 == 0.
//   the first t_wgs workgroups: the low-rank intermediates T' = dY B_cat^T and T = X A_cat of the same call (R % 8 == 0), a chain of
//   round trips that has nothing to do with the weight (in a launch of their own: 2048 x 4096 x 4096 111.6 us a call, now 107.7;
//   544 x 2400 x 15552 136 and 125);
//   the next a_wgs: A_cat's blocks, a 16-byte vector per thread;
//   workgroup (b, z) of the others: rows 64 b .. 64 b + 63 (wave w the 16 rows 16 w ..), chunks [C z / ksl, C (z + 1) / ksl) of
//   the C = ceil(cols / 128) chunks of 128 columns.  Per chunk lane (n = lane%16, g = lane/16) expands byte g of the four
//   bitmap words of row n, as in the small-batch linear, and writes its 32 values into an LDS tile [128 columns][64 rows];
//   after a barrier the 256 threads store the tile's sixteen blocks, two of them (2 KB) in a row each.
//   The packed values of the next chunk are in flight while this one is expanded.
// Bound by memory and by the LDS it transposes through: 4096 x 4096 in 17 us (33 MB out, 19 in).
// ---------------------------------------------------------------------------------------------------
constexpr int kDtWaves = 4;
constexpr int kDtThreads = kDtWaves * 64;
constexpr int kDtRows = 16 * kDtWaves;
constexpr int kDtPitch = kDtRows + 8;     // bf16 elements per tile row: 144 bytes, 16-byte aligned, banks spread
constexpr int kDtSlotDwords = 68;         // per row and chunk: 17 vectors of 16 B (128 values + misalignment)

struct DtStage {
    uint4 bm;
    uint4 vq[3];
    uint32_t off, nv, vbase;
};

// kVec: rows of the bitmap are whole 16-byte vectors (cols % 128 == 0)
template <bool kVec>
__global__ __launch_bounds__(kDtThreads, 4) void decode_transposed_frags_kernel(
    const uint32_t* __restrict__ bitmap, const uint16_t* __restrict__ values, const uint32_t* __restrict__ row_offsets, int64_t rows,
    int64_t cols, int ksl, const uint16_t* __restrict__ a_cat, int R, int r_blocks, int a_wgs, uint16_t* __restrict__ wf, LowRankJob dy_b,
    LowRankJob x_a, int64_t M, int dy_wgs, int t_wgs) {
    // a tile on its way out, and the waves' values; or the tiles of the low-rank intermediates
    constexpr int kTileElems = 128 * kDtPitch;
    __shared__ __attribute__((aligned(16))) uint16_t tile[kTileElems + 2 * (kDtWaves * 16 * kDtSlotDwords + 8)];
    static_assert(sizeof(tile) >= adapter_t_lds_bytes<1, kDtWaves, kFactorRanks>() && sizeof(tile) >= adapter_t_lds_bytes<1, kDtWaves>(), "room");
    if ((int)blockIdx.x < t_wgs) {   // the same for the whole workgroup
        const int Rpad = (R + 31) / 32 * 32, groups = Rpad >> 5, id = (int)blockIdx.x;
        if (id < dy_wgs)
            adapter_t_block<1, kDtWaves, 2, kFactorRanks>(dy_b.in, M, dy_b.C, dy_b.factor, R, Rpad, dy_b.t, id / groups, id % groups, tile, dy_b.t_t);
        else
            adapter_t_block<1, kDtWaves, 2>(x_a.in, M, x_a.C, x_a.factor, R, Rpad, x_a.t, (id - dy_wgs) / groups, (id - dy_wgs) % groups, tile, x_a.t_t);
        return;
    }
    const int wg = (int)blockIdx.x - t_wgs;
    const int64_t out_blocks = rows / 32 + r_blocks, frags = cols / 16;   // blocks per f, number of f
    if (wg < a_wgs) {
        const int64_t v = (int64_t)wg * kDtThreads + threadIdx.x, block = v >> 6;
        const int l = (int)v & 63, rb = (int)(block % r_blocks);
        const int64_t f = block / r_blocks;
        if (f >= frags) return;
        const uint16_t* arow = a_cat + (16 * f + (l & 15)) * R;
        uint32_t e[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int r = 32 * rb + 8 * (l >> 4) + j;
            const uint32_t q = arow[r < R ? r : R - 1];
            e[j] = r < R ? q : 0u;
        }
        *reinterpret_cast<uint4*>(wf + (f * out_blocks + rows / 32 + rb) * 512 + 8 * l) =
            make_uint4(e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16));
        return;
    }
    uint32_t* slots = reinterpret_cast<uint32_t*>(tile + kTileElems);
    __shared__ uint32_t lut[kNibbleLutWords];
    nibble_lut_init(lut);
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, g = lane >> 4;
    const int64_t id = (int64_t)wg - a_wgs, row_blocks = rows / kDtRows;
    const int64_t n0 = id % row_blocks * kDtRows;
    const int64_t row = n0 + 16 * wave + n;
    const int64_t row_c = row;   // rows % 64 == 0: every row of the block exists
    const int64_t wpr = cols >> 5;
    const int64_t chunks = (wpr + 3) >> 2;
    const int z = (int)(id / row_blocks);
    const int64_t c_begin = chunks * z / ksl, c_end = chunks * (z + 1) / ksl;   // the same for the whole workgroup
    const uint32_t* brow = bitmap + row_c * wpr;
    auto load_chunk = [&](int64_t c) -> uint4 {   // words past the row are empty
        if constexpr (kVec) return *reinterpret_cast<const uint4*>(brow + c * 4);
        uint32_t q[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t v = brow[4 * c + i < wpr ? 4 * c + i : wpr - 1];
            q[i] = 4 * c + i < wpr ? v : 0u;
        }
        return make_uint4(q[0], q[1], q[2], q[3]);
    };
    // nonzeros of the row left of the slice: the 4 lanes of a row share the words, 8 loads in flight each
    uint32_t cur = row_offsets[row_c];
    {
        uint32_t before = 0;
        for (int64_t c0 = 0; c0 < c_begin; c0 += 32) {
            uint4 q[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int64_t c = c0 + g + 4 * i;
                q[i] = load_chunk(c < c_begin ? c : 0);
            }
#pragma unroll
            for (int i = 0; i < 8; ++i)
                before += (c0 + g + 4 * i < c_begin) ? __popc(q[i].x) + __popc(q[i].y) + __popc(q[i].z) + __popc(q[i].w) : 0u;
        }
        before += __shfl_xor(before, 16, 64);
        before += __shfl_xor(before, 32, 64);
        cur += before;
    }
    const uint4* values128 = reinterpret_cast<const uint4*>(values);
    uint32_t* slot = slots + (wave * 16 + n) * kDtSlotDwords;
    // chunks past the slice read its last chunk and count as empty (no conditional load in the stream)
    auto issue = [&](DtStage& st, int64_t c) {
        uint4 bm = load_chunk(c < c_end ? c : c_end - 1);
        const uint32_t keep = c < c_end ? 0xFFFFFFFFu : 0u;
        bm.x &= keep; bm.y &= keep; bm.z &= keep; bm.w &= keep;
        st.bm = bm;
        const uint32_t len = __popc(bm.x) + __popc(bm.y) + __popc(bm.z) + __popc(bm.w);
        st.off = cur & 7u;
        st.nv = len ? (st.off + len + 7u) >> 3 : 0u;
        st.vbase = cur >> 3;
        const uint32_t last = st.nv ? st.nv - 1u : 0u;
        // an empty piece reads the output instead (always mapped, and not used)
        const uint4* vb = st.nv ? values128 + st.vbase : reinterpret_cast<const uint4*>(wf);
        cur += len;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const uint32_t v = g + 4 * i;
            st.vq[i] = vb[v < last ? v : last];
        }
    };
    __syncthreads();   // the lookup table
    if (c_begin >= c_end) return;   // the same for the whole workgroup
    DtStage st[2];
    issue(st[0], c_begin);
    issue(st[1], c_begin + 1);
    for (int64_t c = c_begin; c < c_end; c += 2) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            if (c + i < c_end) {   // the same for the whole workgroup
                const DtStage& s0 = st[i];
#pragma unroll
                for (int v = 0; v < 3; ++v) *reinterpret_cast<uint4*>(slot + 4 * (g + 4 * v)) = s0.vq[v];
                if (s0.nv > 12u) {   // a piece of more than 89 values: fetch the rest now
#pragma unroll
                    for (int v3 = 3; v3 < 5; ++v3) {
                        const uint32_t v = g + 4 * v3;
                        if (v < 17u) *reinterpret_cast<uint4*>(slot + 4 * v) = values128[s0.vbase + (v < s0.nv - 1u ? v : s0.nv - 1u)];
                    }
                }
                __builtin_amdgcn_wave_barrier();
                const uint32_t words[4] = {s0.bm.x, s0.bm.y, s0.bm.z, s0.bm.w};
                uint32_t c_local = s0.off;
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const uint32_t word = words[s];
                    const uint32_t m8 = (word >> (8 * g)) & 0xFFu;
                    const uint32_t cb = c_local + __popc(word & ((1u << (8 * g)) - 1u));
                    const uint4 wq = expand_byte(slot, lut, cb, m8);
                    c_local += __popc(word);
                    const uint32_t e[4] = {wq.x, wq.y, wq.z, wq.w};
                    uint16_t* col = tile + (32 * s + 8 * g) * kDtPitch + 16 * wave + n;   // column 32 s + 8 g of the chunk
#pragma unroll
                    for (int j = 0; j < 8; ++j) col[j * kDtPitch] = (uint16_t)(e[j >> 1] >> (16 * (j & 1)));
                }
                issue(st[i], c + i + 2);
                // barriers that wait for LDS traffic only: the requests of the next chunks stay in flight
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // the tile is complete
                // vector l of block (f, nb): column 16 f + l % 16, rows 32 nb + 8 (l / 16) ..
                const int64_t f0 = (c + i) * 8;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int idx = tid + kDtThreads * t;
                    const int f = idx >> 7, nb = (idx >> 6) & 1, l = idx & 63;
                    if (f0 + f < frags)
                        *reinterpret_cast<uint4*>(wf + ((f0 + f) * out_blocks + n0 / 32 + nb) * 512 + 8 * l) =
                            *reinterpret_cast<const uint4*>(tile + (16 * f + (l & 15)) * kDtPitch + 32 * nb + 8 * (l >> 4));
                }
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // the tile may be overwritten
            }
        }
    }
}

hipError_t launch_decode_transposed_frags(const uint32_t* bitmap, const uint16_t* values, const uint32_t* row_offsets, int64_t rows,
                                          int64_t cols, const uint16_t* a_cat, int R, uint16_t* wf, const LowRankJob& dy_b,
                                          const LowRankJob& x_a, int64_t M, hipStream_t stream) {
    const int64_t blocks = rows / kDtRows, chunks = (cols + 127) / 128;
    int64_t ksl = (1024 + blocks - 1) / blocks;   // about four workgroups per CU
    ksl = ksl < 1 ? 1 : (ksl > chunks ? chunks : ksl);
    const int r_blocks = (R + 63) / 64 * 2;
    const int64_t a_wgs = (cols / 16 * r_blocks * 64 + kDtThreads - 1) / kDtThreads;
    const int t_job = (int)((M + 15) / 16) * ((R + 31) / 32);   // workgroups of sixteen rows and 32 ranks
    const int dy_wgs = dy_b.in != nullptr ? t_job : 0, t_wgs = dy_wgs + (x_a.in != nullptr ? t_job : 0);
    const dim3 grid((unsigned)(t_wgs + a_wgs + blocks * ksl));
    if (cols % 128 == 0)
        hipLaunchKernelGGL(decode_transposed_frags_kernel<true>, grid, dim3(kDtThreads), 0, stream, bitmap, values, row_offsets, rows, cols,
                           (int)ksl, a_cat, R, r_blocks, (int)a_wgs, wf, dy_b, x_a, M, dy_wgs, t_wgs);
    else
        hipLaunchKernelGGL(decode_transposed_frags_kernel<false>, grid, dim3(kDtThreads), 0, stream, bitmap, values, row_offsets, rows, cols,
                           (int)ksl, a_cat, R, r_blocks, (int)a_wgs, wf, dy_b, x_a, M, dy_wgs, t_wgs);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------------
// Slice table (see salr_internal.hpp; the block's work is slice_table_block in salr_linear_common.hpp).  Runs once per
// layer.
// ---------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void slice_table_kernel(const uint32_t* __restrict__ bitmap,
                                                          const uint32_t* __restrict__ row_offsets, int64_t N, int64_t K,
                                                          uint32_t* __restrict__ table) {
    slice_table_block(bitmap, row_offsets, N, K, table, (int64_t)blockIdx.x, (int)threadIdx.x);
}

hipError_t launch_build_slice_table(const uint32_t* bitmap, const uint32_t* row_offsets, int64_t N, int64_t K, uint32_t* table,
                                    hipStream_t stream) {
    if (N <= 0) return hipSuccess;
    hipLaunchKernelGGL(slice_table_kernel, dim3((unsigned)((N + kSliceTableRowsPerBlock - 1) / kSliceTableRowsPerBlock)),
                       dim3(256), 0, stream, bitmap, row_offsets, N, K, table);
    return hipGetLastError();
}

}  // namespace salr
