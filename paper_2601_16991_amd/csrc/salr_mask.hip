// Magnitude pruning masks (paper Sec. 2: static mask from a magnitude threshold; Sec. 4: the N:M
// pattern of the inference-throughput comparison).
//
// Row mask, rows of up to 14336 columns in whole 16-byte units, and of 20488 to 28672 where there are many:
// mask_rows_wave_kernel below (see launch_mask_rows).  Other rows: one workgroup per row keeps the `keep` entries of largest |w|, ties to the lower column.
// The threshold is the largest 15-bit magnitude pattern T with count(|w| >= T) >= keep, found by a
// two-level radix select: a histogram of the exponent (the top 8 of the 15 bits) locates T's exponent,
// a histogram of the 7 mantissa bits inside that exponent locates the rest (two passes over the row,
// which sits in LDS when it fits; the histograms are per wave, to spread the LDS atomics);
// every entry above T is kept, and of the entries equal to T the first keep - count(|w| > T) in
// column order (a block scan over the row).  bf16 magnitudes order like their bit patterns, so all of
// it is integer work and the result is exact.  Traffic: the matrix once in, once out.
#include <type_traits>

#include "salr_device.hpp"
#include "salr_internal.hpp"

namespace salr {

constexpr int kMaskThreads = 256;
constexpr int kMaskWaves = kMaskThreads / kWave;
constexpr int64_t kMaskLdsBytesMax = 56 * 1024;  // dynamic LDS a row may take beside the histograms without raising the default limit

__device__ __forceinline__ uint32_t mag15(uint32_t bits16) { return bits16 & 0x7FFFu; }

template <bool kLds, bool kVec>
__global__ __launch_bounds__(kMaskThreads) void mask_rows_kernel(const uint16_t* __restrict__ w, int64_t cols,
                                                                 int64_t keep, uint16_t* __restrict__ out) {
    extern __shared__ uint4 row_lds[];        // kLds: the row, ceil(cols/8) units, zero padded
    __shared__ uint32_t scan_scratch[kMaskWaves + 1];
    const int64_t n = blockIdx.x;
    const uint16_t* row = w + n * cols;
    uint16_t* row_out = out + n * cols;
    const int64_t units = (cols + kUnit - 1) / kUnit;
    const int tid = threadIdx.x;
    const int wave = tid / kWave;

    if constexpr (kLds) {
        for (int64_t u = tid; u < units; u += kMaskThreads) row_lds[u] = load_unit<kVec>(row, cols, u);
        __syncthreads();
    }
    auto unit = [&](int64_t u) -> uint4 {
        if constexpr (kLds) return row_lds[u];
        else return load_unit<kVec>(row, cols, u);
    };
    // Histogram pass: bins[wave][key] += 1 for every entry whose `filter` holds; then the bin of the
    // `want`-th largest key (want >= 1) and the number of entries in bins above it.
    __shared__ uint32_t bins[kMaskWaves][256];
    __shared__ uint32_t found[2];
    auto select_bin = [&](int nbins, auto key_of, auto filter, uint32_t want, uint32_t& bin, uint32_t& above_bin) {
        for (int i = tid; i < kMaskWaves * 256; i += kMaskThreads) bins[i >> 8][i & 255] = 0u;
        __syncthreads();
        for (int64_t u = tid; u < units; u += kMaskThreads) {
            const uint4 q = unit(u);
#pragma unroll
            for (int j = 0; j < kUnit; ++j) {
                const uint32_t m = mag15(unit_elem(q, j));
                if (u * kUnit + j < cols && filter(m)) atomicAdd(&bins[wave][key_of(m)], 1u);
            }
        }
        __syncthreads();
        // thread i owns key nbins - 1 - i: the exclusive scan then counts the entries with a larger key
        const int key = nbins - 1 - tid;
        uint32_t h = 0;
        if (tid < nbins)
#pragma unroll
            for (int w = 0; w < kMaskWaves; ++w) h += bins[w][key];
        uint32_t total;
        const uint32_t larger = block_exclusive_scan<kMaskThreads>(h, scan_scratch, total);
        if (tid < nbins && larger < want && larger + h >= want) {
            found[0] = (uint32_t)key;
            found[1] = larger;
        }
        __syncthreads();
        bin = found[0];
        above_bin = found[1];
        __syncthreads();   // found and bins are reused by the next call
    };

    // T = max { t : count(|w| >= t) >= keep }; above = count(|w| > T).  keep == 0 keeps nothing: T is the largest
    // pattern and nothing is allowed in as a tie.
    uint32_t T = 0x7FFFu, above = 0u;
    if (keep > 0) {
        uint32_t expo, above_expo, mant, above_mant;
        select_bin(256, [](uint32_t m) { return m >> 7; }, [](uint32_t) { return true; }, (uint32_t)keep, expo, above_expo);
        select_bin(128, [](uint32_t m) { return m & 0x7Fu; }, [&](uint32_t m) { return (m >> 7) == expo; },
                   (uint32_t)keep - above_expo, mant, above_mant);
        T = (expo << 7) | mant;
        above = above_expo + above_mant;
    }
    // Entries strictly above T all survive; ties at T fill the remaining places from the left.
    const uint32_t ties_wanted = (uint32_t)(keep - (int64_t)above);

    uint32_t ties_before = 0;  // ties in the columns left of this step
    for (int64_t base = 0; base < units; base += kMaskThreads) {
        const int64_t u = base + tid;
        const int64_t k0 = u * kUnit;
        uint4 q = make_uint4(0, 0, 0, 0);
        if (u < units) q = unit(u);
        uint32_t e[kUnit];
        uint32_t my_ties = 0;
#pragma unroll
        for (int j = 0; j < kUnit; ++j) {
            e[j] = unit_elem(q, j);
            my_ties += (k0 + j < cols) && (mag15(e[j]) == T);
        }
        uint32_t step_ties;
        uint32_t tie_rank = ties_before + block_exclusive_scan<kMaskThreads>(my_ties, scan_scratch, step_ties);
        ties_before += step_ties;
#pragma unroll
        for (int j = 0; j < kUnit; ++j) {
            const uint32_t m = mag15(e[j]);
            bool kept = m > T;
            if (m == T && k0 + j < cols) {
                kept = tie_rank < ties_wanted;
                ++tie_rank;
            }
            if (!kept) e[j] = 0u;
        }
        if (u < units) {
            if constexpr (kVec) {
                uint4 o;
                o.x = e[0] | (e[1] << 16);
                o.y = e[2] | (e[3] << 16);
                o.z = e[4] | (e[5] << 16);
                o.w = e[6] | (e[7] << 16);
                *reinterpret_cast<uint4*>(row_out + k0) = o;
            } else {
#pragma unroll
                for (int j = 0; j < kUnit; ++j)
                    if (k0 + j < cols) row_out[k0 + j] = (uint16_t)e[j];
            }
        }
    }
}

// Two 16-bit counters in a dword: each half of c plus one where that half of v is larger than that half of limit.  Spelled
// out, because the compiler turns the saturating subtraction and the minimum back into compares of single halves.
__device__ __forceinline__ uint32_t count_above(uint32_t c, uint32_t v, uint32_t limit) {
    uint32_t d;
    asm("v_pk_sub_u16 %0, %1, %2 clamp" : "=v"(d) : "v"(v), "s"(limit));
    asm("v_pk_min_u16 %0, %1, %2" : "=v"(d) : "v"(d), "s"(0x00010001u));
    asm("v_pk_add_u16 %0, %1, %2" : "=v"(c) : "v"(c), "v"(d));
    return c;
}

__device__ __forceinline__ void opaque(uint32_t& r) { asm volatile("" : "+v"(r)); }

// f(0), f(1), .. f(kN - 1) as compile-time constants: the rounds index registers, and past a certain length the compiler
// leaves a loop in place and the registers become memory.
template <int kN, typename F>
__device__ __forceinline__ void for_rounds(F&& f) {
    if constexpr (kN > 0) {
        for_rounds<kN - 1>(f);
        f(std::integral_constant<int, kN - 1>{});
    }
}

// Row mask for rows of up to 64 * kUPL units (8 columns each) that allow 16-byte accesses: ONE WAVE per row, the
// row in registers (lane l holds units l, l + 64, ...), the threshold found by counting passes over the registers: no LDS,
// no barrier.  Four rows per workgroup.
//
// The counting passes are what the kernel does besides its two passes over memory.  Entries are kept rotated left by one,
// magnitude on top and sign at the bottom, so they compare with 2 t as they are: a saturating subtraction, a minimum with
// one and an addition, two entries at a time.  Their number is kept low by starting from the threshold of a sample (the
// row's first 256 columns, ranked by ballots) and interpolating between the two sides found so far: about seven passes on
// weights, 15 bisections plus one when each bit of the threshold took a pass of its own.
// 4096 x 4096: 32.8 -> 22.1 us; 4096 x 14336, where a histogram kernel with the row in LDS ran before: 131 -> 67 us (3.5 TB/s).
template <int kUPL>
__global__ __launch_bounds__(kMaskThreads) void mask_rows_wave_kernel(const uint16_t* __restrict__ w, int64_t rows, int64_t cols,
                                                                      int64_t keep, uint16_t* __restrict__ out) {
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int64_t n = (int64_t)blockIdx.x * kMaskWaves + wave;
    if (n >= rows) return;   // wave-uniform; nothing below synchronises across waves
    const uint16_t* row = w + n * cols;
    uint16_t* row_out = out + n * cols;
    const int units = (int)(cols / kUnit);
    uint32_t v[kUPL][4];   // entries rotated left by one, two to a dword; zeros past the row
    for_rounds<kUPL>([&](auto round) __attribute__((always_inline)) {
        constexpr int i = decltype(round)::value;
        const int u = lane + kWave * i;
        const uint4 q = *reinterpret_cast<const uint4*>(row + (int64_t)(u < units ? u : 0) * kUnit);
        const uint32_t e[4] = {u < units ? q.x : 0u, u < units ? q.y : 0u, u < units ? q.z : 0u, u < units ? q.w : 0u};
#pragma unroll
        for (int d = 0; d < 4; ++d) v[i][d] = ((e[d] << 1) & 0xFFFEFFFEu) | ((e[d] >> 15) & 0x00010001u);
    });
    // opaque to the compiler before and after the search: it would keep the entries' other forms alive across it, and the
    // row would take twice the registers
    auto keep_one_form = [&]() __attribute__((always_inline)) {
        for_rounds<kUPL>([&](auto round) __attribute__((always_inline)) {
            constexpr int i = decltype(round)::value;
#pragma unroll
            for (int d = 0; d < 4; ++d) opaque(v[i][d]);
        });
    };
    keep_one_form();
    // entries of the row with magnitude >= t (1 <= t <= 0x7FFF; the zero padding never counts)
    auto row_count_ge = [&](uint32_t t) __attribute__((always_inline)) -> uint32_t {
        const uint32_t limit = (2u * t - 1u) * 0x00010001u;   // an entry is larger iff its magnitude is >= t
        uint32_t c = 0;
        for_rounds<kUPL>([&](auto round) __attribute__((always_inline)) {
            constexpr int i = decltype(round)::value;
            if (kWave * i < units) {   // the same for the whole launch
#pragma unroll
                for (int d = 0; d < 4; ++d) c = count_above(c, v[i][d], limit);
            }
        });
        const uint32_t mine = (c & 0xFFFFu) + (c >> 16);   // at most 8 kUPL < 512: nine bits, each summed over the lanes by a ballot
        uint32_t sum = 0;
#pragma unroll
        for (int bit = 0; bit < 9; ++bit) sum += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64((mine >> bit) & 1u)) << bit;
        return sum;
    };
    // first guess: the threshold of the row's first columns (four entries per lane)
    uint32_t guess = 0;
    {
        const int64_t sample = 4 * (units < kWave ? units : kWave);
        const uint32_t want = (uint32_t)(keep * sample / cols);
        for (int bit = 14; bit >= 3; --bit) {
            const uint32_t cand = guess | (1u << bit);
            uint32_t c = 0;
#pragma unroll
            for (int d = 0; d < 2; ++d) {
                c += __popcll(__builtin_amdgcn_ballot_w64((v[0][d] & 0xFFFFu) >= 2u * cand));
                c += __popcll(__builtin_amdgcn_ballot_w64((v[0][d] >> 16) >= 2u * cand));
            }
            if (c >= want) guess = cand;
        }
    }
    // T = max { t : count(|w| >= t) >= keep }: lo has enough entries above it, hi too few (no magnitude reaches 0x8000)
    uint32_t lo = 0, hi = 0x8000u, count_lo = (uint32_t)cols, count_hi = 0, stride = 16;
    uint32_t t = guess < 1u ? 1u : guess;
    for (int pass = 0; hi - lo > 1u; ++pass) {   // at least every third pass halves the interval
        const uint32_t c = row_count_ge(t);
        if ((int64_t)c == keep) {   // exactly the entries from t on: no ties to rank, and on a row that is pruned already, where
            lo = t - 1u;            // the count stays the same over a wide gap, nothing to creep along (61 us on 4096 x 4096)
            hi = t;
            count_hi = c;
            break;
        }
        if ((int64_t)c >= keep) { lo = t; count_lo = c; }
        else { hi = t; count_hi = c; }
        if (lo == 0u || hi == 0x8000u) {   // one side is still open: reach for it from the guess
            t = lo == 0u ? (hi > stride ? hi - stride : 1u) : lo + stride;
            stride *= 4;
        } else {
            const float f = (float)(count_lo - (uint32_t)keep) / (float)(count_lo - count_hi);
            t = pass % 3 == 2 ? (lo + hi) / 2 : lo + 1u + (uint32_t)(f * (float)(hi - lo - 1u));
        }
        t = t <= lo ? lo + 1u : t >= hi ? hi - 1u : t;
    }
    const uint32_t T = lo, above = count_hi;
    keep_one_form();
    const uint32_t ties_wanted = (uint32_t)(keep - (int64_t)above);
    // Ties fill the remaining places in column order, and rounds are in column order (units run lane-fastest): before the
    // round in which the places run out every tie is kept, after it none, and only in that round do single ties count.
    const uint32_t at_least_T = T > 0u ? (2u * T - 1u) * 0x00010001u : 0u, above_T = (2u * T + 1u) * 0x00010001u;
    const uint32_t any = T > 0u ? 0u : 0x00010001u;   // T == 0: every entry counts as at least T
    uint32_t ties_before = 0;
    for_rounds<kUPL>([&](auto round) __attribute__((always_inline)) {
        constexpr int i = decltype(round)::value;
        const int u = lane + kWave * i;
        if (kWave * i >= units) return;   // the same for the whole launch
        uint32_t kept[4];                 // 1 in each half that survives
#pragma unroll
        for (int d = 0; d < 4; ++d) kept[d] = count_above(0u, v[i][d], above_T);
        if (ties_before < ties_wanted) {  // wave-uniform
            uint32_t ge[4], c = 0;
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                ge[d] = count_above(0u, v[i][d], at_least_T) | any;
                c += ge[d] - kept[d];
            }
            const uint32_t mine = (c & 0xFFFFu) + (c >> 16);
            uint32_t ties = 0;
#pragma unroll
            for (int bit = 0; bit < 4; ++bit) ties += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64((mine >> bit) & 1u)) << bit;
            if (ties_before + ties <= ties_wanted) {
#pragma unroll
                for (int d = 0; d < 4; ++d) kept[d] = ge[d];
            } else {
                uint32_t rank = ties_before + wave_inclusive_scan(mine) - mine;
#pragma unroll
                for (int j = 0; j < kUnit; ++j) {
                    const uint32_t tie = ((ge[j >> 1] - kept[j >> 1]) >> (16 * (j & 1))) & 1u;
                    ge[j >> 1] -= (tie != 0u && rank >= ties_wanted ? 1u : 0u) << (16 * (j & 1));
                    rank += tie;
                }
#pragma unroll
                for (int d = 0; d < 4; ++d) kept[d] = ge[d];
            }
            ties_before += ties;
        }
        if (u < units) {
            uint32_t o[4];
#pragma unroll
            for (int d = 0; d < 4; ++d)
                o[d] = (((v[i][d] >> 1) & 0x7FFF7FFFu) | ((v[i][d] & 0x00010001u) << 15)) & (kept[d] * 0xFFFFu);
            *reinterpret_cast<uint4*>(row_out + (int64_t)u * kUnit) = make_uint4(o[0], o[1], o[2], o[3]);
        }
    });
}

// N:M mask, one thread per group of m consecutive columns: entry i survives iff fewer than n entries
// of its group come before it in the order (larger magnitude first, lower column first among equals).
template <int kM>
__global__ __launch_bounds__(256) void mask_nm_fixed_kernel(const uint16_t* __restrict__ w, int64_t groups,
                                                            int n_keep, uint16_t* __restrict__ out) {
    typedef uint16_t group_t __attribute__((ext_vector_type(kM)));  // 2*kM bytes, aligned because cols % kM == 0
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= groups) return;
    const group_t v = reinterpret_cast<const group_t*>(w)[g];
    group_t o;
#pragma unroll
    for (int i = 0; i < kM; ++i) {
        const uint32_t mi = mag15(v[i]);
        int before = 0;
#pragma unroll
        for (int j = 0; j < kM; ++j) {
            const uint32_t mj = mag15(v[j]);
            before += (mj > mi) || (mj == mi && j < i);
        }
        o[i] = before < n_keep ? v[i] : (uint16_t)0;
    }
    reinterpret_cast<group_t*>(out)[g] = o;
}

__global__ __launch_bounds__(256) void mask_nm_any_kernel(const uint16_t* __restrict__ w, int64_t groups,
                                                          int n_keep, int m_group, uint16_t* __restrict__ out) {
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= groups) return;
    const uint16_t* src = w + g * m_group;
    uint16_t* dst = out + g * m_group;
    for (int i = 0; i < m_group; ++i) {
        const uint32_t mi = mag15(src[i]);
        int before = 0;
        for (int j = 0; j < m_group; ++j) {
            const uint32_t mj = mag15(src[j]);
            before += (mj > mi) || (mj == mi && j < i);
        }
        dst[i] = before < n_keep ? src[i] : (uint16_t)0;
    }
}

hipError_t launch_mask_rows(const uint16_t* w, int64_t rows, int64_t cols, int64_t keep, uint16_t* out,
                            hipStream_t stream) {
    if (rows == 0 || cols == 0) return hipSuccess;
    const int64_t units = (cols + kUnit - 1) / kUnit;
    const size_t row_bytes = (size_t)units * sizeof(uint4);
    const bool lds = row_bytes <= (size_t)kMaskLdsBytesMax;
    const bool vec = (cols % kUnit == 0) && (((reinterpret_cast<uintptr_t>(w) | reinterpret_cast<uintptr_t>(out)) & 15u) == 0);
    // A row in the registers of one wave, or a workgroup per row with the row in LDS.  The registers of 28 units a lane leave two
    // waves on a SIMD (196), those of 56 one (297), too few to cover memory.  Microseconds by rows (1/2 of the entries kept, inputs from
    // memory), wave form / workgroup form:
    //   14336 columns   512: 25/27   1024: 29/42                 2048: 39/72     4096: 68/130    8192: 113/-
    //   16384           512: 41/30   1024: 43/45   1536: 80/67   2048: 82/80     4096: 160/145   8192: 315/275
    //   20480           512: 50/36   1024: 54/67   1536: 99/84   2048: 103/112   4096: 201/213   8192: 396/397
    //   22528           512: 54/39   1024: 57/73   1536: 106/91  2048: 111/123   4096: 213/232   8192: 421/437
    //   24576           512: 57/42   1024: 61/79   1536: 111/100 2048: 117/132   4096: 229/252   8192: 450/470
    //   25600           512: 59/45   1024: 64/86   1536: 117/125 2048: 123/165   4096: 240/320   8192: 471/622
    //   28672           512: 65/49   1024: 71/93   1536: 127/137 2048: 135/180   4096: 262/349   8192: 513/681
    // With 7/10 kept the wave form needs 7 to 10 % more, the other the same.  So 56 units only on rows of more than 20480
    // columns, where the row in LDS leaves three workgroups on a CU, or two from 24584 on, and the rows are more than those
    // hold at once.
    const int64_t held = 256 * (units > kWave * 48 ? 2 : 3);
    if (vec && (units <= kWave * 28 || (units > kWave * 40 && units <= kWave * 56 && rows > held))) {
        const dim3 wgrid((unsigned)((rows + kMaskWaves - 1) / kMaskWaves));
        if (units <= kWave * 4) hipLaunchKernelGGL((mask_rows_wave_kernel<4>), wgrid, dim3(kMaskThreads), 0, stream, w, rows, cols, keep, out);
        else if (units <= kWave * 8) hipLaunchKernelGGL((mask_rows_wave_kernel<8>), wgrid, dim3(kMaskThreads), 0, stream, w, rows, cols, keep, out);
        else if (units <= kWave * 16) hipLaunchKernelGGL((mask_rows_wave_kernel<16>), wgrid, dim3(kMaskThreads), 0, stream, w, rows, cols, keep, out);
        else if (units <= kWave * 28) hipLaunchKernelGGL((mask_rows_wave_kernel<28>), wgrid, dim3(kMaskThreads), 0, stream, w, rows, cols, keep, out);
        else hipLaunchKernelGGL((mask_rows_wave_kernel<56>), wgrid, dim3(kMaskThreads), 0, stream, w, rows, cols, keep, out);
        return hipGetLastError();
    }
    const dim3 grid((unsigned)rows), block(kMaskThreads);
    const size_t dyn = lds ? row_bytes : 0;
    if (lds && vec) hipLaunchKernelGGL((mask_rows_kernel<true, true>), grid, block, dyn, stream, w, cols, keep, out);
    else if (lds) hipLaunchKernelGGL((mask_rows_kernel<true, false>), grid, block, dyn, stream, w, cols, keep, out);
    else if (vec) hipLaunchKernelGGL((mask_rows_kernel<false, true>), grid, block, dyn, stream, w, cols, keep, out);
    else hipLaunchKernelGGL((mask_rows_kernel<false, false>), grid, block, dyn, stream, w, cols, keep, out);
    return hipGetLastError();
}

hipError_t launch_mask_nm(const uint16_t* w, int64_t rows, int64_t cols, int n_keep, int m_group, uint16_t* out,
                          hipStream_t stream) {
    const int64_t groups = rows * (cols / m_group);
    if (groups == 0) return hipSuccess;
    const dim3 grid((unsigned)((groups + 255) / 256)), block(256);
    const bool aligned = (((reinterpret_cast<uintptr_t>(w) | reinterpret_cast<uintptr_t>(out)) & 15u) == 0);
    if (aligned && m_group == 2) hipLaunchKernelGGL((mask_nm_fixed_kernel<2>), grid, block, 0, stream, w, groups, n_keep, out);
    else if (aligned && m_group == 4) hipLaunchKernelGGL((mask_nm_fixed_kernel<4>), grid, block, 0, stream, w, groups, n_keep, out);
    else if (aligned && m_group == 8) hipLaunchKernelGGL((mask_nm_fixed_kernel<8>), grid, block, 0, stream, w, groups, n_keep, out);
    else hipLaunchKernelGGL(mask_nm_any_kernel, grid, block, 0, stream, w, groups, n_keep, m_group, out);
    return hipGetLastError();
}

}  // namespace salr
