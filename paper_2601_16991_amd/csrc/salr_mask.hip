// Magnitude pruning masks (paper Sec. 2: static mask from a magnitude threshold; Sec. 4: the N:M
// pattern of the inference-throughput comparison).
//
// Row mask, rows of up to 57344 columns in whole 16-byte units: mask_rows_wave_kernel below.  Other rows: one workgroup per row keeps the `keep` entries of largest |w|, ties to the lower column.
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
#include "salr_row_stream.hpp"

namespace salr {

constexpr int kMaskThreads = 256;
constexpr int kMaskWaves = kMaskThreads / kWave;
constexpr int kMaskWaveRounds = 14;   // most rounds of 512 columns that a wave takes of a row
constexpr int64_t kMaskLdsBytesMax = 56 * 1024;  // dynamic LDS a row may take beside the histograms without raising the default limit

__device__ __forceinline__ uint32_t mag15(uint32_t bits16) { return bits16 & 0x7FFFu; }

// kLds: the row sits in LDS (rows without 16-byte units only: the others that fit are the kernel's below).
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

// Sum over the wave, in every lane.
__device__ __forceinline__ uint32_t wave_total(uint32_t x) { return last_lane(wave_inclusive_scan(x)); }

constexpr uint32_t kTop = 0x80008000u;   // the top bit of both entries of a dword
constexpr uint32_t kOnes = 0x00010001u;

// Two entries of a row against t (both halves, at most 0x8000): bit 15 of each half says whether that entry's magnitude is at
// least t.  Setting the sign bit keeps one half's subtraction out of the other.
__device__ __forceinline__ uint32_t at_least(uint32_t v, uint32_t top, uint32_t t) { return (v | top) - t; }

// The same, but: the magnitude differs from t.
__device__ __forceinline__ uint32_t differs(uint32_t v, uint32_t top, uint32_t t) { return ((v | top) ^ t) - kOnes; }

// c plus the top bits of the four halves of d0 and d1
__device__ __forceinline__ uint32_t add_tops(uint32_t c, uint32_t d0, uint32_t d1) {
    return c + __popc(__builtin_amdgcn_perm(d0, d1, 0x07050301u) & 0x80808080u);
}

// Row mask for rows of up to 64 * kUPL * kW units (8 columns each) that allow 16-byte accesses: kW waves per row, each with up to
// kUPL consecutive rounds of 64 units, the row in registers, the threshold found by counting passes over them.  Waves of the same
// row exchange their counts through LDS, one barrier a pass; a wave with a row of its own meets no barrier (four to a workgroup).
//
// Bound by the passes over memory and, after each other because registers hold few rows at once, the counting.  A pass takes
// 3.5 instructions per two entries on the entries as they are (at_least, add_tops).  The number of passes is kept low: a first
// guess from 256 entries, ranked by ballots, then two counts over 2048 entries on both sides of it, which give a better one and
// the density of entries around it, and from there Newton steps and interpolation: about 3.5 passes over the row on weights.  Raw
// buffers bound the row, so neither loads nor stores nor passes test for its end (with a compare and a select at each the kernel
// took twice as long).
// Before (one wave per row up to 14336 columns, a pass of 3 instructions on rotated entries, about five passes; rows of 14337 to
// 20480 columns in LDS) and now: 4096 x 14336 60.4 -> 42.5 us (5.5 TB/s), 4096 x 4096 21.0 -> 16.1, 26496 x 1408 46.2 -> 33.9,
// 12788 x 512 21.7 -> 13.5, 2000 x 20000 107.8 -> 32.6, 2000 x 28672 127.9 -> 41.4, 500 x 57344 91.0 -> 24.8.
template <int kUPL, int kW>
__global__ __launch_bounds__(kW == 1 ? kMaskThreads : kW * kWave) void mask_rows_wave_kernel(const uint16_t* __restrict__ w, int64_t rows,
                                                                                          int64_t cols, int64_t keep,
                                                                                          uint16_t* __restrict__ out) {
    __shared__ uint32_t shared_counts[2][kW];
    const int lane = lane_id();
    const int in_group = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int wave = kW == 1 ? 0 : in_group;   // of the row
    const int64_t n = kW == 1 ? (int64_t)blockIdx.x * kMaskWaves + in_group : (int64_t)blockIdx.x;
    if (n >= rows) return;   // only with kW == 1: nothing below synchronises across waves then
    const uint16_t* row = w + n * cols;
    const int row_units = (int)(cols / kUnit);
    const int rounds = ((row_units + kWave - 1) / kWave + kW - 1) / kW;   // of one wave
    const int first_unit = wave * rounds * kWave;
    int units = row_units - first_unit;   // of this wave
    units = units < 0 ? 0 : units < rounds * kWave ? units : rounds * kWave;
    uint32_t v[kUPL][4];   // zeros past the row
    const Buffer in = make_buffer(row + (int64_t)first_unit * kUnit, (uint64_t)units * 16);
    u32x4 q0;   // the row's first 64 units, in every wave
    if constexpr (kW > 1) q0 = buffer_load4(make_buffer(row, (uint64_t)row_units * 16), 16u * lane);
    for_rounds<kUPL>([&](auto round) __attribute__((always_inline)) {
        constexpr int i = decltype(round)::value;
        const u32x4 q = buffer_load4(in, 16u * lane + 1024u * i);
#pragma unroll
        for (int d = 0; d < 4; ++d) v[i][d] = q[d];
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
    uint32_t top = kTop;
    // entries with magnitude >= t (1 <= t <= 0x7FFF; the zero padding never counts) in the first kRounds rounds of this wave, and of
    // all waves of the row
    int parity = 0;
    auto count_ge = [&](auto most, uint32_t t, uint32_t& mine) __attribute__((always_inline)) -> uint32_t {
        constexpr int kRounds = decltype(most)::value;
        const uint32_t t2 = t * kOnes;
        asm volatile("" : "+v"(top));   // anew in each pass, or the compiler keeps `v | top` of the whole row beside it
        uint32_t c = 0;
        for_rounds<kRounds>([&](auto round) __attribute__((always_inline)) {
            constexpr int i = decltype(round)::value;
            c = add_tops(c, at_least(v[i][0], top, t2), at_least(v[i][1], top, t2));
            c = add_tops(c, at_least(v[i][2], top, t2), at_least(v[i][3], top, t2));
        });
        mine = wave_total(c);
        if constexpr (kW == 1) return mine;
        if (lane == 0) shared_counts[parity][wave] = mine;
        __syncthreads();
        uint32_t sum = 0;
#pragma unroll
        for (int i = 0; i < kW; ++i) sum += shared_counts[parity][i];
        parity ^= 1;   // the other half was read before this pass's barrier
        return (uint32_t)__builtin_amdgcn_readfirstlane((int)sum);
    };
    constexpr std::integral_constant<int, kUPL> kAll{};
    // first guess: the threshold of four entries per lane of the first 64 units, to sixteen magnitudes
    uint32_t guess = 0;
    {
        const uint32_t s0 = kW == 1 ? v[0][0] : q0[0], s1 = kW == 1 ? v[0][1] : q0[1];
        const uint32_t a = s0 & 0x7FFFu, b = (s0 >> 16) & 0x7FFFu, c = s1 & 0x7FFFu, d = (s1 >> 16) & 0x7FFFu;
        const float sample = 4.f * (float)(row_units < kWave ? row_units : kWave);
        const uint32_t want = (uint32_t)((float)keep * sample * __builtin_amdgcn_rcpf((float)cols));
        for (int bit = 14; bit >= 4; --bit) {
            const uint32_t cand = guess | (1u << bit);
            const uint32_t ge = __popcll(__builtin_amdgcn_ballot_w64(a >= cand)) + __popcll(__builtin_amdgcn_ballot_w64(b >= cand)) +
                                __popcll(__builtin_amdgcn_ballot_w64(c >= cand)) + __popcll(__builtin_amdgcn_ballot_w64(d >= cand));
            if (ge >= want) guess = cand;
        }
    }
    // T = max { t : count(|w| >= t) >= keep }: lo has enough entries from it on, hi too few (no magnitude reaches 0x8000).
    // mine_lo, mine_hi: this wave's part of the two counts.
    uint32_t lo = 0, hi = 0x8000u, count_lo = (uint32_t)cols, count_hi = 0;
    uint32_t mine_lo = (uint32_t)units * kUnit, mine_hi = 0;
    // the second guess, and how many entries of the row a step of the threshold passes there
    constexpr int kSample = kUPL < (kW < 4 ? 4 / kW : 1) ? kUPL : (kW < 4 ? 4 / kW : 1);
    const uint32_t below = guess > 8u ? guess - 8u : 1u, above_guess = guess < 0x7FE0u ? guess + 24u : 0x7FFFu;
    uint32_t mine_below, mine_above;
    const uint32_t count_below = count_ge(std::integral_constant<int, kSample>{}, below, mine_below);
    const uint32_t count_above = count_ge(std::integral_constant<int, kSample>{}, above_guess, mine_above);
    float density;
    uint32_t t;
    if (rounds <= kSample) {   // the sample was the row: these were passes
        if ((int64_t)count_below >= keep) { lo = below; count_lo = count_below; mine_lo = mine_below; }
        else { hi = below; count_hi = count_below; mine_hi = mine_below; }
        if (lo != 0u) {
            if ((int64_t)count_above >= keep) { lo = above_guess; count_lo = count_above; mine_lo = mine_above; }
            else { hi = above_guess; count_hi = count_above; mine_hi = mine_above; }
        }
        density = 0.f;
        t = 0;
    } else {
        int sampled = 0;   // units
#pragma unroll
        for (int i = 0; i < kW; ++i) {
            const int of_wave = row_units - i * rounds * kWave;
            sampled += of_wave < 0 ? 0 : of_wave < kSample * kWave ? of_wave : kSample * kWave;
        }
        const float scale = (float)row_units * __builtin_amdgcn_rcpf((float)sampled);   // of a count of the sample to the row
        density = scale * (float)(count_below - count_above) * __builtin_amdgcn_rcpf((float)(above_guess - below));
        density = density < 1.f ? 1.f : density;
        float guess2 = (float)below + ((float)count_below * scale - (float)keep) * __builtin_amdgcn_rcpf(density);
        guess2 = guess2 < 1.f ? 1.f : guess2 > 32767.f ? 32767.f : guess2;
        t = (uint32_t)(guess2 + 0.5f);
    }
    uint32_t stride = 1;
    for (int pass = 0;; ++pass) {   // at least every third pass halves the interval once both sides are found
        if (pass > 0 || rounds <= kSample) {
            if (lo == 0u || hi == 0x8000u) {   // one side is still open: reach for it
                const uint32_t off = lo == 0u ? (uint32_t)keep - count_hi : count_lo - (uint32_t)keep;
                uint32_t step = density > 0.f ? (uint32_t)((float)off * __builtin_amdgcn_rcpf(density)) + 1u : 16u;
                step = step < stride ? stride : step > 0x8000u ? 0x8000u : step;
                stride *= 4;
                t = lo == 0u ? (hi > step ? hi - step : 1u) : lo + step;
            } else {
                const float f = (float)(count_lo - (uint32_t)keep) * __builtin_amdgcn_rcpf((float)(count_lo - count_hi));
                t = pass % 3 == 2 ? (lo + hi) / 2 : lo + 1u + (uint32_t)(f * (float)(hi - lo - 1u));
            }
        }
        if (hi - lo <= 1u) break;
        t = t <= lo ? lo + 1u : t >= hi ? hi - 1u : t;
        uint32_t mine;
        const uint32_t c = count_ge(kAll, t, mine);
        if ((int64_t)c == keep) {   // exactly the entries from t on: no ties to rank, and on a row that is pruned already, where
            lo = t - 1u;            // the count stays the same over a wide gap, nothing to creep along
            hi = t;
            count_hi = c;
            break;
        }
        if ((int64_t)c >= keep) { lo = t; count_lo = c; mine_lo = mine; }
        else { hi = t; count_hi = c; mine_hi = mine; }
    }
    const uint32_t T = lo;
    keep_one_form();
    // Ties fill the remaining places in column order: this wave's share of them follows those of the waves before it.
    uint32_t ties_wanted = (uint32_t)(keep - (int64_t)count_hi);
    if constexpr (kW > 1) {
        if (ties_wanted > 0u) {   // the same in all waves of the row
            if (lane == 0) shared_counts[parity][wave] = mine_lo - mine_hi;
            __syncthreads();
            uint32_t before = 0;
#pragma unroll
            for (int i = 0; i < kW - 1; ++i) before += i < wave ? shared_counts[parity][i] : 0u;
            before = (uint32_t)__builtin_amdgcn_readfirstlane((int)before);
            ties_wanted = ties_wanted > before ? ties_wanted - before : 0u;
        }
    }
    // Rounds are in column order (units run lane-fastest): before the group of rounds in which the places run out every tie is
    // kept, after it none, and only in that group do single ties count.
    constexpr int kGroup = 4;
    const uint32_t T2 = T * kOnes;
    const Buffer to = make_buffer(out + n * cols + (int64_t)first_unit * kUnit, (uint64_t)units * 16);   // drops the rest
    uint32_t ties_before = 0;
    auto halves_of = [&](uint32_t d) __attribute__((always_inline)) -> uint32_t {   // all ones in each half whose top bit is set
        typedef short s16x2 __attribute__((ext_vector_type(2)));
        s16x2 h;
        __builtin_memcpy(&h, &d, 4);
        h = h >> (short)15;
        __builtin_memcpy(&d, &h, 4);
        return d;
    };
    auto ties_of = [&](auto round, uint32_t c) __attribute__((always_inline)) -> uint32_t {   // c + the entries that are no ties
        constexpr int i = decltype(round)::value;
        c = add_tops(c, differs(v[i][0], top, T2), differs(v[i][1], top, T2));
        return add_tops(c, differs(v[i][2], top, T2), differs(v[i][3], top, T2));
    };
    for_rounds<(kUPL + kGroup - 1) / kGroup>([&](auto group) __attribute__((always_inline)) {
        constexpr int first = decltype(group)::value * kGroup, count = first + kGroup <= kUPL ? kGroup : kUPL - first;
        uint32_t from[count];   // of each round: entries of at least this magnitude (both halves) are kept
        uint32_t at[count];     // byte offset of this lane's unit
        for_rounds<count>([&](auto round) __attribute__((always_inline)) {
            constexpr int r = decltype(round)::value;
            from[r] = T2 + kOnes;
            at[r] = 16u * lane + 1024u * (first + r);
        });
        if (ties_before < ties_wanted) {   // wave-uniform
            asm volatile("" : "+v"(top));
            uint32_t c = 0;
            for_rounds<count>([&](auto round) __attribute__((always_inline)) {
                c = ties_of(std::integral_constant<int, first + decltype(round)::value>{}, c);
            });
            uint32_t ties = 8u * kWave * count - wave_total(c);
            if (ties_before + ties <= ties_wanted) {
                for_rounds<count>([&](auto round) __attribute__((always_inline)) { from[decltype(round)::value] = T2; });
                ties_before += ties;
            } else {
                // the round in which the places run out goes entry by entry (there is none if they do at a round's end)
                uint32_t e[4] = {0, 0, 0, 0}, e_at = kPastBuffer;
                for_rounds<count>([&](auto round) __attribute__((always_inline)) {
                    constexpr int r = decltype(round)::value;
                    if (ties_before >= ties_wanted) return;
                    ties = 8u * kWave - wave_total(ties_of(std::integral_constant<int, first + r>{}, 0u));
                    if (ties_before + ties <= ties_wanted) {
                        from[r] = T2;
                        ties_before += ties;
                    } else {
#pragma unroll
                        for (int d = 0; d < 4; ++d) e[d] = v[first + r][d];
                        e_at = at[r];
                        at[r] = kPastBuffer;
                        ties = ties_before;
                        ties_before = ties_wanted;
                    }
                });
                uint32_t tied = 0;   // a bit per entry
#pragma unroll
                for (int j = 0; j < kUnit; ++j) tied |= (uint32_t)(((e[j >> 1] >> (16 * (j & 1))) & 0x7FFFu) == T) << j;
                uint32_t rank = ties + wave_inclusive_scan(__popc(tied)) - __popc(tied);
                u32x4 o = {0, 0, 0, 0};
#pragma unroll
                for (int j = 0; j < kUnit; ++j) {
                    const uint32_t x = (e[j >> 1] >> (16 * (j & 1))) & 0xFFFFu, tie = (tied >> j) & 1u;
                    const bool kept = (x & 0x7FFFu) > T || (tie != 0u && rank < ties_wanted);
                    o[j >> 1] |= (kept ? x : 0u) << (16 * (j & 1));
                    rank += tie;
                }
                __builtin_amdgcn_raw_buffer_store_b128(o, to, (int)e_at, 0, 0);
            }
        }
        asm volatile("" : "+v"(top));
        for_rounds<count>([&](auto round) __attribute__((always_inline)) {
            constexpr int r = decltype(round)::value, i = first + r;
            u32x4 o;
#pragma unroll
            for (int d = 0; d < 4; ++d) o[d] = v[i][d] & halves_of(at_least(v[i][d], top, from[r]));
            __builtin_amdgcn_raw_buffer_store_b128(o, to, (int)at[r], 0, 0);
        });
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
    // As few waves a row as leave each at most 14 rounds: more pay a barrier a pass and repeat the search's scalar work, fewer hold so
    // many registers that rows in flight run short.  One, two, four, eight waves: 4324 x 7040 27, 29, 33, 53 us; 4096 x 14336
    // 48, 44, 45, 55; 2000 x 28672 -, 48, 43, 46; 1124 x 22016 -, 30, 26, 30.  The rounds a wave holds are compiled in, in steps that
    // keep the empty ones to a sixth.
    const int64_t all_rounds = (units + kWave - 1) / kWave;
    if (vec && all_rounds <= 8 * kMaskWaveRounds) {
        auto go = [&](auto upl, auto waves) {
            constexpr int kUPL = decltype(upl)::value, kW = decltype(waves)::value;
            const dim3 grid((unsigned)(kW == 1 ? (rows + kMaskWaves - 1) / kMaskWaves : rows)), block(kW == 1 ? kMaskThreads : kW * kWave);
            hipLaunchKernelGGL((mask_rows_wave_kernel<kUPL, kW>), grid, block, 0, stream, w, rows, cols, keep, out);
        };
        auto by_rounds = [&](auto waves) {
            constexpr int kW = decltype(waves)::value;
            const int64_t rounds = (all_rounds + kW - 1) / kW;
            if constexpr (kW == 1) {
                if (rounds <= 1) return go(std::integral_constant<int, 1>{}, waves);
                if (rounds <= 2) return go(std::integral_constant<int, 2>{}, waves);
                if (rounds <= 3) return go(std::integral_constant<int, 3>{}, waves);
                if (rounds <= 4) return go(std::integral_constant<int, 4>{}, waves);
                if (rounds <= 6) return go(std::integral_constant<int, 6>{}, waves);
            }
            if (rounds <= 8) go(std::integral_constant<int, 8>{}, waves);
            else if (rounds <= 10) go(std::integral_constant<int, 10>{}, waves);
            else if (rounds <= 12) go(std::integral_constant<int, 12>{}, waves);
            else go(std::integral_constant<int, kMaskWaveRounds>{}, waves);
        };
        if (all_rounds <= kMaskWaveRounds) by_rounds(std::integral_constant<int, 1>{});
        else if (all_rounds <= 2 * kMaskWaveRounds) by_rounds(std::integral_constant<int, 2>{});
        else if (all_rounds <= 4 * kMaskWaveRounds) by_rounds(std::integral_constant<int, 4>{});
        else by_rounds(std::integral_constant<int, 8>{});
        return hipGetLastError();
    }
    const dim3 grid((unsigned)rows), block(kMaskThreads);
    const size_t dyn = lds && !vec ? row_bytes : 0;
    if (lds && !vec) hipLaunchKernelGGL((mask_rows_kernel<true, false>), grid, block, dyn, stream, w, cols, keep, out);
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
