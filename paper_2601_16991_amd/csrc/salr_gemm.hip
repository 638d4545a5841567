// Large-batch stages of the SALR linear (M > 64) and of its backward pass: the two stages of Sec. 3.3 ("Pipeline Design")
// as two kernels.
//
//   stage 1  bitmap decode of the whole weight, once per call, into MFMA operand order (the layout below), B_cat behind it;
//   stage 2  frag_gemm_kernel: Y = X * W^T (+ T * B_cat, Sec. 3.2) on the matrix cores.
//
// Operand order.  Block (f, kb) is 16 weight rows x 32 columns = 1 KB in the order in which v_mfma_f32_16x16x32_bf16 takes
// them: lane l = 16 g + i holds row i's eight columns 32 kb + 8 g .. + 7.  The blocks of one f follow each other along kb,
// first the blocks of the weight
// (an even number: K / 32, and a zero block when that is odd), then those of B_cat (likewise; the rank dimension is appended to the contraction).
// Block f holds weight rows 16 f .. 16 f + 15.
//
// frag_gemm_kernel.  Workgroup: four waves as kWM x kWN, wave tile 16 kMI (m) x 16 kNI (n); on the largest tiles one wave per
// SIMD, whose accumulators take half of its 512 registers.  W fragments go from memory straight into registers, a whole k-step
// (64 columns) ahead, as contiguous 1 KB loads: they never touch LDS, which would otherwise carry every operand twice (in and
// out) and be as busy as the matrix cores (eight waves of 128 x 64 with both operands in LDS: 192 KB read and 64 KB written
// per step of 2048 MFMA clocks; here 64 + 32 KB).  X goes through LDS: 16-byte-per-lane loads straight into a ring of kStages
// tiles [rows][64 columns], 128-byte rows, segment s of row r at s ^ ((r >> 1) & 7) (conflict-free operand reads).  One barrier
// per k-step, in its middle.  Bound by the matrix cores at the chip's power: 4096 x 8192 x 28672 runs at 1390 to 1430 TFLOP/s
// (1355 us; 1600 us, 1215 TFLOP/s, for the kernel with both operands in LDS), 2048 x 14336 x 4096 at 1180 (206 us; 240).
#include <type_traits>

#include "salr_adapter_t.hpp"
#include "salr_device.hpp"
#include "salr_internal.hpp"
#include "salr_linear_common.hpp"
#include "salr_nf4.hpp"
#include "salr_row_products.hpp"

namespace salr {

constexpr int kGemmXcds = 8;

typedef __bf16 bf16x16 __attribute__((ext_vector_type(16)));

// c += a b on the matrix cores, c in the accumulation registers it is in.  Spelled out, because from the builtin the compiler
// rotates the accumulators through other registers (four copies per MFMA in the loop below).  It does not know the
// instruction's latency then: frag_gemm_kernel reads the accumulators only behind an s_nop of its own.
__device__ __forceinline__ void mfma_in_place(f32x4& c, const bf16x8& a, const bf16x8& b) {
    asm("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}

// The same on the sparse matrix cores (a: four of eight columns and their positions, the half of `index` that kHalf names).
template <int kHalf>
__device__ __forceinline__ void smfmac_in_place(f32x4& c, const bf16x8& a, const bf16x16& b, uint32_t index) {
    if constexpr (kHalf == 0) asm("v_smfmac_f32_16x16x64_bf16 %0, %1, %2, %3" : "+a"(c) : "v"(a), "v"(b), "v"(index));
    else asm("v_smfmac_f32_16x16x64_bf16 %0, %1, %2, %3 abid:1" : "+a"(c) : "v"(a), "v"(b), "v"(index));
}

// LDS of a workgroup: the ring of X tiles, then sixteen output rows per wave on their way out (see the store)
template <int kMI, int kNI, int kWM, int kWN, int kStages, bool kPartial>
constexpr int frag_gemm_lds_bytes() {
    constexpr int kElem = kPartial ? 4 : 2, kOut = kWM * kWN * 16 * (16 * kNI + 32 / kElem) * kElem, kTiles = kStages * 16 * kMI * kWM * 128;
    return kTiles > kOut ? kTiles : kOut;
}

template <int kMI, int kNI, int kWM, int kWN, int kStages, bool kPartial, bool kSparse>
__device__ __forceinline__ void frag_gemm_block(
    const uint16_t* __restrict__ x, int64_t M, int64_t K, int64_t N, const uint16_t* wf,
    const uint16_t* __restrict__ t, int Rpad, uint16_t* __restrict__ y, int m_tiles, int n_tiles, int ksplit,
    float* __restrict__ partial, uint16_t* Xs) {
    constexpr int kWaves = kWM * kWN;
    constexpr int kMT = 16 * kMI * kWM, kNT = 16 * kNI * kWN;
    constexpr int kXLoads = kMT / (8 * kWaves);   // LDS loads per wave and k-step, eight rows each
    static_assert(kMT % (8 * kWaves) == 0 && kNT % 32 == 0, "tile/wave shape");
    typedef typename std::conditional<kPartial, float, uint16_t>::type out_t;
    constexpr int kCols = 16 * kNI, kVec = 16 / sizeof(out_t), kPitch = kCols + 2 * kVec;
    static_assert(frag_gemm_lds_bytes<kMI, kNI, kWM, kWN, kStages, kPartial>() >= kWaves * 16 * kPitch * (int)sizeof(out_t), "room for the results");

    // Consecutive workgroup ids land on different XCDs, each with an L2 of its own: XCD c takes the c-th eighth of the work,
    // ordered so that workgroups running side by side on it share operands: K slice, then blocks of eight m-tiles, then n,
    // then m.
    const int per_k = m_tiles * n_tiles, total = per_k * ksplit, per_xcd = (total + kGemmXcds - 1) / kGemmXcds;
    const int id = (int)blockIdx.x % kGemmXcds * per_xcd + (int)blockIdx.x / kGemmXcds;
    if (id >= total) return;   // uniform for the workgroup, before any barrier
    const int kz = id / per_k, tile = id % per_k;
    const int mg = tile / (8 * n_tiles), in_group = tile - mg * 8 * n_tiles, group_rows = m_tiles - 8 * mg < 8 ? m_tiles - 8 * mg : 8;
    const int nt = in_group / group_rows, mt = 8 * mg + in_group % group_rows;
    const int64_t m0 = (int64_t)mt * kMT, n0 = (int64_t)nt * kNT;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / kWN, wn = wave % kWN;
    const int i16 = lane & 15, g = lane >> 4;

    // k-steps of 64: x_steps over X (the weight is padded with a zero block when K % 64 is 32), then the ones over T;
    // this workgroup takes [s_begin, s_end)
    // (sparse weight: the steps over X only, T follows after the loop)
    const int x_steps = (int)((K + 63) >> 6), steps = x_steps + (kSparse ? 0 : (Rpad + 63) >> 6);
    const int64_t blocks = 2 * (int64_t)steps;
    const int s_begin = (int)((int64_t)steps * kz / ksplit), s_end = (int)((int64_t)steps * (kz + 1) / ksplit);

    // X loader: load j of a wave fills tile rows 8 (wave + kWaves j) .. + 7, lane l slot l % 8 of row l / 8
    const int lrow = 8 * wave + (lane >> 3);
    const int lseg = (lane & 7) ^ ((lrow >> 1) & 7);   // logical 16-byte segment of that slot; the same for every j
    uint32_t row_off[kXLoads];                         // tile row, clamped to the last row of X
#pragma unroll
    for (int j = 0; j < kXLoads; ++j) {
        const int64_t r = lrow + 8 * kWaves * j;
        row_off[j] = (uint32_t)(m0 + r < M ? r : M - 1 - m0);
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)Xs;
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    struct XSource {   // where the X tile of a step comes from (uniform: a raw buffer of 2 GB) and this lane's place in it, in bytes
        u32x4 buffer;
        uint32_t pitch, seg;
    };
    // Second half of a half step: zeros, which a buffer load gives past the buffer's end (the rows of a tile lie below it, see
    // kFragMaxColumns).  That half is multiplied by a zero block, and other columns of the row in its place would make every output
    // of the row NaN where one of them is infinite.  Costs nothing; a condition in the k loop 1 to 3 %, per-lane addresses 1 %.
    constexpr uint32_t kBufferBytes = 0x80000000u, kRawBuffer = 0x00020000u;
    auto x_source = [&](int step) -> XSource {
        const int sc = step < s_end ? step : s_end - 1;   // past the end: reload the last step (unused)
        const bool is_t = sc >= x_steps;
        const int64_t pitch = is_t ? Rpad : K;
        const int k0 = 64 * (is_t ? sc - x_steps : sc);
        const uint64_t base = reinterpret_cast<uint64_t>((is_t ? t : x) + m0 * pitch + k0);
        return {u32x4{(uint32_t)base, (uint32_t)(base >> 32) & 0xFFFFu, kBufferBytes, kRawBuffer}, (uint32_t)pitch * 2,
                k0 + 8 * lseg < pitch ? 16u * lseg : kBufferBytes};
    };
    // Load j of an X tile straight into LDS: lane l lands on the wave's base + 16 l.  Assembly, so that the waits stay under
    // this kernel's control; its memory clobber also keeps the W loads on their side of it, which the wait counts rely on.
    auto fetch_x = [&](const XSource& src, int stage, int j) {
        const uint32_t voff = row_off[j] * src.pitch + src.seg;
        const uint32_t lds = __builtin_amdgcn_readfirstlane(lds0 + stage * (kMT * 128) + (wave + kWaves * j) * 1024);
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds"
                     :
                     : "v"(voff), "s"(src.buffer), "s"(lds)
                     : "memory", "m0");
    };

    // W fragments: block (f, kb) is 512 elements; this wave's f are f0 .. f0 + kNI - 1 (clamped: outputs past N are dropped)
    const int64_t f0 = n0 / 16 + wn * kNI, f_last = (N + 15) / 16 - 1;
    const uint32_t lane_bytes = lane * 16;
    auto load_w = [&](int step, int s, int j) -> bf16x8 {
        const int b0 = 2 * (step < s_end ? step : s_end - 1);
        const int64_t f = f0 + j < f_last ? f0 + j : f_last;
        const char* block = reinterpret_cast<const char*>(wf) + (f * blocks + (b0 + s)) * 1024;
        return *reinterpret_cast<const bf16x8*>(block + lane_bytes);
    };
    const uint16_t* frag_base = Xs + (wm * 16 * kMI + i16) * 64;
    const int fsw = (i16 >> 1) & 7;
    auto load_x = [&](int stage, int s, int i) -> bf16x8 {
        return *reinterpret_cast<const bf16x8*>(frag_base + stage * (kMT * 64) + 16 * i * 64 + ((4 * s + g) ^ fsw) * 8);
    };
    f32x4 acc[kMI][kNI];
#pragma unroll
    for (int i = 0; i < kMI; ++i)
#pragma unroll
        for (int j = 0; j < kNI; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // ---- k loop.  Step s multiplies stage cur in two halves of 32 columns.  A W fragment is requested again, for the next
    // step, as soon as its products of this one are issued; the X fragments of a half are read during the half before it;
    // the second half refills stage cur with step s + kStages.  The barrier between the halves publishes the next stage and
    // retires cur.  Requests are spread between the MFMAs (the scheduling fences keep them there): with one wave per SIMD
    // nothing else fills the matrix pipe.
#pragma unroll
    for (int p = 0; p < kStages; ++p) {
        const XSource src = x_source(s_begin + p);
#pragma unroll
        for (int j = 0; j < kXLoads; ++j) fetch_x(src, p, j);
    }
    if constexpr (!kSparse) {
        bf16x8 w0[kNI], w1[kNI], x0[kMI], x1[kMI];
#pragma unroll
        for (int j = 0; j < kNI; ++j) w0[j] = load_w(s_begin, 0, j);
#pragma unroll
        for (int j = 0; j < kNI; ++j) w1[j] = load_w(s_begin, 1, j);
        asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
        for (int i = 0; i < kMI; ++i) x0[i] = load_x(0, 0, i);
        int cur = 0;
        for (int s = s_begin; s < s_end; ++s) {
            const int nxt = cur + 1 == kStages ? 0 : cur + 1;
#pragma unroll
            for (int j = 0; j < kNI; ++j) {
#pragma unroll
                for (int q = kMI * j / kNI; q < kMI * (j + 1) / kNI; ++q) x1[q] = load_x(cur, 1, q);
#pragma unroll
                for (int i = 0; i < kMI; ++i) mfma_in_place(acc[i][j], w0[j], x0[i]);
                __builtin_amdgcn_sched_barrier(0);
                w0[j] = load_w(s + 1, 0, j);
            }
            // X of step s + 1 has landed: since its last request (second half of step s - 2) there were three halves' W requests
            // and kStages - 2 X tiles
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((kStages - 2) * (kXLoads + 2 * kNI) + kNI) : "memory");
            const XSource src = x_source(s + kStages);
#pragma unroll
            for (int j = 0; j < kNI; ++j) {
#pragma unroll
                for (int q = kXLoads * j / kNI; q < kXLoads * (j + 1) / kNI; ++q) fetch_x(src, cur, q);
#pragma unroll
                for (int q = kMI * j / kNI; q < kMI * (j + 1) / kNI; ++q) x0[q] = load_x(nxt, 0, q);
#pragma unroll
                for (int i = 0; i < kMI; ++i) mfma_in_place(acc[i][j], w1[j], x1[i]);
                __builtin_amdgcn_sched_barrier(0);
                w1[j] = load_w(s + 1, 1, j);
            }
            cur = nxt;
        }
    } else {
        // Sparse weight (256 x 256 and 256 x 224 tiles): one instruction per tile and step of 64 columns, half the steps' matrix time, so W is
        // requested two steps ahead and X fragments are held for two steps.  A pair of
        // steps shares its words of positions (low and high half).  No unit is at its limit (counters at 2048 x 4096 x 14336): the matrix cores are
        // busy 41 % of the cycles, the address units 61, the LDS 33, most of that conflicts of the X reads, and 23 of 64 bytes a clock come to a CU
        // from the L2.  A SIMD has one wave, which is in s_waitcnt for 26 % of its life and waits 33 % for an instruction to be issued: the phases
        // of a step add up.  153 us, 167 with W one step ahead, 203 in the kernel that reads the packed format (gemm_2of4_kernel).
        const int64_t pairs = (steps + 1) / 2, frag = sparse_frag_elems(K, Rpad);
        auto pair_base = [&](int64_t pr, int j) -> const char* {
            const int64_t f = f0 + j < f_last ? f0 + j : f_last;
            return reinterpret_cast<const char*>(wf + f * frag) + (pr < pairs ? pr : pairs - 1) * (kSparsePairElems * 2);
        };
        auto load_ws = [&](int step, int j) -> bf16x8 {
            return *reinterpret_cast<const bf16x8*>(pair_base(step >> 1, j) + (step & 1) * 1024 + lane_bytes);
        };
        auto load_index = [&](int step, int j) -> uint32_t {
            return *reinterpret_cast<const uint32_t*>(pair_base(step >> 1, j) + 2048 + lane * 4);
        };
        auto load_xs = [&](int stage, int i) -> bf16x16 {   // columns 16 g .. 16 g + 15 of the step
            const uint16_t* row = frag_base + stage * (kMT * 64) + 16 * i * 64;
            const bf16x8 lo = *reinterpret_cast<const bf16x8*>(row + ((2 * g) ^ fsw) * 8), hi = *reinterpret_cast<const bf16x8*>(row + ((2 * g + 1) ^ fsw) * 8);
            return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15);
        };
        bf16x8 wa[kNI], wb[kNI];
        uint32_t index[kNI], index_next[kNI];
        bf16x16 xa[kMI], xb[kMI];
#pragma unroll
        for (int j = 0; j < kNI; ++j) wa[j] = load_ws(0, j);
#pragma unroll
        for (int j = 0; j < kNI; ++j) wb[j] = load_ws(1, j);
#pragma unroll
        for (int j = 0; j < kNI; ++j) index[j] = load_index(0, j);
        asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
        for (int i = 0; i < kMI; ++i) xa[i] = load_xs(0, i);
        int cur = 0;
        constexpr int kFirst = kNI / 2;   // n-tiles before the barrier
        auto step = [&](auto half, bf16x8 (&w)[kNI], const bf16x16 (&xc)[kMI], bf16x16 (&xn)[kMI], int s) {
            constexpr int kHalf = decltype(half)::value;
            const int nxt = cur + 1 == kStages ? 0 : cur + 1;
            XSource src{};
#pragma unroll
            for (int j = 0; j < kNI; ++j) {
                if (j == kFirst) {
                    // X of step s + 1 has landed: since its last request (step s + 1 - kStages) there were at least the W
                    // requests and X tiles of kStages - 2 steps, those after the barrier of the one before and kFirst of this
                    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((kStages - 2) * (kXLoads + kNI) + kFirst) : "memory");
                    src = x_source(s + kStages);
                }
                if (j >= kFirst) {
                    constexpr int kRest = kNI - kFirst;
                    const int jj = j - kFirst;
#pragma unroll
                    for (int q = kXLoads * jj / kRest; q < kXLoads * (jj + 1) / kRest; ++q) fetch_x(src, cur, q);
#pragma unroll
                    for (int q = kMI * jj / kRest; q < kMI * (jj + 1) / kRest; ++q) xn[q] = load_xs(nxt, q);
                }
#pragma unroll
                for (int i = 0; i < kMI; ++i) smfmac_in_place<kHalf>(acc[i][j], w[j], xc[i], index[j]);
                __builtin_amdgcn_sched_barrier(0);
                w[j] = load_ws(s + 2, j);
                if constexpr (kHalf == 0) index_next[j] = load_index(s + 2, j);
                else index[j] = index_next[j];
            }
            cur = nxt;
        };
        int s = 0;
        for (; s + 1 < s_end; s += 2) {
            step(std::integral_constant<int, 0>{}, wa, xa, xb, s);
            step(std::integral_constant<int, 1>{}, wb, xb, xa, s + 1);
        }
        if (s < s_end) step(std::integral_constant<int, 0>{}, wa, xa, xb, s);
        // T times B_cat: dense instructions on the same accumulators, both operands from memory
        asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
        const uint16_t* bf = wf + pairs * kSparsePairElems;
        for (int rb = 0; rb < Rpad / 32; ++rb) {
            bf16x8 bq[kNI], tq[kMI];
#pragma unroll
            for (int j = 0; j < kNI; ++j) {
                const int64_t f = f0 + j < f_last ? f0 + j : f_last;
                bq[j] = *reinterpret_cast<const bf16x8*>(bf + f * frag + rb * 512 + lane * 8);
            }
#pragma unroll
            for (int i = 0; i < kMI; ++i) {
                const int64_t m = m0 + wm * 16 * kMI + 16 * i + i16;
                tq[i] = *reinterpret_cast<const bf16x8*>(t + (m < M ? m : M - 1) * Rpad + rb * 32 + 8 * g);
            }
#pragma unroll
            for (int j = 0; j < kNI; ++j)
#pragma unroll
                for (int i = 0; i < kMI; ++i) mfma_in_place(acc[i][j], bq[j], tq[i]);
        }
    }
    // no request lands any more, every wave has read its last tile, the last MFMAs have written their results
    asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier\n\ts_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
    for (int i = 0; i < kMI; ++i)
#pragma unroll
        for (int j = 0; j < kNI; ++j) asm volatile("" : "+a"(acc[i][j]));   // (and no read of them moves up)

    // ---- store, through LDS: a lane holds four outputs n = 16 j + 4 g .. of row m = 16 i + i16.  Sixteen rows at a time go
    // into the wave's own piece of LDS, each shifted to where its first output sits in a 16-byte vector of the result, and
    // leave as whole vectors along n (single elements at the ends).
    out_t* rows = reinterpret_cast<out_t*>(Xs) + wave * 16 * kPitch;
    out_t* dst = kPartial ? reinterpret_cast<out_t*>(partial) + kz * splitk_slice(M * N) : reinterpret_cast<out_t*>(y);
    const int64_t nw = n0 + wn * kCols;
    const int cols = N - nw < kCols ? (int)(N - nw) : kCols;   // may be negative: nothing to store
    const bool quads = (N & 3) == 0;                           // rows start at multiples of four outputs
    // where output (m, nw) sits in its vector
    auto shift_of = [&](int64_t m) -> int { return (int)(((uint32_t)m * (uint32_t)N + (uint32_t)nw) & (kVec - 1)); };
    // a lane stores vector vc of rows vr, vr + kRowStep, .. (of the sixteen); a shifted row has one vector more
    constexpr int kRowVecs = kCols / kVec, kVecs2 = kRowVecs <= 4 ? 4 : kRowVecs <= 8 ? 8 : kRowVecs <= 16 ? 16 : 32;
    constexpr int kRowStep = 64 / kVecs2;
    const int vr = lane / kVecs2, vc = lane % kVecs2;
    const bool whole = cols == kCols && N % kVec == 0 && m0 + kMT <= M;   // uniform: every vector of the tile is whole
    auto store_vec = [&](int64_t mw, int r, int c) {                       // the vector with column 8 c - shift first
        const int64_t m = mw + r;
        const int c0 = c * kVec - shift_of(m);
        if (m >= M) return;
        out_t* to = dst + m * N + nw + c0;
        const out_t* from = rows + r * kPitch + c * kVec;
        if (c0 >= 0 && c0 + kVec <= cols) {
            *reinterpret_cast<uint4*>(to) = *reinterpret_cast<const uint4*>(from);
        } else {
            for (int e = 0; e < kVec; ++e)
                if (c0 + e >= 0 && c0 + e < cols) to[e] = from[e];
        }
    };
#pragma unroll
    for (int i = 0; i < kMI; ++i) {
        const int64_t mw = m0 + wm * 16 * kMI + 16 * i;
        out_t* row = rows + i16 * kPitch + shift_of(mw + i16) + 4 * g;
#pragma unroll
        for (int j = 0; j < kNI; ++j) {
            const f32x4 c = acc[i][j];
            if constexpr (kPartial) {
                if (quads) *reinterpret_cast<float4*>(row + 16 * j) = make_float4(c[0], c[1], c[2], c[3]);
                else
                    for (int e = 0; e < 4; ++e) row[16 * j + e] = c[e];
            } else {
                const uint2 q = make_uint2(pack_bf16_rne(c[0], c[1]), pack_bf16_rne(c[2], c[3]));
                if (quads) {
                    *reinterpret_cast<uint2*>(row + 16 * j) = q;
                } else {
                    row[16 * j] = (uint16_t)q.x;
                    row[16 * j + 1] = (uint16_t)(q.x >> 16);
                    row[16 * j + 2] = (uint16_t)q.y;
                    row[16 * j + 3] = (uint16_t)(q.y >> 16);
                }
            }
        }
        __builtin_amdgcn_wave_barrier();   // LDS executes a wave's accesses in order
        if (whole) {
            if (vc < kRowVecs) {
                out_t* to = dst + (mw + vr) * N + nw + vc * kVec;
                const out_t* from = rows + vr * kPitch + vc * kVec;
#pragma unroll
                for (int t = 0; t < 16 / kRowStep; ++t)
                    *reinterpret_cast<uint4*>(to + t * kRowStep * N) = *reinterpret_cast<const uint4*>(from + t * kRowStep * kPitch);
            }
        } else {
            for (int t = 0; t < 16 / kRowStep; ++t)
                if (vc < kRowVecs) store_vec(mw, vr + t * kRowStep, vc);
            if (N % kVec != 0 && lane < 16) store_vec(mw, lane, kRowVecs);
        }
        __builtin_amdgcn_wave_barrier();
    }
}

template <int kMI, int kNI, int kWM, int kWN, int kStages, bool kPartial, bool kSparse = false>
__global__ __launch_bounds__(64 * kWM * kWN, 1) void frag_gemm_kernel(
    const uint16_t* __restrict__ x, int64_t M, int64_t K, int64_t N, const uint16_t* wf,
    const uint16_t* __restrict__ t, int Rpad, uint16_t* __restrict__ y, int m_tiles, int n_tiles, int ksplit,
    float* __restrict__ partial) {
    __shared__ __attribute__((aligned(16))) uint16_t lds[frag_gemm_lds_bytes<kMI, kNI, kWM, kWN, kStages, kPartial>() / 2];
    frag_gemm_block<kMI, kNI, kWM, kWN, kStages, kPartial, kSparse>(x, M, K, N, wf, t, Rpad, y, m_tiles, n_tiles, ksplit, partial, lds);
}

// The same with the adapter gradients of a backward pass beside it (salr_row_products.hpp), on tiles of which two workgroups fit a CU: workgroups
// behind the stage's `gemm_blocks`, so that they take what room the CUs have left.  The stage keeps the matrix cores busy and those stream X and dY.
// 2048 x 4096 x 4096 rank 32: 99.4 us a step with two launches behind the stage (12.5 and 4.9 us), 89.4 so.
// (Three workgroups a CU on the smaller tiles: four rank tiles take 172 registers of a wave if left alone, and two workgroups cost
// 512 x 2048 x 1024 rank 64 29.7 us for 27.3, 1024 x 2048 x 2048 44.3 for 36.5.)
template <int kMI, int kNI, bool kPartial, int kRT>
__global__ __launch_bounds__(256, kMI == 2 && kNI <= 4 && kRT == 4 ? 3 : 2) void frag_gemm_gradients_kernel(
    const uint16_t* __restrict__ x, int64_t M, int64_t K, int64_t N, const uint16_t* wf,
    const uint16_t* __restrict__ t, int Rpad, uint16_t* __restrict__ y, int m_tiles, int n_tiles, int ksplit,
    float* __restrict__ partial, int gemm_blocks, RowProducts products) {
    constexpr int kBytes = frag_gemm_lds_bytes<kMI, kNI, 2, 2, 3, kPartial>();
    __shared__ __attribute__((aligned(16))) uint16_t lds[(kBytes > kTnLdsBytes ? kBytes : kTnLdsBytes) / 2];
    if ((int)blockIdx.x < gemm_blocks) {   // the same for the whole workgroup
        frag_gemm_block<kMI, kNI, 2, 2, 3, kPartial, false>(x, M, K, N, wf, t, Rpad, y, m_tiles, n_tiles, ksplit, partial, lds);
        return;
    }
    const int id = (int)blockIdx.x - gemm_blocks, blocks = row_product_blocks(products.C[0]) + row_product_blocks(products.C[1]);
    tall_tn_block<kRT, true>(products, id % blocks, id / blocks, lds);
}

static unsigned gemm_grid(int workgroups) { return (unsigned)((workgroups + kGemmXcds - 1) / kGemmXcds * kGemmXcds); }

// A_cat^T in operand order: block (f, kb) = ranks 16 f .. 16 f + 15 (rows past R as zeros) x columns 32 kb .. + 31; an even
// number of blocks per f, as for a weight.  Wave `part` of `parts` takes every parts-th kb.
__device__ __forceinline__ void adapter_frags_block(const uint16_t* __restrict__ a_cat, int64_t K, int R, int Rpad, int part, int parts,
                                                    uint16_t* af) {
    const int lane = lane_id(), i16 = lane & 15, g = lane >> 4;
    const int64_t blocks = (K + 63) / 64 * 2;
    for (int64_t kb = part; kb < blocks; kb += parts) {
        for (int f = 0; f < Rpad / 16; ++f) {
            const int r = 16 * f + i16;
            uint32_t e[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int64_t k = 32 * kb + 8 * g + j;
                const uint32_t v = a_cat[(k < K ? k : K - 1) * R + (r < R ? r : R - 1)];
                e[j] = r < R && k < K ? v : 0u;
            }
            *reinterpret_cast<uint4*>(af + (f * blocks + kb) * 512 + lane * 8) =
                make_uint4(e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16));
        }
    }
}

constexpr int kDfWaves = 4;
constexpr int kDfWords = 8;           // bitmap words of a piece
constexpr int kDfPitch = 140;         // dwords of LDS per row: 33 vectors of 16 bytes and a spread of the 16 rows over the banks
constexpr int kDfAhead = 3;           // vectors per lane and row half fetched ahead: pieces of up to 24 vectors (~70 % dense)

template <bool kPair, bool kNf4>
__global__ __launch_bounds__(kDfWaves * 64, 4) void decode_frag_kernel(const uint32_t* __restrict__ bitmap,
                                                                   const uint16_t* __restrict__ values,
                                                                   const uint32_t* __restrict__ row_offsets, int64_t N, int64_t K,
                                                                   int ksl, const uint16_t* __restrict__ b_cat, int R, int Rpad,
                                                                   const uint16_t* __restrict__ scales, uint32_t scale_last,
                                                                   uint16_t* wf, int a_blocks, const uint16_t* __restrict__ a_cat,
                                                                   uint16_t* __restrict__ af, int t_blocks, const uint16_t* __restrict__ x,
                                                                   int64_t M, uint16_t* __restrict__ t) {
    __shared__ __attribute__((aligned(16))) uint32_t slots[kDfWaves][16 * kDfPitch];
    if ((int)blockIdx.x < t_blocks) {   // the same for the whole workgroup
        static_assert(sizeof(slots) >= adapter_t_lds_bytes<2, kDfWaves>() && sizeof(slots) >= adapter_t_lds_bytes<1, kDfWaves>(), "room for T's tiles");
        adapter_t_block_of<kDfWaves, true>(x, M, K, a_cat, R, Rpad, t, (int)blockIdx.x, reinterpret_cast<uint16_t*>(slots));
        return;
    }
    if ((int)blockIdx.x < a_blocks) {
        adapter_frags_block(a_cat, K, R, Rpad, (int)blockIdx.x * kDfWaves + (threadIdx.x >> 6), a_blocks * kDfWaves, af);
        return;
    }
    __shared__ __attribute__((aligned(16))) uint32_t words_lds[kDfWaves][16 * kDfWords];
    __shared__ uint32_t lut[kNibbleLutWords];
    __shared__ float levels[16];
    __shared__ uint32_t counts[2][kDfWaves][16];   // nonzeros per row: left of the workgroup (a quarter each), of the wave's slice
    nibble_lut_init(lut);
    if (kNf4 && threadIdx.x < 16) levels[threadIdx.x] = kNf4Levels[threadIdx.x];
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, g = lane >> 4;
    const int64_t frags = (N + 15) >> 4, id = (int64_t)blockIdx.x - a_blocks - t_blocks;   // (at most one of the two)
    const int64_t f = id % frags;
    const int z = (int)(id / frags) * kDfWaves + wave;
    const int64_t row = 16 * f + n < N ? 16 * f + n : N - 1;   // rows past N: copies of the last one, their outputs are dropped
    const int64_t wpr = K >> 5, pieces = (wpr + kDfWords - 1) / kDfWords;
    const int64_t w_blocks = (wpr + 1) / 2 * 2, r_blocks = (Rpad + 63) / 64 * 2, blocks = w_blocks + r_blocks;
    const int64_t p_begin = pieces * z / ksl, p_end = pieces * (z + 1) / ksl;
    uint16_t* out = wf + f * blocks * 512 + lane * 8;
    const uint32_t* brow = bitmap + row * wpr;
    uint32_t cur = row_offsets[row];   // index in `values` of the row's next value, the same in its four lanes

    auto load_words = [&](int64_t p) -> uint2 {   // words 2 g, 2 g + 1 of piece p; past the slice or the row they are empty
        const int64_t w = kDfWords * p + 2 * g;
        const bool ok0 = p < p_end && w < wpr, ok1 = p < p_end && w + 1 < wpr;
        uint2 q;
        if constexpr (kPair) {
            q = *reinterpret_cast<const uint2*>(brow + (ok0 ? w : 0));
        } else {
            q.x = brow[ok0 ? w : 0];
            q.y = brow[ok1 ? w + 1 : 0];
        }
        return make_uint2(ok0 ? q.x : 0u, ok1 ? q.y : 0u);
    };
    uint2 b0 = load_words(p_begin), b1 = load_words(p_begin + 1);
    // nonzeros of the row in pieces [p0, p1): the four lanes of a row share the words
    auto count_pieces = [&](int64_t p0, int64_t p1) -> uint32_t {
        const int64_t end = kDfWords * p1 < wpr ? kDfWords * p1 : wpr;
        uint32_t c = 0;
        if ((wpr & 3) == 0) {   // whole 16-byte vectors, eight requests in flight each
            for (int64_t w0 = kDfWords * p0; w0 < end; w0 += 128) {
                uint4 q[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int64_t w = w0 + 16 * i + 4 * g;
                    q[i] = *reinterpret_cast<const uint4*>(brow + (w < end ? w : 0));
                }
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    c += w0 + 16 * i + 4 * g < end ? __popc(q[i].x) + __popc(q[i].y) + __popc(q[i].z) + __popc(q[i].w) : 0u;
            }
        } else {
            for (int64_t w0 = kDfWords * p0; w0 < end; w0 += 32) {
                uint32_t q[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) q[i] = brow[w0 + 4 * i + g < end ? w0 + 4 * i + g : 0];
#pragma unroll
                for (int i = 0; i < 8; ++i) c += w0 + 4 * i + g < end ? __popc(q[i]) : 0u;
            }
        }
        c += __shfl_xor(c, 16, 64);
        return c + __shfl_xor(c, 32, 64);
    };
    const int64_t left = pieces * (z - wave) / ksl;   // pieces left of the workgroup
    const uint32_t left_count = count_pieces(left * wave / kDfWaves, left * (wave + 1) / kDfWaves);
    const uint32_t own_count = count_pieces(p_begin, p_end);
    if (g == 0) {
        counts[0][wave][n] = left_count;
        counts[1][wave][n] = own_count;
    }
    __syncthreads();   // (the lookup tables, too)
#pragma unroll
    for (int w = 0; w < kDfWaves; ++w) cur += counts[0][w][n] + (w < wave ? counts[1][w][n] : 0u);
    for (int rb = z; rb < r_blocks; rb += ksl) {
        uint32_t e[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int rr = 32 * rb + 8 * g + j;
            const uint32_t v = b_cat[(int64_t)(rr < R ? rr : R - 1) * N + row];
            e[j] = rr < R ? v : 0u;
        }
        *reinterpret_cast<uint4*>(out + (w_blocks + rb) * 512) = make_uint4(e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16));
    }
    if (p_begin >= p_end) return;

    const uint4* values128 = reinterpret_cast<const uint4*>(values);
    const uint32_t* codes32 = reinterpret_cast<const uint32_t*>(values);
    uint32_t* slot = slots[wave];
    uint32_t* my_words = words_lds[wave];
    const int r8 = lane >> 3, l8 = lane & 7;   // value loader: rows r8 and r8 + 8, vector l8 of every eight
    struct Stage {
        uint2 bw;
        uint32_t off;               // element offset of this row's piece in its first vector
        uint32_t base[2], nv[2];    // first vector and number of vectors of the pieces of rows r8, r8 + 8
        uint4 v[2][kDfAhead];
    };
    auto fetch = [&](uint32_t base, uint32_t nv, uint32_t v) -> uint4 {   // vector v of a piece, clamped to its last
        const uint32_t j = base + (v < nv ? v : nv - 1u);
        if constexpr (kNf4) {
            const uint32_t i = nv ? j : 0u, blk = i >> 3;
            return make_uint4(codes32[i], scales[blk < scale_last ? blk : scale_last], 0u, 0u);
        } else {   // an empty piece reads what is always there
            return *(nv ? values128 + j : reinterpret_cast<const uint4*>(out));
        }
    };
    auto issue = [&](Stage& st, const uint2 bw) {
        st.bw = bw;
        uint32_t len = __popc(bw.x) + __popc(bw.y);
        len += __shfl_xor(len, 16, 64);
        len += __shfl_xor(len, 32, 64);
        st.off = cur & 7u;
        const uint32_t vec = cur >> 3, nvec = len ? (st.off + len + 7u) >> 3 : 0u;
        cur += len;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            st.base[h] = __shfl(vec, r8 + 8 * h, 64);
            st.nv[h] = __shfl(nvec, r8 + 8 * h, 64);
#pragma unroll
            for (int i = 0; i < kDfAhead; ++i) st.v[h][i] = fetch(st.base[h], st.nv[h], l8 + 8 * i);
        }
    };
    auto park = [&](int h, uint32_t v, const uint4& q) {
        uint4 d = q;
        if constexpr (kNf4) d = nf4_decode8(q.x, bf16_bits_to_f32(q.y), levels);
        *reinterpret_cast<uint4*>(slot + (r8 + 8 * h) * kDfPitch + 4 * v) = d;
    };
    auto consume = [&](const Stage& st, int64_t p) {
        *reinterpret_cast<uint2*>(my_words + n * kDfWords + 2 * g) = st.bw;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int i = 0; i < kDfAhead; ++i) park(h, l8 + 8 * i, st.v[h][i]);
            // more values than were fetched ahead: the rest now (at most 33 vectors)
            for (uint32_t v = l8 + 8 * kDfAhead; v < st.nv[h]; v += 8) park(h, v, fetch(st.base[h], st.nv[h], v));
        }
        __builtin_amdgcn_wave_barrier();   // LDS executes a wave's accesses in order
        const uint4 wa = *reinterpret_cast<const uint4*>(my_words + n * kDfWords), wb = *reinterpret_cast<const uint4*>(my_words + n * kDfWords + 4);
        const uint32_t words[kDfWords] = {wa.x, wa.y, wa.z, wa.w, wb.x, wb.y, wb.z, wb.w};
        uint32_t at = st.off;
        const uint32_t below = (1u << (8 * g)) - 1u;
#pragma unroll
        for (int s = 0; s < kDfWords; ++s) {
            const uint4 q = expand_byte(slot + n * kDfPitch, lut, at + __popc(words[s] & below), (words[s] >> (8 * g)) & 0xFFu);
            at += __popc(words[s]);
            const int64_t kb = kDfWords * p + s;
            if (kb < w_blocks) *reinterpret_cast<uint4*>(out + kb * 512) = q;
        }
        __builtin_amdgcn_wave_barrier();
    };
    Stage s0, s1;
    issue(s0, b0);
    b0 = load_words(p_begin + 2);
    for (int64_t p = p_begin; p < p_end; p += 2) {
        issue(s1, b1);
        b1 = load_words(p + 3);
        consume(s0, p);
        issue(s0, b0);
        b0 = load_words(p + 4);
        if (p + 1 < p_end) consume(s1, p + 1);   // wave-uniform
    }
}

// af: A_cat in operand order, too (null: not wanted); t: T = X A_cat, too, in the launch's first workgroups (null: not wanted; only where
// adapter_t_beside, and not both).  The two have nothing to do with each other, T is a chain of round trips on a few CUs and
// the decode pass fills the memory system: 300 x 2720 x 2731 38.6 -> 32.4 us a call, 2048 x 4096 x 14336
// 252 -> 244.
hipError_t launch_decode_frags(const LinearArgs& a, uint16_t* wf, uint16_t* af, uint16_t* t, hipStream_t stream) {
    const int R = (int)a.R, Rpad = (int)adapter_rank_padded(a.R);
    const int64_t frags = (a.N + 15) / 16, pieces = (a.K + 255) / 256;
    // one round of the four workgroups that fit a CU, more only where the rows are many; two pieces at least to a wave
    int64_t split = 1024 / frags;
    if (split > pieces / (2 * kDfWaves)) split = pieces / (2 * kDfWaves);
    if (split < 1) split = 1;
    const int64_t ksl = split * kDfWaves;
    const int a_blocks = af != nullptr ? (int)((a.K + 32 * kDfWaves - 1) / (32 * kDfWaves)) : 0;
    const int t_blocks = t != nullptr ? adapter_t_blocks<true>(a.M, Rpad) : 0;
    const dim3 grid((unsigned)(t_blocks + a_blocks + frags * split)), block(kDfWaves * 64);
    const uint16_t* src = a.codes != nullptr ? reinterpret_cast<const uint16_t*>(a.codes) : a.values;
    const uint32_t scale_last = a.codes != nullptr ? (uint32_t)((a.nnz + kNf4Block - 1) / kNf4Block - 1) : 0u;
#define SALR_DECODE(PAIR, NF4) \
    hipLaunchKernelGGL((decode_frag_kernel<PAIR, NF4>), grid, block, 0, stream, a.bitmap, src, a.row_offsets, a.N, a.K, (int)ksl, \
                       a.b_cat, R, Rpad, a.scales, scale_last, wf, a_blocks, a.a_cat, af, t_blocks, a.x, a.M, t)
    const bool pair = a.K % 64 == 0;
    if (a.codes != nullptr) {
        if (pair) SALR_DECODE(true, true);
        else SALR_DECODE(false, true);
    } else {
        if (pair) SALR_DECODE(true, false);
        else SALR_DECODE(false, false);
    }
#undef SALR_DECODE
    return hipGetLastError();
}

bool launch_frag_gemm(const uint16_t* x, int64_t M, int64_t K, int64_t N, const uint16_t* wf, const uint16_t* t, int Rpad,
                      uint16_t* y, float* partial, size_t partial_room, const TimingEvents& ev, hipStream_t stream, const RowProducts* beside) {
    const GemmPlan p = gemm_plan(M, K + Rpad, N, partial_room);
    const int m_tiles = (int)((M + p.mt - 1) / p.mt), n_tiles = (int)((N + p.nt - 1) / p.nt);
    const dim3 grid(gemm_grid(m_tiles * n_tiles * p.ksplit));
    // (mt, nt: two of the stage's workgroups fit a CU up to 128 x 256; four rank tiles a pass have the registers up to 128 x 128)
    const bool four = Rpad % 64 == 0 && p.mt * p.nt <= 128 * 128;
    if (beside != nullptr && gradients_beside(M, K, N, p, *beside)) {
        RowProducts products = *beside;
        if (products.ksplit > kBesideSlices) products.ksplit = kBesideSlices;
        const int blocks = (row_product_blocks(products.C[0]) + row_product_blocks(products.C[1])) * products.ksplit;
        const dim3 all(grid.x + (unsigned)blocks);
#define SALR_TN_P(MI, NI, P, RT)                                                                                                                \
    hipLaunchKernelGGL((frag_gemm_gradients_kernel<MI, NI, P, RT>), all, dim3(256), 0, stream, x, M, K, N, wf, t, Rpad, y, m_tiles, n_tiles, \
                       p.ksplit, partial, (int)grid.x, products)
#define SALR_TN(MI, NI, RT)                          \
    do {                                             \
        if (p.ksplit > 1) SALR_TN_P(MI, NI, true, RT); \
        else SALR_TN_P(MI, NI, false, RT);           \
    } while (0)
#define SALR_TN24(MI, NI)           \
    do {                            \
        if (four) SALR_TN(MI, NI, 4); \
        else SALR_TN(MI, NI, 2);    \
    } while (0)
        if (p.mt == 128 && p.nt == 256) SALR_TN(4, 8, 2);
        else if (p.mt == 128) SALR_TN24(4, 4);
        else if (p.nt == 256) SALR_TN24(2, 8);
        else if (p.nt == 128) SALR_TN24(2, 4);
        else SALR_TN24(2, 2);
#undef SALR_TN24
#undef SALR_TN
#undef SALR_TN_P
        if (p.ksplit > 1) launch_splitk_reduce(partial, M * N, p.ksplit, y, stream);
        return true;
    }
#define SALR_GEMM_P(MI, NI, P)                                                                                                     \
    SALR_LAUNCH((frag_gemm_kernel<MI, NI, 2, 2, 3, P>), grid, dim3(256), stream, ev, x, M, K, N, wf, t, Rpad, y, m_tiles, n_tiles, \
                p.ksplit, partial)
#define SALR_GEMM(MI, NI)                        \
    do {                                         \
        if (p.ksplit > 1) SALR_GEMM_P(MI, NI, true); \
        else SALR_GEMM_P(MI, NI, false);         \
    } while (0)
    if (p.mt == 256 && p.nt == 256) SALR_GEMM(8, 8);
    else if (p.mt == 256) SALR_GEMM(8, 7);
    else if (p.mt == 128 && p.nt == 256) SALR_GEMM(4, 8);
    else if (p.mt == 128) SALR_GEMM(4, 4);
    else if (p.nt == 256) SALR_GEMM(2, 8);
    else if (p.nt == 128) SALR_GEMM(2, 4);
    else SALR_GEMM(2, 2);
#undef SALR_GEMM
#undef SALR_GEMM_P
    if (p.ksplit > 1) launch_splitk_reduce(partial, M * N, p.ksplit, y, stream);
    return false;
}

// T = X * A_cat straight to bf16 [M, Rpad] in one launch (more than kAdapterSmallM rows): sixteen waves per 32 rows and 32 ranks.
__global__ __launch_bounds__(1024) void adapter_t_direct_kernel(const uint16_t* __restrict__ x, int64_t M, int64_t K,
                                                                const uint16_t* __restrict__ a_cat, int R, int Rpad,
                                                                uint16_t* __restrict__ t) {
    __shared__ __attribute__((aligned(16))) uint16_t lds[adapter_t_lds_bytes<2, 16>() / 2];
    const int groups = Rpad >> 5;
    adapter_t_block<2, 16, 2>(x, M, K, a_cat, R, Rpad, t, blockIdx.x / groups, (int)blockIdx.x % groups, lds);
}

void launch_adapter_t_direct(const uint16_t* x, int64_t M, int64_t K, const uint16_t* a_cat, int R, int Rpad, uint16_t* t,
                             hipStream_t stream) {
    const dim3 grid((unsigned)((M + 31) / 32 * (Rpad / 32)));
    hipLaunchKernelGGL(adapter_t_direct_kernel, grid, dim3(1024), 0, stream, x, M, K, a_cat, R, Rpad, t);
}

// T = X * A_cat as a product with A_cat in operand order (af): 256 rows x all ranks (128 at a time) per workgroup, K split over
// as many workgroups as the chip holds, fp32 partial sums, their sum to bf16 [M, Rpad] (padding columns as zeros: an infinite
// entry of X made the products with their zero rows NaN, and those every output of the row).
static void launch_adapter_t_product(const uint16_t* x, int64_t M, int64_t K, const uint16_t* af, int R, int Rpad, uint16_t* t,
                                     float* partial, hipStream_t stream) {
    const int m_tiles = (int)((M + 255) / 256), nt = Rpad <= 32 ? 32 : Rpad <= 64 ? 64 : 128, n_tiles = (Rpad + nt - 1) / nt;
    const int ks = adapter_t_product_ksplit(M, K, Rpad);
    const dim3 grid(gemm_grid(m_tiles * n_tiles * ks));
    const uint16_t* no_t = nullptr;
#define SALR_TGEMM(NI)                                                                                                         \
    hipLaunchKernelGGL((frag_gemm_kernel<4, NI, 4, 1, 3, true>), grid, dim3(256), 0, stream, x, M, K, (int64_t)Rpad, af, no_t, 0, t, \
                       m_tiles, n_tiles, ks, partial)
    if (nt == 32) SALR_TGEMM(2);
    else if (nt == 64) SALR_TGEMM(4);
    else SALR_TGEMM(8);
#undef SALR_TGEMM
    launch_splitk_reduce(partial, M * Rpad, ks, t, stream, Rpad, R);
}

hipError_t launch_linear_frag(const LinearArgs& a, hipStream_t stream, const TimingEvents& ev) {
    const int Rpad = (int)adapter_rank_padded(a.R);
    uint16_t* wf = reinterpret_cast<uint16_t*>(reinterpret_cast<char*>(a.t) + frag_weight_offset(a.M, a.K, a.R));
    // T beside the decode pass, or as a product of its own whose operand that pass lays out
    char* af = reinterpret_cast<char*>(a.t) + adapter_t_bytes(a.M, a.R);
    const bool own = a.R > 0 && !adapter_t_beside(a.M, a.K, a.R);
    const hipError_t e = launch_decode_frags(a, wf, own ? reinterpret_cast<uint16_t*>(af) : nullptr, a.R > 0 && !own ? a.t : nullptr, stream);
    if (e != hipSuccess) return e;
    if (own)
        launch_adapter_t_product(a.x, a.M, a.K, reinterpret_cast<const uint16_t*>(af), (int)a.R, Rpad, a.t,
                                 reinterpret_cast<float*>(af + adapter_frag_bytes(a.K, a.R)), stream);
    const size_t base = frag_base_bytes(a.M, a.K, a.N, a.R);
    float* partial = reinterpret_cast<float*>(reinterpret_cast<char*>(a.t) + base);
    launch_frag_gemm(a.x, a.M, a.K, a.N, wf, a.t, Rpad, a.y, partial, a.room - base, ev, stream, nullptr);
    return hipGetLastError();
}

// Sparse operand order of a 2:4-masked weight, B_cat behind it: a permutation of the packed values and the bitmap, no decode.
// Pair (f, p) is 16 weight rows x 128 columns: for each of its two steps of 64 columns 1 KB of values, lane (n, kb) = lane kb 16 +
// n holding two sets of four (columns c .. c + 7 and c + 16 .. c + 23 with c = 32 (kb % 2) + 8 (kb / 2)), then a word per lane with
// the positions of both steps (the index field of v_smfmac_f32_16x16x64_bf16 in the low and the high half; a last single step
// leaves the second half of its pair unread).  Behind the pairs of an f the rank blocks of B_cat, dense, 32 ranks each.
// The first t_blocks workgroups compute T = X A_cat meanwhile (any16 = X; 16 rows and 32 ranks each).
// Value offsets are clamped to the stored count: the 2:4 form is the caller's promise.  Bound by memory: 14336 x 4096, 66 MB in
// and 66 out, 28.7 us.
__global__ __launch_bounds__(256, 5) void pack_2of4_kernel(const uint32_t* __restrict__ bitmap, const uint16_t* __restrict__ values,
                                                        const uint32_t* __restrict__ row_offsets, const uint16_t* __restrict__ any16,
                                                        int64_t N, int64_t K, int split, const uint16_t* __restrict__ b_cat, int R,
                                                        int Rpad, uint16_t* __restrict__ wf, int t_blocks, int64_t M,
                                                        const uint16_t* __restrict__ a_cat, uint16_t* __restrict__ t) {
    if ((int)blockIdx.x < t_blocks) {   // the same for the whole workgroup
        __shared__ __attribute__((aligned(16))) uint16_t lds[adapter_t_lds_bytes<1, 4>() / 2];
        adapter_t_block_of<4, false>(any16, M, K, a_cat, R, Rpad, t, (int)blockIdx.x, lds);
        return;
    }
    const int lane = lane_id(), n = lane & 15, kb = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t frags = (N + 15) / 16, id = ((int64_t)blockIdx.x - t_blocks) * 4 + wave;
    const int64_t f = id / split;
    const int z = (int)(id % split);
    if (f >= frags) return;   // wave-uniform; the kernel has no barrier
    const int64_t row = 16 * f + n < N ? 16 * f + n : N - 1;   // rows past N: copies of the last one, their outputs are dropped
    const int64_t steps = K / 64, pairs = (steps + 1) / 2, frag = sparse_frag_elems(K, Rpad), wpr = K / 32;
    const int64_t p_begin = pairs * z / split, p_end = pairs * (z + 1) / split;
    uint16_t* out = wf + f * frag;
    const uint32_t nnz = row_offsets[N], e_max = nnz >= 8u ? nnz - 8u : 0u;
    const uint16_t* vsrc = nnz >= 8u ? values : any16;   // (a weight this small cannot meet the precondition)
    const uint32_t first = row_offsets[row] + 16u * (uint32_t)(kb & 1);
    const int half = 4 * (kb >> 1), sh = 8 * (kb >> 1);
    const uint32_t* brow = bitmap + row * wpr + (kb & 1);
    auto set = [&](int64_t step, uint32_t h) -> uint2 {   // four values of the vector of eight that holds them
        uint32_t e = first + 32u * (uint32_t)step + 8u * h;
        e = (e < e_max ? e : e_max) & ~7u;
        return *reinterpret_cast<const uint2*>(vsrc + e + half);
    };
    auto code = [&](uint32_t word) -> uint32_t {
        const uint32_t cw = index_codes_2of4(word);
        return ((cw >> sh) & 0xFFu) | ((cw >> (sh + 8)) & 0xFF00u);
    };
    constexpr int kAhead = 4;
    for (int64_t p0 = p_begin; p0 < p_end; p0 += kAhead) {
        uint2 v[kAhead][4];
        uint32_t b[kAhead][2];
#pragma unroll
        for (int d = 0; d < kAhead; ++d) {
            const int64_t p = p0 + d < p_end ? p0 + d : p_end - 1;
            const int64_t s1 = 2 * p + 1 < steps ? 2 * p + 1 : 2 * p;
            v[d][0] = set(2 * p, 0);
            v[d][1] = set(2 * p, 1);
            v[d][2] = set(s1, 0);
            v[d][3] = set(s1, 1);
            b[d][0] = brow[4 * p];
            b[d][1] = brow[2 * s1];
        }
#pragma unroll
        for (int d = 0; d < kAhead; ++d) {
            if (p0 + d < p_end) {   // wave-uniform
                uint16_t* to = out + (p0 + d) * kSparsePairElems;
                *reinterpret_cast<uint4*>(to + 8 * lane) = make_uint4(v[d][0].x, v[d][0].y, v[d][1].x, v[d][1].y);
                *reinterpret_cast<uint4*>(to + 512 + 8 * lane) = make_uint4(v[d][2].x, v[d][2].y, v[d][3].x, v[d][3].y);
                *reinterpret_cast<uint32_t*>(to + 1024 + 2 * lane) = code(b[d][0]) | (code(b[d][1]) << 16);
            }
        }
    }
    for (int rb = z; rb < Rpad / 32; rb += split) {
        uint32_t e[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int r = 32 * rb + 8 * kb + j;
            const uint32_t q = b_cat[(int64_t)(r < R ? r : R - 1) * N + row];
            e[j] = r < R ? q : 0u;
        }
        *reinterpret_cast<uint4*>(out + pairs * kSparsePairElems + rb * 512 + 8 * lane) =
            make_uint4(e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16));
    }
}

// y = x W^T + t B_cat on the sparse matrix cores: the weight into sparse operand order at wf (sparse_weight_bytes), then tiles of
// 256 x 256 or 256 x 224.  K % 64 == 0.  with_t: T first, beside the permutation (adapter_t_in_pass).
void launch_sparse_gemm(const LinearArgs& a, uint16_t* wf, bool narrow, bool with_t, const TimingEvents& ev, hipStream_t stream) {
    const int R = (int)a.R, Rpad = (int)adapter_rank_padded(a.R);
    const int64_t frags = (a.N + 15) / 16, pairs = (a.K / 64 + 1) / 2;
    int64_t split = (8192 + frags - 1) / frags;   // about eight waves per SIMD, four pairs at least to a wave
    if (split > pairs / 4) split = pairs / 4;
    if (split < 1) split = 1;
    const int t_blocks = with_t ? adapter_t_blocks<false>(a.M, Rpad) : 0;
    hipLaunchKernelGGL(pack_2of4_kernel, dim3((unsigned)(t_blocks + (frags * split + 3) / 4)), dim3(256), 0, stream, a.bitmap, a.values,
                       a.row_offsets, a.x, a.N, a.K, (int)split, a.b_cat, R, Rpad, wf, t_blocks, a.M, a.a_cat, a.t);
    const int nt = narrow ? 224 : 256, m_tiles = (int)((a.M + 255) / 256), n_tiles = (int)((a.N + nt - 1) / nt);
    const dim3 grid(gemm_grid(m_tiles * n_tiles));
    float* none = nullptr;
    const uint16_t* t = a.t;
#define SALR_SPARSE(NI)                                                                                                              \
    SALR_LAUNCH((frag_gemm_kernel<8, NI, 2, 2, 3, false, true>), grid, dim3(256), stream, ev, a.x, a.M, a.K, a.N, (const uint16_t*)wf, t, \
                Rpad, a.y, m_tiles, n_tiles, 1, none)
    if (narrow) SALR_SPARSE(7);
    else SALR_SPARSE(8);
#undef SALR_SPARSE
}

}  // namespace salr
