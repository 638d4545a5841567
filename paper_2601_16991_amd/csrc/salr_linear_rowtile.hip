// Row-tiled streaming path of the SALR linear (paper Sec. 3.2 / 3.3) for batches of up to 128 tokens: one pass over the
// compressed weight, the activations shared inside a workgroup through LDS.
//
// A workgroup of eight waves has a CU to itself and takes 128 consecutive rows of What and one slice of K; wave w owns rows
// 16 w .. 16 w + 15 of them for the whole slice.
//   weights      the wave's own stream (salr_row_stream.hpp): bitmap words four chunks at a time, packed values (or their 4-bit codes
//                and block scales, dequantised on the way into LDS) one unit ahead in registers, parked in the wave's LDS slot,
//                expanded straight into an MFMA operand.  A unit is a pair of chunks, one from 65 tokens on.
//   activations  a panel of X (64 KB: 16 chunks of 16 tokens, 4 of 64) is copied to LDS once per workgroup, the next one on its way
//                in registers meanwhile.  No barrier inside a panel: the waves drift apart and the requests of one meet the
//                expansion of another.
//   adapters     T = X A_cat needs all of K before it can be used, so it belongs to neither side of a split of K: the first
//                workgroups of the same launch write its split-K partial sums, and the launch that adds up the slices' partial
//                outputs multiplies T with B_cat and adds that too.  (With a launch of its own in front it cost 4.4 us of the
//                34.9 us of a 16 x 4096 x 14336 call.)
// Where the row tiles alone fill a round of the CUs (rowtile_plan), K is not split over workgroups: 128, 64 or 32 rows a workgroup, the
// waves on one, two or four parts of K beside each other (Q), added up in LDS.  T, formed 3 to 7 us into the launch, is then handed over
// inside it (salr_handover.hpp) and there is no second launch, which takes 4 to 5 us (figures at rowtile_plan).  A part's panels of X are that
// much shorter, and every barrier costs the waves their lead: 0.8 us of a 16 x 4096 x 14336 call.
// The work is cut so that there is one workgroup per CU and one round of them where that can be (rowtile_plan): a slice starts
// with two dependent round trips to memory and the popcounts of the bitmap left of it, 4 us, and the longer a slice the less often
// that is paid.  Two workgroups per CU (half the slice, 128 registers a wave) hide each other's start, but spill: 30.5 us a call.
//
// us a call at p = .5, rank 32, of the kernel before this one (two workgroups per CU, a barrier per chunk or per four, T in a launch of its own) and
// now: 16 x 4096 x 14336 34.2 / 19.9, 32 tokens 37.5 / 22.6, 64 tokens 46.4 / 29.0, 128 tokens 53.8 / 38.5; 64 x 14336 x 4096 56.3 / 30.4;
// 16 x 8192 x 28672 rank 64 101 / 58.1.  The bytes of the first take 13 us at what a large copy reaches; its loop runs at 4.1 TB/s.
// Tried and left out: packed values two units ahead instead of one (+6 %); 32 weight rows per wave, which halves the operand
// reads of X (+18 % at 16 tokens: half as many slices' starts overlap); seven waves, so that 256 instead of 224
// workgroups share the rows of that layer (level); twelve waves on three parts (25.9 us where two took 22.0); the partial outputs of slices
// added up inside the launch by whoever comes last (see salr_handover.hpp); values fetched as whole 256-byte runs of a row, half as many cycles of the
// address unit (the transposition into conflict-free LDS columns then meets conflicts of its own).
#include <hip/hip_ext.h>

#include <type_traits>

#include "salr_handover.hpp"
#include "salr_internal.hpp"
#include "salr_nf4.hpp"
#include "salr_row_stream.hpp"

namespace salr {

constexpr int kRtWaves = 8;
constexpr int kRtThreads = 64 * kRtWaves;

// ---- T = X A_cat, split-K partials: one workgroup sums slice b of K for 16 rows of X and 16 ranks
// kShared: read by other workgroups of the launch, so stored past the caches.  (Where a launch behind it reads them that costs 0.2 to 0.3 us:
// 14 x 15360 x 801, R 64, a table: 17.6 us, 17.3 so.)
template <int W, bool kShared>
__device__ __forceinline__ void adapter_partial_block(const uint16_t* __restrict__ x, int M, int64_t K,
                                                      const uint16_t* __restrict__ a_cat, int R, int Rpad, int block, int slices,
                                                      float* __restrict__ t_partial, float* red, int tid) {
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i16 = lane & 15, g = lane >> 4;
    const int rank_tiles = Rpad >> 4;
    const int b = block % slices, rt = block / slices % rank_tiles, mt = block / (slices * rank_tiles);
    const int units = (int)(K >> 5);   // k-steps of 32 columns
    const int u_begin = units * b / slices, u_end = units * (b + 1) / slices;
    const int r = 16 * rt + i16, m = 16 * mt + i16;
    const int r_c = r < R ? r : R - 1;   // padding columns read a valid one and are zeroed at the store
    const uint16_t* xr = x + (int64_t)(m < M ? m : M - 1) * K + 8 * g;
    constexpr int kBatch = 4;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int u0 = u_begin + wave; u0 < u_end; u0 += W * kBatch) {
        uint4 aq[kBatch], bq[kBatch];
#pragma unroll
        for (int t = 0; t < kBatch; ++t) {
            const int u = u0 + W * t < u_end ? u0 + W * t : u_end - 1;
            aq[t] = *reinterpret_cast<const uint4*>(xr + 32 * (int64_t)u);
            uint32_t e[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) e[j] = a_cat[(32 * (int64_t)u + 8 * g + j) * R + r_c];
            bq[t] = make_uint4(e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16));
        }
#pragma unroll
        for (int t = 0; t < kBatch; ++t)
            if (u0 + W * t < u_end)   // uniform
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(aq[t]), as_bf16x8(bq[t]), acc, 0, 0, 0);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) red[(wave * 4 + e) * 64 + lane] = acc[e];
    __syncthreads();
    for (int i = tid; i < 256; i += 64 * W) {   // lane holds T[16 mt + 4 (lane / 16) + e][16 rt + lane % 16]
        const int l = i & 63, e = i >> 6;
        float s = 0.f;
#pragma unroll
        for (int w = 0; w < W; ++w) s += red[(w * 4 + e) * 64 + l];
        const int mm = 16 * mt + 4 * (l >> 4) + e, rr = 16 * rt + (l & 15);
        if (mm < M) {
            float* to = t_partial + ((int64_t)b * M + mm) * Rpad + rr;
            if constexpr (kShared) __hip_atomic_store(to, rr < R ? s : 0.f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            else *to = rr < R ? s : 0.f;
        }
    }
}

// four consecutive outputs of row m
__device__ __forceinline__ void store_four(uint16_t* __restrict__ y, int M, int64_t N, int m, int64_t col, const f32x4& v) {
    uint16_t* out = y + (int64_t)m * N + col;
    const uint32_t lo = f32_to_bf16_rne(v[0]) | ((uint32_t)f32_to_bf16_rne(v[1]) << 16);
    const uint32_t hi = f32_to_bf16_rne(v[2]) | ((uint32_t)f32_to_bf16_rne(v[3]) << 16);
    if (N % 4 == 0) {
        if (col < N) *reinterpret_cast<uint2*>(out) = make_uint2(lo, hi);
    } else {
        if (col < N) out[0] = (uint16_t)lo;
        if (col + 1 < N) out[1] = (uint16_t)(lo >> 16);
        if (col + 2 < N) out[2] = (uint16_t)hi;
        if (col + 3 < N) out[3] = (uint16_t)(hi >> 16);
    }
}

struct RowtileArgs {
    int t_blocks;        // leading workgroups that compute t_out
    int tiles, ksplit, t_slices;
    float* t_out;        // split-K partials of T written by this launch (kRowtileTSlices)
    const float* t_in;   // or those of an earlier one (kStreamTSlices): slice 0 adds the adapters
    float* partial;      // [ksplit, M, pitch] fp32, or null: y
    int64_t pitch;
    uint64_t* words;     // one slice that adds the adapters in this launch (salr_handover.hpp): a pair per sixteen rows, then t_blocks.  Or null
    uint16_t* t_sum;     // there: T, bf16 [M, Rpad]
    uint64_t tag;
    int polls;
};

// T B_cat for the sixteen rows of a wave, T past the caches
template <int MT>
struct RowtileAdapters {
    const uint16_t* b_cat;
    int M, R, Rpad, n, g;
    int64_t N, n0;
    Buffer t_sum;
    uint32_t e[8];   // B_cat and T of a rank step
    u32x4 tq[MT];

    __device__ __forceinline__ RowtileAdapters(const RowtileArgs& p, int64_t row0, int M_, int64_t N_, const uint16_t* b, int R_, int Rpad_, int lane)
        : b_cat(b), M(M_), R(R_), Rpad(Rpad_), n(lane & 15), g(lane >> 4), N(N_), n0(row0), t_sum(make_buffer(p.t_sum, (uint64_t)M_ * Rpad_ * 2)) {}
    __device__ __forceinline__ void load_b(int rs) {
        const int64_t n_c = n0 + n < N ? n0 + n : N - 1;
#pragma unroll
        for (int j = 0; j < 8; ++j) {   // (past R: dropped by ranks_below)
            const int r = rs * 32 + 8 * g + j;
            e[j] = (uint32_t)b_cat[(int64_t)(r < R ? r : R - 1) * N + n_c];
        }
    }
    __device__ __forceinline__ void load_t(int rs) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const int m = 16 * mt + n;
            tq[mt] = shared_load4(t_sum, (uint32_t)((m < M ? m : M - 1) * Rpad + rs * 32 + 8 * g) * 2);
        }
    }
    // B_cat and T of the first rank step have been asked for
    __device__ __forceinline__ void add(f32x4 (&acc)[MT]) {
        auto packed = [&]() { return make_uint4(e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16)); };
        auto multiply = [&](const uint4& bq) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
                acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(bq), __builtin_bit_cast(bf16x8, tq[mt]), acc[mt], 0, 0, 0);
        };
        const int last = (Rpad >> 5) - 1;
        for (int rs = 0; rs < last; ++rs) {
            __builtin_amdgcn_sched_barrier(0);
            multiply(packed());
            load_b(rs + 1);
            load_t(rs + 1);
        }
        __builtin_amdgcn_sched_barrier(0);
        multiply(ranks_below(packed(), last * 32 + 8 * g, R));
    }
};

// A wave's sums of X What^T in memory, for the case that T comes after them: element (m, column) as in a slice's partial outputs
template <int MT>
__device__ __forceinline__ void rowtile_sums(const RowtileArgs& p, int64_t n0, int M, int lane, bool store, f32x4 (&acc)[MT]) {
    const Buffer partial = make_buffer(p.partial, (uint64_t)M * p.pitch * 4);
    const int n = lane & 15;
    const int64_t col = n0 + 4 * (lane >> 4);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int m = 16 * mt + n;
        const uint32_t at = m < M && col < p.pitch ? (uint32_t)(m * p.pitch + col) * 4 : kPastBuffer;   // (stores past the buffer are dropped)
        if (store) shared_store4(partial, at, __builtin_bit_cast(u32x4, acc[mt]));
        else acc[mt] = __builtin_bit_cast(f32x4, shared_load4(partial, at));
    }
}

template <int MT>
__device__ __forceinline__ void rowtile_store(uint16_t* __restrict__ y, int64_t n0, int M, int64_t N, int lane, const f32x4 (&acc)[MT]) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
        if (16 * mt + (lane & 15) < M) store_four(y, M, N, 16 * mt + (lane & 15), n0 + 4 * (lane >> 4), acc[mt]);
}

// T's workgroups have met, this one came last: T from its partial sums, then T's side of every wave's pair.  Waves that came before T
// have left their sums to it.
template <int MT, int kGroups>
__device__ __forceinline__ void rowtile_hand_out_t(const RowtileArgs& p, int M, int64_t N, const uint16_t* __restrict__ b_cat, int R, int Rpad,
                                                   uint16_t* __restrict__ y, int tid) {
    const int groups = M * (Rpad >> 2);
    const Buffer parts = make_buffer(p.t_out, (uint64_t)p.t_slices * groups * 16), t_sum = make_buffer(p.t_sum, (uint64_t)groups * 8);
    for (int i = tid; i < groups; i += kRtThreads) {
        f32x4 v[kRowtileTSlices], sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int sl = 0; sl < kRowtileTSlices; ++sl)
            v[sl] = __builtin_bit_cast(f32x4, shared_load4(parts, 16u * (uint32_t)((sl < p.t_slices ? sl : 0) * groups + i)));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int sl = 0; sl < kRowtileTSlices; ++sl)
            if (sl < p.t_slices) sum += v[sl];
        shared_store2(t_sum, 8u * (uint32_t)i, u32x2{(uint32_t)f32_to_bf16_rne(sum[0]) | ((uint32_t)f32_to_bf16_rne(sum[1]) << 16),
                                                     (uint32_t)f32_to_bf16_rne(sum[2]) | ((uint32_t)f32_to_bf16_rne(sum[3]) << 16)});
    }
    stores_done();
    __syncthreads();
    const int lane = tid & 63, pairs = p.tiles * kGroups;
    for (int base = __builtin_amdgcn_readfirstlane(tid & ~63); base < pairs; base += kRtThreads) {
        const bool second = base + lane < pairs && meet(p.words + base + lane, p.tag);
        for (uint64_t left = __builtin_amdgcn_ballot_w64(second); left != 0; left &= left - 1) {   // uniform
            const int64_t n0 = (int64_t)(base + __builtin_ctzll(left)) * 16;
            RowtileAdapters<MT> adapters(p, n0, M, N, b_cat, R, Rpad, lane);
            f32x4 acc[MT];
            rowtile_sums<MT>(p, n0, M, lane, false, acc);
            adapters.load_b(0);
            adapters.load_t(0);
            adapters.add(acc);
            rowtile_store<MT>(y, n0, M, N, lane, acc);
        }
    }
}

// MT tiles of sixteen rows of X (M <= 16 MT).  kRagged: K is no multiple of 128.
// Q: the waves of a workgroup share 128 / Q rows, each sixteen of them on one of Q parts of the slice of K, and are added up through LDS.
// kOneLaunch: the only slice, which adds the adapters where p.words is set.
// kCodes: the packed values as 4-bit codes and block scales (`values` points at the codes).
template <int MT, bool kRagged, bool kCodes, int Q, bool kOneLaunch>
__global__ __launch_bounds__(kRtThreads, 2) void linear_rowtile_kernel(
    const uint16_t* __restrict__ x, int M, int64_t K, int64_t N, const uint32_t* __restrict__ bitmap,
    const void* __restrict__ values, const uint16_t* __restrict__ scales, const uint32_t* __restrict__ row_offsets,
    const uint32_t* __restrict__ slice_table, const uint16_t* __restrict__ a_cat, const uint16_t* __restrict__ b_cat, int R, int Rpad,
    uint16_t* __restrict__ y, RowtileArgs p) {
    constexpr int kTileBytes = 16 * MT * kChunkColumns * 2;           // X of one chunk
    constexpr int kGroups = kRtWaves / Q;                             // of sixteen rows
    constexpr int kPartPanel = 16 / MT / Q;                           // chunks of X in LDS, of each part
    constexpr int kPanelBytes = Q * kPartPanel * kTileBytes;          // 64 KB
    constexpr bool kPairs = MT <= 4;                                  // units of two chunks (else there are no registers for them)
    // vectors of a half's piece that starts anywhere in its first one: 128 or 64 values by 8, or codes by 32
    constexpr int kVectors = kCodes ? (kPairs ? 5 : 3) : (kPairs ? 17 : 9), kSlotBytes = slot_bytes(kCodes ? 4 * kVectors : kVectors + 1);
    __shared__ __attribute__((aligned(256))) char lds[256 + kPanelBytes + kRtWaves * kSlotBytes];   // tables, X, values
    const int tid = threadIdx.x;
    if ((int)blockIdx.x < p.t_blocks) {   // the same for the whole workgroup
        adapter_partial_block<kRtWaves, kOneLaunch>(x, M, K, a_cat, R, Rpad, (int)blockIdx.x, p.t_slices, p.t_out, reinterpret_cast<float*>(lds), tid);
        if (!kOneLaunch || p.words == nullptr) return;
        stores_done();
        __syncthreads();   // (the sums in LDS have been read, too)
        int* last = reinterpret_cast<int*>(lds);
        if (tid == 0) *last = knockout(p.words + (int64_t)p.tiles * kGroups, (int)blockIdx.x, p.t_blocks, p.tag);
        __syncthreads();
        if (*last != 0) rowtile_hand_out_t<MT, kGroups>(p, M, N, b_cat, R, Rpad, y, tid);
        return;
    }
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15;
    const int g = lane >> 4;
    const int id = (int)blockIdx.x - p.t_blocks;
    const int z = id / p.tiles, tile = id - z * p.tiles;
    const int part = wave / kGroups;
    const int64_t n0 = ((int64_t)tile * kGroups + wave % kGroups) * 16;
    const int64_t n0_c = n0 < N ? n0 : N;
    const int row_bytes = (int)(K >> 3);     // of the bitmap
    const int chunks = (int)((K + kChunkColumns - 1) / kChunkColumns);
    const int part_of_all = z * Q + part;
    const int c_begin = (int)((uint32_t)(chunks * part_of_all) / (uint32_t)(p.ksplit * Q));
    const int c_end = (int)((uint32_t)(chunks * (part_of_all + 1)) / (uint32_t)(p.ksplit * Q));
    // Chunks that the workgroup goes through: its slice's, or its longest part's (one slice).  With the longest slice's in every workgroup, two
    // rounds of slices of 18 and 19 chunks cost 3.5 % of a call: 8 x 7040 x 20224, R 32, a table: 38.4 us, 37.0 so.
    const int total_chunks = Q == 1 ? c_end - c_begin : (chunks + Q - 1) / Q;

    // ---- the wave's rows of the weight; rows past N read as empty
    const Buffer bits = make_buffer(bitmap + n0_c * (K >> 5), (uint64_t)(N - n0_c) * row_bytes);
    const uint32_t bits_lane = (uint32_t)n * row_bytes;
    // Chunk c starts at column 128 c, the last one of a row of uneven length at K - 128 and its words that belong to the chunk
    // before count as empty.  Chunks past the slice read as empty.
    auto chunk_start = [&](int c) -> int { return kRagged && (c + 1) * kChunkColumns > (int)K ? (int)K - kChunkColumns : c * kChunkColumns; };
    // Bitmap words of four chunks, chunk c + g to lane (n, g): one request of 64 bytes per row.  (One of 16 bytes per row and chunk,
    // the same to its four lanes, keeps the address unit busy for 31 ns whatever it fetches, this one for 20, a KB in one
    // piece for 8.)
    auto load_quad = [&](int c) -> u32x4 {
        const int ct = c + g;
        if constexpr (kRagged) {
            const int start = chunk_start(ct), over = ct * kChunkColumns - start;
            u32x4 q = buffer_load4(bits, ct < c_end ? bits_lane + (start >> 3) : kPastBuffer);
            q.x = over > 0 ? 0u : q.x;
            q.y = over > 32 ? 0u : q.y;
            q.z = over > 64 ? 0u : q.z;
            return q;
        } else {
            return buffer_load4(bits, ct < c_end ? bits_lane + 16 * ct : kPastBuffer);
        }
    };
    u32x4 quad = load_quad(c_begin);
    const int64_t row = n0 + n;
    // Index of the row's first value, or of its value at the last start of a table slice that is not behind this slice's; then the
    // nonzeros from there on (the four lanes of a row share the words).
    int walk_begin = 0;
    uint32_t cur;
    if (slice_table != nullptr) {
        const int w = kSliceTableSlices * c_begin / chunks;
        walk_begin = chunks * w / kSliceTableSlices;
        cur = slice_table[((row < N ? row : N - 1) * kSliceTableSlices + w) * 2];
    } else {
        cur = row_offsets[row < N ? row : N];
    }
    const uint32_t first = row_offsets[n0_c] & (kCodes ? ~63u : ~7u);   // the buffer of the wave's values starts here, in elements
    const uint32_t total = row_offsets[N];
    // The words left of the slice: a request takes sixteen chunks of four rows, 256 bytes each (four chunks of sixteen rows keep the address
    // unit busy for twice as long), and all of up to 112 chunks are in flight at once.  us a call, before / so: 8 x 14336 x 4096 at 70 % zeros
    // 24.5 / 22.4, 64 tokens 34.2 / 32.5, 16 x 12288 x 1024 17.9 / 14.9, 16 x 28672 x 8192 92.4 / 86.6; more of the old requests in flight
    // was worth 0.1 to 0.5 of it.
    constexpr int kWalk = 7;
    u32x4 left[4][kWalk];
    auto walk = [&](int c0) {
#pragma unroll
        for (int i = 0; i < kWalk; ++i) {
            if (c0 + 16 * i >= c_begin) break;   // uniform
            const int c = c0 + 16 * i + n;
#pragma unroll
            for (int r = 0; r < 4; ++r) left[r][i] = buffer_load4(bits, c < c_begin ? (uint32_t)((4 * r + g) * row_bytes + 16 * c) : kPastBuffer);
        }
    };
    walk(walk_begin);
    u32x4 quad_next = load_quad(c_begin + 4);

    // ---- X: the waves of a part move its chunks of a panel
    constexpr int kXRows = 4 * kGroups, kXPer = kPartPanel * 16 * MT / kXRows;   // rows at a time, 16-byte units of a thread
    const Buffer xbuf = make_buffer(x, (uint64_t)M * K * 2);
    const uint32_t lds0 = lds_address(lds), lut = lds0, xs0 = lds0 + 256;
    const int xv = tid & 15, xr = (tid & (16 * kXRows - 1)) >> 4;   // unit j of the thread is vector xv of row (xr + kXRows j) % (16 MT) of chunk (xr + kXRows j) / (16 MT)
    // Vector v of a row at place p(v) ^ (row % 16), p the order in which a unit's steps read them: the operand reads of a wave then
    // meet every bank equally.
    const uint32_t xplace = kPairs ? xv : ((xv & 6) << 1) | ((xv & 1) << 1) | (xv >> 3);
    u32x4 xring[kXPer];
    const uint32_t x_part = xs0 + (uint32_t)part * kPartPanel * kTileBytes;
    auto load_x = [&](int i) {   // the panel that starts i chunks on
#pragma unroll
        for (int j = 0; j < kXPer; ++j) {
            const int t = (xr + kXRows * j) / (16 * MT), r = (xr + kXRows * j) % (16 * MT), ct = c_begin + i + t, start = chunk_start(ct);
            bool in = r < M && ct < c_end;
            if (kRagged) in = in && 8 * xv >= ct * kChunkColumns - start;
            xring[j] = buffer_load4(xbuf, in ? ((uint32_t)r * (uint32_t)K + start + 8 * xv) * 2 : kPastBuffer);
        }
    };
    auto store_x = [&]() {
#pragma unroll
        for (int j = 0; j < kXPer; ++j) lds_write(x_part + (xr + kXRows * j) * 256 + 16 * (xplace ^ ((xr + kXRows * j) & 15)), xring[j]);
    };
    load_x(0);

    if (tid < 16) {
        uint32_t a, b;
        nibble_lut_entry(tid, a, b);
        lds_write(lut + 8 * tid, u32x2{a, b});
        if constexpr (kCodes) reinterpret_cast<float*>(lds + 128)[tid] = kNf4Levels[tid];
    }
    if (walk_begin < c_begin) {   // uniform
        uint32_t before[4] = {0, 0, 0, 0};   // of row 4 r + g
        for (int c0 = walk_begin; c0 < c_begin; c0 += 16 * kWalk) {
            if (c0 > walk_begin) walk(c0);
#pragma unroll
            for (int i = 0; i < kWalk; ++i) {
                if (c0 + 16 * i >= c_begin) break;   // uniform (short rows: counting what is not there was 0.5 us of a call)
#pragma unroll
                for (int r = 0; r < 4; ++r) before[r] = popc4(left[r][i], before[r]);
            }
        }
        // (in registers, by rotations of 16 lanes, and one exchange: as 20 exchanges through LDS they were slower on short rows)
        uint32_t held = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            before[r] += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)before[r], 0x128, 0xF, 0xF, false);   // row_ror:8, 4, 2, 1
            before[r] += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)before[r], 0x124, 0xF, 0xF, false);
            before[r] += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)before[r], 0x122, 0xF, 0xF, false);
            before[r] += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)before[r], 0x121, 0xF, 0xF, false);
            held = n >> 2 == r ? before[r] : held;
        }
        cur += __shfl(held, 16 * (n & 3) + (n & 12), 64);   // row n = 4 (n / 4) + n % 4
    }

    const uint64_t left_over = (uint64_t)total - first;   // values from the buffer's start on; whole vectors of them are readable
    const Buffer vals = kCodes ? make_buffer(static_cast<const uint8_t*>(values) + first / 2, (left_over + 31) / 32 * 16)
                               : make_buffer(static_cast<const uint16_t*>(values) + first, (left_over + 7) / 8 * 16);
    const Buffer scale_buffer = make_buffer(kCodes ? scales + first / 64 : scales, kCodes ? (left_over + 63) / 64 * 2 : 0);
    uint32_t at_next = cur - first;                // the row's next value
    // Lane (n, g) expands half g % 2 of a unit (one of a pair of chunks, or half of a chunk), the bytes g / 2, g / 2 + 2, .. of it: the
    // lanes that read LDS together are sixteen rows of either half, each with a bank of its own.
    const int h = g & 1, gh = g >> 1;
    const uint32_t slot = xs0 + kPanelBytes + wave * kSlotBytes + 64 * h + 4 * n;
    const uint32_t shift[2] = {8u * gh, 8u * gh + 16u}, below[2] = {(1u << shift[0]) - 1u, (1u << shift[1]) - 1u};

    f32x4 acc[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};

    // A lane asks for vectors gh, gh + 2, .. of its piece: always the first few, further ones where any lane of the wave needs them
    // (at 50 % nonzeros the second lot nearly always, at 30 % never).
    constexpr int kLoads = (kVectors + 1) / 2, kFirst = kCodes ? kLoads - 1 : kPairs ? 4 : 3, kSecond = kCodes || !kPairs ? kLoads : 6;
    constexpr uint32_t kPerVector = kCodes ? 32 : 8;
    struct Stage {
        u32x4 v[kLoads];
        uint32_t scale[kCodes ? kLoads : 1];
        uint32_t at;         // the piece's first value
        bool more, most;     // (wave-uniform)
    };
    auto request = [&](Stage& st, int i) {
        const uint32_t v = st.at / kPerVector + gh + 2 * i;
        st.v[i] = buffer_load4(vals, 16 * v);
        // a vector of 32 codes lies in one block of 64 values
        if constexpr (kCodes) st.scale[i] = __builtin_amdgcn_raw_buffer_load_b16(scale_buffer, (int)(v / 2 * 2), 0, 0);
    };
    // Request the pieces of a unit whose lengths are `len` values: those of half 0, then those of half 1.
    auto issue = [&](Stage& st, uint32_t len) {
        uint32_t l0 = len, l1 = len;
        swap_odd_even_groups(l0, l1);   // of half 0 and of half 1, to all lanes of the row
        st.at = at_next + (h ? l0 : 0u);
        at_next += l0 + l1;
        const uint32_t need = st.at % kPerVector + len;
        st.more = __builtin_amdgcn_ballot_w64(need > 2 * kPerVector * kFirst) != 0;
        st.most = kSecond < kLoads && __builtin_amdgcn_ballot_w64(need > 2 * kPerVector * kSecond) != 0;
#pragma unroll
        for (int i = 0; i < kFirst; ++i) request(st, i);
        if (st.more)
#pragma unroll
            for (int i = kFirst; i < kSecond; ++i) request(st, i);
        if (st.most)
#pragma unroll
            for (int i = kSecond; i < kLoads; ++i) request(st, i);
    };
    auto park = [&](const Stage& st) {
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            if (i == kFirst && !st.more) break;
            if (i == kSecond && !st.most) break;
            if constexpr (kCodes) {
                if (i == kLoads - 1 && gh != 0) break;   // an odd number of vectors: the last is the other lane's
                const float scale = __uint_as_float(st.scale[i] << 16);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint4 d = nf4_decode8(st.v[i][j], scale, reinterpret_cast<const float*>(lds + 128));
                    const uint32_t to = slot + 2048 * gh + 4096 * i + 512 * j;
                    lds_write(to, d.x);
                    lds_write(to + 128, d.y);
                    lds_write(to + 256, d.z);
                    lds_write(to + 384, d.w);
                }
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) lds_write(slot + 512 * gh + 1024 * i + 128 * j, st.v[i][j]);
            }
        }
    };
    // Expand the lane's words, whose values start at element `count` of the parked piece, and multiply.
    auto expand = [&](const auto& words, uint32_t count, uint32_t x_operand) {
        constexpr int kSteps = 2 * (int)(sizeof(words) / sizeof(words[0]));
        __builtin_amdgcn_wave_barrier();   // LDS executes a wave's accesses in order: the parked values land first
        ByteWindow w = read_byte_window(words[0], below[0], shift[0], count, slot, lut);
#pragma unroll
        for (int s = 0; s < kSteps; ++s) {
            u32x4 aq[MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) aq[mt] = lds_read<u32x4>((x_operand ^ ((kPairs ? 32 : 64) * s)) + 4096 * mt);
            ByteWindow next;
            if (s + 1 < kSteps) {
                if (s % 2 == 1) count = __popc(words[s / 2]) + count;
                next = read_byte_window(words[(s + 1) / 2], below[(s + 1) % 2], shift[(s + 1) % 2], count, slot, lut);
            }
            __builtin_amdgcn_sched_barrier(0);
            const bf16x8 b = expand_window(w);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
                acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b, __builtin_bit_cast(bf16x8, aq[mt]), acc[mt], 0, 0, 0);
            if (s + 1 < kSteps) w = next;
            __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_wave_barrier();   // reads above are issued before the slots are written again
    };

    // A unit is U words per lane, a round four chunks.
    constexpr int U = kPairs ? 4 : 2, kUnits = kPairs ? 2 : 4, kUnitChunks = 4 / kUnits;
    uint32_t words[kUnits][U], words_next[kUnits][U];
    auto spread = [&](u32x4 q, uint32_t (&w)[kUnits][U]) {   // to the lanes that expand them
        if constexpr (kPairs) {
#pragma unroll
            for (int i = 0; i < 4; ++i) spread_halves(q[i], w[0][i], w[1][i]);
        } else {
            uint32_t a0 = q[0], b0 = q[2], a1 = q[1], b1 = q[3];
            swap_odd_even_groups(a0, b0);
            swap_odd_even_groups(a1, b1);
            spread_halves(a0, w[0][0], w[2][0]);
            spread_halves(b0, w[1][0], w[3][0]);
            spread_halves(a1, w[0][1], w[2][1]);
            spread_halves(b1, w[1][1], w[3][1]);
        }
    };
    auto length = [&](const uint32_t (&w)[U]) -> uint32_t {
        uint32_t l = 0;
#pragma unroll
        for (int i = 0; i < U; ++i) l = __popc(w[i]) + l;
        return l;
    };
    // LDS place of the lane's X vector of step 0 in the unit's first tile (the other steps' differ in two or three bits)
    const uint32_t x_lane = x_part + n * 256 + (kPairs ? h * kTileBytes + 16 * (gh ^ n) : 16 * ((2 * gh + h) ^ n));
    Stage st;
    spread(quad, words);
    quad = quad_next;
    issue(st, length(words[0]));
    // Whether T is there and what of B_cat it meets: asked for before the last unit is multiplied.
    RowtileAdapters<MT> adapters(p, n0, M, N, b_cat, R, Rpad, lane);
    uint64_t* pair = p.words + (int64_t)tile * kGroups + wave % kGroups;
    uint64_t pair_word = 0;
    constexpr int kTurn = kPartPanel < 4 ? 4 : kPartPanel;
    for (int i0 = 0; i0 < total_chunks; i0 += kTurn) {
        if (i0 > 0) __syncthreads();   // the panel before has been read by all waves
        store_x();
        if (kPartPanel < 4 || i0 + kPartPanel < total_chunks) load_x(i0 + kPartPanel);   // (past the slice: zeros)
        __syncthreads();
#pragma unroll 1
        for (int i = i0; i < total_chunks && i < i0 + kTurn; i += 4) {
#pragma unroll
            for (int u = 0; u < kUnits; ++u) {
                if (u > 0 && i + u * kUnitChunks >= total_chunks) break;   // uniform
                if (kPartPanel < 4 && u > 0 && u * kUnitChunks % kPartPanel == 0) {   // (a round is more than one panel)
                    __syncthreads();
                    store_x();
                    load_x(i + u * kUnitChunks + kPartPanel);
                    __syncthreads();
                }
                const uint32_t start = st.at % kPerVector;
                park(st);
                if (u + 1 < kUnits) issue(st, length(words[u + 1]));
                else {
                    spread(quad, words_next);
                    quad = load_quad(c_begin + i + 8);
                    if (i + 4 < total_chunks) issue(st, length(words_next[0]));   // uniform
                }
                if (i + (u + 1) * kUnitChunks >= total_chunks && kOneLaunch && p.words != nullptr) {   // uniform
                    pair_word = look_at(pair);
                    adapters.load_b(0);
                }
                expand(words[u], start, x_lane + (i - i0 + u * kUnitChunks) % kPartPanel * kTileBytes);
            }
#pragma unroll
            for (int u = 0; u < kUnits; ++u)
#pragma unroll
                for (int j = 0; j < U; ++j) words[u][j] = words_next[u][j];
        }
    }
    if constexpr (Q > 1) {   // the parts' sums, in order
        __syncthreads();     // the X panel is retired
        const uint32_t place = xs0 + (uint32_t)(wave % kGroups) * MT * 1024 + 16 * lane;
        if (part > 0)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) lds_write(place + (part - 1) * kGroups * MT * 1024 + 1024 * mt, acc[mt]);
        __syncthreads();
        if (part > 0) return;
#pragma unroll
        for (int q = 0; q + 1 < Q; ++q)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[mt] += lds_read<f32x4>(place + q * kGroups * MT * 1024 + 1024 * mt);
    }

    // ---- adapters from an earlier launch's T (slice 0)
    if (!kOneLaunch && p.t_in != nullptr && z == 0) {
        __syncthreads();   // the X panel is retired
        uint16_t* t_lds = reinterpret_cast<uint16_t*>(lds + 256);   // [M][Rpad]
        const int groups = M * (Rpad >> 2);
        for (int i = tid; i < groups; i += kRtThreads) {
            float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
            const float4* q = reinterpret_cast<const float4*>(p.t_in) + i;
#pragma unroll
            for (int sl = 0; sl < kStreamTSlices; ++sl) {
                const float4 v = q[(int64_t)sl * groups];
                sum.x += v.x; sum.y += v.y; sum.z += v.z; sum.w += v.w;
            }
            uint2 o;
            o.x = (uint32_t)f32_to_bf16_rne(sum.x) | ((uint32_t)f32_to_bf16_rne(sum.y) << 16);
            o.y = (uint32_t)f32_to_bf16_rne(sum.z) | ((uint32_t)f32_to_bf16_rne(sum.w) << 16);
            *reinterpret_cast<uint2*>(&t_lds[4 * i]) = o;
        }
        __syncthreads();
        for (int rs = 0; rs < (Rpad >> 5); ++rs) {
            uint32_t e[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {   // (past R: dropped by ranks_below)
                const int k = rs * 32 + 8 * g + j;
                e[j] = (uint32_t)b_cat[(int64_t)(k < R ? k : R - 1) * N + (row < N ? row : N - 1)];
            }
            const uint4 bq = ranks_below(make_uint4(e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16)), rs * 32 + 8 * g, R);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const int m = 16 * mt + n;
                const uint4 aq = *reinterpret_cast<const uint4*>(&t_lds[(m < M ? m : M - 1) * Rpad + rs * 32 + 8 * g]);
                acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(bq), as_bf16x8(aq), acc[mt], 0, 0, 0);
            }
        }
    }

    // ---- store: lane holds row 16 mt + lane % 16 of Y, columns n0 + 4 g .. + 3
    const int64_t col = n0 + 4 * g;
    if (kOneLaunch && p.words != nullptr) {
        bool t_there = __builtin_amdgcn_ballot_w64(pair_word == p.tag) != 0;   // (the same in all lanes)
        if (t_there) {
            if (lane == 0) leave_clear(pair);
        } else {
            // T is formed within the first 6 to 12 us of the launch.  Where it is not there yet, it soon will be, and its last
            // workgroup would have all rows to finish: wait a little, but not without end.
            rowtile_sums<MT>(p, n0, M, lane, true, acc);
            stores_done();
            if (lane == 0) {
                for (int i = 0; i < p.polls && look_at(pair) != p.tag; ++i) __builtin_amdgcn_s_sleep(1);
                t_there = meet(pair, p.tag);
            }
            if (__builtin_amdgcn_ballot_w64(t_there) == 0) return;
        }
        adapters.load_t(0);
        adapters.add(acc);
        rowtile_store<MT>(y, n0, M, N, lane, acc);
        return;
    }
    if (p.partial == nullptr) {
        rowtile_store<MT>(y, n0, M, N, lane, acc);
        return;
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int m = 16 * mt + n;
        if (m < M && col < p.pitch) *reinterpret_cast<f32x4*>(p.partial + ((int64_t)z * M + m) * p.pitch + col) = acc[mt];
    }
}

// y = sum of the slices' partial outputs + T B_cat.  A few KB a workgroup, so it is as long as its round trips to memory: the requests
// for T, for the first kBatch slices and for B_cat all go out before any of them is used (one after the other, each waited for:
// 4.8 us behind two slices of 16 x 4096 x 14336, so 4.2; 5.3 and 4.1 behind those of 8 x 14336 x 4096).  kBatch: four slices or eight at a time, the fewer
// registers where they are enough, for the workgroups of many rows of X.
template <int kBatch>
__global__ __launch_bounds__(256, kBatch == 4 ? 8 : 4) void rowtile_finish_kernel(const float* __restrict__ partial, int ksplit, int M, int64_t N,
                                                             int64_t pitch, const float* __restrict__ t_partial, int t_slices,
                                                             const uint16_t* __restrict__ b_cat, int R, int Rpad,
                                                             uint16_t* __restrict__ y) {
    constexpr int kTPitch = kMaxRankPadded + 8;
    __shared__ __attribute__((aligned(16))) uint16_t t_lds[16 * kTPitch];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i16 = lane & 15, g = lane >> 4;
    const int64_t n0 = (int64_t)blockIdx.x * 64 + 16 * wave;
    const int m0 = 16 * (int)blockIdx.y, m = m0 + i16;
    const int64_t col = n0 + 4 * g;
    const bool live = m < M && col < pitch;

    // four elements of T: the four k-slices' partials, and their place
    const int rows = M - m0 < 16 ? M - m0 : 16, per_row = Rpad >> 2;
    const int64_t t_slice = (int64_t)M * per_row;
    f32x4 tv[kRowtileTSlices];
    auto load_t = [&](int i) {
        const int r = i / per_row, c = i - r * per_row;
        const f32x4* q = reinterpret_cast<const f32x4*>(t_partial) + (int64_t)(m0 + (r < rows ? r : rows - 1)) * per_row + c;
#pragma unroll
        for (int sl = 0; sl < kRowtileTSlices; ++sl) tv[sl] = q[(sl < t_slices ? sl : 0) * t_slice];
    };
    // nothing below may move up to the requests, where it would wait for them
    auto arrived = [](f32x4& x) __attribute__((always_inline)) { asm volatile("" : "+v"(x)); };
    auto sum_t = [&](int i) {
        const int r = i / per_row, c = i - r * per_row;
        f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int sl = 0; sl < kRowtileTSlices; ++sl) arrived(tv[sl]);
#pragma unroll
        for (int sl = 0; sl < kRowtileTSlices; ++sl)
            if (sl < t_slices) sum += tv[sl];
        uint2 o;
        o.x = (uint32_t)f32_to_bf16_rne(sum[0]) | ((uint32_t)f32_to_bf16_rne(sum[1]) << 16);
        o.y = (uint32_t)f32_to_bf16_rne(sum[2]) | ((uint32_t)f32_to_bf16_rne(sum[3]) << 16);
        *reinterpret_cast<uint2*>(&t_lds[r * kTPitch + 4 * c]) = o;
    };
    const bool has_t = R > 0 && tid < 16 * per_row;
    if (has_t) load_t(tid);

    // the slices' partial outputs
    const float* src = partial + (int64_t)(m < M ? m : M - 1) * pitch + (col < pitch ? col : 0);
    const int64_t slice = (int64_t)M * pitch;
    f32x4 v[kBatch];
    auto load_slices = [&](int z0) {
#pragma unroll
        for (int z = 0; z < kBatch; ++z)
            if (z0 + z < ksplit) v[z] = *reinterpret_cast<const f32x4*>(src + (z0 + z) * slice);
    };
    load_slices(0);

    const int64_t n_c = n0 + i16 < N ? n0 + i16 : N - 1;
    uint32_t e[8];
    auto load_b = [&](int rs) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int r = rs * 32 + 8 * g + j;
            e[j] = (uint32_t)b_cat[(int64_t)(r < R ? r : R - 1) * N + n_c];
        }
    };
#pragma unroll
    for (int j = 0; j < 8; ++j) e[j] = (uint32_t)lane;   // (no constant: the packing would move up, too)
    if (R > 0) load_b(0);

    if (has_t) sum_t(tid);
    for (int i = tid + 256; R > 0 && i < 16 * per_row; i += 256) {
        load_t(i);
        sum_t(i);
    }
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int z0 = 0; z0 < ksplit; z0 += kBatch) {
        if (z0 > 0) load_slices(z0);
#pragma unroll
        for (int z = 0; z < kBatch; ++z)
            if (z0 + z < ksplit) {
                arrived(v[z]);
                acc += v[z];
            }
    }
    if (R > 0) {
        __syncthreads();
        // (Dropping ranks past R in the last step only, behind the loop: with it in every step the requests of the next wait for it, 0.1 to 0.3 us of
        // a call; 64 x 5632 x 1024, R 128, a table: 18.35 us, 18.05 so, 100 x 4096 x 4096, R 256: 29.6 and 29.0.)
        const int last = (Rpad >> 5) - 1;
        auto packed = [&]() { return make_uint4(e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16)); };
        auto multiply = [&](int rs, const uint4& bq) {
            const uint4 tq = *reinterpret_cast<const uint4*>(&t_lds[i16 * kTPitch + rs * 32 + 8 * g]);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(bq), as_bf16x8(tq), acc, 0, 0, 0);
        };
        for (int rs = 0; rs < last; ++rs) {
            multiply(rs, packed());
            load_b(rs + 1);
        }
        multiply(last, ranks_below(packed(), last * 32 + 8 * g, R));
    }
    if (!live) return;
    store_four(y, M, N, m, col, acc);
}

template <int MT, int Q, bool kOne>
static void launch_rowtile_t(const LinearArgs& a, RowtileArgs p, hipStream_t stream, const TimingEvents& ev) {
    const dim3 grid((unsigned)(p.t_blocks + p.tiles * p.ksplit));
    const int R = (int)a.R, Rpad = (int)adapter_rank_padded(a.R);
    const bool ragged = a.K % kChunkColumns != 0;
    auto go = [&](auto kernel, const void* values) {
        SALR_LAUNCH(kernel, grid, dim3(kRtThreads), stream, ev, a.x, (int)a.M, a.K, a.N, a.bitmap, values, a.scales, a.row_offsets, a.slice_table,
                    a.a_cat, a.b_cat, R, Rpad, a.y, p);
    };
    if (a.codes != nullptr) ragged ? go(linear_rowtile_kernel<MT, true, true, Q, kOne>, a.codes) : go(linear_rowtile_kernel<MT, false, true, Q, kOne>, a.codes);
    else ragged ? go(linear_rowtile_kernel<MT, true, false, Q, kOne>, a.values) : go(linear_rowtile_kernel<MT, false, false, Q, kOne>, a.values);
}

// How often a kernel looks for T at the end before it leaves its sums to it (or, salr_shared_t.hpp, forms T itself), a quarter of a
// microsecond each.  For tests: this host thread's next calls, 0 to not wait at all.
constexpr int kHandoverPolls = 64;
static thread_local int g_handover_polls = kHandoverPolls;
int handover_polls() { return g_handover_polls; }
extern "C" void salr_set_handover_polls(int polls) { g_handover_polls = polls >= 0 && polls < kHandoverPolls ? polls : kHandoverPolls; }

hipError_t launch_linear_rowtile(const LinearArgs& a, hipStream_t stream, const TimingEvents& ev) {
    char* base = reinterpret_cast<char*>(a.t);
    const int Rpad = (int)adapter_rank_padded(a.R);
    const RowtilePlan plan = rowtile_plan_in(a.M, a.K, a.N, a.R, a.room);
    RowtileArgs p;
    p.pitch = rowtile_pitch(a.N);
    p.ksplit = plan.ksplit;
    p.t_slices = plan.t_slices;
    p.t_out = reinterpret_cast<float*>(base);
    p.partial = plan.partial ? reinterpret_cast<float*>(base + rowtile_t_out_bytes(a.M, a.R)) : nullptr;
    const bool t_first = a.R > 0 && !plan.partial;
    p.t_in = t_first ? p.t_out : nullptr;
    p.t_blocks = a.R > 0 && !t_first ? plan.t_slices * (Rpad / 16) * (int)((a.M + 15) / 16) : 0;
    if (t_first) launch_adapter_partial_to(a, p.t_out, stream);
    const int rows = 16 * kRtWaves / plan.parts;
    p.tiles = (int)((a.N + rows - 1) / rows);
    p.words = nullptr;
    p.t_sum = nullptr;
    p.polls = g_handover_polls;
    if (handover_aligned(base) && rowtile_hands_over(a.M, a.K, a.N, a.R, plan, a.room)) {
        char* t_sum = base + rowtile_plan_bytes(a.M, a.K, a.N, a.R, plan);
        p.t_sum = reinterpret_cast<uint16_t*>(t_sum);
        p.words = reinterpret_cast<uint64_t*>(t_sum + round_up_256((size_t)a.M * Rpad * sizeof(uint16_t)));
        p.tag = next_handover_tag();
    }
    auto go = [&](auto mt) {
        if (plan.parts == 2) launch_rowtile_t<mt, 2, true>(a, p, stream, ev);
        else if (p.words != nullptr && plan.parts == 1) launch_rowtile_t<mt, 1, true>(a, p, stream, ev);
        else if (plan.parts == 1) launch_rowtile_t<mt, 1, false>(a, p, stream, ev);
        else if constexpr (mt <= 2) launch_rowtile_t<mt, 4, true>(a, p, stream, ev);
    };
    if (a.M <= 16) go(std::integral_constant<int, 1>());
    else if (a.M <= 32) go(std::integral_constant<int, 2>());
    else if (a.M <= 64) go(std::integral_constant<int, 4>());
    else go(std::integral_constant<int, 8>());
    if (p.partial != nullptr && p.words == nullptr)
        hipLaunchKernelGGL(plan.ksplit <= 4 ? rowtile_finish_kernel<4> : rowtile_finish_kernel<8>, dim3((unsigned)((a.N + 63) / 64), (unsigned)((a.M + 15) / 16)), dim3(256), 0, stream, p.partial,
                           plan.ksplit, (int)a.M, a.N, p.pitch, p.t_out, plan.t_slices, a.b_cat, (int)a.R, Rpad, a.y);
    return hipGetLastError();
}

}  // namespace salr
