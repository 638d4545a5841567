// Small-batch (M <= 64) path of the SALR linear: one pass over the compressed weight, HBM-bound.
//
// A workgroup owns 16 consecutive rows of What (= 16 outputs n) for the whole contraction; its NW
// waves split K into contiguous slices and run independently of each other until the final reduction:
//
//   per wave, per chunk of 128 columns (4 bitmap words per row):
//     decode stage  lane (n = lane%16, g = lane/16) takes byte g of each word of row n.  The packed
//                   values of the chunk (one contiguous piece per row) are fetched with 16-byte loads
//                   two chunks ahead, parked in LDS, and expanded by the nibble rule of Sec. 3.3
//                   straight into the B operand of a 16x16x32 bf16 MFMA -- the 8 columns of one byte
//                   mask are exactly the 8 k-values one lane feeds to that instruction;
//     MFMA stage    X rows come from global memory (L2-resident, shared by all workgroups) as the A
//                   operand; fp32 accumulators [16 m x 16 n] per m-tile.
//   adapters       the rank dimension is appended as extra k-steps: A operand = T (summed from the
//                   split-K partials of the adapter pre-kernel), B operand = B_cat columns (Sec. 3.2).
//   epilogue       accumulators of the NW waves are summed through LDS, rounded to bf16, stored.
//
// The row cursor into `values` at the start of a wave's slice is the row offset plus the popcount of
// the row's earlier bitmap words; the waves exchange the counts of their slices for it, or a table holds it.
#include <hip/hip_ext.h>

#include "salr_device.hpp"
#include "salr_internal.hpp"
#include "salr_linear_common.hpp"
#include "salr_row_stream.hpp"
#include "salr_shared_t.hpp"

namespace salr {

constexpr int kStreamRows = 16;         // weight rows per workgroup
constexpr int kChunkWords = 4;          // bitmap words per row per chunk (128 columns)
constexpr int kSlotDwords = 68;         // LDS per row per chunk: 17 vectors of 16 B (128 values + misalignment)
constexpr int kMaxVecPerLane = 5;       // 17 vectors over the 4 lanes of a row

template <int MT, int NV>
struct StreamStage {
    uint4 bm;                           // the chunk's 4 bitmap words of this lane's row
    uint4 vq[NV];                       // this lane's share of the row's packed-value piece
    uint4 xq[kChunkWords * MT];         // X operands of the chunk's 4 k-steps
    uint32_t off;                       // element offset of the piece inside its first 16-byte vector
    uint32_t nv;                        // vectors in the piece
};

// ---- T = X A_cat in every workgroup, for layers whose A_cat is a few KB (see stream_owns_t): one launch instead of two, which is what
// such a call's time is.  The requests for X and A_cat go out with the first of the weight's, the product is formed while the
// packed values are on their way.
// The partials are those of adapter_partial_kernel, summed in the same order, so T has the same bits: the steps of 32 columns of
// a slice are sums of their own, added up in order, and the slices in order.  A wave takes two of the kStreamTSlices slices; its
// rows of A_cat lie side by side, so they come as whole vectors and are read back transposed from its staging slots.
constexpr int kOwnTK = 1024;                        // columns at most: four steps a wave
constexpr int kOwnTSteps = kOwnTK / 32 / 8;
constexpr int kOwnTRank = 32;
constexpr int kOwnTBytes = 4096;                    // of A_cat at most that a wave's steps read: four vectors a lane
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

struct OwnT {
    u32x4_t a[kOwnTBytes / 1024];
    uint4 x[kOwnTSteps];
    int u_begin, u_mid, u_end;   // steps of the wave's first slice and its second
};

__device__ __forceinline__ void own_t_request(OwnT& o, const uint16_t* __restrict__ x, int M, int64_t K,
                                              const uint16_t* __restrict__ a_cat, int R, int wave, int lane) {
    const int units = (int)(K >> 5), i16 = lane & 15, g = lane >> 4;
    static_assert(kStreamTSlices == 16 && kOwnTBytes <= kStreamRows * kSlotDwords * 4);
    o.u_begin = units * wave >> 3;
    o.u_mid = units * (2 * wave + 1) >> 4;
    o.u_end = units * (wave + 1) >> 3;
    const Buffer piece = make_buffer(a_cat + (int64_t)o.u_begin * 32 * R, (uint64_t)(o.u_end - o.u_begin) * 64 * R);
#pragma unroll
    for (int i = 0; i < (int)(sizeof(o.a) / 16); ++i) o.a[i] = buffer_load4(piece, 16u * lane + 1024u * i);
    const int m = i16 < M ? i16 : M - 1;
#pragma unroll
    for (int t = 0; t < kOwnTSteps; ++t) {
        const int u = o.u_begin + t < units ? o.u_begin + t : units - 1;   // steps past the slices are dropped
        o.x[t] = *reinterpret_cast<const uint4*>(x + (int64_t)m * K + 32 * u + 8 * g);
    }
}

// partials: [rank tile][slice][16 rows][16 columns]; slots: 4 KB of this wave's
__device__ __forceinline__ void own_t_partials(const OwnT& o, int R, int Rpad, uint32_t* slots, float* partials, int wave, int lane) {
    const int i16 = lane & 15, g = lane >> 4;
#pragma unroll
    for (int i = 0; i < (int)(sizeof(o.a) / 16); ++i) *reinterpret_cast<u32x4_t*>(slots + 4 * lane + 256 * i) = o.a[i];
    __builtin_amdgcn_wave_barrier();   // LDS executes a wave's accesses in order
    const uint16_t* rows = reinterpret_cast<const uint16_t*>(slots);
#pragma unroll
    for (int rt = 0; rt < kOwnTRank / 16; ++rt) {
        if (16 * rt >= Rpad) break;    // uniform
        const int r = 16 * rt + i16, r_c = r < R ? r : R - 1;   // padded columns read a valid one and become zeros below
        f32x4 product[kOwnTSteps];
#pragma unroll
        for (int t = 0; t < kOwnTSteps; ++t) {
            product[t] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (o.u_begin + t >= o.u_end) break;   // uniform
            uint32_t e[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) e[j] = rows[(32 * t + 8 * g + j) * R + r_c];
            const uint4 b = make_uint4(e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16));
            product[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(o.x[t]), as_bf16x8(b), product[t], 0, 0, 0);
        }
        f32x4 first = {0.f, 0.f, 0.f, 0.f}, second = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < kOwnTSteps; ++t) {
            if (o.u_begin + t < o.u_mid) first += product[t];
            else if (o.u_begin + t < o.u_end) second += product[t];
        }
        float* p = partials + (rt * kStreamTSlices + 2 * wave) * 256 + 64 * g + i16;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            p[16 * q] = r < R ? first[q] : 0.f;
            p[256 + 16 * q] = r < R ? second[q] : 0.f;
        }
    }
    __builtin_amdgcn_wave_barrier();   // the slots are free again
}

// MT m-tiles of 16 rows, NW waves per workgroup, S chunks in flight per wave.
// Where a slice's values start the waves find by exchanging the counts of their slices.  (Each reading the words left of its own again, with no
// barrier before the stream, keeps the address unit busier than the barrier costs.  us a call without adapters, read again / exchanged:
// 4096 x 4096 one token 9.4 / 9.1, 16 tokens 10.7 / 10.4, 32 tokens 14.9 / 14.4; 2048 x 4096 6.5 / 5.8 and 7.6 / 6.8, 2048 x 2048 32 tokens 9.3 / 8.5,
// 1024 x 4096 32 tokens 6.8 / 5.9, 2048 x 7168 16 tokens 13.8 / 12.0; level at 512 columns.)
// kTable: the cursors come ready-made from the layer's slice table (salr_build_slice_table: for every row and each of
// the 8 wave slices the index of the slice's first value and the most nonzeros any chunk of it holds): one 8-byte
// request in place of the row offset, the rest of the slice's bitmap and the words left of it, and no barrier.
// kQuads: the bitmap of four chunks in one request.
// kOwnT: every workgroup computes T itself instead of reading the pre-kernel's partials (see stream_owns_t).  Its rows are a chunk a wave: there
// the waves count what is left of their slices.
// kShareT: the first workgroups form T's partials for all (salr_shared_t.hpp).
template <int MT, int NW, int S, bool kVecBitmap, bool kTable = false, bool kOwnT = false, bool kQuads = false, bool kShareT = false>
__global__ __launch_bounds__(NW * 64, (S == 2 && MT == 1) ? 4 : 1) void linear_stream_kernel(
    const uint16_t* __restrict__ x, int M, int64_t K, int64_t N, const uint32_t* __restrict__ bitmap,
    const uint16_t* __restrict__ values, const uint32_t* __restrict__ row_offsets,
    float* t_partial, const uint16_t* __restrict__ b_cat, int R, int Rpad,
    uint16_t* __restrict__ y, const uint32_t* __restrict__ slice_table, const uint16_t* __restrict__ a_cat, SharedT shared) {
    static_assert(!kShareT || (MT == 1 && NW == kShareWaves && !kOwnT && kShareTileBytes <= kStreamRows * kSlotDwords * 4));
    static_assert(!kTable || NW == kSliceTableSlices, "the table holds one entry per wave slice");
    constexpr int kThreads = NW * 64;
    constexpr int kStageDwords = NW * kStreamRows * kSlotDwords + 8;
    constexpr int kRedFloats = NW * MT * 256;
    constexpr int kSmemDwords = kStageDwords > kRedFloats ? kStageDwords : kRedFloats;
    constexpr int kTRows = 16 * MT;
    __shared__ __attribute__((aligned(16))) uint32_t smem[kSmemDwords];
    __shared__ __attribute__((aligned(16))) uint16_t t_lds[kTRows * kMaxRankPadded];  // T = X * A_cat, bf16
    __shared__ uint32_t lut_all[NW][kNibbleLutWords];  // one copy per wave: filled and used wave-synchronously
    __shared__ uint32_t slice_count[NW][kStreamRows];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // scalar: conditions on it branch uniformly
    const int n = lane & 15;
    const int g = lane >> 4;
    const int group = (int)blockIdx.x - (kShareT ? shared.extra : 0);   // of 16 rows
    if constexpr (kShareT) {
        static_assert(sizeof(t_lds) >= kShareRedBytes);
        if (group < 0) {   // the same for the whole workgroup
            shared_t_workgroup(shared, x, M, K, a_cat, R, Rpad, t_partial, reinterpret_cast<uint16_t*>(smem + wave * kStreamRows * kSlotDwords),
                               reinterpret_cast<float*>(t_lds), wave, lane);
            return;
        }
    }
    const int64_t n0 = (int64_t)group * kStreamRows;
    const int64_t row = n0 + n;
    const bool row_ok = row < N;
    const int64_t wpr = K >> 5;
    const int64_t chunks_total = (wpr + kChunkWords - 1) / kChunkWords;
    const int64_t c_begin = chunks_total * wave / NW;
    const int64_t c_end = chunks_total * (wave + 1) / NW;
    uint32_t* lut = lut_all[wave];
    // Rows past N (last workgroup only) are computed as copies of row N-1 and dropped at the store,
    // so no load below needs a per-lane predicate: every address is clamped into range instead.
    const int64_t row_c = row_ok ? row : N - 1;
    const uint32_t* brow = bitmap + row_c * wpr;

    // first requests of the kernel: row offset, bitmap of the first S chunks, adapter operands
    uint32_t cur;           // element index in `values` of the row's next value
    uint32_t longest = 0;   // most nonzeros any 128-column chunk of the slice holds (per lane)
    if constexpr (kTable) {
        const uint2 e = *reinterpret_cast<const uint2*>(slice_table + ((int64_t)row_c * kSliceTableSlices + wave) * 2);
        cur = e.x;
        longest = e.y;
    } else {
        cur = row_offsets[row_c];
    }

    auto load_bitmap_chunk = [&](int64_t c) -> uint4 {
        uint4 q = make_uint4(0, 0, 0, 0);
        if (c < c_end) {  // wave-uniform when c is
            if constexpr (kVecBitmap) {
                q = *reinterpret_cast<const uint4*>(brow + c * kChunkWords);
            } else {
                const int64_t w0 = c * kChunkWords;
                q.x = brow[w0];
                if (w0 + 1 < wpr) q.y = brow[w0 + 1];
                if (w0 + 2 < wpr) q.z = brow[w0 + 2];
                if (w0 + 3 < wpr) q.w = brow[w0 + 3];
            }
        }
        return q;
    };

    // kQuads: the bitmap of the four chunks in flight comes as one request of 64 bytes a row, chunk c + g to lane (n, g), and goes to the
    // other lanes in registers.  (A request a chunk, the same 16 bytes a row to four lanes, keeps the address unit busy for 31 ns
    // each, this one for 20: 4096 x 4096, one token, 13.7 -> 13.2 us with its pre-kernel, 3000 x 5248 16.4 -> 15.4.)
    static_assert(!kQuads || (S == 4 && kVecBitmap));
    auto load_quad = [&](int64_t c) -> u32x4 {
        u32x4 q = {0, 0, 0, 0};
        if (c + g < c_end) q = *reinterpret_cast<const u32x4*>(brow + (c + g) * kChunkWords);
        return q;
    };
    uint4 bmq[S];  // bitmap ring: chunks [c, c + S) ahead of the stages
    auto spread_quad = [&](u32x4 q) {
        u32x4 w[4];
        spread_chunks(q, w);
#pragma unroll
        for (int i = 0; i < S && i < 4; ++i) bmq[i] = make_uint4(w[i].x, w[i].y, w[i].z, w[i].w);
    };
    u32x4 quad = {0, 0, 0, 0};
    if constexpr (kQuads) quad = load_quad(c_begin);
    else
#pragma unroll
        for (int i = 0; i < S; ++i) bmq[i] = load_bitmap_chunk(c_begin + i);

    // B operand of this wave's rank step (Sec. 3.2): lane (n, g) holds B_cat[32*wave + 8g + j][row], j = 0..7
    const bool has_rank_step = R > 0 && wave * 32 < Rpad;
    uint4 bq = make_uint4(0, 0, 0, 0);
    uint32_t late[8];   // kOwnT: packed where they are used (no constants here: the packing would move up to the loads and wait)
    if constexpr (kOwnT) {
#pragma unroll
        for (int j = 0; j < 8; ++j) late[j] = (uint32_t)lane;
        if (has_rank_step) {
#pragma unroll
            for (int j = 0; j < 8; ++j) late[j] = (uint32_t)b_cat[(int64_t)(8 * g + j < R ? 8 * g + j : R - 1) * N + row_c];
        }
    } else if (has_rank_step) {
        const int r0 = wave * 32 + 8 * g;
        uint32_t e[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {  // clamp instead of predicating; ranks_below drops those past R
            const int r = r0 + j < R ? r0 + j : R - 1;
            e[j] = (uint32_t)b_cat[(int64_t)r * N + row_c];
        }
        bq = make_uint4(e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16));
    }

    __shared__ float own_t[kOwnT ? kOwnTRank / 16 * kStreamTSlices * 256 : 1];
    OwnT own;
    if constexpr (kOwnT) own_t_request(own, x, M, K, a_cat, R, wave, lane);
    // T = sum of the pre-kernel's split-K partials, rounded once to bf16, kept in LDS
    if (R > 0 && !kOwnT && !kShareT) {
        const int groups = M * (Rpad >> 2);  // float4 groups of T
        for (int i = tid; i < groups; i += kThreads) {
            float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
            const float4* p = reinterpret_cast<const float4*>(t_partial) + i;
#pragma unroll
            for (int sl = 0; sl < kStreamTSlices; ++sl) {
                const float4 v = p[(int64_t)sl * groups];
                sum.x += v.x; sum.y += v.y; sum.z += v.z; sum.w += v.w;
            }
            const int m = i / (Rpad >> 2), r4 = i % (Rpad >> 2);
            uint2 o;
            o.x = (uint32_t)f32_to_bf16_rne(sum.x) | ((uint32_t)f32_to_bf16_rne(sum.y) << 16);
            o.y = (uint32_t)f32_to_bf16_rne(sum.z) | ((uint32_t)f32_to_bf16_rne(sum.w) << 16);
            *reinterpret_cast<uint2*>(&t_lds[m * kMaxRankPadded + 4 * r4]) = o;
        }
    }

    const bool forms_t = kShareT && shared.extra == 0 && group < kStreamTSlices * (Rpad >> 5);   // the same for the whole workgroup
    SharedTProducts t_products;
    if constexpr (kShareT)
        if (forms_t) t_products.request(x, M, K, a_cat, R, group, wave, lane);
    // behind the first requests of the stream, whose way is as long as that of the sums
    auto start_hand_out = [&](SharedTHandOut& t_out) {
        if constexpr (kShareT)
            if (forms_t && wave == 0) t_out.start(shared, t_partial, M, R, Rpad, group, (int)gridDim.x, reinterpret_cast<const float*>(t_lds), lane);
    };
    auto finish_hand_out = [&](SharedTHandOut& t_out) {
        if (kShareT && forms_t && wave == 0) t_out.finish(shared);
    };
    auto hand_out = [&]() {
        SharedTHandOut t_out;
        start_hand_out(t_out);
        finish_hand_out(t_out);
    };

    if (lane < 16) {
        uint32_t a, b;
        nibble_lut_entry(lane, a, b);
        lut[2 * lane] = a;
        lut[2 * lane + 1] = b;
    }
    __builtin_amdgcn_wave_barrier();

    if constexpr (kQuads) {
        spread_quad(quad);
        if (!kOwnT && c_begin + S < c_end) quad = load_quad(c_begin + S);   // (uniform, as below)
    }

    // ---- pre-pass: nonzeros of this wave's slice per row.  The first S chunks are already in
    // registers (all 4 lanes of a row hold them); the 4 lanes split the rest.
    if constexpr (!kTable) {
        uint32_t head = 0, tail = 0;
#pragma unroll
        for (int i = 0; i < S; ++i) {
            const uint32_t len = __popc(bmq[i].x) + __popc(bmq[i].y) + __popc(bmq[i].z) + __popc(bmq[i].w);
            head += len;
            longest = len > longest ? len : longest;
        }
        for (int64_t c = c_begin + S + g; c < c_end; c += 4) {
            const uint4 q = load_bitmap_chunk(c);
            const uint32_t len = __popc(q.x) + __popc(q.y) + __popc(q.z) + __popc(q.w);
            tail += len;
            longest = len > longest ? len : longest;
        }
        if constexpr (kOwnT) {
            // nonzeros left of the slice: at most two chunks per lane, in flight at once
            uint32_t before = 0;
            constexpr int kLeft = kOwnTK / 512;
            uint4 left[kLeft];  // no branches: chunks past the slice start re-read chunk 0 and are dropped
#pragma unroll
            for (int i = 0; i < kLeft; ++i) {
                const int64_t c = g + 4 * i;
                left[i] = *reinterpret_cast<const uint4*>(brow + (c < c_begin ? c : 0) * kChunkWords);
            }
#pragma unroll
            for (int i = 0; i < kLeft; ++i) {
                const uint32_t cnt = __popc(left[i].x) + __popc(left[i].y) + __popc(left[i].z) + __popc(left[i].w);
                before += (g + 4 * i < c_begin) ? cnt : 0u;
            }
            before += __shfl_xor(before, 16, 64);
            before += __shfl_xor(before, 32, 64);
            cur += before;
        } else {
            tail += __shfl_xor(tail, 16, 64);
            tail += __shfl_xor(tail, 32, 64);
            if (g == 0) slice_count[wave][n] = head + tail;
        }
    }
    if constexpr (kShareT) {
        if (forms_t) {
            t_products.multiply(reinterpret_cast<uint16_t*>(smem + wave * kStreamRows * kSlotDwords), reinterpret_cast<float*>(t_lds), wave, lane);
            if (kTable) __syncthreads();
        }
    }
    if constexpr (!kOwnT && !kTable) {
        __syncthreads();
        for (int w = 0; w < wave; ++w) cur += slice_count[w][n];
    }

    const uint4* values128 = reinterpret_cast<const uint4*>(values);
    uint32_t* slot = smem + (wave * kStreamRows + n) * kSlotDwords;

    f32x4 acc[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};

    // A piece of up to 89 values spans at most 12 vectors (3 per lane); denser chunks need 5 per lane.
    const bool dense_slice = __builtin_amdgcn_ballot_w64(longest > 89u) != 0;  // wave-uniform

    // X rows of this lane: row 16 mt + n, its 8 k of a k-step at + 8 g (rows past M are computed on row M-1's data
    // and never stored)
    const uint16_t* xrow[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int m = 16 * mt + n;
        xrow[mt] = x + (int64_t)(m < M ? m : M - 1) * K + 8 * g;
    }

    // Fetch everything chunk c needs: NV value vectors per lane and the X operands of its 4 k-steps.
    // Lanes whose vector lies past the piece re-read its last vector (never used); an empty piece reads
    // the start of X instead (always mapped).  No per-lane branches: all requests go out back to back.
    auto issue = [&](auto& st, const uint4 bm, int64_t c) {
        constexpr int NV = sizeof(st.vq) / sizeof(uint4);
        st.bm = bm;
        const uint32_t len = __popc(bm.x) + __popc(bm.y) + __popc(bm.z) + __popc(bm.w);
        st.off = cur & 7u;
        st.nv = len ? (st.off + len + 7u) >> 3 : 0u;
        const uint32_t last = st.nv ? st.nv - 1u : 0u;
        const uint4* vb = st.nv ? values128 + (cur >> 3) : reinterpret_cast<const uint4*>(x);
        cur += len;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const uint32_t v = g + 4 * i;
            st.vq[i] = vb[v < last ? v : last];
        }
        if constexpr (kVecBitmap && MT >= 2) {
            // whole chunks only (K % 128 == 0): one address per row tile, the 4 k-steps at constant offsets (with one
            // row tile the two registers of the hoisted pointer cost more than the address arithmetic they save)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                if (16 * mt + n < M) {   // lanes of rows past M request nothing: their accumulator rows are never stored
                    const uint16_t* xc = xrow[mt] + c * (kChunkWords * 32);
#pragma unroll
                    for (int s = 0; s < kChunkWords; ++s) st.xq[s * MT + mt] = *reinterpret_cast<const uint4*>(xc + 32 * s);
                }
            }
        } else {
#pragma unroll
            for (int s = 0; s < kChunkWords; ++s) {
                int64_t k = (c * kChunkWords + s) * 32 + 8 * g;
                if constexpr (!kVecBitmap) k = k < K ? k : K - 8;  // ragged last chunk: the weight operand is zero there
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    const int m = 16 * mt + n;
                    if (m < M) st.xq[s * MT + mt] = *reinterpret_cast<const uint4*>(x + (int64_t)m * K + k);
                }
            }
        }
    };

    // Park the piece in LDS, expand the 4 byte masks of this lane, run the MFMAs.
    auto consume = [&](const auto& st) {
        constexpr int NV = sizeof(st.vq) / sizeof(uint4);
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const uint32_t v = g + 4 * i;
            if (NV <= 4 || v < 17u) *reinterpret_cast<uint4*>(slot + 4 * v) = st.vq[i];
        }
        __builtin_amdgcn_wave_barrier();  // LDS executes a wave's accesses in order: writes above land first
        const uint32_t words[kChunkWords] = {st.bm.x, st.bm.y, st.bm.z, st.bm.w};
        uint32_t c_local = st.off;
#pragma unroll
        for (int s = 0; s < kChunkWords; ++s) {
            const uint32_t word = words[s];
            const uint32_t m8 = (word >> (8 * g)) & 0xFFu;
            const uint32_t cb = c_local + __popc(word & ((1u << (8 * g)) - 1u));
            const uint4 wq = expand_byte(slot, lut, cb, m8);
            c_local += __popc(word);
            const bf16x8 b = as_bf16x8(wq);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
                acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(st.xq[s * MT + mt]), b, acc[mt], 0, 0, 0);
        }
        __builtin_amdgcn_wave_barrier();  // reads above are issued before the next chunk overwrites the slot
    };

    const int64_t n_chunks = c_end - c_begin;
    SharedTReader t_reader(shared, t_partial, M, Rpad, (int)gridDim.x - shared.extra, group, wave, lane);
    if (n_chunks == 0) hand_out();
    if constexpr (kOwnT) {
        // one chunk at most: its requests, T behind them, and one wait
        static_assert(kOwnTK <= 128 * NW && MT == 1);
        StreamStage<MT, kMaxVecPerLane> st;
        if (n_chunks > 0) issue(st, bmq[0], c_begin);   // wave-uniform
        own_t_partials(own, R, Rpad, smem + wave * kStreamRows * kSlotDwords, own_t, wave, lane);
        __syncthreads();
        {
            const int i = tid & 255, rt = tid >> 8;
            if (16 * rt < Rpad) {
                float sum = 0.f;
#pragma unroll
                for (int b = 0; b < kStreamTSlices; ++b) sum += own_t[(rt * kStreamTSlices + b) * 256 + i];
                t_lds[(i >> 4) * kMaxRankPadded + 16 * rt + (i & 15)] = f32_to_bf16_rne(sum);
            }
        }
        if (has_rank_step) {   // while the values, requested after these, are still on their way
#pragma unroll
            for (int j = 0; j < 8; ++j) asm volatile("" : "+v"(late[j]));
            bq = make_uint4(late[0] | (late[1] << 16), late[2] | (late[3] << 16), late[4] | (late[5] << 16), late[6] | (late[7] << 16));
            bq = ranks_below(bq, 8 * g, R);
        }
        if (n_chunks > 0) consume(st);
    } else if (n_chunks == S && !dense_slice) {
        // the whole slice is in flight at once: straight-line code, each chunk waits for its own data only
        StreamStage<MT, 3> st[S];
#pragma unroll
        for (int i = 0; i < S; ++i) issue(st[i], bmq[i], c_begin + i);
        SharedTHandOut t_out;
        start_hand_out(t_out);
#pragma unroll
        for (int i = 0; i < S; ++i) {
            if (kShareT && i == S - 2) t_reader.look();
            if (kShareT && i == S - 1 && t_reader.check()) t_reader.request();   // (uniform)
            consume(st[i]);
        }
        finish_hand_out(t_out);
    } else if (n_chunks > 0 && !dense_slice) {
        StreamStage<MT, 3> st[S];
#pragma unroll
        for (int i = 0; i < S; ++i) {
            if (c_begin + i < c_end) {
                issue(st[i], bmq[i], c_begin + i);
                if constexpr (!kQuads) bmq[i] = load_bitmap_chunk(c_begin + i + S);
            }
        }
        if (kQuads && c_begin + S < c_end) {
            spread_quad(quad);
            quad = load_quad(c_begin + 2 * S);
        }
        hand_out();
        for (int64_t c = c_begin; c < c_end; c += S) {
#pragma unroll
            for (int i = 0; i < S; ++i) {
                if (c + i < c_end) consume(st[i]);  // wave-uniform conditions
                if (c + i + S < c_end) {
                    issue(st[i], bmq[i], c + i + S);
                    if constexpr (!kQuads) bmq[i] = load_bitmap_chunk(c + i + 2 * S);
                }
            }
            if (kQuads && c + 2 * S < c_end) {
                spread_quad(quad);
                quad = load_quad(c + 3 * S);
            }
        }
    } else if (n_chunks > 0) {
        // dense pieces (more than ~70 % nonzeros in some chunk): 5 vectors per lane, two chunks in flight
        StreamStage<MT, kMaxVecPerLane> da, db;
        uint4 bm_next = bmq[0];
        auto step = [&](auto& st, int64_t c) {
            issue(st, bm_next, c);
            bm_next = (c + 1 - c_begin < S) ? bmq[(c + 1 - c_begin) % S] : load_bitmap_chunk(c + 1);
        };
        step(da, c_begin);
        hand_out();
        for (int64_t c = c_begin; c < c_end; c += 2) {
            if (c + 1 < c_end) step(db, c + 1);
            consume(da);
            if (c + 2 < c_end) step(da, c + 2);
            if (c + 1 < c_end) consume(db);
        }
    }

    __shared__ uint32_t t_missing[kShareT ? NW : 1];
    if constexpr (kShareT) {
        const bool fetched = t_reader.finish(shared, t_lds, Rpad);
        if (lane == 0) t_missing[wave] = fetched ? 0u : 1u;
    }

    __syncthreads();  // every wave is done with its staging slots; T in LDS is complete

    if constexpr (kShareT) {
        uint32_t missing = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) missing |= t_missing[w];
        missing = __builtin_amdgcn_readfirstlane(missing);   // (the same in all lanes)
        if (wave == 0) t_reader.leave(missing == 0);
        if (missing != 0)
            shared_t_alone(x, M, K, a_cat, R, Rpad, reinterpret_cast<uint16_t*>(smem + wave * kStreamRows * kSlotDwords), t_lds, tid, wave, lane);
    }

    // ---- adapter k-step of this wave (Sec. 3.2): A operand = T rows from LDS, B operand = bq
    if (has_rank_step) {
        if constexpr (!kOwnT) {
            int late_tid = tid;   // (rank wave * 32 + 8 g from a register that is there anyway: kept through the stream it spilled six others)
            asm volatile("" : "+v"(late_tid));
            bq = ranks_below(bq, 8 * (late_tid >> 4), R);
        }
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const int m = 16 * mt + n;
            const uint4 aq = *reinterpret_cast<const uint4*>(&t_lds[(m < M ? m : M - 1) * kMaxRankPadded + wave * 32 + 8 * g]);
            acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(aq), as_bf16x8(bq), acc[mt], 0, 0, 0);
        }
    }

    // ---- reduce the waves' accumulators and store
    float* red = reinterpret_cast<float*>(smem);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int e = 0; e < 4; ++e) red[((wave * MT + mt) * 4 + e) * 64 + lane] = acc[mt][e];
    __syncthreads();
    for (int idx = tid; idx < MT * 256; idx += kThreads) {
        const int l = idx & 63;
        const int e = (idx >> 6) & 3;
        const int mt = idx >> 8;
        float s = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) s += red[((w * MT + mt) * 4 + e) * 64 + l];
        const int m = 16 * mt + 4 * (l >> 4) + e;
        const int64_t nn = n0 + (l & 15);
        if (m < M && nn < N) y[(int64_t)m * N + nn] = f32_to_bf16_rne(s);
    }
}

// ---------------------------------------------------------------------------------------------------
// Split-K partials of T = X * A_cat for the small-batch path (Sec. 3.2, first concatenated GEMM).
// Workgroup (slice b, rank tile rt, row block) sums k over its slice for 16 columns of T and 64 rows of X
// with 16x16x32 bf16 MFMAs and writes t_partial[b][m][16 rt + r] (fp32; columns >= R as zeros).
// The main kernel adds the slices up, so no atomics and no zeroed workspace are needed.
//   A operand: lane (m, g) = X[m][k0 + 8g .. +8)            (one 16-byte load)
//   B operand: lane (r, g) = A_cat[k0 + 8g + j][16 rt + r]   (8 two-byte loads, j = 0..7)
// ---------------------------------------------------------------------------------------------------
constexpr int kTpWaves = 4;
constexpr int kTpThreads = kTpWaves * 64;
constexpr int kTpBatch = 4;   // k-steps a wave has in flight

// Blocks past the product's (a one-dimensional grid: product blocks first) build the layer's slice table for this call when
// the caller brought none: the bitmap is read once here, in the shadow of the product's round trips, and the main kernel
// starts from ready cursors (see kTable).
__global__ __launch_bounds__(kTpThreads) void adapter_partial_kernel(const uint16_t* __restrict__ x, int M, int64_t K,
                                                                     const uint16_t* __restrict__ a_cat, int R, int Rpad,
                                                                     int slices, float* __restrict__ t_partial,
                                                                     int product_blocks, const uint32_t* __restrict__ bitmap,
                                                                     const uint32_t* __restrict__ row_offsets, int64_t N,
                                                                     uint32_t* __restrict__ table_out) {
    __shared__ float red[kTpWaves][4][4][64];
    static_assert(kTpThreads == 256, "slice_table_block is written for 256 threads");
    if ((int)blockIdx.x >= product_blocks) {   // the same for the whole workgroup
        slice_table_block(bitmap, row_offsets, N, K, table_out, (int64_t)blockIdx.x - product_blocks, (int)threadIdx.x);
        return;
    }
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i16 = lane & 15, g = lane >> 4;
    const int rank_tiles = Rpad >> 4;
    const int b = (int)blockIdx.x % slices, rt = ((int)blockIdx.x / slices) % rank_tiles;
    const int row_block = (int)blockIdx.x / (slices * rank_tiles);
    const int64_t units = K >> 5;  // k-steps of 32 columns
    const int64_t u_begin = units * b / slices, u_end = units * (b + 1) / slices;
    const int r = 16 * rt + i16;
    const int r_c = r < R ? r : R - 1;  // padded columns read a valid column and are zeroed at the store
    const int m_base = 64 * row_block;  // 64 rows of X per workgroup
    const int mtiles = ((M - m_base < 64 ? M - m_base : 64) + 15) >> 4;
    f32x4 acc[4];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) acc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
    // kTpBatch k-steps per trip with all their loads issued before the first MFMA: the kernel is a handful of dependent
    // round trips long, so they are taken side by side (steps past the slice reload its last step and are skipped)
    for (int64_t u0 = u_begin + wave; u0 < u_end; u0 += kTpWaves * kTpBatch) {
        uint4 bq[kTpBatch], aq[kTpBatch][4];
#pragma unroll
        for (int t = 0; t < kTpBatch; ++t) {
            const int64_t u = u0 + kTpWaves * t < u_end ? u0 + kTpWaves * t : u_end - 1;
            const int64_t k0 = (u << 5) + 8 * g;
            uint32_t e[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) e[j] = a_cat[(k0 + j) * R + r_c];
            bq[t] = make_uint4(e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16));
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
                if (mt < mtiles) {  // uniform
                    const int m = m_base + 16 * mt + i16;
                    aq[t][mt] = *reinterpret_cast<const uint4*>(x + (int64_t)(m < M ? m : M - 1) * K + k0);
                }
            }
        }
#pragma unroll
        for (int t = 0; t < kTpBatch; ++t) {
            if (u0 + kTpWaves * t < u_end) {  // uniform
#pragma unroll
                for (int mt = 0; mt < 4; ++mt)
                    if (mt < mtiles)
                        acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(aq[t][mt]), as_bf16x8(bq[t]), acc[mt], 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int e = 0; e < 4; ++e) red[wave][mt][e][lane] = acc[mt][e];
    __syncthreads();
    // accumulator layout: lane holds T[16 mt + 4 (lane / 16) + e][16 rt + lane % 16]
    for (int idx = threadIdx.x; idx < mtiles * 256; idx += kTpThreads) {
        const int l = idx & 63, e = (idx >> 6) & 3, mt = idx >> 8;
        float s = 0.f;
#pragma unroll
        for (int w = 0; w < kTpWaves; ++w) s += red[w][mt][e][l];
        const int m = m_base + 16 * mt + 4 * (l >> 4) + e;
        const int rr = 16 * rt + (l & 15);
        if (m < M) t_partial[((int64_t)b * M + m) * Rpad + rr] = rr < R ? s : 0.f;
    }
}

static void launch_adapter_partial_impl(const LinearArgs& a, float* partial, bool build_table, hipStream_t stream) {
    const int R = (int)a.R, Rpad = (int)adapter_rank_padded(a.R);
    const int product_blocks = kStreamTSlices * (Rpad / 16) * (int)((a.M + 63) / 64);
    const int table_blocks = build_table ? (int)((a.N + kSliceTableRowsPerBlock - 1) / kSliceTableRowsPerBlock) : 0;
    hipLaunchKernelGGL(adapter_partial_kernel, dim3((unsigned)(product_blocks + table_blocks)), dim3(kTpThreads), 0, stream, a.x,
                       (int)a.M, a.K, a.a_cat, R, Rpad, kStreamTSlices, partial, product_blocks, a.bitmap, a.row_offsets, a.N,
                       const_cast<uint32_t*>(build_table ? a.slice_table : nullptr));
}

void launch_adapter_partial(const LinearArgs& a, hipStream_t stream) {
    launch_adapter_partial_impl(a, reinterpret_cast<float*>(a.t), a.build_table, stream);
}

void launch_adapter_partial_to(const LinearArgs& a, float* partial, hipStream_t stream) {
    launch_adapter_partial_impl(a, partial, false, stream);
}

// Whether the small-batch kernel computes T itself: up to 16 tokens, A_cat of up to 32 KB on rows that are one chunk per wave at most,
// and fewer row groups than two per CU (the other variant has no registers for it).  Both ways, us a call (pre-kernel / here):
// 16 x 512 x 512 rank 16 7.7 / 5.8, 1 x 512 x 1000 7.7 / 5.6, 16 x 1024 x 4096 rank 16 8.7 / 7.3, 16 x 512 x 8000 rank 32 11.0 / 9.1.
// Reading A_cat costs a workgroup 0.3 us per 32 KB; twice that, in columns or rank, takes more of the staging slots than a wave has.
static bool stream_owns_t(int64_t M, int64_t K, int64_t R) {
    return R > 0 && R <= kOwnTRank && M <= 16 && K % 128 == 0 && K <= kOwnTK && (K / 32 + 7) / 8 * 64 * R <= kOwnTBytes;
}

template <int MT, int NW, int S, bool kQ = false>
static void launch_stream_t(const LinearArgs& a, hipStream_t stream, const TimingEvents& ev) {
    const int R = (int)a.R, Rpad = (int)adapter_rank_padded(a.R);
    float* t_partial = reinterpret_cast<float*>(a.t);
    const unsigned grid = (unsigned)((a.N + kStreamRows - 1) / kStreamRows);
    if constexpr (MT == 1 && S > 2 && !kQ) {
        if (stream_owns_t(a.M, a.K, R)) {
            if (a.slice_table != nullptr && !a.build_table)
                SALR_LAUNCH((linear_stream_kernel<MT, NW, S, true, true, true>), dim3(grid), dim3(NW * 64), stream, ev, a.x, (int)a.M,
                            a.K, a.N, a.bitmap, a.values, a.row_offsets, nullptr, a.b_cat, R, Rpad, a.y, a.slice_table, a.a_cat, SharedT());
            else
                SALR_LAUNCH((linear_stream_kernel<MT, NW, S, true, false, true>), dim3(grid), dim3(NW * 64), stream, ev, a.x, (int)a.M,
                            a.K, a.N, a.bitmap, a.values, a.row_offsets, nullptr, a.b_cat, R, Rpad, a.y, nullptr, a.a_cat, SharedT());
            return;
        }
    }
    if constexpr (MT == 1 && S > 2) {
        const SharedT shared = shared_t_of(a, a.room);
        if (shared.words != nullptr) {
            auto go = [&](auto kernel, const uint32_t* table) {
                SALR_LAUNCH(kernel, dim3(grid + shared.extra), dim3(NW * 64), stream, ev, a.x, (int)a.M, a.K, a.N, a.bitmap, a.values, a.row_offsets,
                            t_partial, a.b_cat, R, Rpad, a.y, table, a.a_cat, shared);
            };
            // (a caller's table; without one there is no launch in front to build it in)
            if (a.slice_table != nullptr && !a.build_table) go(linear_stream_kernel<MT, NW, S, true, true, false, kQ, true>, a.slice_table);
            else go(linear_stream_kernel<MT, NW, S, true, false, false, kQ, true>, nullptr);
            return;
        }
    }
    if (R > 0) launch_adapter_partial(a, stream);
    // the optional events take the kernel's own begin/end timestamps (null events = plain launch)
    const int64_t wpr = a.K / 32;
    const uint32_t* no_table = nullptr;
    if (a.slice_table != nullptr && wpr % kChunkWords == 0)   // prepared layer: cursors from its slice table
        SALR_LAUNCH((linear_stream_kernel<MT, NW, S, true, true, false, kQ>), dim3(grid), dim3(NW * 64), stream, ev, a.x, (int)a.M,
                    a.K, a.N, a.bitmap, a.values, a.row_offsets, t_partial, a.b_cat, R, Rpad, a.y, a.slice_table, a.a_cat, SharedT());
    else if (wpr % kChunkWords != 0)  // bitmap rows are not multiples of 16 bytes: scalar bitmap loads
        SALR_LAUNCH((linear_stream_kernel<MT, NW, S, false>), dim3(grid), dim3(NW * 64), stream, ev, a.x, (int)a.M, a.K,
                    a.N, a.bitmap, a.values, a.row_offsets, t_partial, a.b_cat, R, Rpad, a.y, no_table, a.a_cat, SharedT());
    else   // (no ranks: with any there is a table)
        SALR_LAUNCH((linear_stream_kernel<MT, NW, S, true, false, false, kQ>), dim3(grid), dim3(NW * 64), stream, ev, a.x, (int)a.M,
                    a.K, a.N, a.bitmap, a.values, a.row_offsets, t_partial, a.b_cat, R, Rpad, a.y, no_table, a.a_cat, SharedT());
}

hipError_t launch_linear_stream(const LinearArgs& a, hipStream_t stream, const TimingEvents& ev) {
    constexpr int NW = 8;
    // More row groups than two per CU: the leaner variant (2 chunks in flight, 128 registers) lets two
    // workgroups share a CU, so one group's start-up and reduction overlap the other's stream.
    const bool many_groups = (a.N + kStreamRows - 1) / kStreamRows >= 2 * 256;
    if (a.M <= 16 && many_groups) launch_stream_t<1, NW, 2>(a, stream, ev);
    else if (a.M <= 16 && a.K > 2 * NW * kChunkWords * 32) launch_stream_t<1, NW, 4, true>(a, stream, ev);   // (three chunks a wave and more: two come faster one by one)
    else if (a.M <= 16) launch_stream_t<1, NW, 4>(a, stream, ev);
    else if (a.M <= 32) launch_stream_t<2, NW, 3>(a, stream, ev);
    else launch_stream_t<4, NW, 2>(a, stream, ev);
    return hipGetLastError();
}

}  // namespace salr
