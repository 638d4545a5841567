// T = X A_cat of a decoding call (up to 16 tokens), formed and handed over inside the launch that needs it.
//
// A launch for T in front costs the small-batch kernels 4 us of 12 to 16, whatever it does.  Their own workgroups, one a CU, need T only at
// their end, 8 us after their start, so the first kStreamTSlices * Rpad / 32 of them each form the product over one slice of K for 32 ranks
// beside their own start (two requests a step of 32 columns) and leave it to all.  Where CUs would be idle, workgroups of their own do.
//   partial sums   kStreamTSlices fp32 slices, the same sums in the same order as adapter_partial_kernel's: T has the same bits
//   words          one per slice and workgroup (salr_handover.hpp): a slice's workgroup meets every workgroup's word once its sums have
//                  reached memory.  A workgroup that finds the tag in all of its words at the end reads the sums and clears the words; one that
//                  has looked often enough in vain leaves its tag there, so that what comes later is cleared, and forms T itself.
//                  So nobody depends on which workgroups run at the same time.
// us a call, launch in front / so: see shares_t.
#pragma once

#include "salr_adapter_t.hpp"
#include "salr_handover.hpp"
#include "salr_internal.hpp"
#include "salr_linear_common.hpp"

namespace salr {

constexpr int kShareWaves = 8;
constexpr int kShareSteps = (int)(kSharedMaxColumns / 32 / kStreamTSlices / 4);   // of a wave at most
constexpr int kShareTileBytes = kShareSteps * 1024;             // of a wave
constexpr int kShareRedBytes = kShareWaves * 256 * 4;
constexpr int kShareMaxPairs = kSharedMaxRank / 32;

// The sums of slice `block` % kStreamTSlices for ranks 32 (block / kStreamTSlices) .. + 31: waves 0 to 3 the first sixteen ranks, every fourth
// step each, waves 4 to 7 the others.  R % 8 == 0.
struct SharedTProducts {
    uint4 a[kShareSteps], x[kShareSteps];
    int first, end;   // steps of 32 columns of this wave: first, first + 4, ..

    __device__ __forceinline__ void request(const uint16_t* __restrict__ x_in, int M, int64_t K, const uint16_t* __restrict__ a_cat, int R, int block,
                                            int wave, int lane) {
        const int i16 = lane & 15, g = lane >> 4;
        const int b = block % kStreamTSlices, rt = 2 * (block / kStreamTSlices) + (wave >> 2), units = (int)(K >> 5);
        first = units * b / kStreamTSlices + (wave & 3);
        end = 16 * rt < R ? units * (b + 1) / kStreamTSlices : 0;   // (ranks past R: nothing)
        const uint16_t* xr = x_in + (int64_t)(i16 < M ? i16 : M - 1) * K + 8 * g;
        // sixteen ranks of 32 rows of A_cat: 16 bytes a lane, row lane / 2 (ranks past R read valid ones and are dropped)
        const int r0 = 16 * rt + 8 * (lane & 1);
        const uint16_t* ar = a_cat + (int64_t)(lane >> 1) * R + (r0 < R ? r0 : R - 8);
#pragma unroll
        for (int t = 0; t < kShareSteps; ++t) {
            a[t] = x[t] = make_uint4(0, 0, 0, 0);
            if (first + 4 * t < end) {   // uniform
                a[t] = *reinterpret_cast<const uint4*>(ar + (int64_t)(first + 4 * t) * 32 * R);
                x[t] = *reinterpret_cast<const uint4*>(xr + 32 * (int64_t)(first + 4 * t));
            }
        }
    }
    // As accumulators of eight waves in `red` [8][4][64].  tiles: kShareTileBytes of this wave.
    __device__ __forceinline__ void multiply(uint16_t* tiles, float* red, int wave, int lane) {
        const int i16 = lane & 15, g = lane >> 4;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < kShareSteps; ++t) *reinterpret_cast<uint4*>(tiles + 512 * t + 8 * lane) = a[t];
        __builtin_amdgcn_wave_barrier();   // LDS executes a wave's accesses in order
#pragma unroll
        for (int t = 0; t < kShareSteps; ++t)
            if (first + 4 * t < end) {     // uniform
                const uint16_t* col = tiles + 512 * t + (8 * g + (i16 >> 2)) * 16 + 4 * (i16 & 3);
                const uint2 lo = lds_read_tr4(col), hi = lds_read_tr4(col + 64);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(x[t]), as_bf16x8(make_uint4(lo.x, lo.y, hi.x, hi.y)), acc, 0, 0, 0);
            }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int e = 0; e < 4; ++e) red[(wave * 4 + e) * 64 + lane] = acc[e];
    }
};

// One wave leaves what the waves have formed to all workgroups: sums [slice][M][Rpad], then the words.  What the last words held, which only
// matters where a workgroup has given up, is looked at by finish(), so that the wave goes on with its stream meanwhile.
struct SharedTHandOut {
    static constexpr int kAtOnce = 4;
    uint64_t before[kAtOnce];
    uint64_t* last;   // the words of the last exchanges, this lane's every 64th

    __device__ __forceinline__ void exchange(const SharedT& p, int left) {
#pragma unroll
        for (int i = 0; i < kAtOnce; ++i) {
            before[i] = 0;
            if (64 * i < left) before[i] = __hip_atomic_exchange(last + 64 * i, p.tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    __device__ __forceinline__ void start(const SharedT& p, float* sums, int M, int R, int Rpad, int block, int workgroups, const float* red, int lane) {
        const int b = block % kStreamTSlices, rp = block / kStreamTSlices;
        const Buffer out = make_buffer(sums, (uint64_t)kStreamTSlices * M * Rpad * 4);
#pragma unroll
        for (int i = 0; i < 2; ++i) {   // four ranks of a token each
            const int q = lane + 64 * i, m = q >> 3, rt = (q >> 2) & 1, col = 4 * (q & 3), r = 32 * rp + 16 * rt + col;
            f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < 4; ++w) s += *reinterpret_cast<const f32x4*>(red + ((4 * rt + w) * 4 + (m & 3)) * 64 + 16 * (m >> 2) + col);
            if (r >= R) s = f32x4{0.f, 0.f, 0.f, 0.f};   // (R % 8 == 0: all four or none)
            shared_store4(out, m < M ? (uint32_t)((b * M + m) * Rpad + r) * 4 : kPastBuffer, __builtin_bit_cast(u32x4, s));
        }
        stores_done();
        last = p.words + (int64_t)block * workgroups + lane;
        int left = workgroups - lane;
        exchange(p, left);
        while (workgroups > 64 * kAtOnce) {   // (uniform)
            finish(p);
            last += 64 * kAtOnce;
            left -= 64 * kAtOnce;
            workgroups -= 64 * kAtOnce;
            exchange(p, left);
        }
    }
    __device__ __forceinline__ void finish(const SharedT& p) {
#pragma unroll
        for (int i = 0; i < kAtOnce; ++i)
            if (before[i] == p.tag) leave_clear(last + 64 * i);   // that workgroup has formed T itself
    }
};

// A workgroup that does nothing else
__device__ __forceinline__ void shared_t_workgroup(const SharedT& p, const uint16_t* __restrict__ x, int M, int64_t K,
                                                   const uint16_t* __restrict__ a_cat, int R, int Rpad, float* sums, uint16_t* tiles, float* red,
                                                   int wave, int lane) {
    SharedTProducts products;
    products.request(x, M, K, a_cat, R, (int)blockIdx.x, wave, lane);
    products.multiply(tiles, red, wave, lane);
    __syncthreads();
    if (wave == 0) {
        SharedTHandOut out;
        out.start(p, sums, M, R, Rpad, (int)blockIdx.x, (int)gridDim.x - p.extra, red, lane);
        out.finish(p);
    }
}

// A workgroup's side, wave by wave: waves of the first M Rpad / 4 lanes each sum four ranks of a token per lane into t_lds
// [16][kMaxRankPadded]; M Rpad / 4 <= 512.
struct SharedTReader {
    uint64_t* word;      // this lane's slice
    uint64_t seen;
    bool asks, mine;     // this lane looks at a word; this wave has sums to read (uniform)
    bool there;          // (uniform)
    uint64_t tag;
    Buffer sums;
    int groups, item;
    f32x4 v[kStreamTSlices];

    __device__ __forceinline__ SharedTReader(const SharedT& p, const float* t_sums, int M, int Rpad, int workgroups, int workgroup, int wave, int lane)
        : word(p.words + (int64_t)lane * workgroups + workgroup), seen(0), asks(lane < kStreamTSlices * (Rpad >> 5)), there(false), tag(p.tag),
          sums(make_buffer(const_cast<float*>(t_sums), (uint64_t)kStreamTSlices * M * Rpad * 4)), groups(M * (Rpad >> 2)), item(64 * wave + lane) {
        mine = 64 * wave < groups;
    }
    __device__ __forceinline__ void look() {
        if (mine && asks) seen = look_at(word);
    }
    __device__ __forceinline__ bool check() {
        there = mine && __builtin_amdgcn_ballot_w64(asks && seen != tag) == 0;
        return there;
    }
    __device__ __forceinline__ void request() {
#pragma unroll
        for (int sl = 0; sl < kStreamTSlices; ++sl)
            v[sl] = __builtin_bit_cast(f32x4, shared_load4(sums, item < groups ? 16u * (uint32_t)(sl * groups + item) : kPastBuffer));
    }
    __device__ __forceinline__ void add_up(uint16_t* t_lds, int Rpad) {
        f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int sl = 0; sl < kStreamTSlices; ++sl) sum += v[sl];
        if (item < groups) {
            const int m = item / (Rpad >> 2), r4 = item % (Rpad >> 2);
            uint2 o;
            o.x = (uint32_t)f32_to_bf16_rne(sum[0]) | ((uint32_t)f32_to_bf16_rne(sum[1]) << 16);
            o.y = (uint32_t)f32_to_bf16_rne(sum[2]) | ((uint32_t)f32_to_bf16_rne(sum[3]) << 16);
            *reinterpret_cast<uint2*>(&t_lds[m * kMaxRankPadded + 4 * r4]) = o;
        }
    }
    // The wave has nothing left to do but this.  True where T is in t_lds or not this wave's to fetch.
    __device__ __forceinline__ bool finish(const SharedT& p, uint16_t* t_lds, int Rpad) {
        if (!mine) return true;
        if (!there) {
            for (int i = 0; i < p.polls; ++i) {
                look();
                if (check()) break;   // uniform
                __builtin_amdgcn_s_sleep(1);
            }
            if (!there) return false;
            request();
        }
        add_up(t_lds, Rpad);
        return true;
    }
    // By one wave, when all are past finish()
    __device__ __forceinline__ void leave(bool all_there) {
        if (!asks) return;
        if (all_there) leave_clear(word);
        else meet(word, tag);
    }
};

// T by this workgroup alone (512 threads; LDS is free but for t_lds, whose bytes are `red` until the end)
__device__ __forceinline__ void shared_t_alone(const uint16_t* __restrict__ x, int M, int64_t K, const uint16_t* __restrict__ a_cat, int R, int Rpad,
                                               uint16_t* tiles, uint16_t* t_lds, int tid, int wave, int lane) {
    float total[kShareMaxPairs];
    float* red = reinterpret_cast<float*>(t_lds);
    const int rt = tid >> 8, e = (tid >> 6) & 3;
#pragma unroll
    for (int rp = 0; rp < kShareMaxPairs; ++rp) {
        total[rp] = 0.f;
        if (32 * rp < Rpad)   // uniform
#pragma unroll 1
            for (int b = 0; b < kStreamTSlices; ++b) {
                __syncthreads();
                SharedTProducts products;
                products.request(x, M, K, a_cat, R, rp * kStreamTSlices + b, wave, lane);
                products.multiply(tiles, red, wave, lane);
                __syncthreads();
                float s = 0.f;
#pragma unroll
                for (int w = 0; w < 4; ++w) s += red[((4 * rt + w) * 4 + e) * 64 + lane];
                total[rp] += s;
            }
    }
    __syncthreads();
#pragma unroll
    for (int rp = 0; rp < kShareMaxPairs; ++rp) {
        const int r = 32 * rp + 16 * rt + (lane & 15);
        if (32 * rp < Rpad) t_lds[(4 * (lane >> 4) + e) * kMaxRankPadded + r] = r < R ? f32_to_bf16_rne(total[rp]) : (uint16_t)0;
    }
    __syncthreads();
}

}  // namespace salr
