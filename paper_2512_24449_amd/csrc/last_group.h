// The end of a split context in the kernel that split it: every workgroup counts itself off at its stream's counter when
// its partial rows are stored, and the last one merges the stream's rows, one wave per query head.  Saves the launch
// of a merging kernel where launches are what a call costs: few streams, short contexts.
//
// The partial rows go out with agent-scope stores and are read with agent-scope loads: the dies' L2 caches are not
// coherent with each other for ordinary accesses inside a kernel.  Nothing waits: a workgroup that is not the
// last one ends.  The counters are zero between calls (calls on one cache do not overlap).  A stream has one for each
// of the calls that merge, a byte of one word each: calls that overlap all the same, which kv_v_matvec_noalloc may with those
// that use the workspace, do not count for one another, and two of one kind and size leave zero behind.
#pragma once

#include "unpack.h"

namespace packkv {

// The rule.  Counting costs every workgroup the way of its rows to memory and an atomic, and the last one its merge; the launch
// it saves costs the host some 3 us and the GPU a gap.  Passes back to back / replayed from a graph, merged here and by a
// kernel of its own: fused attention, 1 stream in 4 workgroups 12.7 / 11.5 and 16.2 / 12.2 us, 32 in 128 13.0 / 12.3 and 16.2 /
// 13.0, 8 of four heads in 128 14.7 / 14.3 and 16.4 / 14.5, 32 in 512 16.1 / 16.0 and 16.0 / 15.4; three steps, 1 in 4 23.2 /
// 15.8 and 26.4 / 16.7.  Wide chunks, whose kernels run longer than the host takes: 16 in 128 17.0 / 17.1 and 16.6 / 16.4.
// A wave merges a head, so more than four heads take it a second turn, and with seven and eight the merge held registers in scratch:
// 2 streams of packs of 8 in 16 workgroups, merged here and by a kernel of its own, fused attention at five heads 13.5 / 11.7 us,
// six 14.4 / 12.3, seven 15.1 / 12.9, eight 19.9 / 13.4, V product 8.3 / 7.5, 8.4 / 7.6, 8.6 / 7.6, 8.7 / 7.7 (four heads 10.6 /
// 11.2 and 6.9 / 7.4).
constexpr int MERGED_HEADS = 4;
inline bool merge_in_kernel(int64_t groups, int64_t streams, int heads, bool wide = false) {
    return heads <= MERGED_HEADS && streams <= COUNTED_STREAMS && groups <= (wide ? 64 : 128);
}

__device__ inline void store_shared(float *to, float x, float y) {
    const uint64_t v = uint64_t(__float_as_uint(x)) | (uint64_t(__float_as_uint(y)) << 32);
    __hip_atomic_store(reinterpret_cast<uint64_t *>(to), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline float2 load_shared(const float *from) {
    const uint64_t v = __hip_atomic_load(reinterpret_cast<const uint64_t *>(from), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return make_float2(__uint_as_float(uint32_t(v)), __uint_as_float(uint32_t(v >> 32)));
}

enum { COUNT_ATTENTION = 0, COUNT_V = 1, COUNT_V_NOALLOC = 2 };  // byte of the word

// Whether this workgroup is the last of `expected` (at most 64) at the counter, a byte (which it then sets back).  All
// threads call, with their agent-scope stores issued; flag: a word of LDS.  Contains two workgroup barriers.
__device__ inline bool last_group(uint8_t *counter, uint32_t expected, uint32_t *flag) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's stores are where the others will read
    __syncthreads();
    if (threadIdx.x == 0) {
        const int byte = int(reinterpret_cast<uintptr_t>(counter) & 3u), shift = 8 * byte;
        uint32_t *word = reinterpret_cast<uint32_t *>(counter - byte);
        const uint32_t before = __hip_atomic_fetch_add(word, 1u << shift, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t mine = ((before >> shift) & 255u) + 1;
        const bool last = mine == expected || mine == 2 * expected;   // (2: of two calls that overlap)
        if (last) __hip_atomic_fetch_sub(word, expected << shift, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *flag = last;
    }
    __syncthreads();
    return *flag != 0;
}

// Channels 2 lane, 2 lane + 1 of the weighted sum of n <= 64 partial rows, `stride` floats apart; weight: lane s holds row
// s's.  The first rows are loaded ahead of their weights.
struct RowSum {
    static constexpr int BATCH = 8;
    float2 v[BATCH];
    __device__ inline void load(const float *rows, int64_t stride, int first, int n, int lane) {
#pragma unroll
        for (int k = 0; k < BATCH; ++k)
            if (first + k < n) v[k] = load_shared(rows + (first + k) * stride + 2 * lane);
    }
    __device__ inline float2 sum(const float *rows, int64_t stride, int n, float weight, int lane) {
        float2 acc = make_float2(0.0f, 0.0f);
#pragma unroll 1
        for (int first = 0; first < n; first += BATCH) {
            if (first) load(rows, stride, first, n, lane);
#pragma unroll
            for (int k = 0; k < BATCH; ++k) {
                if (first + k < n) {
                    const float w = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(weight), first + k));
                    acc.x = fmaf(w, v[k].x, acc.x), acc.y = fmaf(w, v[k].y, acc.y);
                }
            }
        }
        return acc;
    }
};

// Raw fp16 V tail, one wave: channels 8 (lane % 16) .. of the tokens lane / 16 + 4 i, 16 bytes per load, 32 tokens at a time
// (the first of them loaded ahead of their weights).
struct TailSum {
    uint4 raw[8];
    // vrow: the head's 128 values of tail token 0; token_stride in elements
    __device__ inline void load(const __half *vrow, int64_t token_stride, int first, int n_tail, int lane) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int t = first + (lane >> 4) + 4 * i;
            raw[i] = make_uint4(0, 0, 0, 0);
            if (t < n_tail) raw[i] = *reinterpret_cast<const uint4 *>(vrow + t * token_stride + 8 * (lane & 15));
        }
    }
    // weight: 64 floats in LDS, 0 from n_tail on.  The sums of channels 2 lane, 2 lane + 1.
    __device__ inline float2 sum(const __half *vrow, int64_t token_stride, const float *weight, int n_tail, float *lds128, int lane) {
        float acc[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) acc[k] = 0.0f;
#pragma unroll 1
        for (int first = 0; first < n_tail; first += 32) {
            if (first) load(vrow, token_stride, first, n_tail, lane);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const __half *hv = reinterpret_cast<const __half *>(&raw[i]);
                const float w = weight[first + (lane >> 4) + 4 * i];
#pragma unroll
                for (int k = 0; k < 8; ++k) acc[k] = fmaf(w, __half2float(hv[k]), acc[k]);
            }
        }
        // the four rows' sums; row r keeps two of the eight channels
        float two[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            uint32_t a = __float_as_uint(acc[k]), b = __float_as_uint(acc[4 + k]), c = __float_as_uint(acc[2 + k]), d = __float_as_uint(acc[6 + k]);
            swap_rows32(a, b);
            swap_rows32(c, d);
            uint32_t lo = __float_as_uint(__uint_as_float(a) + __uint_as_float(b)), hi = __float_as_uint(__uint_as_float(c) + __uint_as_float(d));
            swap_rows16(lo, hi);
            two[k] = __uint_as_float(lo) + __uint_as_float(hi);
        }
        // row 0: channels 0, 1 of the eight, row 1: 2, 3, row 2: 4, 5, row 3: 6, 7; to lane = channel pair
        *reinterpret_cast<float2 *>(lds128 + 8 * (lane & 15) + 4 * (lane >> 5) + 2 * ((lane >> 4) & 1)) = make_float2(two[0], two[1]);
        wave_lds_fence();
        const float2 r = *reinterpret_cast<const float2 *>(lds128 + 2 * lane);
        wave_lds_fence();
        return r;
    }
};

}  // namespace packkv
