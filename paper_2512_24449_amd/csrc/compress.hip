// Append-side compressor: token-wise quantization, bit-packing, appending
// (PackKV Sec. III-B.1 .. III-B.4).  Cold path: runs once per 64 decode steps.
//
// In a contiguous arena whose free space takes even the largest chunks, or in a
// paged arena if the staging area takes the whole round (staged path, the input is read and quantized once; codes up to 127):
//   quantize       resident workgroups, 16 tokens of all kv-heads at a time each: min/max over a token's
//                  H*128 values -> fp16 scale = rel*(max-min), fp16 min; the codes, pack headers and pack bytes per
//                  token group to a fixed slot per chunk of the staging area
//   place_small    (paged) chunk positions, from the pack bytes
//   assemble       one wave per chunk: codes to bit planes (packs of 8: consecutive bits) at the chunk's place in the arena; contiguous: the
//                  workgroup adds up the sizes before its chunks and sets their index words
// with more than 64 kv-heads or V-median repacking the scales come first:
//   token_params   a workgroup or a wave per (token, batch)
//   v_median_key, block_order   (V-median repacking only) sort key per token,
//                  order of the 64 tokens of a block, metadata into storage order
// else (two-pass path: large rounds of paged arenas or small staging areas, a nearly full arena, codes above 127):
//   quantize       as above, metadata and width sums only; or token_params and
//   chunk_sizes    one workgroup per chunk: quantize, per-pack width -> bytes
//   scan_offsets / place_small, place_chunks (paged arena) one workgroup: chunk positions -> index;
//                  paged: inside pages taken from a shared pool, index of (start, end) pairs
//   pack_chunks    one workgroup per chunk: quantize again and write header +
//                  payload at its final place
// K and V share every launch.  The arena bytes are a pure function of the input, whichever way a round takes: the rules for a code agree on every
// bit pattern (quantize_value.h), and the atomics are ORs and counts in LDS, in any order the same, and the page stack's update.
// (Only the metadata of a token without a single number differs between the ways.)
#include <algorithm>
#include <atomic>

#include "quantize_value.h"
#include "unpack.h"

namespace packkv {

// Eight consecutive input values as fp16.  fp16 inputs pass as they are; bf16 inputs are rounded
// to fp16 (to nearest even; exact for every value in fp16's normal range, fp16 having the longer
// significand) -- from there on the path does not know the input type.
__device__ inline uint4 as_fp16(uint4 raw, bool bf16) {
    if (bf16) {
        uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            typedef float f32x2 __attribute__((ext_vector_type(2)));
            typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
            const f32x2 both = {__uint_as_float(w[k] << 16), __uint_as_float(w[k] & 0xFFFF0000u)};
            w[k] = __builtin_bit_cast(uint32_t, __builtin_convertvector(both, f16x2));   // one instruction, to nearest even
        }
        raw = make_uint4(w[0], w[1], w[2], w[3]);
    }
    return raw;
}
// A round whose input is larger than the last-level cache (256 MB; both tensors): its kernels read with the non-
// temporal hint (STREAM), which keeps the input from pushing out what is read again, the staged chunks for one. The
// input of a smaller round may still be in the caches from what wrote it or is read again from them (packs of 8, repacked
// tokens), which the hint would not make use of.  Without / with the hint: packs of 8, 67 MB 80 / 84 us, 262 MB 243 / 265, 393 MB 389 / 381, 1.7 GB
// 1648 / 1618; packs of 16, 67 MB 28.9 / 29.5 (repacked 53.0 / 54.5), 255 MB 116.8 / 116.0, 788 MB 277 / 267, a block of
// 416 streams 16.1 / 17.4.
inline bool larger_than_caches(int64_t n_chunks) { return n_chunks * 2 * (N * D * 2) > (int64_t(256) << 20); }

__device__ inline uint4 load8_nt(const __half *p) {
    typedef uint32_t u32x4n __attribute__((ext_vector_type(4)));
    const u32x4n v = __builtin_nontemporal_load(reinterpret_cast<const u32x4n *>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
}
template <bool STREAM>
__device__ inline uint4 load8(const __half *p) {
    return STREAM ? load8_nt(p) : *reinterpret_cast<const uint4 *>(p);
}
template <bool STREAM>
__device__ inline uint4 load8_as_fp16(const __half *p, bool bf16) {
    return as_fp16(load8<STREAM>(p), bf16);
}

// A token's metadata word from its smallest and largest value: fp16 scale | fp16 minimum << 16.
__device__ inline uint32_t token_meta_word(float mn, float mx, float rel) {
    float range = mx - mn;
    float s = rel * range;
    // The product is rounded to fp32 first and to fp16 second; keep the
    // compiler from fusing both into one mixed-precision FMA (one rounding).
    asm volatile("" : "+v"(s));
    const uint32_t s16 = __half_as_ushort(__float2half_rn(s)) & 0x7FFFu;  // the range of zeros of either sign is +0
    uint32_t m16 = __half_as_ushort(__float2half_rn(mn));                // exact: mn is an fp16 value
    m16 = m16 == 0x8000u ? 0u : m16;                                      // a zero minimum is stored as +0
    return s16 | (m16 << 16);
}

// ---------------------------------------------------------------------------
// Both tensors of an append share every launch (blockIdx.z or the item number says which): the
// launches of a small round cost more than its work.
struct ParamTensor {
    const __half *src;
    float rel;
    uint32_t *meta;
};
struct ParamArgs {
    ParamTensor t[2];
    int64_t batch_stride, token_stride, meta_stride, first_token;
    int row_elems;
    bool bf16;
};

// A workgroup per token, or (WAVE: rows of up to 2048 values, which would leave lanes of a workgroup
// idle) a wave per token, four tokens to a workgroup.
template <bool WAVE, bool STREAM>
__global__ __launch_bounds__(256) void token_params_kernel(ParamArgs a, int n_tokens) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int t = WAVE ? blockIdx.x * 4 + wave : blockIdx.x, b = blockIdx.y;
    if (WAVE && t >= n_tokens) return;
    const ParamTensor &pt = a.t[blockIdx.z];
    const __half *row = pt.src + b * a.batch_stride + t * a.token_stride;
    float mn = INFINITY, mx = -INFINITY;
    constexpr int STEP = (WAVE ? 64 : 256) * 8;
    for (int i = (WAVE ? lane : int(threadIdx.x)) * 8; i < a.row_elems; i += STEP) {
        uint4 raw = load8_as_fp16<STREAM>(row + i, a.bf16);
        const __half *h = reinterpret_cast<const __half *>(&raw);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            float v = __half2float(h[k]);
            mn = fminf(mn, v);
            mx = fmaxf(mx, v);
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        mn = fminf(mn, __shfl_xor(mn, o));
        mx = fmaxf(mx, __shfl_xor(mx, o));
    }
    if constexpr (!WAVE) {
        __shared__ float smn[4], smx[4];
        if (lane == 0) {
            smn[wave] = mn;
            smx[wave] = mx;
        }
        __syncthreads();
        mn = fminf(fminf(smn[0], smn[1]), fminf(smn[2], smn[3]));
        mx = fmaxf(fmaxf(smx[0], smx[1]), fmaxf(smx[2], smx[3]));
    }
    if (WAVE ? lane == 0 : threadIdx.x == 0)
        pt.meta[b * a.meta_stride + a.first_token + t] = token_meta_word(mn, mx, pt.rel);
}

// Quantize the PK tokens of one pack (channel d of token group g) and derive
// its minimum, width and code bits.
struct PackBits {
    uint64_t bits;
    int w, m;
};

// A token's (scale, minimum, 1 / scale) from its metadata word (fp16 scale | fp16 minimum << 16).
__device__ inline float4 token_scale_min(uint32_t mt) {
    const float s = __half2float(__ushort_as_half(uint16_t(mt & 0xFFFFu)));
    const float mn = __half2float(__ushort_as_half(uint16_t(mt >> 16)));
    return make_float4(s, mn, s != 0.0f ? 1.0f / s : 0.0f, 0.0f);
}

// tile: the block's 64 x 128 values in LDS, rows already in storage order; the pack holds rows
// PK*g..PK*g+PK-1 of channel d; sm: token_scale_min of the block's 64 tokens (storage order), in LDS.
template <int PK>
__device__ inline PackBits make_pack(const __half *tile, int g, int d, const float4 *sm, int qmax) {
    int q[PK];
    int lo = 255, hi = 0;
#pragma unroll
    for (int i = 0; i < PK; ++i) {
        const float4 t = sm[g * PK + i];
        const int v = quantize_value(__half2float(tile[(g * PK + i) * D + d]), t.x, t.y, t.z, qmax);
        q[i] = v;
        lo = min(lo, v);
        hi = max(hi, v);
    }
    PackBits pb;
    int range = hi - lo;
    pb.w = range == 0 ? 0 : 32 - __clz(range);
    pb.m = lo;
    // two halves of PK/2 codes, at most 32 bits each, built with 32-bit shift-and-or steps from
    // the top code down; one 64-bit shift joins them
    uint32_t half_lo = 0, half_hi = 0;
#pragma unroll
    for (int i = PK / 2 - 1; i >= 0; --i) {
        half_lo = (half_lo << pb.w) | uint32_t(q[i] - lo);
        half_hi = (half_hi << pb.w) | uint32_t(q[PK / 2 + i] - lo);
    }
    pb.bits = uint64_t(half_lo) | (uint64_t(half_hi) << (PK / 2 * pb.w));
    return pb;
}

// Exclusive prefix sum over the 256 threads of a workgroup; also returns the total.
__device__ inline int block_exclusive_scan(int v, int *total) {
    __shared__ int wave_sum[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int inc = wave_inclusive_scan(v);
    __syncthreads();  // protects wave_sum against a previous call
    if (lane == 63) wave_sum[wave] = inc;
    __syncthreads();
    int base = 0;
    for (int k = 0; k < wave; ++k) base += wave_sum[k];
    *total = wave_sum[0] + wave_sum[1] + wave_sum[2] + wave_sum[3];
    return base + inc - v;
}

struct ChunkSource {
    const __half *src;
    int64_t batch_stride, token_stride;
    int B, H, qmax;
    uint64_t magic_h, magic_hb;  // floor(2^32 / H) + 1, floor(2^32 / (H * B)) + 1
    uint32_t *meta;
    int64_t meta_stride, first_token;
    const uint8_t *order;
    bool bf16;
    int pack_order;
};

// One tensor's side of a round or part.
struct PackTensor {
    ChunkSource cs;
    StagedRound round;
    uint32_t *index;
    uint8_t *arena;
    uint32_t *sizes16;      // two-pass: sizes of the round's chunks, 16-byte units
    uint16_t *widths;       // staged: sums of the pack widths of the part's chunks, [chunk][token group] (8-byte aligned)
    float rel;
    bool cap_all;           // staged: see QuantRange
    float small_scale;
    bool wide;              // packs of 8: wide chunk layout
    uint32_t stage_at, slot;  // staged: where the tensor's slots start in the staging area, bytes of a slot
    uint32_t header16, unit_shift;  // size of a chunk from its width sums: chunk_units
    uint64_t arena_cap16;
    uint32_t *status;       // set when the round does not fit
    uint32_t *page_list;    // paged arena
    int64_t max_pages;
    __half *tail;           // raw tail, and what of the new tokens the round's last kernel copies to its start
    const __half *rest;
};
struct PackArgs {
    PackTensor t[2];        // K, V
    int part_first, n;      // chunks part_first .. part_first + n - 1 of the round, in both tensors
    int part_row, rows;     // the same in rows of H chunks (row = blk*B + b)
    int round_rows;         // rows of the whole round
    uint64_t magic_b;       // floor(2^32 / B) + 1
    int index_words;
    int first_tensor;       // a launch whose grid covers one tensor: which (else 0)
    uint32_t *pool_state;   // paged arena
    int split;              // workgroups that share an item's quantization (quantize16_kernel)
    int held;               // > 0: the round is one block, and its first `held` tokens are in the tail
    uint8_t *keys;          // codes moved into storage order (move_codes_kernel): the tokens' sort keys, later their order
    int rest_units;         // 16-byte units of a batch element that the tail takes behind the round, 0: none
    int64_t rest_stride;    // elements between the batch elements of `rest`
    bool rest_bf16;
    uint8_t *staging;       // chunk i of the part in the tensor's slot i: the pack headers [group][channel], then the codes
                            // of the packs (quantize16_kernel)
};

// Two-pass path, packs of 8 (Sec. IV-B; packs of 16 have their own kernel below).  One workgroup per new chunk: the chunk has 64/PK token groups of 128 packs, thread tau owns packs tau + 256k
// (token group (tau >> 7) + 2k, channel tau & 127).  A pack takes PK*w/8 payload bytes.  WIDE (codes above 15, packs of 8): the
// header is a width byte per pack followed by a minimum byte per pack, widths go up to 8.
template <bool WRITE, int PK, bool WIDE, bool STREAM>
__global__ __launch_bounds__(256) void chunk_kernel(PackArgs a) {
    static_assert(PK == 8, "contiguous packs are packs of 8 tokens");
    constexpr int NPACKS = N / PK * D;
    constexpr int HDR = WIDE ? 2 * NPACKS : NPACKS;  // header bytes
    constexpr int PER = N / PK * D / 256;  // packs per thread
    const PackTensor &t = a.t[a.first_tensor + blockIdx.y];
    const ChunkSource &cs = t.cs;
    const int cl = blockIdx.x;  // chunk within this round: (blk*B + b)*H + h
    const int h = cl % cs.H;
    const int b = (cl / cs.H) % cs.B;
    const int blk = cl / (cs.H * cs.B);
    const int tau = threadIdx.x;
    const int d = tau & 127;

    uint8_t *dst = nullptr;
    uint32_t room16 = 0;
    if (WRITE) {
        const int64_t e = (t.round.first_chunk + cl) * a.index_words;
        uint32_t o0 = t.index[e], o1 = t.index[e + 1];
        if (o1 == o0) return;  // dropped: the arena was full
        dst = t.arena + size_t(o0) * 16;
        room16 = o1 - o0;
    }

    // stage the block's 64 x 128 values in LDS with 16-byte loads, rows in storage order, and the
    // tokens' scales and minimums as floats (every thread needs all 64 of them)
    __shared__ __attribute__((aligned(16))) __half tile[N * D];
    __shared__ float4 sm[N];
    if (tau < N) sm[tau] = token_scale_min(cs.meta[b * cs.meta_stride + cs.first_token + int64_t(blk) * N + tau]);
    {
        const __half *x_blk = cs.src + b * cs.batch_stride + int64_t(blk) * N * cs.token_stride + h * D;
        const uint8_t *ord = cs.order ? cs.order + b * cs.meta_stride + cs.first_token + int64_t(blk) * N : nullptr;
#pragma unroll
        for (int pass = 0; pass < 4; ++pass) {
            const int row = pass * 16 + (tau >> 4), c8 = (tau & 15) * 8;
            const int src_row = ord ? ord[row] : row;
            *reinterpret_cast<uint4 *>(tile + row * D + c8) = load8_as_fp16<STREAM>(x_blk + src_row * cs.token_stride + c8, cs.bf16);
        }
    }
    __syncthreads();

    PackBits pb[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int g = (tau >> 7) + 2 * k;
        pb[k] = make_pack<PK>(tile, g, d, sm, cs.qmax);
    }
    // all packs are quantized before the first barrier of the scans
    int off[PER];
    int payload = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        int total;
        off[k] = payload + block_exclusive_scan(PK / 8 * pb[k].w, &total);
        payload += total;
    }
    const int padded = (HDR + payload + 15) & ~15;

    if (!WRITE) {
        if (tau == 0) t.sizes16[cl] = uint32_t(padded >> 4);
        return;
    }
    // The sizes come from the same codes, so this never happens; should it all the same, nothing is written behind the chunk's place, and a
    // header of zeros makes it 64 tokens of code 0.
    if (uint32_t(padded) > 16 * room16) {
        for (int i = tau; i < HDR && uint32_t(i) < 16 * room16; i += 256) dst[i] = 0;
        return;
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        if constexpr (WIDE) {
            dst[tau + 256 * k] = uint8_t(pb[k].w);
            dst[NPACKS + tau + 256 * k] = uint8_t(pb[k].m);
        } else {
            dst[tau + 256 * k] = uint8_t((pb[k].w << 4) | pb[k].m);
        }
        uint8_t *out = dst + HDR + off[k];
        for (int j = 0; j < pb[k].w; ++j) out[j] = uint8_t(pb[k].bits >> (8 * j));
    }
    if (tau < padded - HDR - payload) dst[HDR + payload + tau] = 0;
}

// ---- packs of 16 tokens, plane layout (packkv.h) --------------------------------------------
// One workgroup per chunk, wave w = token group w.  Lane (cg = lane % 16, q = lane / 16) loads the
// channels 8 cg .. 8 cg + 7 of the four tokens 16 w + 8 (q / 2) + q % 2 + 2 i and quantizes them; a
// 4 x 4 exchange between the lanes of one cg (eight row swaps) then leaves each lane all sixteen
// tokens of the channels 8 cg + 2 q and 8 cg + 2 q + 1: its two packs.  No LDS tile and no barrier
// on the way; the waves meet once for the byte counts of their packs and once when the chunk's
// bytes are complete in LDS.

struct PlaneBits {
    uint32_t low, high, top;  // top: in the low 16 bits
    int w, m;
};

// n0, n1: the 16 codes of a pack as nibbles (tokens 0..7, 8..15); lo, hi: their minimum and maximum.
__device__ inline PlaneBits planes_from_nibbles(uint32_t n0, uint32_t n1, uint32_t lo, uint32_t hi) {
    PlaneBits pb;
    pb.w = 32 - __clz(int(hi - lo));  // 0 for equal codes
    pb.m = int(lo);
    // codes minus the pack minimum: no nibble borrows (every code is at least the minimum)
    uint32_t all = lo | (lo << 4);
    all |= all << 8;
    all |= all << 16;
    n0 -= all;
    n1 -= all;
    // planes of two-bit fields: token i at bits [4i, 4i+2) for i < 8, at [4(i-8)+2, 4(i-8)+4) for i >= 8
    pb.low = (n0 & 0x33333333u) | ((n1 << 2) & 0xCCCCCCCCu);
    pb.high = ((n0 >> 2) & 0x33333333u) | (n1 & 0xCCCCCCCCu);
    // top bit of every code, token i at bit 4 (i % 4) + i / 4
    const int top_bit = max(pb.w - 1, 0);
    const uint32_t t0 = (n0 >> top_bit) & 0x11111111u, t1 = (n1 >> top_bit) & 0x11111111u;
    const uint32_t y0 = t0 | (t0 >> 15), y1 = t1 | (t1 >> 15);
    pb.top = y0 | (y1 << 2);
    return pb;
}

typedef unsigned short pk_u16 __attribute__((ext_vector_type(2)));
__device__ inline uint32_t pk_min(uint32_t x, uint32_t y) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(pk_u16, x), __builtin_bit_cast(pk_u16, y)));
}
__device__ inline uint32_t pk_max(uint32_t x, uint32_t y) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(pk_u16, x), __builtin_bit_cast(pk_u16, y)));
}

// What a lane loads of a chunk: eight channels of its four tokens, and the metadata word of token
// 16 w + lane % 16 of the block (storage order).
struct ChunkInput {
    uint4 raw[4];
    uint32_t mt;
};

// LDS of a workgroup that builds a chunk.
struct ChunkLds {
    float4 tok[N];              // token_quant of the block's tokens
    __attribute__((aligned(16))) uint32_t counts[4][64];  // per wave: byte counts of the packs (see build_plane_chunk)
    __attribute__((aligned(16))) uint8_t image[CHUNK_MAX];
};

// Chunk cl of the round is (blk*B + b)*H + h.  cl is the same for the whole workgroup, so the
// quotients are scalar work: x / d = (x * (floor(2^32 / d) + 1)) >> 32 for x * d < 2^32
// (cl < 2^16 here, H * B <= 2^16).
struct ChunkCoord {
    int h, b, blk;
};
__device__ inline ChunkCoord chunk_coord(const ChunkSource &cs, int cl) {
    const uint32_t c = uint32_t(__builtin_amdgcn_readfirstlane(cl));
    const uint32_t by_h = uint32_t((uint64_t(c) * cs.magic_h) >> 32);
    const uint32_t blk = uint32_t((uint64_t(c) * cs.magic_hb) >> 32);
    ChunkCoord k;
    k.h = int(c - by_h * uint32_t(cs.H));
    k.b = int(by_h - blk * uint32_t(cs.B));
    k.blk = int(blk);
    return k;
}

// Loads chunk cl of the round, (blk*B + b)*H + h: the lane's four tokens are rows row0 + 2i of the block in storage order,
// at the source positions the token order gives.
__device__ inline ChunkInput load_chunk_input(const ChunkSource &cs, int cl) {
    const ChunkCoord k = chunk_coord(cs, cl);
    const int h = k.h, b = k.b, blk = k.blk;
    const int cg = threadIdx.x & 15, q = threadIdx.x >> 4;  // q: 4 * wave + lane / 16
    const int row0 = 16 * (q >> 2) + 8 * ((q >> 1) & 1) + (q & 1);
    const __half *x_blk = cs.src + b * cs.batch_stride + int64_t(blk) * N * cs.token_stride + h * D + cg * 8;
    const int64_t tok0 = b * cs.meta_stride + cs.first_token + int64_t(blk) * N;
    int row[4];
    if (cs.order) {
#pragma unroll
        for (int i = 0; i < 4; ++i) row[i] = cs.order[tok0 + row0 + 2 * i];
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) row[i] = row0 + 2 * i;
    }
    ChunkInput in;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        in.raw[i] = *reinterpret_cast<const uint4 *>(x_blk + row[i] * cs.token_stride);  // converted where it is used
    in.mt = cs.meta[tok0 + 16 * (threadIdx.x >> 6) + cg];
    return in;
}

// Quantization (Sec. III-B.2: clamp(rint(fl((x - mn) / s)), 0, qmax), the quotient rounded to fp32
// as an IEEE divide does), qmax < 16.  Fast path, one fused multiply-add per value:
//     t = fl(x * r + c),   r = 1 / s to within an ulp,   c = fl(128 + 1/2 + g * 2^-16 - mn * r)
// The quotient (x - mn) * r is below 24 (the largest value over an fp16 scale that may have been
// rounded down from half a subnormal step more), so t lies in [128, 256), where a float is a fixed-
// point number with 16 fraction bits: bits 16.. of its pattern are 0x4300 + floor(quotient + 1/2 + g).
// Error of t against quotient + 1/2 + g, in units of 2^-16: half for t's own rounding, half an ulp
// of c (half a unit for |c| < 256, 2^(e-8) for |c| below 2^(e+1)), 0.19 for r, 0.16 for the roundings of
// the subtraction and the quotient in the definition: below 1.4 + 2^(e-8).  With g = 3 (+ 2^(e-7) for
// e >= 8) the quotient can only be on the other side of a rounding tie, or on one, if the fraction
// field of t is below 2g: then the token's eight values take the divide.  A token whose offset is so
// large against its scale that g reaches 1/2 always does, infinite offsets and scales among them.  A NaN
// gets qmax: its pattern is above the clamp's on the fast path, and the divide's minimum
// takes qmax.  s = 0: r = 0, code 0; t is then 128 + (1 - 2^-16) for every number, at the guard, while a NaN, from infinite values too, lies below it (its
// low 13 bits are 0) and takes the divide, which gives 0.
struct TokenQuant {
    float r, c;
    uint32_t guard;  // 2g
    uint32_t mt;     // fp16 scale | fp16 minimum << 16
};
__device__ inline float4 token_quant(uint32_t mt) {
    const float s = __half2float(__ushort_as_half(uint16_t(mt & 0xFFFFu)));
    const float mn = __half2float(__ushort_as_half(uint16_t(mt >> 16)));
    const float r = s != 0.0f ? __builtin_amdgcn_rcpf(s) : 0.0f;
    const int e = int((__float_as_uint(fmaf(-mn, r, 128.5f)) >> 23) & 0xFFu) - 127;
    const uint32_t g = 3u + (e >= 8 ? 2u << min(e - 8, 14) : 0u);
    const float c = s != 0.0f ? fmaf(-mn, r, 128.5f + float(g) * (1.0f / 65536.0f)) : __uint_as_float(0x4300FFFFu);
    return make_float4(r, c, __uint_as_float(s != 0.0f ? 2u * g : 0xFFFFu), __uint_as_float(mt));
}

// x * r + c for the low (HI = false) or high half x of a word of two fp16 values, rounded once.
template <bool HI>
__device__ inline float half_mul_add(uint32_t two_halves, float r, float c) {
    float t;
    if (HI)
        asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(t) : "v"(two_halves), "v"(r), "v"(c));
    else
        asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel_hi:[1,0,0]" : "=v"(t) : "v"(two_halves), "v"(r), "v"(c));
    return t;
}

// The eight values of one token a lane holds: pair[k] = 0x4300 + code of values 2k (low half) and 2k + 1.
__device__ inline void quantize_token8(uint4 values, float4 tq, uint32_t qmax, uint32_t (&pair)[4]) {
    const uint32_t w[4] = {values.x, values.y, values.z, values.w};
    const uint32_t cap = (0x4300u + qmax) * 0x10001u;
    uint32_t t[8];
    unsigned short near = 0xFFFF;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        t[2 * k] = __float_as_uint(half_mul_add<false>(w[k], tq.x, tq.y));
        t[2 * k + 1] = __float_as_uint(half_mul_add<true>(w[k], tq.x, tq.y));
        near = min(min(near, (unsigned short)t[2 * k]), (unsigned short)t[2 * k + 1]);
        pair[k] = pk_min(__builtin_amdgcn_perm(t[2 * k + 1], t[2 * k], 0x07060302u), cap);
    }
    if (near < __float_as_uint(tq.z)) {  // rare: a value near a rounding tie: the divide decides
        const uint32_t mt = __float_as_uint(tq.w);
        const float s = __half2float(__ushort_as_half(uint16_t(mt & 0xFFFFu)));
        const float mn = __half2float(__ushort_as_half(uint16_t(mt >> 16)));
        const float top = float(qmax);
        const __half *x = reinterpret_cast<const __half *>(&values);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            uint32_t code[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const float qd = s != 0.0f ? (__half2float(x[2 * k + j]) - mn) / s : 0.0f;  // IEEE fp32 divide
                code[j] = __builtin_amdgcn_cvt_pk_u8_f32(fminf(qd, top), 0u, 0u);            // to nearest even, 0 .. 255
            }
            pair[k] = 0x43004300u + (code[0] | (code[1] << 16));
        }
    }
}

// Sum over the four lanes of one cg (rows 0..3) of x, and the part of it in the rows before this one.
__device__ inline void rows4_sum(uint32_t x, uint32_t &before, uint32_t &total) {
    const int q = (threadIdx.x >> 4) & 3;
    uint32_t a = x, b = x;
    swap_rows16(a, b);  // a: the even row's value, b: the odd row's, in both rows of a pair
    uint32_t c = a + b, d = c;
    swap_rows32(c, d);  // c: the lower pair's sum, d: the upper pair's
    total = c + d;
    before = ((q & 1) ? a : 0u) + ((q & 2) ? c : 0u);
}

// Inclusive prefix sum over the 16 lanes of a row.
__device__ inline uint32_t row_inclusive_scan(uint32_t x) {
    int v = int(x);
    v += dpp_shift0<DPP_ROW_SHR1, 0xF>(v);
    v += dpp_shift0<DPP_ROW_SHR2, 0xF>(v);
    v += dpp_shift0<DPP_ROW_SHR4, 0xF>(v);
    v += dpp_shift0<DPP_ROW_SHR8, 0xF>(v);
    return uint32_t(v);
}

// Quantizes a chunk and, if WRITE, puts its bytes together in lds.image (complete in every
// thread's view on return).  Returns the chunk's size in 16-byte units.  All 256 threads call;
// contains workgroup barriers (one without WRITE).
//
// Bound by vector instructions next to memory (both passes read the input): per value one fused
// multiply-add, half a byte permute, half a clamp, a third of a minimum for the tie test.
template <bool WRITE>
__device__ inline int build_plane_chunk(const ChunkSource &cs, const ChunkInput &in, ChunkLds &lds) {
    const int tau = threadIdx.x, lane = tau & 63, cg = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tau >> 6);
    if (lane < 16) lds.tok[16 * wave + lane] = token_quant(in.mt);
    wave_lds_fence();
    // codes of the lane's 8 channels x 4 tokens: word[j] = channel 8 cg + j, token i in byte i
    uint32_t word[8], mn2[4], mx2[4];
    {
        const int tok0 = 16 * wave + 8 * (q >> 1) + (q & 1);
        uint32_t pair[4][4];
#pragma unroll
        for (int i = 0; i < 4; ++i) quantize_token8(as_fp16(in.raw[i], cs.bf16), lds.tok[tok0 + 2 * i], uint32_t(cs.qmax), pair[i]);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            mn2[k] = pk_min(pk_min(pair[0][k], pair[1][k]), pk_min(pair[2][k], pair[3][k]));
            mx2[k] = pk_max(pk_max(pair[0][k], pair[1][k]), pk_max(pair[2][k], pair[3][k]));
            const uint32_t p01 = __builtin_amdgcn_perm(pair[1][k], pair[0][k], 0x06020400u);  // even ch. tokens 0 1, odd ch. tokens 0 1
            const uint32_t p23 = __builtin_amdgcn_perm(pair[3][k], pair[2][k], 0x06020400u);
            word[2 * k] = __builtin_amdgcn_perm(p23, p01, 0x05040100u);
            word[2 * k + 1] = __builtin_amdgcn_perm(p23, p01, 0x07060302u);
        }
    }
    // 4 x 4 exchange between rows: rows 0, 1 keep channels 0..3, rows 2, 3 channels 4..7; then even
    // rows the lower pair of those, odd rows the upper.  Row q ends with channels 2q, 2q + 1; word
    // 2q + j of row q' goes to: j (from row 0), j + 2 (row 1), j + 4 (row 2), j + 6 (row 3).
#pragma unroll
    for (int j = 0; j < 4; ++j) swap_rows32(word[j], word[j + 4]);
#pragma unroll
    for (int j = 0; j < 2; ++j) swap_rows16(word[j], word[j + 2]), swap_rows16(word[j + 4], word[j + 6]);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        swap_rows32(mn2[k], mn2[k + 2]);
        swap_rows32(mx2[k], mx2[k + 2]);
        mn2[k] = pk_min(mn2[k], mn2[k + 2]);
        mx2[k] = pk_max(mx2[k], mx2[k + 2]);
    }
    swap_rows16(mn2[0], mn2[1]);
    swap_rows16(mx2[0], mx2[1]);
    const uint32_t mn = pk_min(mn2[0], mn2[1]), mx = pk_max(mx2[0], mx2[1]);
    PlaneBits pb[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const uint32_t lo = (mn >> (16 * j)) & 0xFFu, hi = (mx >> (16 * j)) & 0xFFu;
        pb[j] = planes_from_nibbles(word[j] | (word[j + 2] << 4), word[j + 4] | (word[j + 6] << 4), lo, hi);
    }
    const int w0 = pb[0].w, w1 = pb[1].w;
    // Bytes of the lane's packs in the two regions.  Where a pack's planes go: behind those of all
    // packs before it in the list.  Sums carry region E in the low half and region O in the high half.
    const uint32_t e0 = 4u * uint32_t(w0 >> 1), e1 = 4u * uint32_t(w1 >> 1), o0 = 2u * uint32_t(w0 & 1), o1 = 2u * uint32_t(w1 & 1);
    uint32_t off0, off1, total;
    if (cs.pack_order == 0) {
        // group-major (V): wave after wave, channels ascending inside a wave
        const uint32_t mine = (e0 + e1) | ((o0 + o1) << 16);
        uint32_t before, four;
        rows4_sum(mine, before, four);
        const uint32_t inc = row_inclusive_scan(four);
        if (lane == 15) lds.counts[0][wave] = inc;
        __syncthreads();
        const uint4 t = *reinterpret_cast<const uint4 *>(&lds.counts[0][0]);
        total = (t.x + t.y) + (t.z + t.w);
        off0 = inc - four + before + (wave > 0 ? t.x : 0u) + (wave > 1 ? t.y : 0u) + (wave > 2 ? t.z : 0u);
        off1 = off0 + (e0 | (o0 << 16));
    } else {
        // channel-major (K): for every channel the four groups, i.e. the four waves
        lds.counts[wave][lane] = e0 | (o0 << 8) | (e1 << 16) | (o1 << 24);  // sums of four stay below 256
        __syncthreads();
        const uint32_t n0 = lds.counts[0][lane], n1 = lds.counts[1][lane];
        const uint32_t n2 = lds.counts[2][lane], n3 = lds.counts[3][lane];
        const uint32_t all = (n0 + n1) + (n2 + n3);
        const uint32_t earlier = (wave > 0 ? n0 : 0u) + (wave > 1 ? n1 : 0u) + (wave > 2 ? n2 : 0u);
        const uint32_t all0 = (all & 0xFFu) | ((all & 0xFF00u) << 8), all1 = ((all >> 16) & 0xFFu) | ((all >> 8) & 0xFF0000u);
        uint32_t before, four;
        rows4_sum(all0 + all1, before, four);
        const uint32_t inc = row_inclusive_scan(four);
        total = uint32_t(__builtin_amdgcn_readlane(int(inc), 15));
        off0 = inc - four + before;
        off1 = off0 + all0 + (((earlier >> 16) & 0xFFu) | ((earlier >> 8) & 0xFF0000u));
        off0 += (earlier & 0xFFu) | ((earlier & 0xFF00u) << 8);
    }
    const int e_bytes = int(total & 0xFFFFu), used = HEADER + e_bytes + int(total >> 16);
    const int padded = (used + 15) & ~15;
    if constexpr (WRITE) {
        uint8_t *img = lds.image;
        const int d = 8 * cg + 2 * q;
        const uint32_t h0 = uint32_t((w0 << 4) | pb[0].m), h1 = uint32_t((w1 << 4) | pb[1].m);
        if (cs.pack_order == 0) {
            *reinterpret_cast<uint16_t *>(img + 128 * wave + d) = uint16_t(h0 | (h1 << 8));
        } else {
            img[4 * d + wave] = uint8_t(h0);
            img[4 * d + 4 + wave] = uint8_t(h1);
        }
        uint32_t *ea = reinterpret_cast<uint32_t *>(img + HEADER + (off0 & 0xFFFFu));
        uint32_t *eb = reinterpret_cast<uint32_t *>(img + HEADER + (off1 & 0xFFFFu));
        if (w0 >= 2) ea[0] = pb[0].low;
        if (w0 == 4) ea[1] = pb[0].high;
        if (w1 >= 2) eb[0] = pb[1].low;
        if (w1 == 4) eb[1] = pb[1].high;
        if (w0 & 1) *reinterpret_cast<uint16_t *>(img + HEADER + e_bytes + (off0 >> 16)) = uint16_t(pb[0].top);
        if (w1 & 1) *reinterpret_cast<uint16_t *>(img + HEADER + e_bytes + (off1 >> 16)) = uint16_t(pb[1].top);
        if (tau < padded - used) img[used + tau] = 0;
        __syncthreads();
    }
    return padded >> 4;
}

// The finished bytes of a chunk to global memory.
__device__ inline void copy_image(const ChunkLds &lds, int n16, uint8_t *__restrict__ to) {
    static_assert(CHUNK_MAX <= 2 * 256 * 16, "two 16-byte units per thread move a chunk");
    const int tau = threadIdx.x;
    const uint4 *image = reinterpret_cast<const uint4 *>(lds.image);
    uint4 *dst = reinterpret_cast<uint4 *>(to);
    if (tau < n16) dst[tau] = image[tau];
    if (tau + 256 < n16) dst[tau + 256] = image[tau + 256];
}

// Staged path: the input is read and quantized once.
//   quantize  a workgroup holds 16 tokens of all kv-heads in registers: their scales and minimums, then
//             their codes as nibbles (wide chunks: bytes), pack headers and bytes per pack list, into the chunk's slot
//             (the largest chunk's bytes) of the staging area in the workspace
//   assemble  one wave per chunk: turns the codes into planes and puts the chunk's bytes at their place in the arena
// A chunk's place depends on the sizes of all chunks before it, so some second step is needed;
// this one reads the codes (a quarter of the input, and still in the last-level cache: the staging area is a
// few tens of MB) instead of the input.  A round is cut into parts
// that fit the staging area.  The path runs when even the largest chunks fit the arena (worst16 =
// chunks of the round times the largest chunk, checked on the device, where the fill level is), so
// no part can overflow and a round keeps or drops its chunks as a whole; otherwise the first kernel finds the token
// metadata only (nothing where it is given), the second returns at once and the two-pass kernels do the round, and the
// other way round.
__device__ inline bool staged_round(const StagedRound &r, const uint32_t *index) {
    return r.worst16 != 0 && uint64_t(index[r.first_chunk]) + r.worst16 <= r.arena_cap16;
}

// Two-pass path, packs of 16: WRITE false = sizes only, true = bytes at the offsets of the index.
// blockIdx.y: tensor.
template <bool WRITE>
__global__ __launch_bounds__(256) void chunk16_kernel(PackArgs a) {
    const PackTensor &t = a.t[a.first_tensor + blockIdx.y];
    if (staged_round(t.round, t.index)) return;  // the staged path writes this round
    const int cl = blockIdx.x;
    uint8_t *dst = nullptr;
    int room16 = 0;
    if (WRITE) {
        const int64_t e = (t.round.first_chunk + cl) * a.index_words;
        uint32_t o0 = t.index[e], o1 = t.index[e + 1];
        if (o1 == o0) return;  // dropped: the arena was full
        dst = t.arena + size_t(o0) * 16;
        room16 = int(o1 - o0);
    }
    __shared__ ChunkLds lds;
    const int n16 = build_plane_chunk<WRITE>(t.cs, load_chunk_input(t.cs, cl), lds);
    if (WRITE)
        copy_image(lds, min(n16, room16), dst);   // (they are equal; nothing is written behind the chunk's place in any case)
    else if (threadIdx.x == 0)
        t.sizes16[cl] = uint32_t(n16);
}

// Smaller halves of two pairs of fp16 values; the larger ones.  (The builtin forms put a canonicalizing instruction
// in front of every loaded operand.)
__device__ inline uint32_t pk_min_f16(uint32_t x, uint32_t y) {
    uint32_t r;
    asm("v_pk_min_f16 %0, %1, %2" : "=v"(r) : "v"(x), "v"(y));
    return r;
}
__device__ inline uint32_t pk_max_f16(uint32_t x, uint32_t y) {
    uint32_t r;
    asm("v_pk_max_f16 %0, %1, %2" : "=v"(r) : "v"(x), "v"(y));
    return r;
}
// Smallest and largest of three pairs of fp16 values that are no NaN.
__device__ inline uint32_t pk_min3_f16(uint32_t x, uint32_t y, uint32_t z) {
    uint32_t r;
    asm("v_pk_minimum3_f16 %0, %1, %2, %3" : "=v"(r) : "v"(x), "v"(y), "v"(z));
    return r;
}
__device__ inline uint32_t pk_max3_f16(uint32_t x, uint32_t y, uint32_t z) {
    uint32_t r;
    asm("v_pk_maximum3_f16 %0, %1, %2, %3" : "=v"(r) : "v"(x), "v"(y), "v"(z));
    return r;
}
// The two above take the other operand where one is a NaN.  With the mode register's IEEE bit (9) set, as kernels start, a
// signalling NaN would come out as a quiet one instead, and the other operand be lost.
__device__ inline void ieee_mode_off() { __builtin_amdgcn_s_setreg(1 | (9 << 6), 0); }
template <int CTRL>
__device__ inline uint32_t dpp_u32(uint32_t v) {
    return uint32_t(__builtin_amdgcn_update_dpp(0, int(v), CTRL, 0xF, 0xF, true));
}
// Lane i <- lane i ^ 4 of its row (two rotations, each written to half of the lanes).
__device__ inline uint32_t dpp_xor4(uint32_t v) {
    const int up = __builtin_amdgcn_update_dpp(0, int(v), 0x12C, 0xF, 0x5, true);   // banks 0, 2: from the lane four above
    return uint32_t(__builtin_amdgcn_update_dpp(up, int(v), DPP_ROW_ROR4, 0xF, 0xA, true));
}

// Widths of four packs from the ranges of their codes (a byte 0..15 each): bits of the range.
__device__ inline uint32_t width_bytes(uint32_t range) {
    const uint32_t half = (range >> 1) & 0x07070707u;
    const uint32_t w = __builtin_amdgcn_perm(0x04040404u, 0x03030200u, half);   // half = 0: range itself, below
    const uint32_t low = __builtin_amdgcn_perm(0u, 0x00000001u, half);
    return w | (range & low);
}

// Widths of codes up to 127.
__device__ inline uint32_t width_bytes7(uint32_t range) {
    const uint32_t low = width_bytes(range & 0x0F0F0F0Fu), high = width_bytes((range >> 4) & 0x07070707u);
    const uint32_t any = ((high + 0x7F7F7F7Fu) & 0x80808080u) >> 7, mask = (any << 8) - any;   // bytes whose upper half is not 0
    return (low & ~mask) | ((high + 0x04040404u) & mask);
}

// Size of a chunk in 16-byte units from the width sums of its four groups of 16 tokens: a pack of width w takes 2 w bytes
// (w bytes with packs of 8).
constexpr uint32_t UNIT_SHIFT16 = 3, UNIT_SHIFT8 = 4;
__device__ inline uint32_t chunk_units(uint2 sums, uint32_t header16 = HEADER / 16, uint32_t unit_shift = UNIT_SHIFT16) {
    const uint32_t w = (sums.x & 0xFFFFu) + (sums.x >> 16) + (sums.y & 0xFFFFu) + (sums.y >> 16);
    return header16 + ((w + (1u << unit_shift) - 1) >> unit_shift);
}

// Sixteen words of a lane (v[k], k < 8: minimums of tokens 2k, 2k + 1; v[8 + k]: their negated maximums), smallest
// over the 16 lanes of a row: lane i of the row returns word i.
__device__ inline uint32_t row_min_scatter16(const uint32_t (&v)[16]) {
    const int lane = threadIdx.x & 63;
    const bool b3 = lane & 8, b2 = lane & 4, b1 = lane & 2, b0 = lane & 1;
    uint32_t a[8], b[4], c[2];
#pragma unroll
    for (int k = 0; k < 8; ++k) a[k] = pk_min_f16(b3 ? v[8 + k] : v[k], dpp_u32<DPP_ROW_ROR8>(b3 ? v[k] : v[8 + k]));
#pragma unroll
    for (int k = 0; k < 4; ++k) b[k] = pk_min_f16(b2 ? a[4 + k] : a[k], dpp_xor4(b2 ? a[k] : a[4 + k]));
#pragma unroll
    for (int k = 0; k < 2; ++k) c[k] = pk_min_f16(b1 ? b[2 + k] : b[k], dpp_u32<DPP_QUAD_XOR2>(b1 ? b[k] : b[2 + k]));
    return pk_min_f16(b0 ? c[1] : c[0], dpp_u32<DPP_QUAD_XOR1>(b0 ? c[0] : c[1]));
}
// The same over all 64 lanes: lane l returns word 8 (l / 32) + 4 (l / 16 % 2) + l / 4 % 4.
__device__ inline uint32_t wave_min_scatter16(const uint32_t (&v)[16]) {
    const int lane = threadIdx.x & 63;
    const bool b3 = lane & 8, b2 = lane & 4;
    uint32_t a[8], b[4], c[2];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        uint32_t x = v[k], y = v[8 + k];
        swap_rows32(x, y);   // the lower half of the wave keeps word k, the upper half word 8 + k
        a[k] = pk_min_f16(x, y);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        uint32_t x = a[k], y = a[4 + k];
        swap_rows16(x, y);   // even rows keep a[k], odd rows a[4 + k]
        b[k] = pk_min_f16(x, y);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) c[k] = pk_min_f16(b3 ? b[2 + k] : b[k], dpp_u32<DPP_ROW_ROR8>(b3 ? b[k] : b[2 + k]));
    uint32_t r = pk_min_f16(b2 ? c[1] : c[0], dpp_xor4(b2 ? c[0] : c[1]));
    r = pk_min_f16(r, dpp_u32<DPP_QUAD_XOR2>(r));
    return pk_min_f16(r, dpp_u32<DPP_QUAD_XOR1>(r));
}

// token_quant with a closer guard, for quotients below 15.5 (larger ones, over tiny scales, take the divide): the error of
// t against quotient + 1/2 + g is below 0.5 (its rounding) + 0.5 (c; 2^(e-8) for e >= 8) + 0.12 (r) + 0.13 (the
// definition's roundings) units, so g = 2 (+ 2^(e-7)) does: a third fewer divides, which matters here, where all waves
// of a token wait for the slowest.  A token whose scale is so small that codes could pass qmax always divides.
// For quotients up to 127.5 (WIDE) r contributes up to 1 unit and the definition's roundings 1: g = 4 (+ 2^(e-7)).
// r and c come divided by 256 (exactly: they are powers of two away from underflow), for half_mul_add_unit.
template <bool WIDE = false>
__device__ inline float4 token_quant_near(uint32_t mt, float small_scale) {
    const float s = __half2float(__ushort_as_half(uint16_t(mt & 0xFFFFu)));
    const float mn = __half2float(__ushort_as_half(uint16_t(mt >> 16)));
    const float r = s != 0.0f ? __builtin_amdgcn_rcpf(s) : 0.0f;
    const int e = int((__float_as_uint(fmaf(-mn, r, 128.5f)) >> 23) & 0xFFu) - 127;
    uint32_t g = (WIDE ? 4u : 2u) + (e >= 8 ? 2u << min(e - 8, 14) : 0u);
    const float c = fmaf(-mn, r, 128.5f + float(g) * (1.0f / 65536.0f));
    if (s > 0.0f && s < small_scale) g = 1u << 15;
    return make_float4(r * (1.0f / 256.0f), c * (1.0f / 256.0f), __uint_as_float(2u * g), __uint_as_float(mt));
}

// half_mul_add clamped to 0 .. 1: with the operands of token_quant_near t / 256, in [1/2, 1), whose bits 16.. are 0x3F00 + code.
// A NaN becomes 0 (the mode register's DX10_CLAMP bit, set as kernels start) and what is too large 1: their low 16 bits are 0, so both take the divide, whose minimum gives them a code
// in range, and no other token's code sees them.
template <bool HI>
__device__ inline float half_mul_add_unit(uint32_t two_halves, float r, float c) {
    float t;
    if (HI)
        asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[1,0,0] op_sel_hi:[1,0,0] clamp" : "=v"(t) : "v"(two_halves), "v"(r), "v"(c));
    else
        asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel_hi:[1,0,0] clamp" : "=v"(t) : "v"(two_halves), "v"(r), "v"(c));
    return t;
}

// Quantizes four tokens (eight channels each): pair[i][k] = 0x3F00 + code of values 2k (low half) and 2k + 1 of token i.  The tokens that hold a
// value near a rounding tie take the divide, one after the other (every second wave meets one in 16 tokens).
// tok: token_quant_near of the four tokens, every second entry.  cap_all: clamp every value (see QuantRange).
__device__ inline void quantize_quad(const uint4 (&x)[4], const float4 *tok, uint32_t qmax, bool cap_all, uint32_t (&pair)[4][4]) {
    uint64_t near_lanes[4], any = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t w[4] = {x[i].x, x[i].y, x[i].z, x[i].w};
        const float4 tq = tok[2 * i];
        unsigned short near = 0xFFFF;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t t0 = __float_as_uint(half_mul_add_unit<false>(w[k], tq.x, tq.y));
            const uint32_t t1 = __float_as_uint(half_mul_add_unit<true>(w[k], tq.x, tq.y));
            near = min(min(near, (unsigned short)t0), (unsigned short)t1);
            pair[i][k] = __builtin_amdgcn_perm(t1, t0, 0x07060302u);
        }
        near_lanes[i] = __builtin_amdgcn_ballot_w64(near < __float_as_uint(tq.z));
        any |= near_lanes[i];
    }
    if (cap_all) {
        const uint32_t cap = (0x3F00u + qmax) * 0x10001u;
#pragma unroll
        for (int i = 0; i < 16; ++i) pair[i >> 2][i & 3] = pk_min(pair[i >> 2][i & 3], cap);
    }
    if (any == 0) return;
    uint32_t todo = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) todo |= __builtin_amdgcn_inverse_ballot_w64(near_lanes[i]) ? 1u << i : 0u;
    while (todo) {
        const int i = __builtin_ctz(todo);
        const uint32_t mt = __float_as_uint(tok[2 * i].w);
        uint32_t w[4] = {x[0].x, x[0].y, x[0].z, x[0].w};
#pragma unroll
        for (int j = 1; j < 4; ++j) {
            if (i == j) w[0] = x[j].x, w[1] = x[j].y, w[2] = x[j].z, w[3] = x[j].w;
        }
        const float s = __half2float(__ushort_as_half(uint16_t(mt & 0xFFFFu)));
        const float mn = __half2float(__ushort_as_half(uint16_t(mt >> 16)));
        const float top = float(qmax);
        const uint32_t keep = s != 0.0f ? ~0u : 0x3F003F00u;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            __builtin_amdgcn_sched_barrier(0);   // two at a time, in few registers
            const float q0 = (half_lo(w[k]) - mn) / s, q1 = (half_hi(w[k]) - mn) / s;   // IEEE fp32 divide
            const uint32_t c0 = __builtin_amdgcn_cvt_pk_u8_f32(fminf(q0, top), 0u, 0u), c1 = __builtin_amdgcn_cvt_pk_u8_f32(fminf(q1, top), 0u, 0u);
            const uint32_t both = (0x3F003F00u + (c0 | (c1 << 16))) & keep;
#pragma unroll
            for (int j = 0; j < 4; ++j) pair[j][k] = i == j ? both : pair[j][k];
        }
        todo &= todo - 1;
    }
}

// Codes above qmax come out of the multiply-add only where the scale's own rounding to fp16 makes the quotient of the
// largest value pass qmax + 1/2: by less than 2^-11 of it for a scale in fp16's normal range, which reaches there only if
// 1 / rel is within 2^-11 of qmax + 1/2 already (cap_all: the tensor's values are all clamped), by more for a subnormal
// scale (below small_scale the divide and its clamp take the token).  The host's part:
struct QuantRange {
    bool cap_all;
    float small_scale;
};
inline QuantRange quant_range(float rel, int qmax) {
    // the largest quotient is below (s + u) / (rel s) (1 + 2^-20), u half a unit of the scale's last place; with the
    // guard of token_quant_near, its error and the half that rounds it must stay below qmax + 1
    const double room = (qmax + 0.5 - (qmax > 15 ? 8.0 : 4.0) / 65536.0) * double(rel) / (1.0 + 1.0 / (1 << 20)) - 1.0;   // must exceed u / s
    QuantRange q;
    q.cap_all = !(room > 1.0 / 2048.0);
    q.small_scale = q.cap_all ? 0.0f : float(1.0 / (1 << 25) / room * 1.0001);
    return q;
}

// Reads and quantizes the input of a part, once.  A workgroup takes 16 tokens of all kv-heads at a time (an item), a
// wave four heads of them, a lane eight channels (lane % 16) of all 16 tokens: the item's 4 H KB sit in registers while
// the tokens' minimums and maximums are found across the workgroup, so the input is not read a second time.  A token's
// registers are loaded with the next item's as soon as its codes are there.
// HP < 4 (that many kv-heads): the rows of a wave hold 4 / HP token groups.  GIVEN: the token metadata is there
// already (more than 64 kv-heads, or tokens that are repacked, whose order depends on it): the waves are independent.
// Eight codes of a pack make a word, token 2 i in the low half of byte i and token 2 i + 1 in the high half; the words
// of a chunk go out in the order [group][tokens 0..7, 8..15][channel % 8 / 4][channel / 8][channel % 4], which every
// store instruction covers without gaps.
// Bound by memory and arithmetic alike: 8192 chunks of 52 heads of each tensor (268 MB in, 75 MB out) 64 us, about 950 vector
// instructions per wave and item; the token parameters and the quantizer as two kernels that both read the input
// took 38 + 71.  6.8 GB with the assembly below 3330 -> 2280 us, 67 MB 41.6 -> 28.9 (8 heads, 268 MB: 144 -> 104).  Landing half of the next
// item in LDS early, which keeps more loads in flight, gained nothing (2280 -> 2315, 104 -> 114).
// split: few items leave most of the chip idle, and up to 16 waves of one compute unit then share its
// vector units; with split workgroups per item, each reads it all and quantizes a part of the heads (8 x 52 heads, one block:
// flush 19.0 us with one workgroup per item, 16.4 with two, 15.5 with four).
// MIXED: the round is the block that the new tokens complete: its first `held` tokens are read from the tail, the others
// where the caller has them, and those are left in the tail as well, so that no copy has to run first (the appends that
// complete a block of 8 x 52 heads 16.1 -> 14.6 us, of 4 x 1 heads 15.4 -> 11.6).  One item to a workgroup.
// PACK8: a channel's 16 tokens are two packs, whose minimum and maximum are complete after every second quad.  Wide chunks
// (codes up to MOST_STAGED_CODE) keep their codes in bytes, [group][quad][channel % 8 / 4][channel / 8][channel % 4],
// and two header bytes to a pack.  One read of the input instead of three (parameters, sizes, bytes): 8 x 52 heads
// of 8000 tokens 1603 -> 653 us, wide 1670 -> 947; 4 x 8 heads 134 -> 61; a block of 2 x 40 heads, V wide, 44.7 -> 16.1 (eight
// launches before, two now).
// SIZES: token metadata and width sums only, of a whole round that is written in a second pass over the input.
// UNSURE: the round may not be staged, and the kernel finds out first (at run time the question alone cost sure rounds 1 %, a
// block of 8 x 52 heads 16.0 -> 16.4 us).  Not staged, 8000 tokens of 8 x 52 heads take 1025 us, 4096 of 32 55; quantized
// all the same, and thrown away, 1305 and 67.
template <int HP, bool GIVEN, bool STREAM, bool UNSURE, bool MIXED, bool PACK8, bool SIZES = false>
__global__ __launch_bounds__(HP < 4 ? 64 : GIVEN ? 256 : 1024) void quantize16_kernel(PackArgs a) {
    static_assert(!SIZES || (!GIVEN && !UNSURE && !MIXED), "whole rounds that are written in a second pass");
    static_assert(!PACK8 || !UNSURE, "packs of 8 are staged in rounds that fit for sure");
    static_assert(!MIXED || (!GIVEN && !UNSURE), "the block of the tail: rounds that are staged for sure and find their parameters");
    constexpr int MOST_WAVES = HP < 4 ? 1 : GIVEN ? 4 : 16;
    ieee_mode_off();
    __shared__ uint32_t red[2][MOST_WAVES][16];
    __shared__ float4 tok_all[MOST_WAVES][HP < 4 ? 64 : 16];
    __shared__ uint32_t first_sums[PACK8 ? MOST_WAVES : 1][64];
    const int lane = threadIdx.x & 63, cg = lane & 15, row4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = int(blockDim.x >> 6);
    float4 *tok = tok_all[wave];
    const int H = a.t[0].cs.H, B = a.t[0].cs.B;
    const int sets = HP == 4 && GIVEN ? (H + 15) / 16 : 1;   // workgroups that share the heads of an item
    // of a tensor whose round is not staged the first part takes the token metadata of the whole round, if it is not given
    const bool skip_k = UNSURE && !staged_round(a.t[0].round, a.t[0].index), skip_v = UNSURE && !staged_round(a.t[1].round, a.t[1].index);
    const int skip_rows = GIVEN || a.part_row ? 0 : a.round_rows;
    const int items_k = (skip_k ? skip_rows : a.rows) * HP * sets, n_items = items_k + (skip_v ? skip_rows : a.rows) * HP * sets;
    const int token_bytes = int(2 * a.t[0].cs.token_stride);

    struct Item {
        int v, row, blk, b, g0, set;   // tensor, row of the part, block and batch element, first token group, head set
    };
    auto locate = [&](int item) {
        Item m;
        m.v = item >= items_k;
        int rest = item - (m.v ? items_k : 0);
        m.set = 0;
        if (sets > 1) {
            m.set = rest % sets;
            rest /= sets;
        }
        m.row = rest / HP;
        m.g0 = (rest % HP) * (4 / HP);
        const uint32_t full = uint32_t(a.part_row + m.row);
        m.blk = int((uint64_t(full) * a.magic_b) >> 32);
        m.b = int(full) - m.blk * B;
        return m;
    };
    const int head_in_set = HP == 4 ? 4 * wave + row4 : HP == 2 ? row4 & 1 : 0;
    const int group_in_item = HP == 4 ? 0 : HP == 2 ? row4 >> 1 : row4;
    auto head_of = [&](const Item &m) { return head_in_set + 16 * m.set; };
    // storage order of the item's tokens, a byte each (GIVEN, repacked)
    auto order_of = [&](const Item &m) {
        const ChunkSource &cs = a.t[m.v].cs;
        return *reinterpret_cast<const uint4 *>(cs.order + m.b * cs.meta_stride + cs.first_token + int64_t(m.blk) * N +
                                                16 * (m.g0 + group_in_item));
    };
    const bool ordered = GIVEN && a.t[0].cs.order != nullptr;
    auto block_of = [&](const Item &m) {
        const ChunkSource &cs = a.t[m.v].cs;
        return cs.src + m.b * cs.batch_stride + int64_t(m.blk) * N * cs.token_stride;
    };
    // where the lane finds token t: bytes behind the block's first token, the same for all lanes and the lane's own
    auto offset_of = [&](const Item &m, const uint4 &order, int t, int &base) {
        int off = min(head_of(m), H - 1) * (2 * D) + 16 * cg;
        base = (16 * m.g0 + t) * token_bytes;
        if (ordered) {
            const uint32_t w = t < 4 ? order.x : t < 8 ? order.y : t < 12 ? order.z : order.w;
            off += int((w >> (8 * (t & 3))) & 0xFFu) * token_bytes;
            base = 0;
        } else if (HP < 4) {
            off += 16 * group_in_item * token_bytes;
        }
        return off;
    };
    // the block's 64 tokens as a buffer (an empty one if there is no such item: its loads touch no memory)
    auto buffer_of = [&](const Item &m, bool present) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<__half *>(block_of(m)), 0, present ? int(N * token_bytes) : 0, 0x00027000);
    };
    auto load_token = [&](const Item &m, __amdgpu_buffer_rsrc_t buffer, const uint4 &order, int t) {
        int base;
        const int off = offset_of(m, order, t, base);
        typedef uint32_t u32x4n __attribute__((ext_vector_type(4)));
        const u32x4n v = __builtin_amdgcn_raw_buffer_load_b128(buffer, off, base, STREAM ? 2 : 0);   // 2: non-temporal
        return make_uint4(v.x, v.y, v.z, v.w);
    };
    // split > 1: n_items * split workgroups, one item each (those of an item on the same die)
    const int split = HP == 4 && !GIVEN && !skip_k && !skip_v ? a.split : 1;
    int item = split > 1 ? int(blockIdx.x) % n_items : int(blockIdx.x);
    if (item >= n_items) return;
    Item cur = locate(item);
    uint4 raw[16];
    uint4 order = make_uint4(0, 0, 0, 0), order_next = order;   // storage order of the item's tokens, and of the next one's
    // token metadata (GIVEN) of the lane's token cg, of the item and of the next one: ahead of what waits for the order
    auto meta_of = [&](const Item &m) {
        const ChunkSource &cs = a.t[m.v].cs;
        return cs.meta + m.b * cs.meta_stride + cs.first_token + int64_t(m.blk) * N + 16 * (m.g0 + group_in_item);
    };
    uint32_t given = 0;
    if constexpr (GIVEN) given = meta_of(cur)[cg];
    if (ordered) order = order_of(cur), order_next = order_of(locate(min(item + int(gridDim.x), n_items - 1)));
    // MIXED: token t of the lane's group is in the tail already; the lane's place in the tail's token 0
    auto from_tail = [&](int t) { return 16 * (cur.g0 + group_in_item) + t < a.held; };
    auto tail_of = [&](int b, int head) { return a.t[cur.v].tail + (int64_t(b) * N * H + head) * D + 8 * cg; };
    if constexpr (MIXED) {
        const ChunkSource &cs = a.t[cur.v].cs;
        const int head = min(head_of(cur), H - 1);
        const __half *const old = tail_of(cur.b, head);
        const __half *const fresh = cs.src + cur.b * cs.batch_stride + head * D + 8 * cg;   // the first new token
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            const int token = 16 * (cur.g0 + group_in_item) + t;
            raw[t] = load8<STREAM>((from_tail(t) ? old + token * cs.token_stride : fresh + (token - a.held) * cs.token_stride));
        }
    } else {
        const __amdgpu_buffer_rsrc_t buffer = buffer_of(cur, true);
#pragma unroll
        for (int t = 0; t < 16; ++t) raw[t] = load_token(cur, buffer, order, t);
    }
    for (int slot = 0;; slot ^= 1) {
        const PackTensor &pt = a.t[cur.v];
        const ChunkSource &cs = pt.cs;
        const int g = cur.g0 + group_in_item;
        const int next = item + int(gridDim.x);   // (split: past the end)
        const bool more = !MIXED && next < n_items;
        const Item nxt = locate(more ? next : item);
        order = order_next;
        if (ordered) order_next = order_of(locate(min(next + int(gridDim.x), n_items - 1)));
        if (cs.bf16) {
#pragma unroll
            for (int t = 0; t < 16; ++t) raw[t] = as_fp16(raw[t], !MIXED || !from_tail(t));
        }
        if constexpr (GIVEN) {
            const uint32_t now = given;
            given = meta_of(nxt)[cg];
            tok[HP < 4 ? lane : cg] = PACK8 && pt.wide ? token_quant_near<true>(now, pt.small_scale) : token_quant_near(now, pt.small_scale);
        } else {
            uint32_t v[16];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const uint4 p = raw[2 * k], q = raw[2 * k + 1];
                const uint32_t p_mn = pk_min_f16(pk_min_f16(p.x, p.y), pk_min_f16(p.z, p.w)), q_mn = pk_min_f16(pk_min_f16(q.x, q.y), pk_min_f16(q.z, q.w));
                const uint32_t p_mx = pk_max_f16(pk_max_f16(p.x, p.y), pk_max_f16(p.z, p.w)), q_mx = pk_max_f16(pk_max_f16(q.x, q.y), pk_max_f16(q.z, q.w));
                v[k] = pk_min_f16(__builtin_amdgcn_perm(q_mn, p_mn, 0x05040100u), __builtin_amdgcn_perm(q_mn, p_mn, 0x07060302u));
                v[8 + k] = pk_max_f16(__builtin_amdgcn_perm(q_mx, p_mx, 0x05040100u), __builtin_amdgcn_perm(q_mx, p_mx, 0x07060302u)) ^ 0x80008000u;
            }
            const bool skip = cur.v ? skip_v : skip_k;
            if (skip) {
                const __amdgpu_buffer_rsrc_t buffer = buffer_of(nxt, more);
#pragma unroll
                for (int t = 0; t < 16; ++t) raw[t] = load_token(nxt, buffer, order, t);
            }
            // word cg (of v) over the whole item, in every row
            uint32_t word;
            if constexpr (HP == 4) {
                const uint32_t part = wave_min_scatter16(v);
                if ((lane & 3) == 0) red[slot][wave][8 * (row4 >> 1) + 4 * (row4 & 1) + (cg >> 2)] = part;
                if (waves > 1)
                    __syncthreads();   // one per item: the words of the next item go to the other slot
                else
                    wave_lds_fence();
                word = red[slot][min(row4, waves - 1)][cg];
                for (int w = row4 + 4; w < waves; w += 4) word = pk_min_f16(word, red[slot][w][cg]);
                uint32_t x = word, y = word;
                swap_rows16(x, y);
                x = y = pk_min_f16(x, y);
                swap_rows32(x, y);
                word = pk_min_f16(x, y);
            } else {
                word = row_min_scatter16(v);
                if constexpr (HP == 2) {
                    uint32_t x = word, y = word;
                    swap_rows16(x, y);
                    word = pk_min_f16(x, y);
                }
            }
            // lane i: token 2i (i < 8) or 2 (i - 8) + 1; its minimum and negated maximum in one half of the two words
            const uint32_t other = dpp_u32<DPP_ROW_ROR8>(word);
            const uint32_t mnw = cg < 8 ? word : other >> 16, mxw = cg < 8 ? other : word >> 16;
            const int t = 2 * (cg & 7) + (cg >> 3);
            const uint32_t mt = token_meta_word(half_lo(mnw), -half_lo(mxw), pt.rel);
            tok[HP < 4 ? 16 * row4 + t : t] = PACK8 && pt.wide ? token_quant_near<true>(mt, pt.small_scale) : token_quant_near(mt, pt.small_scale);
            if (HP == 4 ? threadIdx.x < 16 : head_in_set == 0) meta_of(cur)[t] = mt;
            if (skip) {
                if (!more) break;
                cur = nxt;
                item = next;
                continue;
            }
            if (split > 1 && ((wave >> 2) & (split - 1)) != int(blockIdx.x) / n_items) return;   // another workgroup's heads
        }
        wave_lds_fence();
        const __amdgpu_buffer_rsrc_t next_buffer = buffer_of(nxt, more);
        const int head = head_of(cur);
        const bool present = head < H;
        if constexpr (MIXED) {
            __half *const to = tail_of(cur.b, head) + 16 * g * cs.token_stride;
#pragma unroll
            for (int t = 0; t < 16; ++t)
                if (present && !from_tail(t)) *reinterpret_cast<uint4 *>(to + t * cs.token_stride) = raw[t];
        }
        const bool wide = PACK8 && pt.wide;
        const uint32_t at = pt.stage_at + uint32_t(cur.row * H + head) * pt.slot + uint32_t(16 * cg);
        uint32_t codes[8], mn2[4], mx2[4];   // codes: channel c, eight tokens as nibbles (wide: four as bytes)
        uint32_t width_sum = 0;              // in bytes: at most 28 each
        // header bytes of the lane's eight packs of group `group`: (width << 4) | minimum, or (wide) the widths and the minimums
        // (codes are at most 15 or 127; the masks keep the header one for any bytes, of which width_bytes makes at most 4)
        auto headers = [&](int group) {
            uint8_t *const to = a.staging + (at + uint32_t(D * group) - uint32_t(8 * cg));
            const uint32_t m_lo = __builtin_amdgcn_perm(mn2[1], mn2[0], 0x06040200u), m_hi = __builtin_amdgcn_perm(mn2[3], mn2[2], 0x06040200u);
            const uint32_t x_lo = __builtin_amdgcn_perm(mx2[1], mx2[0], 0x06040200u), x_hi = __builtin_amdgcn_perm(mx2[3], mx2[2], 0x06040200u);
            if (wide) {
                const uint32_t m0 = m_lo & 0x7F7F7F7Fu, m1 = m_hi & 0x7F7F7F7Fu, w0 = width_bytes7(x_lo - m0), w1 = width_bytes7(x_hi - m1);
                width_sum += w0 + w1;
                if (present && !SIZES) *reinterpret_cast<uint2 *>(to) = make_uint2(w0, w1);
                if (present && !SIZES) *reinterpret_cast<uint2 *>(to + HEADERW / 2) = make_uint2(m0, m1);
            } else {
                const uint32_t m0 = m_lo & 0x0F0F0F0Fu, m1 = m_hi & 0x0F0F0F0Fu, w0 = width_bytes(x_lo - m0), w1 = width_bytes(x_hi - m1);
                width_sum += w0 + w1;
                if (present && !SIZES) *reinterpret_cast<uint2 *>(to) = make_uint2((w0 << 4) | m0, (w1 << 4) | m1);
            }
        };
#pragma unroll
        for (int quad = 0; quad < 4; ++quad) {
            // tokens first, first + 2, .. first + 6
            const int first = 8 * (quad >> 1) + (quad & 1);
            uint4 x[4];
            uint32_t pair[4][4];
            __builtin_amdgcn_sched_barrier(0);   // one quad after the other: the registers do not take more
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = raw[first + 2 * i];
            quantize_quad(x, tok + (HP < 4 ? 16 * row4 : 0) + first, uint32_t(cs.qmax), pt.cap_all, pair);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (!MIXED) raw[first + 2 * i] = load_token(nxt, next_buffer, order, first + 2 * i);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                // (0x3F00 + code is an fp16 number between 1.75 and 1.77)
                const uint32_t lo = pk_min3_f16(pair[0][k], pair[1][k], pair[2][k]), hi = pk_max3_f16(pair[0][k], pair[1][k], pair[2][k]);
                const bool first_quad = PACK8 ? quad % 2 == 0 : quad == 0;
                mn2[k] = first_quad ? pk_min(lo, pair[3][k]) : pk_min3_f16(mn2[k], lo, pair[3][k]);
                mx2[k] = first_quad ? pk_max(hi, pair[3][k]) : pk_max3_f16(mx2[k], hi, pair[3][k]);
                const uint32_t p01 = __builtin_amdgcn_perm(pair[1][k], pair[0][k], 0x06020400u);  // even ch. tokens 0 1, odd ch. tokens 0 1
                const uint32_t p23 = __builtin_amdgcn_perm(pair[3][k], pair[2][k], 0x06020400u);
                const uint32_t e = __builtin_amdgcn_perm(p23, p01, 0x05040100u), o = __builtin_amdgcn_perm(p23, p01, 0x07060302u);
                if ((quad & 1) && !wide)
                    codes[2 * k] |= e << 4, codes[2 * k + 1] |= o << 4;
                else
                    codes[2 * k] = e, codes[2 * k + 1] = o;
            }
            // what the quad leaves is computed here: moved to where it is used, it would keep all pairs in registers
#pragma unroll
            for (int k = 0; k < 4; ++k) consume_here(mn2[k]), consume_here(mx2[k]), consume_here(codes[2 * k]), consume_here(codes[2 * k + 1]);
            if (!SIZES && ((quad & 1) || wide) && present) {
                const uint32_t place = wide ? HEADERW + 2048 * g + 512 * quad : (PACK8 ? HEADER8 : HEADER) + 1024 * g + 512 * (quad >> 1);
                uint8_t *const to = a.staging + (at + place);
                *reinterpret_cast<uint4 *>(to) = make_uint4(codes[0], codes[1], codes[2], codes[3]);
                *reinterpret_cast<uint4 *>(to + 256) = make_uint4(codes[4], codes[5], codes[6], codes[7]);
            }
            if constexpr (PACK8) {
                __builtin_amdgcn_sched_barrier(0);
                if (quad & 1) headers(2 * g + (quad >> 1));
                if (quad == 1) first_sums[wave][lane] = width_sum, width_sum = 0;   // (not in a register: one too many)
            }
        }
        if constexpr (!PACK8) headers(g);
        uint32_t sum = width_sum;
        if (PACK8) sum += first_sums[wave][lane];
        sum += sum >> 16;
        sum = (sum + (sum >> 8)) & 0xFFu;
        sum = row_inclusive_scan(sum);
        if (present && cg == 15) pt.widths[4 * (cur.row * H + head) + g] = uint16_t(sum);
        if (!more) break;
        cur = nxt;
        item = next;
    }
}

// Sum over the 256 threads of a workgroup, in every thread.
__device__ inline uint32_t block_sum(uint32_t v) {
    __shared__ uint32_t wave_sum[4];
    const int inc = wave_inclusive_scan(int(v));
    if ((threadIdx.x & 63) == 63) wave_sum[threadIdx.x >> 6] = uint32_t(inc);
    __syncthreads();
    return wave_sum[0] + wave_sum[1] + wave_sum[2] + wave_sum[3];
}

// A lane's part of a staged chunk: channels 2 lane, 2 lane + 1 in all four token groups.
struct StagedLane {
    uint2 codes[4][2];   // [group][half]: eight codes of the two channels
    uint32_t header[4];  // [group]: two header bytes
    __device__ inline void load(const uint8_t *slot, int lane) {
        typedef uint32_t u32x2n __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            header[g] = *reinterpret_cast<const uint16_t *>(slot + D * g + 2 * lane);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const u32x2n v = __builtin_nontemporal_load(reinterpret_cast<const u32x2n *>(
                    slot + HEADER + 1024 * g + 512 * h + 256 * ((lane >> 1) & 1) + 16 * (lane >> 2) + 8 * (lane & 1)));
                codes[g][h] = make_uint2(v.x, v.y);
            }
        }
    }
};

// The bytes of one chunk from its staged codes, in the wave's LDS image.  channel_major: the pack list of K chunks.
// The image is zero from its last byte in use to the next multiple of 16.
__device__ inline void assemble_chunk(const StagedLane &in, bool channel_major, uint8_t *img) {
    const int lane = threadIdx.x & 63;
    // header bytes by channel, group g in byte g
    const uint32_t h01 = __builtin_amdgcn_perm(in.header[1], in.header[0], 0x05010400u), h23 = __builtin_amdgcn_perm(in.header[3], in.header[2], 0x05010400u);
    const uint32_t hdr[2] = {__builtin_amdgcn_perm(h23, h01, 0x05040100u), __builtin_amdgcn_perm(h23, h01, 0x07060302u)};
    // where the planes of the lane's packs go: words of region E, halfwords of region O before them
    uint32_t e_at[2][4], o_at[2][4], e_words, o_halves;
    const uint32_t e0 = (hdr[0] >> 5) & 0x03030303u, e1 = (hdr[1] >> 5) & 0x03030303u;
    const uint32_t o0 = (hdr[0] >> 4) & 0x01010101u, o1 = (hdr[1] >> 4) & 0x01010101u;
    if (channel_major) {
        const uint32_t ep0 = byte_prefix_sums(e0), ep1 = byte_prefix_sums(e1), op0 = byte_prefix_sums(o0), op1 = byte_prefix_sums(o1);
        const uint32_t both = ((ep0 >> 24) + (ep1 >> 24)) | (((op0 >> 24) + (op1 >> 24)) << 16);
        const uint32_t inc = uint32_t(wave_inclusive_scan(int(both)));
        const uint32_t total = uint32_t(__builtin_amdgcn_readlane(int(inc), 63)), before = inc - both;
        e_words = total & 0xFFFFu, o_halves = total >> 16;
        const uint32_t eb = before & 0xFFFFu, ob = before >> 16;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            e_at[0][g] = eb + (g ? (ep0 >> (8 * (g - 1))) & 0xFFu : 0u);
            o_at[0][g] = ob + (g ? (op0 >> (8 * (g - 1))) & 0xFFu : 0u);
            e_at[1][g] = eb + (ep0 >> 24) + (g ? (ep1 >> (8 * (g - 1))) & 0xFFu : 0u);
            o_at[1][g] = ob + (op0 >> 24) + (g ? (op1 >> (8 * (g - 1))) & 0xFFu : 0u);
        }
    } else {
        const uint32_t es = e0 + e1, os = o0 + o1;
        uint32_t run = 0;   // words | halfwords << 16 of the groups before
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const uint32_t both = ((es >> (8 * g)) & 0xFFu) | (((os >> (8 * g)) & 0xFFu) << 16);
            const uint32_t inc = uint32_t(wave_inclusive_scan(int(both))), before = run + inc - both;
            e_at[0][g] = before & 0xFFFFu, o_at[0][g] = before >> 16;
            e_at[1][g] = e_at[0][g] + ((e0 >> (8 * g)) & 0xFFu);
            o_at[1][g] = o_at[0][g] + ((o0 >> (8 * g)) & 0xFFu);
            run += uint32_t(__builtin_amdgcn_readlane(int(inc), 63));
        }
        e_words = run & 0xFFFFu, o_halves = run >> 16;
    }
    const int used = HEADER + 4 * int(e_words) + 2 * int(o_halves);
    if (lane < 8) *reinterpret_cast<uint16_t *>(img + used + 2 * lane) = 0;
    if (channel_major) {
        *reinterpret_cast<uint2 *>(img + 8 * lane) = make_uint2(hdr[0], hdr[1]);
    } else {
#pragma unroll
        for (int g = 0; g < 4; ++g) *reinterpret_cast<uint16_t *>(img + D * g + 2 * lane) = uint16_t(in.header[g]);
    }
    uint8_t *const e_region = img + HEADER, *const o_region = img + HEADER + 4 * e_words;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const uint32_t hb = (hdr[c] >> (8 * g)) & 0xFFu, w = hb >> 4;
            uint32_t all = hb & 15u;   // the minimum in every nibble: no nibble borrows
            all |= all << 4;
            all = __builtin_amdgcn_perm(0u, all, 0u);
            const uint32_t n0 = (c ? in.codes[g][0].y : in.codes[g][0].x) - all, n1 = (c ? in.codes[g][1].y : in.codes[g][1].x) - all;
            uint32_t *e = reinterpret_cast<uint32_t *>(e_region + 4 * e_at[c][g]);
            if (w >= 2) e[0] = (n0 & 0x33333333u) | ((n1 << 2) & 0xCCCCCCCCu);
            if (w == 4) e[1] = ((n0 >> 2) & 0x33333333u) | (n1 & 0xCCCCCCCCu);
            if (w & 1) {
                // top bit of every code, token i at bit 4 (i % 4) + i / 4
                const uint32_t z = ((n0 >> (w - 1)) & 0x11111111u) | (((n1 >> (w - 1)) & 0x11111111u) << 2);
                *reinterpret_cast<uint16_t *>(o_region + 2 * o_at[c][g]) = uint16_t(z | (z >> 15));
            }
        }
    }
    wave_lds_fence();
}

// New tokens behind the last full block to the start of the raw tail, by the workgroups behind those of the chunks, REST_UNITS
// 16-byte units of a batch element each (a launch less: 4 x 3522 tokens of one head 19.4 -> 15.8 us,
// 2 x 40 heads of 26 blocks and 63 tokens 35.1 -> 33.0; of 58 blocks, 61.5 / 61.6, and more the copy costs what its launch did).
constexpr int REST_UNITS = 512;
__device__ inline void copy_rest(const PackArgs &a, const PackTensor &t, int wg) {
    const int B = t.cs.B, slice = wg / B, b = wg - slice * B;
    const uint4 *src = reinterpret_cast<const uint4 *>(t.rest + b * a.rest_stride);
    uint4 *dst = reinterpret_cast<uint4 *>(t.tail + int64_t(b) * N * t.cs.H * D);
    const int end = min((slice + 1) * REST_UNITS, a.rest_units);
    for (int i = slice * REST_UNITS + int(threadIdx.x); i < end; i += 256)
        dst[i] = load8_as_fp16<true>(reinterpret_cast<const __half *>(src + i), a.rest_bf16);
}

// Storage rank of token `lane` of a block among its 64 sort keys: ascending, equal keys in arrival order.
__device__ inline int storage_rank(int key, int qmax) {
    const int lane = threadIdx.x & 63;
    int rank = 0, base = 0;
    for (int v = 0; v <= qmax; ++v) {
        const uint64_t mask = __builtin_amdgcn_ballot_w64(key == v);
        if (key == v) rank = base + __popcll(mask & ((1ull << lane) - 1ull));
        base += __popcll(mask);
    }
    return rank;
}

// The block's sort keys become its order, and the token metadata of both tensors goes into storage order: one wave, behind the
// last reader of the keys.  scratch: 64 bytes of LDS.
__device__ inline void reorder_block(const PackArgs &a, const ChunkCoord &k, uint8_t *scratch) {
    const int lane = threadIdx.x & 63;
    const ChunkSource &cs = a.t[1].cs;
    const int64_t pos = k.b * cs.meta_stride + cs.first_token + int64_t(k.blk) * N;
    const int key = a.keys[pos + lane];
    const uint32_t km = a.t[0].cs.meta[pos + lane], vm = cs.meta[pos + lane];
    const int rank = storage_rank(key, cs.qmax);
    a.t[0].cs.meta[pos + rank] = km;
    cs.meta[pos + rank] = vm;
    scratch[rank] = uint8_t(lane);
    wave_lds_fence();
    a.keys[pos + lane] = scratch[lane];
    wave_lds_fence();
}

// Chunks of a part from their staged codes to their place, and their index words.  blockIdx.y: tensor; a wave
// takes one chunk, so a workgroup four (waves that walk several, the next one's codes on their way, are slower: 16384 chunks
// 25 us, two per wave 27, three 31).  Every workgroup adds up the sizes of the part's chunks
// before its own by itself (at most 64 KB, in the L2 cache of its die after the first): no launch of a scan in between.
// EXTRAS: there is a rest to copy or a block order to finish (the question alone cost the others 2 %).
template <bool UNSURE, bool EXTRAS>
__global__ __launch_bounds__(256) void assemble16_kernel(PackArgs a) {
    static_assert(!(UNSURE && EXTRAS), "rounds that may not be staged leave both to other kernels");
    __shared__ __attribute__((aligned(16))) uint8_t images[4][CHUNK_MAX + 16];
    const PackTensor &t = a.t[blockIdx.y];
    if (EXTRAS && int(blockIdx.x) >= (a.n + 3) / 4) {
        copy_rest(a, t, int(blockIdx.x) - (a.n + 3) / 4);
        return;
    }
    if (UNSURE && !staged_round(t.round, t.index)) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool paged = a.index_words == 2;  // the placement kernel has set the chunks' index pairs
    const int wg_first = blockIdx.x * 4, cl = wg_first + wave;
    const bool present = cl < a.n;
    uint32_t *const index = t.index + (t.round.first_chunk + a.part_first) * a.index_words;
    const uint2 *widths = reinterpret_cast<const uint2 *>(t.widths);
    // one memory latency for all that the start needs
    StagedLane in;
    if (present) in.load(a.staging + (t.stage_at + uint32_t(cl) * uint32_t(CHUNK_MAX)), lane);
    const uint32_t first = t.index[t.round.first_chunk];
    uint32_t place, units = 0;
    if (paged) {
        const uint2 pair = *reinterpret_cast<const uint2 *>(index + 2 * min(cl, a.n - 1));
        place = pair.x;
        units = present ? pair.y - pair.x : 0;   // 0: dropped, the pool could not cover the call
    } else {
        place = index[0];
        uint32_t before = 0;
#pragma unroll 4
        for (int i = 2 * int(threadIdx.x); i < wg_first; i += 512) {
            const uint4 q = *reinterpret_cast<const uint4 *>(widths + i);
            before += chunk_units(make_uint2(q.x, q.y)) + chunk_units(make_uint2(q.z, q.w));
        }
        // the workgroup's four chunks (the sizes area goes on behind the last one)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t u = chunk_units(widths[wg_first + k]);
            if (k < wave) place += u;
            if (k == wave) units = u;
        }
        place += block_sum(before);
    }
    if (t.round.worst16 == 0 || uint64_t(first) + t.round.worst16 > t.round.arena_cap16) return;   // not a staged round
    if (EXTRAS && a.keys && blockIdx.y == 1 && present) {
        const ChunkCoord k = chunk_coord(t.cs, a.part_first + cl);
        if (k.h == 0) reorder_block(a, k, images[wave]);
    }
    if (!present || units == 0) return;
    if (!paged && lane == 0) index[cl + 1] = place + units;
    uint8_t *const img = images[wave];
    assemble_chunk(in, blockIdx.y == 0, img);
    typedef uint32_t u32x4n __attribute__((ext_vector_type(4)));
    u32x4n *dst = reinterpret_cast<u32x4n *>(t.arena + size_t(place) * 16);
#pragma unroll
    for (int i = 0; i < (CHUNK_MAX / 16 + 63) / 64; ++i) {
        if (lane + 64 * i < int(units)) {
            const uint4 q = *reinterpret_cast<const uint4 *>(img + 16 * (lane + 64 * i));
            __builtin_nontemporal_store(u32x4n{q.x, q.y, q.z, q.w}, dst + lane + 64 * i);
        }
    }
}

// The same for packs of 8 tokens, narrow or wide: consecutive codes of w bits, w bytes to a pack, packs in [group][channel]
// order.  A lane's part: channels 2 lane, 2 lane + 1 in all eight token groups, two packs next to each other in each.
template <bool WIDE>
struct StagedLane8 {
    uint2 codes[8][WIDE ? 2 : 1];   // [group][quad: tokens 0 2 4 6, 1 3 5 7]: bytes; narrow: eight nibbles
    uint32_t width[8], least[8];    // [group]: two header bytes (narrow: both in `width`)
    __device__ inline void load(const uint8_t *slot, int lane) {
        typedef uint32_t u32x2n __attribute__((ext_vector_type(2)));
        const int at = 256 * ((lane >> 1) & 1) + 16 * (lane >> 2) + 8 * (lane & 1);
#pragma unroll
        for (int g = 0; g < 8; ++g) {
            width[g] = *reinterpret_cast<const uint16_t *>(slot + D * g + 2 * lane);
            if (WIDE) least[g] = *reinterpret_cast<const uint16_t *>(slot + HEADERW / 2 + D * g + 2 * lane);
#pragma unroll
            for (int q = 0; q < (WIDE ? 2 : 1); ++q) {
                const u32x2n v = __builtin_nontemporal_load(reinterpret_cast<const u32x2n *>(
                    slot + (WIDE ? HEADERW + 1024 * g + 512 * q : HEADER8 + 512 * g) + at));
                codes[g][q] = make_uint2(v.x, v.y);
            }
        }
    }
};

// Bits `from` .. of the image's payload |= value.  (The image is zero there before; the packs of neighbouring lanes share words.)
__device__ inline void or_bits(uint32_t *payload, uint32_t byte, uint64_t value, int bytes) {
    uint32_t *const at = payload + (byte >> 2);
    const uint32_t shift = 8 * (byte & 3);
    const uint64_t low = value << shift;
    if (bytes > 0) atomicOr(at, uint32_t(low));
    if (int(byte & 3) + bytes > 4) atomicOr(at + 1, uint32_t(low >> 32));
    if (int(byte & 3) + bytes > 8) atomicOr(at + 2, uint32_t((value >> 32) >> (32 - shift)));   // (shift > 0 here)
}

// The bytes of a chunk of packs of 8 from its staged codes, in the wave's LDS image of `units` 16-byte units.
template <bool WIDE>
__device__ inline void assemble_chunk8(const StagedLane8<WIDE> &in, uint32_t units, uint8_t *img) {
    constexpr int HDR = WIDE ? HEADERW : HEADER8;
    const int lane = threadIdx.x & 63;
    uint4 *const words = reinterpret_cast<uint4 *>(img);
    for (uint32_t i = HDR / 16 + lane; i < units; i += 64) words[i] = make_uint4(0, 0, 0, 0);
    wave_lds_fence();
#pragma unroll
    for (int g = 0; g < 8; ++g) {
        *reinterpret_cast<uint16_t *>(img + D * g + 2 * lane) = uint16_t(in.width[g]);
        if (WIDE) *reinterpret_cast<uint16_t *>(img + HEADERW / 2 + D * g + 2 * lane) = uint16_t(in.least[g]);
    }
    uint32_t *const payload = reinterpret_cast<uint32_t *>(img + HDR);
    uint32_t run = 0;   // bytes of the groups before
#pragma unroll
    for (int g2 = 0; g2 < 4; ++g2) {
        // the widths of two groups in the halves of a word: at most 1024 bytes each
        uint32_t w[2][2], both = 0;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint32_t h = in.width[2 * g2 + i];
            w[i][0] = WIDE ? h & 0xFFu : (h >> 4) & 0xFu, w[i][1] = WIDE ? h >> 8 : h >> 12;
            both |= (w[i][0] + w[i][1]) << (16 * i);
        }
        const uint32_t inc = uint32_t(wave_inclusive_scan(int(both))), before = inc - both;
        const uint32_t total = uint32_t(__builtin_amdgcn_readlane(int(inc), 63));
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int g = 2 * g2 + i;
            const uint32_t at = run + (i ? (total & 0xFFFFu) + (before >> 16) : before & 0xFFFFu);
            uint64_t bits[2];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const uint32_t wc = w[i][c];
                uint32_t p0, p1;   // halfwords: codes 2 j and 2 j + 1 of the pack, j = 0, 1 and 2, 3
                if constexpr (WIDE) {
                    uint32_t all = (in.least[g] >> (8 * c)) & 0xFFu;
                    all = __builtin_amdgcn_perm(0u, all, 0u);   // the minimum in every byte: no byte borrows
                    const uint32_t e = (c ? in.codes[g][0].y : in.codes[g][0].x) - all, o = (c ? in.codes[g][WIDE].y : in.codes[g][WIDE].x) - all;
                    // (codes of up to 7 bits: a pair stays in its halfword)
                    p0 = __builtin_amdgcn_perm(0u, e, 0x0C010C00u) | (__builtin_amdgcn_perm(0u, o, 0x0C010C00u) << wc);
                    p1 = __builtin_amdgcn_perm(0u, e, 0x0C030C02u) | (__builtin_amdgcn_perm(0u, o, 0x0C030C02u) << wc);
                    const uint32_t h0 = (p0 & 0xFFFFu) | ((p0 >> 16) << (2 * wc)), h1 = (p1 & 0xFFFFu) | ((p1 >> 16) << (2 * wc));
                    bits[c] = uint64_t(h0) | (uint64_t(h1) << (4 * wc));
                } else {
                    uint32_t all = (in.width[g] >> (8 * c)) & 0xFu;
                    all |= all << 4;
                    all = __builtin_amdgcn_perm(0u, all, 0u);
                    const uint32_t n = (c ? in.codes[g][0].y : in.codes[g][0].x) - all;
                    p0 = (n & 0x0F0F0F0Fu) | (((n >> 4) & 0x0F0F0F0Fu) << wc);           // bytes of 2 w bits
                    p1 = (p0 & 0x00FF00FFu) | (((p0 >> 8) & 0x00FF00FFu) << (2 * wc));   // halfwords of 4 w bits
                    bits[c] = (p1 & 0xFFFFu) | ((p1 >> 16) << (4 * wc));
                }
            }
            if constexpr (WIDE) {
                or_bits(payload, at, bits[0], int(w[i][0]));
                or_bits(payload, at + w[i][0], bits[1], int(w[i][1]));
            } else {
                or_bits(payload, at, bits[0] | (bits[1] << (8 * w[i][0])), int(w[i][0] + w[i][1]));
            }
        }
        run += (total & 0xFFFFu) + (total >> 16);
    }
    wave_lds_fence();
}

// assemble16_kernel for packs of 8.  LDS: an image of a slot's size to each wave.
__global__ __launch_bounds__(256) void assemble8_kernel(PackArgs a) {
    extern __shared__ __attribute__((aligned(16))) uint8_t images8[];
    const PackTensor &t = a.t[blockIdx.y];
    if (int(blockIdx.x) >= (a.n + 3) / 4) {
        copy_rest(a, t, int(blockIdx.x) - (a.n + 3) / 4);
        return;
    }
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wg_first = blockIdx.x * 4, cl = wg_first + wave;
    const bool present = cl < a.n;
    const uint8_t *const slot = a.staging + (t.stage_at + uint32_t(min(cl, a.n - 1)) * t.slot);
    uint32_t place = 0, units = 0;
    auto find_place = [&]() {
        uint32_t *const index = t.index + (t.round.first_chunk + a.part_first) * a.index_words;
        const uint2 *widths = reinterpret_cast<const uint2 *>(t.widths);
        if (a.index_words == 2) {   // paged: the placement kernel has set the chunks' index pairs
            const uint2 pair = *reinterpret_cast<const uint2 *>(index + 2 * min(cl, a.n - 1));
            place = pair.x;
            units = present ? pair.y - pair.x : 0;   // 0: dropped, the pool could not cover the call
            return;
        }
        place = index[0];
        uint32_t before = 0;
#pragma unroll 4
        for (int i = 2 * int(threadIdx.x); i < wg_first; i += 512) {
            const uint4 q = *reinterpret_cast<const uint4 *>(widths + i);
            before += chunk_units(make_uint2(q.x, q.y), t.header16, UNIT_SHIFT8) + chunk_units(make_uint2(q.z, q.w), t.header16, UNIT_SHIFT8);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t u = chunk_units(widths[wg_first + k], t.header16, UNIT_SHIFT8);
            if (k < wave) place += u;
            if (k == wave) units = present ? u : 0;
        }
        place += block_sum(before);
        if (present && lane == 0) index[cl + 1] = place + units;
    };
    uint8_t *const img = images8 + wave * t.slot;
    if (a.keys && blockIdx.y == 1 && present) {
        const ChunkCoord k = chunk_coord(t.cs, a.part_first + cl);
        if (k.h == 0) reorder_block(a, k, img);
    }
    if (t.wide) {
        StagedLane8<true> in;
        in.load(slot, lane);
        find_place();
        if (units == 0) return;
        assemble_chunk8<true>(in, units, img);
    } else {
        StagedLane8<false> in;
        in.load(slot, lane);
        find_place();
        if (units == 0) return;
        assemble_chunk8<false>(in, units, img);
    }
    typedef uint32_t u32x4n __attribute__((ext_vector_type(4)));
    u32x4n *dst = reinterpret_cast<u32x4n *>(t.arena + size_t(place) * 16);
    for (uint32_t i = lane; i < units; i += 64) {
        const uint4 q = *reinterpret_cast<const uint4 *>(img + 16 * i);
        __builtin_nontemporal_store(u32x4n{q.x, q.y, q.z, q.w}, dst + i);
    }
}

// Two-pass rounds, one workgroup per tensor (blockIdx.x): index[first+i+1] = index[first] + sum_{j<=i} sizes16[j].
// If the new chunks do not fit, all of them get size 0 and the flag is set.
// Wave w owns a run of `per` consecutive sizes (a multiple of 256) and walks it 256 at a time,
// four per lane, so loads and stores of a wave cover consecutive memory.
__global__ __launch_bounds__(1024) void scan_offsets_kernel(PackArgs a) {
    const PackTensor &t = a.t[a.first_tensor + blockIdx.x];
    const uint32_t *sizes16 = t.sizes16;
    uint32_t *index = t.index;
    const int64_t first_chunk = t.round.first_chunk;
    const int n = a.n;
    if (staged_round(t.round, index)) return;  // the staged path writes this round
    __shared__ uint32_t wsum[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int per = ((n + 15) / 16 + 255) & ~255;
    const int lo = min(wave * per, n), hi = min(lo + per, n);
    // sizes lo + 256 r + 4 lane .. + 3 (sizes16 is 256-byte aligned and its area a multiple of 16 bytes)
    const uint2 *widths = reinterpret_cast<const uint2 *>(t.widths);   // or the width sums, where the round has those
    auto load4 = [&](int r) {
        const int i = lo + 256 * r + 4 * lane;
        uint4 q = make_uint4(0, 0, 0, 0);
        if (widths) {
            if (i < hi) {   // (the area goes on behind the last one)
                const uint4 x = *reinterpret_cast<const uint4 *>(widths + i), y = *reinterpret_cast<const uint4 *>(widths + i + 2);
                q.x = chunk_units(make_uint2(x.x, x.y), t.header16, t.unit_shift), q.y = chunk_units(make_uint2(x.z, x.w), t.header16, t.unit_shift);
                q.z = chunk_units(make_uint2(y.x, y.y), t.header16, t.unit_shift), q.w = chunk_units(make_uint2(y.z, y.w), t.header16, t.unit_shift);
            }
        } else
            q = i < hi ? *reinterpret_cast<const uint4 *>(sizes16 + i) : make_uint4(0, 0, 0, 0);
        if (i + 1 >= hi) q.y = 0;
        if (i + 2 >= hi) q.z = 0;
        if (i + 3 >= hi) q.w = 0;
        return q;
    };
    const int rounds = (hi - lo + 255) / 256;
    // the first four rounds (all of them for up to 16384 chunks) go out at once and stay in registers
    uint4 held[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) held[r] = load4(r);
    const uint32_t start = index[first_chunk];
    uint32_t local = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) local += held[r].x + held[r].y + held[r].z + held[r].w;
    for (int r = 4; r < rounds; ++r) {
        const uint4 q = load4(r);
        local += q.x + q.y + q.z + q.w;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) local += __shfl_xor(local, o);
    if (lane == 0) wsum[wave] = local;
    __syncthreads();
    uint32_t run = start, total = 0;
    for (int k = 0; k < 16; ++k) {
        if (k < wave) run += wsum[k];
        total += wsum[k];
    }
    const bool fits = uint64_t(start) + total <= t.arena_cap16;
    if (!fits && tid == 0) t.status[0] = 1;
    auto place = [&](int r, uint4 q) {
        const uint32_t mine = q.x + q.y + q.z + q.w;
        uint32_t inc = mine;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t v = __shfl_up(inc, o);
            if (lane >= o) inc += v;
        }
        const int i = lo + 256 * r + 4 * lane;
        uint32_t at = run + inc - mine;
        const uint32_t ends[4] = {at + q.x, at + q.x + q.y, at + q.x + q.y + q.z, at + mine};
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (i + k < hi) index[first_chunk + i + k + 1] = fits ? ends[k] : start;
        run += __shfl(inc, 63);
    };
#pragma unroll
    for (int r = 0; r < 4; ++r)
        if (r < rounds) place(r, held[r]);
    for (int r = 4; r < rounds; ++r) place(r, load4(r));
}

// Paged arena: places the n new chunks of one tensor (sizes16: their sizes in 16-byte units;
// overwritten with their exclusive prefix sums) in chunk order.  A chunk goes right behind the
// previous one while it still fits into the tensor's newest page, else to the start of a fresh
// page, so no chunk crosses a page boundary; positions count 16-byte units from the start of the
// pool.  The fresh pages come off the pool's stack, all of them with one atomic update of its
// height.  If the pool (or the tensor's page list) cannot take them, nothing is taken, every
// chunk of the call is dropped (start = end) and the flag is set, as with a full contiguous arena.
//
// One workgroup.  The rule is sequential in the fill level only, so the work is split: (1) prefix
// sums S of the sizes; (2) for every chunk j, in parallel, how many chunks a page holds that
// starts with j (two pointers over S); (3) one thread follows that chain from the first chunk
// that does not fit the newest page -- one LDS step per fresh page, not per chunk -- and marks
// the chunks that start a page; (4) in parallel again, every chunk finds its page (a count of the
// marks before it) and its offset inside it (S[j] - S[page start]).
__global__ __launch_bounds__(1024) void place_chunks_kernel(PackArgs a, int n_tensors) {
    uint32_t *const pool_state = a.pool_state;
    const int n = a.n;
    // bit 7: the chunk starts a fresh page; bits 0..6: chunks that fit a page starting here, minus 1
    // (a chunk is at least 512 bytes, so a page holds at most 128)
    __shared__ uint8_t step[MAX_NEW_CHUNKS];
    __shared__ uint32_t wave_a[16], wave_b[16];
    __shared__ uint32_t sh_total, sh_top, sh_ok;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int per = (n + 1023) / 1024;
    const int lo = min(tid * per, n), hi = min(lo + per, n);
    constexpr uint32_t P = PAGE16;
    constexpr int WAVES = 16, ENTRIES = 128;
    __shared__ uint32_t seg_exit[WAVES][ENTRIES];
    __shared__ uint16_t seg_pages[WAVES][ENTRIES];
    __shared__ uint32_t seg_entry[WAVES];

    // the tensors one after the other: V's fresh pages are the ones below K's on the pool's stack
    for (int tensor = 0; tensor < n_tensors; ++tensor) {
    const PackTensor &pt = a.t[a.first_tensor + tensor];
    uint32_t *const sizes16 = pt.sizes16;
    uint32_t *const index2 = pt.index;
    const int64_t first_chunk = pt.round.first_chunk;
    uint32_t *const page_list = pt.page_list;
    const int64_t max_pages = pt.max_pages;
    const uint2 *widths = reinterpret_cast<const uint2 *>(pt.widths);
    if (tensor) __syncthreads();  // the shared arrays and the pool's state of the tensor before are done with

    // (1) exclusive prefix sums, in place (width sums: both tensors use the same sizes, one after the other)
    uint32_t local = 0;
    for (int i = lo; i < hi; ++i) {
        if (widths) sizes16[i] = chunk_units(widths[i], pt.header16, pt.unit_shift);
        local += sizes16[i];
    }
    uint32_t inc = local;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t v = __shfl_up(inc, o);
        if (lane >= o) inc += v;
    }
    if (lane == 63) wave_a[wave] = inc;
    __syncthreads();
    uint32_t run = inc - local;
    for (int k = 0; k < wave; ++k) run += wave_a[k];
    if (tid == 1023) sh_total = run + local;
    for (int i = lo; i < hi; ++i) {
        const uint32_t sz = sizes16[i];
        sizes16[i] = run;
        run += sz;
    }
    __syncthreads();
    const uint32_t total = sh_total;
    auto S = [&](int i) -> uint32_t { return i < n ? sizes16[i] : total; };

    // (2) chunks per page for a page that starts with chunk j
    {
        int k = lo;
        for (int j = lo; j < hi; ++j) {
            k = max(k, j + 1);
            const uint32_t limit = S(j) + P;
            while (k < n && S(k + 1) <= limit) ++k;
            step[j] = uint8_t(k - j - 1);
        }
    }
    __syncthreads();

    // (3) the chain of page starts, and the pages for it.  Following the chain is one dependent LDS
    // read per fresh page; with many chunks it is cut into sixteen segments, one per wave: a chain
    // enters a segment within its first 128 chunks (a page holds no more), so every wave follows
    // the chain from each of these 128 possible entries to the segment's end (lanes in parallel)
    // and notes where it leaves and how many pages it starts; thread 0 then hops through the
    // sixteen tables, and every wave marks its own segment from its true entry.
    const int seg = (n + WAVES - 1) / WAVES;
    const bool segmented = seg >= ENTRIES;
    const int seg_a = min(wave * seg, n), seg_e = min(seg_a + seg, n);
    if (segmented) {
        for (int c = lane; c < ENTRIES; c += 64) {
            int j = seg_a + c;
            uint32_t pages = 0;
            while (j < seg_e) {
                ++pages;
                j += int(step[j]) + 1;
            }
            seg_exit[wave][c] = uint32_t(j);
            seg_pages[wave][c] = uint16_t(pages);
        }
    }
    __syncthreads();
    const uint32_t held = page_list[0];
    const uint32_t fill0 = held ? page_list[1] : P;  // no page yet: like a full one
    if (tid == 0) {
        int j = 0;
        while (j < n && fill0 + S(j + 1) <= P) ++j;  // these still go into the newest page
        uint32_t need = 0;
        for (int w = 0; w < (segmented ? WAVES : 1); ++w) {
            const int a = segmented ? min(w * seg, n) : 0, e = segmented ? min(a + seg, n) : n;
            seg_entry[w] = uint32_t(j);
            if (segmented && j < e && j - a < ENTRIES) {
                need += seg_pages[w][j - a];
                j = int(seg_exit[w][j - a]);
            } else {
                while (j < e) {  // few chunks, or an entry the tables do not cover: step by step
                    ++need;
                    j += int(step[j]) + 1;
                }
            }
        }
        uint32_t ok = held + need <= uint64_t(max_pages), top = 0;
        if (ok && need) {
            uint32_t old = __atomic_load_n(&pool_state[0], __ATOMIC_RELAXED);
            while (true) {
                if (old < need) {
                    ok = 0;
                    break;
                }
                const uint32_t seen = atomicCAS(&pool_state[0], old, old - need);
                if (seen == old) break;
                old = seen;
            }
            top = old;
        }
        sh_ok = ok;
        sh_top = top;
    }
    __syncthreads();
    if (sh_ok && lane == 0 && (segmented || wave == 0)) {  // mark the page starts of this wave's part
        int j = int(seg_entry[wave]);
        const int e = segmented ? seg_e : n;
        while (j < e) {
            const uint32_t c = step[j];
            step[j] = uint8_t(c | 0x80u);
            j += int(c) + 1;
        }
    }
    __syncthreads();
    if (!sh_ok) {
        if (tid == 0) pt.status[0] = 1;
        for (int i = lo; i < hi; ++i) {
            index2[2 * (first_chunk + i)] = 0;
            index2[2 * (first_chunk + i) + 1] = 0;
        }
        continue;
    }
    const uint32_t top = sh_top;

    // (4) marks before this thread's slice, and the last marked chunk before it (+1; 0 = none)
    uint32_t marks = 0, last = 0;
    for (int j = lo; j < hi; ++j)
        if (step[j] & 0x80u) ++marks, last = uint32_t(j) + 1;
    uint32_t marks_inc = marks, last_inc = last;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t a = __shfl_up(marks_inc, o), b = __shfl_up(last_inc, o);
        if (lane >= o) marks_inc += a, last_inc = max(last_inc, b);
    }
    if (lane == 63) wave_a[wave] = marks_inc, wave_b[wave] = last_inc;
    __syncthreads();
    uint32_t ord = marks_inc - marks;      // fresh pages started before the slice
    uint32_t start_j = __shfl_up(last_inc, 1);
    if (lane == 0) start_j = 0;
    for (int k = 0; k < wave; ++k) ord += wave_a[k], start_j = max(start_j, wave_b[k]);
    const uint32_t newest = held ? page_list[1 + held] : 0u;
    uint32_t page = 0, page_s = 0;  // the page the slice starts in, S of the chunk that starts it
    if (start_j) page = pool_state[top - (ord - 1)], page_s = S(int(start_j) - 1);
    for (int j = lo; j < hi; ++j) {
        if (step[j] & 0x80u) {
            page = pool_state[top - ord];  // stack entry top - 1 - ord sits at word top - ord
            page_list[2 + held + ord] = page;
            ++ord;
            page_s = S(j);
        }
        const uint32_t at = ord ? page * P + (S(j) - page_s) : newest * P + fill0 + S(j);
        index2[2 * (first_chunk + j)] = at;
        index2[2 * (first_chunk + j) + 1] = at + (S(j + 1) - S(j));
    }
    if (tid == 1023) {
        const uint32_t all_last = max(last_inc, start_j);  // with the waves before: the last marked chunk of all
        uint32_t l = all_last;
        for (int k = 0; k < 16; ++k) l = max(l, wave_b[k]);
        page_list[0] = held + ord;
        page_list[1] = l ? total - S(int(l) - 1) : fill0 + total;
    }
    }
}

// The same for rounds of up to PLACE_SMALL_CHUNKS chunks per tensor: sizes and prefix sums stay in LDS, the
// two tensors run side by side in half a workgroup each, and the pages of both are taken in one step (K's
// first).  The chain of page starts is followed as in place_chunks_kernel, the eight waves of a tensor a segment each.
// This kernel is one chain of latencies: 2 x 1504 chunks took 14.5 us with one thread following the chain and ends
// of pages found by stepping through the chunks, 11.8 with this (marks sent ahead by doubled jumps: 16.7).
constexpr int PLACE_SMALL_CHUNKS = 8192;
__global__ __launch_bounds__(1024) void place_small_kernel(PackArgs a) {
    constexpr int T = 512;
    constexpr uint32_t P = PAGE16;
    __shared__ uint32_t sums[2][PLACE_SMALL_CHUNKS + 1];
    __shared__ uint16_t nexts[2][PLACE_SMALL_CHUNKS];       // where the page behind one that starts with chunk j starts
    __shared__ uint8_t marks_of[2][PLACE_SMALL_CHUNKS];     // the chunk starts a fresh page
    constexpr int WAVES = T / 64, ENTRIES = 128;            // a page holds at most 128 chunks (of 512 bytes)
    __shared__ uint16_t seg_exit[2][WAVES][ENTRIES];
    __shared__ uint16_t first_start[2];
    __shared__ uint32_t wave_a[2][T / 64], wave_b[2][T / 64];
    __shared__ uint32_t sh_need[2], sh_top[2], sh_ok[2];
    const int half = __builtin_amdgcn_readfirstlane(threadIdx.x / T);
    const int tid = threadIdx.x % T, lane = tid & 63, wave = tid >> 6, n = a.n;
    const PackTensor &t = a.t[half];
    uint32_t *const S = sums[half];
    uint16_t *const next = nexts[half];
    uint8_t *const mark = marks_of[half];
    const uint32_t held = t.page_list[0], newest_fill = t.page_list[1];
    uint32_t old = 0, held_of[2] = {0, 0};   // thread 0: what the pages are taken from, long before they are
    if (threadIdx.x == 0) {
        old = __atomic_load_n(&a.pool_state[0], __ATOMIC_RELAXED);
        held_of[0] = a.t[0].page_list[0], held_of[1] = a.t[1].page_list[0];
    }
#pragma unroll 4
    for (int i = tid; i < n; i += T) {
        S[i] = t.widths ? chunk_units(reinterpret_cast<const uint2 *>(t.widths)[i], t.header16, t.unit_shift) : t.sizes16[i];
        mark[i] = 0;
    }
    const uint32_t newest = held ? t.page_list[1 + held] : 0u;
    const uint32_t fill0 = held ? newest_fill : P;  // no page yet: like a full one
    __syncthreads();
    // exclusive prefix sums, S[n] = total
    const int per = (n + T - 1) / T, lo = min(tid * per, n), hi = min(lo + per, n);
    uint32_t local = 0;
    for (int i = lo; i < hi; ++i) local += S[i];
    const uint32_t inc = uint32_t(wave_inclusive_scan(int(local)));
    if (lane == 63) wave_a[half][wave] = inc;
    __syncthreads();
    uint32_t run = inc - local;
    for (int k = 0; k < wave; ++k) run += wave_a[half][k];
    for (int i = lo; i < hi; ++i) {
        const uint32_t sz = S[i];
        S[i] = run;
        run += sz;
    }
    if (tid == T - 1) S[n] = run;
    __syncthreads();
    // the largest k with S[k] <= limit and below <= k <= min(n, j + 128), four searches at a time
    for (int j0 = tid; j0 < n; j0 += 4 * T) {
        int below[4], above[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) below[i] = min(j0 + T * i + 1, n), above[i] = min(j0 + T * i + ENTRIES, n);
#pragma unroll
        for (int r = 0; r < 7; ++r) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int mid = (below[i] + above[i] + 1) >> 1;   // (equal ends stay as they are)
                if (S[mid] <= S[min(j0 + T * i, n)] + P) below[i] = mid; else above[i] = max(mid - 1, below[i]);
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (j0 + T * i < n) next[j0 + T * i] = uint16_t(below[i]);
    }
    if (wave == WAVES - 1) {
        // chunks 0 .. j - 1 still go into the newest page: the largest j with fill0 + S[j] <= P
        int below = 0, above = min(n, ENTRIES);
        while (above > below) {
            const int mid = (below + above + 1) >> 1;
            if (fill0 + S[mid] <= P) below = mid; else above = mid - 1;
        }
        if (lane == 0) first_start[half] = uint16_t(below);
    }
    __syncthreads();
    // the chain from every chunk a segment may be entered at to where it leaves the segment, lanes in parallel
    const int seg = (n + WAVES - 1) / WAVES, seg_a = min(wave * seg, n), seg_e = min(seg_a + seg, n);
    {
        int j[2] = {seg_a + lane, seg_a + lane + 64};
        while (__builtin_amdgcn_ballot_w64(min(j[0], j[1]) < seg_e)) {
#pragma unroll
            for (int i = 0; i < 2; ++i)
                if (j[i] < seg_e) j[i] = next[j[i]];
        }
        seg_exit[half][wave][lane] = uint16_t(j[0]), seg_exit[half][wave][lane + 64] = uint16_t(j[1]);
    }
    __syncthreads();
    // this wave's entry, through the segments before it, and its marks
    {
        int j = first_start[half];
        for (int w = 0; w < wave; ++w) {
            const int wa = min(w * seg, n), we = min(wa + seg, n);
            if (j < we) j = seg_exit[half][w][j - wa];
        }
        while (j < seg_e) {
            if (lane == 0) mark[j] = 1;
            j = next[j];
        }
    }
    __syncthreads();
    // page starts before this thread's slice, and the last of them (+1; 0 = none)
    uint32_t marks = 0, last = 0;
    for (int j = lo; j < hi; ++j)
        if (mark[j]) ++marks, last = uint32_t(j) + 1;
    const uint32_t marks_inc = uint32_t(wave_inclusive_scan(int(marks)));
    uint32_t last_inc = last;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(last_inc, o);
        if (lane >= o) last_inc = max(last_inc, y);
    }
    if (lane == 63) wave_a[half][wave] = marks_inc, wave_b[half][wave] = last_inc;
    __syncthreads();
    uint32_t ord = marks_inc - marks, start_j = __shfl_up(last_inc, 1);
    if (lane == 0) start_j = 0;
    for (int k = 0; k < wave; ++k) ord += wave_a[half][k], start_j = max(start_j, wave_b[half][k]);
    if (tid == T - 1) sh_need[half] = ord + marks;
    __syncthreads();
    if (threadIdx.x == 0) {
        bool ok[2];
        uint32_t top[2];
        while (true) {  // K's pages come first; a tensor the pool or its list cannot cover takes none
            uint32_t left = old;
            for (int v = 0; v < 2; ++v) {
                const uint32_t need = sh_need[v];
                ok[v] = held_of[v] + need <= uint64_t(a.t[v].max_pages) && need <= left;
                top[v] = left;
                if (ok[v]) left -= need;
            }
            if (left == old) break;
            const uint32_t seen = atomicCAS(&a.pool_state[0], old, left);
            if (seen == old) break;
            old = seen;
        }
        for (int v = 0; v < 2; ++v) sh_ok[v] = ok[v], sh_top[v] = top[v];
    }
    __syncthreads();
    uint32_t *const index2 = t.index + 2 * t.round.first_chunk;
    const uint32_t top = sh_top[half];
    if (!sh_ok[half]) {
        if (tid == 0) t.status[0] = 1;
        for (int i = tid; i < 2 * n; i += T) index2[i] = 0;
        return;
    }
    uint32_t page = 0, page_s = 0;  // the page the slice starts in, S of the chunk that starts it
    if (start_j) page = a.pool_state[top - (ord - 1)], page_s = S[start_j - 1];
    for (int j = lo; j < hi; ++j) {
        if (mark[j]) {
            page = a.pool_state[top - ord];  // stack entry top - 1 - ord sits at word top - ord
            t.page_list[2 + held + ord] = page;
            ++ord;
            page_s = S[j];
        }
        const uint32_t at = ord ? page * P + (S[j] - page_s) : newest * P + fill0 + S[j];
        index2[2 * j] = at;
        index2[2 * j + 1] = at + (S[j + 1] - S[j]);
    }
    if (tid == T - 1) {
        uint32_t l = max(last_inc, start_j);  // the last page start of all
        for (int k = 0; k < T / 64; ++k) l = max(l, wave_b[half][k]);
        t.page_list[0] = held + ord;
        t.page_list[1] = l ? S[n] - S[l - 1] : fill0 + S[n];
    }
}

// Pool of n free pages: the stack holds n - 1 down to 0, so page 0 is handed out first.
__global__ void pool_init_kernel(uint32_t *state, int64_t n_pages) {
    const int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
    if (i == 0) state[0] = uint32_t(n_pages);
    if (i < n_pages) state[1 + i] = uint32_t(n_pages - 1 - i);
}

// What a new or released cache starts from.
__device__ inline void init_words(uint32_t *status, uint32_t *k_index, uint32_t *v_index) {
    if (threadIdx.x < 64) status[threadIdx.x] = 0;
    if (threadIdx.x == 0) k_index[0] = v_index[0] = 0;
}

// Pushes the pages of both tensors back onto the pool's stack (the newest page of a list first,
// so a cache that refills an otherwise idle pool gets its pages in the same order again) and
// empties the lists; status and index start anew with it.  One wave.
__global__ __launch_bounds__(64) void release_pages_kernel(uint32_t *k_list, uint32_t *v_list, uint32_t *pool_state,
                                                           int64_t n_pages, uint32_t *status, uint32_t *k_index, uint32_t *v_index) {
    const int lane = threadIdx.x;
    init_words(status, k_index, v_index);
    for (int t = 0; t < 2; ++t) {
        uint32_t *list = t ? v_list : k_list;
        const uint32_t cnt = list[0];
        uint32_t base = 0;
        if (lane == 0 && cnt) base = atomicAdd(&pool_state[0], cnt);
        base = __builtin_amdgcn_readfirstlane(base);
        for (uint32_t i = lane; i < cnt; i += 64)
            if (int64_t(base) + i < n_pages) pool_state[1 + base + i] = list[2 + cnt - 1 - i];
    }
    __syncthreads();
    if (lane == 0) k_list[0] = k_list[1] = v_list[0] = v_list[1] = 0;
}

// New tokens of both tensors into their raw tails: blockIdx.z = 0 copies K, 1 copies V.
__global__ void tail_copy_kernel(const uint4 *__restrict__ ksrc, const uint4 *__restrict__ vsrc,
                                 int64_t src_batch_stride16, uint4 *__restrict__ kdst,
                                 uint4 *__restrict__ vdst, int64_t dst_batch_stride16, int64_t n16,
                                 bool bf16) {
    const int b = blockIdx.y;
    const uint4 *src = blockIdx.z ? vsrc : ksrc;
    uint4 *dst = blockIdx.z ? vdst : kdst;
    for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < n16;
         i += int64_t(gridDim.x) * blockDim.x)
        dst[b * dst_batch_stride16 + i] =
            load8_as_fp16<true>(reinterpret_cast<const __half *>(src + b * src_batch_stride16 + i), bf16);
}

__global__ void init_kernel(uint32_t *status, uint32_t *k_index, uint32_t *v_index, uint32_t *k_pages,
                            uint32_t *v_pages) {
    init_words(status, k_index, v_index);
    if (threadIdx.x == 0 && k_pages) k_pages[0] = k_pages[1] = v_pages[0] = v_pages[1] = 0;
}

// Minimum (low half) and negated maximum (high half) of a wave's values; mn, mx: two of each to a lane.
__device__ inline uint32_t wave_extremes(uint32_t mn, uint32_t mx) {
    mx ^= 0x80008000u;
    uint32_t w = pk_min_f16(__builtin_amdgcn_perm(mx, mn, 0x05040100u), __builtin_amdgcn_perm(mx, mn, 0x07060302u)), y = w;
    swap_rows32(w, y);
    y = w = pk_min_f16(w, y);
    swap_rows16(w, y);
    w = pk_min_f16(w, y);
    w = pk_min_f16(w, dpp_u32<DPP_ROW_ROR8>(w));
    w = pk_min_f16(w, dpp_u32<DPP_ROW_ROR4>(w));
    w = pk_min_f16(w, dpp_u32<DPP_QUAD_XOR2>(w));
    w = pk_min_f16(w, dpp_u32<DPP_QUAD_XOR1>(w));
    return w;
}

// Token parameters of both tensors (blockIdx.z) and V-median repacking, step 1, in one, codes below 16 (packs of 16): a
// wave holds a token's row of up to NREG * 512 values in registers, finds its scale and minimum, and of V
// quantizes it with the packs' fixed-point rule and counts every code with ballots; the lower median is the first code
// whose running count passes the middle.  NREG = 0, longer rows: read again for the codes.
// Bound by the counts, eight ballots for 512 values and each code but the last (five levels 40, fifteen 120).  One kernel instead of two that both read V: 12032 tokens of 1024
// values 12 + 15.5 -> 17.6 us, 7936 tokens of 6656 values 31 + 39 -> 63 (those all in registers: 140, the unrolled
// counts overflow the instruction cache; 4096 values read twice: 40.0 instead of 35.5).
template <int NREG, bool STREAM>
__global__ __launch_bounds__(256) void token_params_keys_kernel(ParamArgs a, int n_tokens, int qmax, uint8_t *__restrict__ keys) {
    const int lane = threadIdx.x & 63, t = blockIdx.x * 4 + (threadIdx.x >> 6), b = blockIdx.y;
    if (t >= n_tokens) return;
    ieee_mode_off();
    const ParamTensor &pt = a.t[blockIdx.z];
    const __half *row = pt.src + b * a.batch_stride + t * a.token_stride;
    uint4 x[NREG ? NREG : 1];
    uint32_t mn = 0x7C007C00u, mx = 0xFC00FC00u;
    auto widen = [&](const uint4 &v) {
        mn = pk_min_f16(mn, pk_min_f16(pk_min_f16(v.x, v.y), pk_min_f16(v.z, v.w)));
        mx = pk_max_f16(mx, pk_max_f16(pk_max_f16(v.x, v.y), pk_max_f16(v.z, v.w)));
    };
    if constexpr (NREG == 0) {
        for (int e = 8 * lane; e < a.row_elems; e += 512) widen(as_fp16(load8<STREAM>(row + e), a.bf16));
    }
#pragma unroll
    for (int k = 0; k < NREG; ++k)
        if (512 * k + 8 * lane < a.row_elems) x[k] = load8<STREAM>(row + 512 * k + 8 * lane);
#pragma unroll
    for (int k = 0; k < NREG; ++k)
        if (512 * k + 8 * lane < a.row_elems) widen(x[k] = as_fp16(x[k], a.bf16));
    const uint32_t w = wave_extremes(mn, mx);
    const uint32_t mt = token_meta_word(half_lo(w), -half_hi(w), pt.rel);
    const int64_t at = b * a.meta_stride + a.first_token + t;
    if (lane == 0) pt.meta[at] = mt;
    if (blockIdx.z == 0) return;
    const float4 tq = token_quant(mt);
    int count[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) count[v] = 0;
    auto tally = [&](const uint4 &v, bool present) {
        uint32_t pair[4] = {0, 0, 0, 0};  // no code where the row has ended
        if (present) quantize_token8(v, tq, uint32_t(qmax), pair);
#pragma unroll
        for (int c = 0; c < 16; ++c) {
            if (c < qmax) {  // the last code's count is what is left
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    count[c] += __popcll(__builtin_amdgcn_ballot_w64((pair[i] & 0xFFFFu) == 0x4300u + c));
                    count[c] += __popcll(__builtin_amdgcn_ballot_w64((pair[i] >> 16) == 0x4300u + c));
                }
            }
        }
    };
    if constexpr (NREG == 0) {
        for (int e0 = 0; e0 < a.row_elems; e0 += 512) {
            const int e = e0 + 8 * lane;
            x[0] = make_uint4(0, 0, 0, 0);
            if (e < a.row_elems) x[0] = as_fp16(load8<STREAM>(row + e), a.bf16);
            tally(x[0], e < a.row_elems);
        }
    }
#pragma unroll
    for (int k = 0; k < NREG; ++k) {
        if (512 * k >= a.row_elems) break;
        tally(x[k], 512 * k + 8 * lane < a.row_elems);
    }
    const int rank = (a.row_elems - 1) / 2;
    int seen = 0, key = qmax;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        if (v < qmax) {
            seen += count[v];
            if (seen > rank && key == qmax) key = v;
        }
    }
    if (lane == 0) keys[at] = uint8_t(key);
}

// Repacked tokens, staged rounds of codes up to 15 and at most 64 kv-heads: the tokens are quantized in arrival order, their
// codes moved into storage order afterwards, so the input is read once (before: by the kernel above and again, in storage
// order, by quantize16_kernel).  This kernel is the one above plus the codes of both tensors, eight nibbles to a word, to the
// chunk's slot as [token][channel]; the tail's tokens of a block that is being completed are handled as in quantize16_kernel.
// A wave (WAVES = 1: rows of up to 2048 values) or four waves take a token, NREG 16-byte registers to a lane.  The key is found
// by bisection: the codes up to a bound are counted with ballots, three times for five levels (every code counted: 40 ballots
// for 512 values instead of 24).  Bound by latency: waves that take several tokens, the next one's values on their way, are
// slower (12032 tokens of 8 heads, whole append 45.9 us with a token to a wave, 49.2 with four).
// Appends of repacked tokens, input read twice -> once: 8 x 52 heads of 32 000 tokens 4043 -> 2782 us, 8 x 32 of 8000 552 -> 462,
// 4 x 8 of 3001 bf16 tokens in pages 62.5 -> 46.1 (of which this kernel 18, 49 MB in), packs of 8, 32 heads of 4000 102 -> 39.
template <int NREG, int WAVES, bool STREAM>
__global__ __launch_bounds__(256) void quantize_tokens_kernel(PackArgs a) {
    ieee_mode_off();
    __shared__ __attribute__((aligned(16))) uint32_t extremes[4];
    __shared__ __attribute__((aligned(16))) int counts[2][4];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const PackTensor &pt = a.t[blockIdx.y];
    const ChunkSource &cs = pt.cs;
    const int i = WAVES == 1 ? int(blockIdx.x) * 4 + wave : int(blockIdx.x), token = i & (N - 1), row = i / N;   // row of the part
    const uint32_t full = uint32_t(a.part_row + row), cap = uint32_t(cs.qmax);
    const int blk = int((uint64_t(full) * a.magic_b) >> 32), b = int(full) - blk * cs.B;
    const int row_elems = cs.H * D;
    const int wave_first = WAVES == 1 ? 0 : wave * NREG * 512, first = wave_first + 8 * lane;   // the lane's value of register k: + 512 k
    const bool old = token < a.held;   // (held is 0 but in a block that is being completed)
    __half *const tail = pt.tail + (int64_t(b) * N + token) * row_elems;
    const __half *const src = old ? tail : cs.src + b * cs.batch_stride + (int64_t(blk) * N + token - a.held) * cs.token_stride;
    uint4 x[NREG];
#pragma unroll
    for (int k = 0; k < NREG; ++k)
        if (first + 512 * k < row_elems) x[k] = load8<STREAM>(src + first + 512 * k);
    uint32_t mn = 0x7C007C00u, mx = 0xFC00FC00u;
#pragma unroll
    for (int k = 0; k < NREG; ++k) {
        if (first + 512 * k < row_elems) {
            const uint4 v = x[k] = as_fp16(x[k], cs.bf16 && !old);
            mn = pk_min_f16(mn, pk_min_f16(pk_min_f16(v.x, v.y), pk_min_f16(v.z, v.w)));
            mx = pk_max_f16(mx, pk_max_f16(pk_max_f16(v.x, v.y), pk_max_f16(v.z, v.w)));
        }
    }
    uint32_t w = wave_extremes(mn, mx);
    if constexpr (WAVES > 1) {
        if (lane == 0) extremes[wave] = w;
        __syncthreads();
        const uint4 all = *reinterpret_cast<const uint4 *>(extremes);
        w = pk_min_f16(pk_min_f16(all.x, all.y), pk_min_f16(all.z, all.w));
    }
    const uint32_t mt = token_meta_word(half_lo(w), -half_hi(w), pt.rel);
    const int64_t at = b * cs.meta_stride + cs.first_token + int64_t(blk) * N + token;
    if (lane == 0 && (WAVES == 1 || wave == 0)) cs.meta[at] = mt;
    const float4 tq = token_quant(mt);
    const uint32_t codes_at = pt.stage_at + uint32_t(row * cs.H) * pt.slot + pt.header16 * 16 + uint32_t(token * (D / 2)) + 4 * (lane & 15);
    uint32_t low[NREG][4], high[NREG][4];   // 0x4300 + code of the even and odd channels; past the row's end above all codes
#pragma unroll
    for (int k = 0; k < NREG; ++k) {
#pragma unroll
        for (int j = 0; j < 4; ++j) low[k][j] = high[k][j] = 0xFFFFu;
        const int e = first + 512 * k;
        if (e < row_elems) {
            uint32_t pair[4];
            quantize_token8(x[k], tq, cap, pair);
            const uint32_t p01 = __builtin_amdgcn_perm(pair[1], pair[0], 0x06020400u), p23 = __builtin_amdgcn_perm(pair[3], pair[2], 0x06020400u);
            const uint32_t even = __builtin_amdgcn_perm(p23, p01, 0x05040100u), odd = __builtin_amdgcn_perm(p23, p01, 0x07060302u);
            *reinterpret_cast<uint32_t *>(a.staging + (codes_at + uint32_t(e / D) * pt.slot)) = even | (odd << 4);
            if (!old && a.held) *reinterpret_cast<uint4 *>(tail + e) = x[k];
#pragma unroll
            for (int j = 0; j < 4; ++j) low[k][j] = pair[j] & 0xFFFFu, high[k][j] = pair[j] >> 16;
        }
    }
    if (blockIdx.y == 0) return;
    // lower median: the smallest code with more than `rank` codes up to it
    const int rank = (row_elems - 1) / 2;
    uint32_t below = 0, above = cap;   // it is one of below .. above
    for (int flip = 0; below < above; flip ^= 1) {
        const uint32_t mid = (below + above) >> 1, bound = 0x4300u + mid;
        int n = 0;
#pragma unroll
        for (int k = 0; k < NREG; ++k) {
            if (wave_first + 512 * k >= row_elems) break;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                n += __popcll(__builtin_amdgcn_ballot_w64(low[k][j] <= bound)) + __popcll(__builtin_amdgcn_ballot_w64(high[k][j] <= bound));
        }
        if constexpr (WAVES > 1) {
            if (lane == 0) counts[flip][wave] = n;
            __syncthreads();   // (one a step: the next step's counts go to the other row)
            const int4 all = *reinterpret_cast<const int4 *>(counts[flip]);
            n = __builtin_amdgcn_readfirstlane((all.x + all.y) + (all.z + all.w));
        }
        if (n > rank) above = mid; else below = mid + 1;
    }
    if (lane == 0 && (WAVES == 1 || wave == 0)) a.keys[at] = uint8_t(below);
}

// Codes of a chunk from arrival order [token][channel] to packs in storage order, in place in the chunk's slot, with the pack
// headers and width sums that quantize16_kernel leaves.  A wave to a chunk; lane (row g, cg): the sixteen tokens of group g,
// channels 8 cg .. 8 cg + 7, two 8 x 8 transpositions of nibbles.  2 x 1504 chunks 6.8 us
// (12 MB in and out; the quantizer that read the input again 18.4, and the order's kernel 4).
template <bool PACK8>
__global__ __launch_bounds__(256) void move_codes_kernel(PackArgs a) {
    __shared__ __attribute__((aligned(16))) uint8_t orders[4][N];
    const PackTensor &pt = a.t[blockIdx.y];
    const int lane = threadIdx.x & 63, cg = lane & 15, g = lane >> 4, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int cl = int(blockIdx.x) * 4 + wave;
    if (cl >= a.n) return;
    const ChunkCoord k = chunk_coord(pt.cs, a.part_first + cl);
    const int key = a.keys[k.b * pt.cs.meta_stride + pt.cs.first_token + int64_t(k.blk) * N + lane];
    orders[wave][storage_rank(key, a.t[1].cs.qmax)] = uint8_t(lane);
    wave_lds_fence();
    const uint4 order = *reinterpret_cast<const uint4 *>(&orders[wave][16 * g]);
    uint8_t *const slot = a.staging + (pt.stage_at + uint32_t(cl) * pt.slot);
    uint8_t *const codes = slot + (PACK8 ? HEADER8 : HEADER);
    uint32_t x[16];
#pragma unroll
    for (int t = 0; t < 16; ++t) {
        const uint32_t o = t < 4 ? order.x : t < 8 ? order.y : t < 12 ? order.z : order.w;
        x[t] = *reinterpret_cast<const uint32_t *>(codes + ((o >> (8 * (t & 3))) & 0xFFu) * (D / 2) + 4 * cg);
    }
    uint32_t mn[4], mx[4], sum = 0;   // halves: channels j and j + 4
    auto headers = [&](int group) {
        const uint32_t m01 = __builtin_amdgcn_perm(mn[1], mn[0], 0x06020400u), m23 = __builtin_amdgcn_perm(mn[3], mn[2], 0x06020400u);
        const uint32_t x01 = __builtin_amdgcn_perm(mx[1], mx[0], 0x06020400u), x23 = __builtin_amdgcn_perm(mx[3], mx[2], 0x06020400u);
        const uint32_t m_lo = __builtin_amdgcn_perm(m23, m01, 0x05040100u), m_hi = __builtin_amdgcn_perm(m23, m01, 0x07060302u);
        const uint32_t w_lo = width_bytes(__builtin_amdgcn_perm(x23, x01, 0x05040100u) - m_lo);
        const uint32_t w_hi = width_bytes(__builtin_amdgcn_perm(x23, x01, 0x07060302u) - m_hi);
        sum += w_lo + w_hi;
        *reinterpret_cast<uint2 *>(slot + D * group + 8 * cg) = make_uint2((w_lo << 4) | m_lo, (w_hi << 4) | m_hi);
    };
#pragma unroll
    for (int half = 0; half < 2; ++half) {
#pragma unroll
        for (int t = 8 * half; t < 8 * half + 8; t += 2) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                // (codes are fp16 subnormals)
                const uint32_t p = (x[t] >> (4 * j)) & 0x000F000Fu, q = (x[t + 1] >> (4 * j)) & 0x000F000Fu;
                const bool first = t == (PACK8 ? 8 * half : 0);
                mn[j] = first ? pk_min(p, q) : pk_min3_f16(mn[j], p, q);
                mx[j] = first ? pk_max(p, q) : pk_max3_f16(mx[j], p, q);
            }
        }
        if (PACK8) headers(2 * g + half);
    }
    if (!PACK8) headers(g);
    // all codes are in registers before the first of them is overwritten, by whichever lane
#pragma unroll
    for (int t = 0; t < 16; ++t) asm volatile("" ::"v"(x[t]));
    vmem_order_fence();
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        uint32_t y[8];
#pragma unroll
        for (int t = 0; t < 8; t += 2) {
            const uint32_t p = x[8 * half + t], q = x[8 * half + t + 1];
            y[t] = (p & 0x0F0F0F0Fu) | ((q << 4) & 0xF0F0F0F0u);
            y[t + 1] = ((p >> 4) & 0x0F0F0F0Fu) | (q & 0xF0F0F0F0u);
        }
#pragma unroll
        for (int t = 0; t < 8; t = t % 4 == 1 ? t + 3 : t + 1) {   // 0 1 4 5
            const uint32_t p = y[t], q = y[t + 2];
            y[t] = __builtin_amdgcn_perm(q, p, 0x06020400u);
            y[t + 2] = __builtin_amdgcn_perm(q, p, 0x07030501u);
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const uint32_t p = y[t], q = y[t + 4];
            y[t] = __builtin_amdgcn_perm(q, p, 0x05040100u);
            y[t + 4] = __builtin_amdgcn_perm(q, p, 0x07060302u);
        }
        uint8_t *const to = codes + 1024 * g + 512 * half + 16 * cg;
        *reinterpret_cast<uint4 *>(to) = make_uint4(y[0], y[1], y[2], y[3]);
        *reinterpret_cast<uint4 *>(to + 256) = make_uint4(y[4], y[5], y[6], y[7]);
    }
    sum += sum >> 16;
    sum = (sum + (sum >> 8)) & 0xFFu;
    sum = row_inclusive_scan(sum);
    if (cg == 15) pt.widths[4 * cl + g] = uint16_t(sum);
}

// V-median repacking, step 1 (Sec. III-B.3): the lower median of the H*128 quantized V codes of
// one token, written as a sort key.  One workgroup per (token, batch).
template <bool STREAM>
__global__ __launch_bounds__(256) void v_median_key_kernel(const __half *__restrict__ src,
                                                           int64_t batch_stride, int64_t token_stride,
                                                           int row_elems, int qmax,
                                                           const uint32_t *__restrict__ meta,
                                                           int64_t meta_stride, int64_t first_token,
                                                           uint8_t *__restrict__ keys, bool bf16) {
    __shared__ int hist[256];
    const int t = blockIdx.x, b = blockIdx.y;
    hist[threadIdx.x] = 0;
    __syncthreads();
    const __half *row = src + b * batch_stride + t * token_stride;
    const float4 tsm = token_scale_min(meta[b * meta_stride + first_token + t]);
    if (qmax > 15) {
        // codes up to 255: count straight into the LDS histogram
        for (int i = threadIdx.x * 8; i < row_elems; i += 256 * 8) {
            uint4 raw = load8_as_fp16<STREAM>(row + i, bf16);
            const __half *hv = reinterpret_cast<const __half *>(&raw);
#pragma unroll
            for (int k = 0; k < 8; ++k) atomicAdd(&hist[quantize_value(__half2float(hv[k]), tsm.x, tsm.y, tsm.z, qmax)], 1);
        }
    } else {
        // sixteen 8-bit counters in two words; a thread sees at most 8 * ceil(row_elems / 2048) values
        uint64_t lo = 0, hi = 0;
        for (int i = threadIdx.x * 8; i < row_elems; i += 256 * 8) {
            uint4 raw = load8_as_fp16<STREAM>(row + i, bf16);
            const __half *hv = reinterpret_cast<const __half *>(&raw);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int v = quantize_value(__half2float(hv[k]), tsm.x, tsm.y, tsm.z, qmax);
                const uint64_t one = 1ull << (8 * (v & 7));
                if (v < 8) lo += one; else hi += one;
            }
        }
        for (int bin = 0; bin <= qmax; ++bin) {
            int c = int(((bin < 8 ? lo : hi) >> (8 * (bin & 7))) & 0xFFu);
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o);
            if ((threadIdx.x & 63) == 0) atomicAdd(&hist[bin], c);
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const int rank = (row_elems - 1) / 2;
        int seen = 0, v = 0;
        for (; v < qmax; ++v) {
            seen += hist[v];
            if (seen > rank) break;
        }
        keys[b * meta_stride + first_token + t] = uint8_t(v);
    }
}

// Step 2: one wave per (block, batch) ranks the 64 keys (ascending, equal keys in arrival order),
// replaces them by the order and moves the token metadata of both tensors into storage order.
__global__ __launch_bounds__(64) void block_order_kernel(uint8_t *__restrict__ order, int qmax,
                                                         uint32_t *__restrict__ k_meta,
                                                         uint32_t *__restrict__ v_meta,
                                                         int64_t meta_stride, int64_t first_token) {
    __shared__ uint8_t ord[N];
    const int lane = threadIdx.x;
    const int64_t pos = blockIdx.y * meta_stride + first_token + int64_t(blockIdx.x) * N;
    const int key = order[pos + lane];
    const uint32_t km = k_meta[pos + lane], vm = v_meta[pos + lane];
    const int rank = storage_rank(key, qmax);
    ord[rank] = uint8_t(lane);
    k_meta[pos + rank] = km;
    v_meta[pos + rank] = vm;
    __syncthreads();
    order[pos + lane] = ord[lane];
}

// ---------------------------------------------------------------------------
int launch_init(const kv_cache *c, hipStream_t s) {
    uint8_t *ws = static_cast<uint8_t *>(c->buf.workspace);
    hipLaunchKernelGGL(init_kernel, dim3(1), dim3(64), 0, s,
                       reinterpret_cast<uint32_t *>(ws + WS_STATUS),
                       static_cast<uint32_t *>(c->buf.k_index),
                       static_cast<uint32_t *>(c->buf.v_index),
                       c->pool ? static_cast<uint32_t *>(c->buf.k_pages) : nullptr,
                       c->pool ? static_cast<uint32_t *>(c->buf.v_pages) : nullptr);
    KV_HIP_CHECK(hipGetLastError());
    return KV_OK;
}

int launch_pool_init(const kv_page_pool *pool, hipStream_t s) {
    const int64_t blocks = (pool->n_pages + 255) / 256;
    hipLaunchKernelGGL(pool_init_kernel, dim3(uint32_t(blocks)), dim3(256), 0, s, pool->state, pool->n_pages);
    KV_HIP_CHECK(hipGetLastError());
    return KV_OK;
}

int launch_release_pages(const kv_cache *c, hipStream_t s) {
    if (!c->pool) return KV_ERR_ARG;
    hipLaunchKernelGGL(release_pages_kernel, dim3(1), dim3(64), 0, s,
                       static_cast<uint32_t *>(c->buf.k_pages), static_cast<uint32_t *>(c->buf.v_pages),
                       c->pool->state, c->pool->n_pages, reinterpret_cast<uint32_t *>(static_cast<uint8_t *>(c->buf.workspace) + WS_STATUS),
                       static_cast<uint32_t *>(c->buf.k_index), static_cast<uint32_t *>(c->buf.v_index));
    KV_HIP_CHECK(hipGetLastError());
    return KV_OK;
}

int launch_tail_copy(const kv_cache *c, const __half *ksrc, const __half *vsrc, int64_t src_batch_stride,
                     int n, int tail_pos, bool bf16, hipStream_t s) {
    const int64_t row = int64_t(c->cfg.n_kv_heads) * D;  // elements per token
    const int64_t n16 = n * row / 8;
    if (n16 == 0) return KV_OK;
    const int threads = 256;
    const int blocks = int(std::min<int64_t>((n16 + threads - 1) / threads, 1024));
    __half *ktail = static_cast<__half *>(c->buf.k_tail), *vtail = static_cast<__half *>(c->buf.v_tail);
    hipLaunchKernelGGL(tail_copy_kernel, dim3(blocks, c->cfg.batch, 2), dim3(threads), 0, s,
                       reinterpret_cast<const uint4 *>(ksrc), reinterpret_cast<const uint4 *>(vsrc),
                       src_batch_stride / 8, reinterpret_cast<uint4 *>(ktail + int64_t(tail_pos) * row),
                       reinterpret_cast<uint4 *>(vtail + int64_t(tail_pos) * row),
                       int64_t(c->cfg.tail_capacity) * row / 8, n16, bf16);
    KV_HIP_CHECK(hipGetLastError());
    return KV_OK;
}

// The V-median keys come with the token parameters (codes of the fixed-point rule).
static bool keys_with_params(const kv_cache *c) {
    return c->cfg.repack == KV_REPACK_V_MEDIAN && c->qmax_v < 16;
}

int launch_token_params(const kv_cache *c, const CompressJob &kjob, const CompressJob &vjob, hipStream_t s) {
    const int B = c->cfg.batch, H = c->cfg.n_kv_heads;
    const int n_tokens = kjob.n_blocks * N;
    if (n_tokens <= 0) return KV_ERR_ARG;
    ParamArgs a;
    a.t[0] = ParamTensor{kjob.src, kjob.rel, kjob.meta};
    a.t[1] = ParamTensor{vjob.src, vjob.rel, vjob.meta};
    a.batch_stride = kjob.batch_stride;
    a.token_stride = kjob.token_stride;
    a.meta_stride = c->max_tokens;
    a.first_token = kjob.first_token;
    a.row_elems = H * D;
    a.bf16 = kjob.bf16;
    const bool wave = a.row_elems <= 2048, stream = larger_than_caches(int64_t(kjob.n_blocks) * B * H);
    if (keys_with_params(c)) {
        uint8_t *keys = static_cast<uint8_t *>(c->buf.token_order);
        const dim3 grid((n_tokens + 3) / 4, B, 2);
#define PACKKV_LAUNCH_KEYS(nreg)                                                                                                   \
    hipLaunchKernelGGL((stream ? token_params_keys_kernel<nreg, true> : token_params_keys_kernel<nreg, false>), grid, dim3(256), 0, s, a, \
                       n_tokens, vjob.qmax, keys)
        if (a.row_elems <= 1024) PACKKV_LAUNCH_KEYS(2);
        else if (a.row_elems <= 2048) PACKKV_LAUNCH_KEYS(4);
        else if (a.row_elems <= 4096) PACKKV_LAUNCH_KEYS(8);
        else PACKKV_LAUNCH_KEYS(0);
#undef PACKKV_LAUNCH_KEYS
        KV_HIP_CHECK(hipGetLastError());
        return KV_OK;
    }
    auto kernel = wave ? (stream ? token_params_kernel<true, true> : token_params_kernel<true, false>)
                       : (stream ? token_params_kernel<false, true> : token_params_kernel<false, false>);
    hipLaunchKernelGGL(kernel, dim3(wave ? (n_tokens + 3) / 4 : n_tokens, B, 2), dim3(256), 0, s, a, n_tokens);
    KV_HIP_CHECK(hipGetLastError());
    return KV_OK;
}

int launch_v_median_order(const kv_cache *c, const CompressJob &vjob, uint32_t *k_meta, uint8_t *order,
                          hipStream_t s) {
    const int B = c->cfg.batch, H = c->cfg.n_kv_heads;
    const int n_tokens = vjob.n_blocks * N;
    if (n_tokens <= 0 || H * D / 2048 + 1 > 31) return KV_ERR_ARG;  // 8-bit per-thread counters
    const bool stream = larger_than_caches(int64_t(vjob.n_blocks) * B * H);
    if (!keys_with_params(c))
        hipLaunchKernelGGL(stream ? v_median_key_kernel<true> : v_median_key_kernel<false>, dim3(n_tokens, B), dim3(256), 0, s, vjob.src,
                           vjob.batch_stride, vjob.token_stride, H * D, vjob.qmax, vjob.meta,
                           c->max_tokens, vjob.first_token, order, vjob.bf16);
    hipLaunchKernelGGL(block_order_kernel, dim3(vjob.n_blocks, B), dim3(64), 0, s, order, vjob.qmax,
                       k_meta, vjob.meta, c->max_tokens, vjob.first_token);
    KV_HIP_CHECK(hipGetLastError());
    return KV_OK;
}

template <bool WRITE, bool WIDE>
static auto chunk8(bool stream) {
    return stream ? chunk_kernel<WRITE, 8, WIDE, true> : chunk_kernel<WRITE, 8, WIDE, false>;
}

// Whether the arenas take the next n_chunks chunks of each tensor at their largest, by the host's bound of the fill level.
static bool fits_for_sure(const kv_cache *c, int n_chunks) {
    if (c->pool) return true;
    auto worst16 = [&](bool wide) { return uint64_t(n_chunks) * uint64_t(chunk_max_bytes(c->cfg.pack_size, wide) / 16); };
    return c->fill_bound16[0] + worst16(c->wide_k) <= arena_units(c->sizes.k_arena) && c->fill_bound16[1] + worst16(c->wide_v) <= arena_units(c->sizes.v_arena);
}

// Whether a round in two passes over the input finds its metadata and sizes with the staged path's quantizer (the width sums go to the
// staging area): one read of the input for both, where token parameters and sizes took one each (pages, 8 x 10 heads of 22 090 tokens 847 -> 759 us, 3 x 1 of
// 11 032 43.7 -> 29.9; packs of 8, 32 heads of 10 000 188 -> 150).
static bool sizes_in_one(const kv_cache *c, int n_chunks) {
    const size_t area = size_t(c->stage_chunks / 2) * stage_pair_bytes(c->cfg.pack_size, c->wide_k, c->wide_v);
    return std::max(c->qmax_k, c->qmax_v) <= MOST_STAGED_CODE && c->cfg.n_kv_heads <= 64 && c->cfg.repack == KV_REPACK_NONE &&
           area >= size_t(2) * 8 * (size_t(n_chunks) + 8);
}

// Whether a round that could be staged in parts of at most `most` chunks is better done in two passes over all of it: parts leave
// the chip idle and cost two launches each; the second read comes from the last-level cache or costs less than they do.  Staged / two passes:
// packs of 16, parts of 256 chunks (4 heads of 40 000 tokens) 128 / 50 us, 512 (8 heads of 13 000) 60 / 41, 1024 (2 x 8 of 30 000) 155 / 107, 2048 (32 of
// 20 000) 151 / 137, two of 2048 58 / 65, 2560 (4 x 10 of 30 000) 274 / 252, 3328 (52 of 20 000) 214 / 227, 5120 (8 x 10 of 22 090) 327 / 384; packs of 8, whose second pass is
// slower, 256 (4 heads of 13 000) 55 / 41, 512 (8 heads) 64 / 58, 1024 (2 x 8 of 20 000) 105 / 126.  Repacked packs of 8, whose token parameters
// and sizes are two passes themselves, 4 heads of 30 000, wide, in 8 parts of 256 174 / 116.
static bool two_passes_pay(const kv_cache *c, int n_chunks, int most) {
    const int parts = (n_chunks + most - 1) / most;
    if (!sizes_in_one(c, n_chunks)) return c->cfg.pack_size == 8 && most < 1024 && parts > 4;
    if (c->cfg.pack_size == 8) return parts > 1 && most <= 640;
    // (an arena that may be too full: the staged kernels find out before they have read anything twice)
    return ((parts > 2 && most <= 2560) || (parts > 1 && most <= 512)) && fits_for_sure(c, n_chunks);
}

// Whether a round of n_chunks chunks (per tensor) is staged, unless (packs of 16) the arena turns out to be too full.
// Packs of 8: only where no arena can be too full, and for codes the fixed-point quantizer takes.
static bool staged_rounds(const kv_cache *c, int n_chunks) {
    const int most = c->stage_chunks / 2;
    if (most < c->cfg.n_kv_heads || (c->pool && n_chunks > most) || two_passes_pay(c, n_chunks, most)) return false;
    return c->cfg.pack_size == 16 || (std::max(c->qmax_k, c->qmax_v) <= MOST_STAGED_CODE && fits_for_sure(c, n_chunks));
}

bool finds_params(const kv_cache *c, int n_chunks) {
    return c->cfg.n_kv_heads <= 64 && c->cfg.repack == KV_REPACK_NONE && (staged_rounds(c, n_chunks) || sizes_in_one(c, n_chunks));
}

// A round of many small parts is left to the token parameters of the whole round and two kernels to a part, instead of three
// (40 000 tokens of 1, 2, 4, 8 streams, 256 and, of eight, 512 chunks to a part: 68, 94, 164, 201 us; moved 75, 101, 175, 197).
bool moves_codes(const kv_cache *c, int n_chunks) {
    const int most = c->stage_chunks / 2;
    return c->cfg.repack == KV_REPACK_V_MEDIAN && staged_rounds(c, n_chunks) && fits_for_sure(c, n_chunks) && c->cfg.n_kv_heads <= 64 &&
           std::max(c->qmax_k, c->qmax_v) <= 15 && (n_chunks <= most || most >= 512);
}

static void launch_quantize_tokens(const PackArgs &a, int H, bool stream, hipStream_t s) {
    const dim3 grid(a.rows * (H <= 16 ? N / 4 : N), 2);
#define PACKKV_LAUNCH_TOKENS(nreg, waves) \
    hipLaunchKernelGGL((stream ? quantize_tokens_kernel<nreg, waves, true> : quantize_tokens_kernel<nreg, waves, false>), grid, dim3(256), 0, s, a)
    if (H <= 8) PACKKV_LAUNCH_TOKENS(2, 1);
    else if (H <= 16) PACKKV_LAUNCH_TOKENS(4, 1);
    else if (H <= 32) PACKKV_LAUNCH_TOKENS(2, 4);
    else PACKKV_LAUNCH_TOKENS(4, 4);
#undef PACKKV_LAUNCH_TOKENS
}

template <int HP, bool GIVEN, bool PACK8>
static void launch_quantize16_as(PackArgs &a, int H, bool stream, bool unsure, bool mixed, bool sizes, hipStream_t s) {
    const int waves = HP < 4 ? 1 : std::min((H + 3) / 4, GIVEN ? 4 : 16);
    // workgroups of that many waves that fit a compute unit (0: not asked yet)
    static std::atomic<int> per_cu_of[17];
    int per_cu = per_cu_of[waves].load(std::memory_order_relaxed);
    if (!per_cu) {
        per_cu = resident_workgroups(reinterpret_cast<const void *>(quantize16_kernel<HP, GIVEN, false, false, false, PACK8>), 64 * waves);
        per_cu_of[waves].store(per_cu, std::memory_order_relaxed);
    }
    const int64_t items = int64_t(2) * a.rows * HP * (HP == 4 && GIVEN ? (H + 15) / 16 : 1);
    int groups = mixed ? int(items) : flat_groups_for(items * 4, per_cu, int64_t(1) << 30);   // all resident, at most one per item
    a.split = 1;
    if (HP == 4 && !GIVEN) {
        const int room = flat_groups_for(int64_t(1) << 40, 1, int64_t(1) << 30);
        while (a.split < 4 && 4 * a.split < waves && items * a.split * 2 <= room) a.split *= 2;
        groups *= a.split;
    }
    auto kernel = stream ? quantize16_kernel<HP, GIVEN, true, false, false, PACK8> : quantize16_kernel<HP, GIVEN, false, false, false, PACK8>;
    if constexpr (!PACK8)
        if (unsure) kernel = stream ? quantize16_kernel<HP, GIVEN, true, true, false, false> : quantize16_kernel<HP, GIVEN, false, true, false, false>;
    if constexpr (!GIVEN)
        if (mixed) kernel = quantize16_kernel<HP, false, false, false, true, PACK8>;
    if constexpr (!GIVEN)
        if (sizes) kernel = stream ? quantize16_kernel<HP, false, true, false, false, PACK8, true> : quantize16_kernel<HP, false, false, false, false, PACK8, true>;
    hipLaunchKernelGGL(kernel, dim3(groups), dim3(64 * waves), 0, s, a);
}

template <bool PACK8>
static void launch_quantize16(PackArgs &a, int H, bool given, bool stream, bool unsure, bool mixed, bool sizes, hipStream_t s) {
#define PACKKV_LAUNCH_QUANTIZE(hp)                                        \
    given ? launch_quantize16_as<hp, true, PACK8>(a, H, stream, unsure, false, false, s) \
          : launch_quantize16_as<hp, false, PACK8>(a, H, stream, unsure, mixed, sizes, s)
    if (H == 1) PACKKV_LAUNCH_QUANTIZE(1);
    else if (H == 2) PACKKV_LAUNCH_QUANTIZE(2);
    else PACKKV_LAUNCH_QUANTIZE(4);
#undef PACKKV_LAUNCH_QUANTIZE
}

bool completes_in_place(const kv_cache *c) {
    const int n_chunks = c->cfg.batch * c->cfg.n_kv_heads;
    return ((staged_rounds(c, n_chunks) && finds_params(c, n_chunks) && fits_for_sure(c, n_chunks)) || moves_codes(c, n_chunks)) && !larger_than_caches(n_chunks);
}

int launch_pack(const kv_cache *c, const CompressJob &kjob, const CompressJob &vjob, TailRest *rest, hipStream_t s) {
    const int B = c->cfg.batch, H = c->cfg.n_kv_heads;
    const int n_chunks = kjob.n_blocks * B * H;
    if (n_chunks <= 0 || n_chunks > MAX_NEW_CHUNKS) return KV_ERR_ARG;
    uint8_t *ws = static_cast<uint8_t *>(c->buf.workspace);
    uint32_t *sizes16 = reinterpret_cast<uint32_t *>(ws + WS_SIZES);
    const bool planes = c->cfg.pack_size == 16;
    // packs of 16, contiguous arena: the staged path when even the largest chunks fit (decided on
    // the device, where the fill level is); the kernels of the other path return at once, but for the token
    // metadata, which the first kernel of the staged path finds either way.  The
    // host knows an upper bound of the fill level: where that already says "fits", the two-pass
    // kernels are not launched at all.
    // Paged arena: the placement needs the sizes of the whole round, so the staged path takes the
    // rounds that fit the staging area whole (the input is then quantized once, not twice: 33 -> 21 us for
    // 2 x 1504 repacked bf16 chunks); it places whatever the pool covers, so no fill level is tested.
    const bool staged = staged_rounds(c, n_chunks);
    bool two_pass = !staged || !fits_for_sure(c, n_chunks);
    const bool stream = larger_than_caches(n_chunks);
    PackArgs a;
    for (int i = 0; i < 2; ++i) {
        const CompressJob &job = i ? vjob : kjob;
        PackTensor &t = a.t[i];
        t.cs.src = job.src;
        t.cs.batch_stride = job.batch_stride;
        t.cs.token_stride = job.token_stride;
        t.cs.B = B;
        t.cs.H = H;
        t.cs.qmax = job.qmax;
        t.cs.magic_h = (uint64_t(1) << 32) / uint64_t(H) + 1;
        t.cs.magic_hb = (uint64_t(1) << 32) / (uint64_t(H) * uint64_t(B)) + 1;
        t.cs.meta = job.meta;
        t.rel = job.rel;
        const QuantRange range = quant_range(job.rel, job.qmax);
        t.cap_all = range.cap_all;
        t.small_scale = range.small_scale;
        t.widths = nullptr;
        t.cs.meta_stride = c->max_tokens;
        t.cs.first_token = job.first_token;
        t.cs.order = job.order;
        t.cs.bf16 = job.bf16;
        t.cs.pack_order = job.pack_order;
        t.round.first_chunk = job.first_chunk;
        t.wide = job.wide;
        t.slot = uint32_t(chunk_max_bytes(c->cfg.pack_size, job.wide));
        t.header16 = uint32_t(chunk_header_bytes(c->cfg.pack_size, job.wide) / 16);
        t.unit_shift = planes ? UNIT_SHIFT16 : UNIT_SHIFT8;
        t.round.worst16 = staged ? uint32_t(n_chunks) * (t.slot / 16) : 0;
        t.round.arena_cap16 = c->pool ? ~uint64_t(0) : job.arena_cap16;
        t.index = job.index;
        t.arena = job.arena;
        t.arena_cap16 = job.arena_cap16;
        t.status = job.status;
        t.page_list = job.page_list;
        t.max_pages = job.max_pages;
        t.tail = static_cast<__half *>(i ? c->buf.v_tail : c->buf.k_tail);
        t.rest = rest ? rest->src[i] : nullptr;
    }
    const bool unsure = two_pass;   // the device decides (staged_round)
    a.index_words = c->index_words;
    a.magic_b = (uint64_t(1) << 32) / uint64_t(B) + 1;
    a.first_tensor = 0;
    a.pool_state = c->pool ? c->pool->state : nullptr;
    a.staging = ws + c->stage_offset;
    a.held = kjob.held;
    a.keys = staged && moves_codes(c, n_chunks) ? static_cast<uint8_t *>(c->buf.token_order) : nullptr;
    a.rest_units = 0;
    if (staged) {
        // equal parts of whole rows that fit the staging area, half of its slots for each tensor
        const int rows = n_chunks / H, most = c->stage_chunks / 2 / H;
        const int parts = (rows + most - 1) / most, per_part = (rows + parts - 1) / parts;
        a.round_rows = rows;
        for (int part = 0; part < rows; part += per_part) {
            a.part_row = part;
            a.rows = std::min(per_part, rows - part);
            a.part_first = part * H;
            a.n = a.rows * H;
            a.t[0].widths = reinterpret_cast<uint16_t *>(sizes16);
            a.t[1].widths = a.t[0].widths + 4 * ((a.n + 1) & ~1);
            a.t[0].stage_at = 0;
            a.t[1].stage_at = uint32_t(a.n) * a.t[0].slot;
            if (a.keys) {
                launch_quantize_tokens(a, H, stream, s);
                hipLaunchKernelGGL(planes ? move_codes_kernel<false> : move_codes_kernel<true>, dim3((a.n + 3) / 4, 2), dim3(256), 0, s, a);
            } else
                (planes ? launch_quantize16<false> : launch_quantize16<true>)(a, H, !finds_params(c, n_chunks), stream, unsure, kjob.held > 0, false, s);
            static_assert(PLACE_SMALL_CHUNKS >= 16384 / 2, "a staged round of a paged cache fits the placement kernel");
            static_assert(16384 * 8 + 64 <= WS_SIZES_BYTES, "the width sums of a part fit the sizes area");
            if (c->pool) hipLaunchKernelGGL(place_small_kernel, dim3(1), dim3(1024), 0, s, a);
            int groups = (a.n + 3) / 4;
            if (rest && rest->tokens > 0 && !two_pass && part + per_part >= rows) {   // behind the last read of the tail
                a.rest_units = rest->tokens * (H * D / 8);
                a.rest_stride = rest->batch_stride;
                a.rest_bf16 = rest->bf16;
                groups += (a.rest_units + REST_UNITS - 1) / REST_UNITS * B;
                rest->tokens = 0;
            }
            if (planes) {
                auto assemble = a.keys || a.rest_units ? assemble16_kernel<false, true> : assemble16_kernel<false, false>;
                if (unsure) assemble = assemble16_kernel<true, false>;
                hipLaunchKernelGGL(assemble, dim3(groups, 2), dim3(256), 0, s, a);
            }
            else
                hipLaunchKernelGGL(assemble8_kernel, dim3(groups, 2), dim3(256), 4 * std::max(a.t[0].slot, a.t[1].slot), s, a);
        }
    }
    if (two_pass) {
        // both tensors per launch where the sizes area takes both (and, packs of 8, the layouts agree)
        a.part_first = a.part_row = 0;
        a.n = n_chunks;
        a.rows = a.round_rows = n_chunks / H;
        const bool sized = !staged && finds_params(c, n_chunks);
        a.t[0].widths = sized ? reinterpret_cast<uint16_t *>(a.staging) : nullptr;
        a.t[1].widths = sized ? a.t[0].widths + 4 * ((n_chunks + 7) & ~3) : nullptr;
        const bool both = sized || 2 * ((n_chunks + 3) & ~3) <= MAX_NEW_CHUNKS;
        const bool same = planes || kjob.wide == vjob.wide;
        if (sized) (planes ? launch_quantize16<false> : launch_quantize16<true>)(a, H, false, stream, false, false, true, s);
        for (int i = 0; i < 2; i += both ? 2 : 1) {
            a.first_tensor = i;
            a.t[0].sizes16 = sizes16;
            a.t[1].sizes16 = both && !sized ? sizes16 + ((n_chunks + 3) & ~3) : sizes16;
            const int n_tensors = both ? 2 : 1;
            auto pass = [&](bool write) {
                for (int j = i; j < i + n_tensors; j += same ? n_tensors : 1) {
                    a.first_tensor = j;
                    const dim3 grid(n_chunks, same ? n_tensors : 1);
                    const bool wide = j ? vjob.wide : kjob.wide;
                    auto kernel = planes ? (write ? chunk16_kernel<true> : chunk16_kernel<false>)
                                  : wide ? (write ? chunk8<true, true>(stream) : chunk8<false, true>(stream))
                                         : (write ? chunk8<true, false>(stream) : chunk8<false, false>(stream));
                    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, a);
                }
                a.first_tensor = i;
            };
            if (!sized) pass(false);
            if (c->pool && n_tensors == 2 && n_chunks <= PLACE_SMALL_CHUNKS)
                hipLaunchKernelGGL(place_small_kernel, dim3(1), dim3(1024), 0, s, a);
            else if (c->pool)
                hipLaunchKernelGGL(place_chunks_kernel, dim3(1), dim3(1024), 0, s, a, n_tensors);
            else
                hipLaunchKernelGGL(scan_offsets_kernel, dim3(n_tensors), dim3(1024), 0, s, a);
            pass(true);
        }
    }
    KV_HIP_CHECK(hipGetLastError());
    return KV_OK;
}

}  // namespace packkv
