// Fused V path (PackKV Sec. III-C.2): out = p^T Vhat, streaming the packed V cache once and
// decoding it on chip.
//
// The paper gives each thread one pack (a dot-product segment along ctx_len) and combines
// segments with fp32 atomic adds.  Here the contraction runs along the pack direction, so it maps
// onto the matrix cores without any transposition: the planes of a pack are FP4 operands as they
// are stored (v_planes.h; packs of 8 tokens and wide chunks: fp16 operands, pack8.h), the
// softmax weights times the token scales are the other operand, and the G query heads of a group
// share one decode.  Accumulation is fp32 inside the matrix instruction, in a fixed order: the
// context axis is split over workgroups whose partial sums are combined by a second small kernel or the last workgroup of
// a stream -- no floating-point atomics, bitwise reproducible.  De-quantization is folded in:
//   out_d = sum_t w_t code[t,d] + sum_g m[g,d] sum_{t in g} w_t + sum_t p_t min_t
// (wide chunks: centred codes and minimums, vw_chunk).
#include <algorithm>
#include <mutex>

#include "last_group.h"
#include "pack8.h"
#include "v_chunk.h"
#include "v_planes.h"

#ifndef PACKKV_V_NBUF
#define PACKKV_V_NBUF 2
#endif

namespace packkv {

struct VArgs {
    const uint8_t *arena;
    const uint32_t *index;
    const uint32_t *meta;   // [B][meta_stride]
    const float *p;         // [B][Hq][ld]
    float *partial;         // [splits][B*Hq][V_PART_STRIDE]
    int64_t ld;
    int64_t meta_stride;
    int B, H;
    int index_words;        // index words per chunk: 1 back to back, 2 with a paged arena
    int dup;                // H counts every kv-head dup times (query groups above 8 are split): kv-head = h / dup
    int n_blocks;           // packed blocks per stream
    int blocks_per_split;
    // MERGE: the last workgroup of a stream merges its rows (else v_reduce_kernel does)
    uint8_t *counters;      // of stream 0, a word per stream
    const __half *tail;     // [B][tail_cap][kv-heads][128]
    int64_t packed_tokens;
    int n_tail, tail_cap;
    float *out;
};

// The sums of a workgroup's four waves, red[4][G][..], to the partial rows dst[g].
template <int G, bool MERGE>
__device__ inline void v_store_partial(const VArgs &a, const float (*red)[G][D + 4], float *dst) {
    if (threadIdx.x < G * (D / 4)) {
        const int g = threadIdx.x / (D / 4), d4 = threadIdx.x % (D / 4);
        const float4 x = *reinterpret_cast<const float4 *>(&red[0][g][4 * d4]), y = *reinterpret_cast<const float4 *>(&red[1][g][4 * d4]);
        const float4 z = *reinterpret_cast<const float4 *>(&red[2][g][4 * d4]), w = *reinterpret_cast<const float4 *>(&red[3][g][4 * d4]);
        const float4 sum = make_float4((x.x + y.x) + (z.x + w.x), (x.y + y.y) + (z.y + w.y), (x.z + y.z) + (z.z + w.z), (x.w + y.w) + (z.w + w.w));
        const float pmin = (red[0][g][D] + red[1][g][D]) + (red[2][g][D] + red[3][g][D]);
        float *row = dst + g * V_PART_STRIDE;
        if constexpr (MERGE) {
            store_shared(row + 4 * d4, sum.x, sum.y);
            store_shared(row + 4 * d4 + 2, sum.z, sum.w);
            if (d4 == 0) store_shared(row + D, pmin, 0.0f);
        } else {
            *reinterpret_cast<float4 *>(row + 4 * d4) = sum;
            if (d4 == 0) row[D] = pmin;
        }
    }
}

// The last workgroup of a stream: adds its n_sets row sets (the first at first_set, set_stride floats apart) and the raw
// fp16 tail, in an order of its own, a wave, or with one or two heads several waves, per query head.
template <int G>
__device__ inline void v_merge_stream(const VArgs &a, int stream, int b, int h, const float *first_set, int n_sets, int64_t set_stride,
                                      uint32_t *flag, float *scratch) {
    if (!last_group(a.counters + 4 * stream, uint32_t(n_sets), flag)) return;
    constexpr int W = G == 1 ? 4 : G == 2 ? 2 : 1;   // waves per head: each takes every W-th row set and 64 / W tail tokens
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), part = wave % W;
    float *const weights = scratch + 256 * wave, *const sums = weights + 64;
    const int kvh = h / a.dup, Hkv = a.H / a.dup;
    const int sets = (n_sets - part + W - 1) / W, tail0 = part * (N / W), n_tail = max(0, min(a.n_tail - tail0, N / W));
    for (int g = wave / W; g < G; g += 4 / W) {
        const int64_t row = int64_t(stream) * G + g;
        const float *first = first_set + g * V_PART_STRIDE + part * set_stride;
        const __half *vrow = a.tail + ((int64_t(b) * a.tail_cap + tail0) * Hkv + kvh) * D;
        RowSum rows;
        TailSum tail;
        rows.load(first, W * set_stride, 0, sets, lane);
        float pmin = 0.0f;
        if (lane < sets) pmin = load_shared(first + lane * W * set_stride + D).x;
        if (n_tail > 0) {
            tail.load(vrow, int64_t(Hkv) * D, 0, n_tail, lane);
            weights[lane] = lane < n_tail ? a.p[row * a.ld + a.packed_tokens + tail0 + lane] : 0.0f;
            wave_lds_fence();
        }
        pmin = wave_all_sum(pmin);
        float2 o = rows.sum(first, W * set_stride, sets, 1.0f, lane);
        o.x += pmin, o.y += pmin;
        if (n_tail > 0) {
            const float2 t = tail.sum(vrow, int64_t(Hkv) * D, weights, n_tail, sums, lane);
            o.x += t.x, o.y += t.y;
        }
        if constexpr (W > 1) {
            *reinterpret_cast<float2 *>(sums + 2 * lane) = o;
            __syncthreads();
            if (part != 0) continue;
            o = make_float2(0.0f, 0.0f);
#pragma unroll
            for (int p = 0; p < W; ++p) {
                const float2 v = *reinterpret_cast<const float2 *>(sums + 256 * p + 2 * lane);
                o.x += v.x, o.y += v.y;
            }
        }
        *reinterpret_cast<float2 *>(a.out + row * D + 2 * lane) = o;
    }
}

// SOLO: a workgroup has its stream to itself, tail included.  Wave w of WAVES takes the tail's tokens 64 / WAVES * w ..; their values and
// weights are loaded ahead of the first chunk and stay in registers.
template <int G, int WAVES>
struct VSoloTail {
    static constexpr int PER = N / WAVES;
    uint4 v[PER / 4];        // token lane / 16 + 4 i, channels 8 (lane % 16) ..
    float w[G][PER / 4];
    __device__ inline void load(const VArgs &a, const float *prow, int b, int h, int wave, int lane) {
        const int Hkv = a.H / a.dup, left = a.n_tail - PER * wave;
        const int64_t step = int64_t(Hkv) * D;
        const __half *vrow = a.tail + ((int64_t(b) * a.tail_cap + PER * wave + (lane >> 4)) * Hkv + h / a.dup) * D + 8 * (lane & 15);
#pragma unroll
        for (int i = 0; i < PER / 4; ++i) {
            const int t = (lane >> 4) + 4 * i;
            v[i] = make_uint4(0, 0, 0, 0);
            if (t < left) v[i] = *reinterpret_cast<const uint4 *>(vrow + 4 * i * step);
#pragma unroll
            for (int g = 0; g < G; ++g) w[g][i] = t < left ? prow[g * a.ld + a.packed_tokens + PER * wave + t] : 0.0f;
        }
    }
    __device__ inline void consume() {
#pragma unroll
        for (int i = 0; i < PER / 4; ++i) {
            consume_here(v[i].x), consume_here(v[i].y), consume_here(v[i].z), consume_here(v[i].w);
#pragma unroll
            for (int g = 0; g < G; ++g) {
                uint32_t bits = __float_as_uint(w[g][i]);
                consume_here(bits);
                w[g][i] = __uint_as_float(bits);
            }
        }
    }
    // Adds the wave's tail tokens to its rows red[g].
    __device__ inline void add(const VArgs &a, float (*red)[D + 4], int wave, int lane) const {
        if (a.n_tail <= PER * wave) return;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            float acc[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e] = 0.0f;
#pragma unroll
            for (int i = 0; i < PER / 4; ++i) {
                const __half *hv = reinterpret_cast<const __half *>(&v[i]);
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[e] = fmaf(w[g][i], __half2float(hv[e]), acc[e]);
            }
            const float2 two = row_sums8(acc);
            float2 *const place = row_sums8_place(red[g], lane);
            const float2 before = *place;
            *place = make_float2(before.x + two.x, before.y + two.y);
        }
    }
};

// The waves' rows of a stream, tail included, to its outputs.
template <int G, int WAVES>
__device__ inline void v_solo_store(const VArgs &a, const float (*red)[G][D + 4], int64_t head0) {
    for (int i = threadIdx.x; i < G * D / 2; i += 64 * WAVES) {
        const int g = i / (D / 2), d = 2 * (i % (D / 2));
        float x = 0.0f, y = 0.0f, pmin = 0.0f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            const float2 v = *reinterpret_cast<const float2 *>(&red[w][g][d]);
            x += v.x, y += v.y, pmin += red[w][g][D];
        }
        *reinterpret_cast<float2 *>(a.out + (head0 + g) * D + d) = make_float2(x + pmin, y + pmin);
    }
}

// Packs of 16 tokens, plane layout (v_planes.h).  HIGH: the codes of the cache may need four bits
// (otherwise a chunk is at most 512 + 512 * 6 bytes).  The chunks of all streams form one work
// list that is cut into equal ranges, one per workgroup (FlatPlan): a launch is one round of
// long-lived workgroups whatever the numbers of streams and blocks are.  The four waves of a
// workgroup take every fourth block of its range.  A wave keeps NBUF chunk buffers: the next
// chunks stream in while one is decoded, and the token metadata and the weights of a chunk
// travel the same way (one dword per lane, global memory -> LDS, behind the chunk in its buffer):
// no vector memory instruction of the loop is visible to the compiler, so the only waits are the
// counted ones below.
// SOLO > 0: a workgroup of that many waves to a stream (blockIdx.x), which does it all, tail included: no partial rows through memory and no second
// kernel (v_solo_waves says where).
template <int G, bool HIGH, bool MERGE, int SOLO = 0>
__global__ __launch_bounds__(SOLO ? 64 * SOLO : 256) void v_matvec_kernel(VArgs a, FlatPlan plan) {
    constexpr int WAVES = SOLO ? SOLO : 4;
    static_assert(!SOLO || !MERGE, "a stream of its own needs no merge");
    constexpr int CHUNK_BYTES = HIGH ? CHUNK_MAX : HEADER + PACKS * 6;
    constexpr int SLICES = (CHUNK_BYTES + 1023) / 1024;
    constexpr int SIDE = CHUNK_BYTES + LDS_TAIL_PAD;   // metadata row, then G weight rows
    constexpr int BUF = SIDE + (1 + G) * 256;          // bytes of one chunk buffer
    constexpr int NBUF = PACKKV_V_NBUF;                // chunks n+1 .. n+NBUF-1 in flight
    static_assert(NBUF == 2 || NBUF == 3, "wait counts below");
    // between the ranges of two streams the chunk buffers hold the cross-wave reduction array
    __shared__ __attribute__((aligned(16))) uint8_t lds_all[WAVES * NBUF * BUF];
    constexpr int VB = vb_bytes<G>();
    __shared__ __attribute__((aligned(16))) uint8_t vb_all[WAVES * VB];
    __shared__ uint4 table[PLANE_TABLE_ENTRIES];
    __shared__ uint32_t highs[PLANE_TABLE_ENTRIES];
    __shared__ uint32_t merge_flag;
    static_assert(sizeof(float) * G * (D + 4) <= NBUF * BUF, "reduction array must fit");
    static_assert(BUF % 16 == 0, "buffers are 16-byte aligned");
    float(*red)[G][D + 4] = reinterpret_cast<float(*)[G][D + 4]>(lds_all);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int buf_base = wave * NBUF * BUF;
    bool tables = false;
    uint8_t *vb = vb_all + wave * VB;
    const int grp = blockIdx.x;
    const int64_t range_end = SOLO ? int64_t(grp + 1) * a.n_blocks : plan.begin(grp + 1);
    VSoloTail<G, WAVES> tail;

    for (int64_t f = SOLO ? int64_t(grp) * a.n_blocks : plan.begin(grp); f < range_end;) {
        const FlatPlan::Segment seg = plan.segment(f, range_end);
        const int stream = seg.stream, b = seg.b, h = seg.h, blk_begin = seg.blk_begin, blk_end = seg.blk_end;
        f += blk_end - blk_begin;
        const uint32_t *meta = a.meta + b * a.meta_stride;
        const float *prow = a.p + int64_t(stream) * G * a.ld;
        VPlaneState<G> st;
        st.clear();

        // everything chunk `blk` needs, into buffer `slot`: 1 + G row transfers, then the chunk
        // itself (with the streaming hint: the weights, which the softmax kernel has just written,
        // then stay in the caches); returns the number of transfer instructions of the chunk
        auto issue = [&](const IndexBatch &ib, int it, int blk, int slot) -> int {
            uint8_t *buf = lds_all + buf_base + slot * BUF;
            row_issue_lds(meta + int64_t(blk) * N, buf + SIDE, lane);
#pragma unroll
            for (int g = 0; g < G; ++g) row_issue_lds(prow + g * a.ld + int64_t(blk) * N, buf + SIDE + 256 * (1 + g), lane);
            return chunk_issue_lds_counted<CHUNK_BYTES, HEADER, true>(a.arena, ib.start16(it), ib.end16(it), buf, lane);
        };

        IndexBatch ib;
        auto load_index = [&](int first) {
            if (first < blk_end) ib.load(a.index, a.index_words, first, WAVES, blk_end, a.B, a.H / a.dup, b, h / a.dup, lane);
        };
        load_index(blk_begin + wave);
        if constexpr (SOLO > 0) tail.load(a, prow, b, h, wave, lane);
        if (!tables) {  // while the index words are on their way
            for (int i = threadIdx.x; i < WAVES * VB / 4; i += 64 * WAVES) reinterpret_cast<uint32_t *>(vb_all)[i] = 0;
            build_plane_table(table, highs);
            tables = true;
        }
        for (int first = blk_begin + wave; first < blk_end; first += WAVES * 64) {
            const int n_it = min(64, (blk_end - first + WAVES - 1) / WAVES);
            wait_chunk_landed();  // the index words (the only loads the compiler sees)
            if constexpr (SOLO > 0) {
                if (first == blk_begin + wave) tail.consume();
            }
            issue(ib, 0, first, 0);
            int slices_next = 0;  // transfer instructions of chunk it + 1
            if (NBUF == 3 && n_it > 1) slices_next = issue(ib, 1, first + WAVES, 1);
            int slot = 0;         // buffer of chunk it
            for (int it = 0; it < n_it; ++it) {
                const int cur = buf_base + slot * BUF;
                const bool valid = ib.end16(it) - ib.start16(it) >= uint32_t(HEADER / 16);
                // chunk it with its rows has landed; with three buffers the 1 + G rows and the
                // chunk of it + 1 may still be in flight
                if (NBUF == 3 && it + 1 < n_it)
                    wait_vmem_except<1 + G, SLICES>(slices_next);
                else
                    wait_chunk_landed();
                if (it + NBUF - 1 < n_it) {
                    // into the buffer chunk it - 1 was decoded from: its LDS reads have returned
                    lds_reads_returned();
                    slices_next = issue(ib, it + NBUF - 1, first + WAVES * (it + NBUF - 1), slot == 0 ? NBUF - 1 : slot - 1);
                }
                slot = slot == NBUF - 1 ? 0 : slot + 1;
                if (!valid) continue;  // a block dropped by an arena overflow contributes nothing
                const uint32_t mt = *reinterpret_cast<const uint32_t *>(lds_all + cur + SIDE + 4 * lane);
                float pt[G];
#pragma unroll
                for (int g = 0; g < G; ++g)
                    pt[g] = *reinterpret_cast<const float *>(lds_all + cur + SIDE + 256 * (1 + g) + 4 * lane);
                v_planes_chunk<G, HIGH>(lds_all, cur, table, highs, vb, mt, pt, st);
            }
            wait_chunk_landed();
            load_index(first + WAVES * 64);
        }
        __syncthreads();  // every wave is done with its chunk buffers: reuse them as red[][][]

        v_planes_store<G>(st, red[wave], lane);
        if constexpr (SOLO > 0) {
            wave_lds_fence();
            tail.add(a, red[wave], wave, lane);
            __syncthreads();
            v_solo_store<G, WAVES>(a, red, int64_t(stream) * G);
            return;
        }
        __syncthreads();
        float *dst = a.partial + int64_t(grp + stream) * G * V_PART_STRIDE;
        v_store_partial<G, MERGE>(a, red, dst);
        if constexpr (MERGE) {
            const int w_lo = plan.group_of(int64_t(stream) * plan.n_blocks), w_hi = plan.group_of(int64_t(stream + 1) * plan.n_blocks - 1);
            v_merge_stream<G>(a, stream, b, h, a.partial + int64_t(w_lo + stream) * G * V_PART_STRIDE, w_hi - w_lo + 1,
                              int64_t(G) * V_PART_STRIDE, &merge_flag, reinterpret_cast<float *>(lds_all));
        }
        __syncthreads();  // red[][][] has been read: the buffers may be filled again
    }
}

// The same for chunks with packs of 8 tokens (Sec. IV-B; pack8.h).  Here and for wide chunks the transfers carry the
// non-temporal hint too (cache read from memory: 15.6 -> 15.1 us for 32 streams of 156 blocks at four heads, wide
// 23.0 -> 20.4 for 64 of 127; the K products gain less and lose 1 % on large caches, and go without).
// MID: wide chunks without codes above 31, of which two fit as well (pack8.h; with one buffer, as below, 64 streams of 127
// blocks took 22.6 us).
template <int G, bool MID, bool MERGE>
__global__ __launch_bounds__(256) void v8_matvec_kernel(VArgs a, VCentre centre) {
    constexpr int LDS = MID ? CHUNKM_LDS : CHUNK8_LDS, MAXB = MID ? CHUNKM_MAX : CHUNK8_MAX, HDR = MID ? HEADERW : HEADER8;
    // two chunk buffers per wave; after the main loop the same memory holds the
    // cross-wave reduction array red[4][G][D + 4]
    __shared__ __attribute__((aligned(16))) uint8_t lds_all[4 * 2 * LDS + LDS_TAIL_PAD];
    __shared__ __attribute__((aligned(16))) uint8_t blds_all[4 * BLds<G>::BYTES];
    __shared__ uint4 table[MID ? 16 : PACK_TABLE_ENTRIES];
    static_assert(sizeof(float) * 4 * G * (D + 4) <= 4 * 2 * LDS, "reduction array must fit");
    float(*red)[G][D + 4] = reinterpret_cast<float(*)[G][D + 4]>(lds_all);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int split = blockIdx.x;
    const int bh = blockIdx.y;
    const int h = bh % a.H, b = bh / a.H;
    const int buf_base = wave * 2 * LDS;
    const int blk_begin = split * a.blocks_per_split;
    const int blk_end = min(blk_begin + a.blocks_per_split, a.n_blocks);
    IndexBatch ib;
    auto load_index = [&](int first) {
        if (first < blk_end) ib.load(a.index, a.index_words, first, 4, blk_end, a.B, a.H / a.dup, b, h / a.dup, lane);
    };
    load_index(blk_begin + wave);
    if constexpr (MID) build_wide_tables(nullptr, table);
    else build_pack_table(table, CODE_LIFT, fold_min<G>());
    VLane<G> vl;
    vl.init(blds_all + wave * BLds<G>::BYTES, lane);
    vl.bslot = v8_bslot<G>(lane);  // lane l is token l of the block
    VState<G, MID || fold_min<G>()> st;
    st.clear();

    for (int first = blk_begin + wave; first < blk_end; first += 4 * 64) {
        const int n_it = min(64, (blk_end - first + 3) / 4);
        chunk_issue_lds<MAXB, HDR, true>(a.arena, ib.start16(0), ib.end16(0), lds_all + buf_base, lane);
        uint32_t mt_next = a.meta[b * a.meta_stride + int64_t(first) * N + lane];
        float p_next[G];
#pragma unroll
        for (int g = 0; g < G; ++g)
            p_next[g] = a.p[(int64_t(b) * a.H * G + h * G + g) * a.ld + int64_t(first) * N + lane];
        for (int it = 0; it < n_it; ++it) {
            const int cur = buf_base + (it & 1) * LDS;
            const bool valid = ib.end16(it) - ib.start16(it) >= uint32_t(HDR / 16);
            wait_chunk_landed();
            uint32_t mt = mt_next;
            consume_here(mt);
            float pt[G];
#pragma unroll
            for (int g = 0; g < G; ++g) {
                pt[g] = p_next[g];
                consume_here(pt[g]);
            }
            // the next chunk streams into the other buffer while this one is unpacked
            if (it + 1 < n_it) {
                chunk_issue_lds<MAXB, HDR, true>(a.arena, ib.start16(it + 1), ib.end16(it + 1),
                                lds_all + buf_base + ((it + 1) & 1) * LDS, lane);
                const int64_t tok = int64_t(first + 4 * (it + 1)) * N + lane;
                mt_next = a.meta[b * a.meta_stride + tok];
#pragma unroll
                for (int g = 0; g < G; ++g) p_next[g] = a.p[(int64_t(b) * a.H * G + h * G + g) * a.ld + tok];
            }
            if (!valid) continue;  // a block dropped by an arena overflow contributes nothing
            if constexpr (MID) vw_chunk<G, true>(lds_all, cur, table, vl, mt, pt, centre, st);
            else v8_chunk<G>(lds_all, cur, table, vl, mt, pt, st);
        }
        wait_chunk_landed();
        load_index(first + 4 * 64);
    }
    __syncthreads();  // every wave is done with its chunk buffers: reuse them as red[][][]

    v_state_store<G, MID>(st, red[wave], lane, MID ? 1.0f : CODE_SCALE_LIFTED);  // the wide path feeds the codes as numbers
    __syncthreads();
    const int64_t set_stride = int64_t(a.B) * a.H * G * V_PART_STRIDE;
    float *first_set = a.partial + int64_t(bh) * G * V_PART_STRIDE;
    v_store_partial<G, MERGE>(a, red, first_set + split * set_stride);
    if constexpr (MERGE) {
        v_merge_stream<G>(a, bh, b, h, first_set, gridDim.x, set_stride, reinterpret_cast<uint32_t *>(table), reinterpret_cast<float *>(lds_all));
    }
}

// Wide chunks (codes above 15; pack8.h): one buffer per wave (a chunk is up to 10 KB), so the
// transfer is waited for before the unpack; the other waves of the compute unit overlap with it.
template <int G, bool MERGE>
__global__ __launch_bounds__(256) void vw_matvec_kernel(VArgs a, VCentre centre) {
    __shared__ __attribute__((aligned(16))) uint8_t lds_all[4 * CHUNKW_LDS + LDS_TAIL_PAD];
    __shared__ __attribute__((aligned(16))) uint8_t blds_all[4 * BLds<G>::BYTES];
    __shared__ uint4 vtable[16];
    static_assert(sizeof(float) * 4 * G * (D + 4) <= 4 * CHUNKW_LDS, "reduction array must fit");
    float(*red)[G][D + 4] = reinterpret_cast<float(*)[G][D + 4]>(lds_all);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int split = blockIdx.x;
    const int bh = blockIdx.y;
    const int h = bh % a.H, b = bh / a.H;
    const int buf = wave * CHUNKW_LDS;
    const int blk_begin = split * a.blocks_per_split;
    const int blk_end = min(blk_begin + a.blocks_per_split, a.n_blocks);
    IndexBatch ib;
    auto load_index = [&](int first) {
        if (first < blk_end) ib.load(a.index, a.index_words, first, 4, blk_end, a.B, a.H / a.dup, b, h / a.dup, lane);
    };
    load_index(blk_begin + wave);
    build_wide_tables(nullptr, vtable);
    VLane<G> vl;
    vl.init(blds_all + wave * BLds<G>::BYTES, lane);
    vl.bslot = v8_bslot<G>(lane);  // lane l is token l of the block
    VState<G, true> st;
    st.clear();

    for (int first = blk_begin + wave; first < blk_end; first += 4 * 64) {
        const int n_it = min(64, (blk_end - first + 3) / 4);
        for (int it = 0; it < n_it; ++it) {
            const bool valid = ib.end16(it) - ib.start16(it) >= uint32_t(HEADERW / 16);
            lds_reads_returned();  // one buffer: the previous chunk has been read completely
            chunk_issue_lds<CHUNKW_MAX, HEADERW, true>(a.arena, ib.start16(it), ib.end16(it), lds_all + buf, lane);
            const int64_t tok = int64_t(first + 4 * it) * N + lane;
            const uint32_t mt = a.meta[b * a.meta_stride + tok];
            float pt[G];
#pragma unroll
            for (int g = 0; g < G; ++g) pt[g] = a.p[(int64_t(b) * a.H * G + h * G + g) * a.ld + tok];
            wait_chunk_landed();
            if (!valid) continue;  // a block dropped by an arena overflow contributes nothing
            vw_chunk<G, true>(lds_all, buf, vtable, vl, mt, pt, centre, st);
        }
        load_index(first + 4 * 64);
    }
    __syncthreads();  // every wave is done with its chunk buffer: reuse the memory as red[][][]

    v_state_store<G, true>(st, red[wave], lane, 1.0f);  // the wide path feeds the codes as numbers
    __syncthreads();
    const int64_t set_stride = int64_t(a.B) * a.H * G * V_PART_STRIDE;
    float *first_set = a.partial + int64_t(bh) * G * V_PART_STRIDE;
    v_store_partial<G, MERGE>(a, red, first_set + split * set_stride);
    if constexpr (MERGE) {
        v_merge_stream<G>(a, bh, b, h, first_set, gridDim.x, set_stride, reinterpret_cast<uint32_t *>(vtable), reinterpret_cast<float *>(lds_all));
    }
}

// Fixed-order combination of the split partial sums, plus the raw fp16 tail.  plan.n_groups > 0:
// the partial rows come from a kernel that walks the flat work list (kv-head group size Gk per
// stream); the row sets of stream s are those of the workgroups that hold one of its chunks.
__global__ __launch_bounds__(256) void v_reduce_kernel(const float *__restrict__ partial,
                                                       int n_splits, int n_rows, FlatPlan plan, int Gk,
                                                       const float *__restrict__ p, int64_t ld,
                                                       int64_t packed_tokens,
                                                       const __half *__restrict__ tail, int n_tail,
                                                       int tail_cap, int H, int G,
                                                       float *__restrict__ out) {
    __shared__ float lds[16][V_PART_STRIDE];
    __shared__ float wt[N];
    const int r = blockIdx.x;  // b*Hq + hq
    const int d = threadIdx.x;
    const int hq = r % (H * G), b = r / (H * G);
    const int h = hq / G;
    // every global load of the kernel is issued before the first result is needed
    SplitRows rows;
    TailRows trows;
    if (plan.n_groups > 0) {
        const int stream = r / Gk, g = r % Gk;
        const int w_lo = plan.group_of(int64_t(stream) * plan.n_blocks);
        const int w_hi = plan.group_of(int64_t(stream + 1) * plan.n_blocks - 1);
        n_splits = w_hi - w_lo + 1;
        rows.load_strided(partial + (int64_t(w_lo + stream) * Gk + g) * V_PART_STRIDE, n_splits, Gk);
    } else {
        rows.load(partial, n_splits, n_rows, r);
    }
    trows.load(tail + (int64_t(b) * tail_cap * H + h) * D, int64_t(H) * D, n_tail);
    if (d < n_tail) wt[d] = p[int64_t(r) * ld + packed_tokens + d];
    float pmin;
    float acc = rows.sum(n_splits, lds, &pmin);  // its barriers also publish wt
    acc += pmin;
    if (n_tail > 0) acc += trows.sum(wt, n_tail, lds);
    if (d < D) out[int64_t(r) * D + d] = acc;
}

// partial: [splits][B * H_q][V_PART_STRIDE] floats for the split sums; max_split_rows: how many
// such rows it can take (the split count is lowered to fit).
// Workgroups of `kernel` that fit one compute unit (registers, LDS); 1 if the
// runtime cannot tell.
int resident_workgroups(const void *kernel, int threads) {
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, threads, 0) != hipSuccess || n < 1) n = 1;
    return n;
}

static int64_t resident_room(int per_cu) {
    static int n_cu = 0;
    if (n_cu == 0) {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0)
            n_cu = v;
        else
            n_cu = 256;
    }
    return int64_t(n_cu) * per_cu;
}
int flat_groups_for(int64_t total, int per_cu, int64_t most) { return int(flat_groups(total, resident_room(per_cu), most)); }
int plan_groups_for(int n_blocks, int streams, int per_cu, int64_t most) {
    return plan_groups(n_blocks, streams, resident_room(per_cu), most);
}
StreamSplits splits_for(int n_blocks, int streams, int per_cu, int most) {
    return stream_splits(n_blocks, streams, int(resident_room(1)), per_cu, most);
}

// Waves of a workgroup that has a stream to itself, 0: the streams are split (as in the fused attention, where a block is twice the
// work; four waves only where eight would not let two workgroups share a compute unit).  Split, the reduction included / solo, replayed, us:
// one stream, one head, 4 blocks 6.8 / 4.7, 16 6.8 / 6.2, 24 6.9 / 7.4; 8, four heads, 8 8.1 / 6.5, 16 8.2 / 8.3; 128 of 16 8.9 / 6.9, of 32 10.4 / 9.0,
// of 60 12.3 / 12.7; 256 of 15 blocks at four heads 14.4 / 9.0, of 90 29.4 / 26.2; one head, 120 23.4 / 21.9, 160 27.9 / 27.9; 320 of 30 13.9 / 13.0, of 60 19.5 / 19.6;
// 416 of 16 12.5 / 9.5, of 120 34.7 / 33.8; 384 at four heads 30 23.0 / 20.4, 60 31.8 / 32.9.
static int v_solo_waves(int n_blocks, int streams, int heads) {
    const int cus = int(resident_room(1));
    if (streams <= cus) return n_blocks <= (4 * streams >= 3 * cus ? 120 : 2 * streams >= cus ? 32 : heads <= 2 ? 16 : 8) ? 8 : 0;
    if (streams > 2 * cus) return 0;
    if (heads <= 2) return n_blocks <= (2 * streams > 3 * cus ? 120 : 30) ? 8 : 0;
    return n_blocks <= 30 ? 4 : 0;
}

// partial: [row sets][V_PART_STRIDE] floats for the split sums; max_split_rows: how many rows
// (one per query head and split or row set) it can take; counter: COUNT_V or COUNT_V_NOALLOC.
static int launch_v_matvec_into(const kv_cache *c, const float *p, int64_t ld_p, float *out, float *partial,
                                int64_t max_split_rows, int counter, hipStream_t s) {
    // Hs: kv-heads as the stream kernels count them (each dup times, see head_split); the combine
    // kernel works per query head and sees the real kv-head count and the whole group
    const int B = c->cfg.batch, H = c->cfg.n_kv_heads, G = c->group, Hs = H * c->head_split, Gq = G * c->head_split;
    const int n_blocks = int(c->packed_tokens / N);
    const int64_t rows = int64_t(B) * H * Gq;
    if (rows > max_split_rows) return KV_ERR_CAPACITY;
    const bool planes = !c->wide_v && c->cfg.pack_size == PACK;
    int n_splits = 0;
    FlatPlan plan = FlatPlan::make(n_blocks, B, Hs);
    VArgs a;
    a.arena = static_cast<const uint8_t *>(c->buf.v_arena);
    a.index = static_cast<const uint32_t *>(c->buf.v_index);
    a.meta = static_cast<const uint32_t *>(c->buf.v_token_meta);
    a.p = p;
    a.partial = partial;
    a.ld = ld_p;
    a.meta_stride = c->max_tokens;
    a.B = B;
    a.index_words = c->index_words;
    a.H = Hs;
    a.dup = c->head_split;
    a.n_blocks = n_blocks;
    a.blocks_per_split = 0;
    a.tail = static_cast<const __half *>(c->buf.v_tail);
    a.packed_tokens = c->packed_tokens;
    a.n_tail = c->tail_tokens;
    a.tail_cap = c->cfg.tail_capacity;
    a.out = out;
    a.counters = static_cast<uint8_t *>(c->buf.workspace) + WS_STATUS + 4 * ST_COUNTERS + counter;
    bool merged = false;
    if (n_blocks > 0 && planes) {
        // row sets: one per (workgroup, stream it touches), G rows each
        if (max_split_rows / G <= int64_t(B) * Hs) return KV_ERR_CAPACITY;
        // one round of resident workgroups: how many fit a compute unit depends on the instance; at
        // most 62 per stream (the combine kernel takes up to 64 row sets per stream)
        const int64_t most_groups = std::min<int64_t>(int64_t(62) * B * Hs, max_split_rows / G - int64_t(B) * Hs);
        const int solo = v_solo_waves(n_blocks, B * Hs, G);
#define PACKKV_LAUNCH_VX(g, high)                                                                          \
    {                                                                                                      \
        static const int per_cu = resident_workgroups(reinterpret_cast<const void *>(v_matvec_kernel<g, high, false>)); \
        plan.split(plan_groups_for(n_blocks, B * Hs, per_cu, most_groups));                               \
        merged = solo || merge_in_kernel(plan.n_groups, int64_t(B) * Hs, G);                              \
        if (solo == 8) hipLaunchKernelGGL((v_matvec_kernel<g, high, false, 8>), dim3(B * Hs), dim3(512), 0, s, a, plan); \
        else if (solo) hipLaunchKernelGGL((v_matvec_kernel<(g < 3 ? 3 : g), high, false, 4>), dim3(B * Hs), dim3(256), 0, s, a, plan); \
        else if (merged) hipLaunchKernelGGL((v_matvec_kernel<g, high, true>), dim3(plan.n_groups), dim3(256), 0, s, a, plan); \
        else hipLaunchKernelGGL((v_matvec_kernel<g, high, false>), dim3(plan.n_groups), dim3(256), 0, s, a, plan); \
    }
#define PACKKV_LAUNCH_V(g) PACKKV_LAUNCH_VX(g, false)
#define PACKKV_LAUNCH_VH(g) PACKKV_LAUNCH_VX(g, true)
        if (c->qmax_v > 7) {
            PACKKV_DISPATCH_GROUP4(G, PACKKV_LAUNCH_VH)
        } else {
            PACKKV_DISPATCH_GROUP4(G, PACKKV_LAUNCH_V)
        }
#undef PACKKV_LAUNCH_VH
#undef PACKKV_LAUNCH_V
#undef PACKKV_LAUNCH_VX
    } else if (n_blocks > 0) {
        const bool mid = c->wide_v && c->qmax_v <= MID_QMAX;
        int per_cu = 1;
#define PACKKV_ROOM(kernel) { static const int n = resident_workgroups(reinterpret_cast<const void *>(kernel)); per_cu = n; }
#define PACKKV_ROOM_VM(g) PACKKV_ROOM((v8_matvec_kernel<g, true, false>))
#define PACKKV_ROOM_VW(g) PACKKV_ROOM((vw_matvec_kernel<g, false>))
#define PACKKV_ROOM_V8(g) PACKKV_ROOM((v8_matvec_kernel<g, false, false>))
        if (mid) {
            PACKKV_DISPATCH_GROUP(G, PACKKV_ROOM_VM)
        } else if (c->wide_v) {
            PACKKV_DISPATCH_GROUP(G, PACKKV_ROOM_VW)
        } else {
            PACKKV_DISPATCH_GROUP(G, PACKKV_ROOM_V8)
        }
#undef PACKKV_ROOM_VM
#undef PACKKV_ROOM_VW
#undef PACKKV_ROOM_V8
#undef PACKKV_ROOM
        n_splits = int(std::min<int64_t>(splits_for(n_blocks, B * Hs, per_cu).n, max_split_rows / rows));
        a.blocks_per_split = (n_blocks + n_splits - 1) / n_splits;
        n_splits = (n_blocks + a.blocks_per_split - 1) / a.blocks_per_split;
        dim3 grid(n_splits, B * Hs);
        merged = merge_in_kernel(int64_t(n_splits) * B * Hs, int64_t(B) * Hs, G, c->wide_v);
#define PACKKV_LAUNCH_VW(g)                                                                     \
    if (merged) hipLaunchKernelGGL((vw_matvec_kernel<g, (g <= MERGED_HEADS)>), grid, dim3(256), 0, s, a, VCentre::of(c->qmax_v));      \
    else hipLaunchKernelGGL((vw_matvec_kernel<g, false>), grid, dim3(256), 0, s, a, VCentre::of(c->qmax_v))
#define PACKKV_LAUNCH_V8X(g, mid)                                                               \
    if (merged) hipLaunchKernelGGL((v8_matvec_kernel<g, mid, (g <= MERGED_HEADS)>), grid, dim3(256), 0, s, a, VCentre::of(c->qmax_v)); \
    else hipLaunchKernelGGL((v8_matvec_kernel<g, mid, false>), grid, dim3(256), 0, s, a, VCentre::of(c->qmax_v))
#define PACKKV_LAUNCH_V8(g) PACKKV_LAUNCH_V8X(g, false)
#define PACKKV_LAUNCH_VM(g) PACKKV_LAUNCH_V8X(g, true)
        if (mid) {
            PACKKV_DISPATCH_GROUP(G, PACKKV_LAUNCH_VM)
        } else if (c->wide_v) {
            PACKKV_DISPATCH_GROUP(G, PACKKV_LAUNCH_VW)
        } else {
            PACKKV_DISPATCH_GROUP(G, PACKKV_LAUNCH_V8)
        }
#undef PACKKV_LAUNCH_VW
#undef PACKKV_LAUNCH_V8
#undef PACKKV_LAUNCH_VM
#undef PACKKV_LAUNCH_V8X
    }
    if (merged) {
        KV_HIP_CHECK(hipGetLastError());
        return KV_OK;
    }
    hipLaunchKernelGGL(v_reduce_kernel, dim3(B * H * Gq), dim3(256), 0, s, partial, n_splits,
                       B * H * Gq, plan, G, p, ld_p, c->packed_tokens,
                       static_cast<const __half *>(c->buf.v_tail), c->tail_tokens,
                       c->cfg.tail_capacity, H, Gq, out);
    KV_HIP_CHECK(hipGetLastError());
    return KV_OK;
}

int launch_v_matvec(const kv_cache *c, const float *p, int64_t ld_p, float *out, hipStream_t s) {
    uint8_t *ws = static_cast<uint8_t *>(c->buf.workspace);
    return launch_v_matvec_into(c, p, ld_p, out, reinterpret_cast<float *>(ws + WS_VPART),
                                int64_t(V_SPLITS_MAX) * c->cfg.batch * c->cfg.n_q_heads, COUNT_V, s);
}

// ---- the V product for callers that cannot allocate ------------------------------------------
// The split sums go to a file-scope device array instead of the caller's workspace.  Every GPU
// the library runs on holds its own copy of the array (at its own address) until the process
// ends; the address is looked up once per device, with that device current, and kept.
static __device__ __align__(256) float scratch[size_t(KV_NOALLOC_MAX_SPLIT_ROWS) * V_PART_STRIDE];

static int scratch_of_current_device(float **out) {
    constexpr int MAX_DEVICES = 64;
    static float *ptr_of_device[MAX_DEVICES];
    static std::mutex lock;
    int dev = -1;
    KV_HIP_CHECK(hipGetDevice(&dev));
    if (dev < 0 || dev >= MAX_DEVICES) return KV_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> guard(lock);
    if (!ptr_of_device[dev]) {
        float *p = nullptr;
        KV_HIP_CHECK(hipGetSymbolAddress(reinterpret_cast<void **>(&p), HIP_SYMBOL(scratch)));
        if (!p) return KV_ERR_HIP;
        ptr_of_device[dev] = p;
    }
    *out = ptr_of_device[dev];
    return KV_OK;
}

int launch_v_matvec_noalloc(const kv_cache *c, const float *p, int64_t ld_p, float *out, hipStream_t s) {
    float *partial = nullptr;
    const int rc = scratch_of_current_device(&partial);
    if (rc != KV_OK) return rc;
    // every split row that the combine kernel reads is written in full by the stream kernel of
    // the same call: nothing in the array has to start at zero
    return launch_v_matvec_into(c, p, ld_p, out, partial, KV_NOALLOC_MAX_SPLIT_ROWS, COUNT_V_NOALLOC, s);
}

}  // namespace packkv
