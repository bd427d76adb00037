// Fused decode attention over the packed cache: Att(q, K, V) = softmax(sm_scale * K q)^T V
// (definition in PackKV Sec. III-B.3) in one pass, with the per-chunk K and V work of
// Sec. III-C.1 / III-C.2 (k_planes.h, v_planes.h; pack8.h) and an online softmax in between, so the
// fp32 scores and probabilities never travel through HBM.
//
// A wave walks blocks of one (batch, kv-head) stream.  Per block it unpacks the K chunk
// into the 64 scores of the block (lane = token), turns them into weights
// p_t = 2^(s_t - m_ref) against a wave-uniform reference m_ref per head, and feeds the V
// chunk of the same block with them.  m_ref is only raised when some score exceeds it by
// more than 8 (in log2 units): then the exact wave maximum becomes the new reference and
// all running sums are rescaled once.  Weights therefore stay below 2^8, inside the range
// the V operand's weight split represents, and a reference below the true
// maximum cancels in the final division.  The wave holds one K and one V chunk buffer:
// the V chunk streams in while K is unpacked, the next K chunk while V is unpacked.
//
// The context axis is split over workgroups.  Each wave ends with (m_ref, l = sum p,
// o[128]) per head; the four waves of a workgroup and then the splits are merged in a
// fixed order with the usual 2^(m_i - M) factors by attn_combine_kernel, which also
// handles the raw fp16 tail.  No floating-point atomics: bitwise reproducible.
#include <algorithm>

#include "k_planes.h"
#include "last_group.h"
#include "pack8.h"
#include "v_chunk.h"
#include "v_planes.h"

namespace packkv {

constexpr float LOG2E = 1.4426950408889634f;
constexpr float RAISE_MARGIN = 8.0f;  // log2 units a score may exceed the reference by
constexpr int A_L = D;                // partial row: [0..127] outputs, [128] sum of weights,
constexpr int A_M = D + 1;            // [129] reference exponent (log2 units)

struct AArgs {
    const uint8_t *k_arena, *v_arena;
    const uint32_t *k_index, *v_index;
    const uint32_t *k_meta, *v_meta;  // [B][meta_stride]
    const __half *q;                  // [B][Hq][128]
    float *partial;                   // [row sets][G][V_PART_STRIDE], see FlatPlan
    int64_t meta_stride;
    int B, H;
    int index_words;        // index words per chunk: 1 back to back, 2 with a paged arena
    int dup;                // H counts every kv-head dup times (query groups above 8 are split): kv-head = h / dup
    int n_blocks;                     // packed blocks per stream
    int blocks_per_split;             // not FLAT: blocks of a workgroup
    float sm_log2;                    // sm_scale * log2(e)
    // MERGE: the last workgroup of a stream merges its rows (else attn_combine_kernel does)
    uint8_t *counters;      // of stream 0, a word per stream
    const __half *k_tail, *v_tail;
    int n_tail, tail_cap;
    float *out;
};

// Maximum over the 64 lanes of a wave, in every lane (see wave_all_sum).
__device__ inline float wave_all_max(float v) {
    uint32_t a = __float_as_uint(v), b = a;
    swap_rows32(a, b);
    v = fmaxf(__uint_as_float(a), __uint_as_float(b));
    a = b = __float_as_uint(v);
    swap_rows16(a, b);
    v = fmaxf(__uint_as_float(a), __uint_as_float(b));
    v = fmaxf(v, dpp_f32<DPP_ROW_ROR8>(v));
    v = fmaxf(v, dpp_f32<DPP_ROW_ROR4>(v));
    v = fmaxf(v, dpp_f32<DPP_QUAD_XOR2>(v));
    return fmaxf(v, dpp_f32<DPP_QUAD_XOR1>(v));
}

// 2^(a - b) with the convention that an empty side (a = -inf) weighs nothing.
__device__ inline float exp2_diff(float a, float b) { return a == -INFINITY ? 0.0f : exp2f(a - b); }

// Online softmax bookkeeping: raise a head's reference only when a score of this block runs
// away from it, and rescale the running sums then.  s: this lane's scores (log2 units).
template <int G, bool FOLD>
__device__ inline void attn_raise_reference(const float (&s)[G], float (&m_ref)[G], float (&l_lane)[G],
                                            VState<G, FOLD> &st, int col) {
    bool raise = false;
#pragma unroll
    for (int g = 0; g < G; ++g) raise |= s[g] > m_ref[g] + RAISE_MARGIN;
    if (__builtin_amdgcn_ballot_w64(raise) != 0) {
        float alpha_col = 1.0f;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            // the same value in every lane: keep it in a scalar register
            const float m_new = __int_as_float(__builtin_amdgcn_readfirstlane(
                __float_as_int(fmaxf(m_ref[g], wave_all_max(s[g])))));
            const float alpha = exp2_diff(m_ref[g], m_new);
            m_ref[g] = m_new;
            l_lane[g] *= alpha;
            st.pm[g] *= alpha;
            if constexpr (!FOLD) {
#pragma unroll
                for (int j = 0; j < 8; ++j) st.macc[g][j] *= alpha;
            }
            if ((col >> 1) == g) alpha_col = alpha;
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) st.acc[j] *= alpha_col;
    }
}

// The same for the running sums of the plane-layout V phase (v_planes.h): the result tiles hold
// one digit of one head per column.
template <int G>
__device__ inline void attn_raise_reference(const float (&s)[G], float (&m_ref)[G], float (&l_lane)[G],
                                            VPlaneState<G> &st, int col) {
    bool raise = false;
#pragma unroll
    for (int g = 0; g < G; ++g) raise |= s[g] > m_ref[g] + RAISE_MARGIN;
    if (__builtin_amdgcn_ballot_w64(raise) != 0) {
        float alpha_col = 1.0f;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const float m_new = __int_as_float(__builtin_amdgcn_readfirstlane(
                __float_as_int(fmaxf(m_ref[g], wave_all_max(s[g])))));
            const float alpha = exp2_diff(m_ref[g], m_new);
            m_ref[g] = m_new;
            l_lane[g] *= alpha;
            st.pm[g] *= alpha;
#pragma unroll
            for (int j = 0; j < 8; ++j) st.macc[g][j] *= alpha;
            if (col / v_pieces<G>() == g) alpha_col = alpha;
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) st.acc[j] *= alpha_col;
    }
}

template <int G, bool FOLD>
__device__ inline void attn_store_state(const VState<G, FOLD> &st, float (*red)[D + 4], int lane, float code_scale) {
    v_state_store<G, false>(st, red, lane, code_scale);
}
template <int G>
__device__ inline void attn_store_state(const VPlaneState<G> &st, float (*red)[D + 4], int lane, float) {
    v_planes_store<G>(st, red, lane);
}

// End of a workgroup's part of a stream: merges the four waves' running sums (each with its own
// softmax reference) and writes the partial rows.  red aliases the chunk buffers (a caller that fills them
// again passes a barrier first).
template <int G, bool MERGE, class State>
__device__ inline void attn_store_partial(const AArgs &a, const State &st, const float (&l_lane)[G],
                                          const float (&m_ref)[G], float (*red)[G][D + 4], int wave,
                                          int lane, int64_t row_set,
                                          float code_scale = CODE_SCALE_LIFTED) {
    __syncthreads();  // every wave is done with its chunk buffers: reuse them as red[][][]

    attn_store_state<G>(st, red[wave], lane, code_scale);
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const float l = wave_all_sum(l_lane[g]);
        if (lane == 0) {
            red[wave][g][D + 1] = l;
            red[wave][g][D + 2] = m_ref[g];
        }
    }
    __syncthreads();
    // four outputs to a thread
    if (threadIdx.x < G * (D / 4)) {
        const int g = threadIdx.x / (D / 4), d4 = threadIdx.x % (D / 4);
        const float m0 = red[0][g][D + 2], m1 = red[1][g][D + 2], m2 = red[2][g][D + 2], m3 = red[3][g][D + 2];
        const float M = fmaxf(fmaxf(m0, m1), fmaxf(m2, m3));
        const float f[4] = {exp2_diff(m0, M), exp2_diff(m1, M), exp2_diff(m2, M), exp2_diff(m3, M)};
        float4 o[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            // outputs carry the per-head sum p*min term
            const float4 x = *reinterpret_cast<const float4 *>(&red[w][g][4 * d4]);
            const float pmin = red[w][g][D];
            o[w] = make_float4(f[w] * (x.x + pmin), f[w] * (x.y + pmin), f[w] * (x.z + pmin), f[w] * (x.w + pmin));
        }
        float *dst = a.partial + (row_set * G + g) * V_PART_STRIDE;
        const float4 sum = make_float4((o[0].x + o[1].x) + (o[2].x + o[3].x), (o[0].y + o[1].y) + (o[2].y + o[3].y),
                                       (o[0].z + o[1].z) + (o[2].z + o[3].z), (o[0].w + o[1].w) + (o[2].w + o[3].w));
        const float l = (f[0] * red[0][g][D + 1] + f[1] * red[1][g][D + 1]) + (f[2] * red[2][g][D + 1] + f[3] * red[3][g][D + 1]);
        if constexpr (MERGE) {
            store_shared(dst + 4 * d4, sum.x, sum.y);
            store_shared(dst + 4 * d4 + 2, sum.z, sum.w);
            if (d4 == 0) store_shared(dst + A_L, l, M);
        } else {
            *reinterpret_cast<float4 *>(dst + 4 * d4) = sum;
            if (d4 == 0) *reinterpret_cast<float2 *>(dst + A_L) = make_float2(l, M);
        }
    }
}

// The last workgroup of a stream: merges its n_sets row sets and the raw fp16 tail, by attn_combine_kernel's formulas in an
// order of its own, a wave, or with one or two heads several waves, per query head.  flag, scratch: a word and 4 * 256 floats of LDS that
// nothing else uses any more.
template <int G>
__device__ inline void attn_merge_stream(const AArgs &a, int stream, int b, int h, int n_sets, int64_t set_stride, uint32_t *flag,
                                         float *scratch) {
    if (!last_group(a.counters + 4 * stream, uint32_t(n_sets), flag)) return;
    constexpr int W = G == 1 ? 4 : G == 2 ? 2 : 1;   // waves per head: each takes every W-th row set and 64 / W tail tokens
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), part = wave % W;
    float *const weights = scratch + 256 * wave, *const sums = weights + 64;
    const int kvh = h / a.dup, Hkv = a.H / a.dup;
    const int sets = (n_sets - part + W - 1) / W, tail0 = part * (N / W), n_tail = max(0, min(a.n_tail - tail0, N / W));
    for (int g = wave / W; g < G; g += 4 / W) {
        const int64_t row = int64_t(stream) * G + g;
        const int64_t stride = set_stride * G * V_PART_STRIDE;
        const float *first = a.partial + row * V_PART_STRIDE + part * stride;
        const int64_t tail_at = ((int64_t(b) * a.tail_cap + tail0) * Hkv + kvh) * D;
        RowSum rows;
        TailSum tail;
        rows.load(first, W * stride, 0, sets, lane);
        float2 lm = make_float2(0.0f, -INFINITY);
        if (lane < sets) lm = load_shared(first + lane * W * stride + A_L);
        if (n_tail > 0) {
            tail.load(a.v_tail + tail_at, int64_t(Hkv) * D, 0, n_tail, lane);
            // scores: four lanes per token, 32 channels each, sixteen tokens at a time
            const __half *q = a.q + row * D + 32 * (lane & 3);
            uint4 qr[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) qr[c] = *reinterpret_cast<const uint4 *>(q + 8 * c);
#pragma unroll 1
            for (int t0 = 0; t0 < n_tail; t0 += 16) {
                const int t = t0 + (lane >> 2);
                float s = 0.0f;
                if (t < n_tail) {
                    const __half *krow = a.k_tail + tail_at + int64_t(t) * Hkv * D + 32 * (lane & 3);
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const uint4 kr = *reinterpret_cast<const uint4 *>(krow + 8 * c);
                        const __half *kk = reinterpret_cast<const __half *>(&kr), *qq = reinterpret_cast<const __half *>(&qr[c]);
#pragma unroll
                        for (int e = 0; e < 8; ++e) s = fmaf(__half2float(kk[e]), __half2float(qq[e]), s);
                    }
                }
                s += dpp_f32<DPP_QUAD_XOR1>(s);
                s += dpp_f32<DPP_QUAD_XOR2>(s);
                if ((lane & 3) == 0) weights[t] = a.sm_log2 * s;
            }
            wave_lds_fence();
        }
        const float my_tail = lane < n_tail ? weights[lane] : -INFINITY;
        float M = wave_all_max(fmaxf(lm.y, my_tail));
        if constexpr (W > 1) {   // the waves of a head agree on its reference
            if (lane == 0) sums[128] = M;
            __syncthreads();
#pragma unroll
            for (int w = 0; w < W; ++w) M = fmaxf(M, scratch[256 * (wave - part + w) + 192]);
        }
        const float f = lane < sets ? exp2_diff(lm.y, M) : 0.0f, w = lane < n_tail ? exp2f(my_tail - M) : 0.0f;
        float l = wave_all_sum(fmaf(f, lm.x, w));
        float2 o = rows.sum(first, W * stride, sets, f, lane);
        if (n_tail > 0) {
            weights[lane] = w;
            wave_lds_fence();
            const float2 t = tail.sum(a.v_tail + tail_at, int64_t(Hkv) * D, weights, n_tail, sums, lane);
            o.x += t.x, o.y += t.y;
        }
        if constexpr (W > 1) {
            *reinterpret_cast<float2 *>(sums + 2 * lane) = o;
            if (lane == 0) sums[129] = l;
            __syncthreads();
            if (part != 0) continue;
            o = make_float2(0.0f, 0.0f), l = 0.0f;
#pragma unroll
            for (int p = 0; p < W; ++p) {
                const float *theirs = sums + 256 * p;
                const float2 v = *reinterpret_cast<const float2 *>(theirs + 2 * lane);
                o.x += v.x, o.y += v.y, l += theirs[129];
            }
        }
        const bool some = l > 0.0f;  // every block dropped and no tail: defined output
        *reinterpret_cast<float2 *>(a.out + row * D + 2 * lane) = make_float2(some ? o.x / l : 0.0f, some ? o.y / l : 0.0f);
    }
}

// SOLO: a workgroup has its stream to itself, tail included.  Wave w of WAVES takes the tail's tokens 64 / WAVES * w ..; their K and V values
// are loaded ahead of the first chunks and stay in registers.
template <int G, int WAVES>
struct SoloTail {
    static constexpr int PER = N / WAVES, SEGS = 64 / PER, CH = D / SEGS;   // tokens to a wave; K: lanes to a token, channels to a lane
    uint4 k[CH / 8], v[PER / 4];                                            // V: token lane / 16 + 4 i, channels 8 (lane % 16) ..
    __device__ inline void load(const AArgs &a, int b, int h, int wave, int lane) {
        const int Hkv = a.H / a.dup;
        const int64_t at = ((int64_t(b) * a.tail_cap + PER * wave) * Hkv + h / a.dup) * D, step = int64_t(Hkv) * D;
        const int left = a.n_tail - PER * wave;
        const __half *krow = a.k_tail + at + (lane / SEGS) * step + CH * (lane % SEGS);
        const __half *vrow = a.v_tail + at + (lane >> 4) * step + 8 * (lane & 15);
#pragma unroll
        for (int c = 0; c < CH / 8; ++c) {
            k[c] = make_uint4(0, 0, 0, 0);
            if (lane / SEGS < left) k[c] = *reinterpret_cast<const uint4 *>(krow + 8 * c);
        }
#pragma unroll
        for (int i = 0; i < PER / 4; ++i) {
            v[i] = make_uint4(0, 0, 0, 0);
            if ((lane >> 4) + 4 * i < left) v[i] = *reinterpret_cast<const uint4 *>(vrow + 4 * i * step);
        }
    }
    __device__ inline void consume() {
#pragma unroll
        for (int c = 0; c < CH / 8; ++c) consume_here(k[c].x), consume_here(k[c].y), consume_here(k[c].z), consume_here(k[c].w);
#pragma unroll
        for (int i = 0; i < PER / 4; ++i) consume_here(v[i].x), consume_here(v[i].y), consume_here(v[i].z), consume_here(v[i].w);
    }
    // Adds the wave's tail tokens to its rows red[g] (outputs), l[g], m[g] of every head; q: the G heads' queries, in LDS;
    // weights: 64 floats of LDS.
    __device__ inline void add(const AArgs &a, const __half *q, float (*red)[D + 4], const float (&l_lane)[G], const float (&m_ref)[G],
                               float *weights, int wave, int lane) {
        const int left = a.n_tail - PER * wave;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            float l = wave_all_sum(l_lane[g]), m = m_ref[g];
            float2 *const row = row_sums8_place(red[g], lane);
            if (left > 0) {
                float s = 0.0f;
#pragma unroll
                for (int c = 0; c < CH / 8; ++c) {
                    const uint4 qv = *reinterpret_cast<const uint4 *>(q + g * D + CH * (lane % SEGS) + 8 * c);
                    const __half *kk = reinterpret_cast<const __half *>(&k[c]), *qq = reinterpret_cast<const __half *>(&qv);
#pragma unroll
                    for (int e = 0; e < 8; ++e) s = fmaf(__half2float(kk[e]), __half2float(qq[e]), s);
                }
                s += dpp_f32<DPP_QUAD_XOR1>(s);
                s += dpp_f32<DPP_QUAD_XOR2>(s);
                if constexpr (SEGS == 8) s += dpp_f32<DPP_ROW_HALF_MIRROR>(s);
                const bool some = lane / SEGS < left;
                s = some ? a.sm_log2 * s : -INFINITY;   // in all lanes of its token
                const float M = fmaxf(m, wave_all_max(s)), f = exp2_diff(m, M);
                const float w = exp2_diff(s, M);   // (M too is -inf where the wave has no block and only such tokens)
                if (lane % SEGS == 0) weights[lane / SEGS] = w;
                wave_lds_fence();
                l = fmaf(f, l, wave_all_sum(lane % SEGS == 0 ? w : 0.0f));
                m = M;
                float acc[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[e] = 0.0f;
#pragma unroll
                for (int i = 0; i < PER / 4; ++i) {
                    const __half *hv = reinterpret_cast<const __half *>(&v[i]);
                    const float wt = weights[(lane >> 4) + 4 * i];
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc[e] = fmaf(wt, __half2float(hv[e]), acc[e]);
                }
                const float2 two = row_sums8(acc);
                const float pmin = red[g][D];
                wave_lds_fence();
                const float2 before = *row;
                *row = make_float2(fmaf(f, before.x + pmin, two.x), fmaf(f, before.y + pmin, two.y));
                if (lane == 0) red[g][D] = 0.0f;
                wave_lds_fence();
            }
            if (lane == 0) red[g][D + 1] = l, red[g][D + 2] = m;
        }
    }
};

// The waves' rows of a stream, tail included, to its outputs.
template <int G, int WAVES>
__device__ inline void attn_solo_store(const AArgs &a, const float (*red)[G][D + 4], int64_t head0) {
    for (int i = threadIdx.x; i < G * D / 2; i += 64 * WAVES) {
        const int g = i / (D / 2), d = 2 * (i % (D / 2));
        float M = red[0][g][D + 2];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) M = fmaxf(M, red[w][g][D + 2]);
        float x = 0.0f, y = 0.0f, l = 0.0f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            const float f = exp2_diff(red[w][g][D + 2], M), pmin = red[w][g][D];
            const float2 v = *reinterpret_cast<const float2 *>(&red[w][g][d]);
            x = fmaf(f, v.x + pmin, x), y = fmaf(f, v.y + pmin, y), l = fmaf(f, red[w][g][D + 1], l);
        }
        const bool some = l > 0.0f;  // every block dropped and no tail: defined output
        *reinterpret_cast<float2 *>(a.out + (head0 + g) * D + d) = make_float2(some ? x / l : 0.0f, some ? y / l : 0.0f);
    }
}

// HIGH: the V codes of the cache may need four bits (a plane H exists).  The blocks of all streams form
// one work list cut into equal ranges, one per workgroup and one round of resident workgroups
// (FlatPlan), so no last round runs nearly empty; a workgroup whose range crosses a stream
// boundary writes a partial row set per stream.
// SOLO > 0: a workgroup of that many waves to a stream, which does it all: no partial rows through memory, no counter and no
// second kernel (solo_waves says where).
template <int G, bool HIGH, bool FLAT, bool MERGE, int SOLO = 0>
__global__ __launch_bounds__(SOLO ? 64 * SOLO : 256) void attn_kernel(AArgs a, FlatPlan plan) {
    constexpr int WAVES = SOLO ? SOLO : 4;
    static_assert(!SOLO || (!FLAT && !MERGE), "a stream of its own needs neither");
    // per wave: buffer 0 holds the K chunk (and then its tiles, k_planes.h), buffer 1 the V chunk of
    // the block in flight; between two streams the same memory holds the cross-wave reduction array
    // red[4][G][D + 4].  (A second K buffer, the next K chunk on its way while one is decoded: 41.7 -> 42.6 us for
    // 4 x 8 streams of 512 blocks at four heads, 69.3 -> 75.9 for twice as many: two workgroups per compute unit, not three.)
    __shared__ __attribute__((aligned(16))) uint8_t lds_all[WAVES * 2 * CHUNK_LDS + LDS_TAIL_PAD];
    constexpr int VB = vb_bytes<G>();
    __shared__ __attribute__((aligned(16))) uint8_t vb_all[WAVES * VB];  // digit staging of the V phase
    __shared__ uint4 ktable[5];                                      // K chunks: plane layout, channel-major
    __shared__ uint4 vtable[PLANE_TABLE_ENTRIES];                    // V chunks: plane layout, group-major
    __shared__ uint32_t vhighs[PLANE_TABLE_ENTRIES];
    __shared__ __attribute__((aligned(16))) __half q_lds[SOLO ? G * D : 8];
    static_assert(sizeof(float) * G * (D + 4) <= 2 * CHUNK_LDS, "reduction array must fit");
    static_assert(K_TILES_BYTES <= CHUNK_LDS && CHUNK_LDS % 16 == 0, "the K tiles are built in the K buffer");
    float(*red)[G][D + 4] = reinterpret_cast<float(*)[G][D + 4]>(lds_all);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int grp = blockIdx.x;
    const int col = lane & 15;
    const int kbuf = wave * 2 * CHUNK_LDS, vbuf = kbuf + CHUNK_LDS;
    uint8_t *vb = vb_all + wave * VB;
    bool tables = false;
    const int64_t range_end = FLAT ? plan.begin(grp + 1) : 1;
    SoloTail<G, WAVES> tail;

    for (int64_t f = FLAT ? plan.begin(grp) : 0; f < range_end;) {
        FlatPlan::Segment seg;
        int64_t row_set;
        if constexpr (FLAT) {
            seg = plan.segment(f, range_end);
            row_set = int64_t(grp) + seg.stream;
            f += seg.blk_end - seg.blk_begin;
        } else {
            seg.stream = blockIdx.y;
            seg.b = seg.stream / a.H, seg.h = seg.stream % a.H;
            seg.blk_begin = grp * a.blocks_per_split;
            seg.blk_end = min(seg.blk_begin + a.blocks_per_split, a.n_blocks);
            row_set = int64_t(grp) * gridDim.y + seg.stream;
            f = 1;
        }
        const int stream = seg.stream, b = seg.b, h = seg.h, blk_begin = seg.blk_begin, blk_end = seg.blk_end;
        const int64_t head0 = int64_t(stream) * G;

        KQueryPlanes<G> kq;
        kq.fetch(a.q + head0 * D, lane);
        VPlaneState<G> st;
        st.clear();
        float m_ref[G], l_lane[G];
#pragma unroll
        for (int g = 0; g < G; ++g) m_ref[g] = -INFINITY, l_lane[g] = 0.0f;

        IndexBatch ik, iv;
        uint32_t kmt_next = 0, vmt_next = 0;
        // index words of up to 64 blocks of this wave
        auto load_index = [&](int first) {
            if (first >= blk_end) return;
            ik.load(a.k_index, a.index_words, first, WAVES, blk_end, a.B, a.H / a.dup, b, h / a.dup, lane);
            iv.load(a.v_index, a.index_words, first, WAVES, blk_end, a.B, a.H / a.dup, b, h / a.dup, lane);
            const int64_t tok0 = b * a.meta_stride + int64_t(first) * N + lane;
            kmt_next = a.k_meta[tok0], vmt_next = a.v_meta[tok0];
        };
        // the chunks of block `it` of the batch
        auto issue_k = [&](int it) {
            chunk_issue_lds<CHUNK_MAX, HEADER, true>(a.k_arena, ik.start16(it), ik.end16(it), lds_all + kbuf, lane);
        };
        auto issue_v = [&](int it) {
            chunk_issue_lds<CHUNK_MAX, HEADER, true>(a.v_arena, iv.start16(it), iv.end16(it), lds_all + vbuf, lane);
        };
        auto issue_first = [&](int first) {
            if (first >= blk_end) return;
            issue_k(0);
            issue_v(0);
        };
        load_index(blk_begin + wave);
        if constexpr (SOLO > 0) {
            tail.load(a, b, h, wave, lane);
            for (int i = threadIdx.x; i < G * D / 8; i += 64 * WAVES) reinterpret_cast<uint4 *>(q_lds)[i] = reinterpret_cast<const uint4 *>(a.q + head0 * D)[i];
        }
        if (!tables) {  // while the index words are on their way
            for (int i = threadIdx.x; i < WAVES * VB / 4; i += 64 * WAVES) reinterpret_cast<uint32_t *>(vb_all)[i] = 0;
            build_k_plane_table<false>(ktable);
            build_plane_table<false>(vtable, vhighs);
            __syncthreads();
            tables = true;
        }
        issue_first(blk_begin + wave);
        kq.build(lane);  // while the first chunks are on their way
        for (int first = blk_begin + wave; first < blk_end; first += WAVES * 64) {
            const int n_it = min(64, (blk_end - first + WAVES - 1) / WAVES);
            for (int it = 0; it < n_it; ++it) {
                // a block dropped by an arena overflow (in either tensor) takes no part
                const bool valid = ik.end16(it) - ik.start16(it) >= uint32_t(HEADER / 16) &&
                                   iv.end16(it) - iv.start16(it) >= uint32_t(HEADER / 16);
                wait_chunk_landed();  // K chunk of this block
                uint32_t kmt = kmt_next, vmt = vmt_next;
                consume_here(kmt), consume_here(vmt);
                if constexpr (SOLO > 0) {
                    if (it == 0) tail.consume();
                }
                if (it > 0) {
                    lds_reads_returned();  // the previous V chunk has been read completely
                    issue_v(it);
                }
                if (it + 1 < n_it) {
                    const int64_t tok = b * a.meta_stride + int64_t(first + WAVES * (it + 1)) * N + lane;
                    kmt_next = a.k_meta[tok];
                    vmt_next = a.v_meta[tok];
                }

                float s[G];  // scores of token `lane` in log2 units
                if (valid) {
                    float u[G];
                    k_planes_chunk<G>(lds_all, kbuf, ktable, lds_all + kbuf, kq, u, []() {});
                    const float kscale = __half2float(__ushort_as_half(uint16_t(kmt & 0xFFFFu)));
                    const float kmn = __half2float(__ushort_as_half(uint16_t(kmt >> 16)));
#pragma unroll
                    for (int g = 0; g < G; ++g) s[g] = a.sm_log2 * fmaf(kscale, u[g], kmn * kq.qsum[g]);

                    attn_raise_reference<G>(s, m_ref, l_lane, st, col);
                }
                wait_chunk_landed();  // V chunk of this block
                lds_reads_returned();  // the K tiles have been read completely before the next chunk overwrites them
                if (it + 1 < n_it) issue_k(it + 1);
                if (!valid) continue;
                float pt[G];
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    pt[g] = exp2f(s[g] - m_ref[g]);  // subnormals too: they are the output where larger weights meet values of 0
                    l_lane[g] += pt[g];
                }
                v_planes_chunk<G, HIGH>(lds_all, vbuf, vtable, vhighs, vb, vmt, pt, st);
            }
            wait_chunk_landed();
            lds_reads_returned();  // the last V chunk has been read before the next batch's first overwrites it
            load_index(first + WAVES * 64);
            issue_first(first + WAVES * 64);
        }
        if constexpr (SOLO > 0) {
            __syncthreads();  // every wave is done with its chunk buffers: reuse them as red[][][]
            attn_store_state<G>(st, red[wave], lane, 0.0f);
            wave_lds_fence();
            tail.add(a, q_lds, red[wave], l_lane, m_ref, reinterpret_cast<float *>(vb), wave, lane);
            __syncthreads();
            attn_solo_store<G, WAVES>(a, red, head0);
            return;
        }
        attn_store_partial<G, MERGE>(a, st, l_lane, m_ref, red, wave, lane, row_set);
        if constexpr (FLAT)
            __syncthreads();  // red[][][] has been read: the buffers may be filled again
        else if constexpr (MERGE)
            attn_merge_stream<G>(a, stream, b, h, gridDim.x, gridDim.y, reinterpret_cast<uint32_t *>(vhighs),
                                 reinterpret_cast<float *>(lds_all));
    }
}

// The same for chunks with packs of 8 tokens (Sec. IV-B; pack8.h): the K phase runs the
// pairwise dot-product form for all G heads and leaves lane l with token
// k8_token_of_block_lane(l) of the block; the V phase stages the weights in that order.
// KW / VW: that tensor uses the wide chunk layout (codes above 15); the two tensors choose
// their layout independently, and a wide chunk needs a buffer twice as large.  With both wide,
// two buffers per wave would leave room for one workgroup per compute unit only (measured 0.76 ms
// at the headline shape, slower than the three-step path); the K and the V chunk then take turns
// in ONE buffer, transfers overlap with the unpacking of other waves only, and three workgroups
// fit.  MID: no code above 31 in a wide tensor, so that a chunk fits a smaller buffer and K and V have
// one each (two workgroups per compute unit).  The transfers carry the non-temporal hint, as those of the plane layout do: with the cache read from memory
// 29.6 -> 28.4 us (4 x 8 streams of 156 blocks, four heads), 35.1 -> 33.0 (2 x 32 of 127, both tensors wide).
// (Three waves per SIMD where the buffers leave room for them, two with more heads.)
template <int G, bool KW, bool VW, bool MID, bool MERGE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(G <= 4 && KW == VW && !MID ? 3 : 2))) void attn8_kernel(AArgs a, VCentre centre) {
    constexpr bool SHARED = KW && VW && !MID;
    constexpr int WLDS = MID ? CHUNKM_LDS : CHUNKW_LDS, WMAX = MID ? CHUNKM_MAX : CHUNKW_MAX;
    constexpr int KLDS = KW ? WLDS : CHUNK8_LDS, VLDS = SHARED ? 0 : (VW ? WLDS : CHUNK8_LDS);
    constexpr int KMAX = KW ? WMAX : CHUNK8_MAX, VMAX = VW ? WMAX : CHUNK8_MAX;
    constexpr int KHDR = KW ? HEADERW : HEADER8, VHDR = VW ? HEADERW : HEADER8;
    __shared__ __attribute__((aligned(16))) uint8_t lds_all[4 * (KLDS + VLDS) + LDS_TAIL_PAD];
    __shared__ __attribute__((aligned(16))) uint8_t blds_all[4 * BLds<G>::BYTES];
    __shared__ uint2 table[KW ? 16 : PACK_TABLE_ENTRIES];   // K: the wide K table, or the pair table
    __shared__ uint4 vtable[VW ? 16 : PACK_TABLE_ENTRIES];  // V: the wide V table, or lifted codes
    static_assert(sizeof(float) * 4 * G * (D + 4) <= 4 * (KLDS + VLDS), "reduction array must fit");
    static_assert(WIDE_TABLE_ENTRIES <= 16, "table sizes above");
    float(*red)[G][D + 4] = reinterpret_cast<float(*)[G][D + 4]>(lds_all);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int split = blockIdx.x;
    const int bh = blockIdx.y;
    const int h = bh % a.H, b = bh / a.H;
    const int col = lane & 15;
    const int kbuf = wave * (KLDS + VLDS), vbuf = SHARED ? kbuf : kbuf + KLDS;
    const int64_t head0 = int64_t(b) * a.H * G + h * G;
    const int tok_in_blk = k8_token_of_block_lane(lane);

    const int blk_begin = split * a.blocks_per_split;
    const int blk_end = min(blk_begin + a.blocks_per_split, a.n_blocks);
    IndexBatch ik, iv;
    auto load_index = [&](int first) {
        if (first >= blk_end) return;
        ik.load(a.k_index, a.index_words, first, 4, blk_end, a.B, a.H / a.dup, b, h / a.dup, lane);
        iv.load(a.v_index, a.index_words, first, 4, blk_end, a.B, a.H / a.dup, b, h / a.dup, lane);
    };
    load_index(blk_begin + wave);
    // while the index words are on their way
    if constexpr (!KW) build_pair_table(table);
    if constexpr (!VW) build_pack_table(vtable, CODE_LIFT, fold_min<G>());
    if constexpr (KW || VW) build_wide_tables(KW ? table : nullptr, VW ? vtable : nullptr);
    KQuery8<G> kq;
    kq.load(a.q + head0 * D, lane);
    VLane<G> vl;
    vl.init(blds_all + wave * BLds<G>::BYTES, lane);
    vl.bslot = v8_bslot<G>(tok_in_blk);
    VState<G, VW || fold_min<G>()> st;
    st.clear();
    float m_ref[G], l_lane[G];
#pragma unroll
    for (int g = 0; g < G; ++g) m_ref[g] = -INFINITY, l_lane[g] = 0.0f;

    for (int first = blk_begin + wave; first < blk_end; first += 4 * 64) {
        const int n_it = min(64, (blk_end - first + 3) / 4);
        chunk_issue_lds<KMAX, KHDR, true>(a.k_arena, ik.start16(0), ik.end16(0), lds_all + kbuf, lane);
        const int64_t tok0 = b * a.meta_stride + int64_t(first) * N + tok_in_blk;
        uint32_t kmt_next = a.k_meta[tok0], vmt_next = a.v_meta[tok0];
        for (int it = 0; it < n_it; ++it) {
            // a block dropped by an arena overflow (in either tensor) takes no part
            const bool valid = ik.end16(it) - ik.start16(it) >= uint32_t(KHDR / 16) &&
                               iv.end16(it) - iv.start16(it) >= uint32_t(VHDR / 16);
            wait_chunk_landed();  // K chunk of this block
            uint32_t kmt = kmt_next, vmt = vmt_next;
            consume_here(kmt), consume_here(vmt);
            if constexpr (!SHARED) {
                lds_reads_returned();  // the previous V chunk has been read completely
                chunk_issue_lds<VMAX, VHDR, true>(a.v_arena, iv.start16(it), iv.end16(it), lds_all + vbuf, lane);
            }
            if (it + 1 < n_it) {
                const int64_t tok = b * a.meta_stride + int64_t(first + 4 * (it + 1)) * N + tok_in_blk;
                kmt_next = a.k_meta[tok];
                vmt_next = a.v_meta[tok];
            }

            float s[G];  // scores of this lane's token in log2 units
            if (valid) {
                float u0[G], u1[G];
                if constexpr (KW) {
                    kw_chunk<G>(lds_all, kbuf, table, kq, lane, u0, u1);
                } else {
                    const uint2 hdr0 = *reinterpret_cast<const uint2 *>(lds_all + kbuf + lane * 8);
                    LanePacks8 lp0;
                    lp0.init(hdr0.x, hdr0.y, kbuf + HEADER8);
                    k8_half<G>(lds_all, table, lp0, kq, lane, u0);
                    const uint2 hdr1 = *reinterpret_cast<const uint2 *>(lds_all + kbuf + 512 + lane * 8);
                    LanePacks8 lp1;
                    lp1.init(hdr1.x, hdr1.y, lp0.end_all);
                    k8_half<G>(lds_all, table, lp1, kq, lane, u1);
                }
                const float kscale = __half2float(__ushort_as_half(uint16_t(kmt & 0xFFFFu)));
                const float kmn = __half2float(__ushort_as_half(uint16_t(kmt >> 16)));
#pragma unroll
                for (int g = 0; g < G; ++g)
                    s[g] = a.sm_log2 * fmaf(kscale, (lane & 1) ? u1[g] : u0[g], kmn * kq.qsum[g]);
                attn_raise_reference<G>(s, m_ref, l_lane, st, col);
            }
            if constexpr (SHARED) {
                // one buffer: the K chunk has been read completely before the V chunk overwrites it
                lds_reads_returned();
                chunk_issue_lds<VMAX, VHDR, true>(a.v_arena, iv.start16(it), iv.end16(it), lds_all + vbuf, lane);
            }
            wait_chunk_landed();  // V chunk of this block
            if constexpr (!SHARED) {
                lds_reads_returned();  // the K chunk has been read completely before the next one overwrites it
                if (it + 1 < n_it)
                    chunk_issue_lds<KMAX, KHDR, true>(a.k_arena, ik.start16(it + 1), ik.end16(it + 1), lds_all + kbuf, lane);
            }
            if (valid) {
                float pt[G];
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    pt[g] = exp2f(s[g] - m_ref[g]);  // subnormals too: they are the output where larger weights meet values of 0
                    l_lane[g] += pt[g];
                }
                if constexpr (VW)
                    vw_chunk<G>(lds_all, vbuf, vtable, vl, vmt, pt, centre, st);
                else
                    v8_chunk<G, true>(lds_all, vbuf, vtable, vl, vmt, pt, st);
            }
            if constexpr (SHARED) {
                lds_reads_returned();
                if (it + 1 < n_it)
                    chunk_issue_lds<KMAX, KHDR, true>(a.k_arena, ik.start16(it + 1), ik.end16(it + 1), lds_all + kbuf, lane);
            }
        }
        wait_chunk_landed();
        load_index(first + 4 * 64);
    }
    // wide V codes enter the matrix cores as the numbers themselves
    attn_store_partial<G, MERGE>(a, st, l_lane, m_ref, red, wave, lane, int64_t(split) * gridDim.y + bh, VW ? 1.0f : CODE_SCALE_LIFTED);
    if constexpr (MERGE)
        attn_merge_stream<G>(a, bh, b, h, gridDim.x, gridDim.y, reinterpret_cast<uint32_t *>(table), reinterpret_cast<float *>(lds_all));
}

// Merges the splits of one (batch, query head) row in a fixed order and adds the raw fp16
// tail tokens (Sec. III-B.1 buffer), whose scores are plain dot products.
// FLAT: the rows lie as a flat plan wrote them.  A form of its own: reading the plan in front of the first
// address cost every launch without one 0.2-0.3 us.
// Bound by its chain of latencies.  Whole fused attention, 1 x 32 streams of 4096 tokens and a tail of 0 / 8 / 24 /
// 62 tokens, replayed: references and weight sums walked element by element from LDS 13.3 / 14.4 / 14.6 / 16.5 us,
// across the lanes with shuffles 13.6 / 14.7 / 14.5 / 15.6, with row swaps and DPP, a barrier less and the
// tail's weight sum at the end 13.2 / 14.4 / 14.2 / 15.3.
template <bool FLAT>
__global__ __launch_bounds__(256) void attn_combine_kernel(const float *__restrict__ partial,
                                                           int n_splits, int n_rows, FlatPlan plan,
                                                           const __half *__restrict__ q,
                                                           const __half *__restrict__ k_tail,
                                                           const __half *__restrict__ v_tail,
                                                           int n_tail, int tail_cap, int H, int G,
                                                           float sm_log2, float *__restrict__ out) {
    __shared__ float st[N], tw[N];                        // tail scores (log2 units), tail weights
    __shared__ float ms[V_SPLITS_MAX], mf[V_SPLITS_MAX];  // split references, split factors
    __shared__ float red[16][V_PART_STRIDE];
    static_assert(A_L == 128, "the splits' weight sums sit in the column the reduction returns separately");
    const int r = blockIdx.x;           // b*Hq + hq
    const int hq = r % (H * G), b = r / (H * G);
    const int h = hq / G;
    // every global load of the kernel is issued before the first result is needed
    SplitRows rows;
    TailRows trows;
    // the row sets of the row's stream: one per split, or with a flat plan (one head per kv-head: row =
    // stream) those of the workgroups that hold one of its blocks
    int first_row = r, row_stride = n_rows;
    if constexpr (FLAT) {
        const int w_lo = plan.group_of(int64_t(r) * plan.n_blocks);
        const int w_hi = plan.group_of(int64_t(r + 1) * plan.n_blocks - 1);
        n_splits = w_hi - w_lo + 1;
        first_row = w_lo + r;
        row_stride = 1;
    }
    partial += int64_t(first_row) * V_PART_STRIDE;
    rows.load_strided(partial, n_splits, row_stride);
    trows.load(v_tail + (int64_t(b) * tail_cap * H + h) * D, int64_t(H) * D, n_tail);
    if (int(threadIdx.x) < n_splits)
        ms[threadIdx.x] = partial[(int64_t(threadIdx.x) * row_stride) * V_PART_STRIDE + A_M];
    // tail scores: thread (t, seg) takes 32 channels of tail token t, four threads per token
    {
        const int t = threadIdx.x >> 2, seg = threadIdx.x & 3;
        float s = 0.0f;
        if (t < n_tail) {
            const __half *krow = k_tail + ((int64_t(b) * tail_cap + t) * H + h) * D + 32 * seg;
            const __half *qrow = q + int64_t(r) * D + 32 * seg;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const uint4 kr = *reinterpret_cast<const uint4 *>(krow + 8 * c);
                const uint4 qr = *reinterpret_cast<const uint4 *>(qrow + 8 * c);
                const __half *kk = reinterpret_cast<const __half *>(&kr);
                const __half *qq = reinterpret_cast<const __half *>(&qr);
#pragma unroll
                for (int e = 0; e < 8; ++e) s = fmaf(__half2float(kk[e]), __half2float(qq[e]), s);
            }
        }
        s += dpp_f32<DPP_QUAD_XOR1>(s);
        s += dpp_f32<DPP_QUAD_XOR2>(s);
        if (seg == 0 && t < n_tail) st[t] = sm_log2 * s;
    }
    __syncthreads();
    // at most 64 splits and 64 tail tokens: one of each per lane; every wave finds the row's reference by itself
    // (element after element from LDS reference and weight sum took 3 us with 62 tail tokens)
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const float my_split = lane < n_splits ? ms[lane] : -INFINITY, my_tail = lane < n_tail ? st[lane] : -INFINITY;
    const float M = wave_all_max(fmaxf(my_split, my_tail));
    const float tail_weight = lane < n_tail ? exp2f(my_tail - M) : 0.0f;
    if (wave == 0 && lane < n_splits) mf[lane] = exp2_diff(my_split, M);
    if (wave == 1 && lane < n_tail) tw[lane] = tail_weight;
    __syncthreads();
    // weighted sum of the split rows (column 128 = the splits' weight sums), then the tail tokens
    float l;
    float o = rows.sum(n_splits, red, &l, mf);
    if (n_tail > 0) {
        o += trows.sum(tw, n_tail, red);
        l += wave_all_sum(tail_weight);
    }
    const int d = threadIdx.x;
    if (d < D) out[int64_t(r) * D + d] = l > 0.0f ? o / l : 0.0f;  // every block dropped and no tail: defined output
}

// Waves of a workgroup that has a stream to itself, 0: the streams are split.  A solo workgroup saves the way of the partial rows through
// memory and the merge (2 us in the same kernel, 5 with a kernel of its own); against that stands that a stream cannot have more
// than one compute unit.  Eight waves: every stream of up to four blocks; up to 72 where the streams fill three quarters of the
// chip, 16 where they fill half of it.  Beyond one stream to a compute unit, four waves (one head; two workgroups fit): short contexts,
// and up to 56 blocks where two workgroups to a stream would not all be resident.  Split / solo, replayed, us:
// 32 streams, one head, 4 blocks 10.1 / 8.2, 8 blocks 10.2 / 10.2; 128 of 12 13.1 / 11.2, of 16 13.3 / 13.3; 208 of 10 15.2 / 11.2, of 56 28.6 / 26.1;
// 256 of 3, 20, 60, 80, 95 blocks at four heads 13.6 / 11.1, 23.5 / 18.4, 37.6 / 34.9, 45.3 / 43.8, 49.9 / 50.3; 320 of 10 17.4 / 16.5, of 24 22.6 / 24.5;
// 416 of 6, 16, 32, 56 18.5 / 14.0, 23.6 / 19.5, 33.0 / 29.7, 47.5 / 44.7.
static int solo_waves(int n_blocks, int streams, int heads) {
    const int cus = flat_groups_for(int64_t(1) << 40, 1, int64_t(1) << 30);
    if (streams <= cus) return n_blocks <= (4 * streams >= 3 * cus ? 72 : 2 * streams >= cus ? 16 : 4) ? 8 : 0;
    return heads == 1 && streams <= 2 * cus && n_blocks <= (2 * streams > 3 * cus ? 56 : 10) ? 4 : 0;
}

int launch_decode_attention(const kv_cache *c, const __half *q, float sm_scale, float *out, hipStream_t s) {
    // Hs: kv-heads as the stream kernels count them (each dup times, see head_split); the combine
    // kernel works per query head and sees the real kv-head count and the whole group
    const int B = c->cfg.batch, H = c->cfg.n_kv_heads, G = c->group, Hs = H * c->head_split, Gq = G * c->head_split;
    const int n_blocks = int(c->packed_tokens / N);
    uint8_t *ws = static_cast<uint8_t *>(c->buf.workspace);
    float *partial = reinterpret_cast<float *>(ws + WS_VPART);
    const float sm_log2 = sm_scale * LOG2E;
    FlatPlan plan = FlatPlan::make(n_blocks, B, Hs);
    int n_splits = 0, solo = 0;
    bool flat = false, merged = false;
    if (n_blocks > 0) {
        AArgs a;
        a.k_arena = static_cast<const uint8_t *>(c->buf.k_arena);
        a.v_arena = static_cast<const uint8_t *>(c->buf.v_arena);
        a.k_index = static_cast<const uint32_t *>(c->buf.k_index);
        a.v_index = static_cast<const uint32_t *>(c->buf.v_index);
        a.k_meta = static_cast<const uint32_t *>(c->buf.k_token_meta);
        a.v_meta = static_cast<const uint32_t *>(c->buf.v_token_meta);
        a.q = q;
        a.partial = partial;
        a.meta_stride = c->max_tokens;
        a.B = B;
        a.index_words = c->index_words;
        a.H = Hs;
        a.dup = c->head_split;
        a.n_blocks = n_blocks;
        a.sm_log2 = sm_log2;
        // MID with both tensors wide: where it is cheaper with all its workgroups, two to a compute unit, at once; else three with
        // one buffer that K and V share do as well or better (with MID / without: 16000 chunks 45.0 / 51.1 us, four
        // heads 59.6 / 67.8, 25600 in 512 workgroups 64.1 / 73.1, 166400 in 416 426 / 369).  With one wide
        // tensor two workgroups fit either way, and MID is faster at all sizes (208000 chunks 351 / 406, 382 / 432).
        const bool both = c->wide_k && c->wide_v;
        bool mid = (c->wide_k || c->wide_v) && (!c->wide_k || c->qmax_k <= MID_QMAX) && (!c->wide_v || c->qmax_v <= MID_QMAX);
        int per_cu = 1;
#define PACKKV_ROOM(...) { static const int n = resident_workgroups(reinterpret_cast<const void *>(__VA_ARGS__)); per_cu = n; }
#define PACKKV_ROOM_8(g) \
    if (both) PACKKV_ROOM(attn8_kernel<g, true, true, false, false>) \
    else if (c->wide_k) { if (mid) PACKKV_ROOM(attn8_kernel<g, true, false, true, false>) else PACKKV_ROOM(attn8_kernel<g, true, false, false, false>) } \
    else if (c->wide_v) { if (mid) PACKKV_ROOM(attn8_kernel<g, false, true, true, false>) else PACKKV_ROOM(attn8_kernel<g, false, true, false, false>) } \
    else PACKKV_ROOM(attn8_kernel<g, false, false, false, false>)
#define PACKKV_ROOM_16(g) if (c->qmax_v > 7) PACKKV_ROOM(attn_kernel<g, true, false, false>) else PACKKV_ROOM(attn_kernel<g, false, false, false>)
        if (c->cfg.pack_size == 8) {
            PACKKV_DISPATCH_GROUP(G, PACKKV_ROOM_8)
        } else {
            PACKKV_DISPATCH_GROUP4(G, PACKKV_ROOM_16)
        }
#undef PACKKV_ROOM_8
#undef PACKKV_ROOM_16
#undef PACKKV_ROOM
        StreamSplits splits = splits_for(n_blocks, B * Hs, per_cu);
        if (both && mid) {
            const StreamSplits with_mid = splits_for(n_blocks, B * Hs, 2);
            mid = with_mid.n * B * Hs <= mid_room() && with_mid.cost <= splits.cost;
            if (mid) splits = with_mid;
        }
        n_splits = splits.n;
        a.blocks_per_split = (n_blocks + n_splits - 1) / n_splits;
        n_splits = (n_blocks + a.blocks_per_split - 1) / a.blocks_per_split;
        merged = merge_in_kernel(int64_t(n_splits) * B * Hs, int64_t(B) * Hs, G, c->wide_k || c->wide_v);
        solo = c->cfg.pack_size == PACK ? solo_waves(n_blocks, B * Hs, G) : 0;
        if (solo) a.blocks_per_split = n_blocks;
        a.counters = ws + WS_STATUS + 4 * ST_COUNTERS + COUNT_ATTENTION;
        a.k_tail = static_cast<const __half *>(c->buf.k_tail);
        a.v_tail = static_cast<const __half *>(c->buf.v_tail);
        a.n_tail = c->tail_tokens;
        a.tail_cap = c->cfg.tail_capacity;
        a.out = out;
        const dim3 grid(n_splits, B * Hs);
#define PACKKV_LAUNCH_A8X(g, kw, vw, mid)                                                                    \
    if (merged) hipLaunchKernelGGL((attn8_kernel<g, kw, vw, mid, (g <= MERGED_HEADS)>), grid, dim3(256), 0, s, a, VCentre::of(c->qmax_v)); \
    else hipLaunchKernelGGL((attn8_kernel<g, kw, vw, mid, false>), grid, dim3(256), 0, s, a, VCentre::of(c->qmax_v))
#define PACKKV_LAUNCH_A8W(g, kw, vw)              \
    if (mid) { PACKKV_LAUNCH_A8X(g, kw, vw, true); } \
    else { PACKKV_LAUNCH_A8X(g, kw, vw, false); }
#define PACKKV_LAUNCH_A8NN(g) PACKKV_LAUNCH_A8X(g, false, false, false)
#define PACKKV_LAUNCH_A8WN(g) PACKKV_LAUNCH_A8W(g, true, false)
#define PACKKV_LAUNCH_A8NW(g) PACKKV_LAUNCH_A8W(g, false, true)
#define PACKKV_LAUNCH_A8WW(g) PACKKV_LAUNCH_A8W(g, true, true)
#define PACKKV_LAUNCH_AX(g, high)                                                                            \
    if (solo == 8) hipLaunchKernelGGL((attn_kernel<g, high, false, false, 8>), dim3(1, B * Hs), dim3(512), 0, s, a, plan); \
    else if (solo) hipLaunchKernelGGL((attn_kernel<1, high, false, false, 4>), dim3(1, B * Hs), dim3(256), 0, s, a, plan); \
    else if (merged) hipLaunchKernelGGL((attn_kernel<g, high, false, true>), grid, dim3(256), 0, s, a, plan);     \
    else hipLaunchKernelGGL((attn_kernel<g, high, false, false>), grid, dim3(256), 0, s, a, plan)
#define PACKKV_LAUNCH_A(g) PACKKV_LAUNCH_AX(g, false)
#define PACKKV_LAUNCH_AH(g) PACKKV_LAUNCH_AX(g, true)
        // One head per kv-head and at least eight blocks for every wave of one round of resident workgroups:
        // a flat plan (8 x 52 streams of 500 blocks: 4160 workgroups at 768 resident ended in a round that was
        // two fifths full; 258 -> 239 us, 1 x 32 of 1000: 55 -> 49).  Below that the longer start-up of the plan
        // shows (1 x 32 streams of 250 blocks: 21.7 / 23.5 us).  With more heads the sums of a second stream's
        // part do not fit the registers next to the loop (4 x 8 streams of 512, four heads: 46 -> 50 us), and
        // packs of 8 gain nothing (30.1 / 30.6 us, wide 35.3 / 35.2).
#define PACKKV_LAUNCH_FLAT(...)                                                                        \
    {                                                                                                  \
        static const int per_cu = resident_workgroups(reinterpret_cast<const void *>(__VA_ARGS__));    \
        const int groups = plan_groups_for(n_blocks, B * Hs, per_cu, int64_t(V_SPLITS_MAX - 2) * B * Hs); \
        flat = plan.total >= int64_t(groups) * 4 * 8;                                                  \
        if (flat) {                                                                                    \
            plan.split(groups);                                                                        \
            hipLaunchKernelGGL((__VA_ARGS__), dim3(groups), dim3(256), 0, s, a, plan);                 \
        }                                                                                              \
    }
        if (c->cfg.pack_size == 16 && G == 1 && !solo) {
            if (c->qmax_v > 7) PACKKV_LAUNCH_FLAT(attn_kernel<1, true, true, false>)
            else PACKKV_LAUNCH_FLAT(attn_kernel<1, false, true, false>)
        }
        if (flat) {
        } else if (c->cfg.pack_size == 8) {
            if (c->wide_k && c->wide_v) {
                PACKKV_DISPATCH_GROUP(G, PACKKV_LAUNCH_A8WW)
            } else if (c->wide_k) {
                PACKKV_DISPATCH_GROUP(G, PACKKV_LAUNCH_A8WN)
            } else if (c->wide_v) {
                PACKKV_DISPATCH_GROUP(G, PACKKV_LAUNCH_A8NW)
            } else {
                PACKKV_DISPATCH_GROUP(G, PACKKV_LAUNCH_A8NN)
            }
        } else if (c->qmax_v > 7) {
            PACKKV_DISPATCH_GROUP4(G, PACKKV_LAUNCH_AH)
        } else {
            PACKKV_DISPATCH_GROUP4(G, PACKKV_LAUNCH_A)
        }
#undef PACKKV_LAUNCH_A8X
#undef PACKKV_LAUNCH_A8W
#undef PACKKV_LAUNCH_AX
#undef PACKKV_LAUNCH_A8NN
#undef PACKKV_LAUNCH_A8WN
#undef PACKKV_LAUNCH_A8NW
#undef PACKKV_LAUNCH_A8WW
#undef PACKKV_LAUNCH_A
#undef PACKKV_LAUNCH_AH
#undef PACKKV_LAUNCH_FLAT
    }
    if (flat || !(merged || solo))
        hipLaunchKernelGGL(flat ? attn_combine_kernel<true> : attn_combine_kernel<false>, dim3(B * H * Gq), dim3(256), 0, s, partial,
                           n_splits, B * H * Gq, plan, q, static_cast<const __half *>(c->buf.k_tail),
                           static_cast<const __half *>(c->buf.v_tail), c->tail_tokens,
                           c->cfg.tail_capacity, H, Gq, sm_log2, out);
    KV_HIP_CHECK(hipGetLastError());
    return KV_OK;
}

}  // namespace packkv
