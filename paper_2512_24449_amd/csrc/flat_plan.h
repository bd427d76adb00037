// How the decode kernels cut the chunks of all streams into workgroups.  Plain arithmetic, the same on the host
// and in the kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

namespace packkv {

// All divisions are multiplications by numbers the host has prepared: a 64-bit division is some 130
// instructions, and a workgroup needs several before its first load (1 to 2 us at the
// start of every workgroup).
struct Divisor {
    uint64_t m = 0;  // floor(2^64 / d) + 1; 0 for d = 1
    static Divisor of(uint64_t d) {
        Divisor r;
        r.m = d > 1 ? ~uint64_t(0) / d + 1 : 0;
        return r;
    }
    // x / d for x * d < 2^64 (m * d exceeds 2^64 by at most d; ~0 / d is floor(2^64 / d) but for
    // powers of two, where m is exactly 2^64 / d)
    __host__ __device__ inline uint64_t divide(uint64_t x) const {
#if defined(__HIP_DEVICE_COMPILE__)
        return m ? __umul64hi(x, m) : x;
#else
        return m ? uint64_t((static_cast<unsigned __int128>(x) * m) >> 64) : x;
#endif
    }
};

// A value that is the same in every lane, in a scalar register.
__host__ __device__ inline int uniform_value(int v) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_readfirstlane(v);
#else
    return v;
#endif
}

// Work list of the kernels that walk chunks in the plane layout: the chunks of all streams in one
// sequence (stream-major, n_blocks per stream), cut into n_groups equal ranges, one per workgroup.
// A workgroup that crosses a stream boundary writes one partial row set per stream it touches:
// the set of workgroup w for stream s has number w + s (unique, below n_groups + streams).
struct FlatPlan {
    int n_blocks;    // packed blocks per stream
    int n_groups;    // workgroups
    int64_t total;   // streams * n_blocks
    int heads;
    Divisor by_groups, by_blocks, by_heads, by_total;  // by_total: m = 0 if the products below do not fit it

    // streams = batch * heads.  n_groups may be set later, by split().
    static FlatPlan make(int n_blocks, int batch, int heads) {
        FlatPlan p;
        p.n_blocks = n_blocks;
        p.n_groups = 0;
        p.total = int64_t(n_blocks) * batch * heads;
        p.heads = heads;
        p.by_blocks = Divisor::of(uint64_t(n_blocks > 0 ? n_blocks : 1));
        p.by_heads = Divisor::of(uint64_t(heads));
        return p;
    }
    void split(int groups) {
        n_groups = groups;
        by_groups = Divisor::of(uint64_t(groups));
        by_total = Divisor::of(uint64_t(total));
        if (double(total) * double(total) * groups >= 1e19) by_total.m = 0;
    }
    // The longer ranges are spread evenly, so that ranges end at stream boundaries wherever the
    // numbers allow it (a workgroup with parts of two streams pays its start-up and its end twice:
    // 25 -> 30 us for the V product of 8 streams of 2048 blocks).
    __host__ __device__ inline int64_t begin(int w) const { return int64_t(by_groups.divide(uint64_t(w) * uint64_t(total))); }
    // workgroup that holds flattened chunk f (for the largest plans an estimate, off by one at most, put right)
    __host__ __device__ inline int group_of(int64_t f) const {
        if (by_total.m) return int(by_total.divide(uint64_t((f + 1) * n_groups - 1)));
        int w = int(double(f) * n_groups / double(total));
        w = w < n_groups ? w : n_groups - 1;
        while (begin(w) > f) --w;
        while (begin(w + 1) <= f) ++w;
        return w;
    }
    // The part of one stream at the head of the range [f, range_end).
    struct Segment {
        int stream, b, h, blk_begin, blk_end;
    };
    __host__ __device__ inline Segment segment(int64_t f, int64_t range_end) const {
        Segment g;
        // (scalar from here on: everything the loops derive from them stays in scalar registers)
        g.stream = uniform_value(int(by_blocks.divide(uint64_t(f))));
        g.b = uniform_value(int(by_heads.divide(uint64_t(g.stream))));
        g.h = g.stream - g.b * heads;
        g.blk_begin = int(f - int64_t(g.stream) * n_blocks);
        const int64_t left = g.blk_begin + (range_end - f);
        g.blk_end = left < n_blocks ? int(left) : n_blocks;
        return g;
    }
};

// Workgroups for a flat work list of `total` chunks where `room` of them are resident at a time: one round,
// never less than one block per wave, at most `most`.
inline int64_t flat_groups(int64_t total, int64_t room, int64_t most) {
    return std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(room, (total + 3) / 4), most));
}

// Workgroups for a flat plan over `streams` streams of n_blocks chunks, at most `most`.  Either one round
// of resident workgroups that cut the list as it comes, or a whole number of workgroups per
// stream: then none has parts of two streams, each of which costs its start-up (query, index, first
// chunk) and its end (merge, store) -- about the time of PART_COST chunks of a wave.  The cheaper one by the
// chunks its longest wave walks: 256 streams of 7 blocks run as 512 workgroups of one stream each (K product 5.9 us,
// V product 8.9; 448 that cross the boundaries 8.1 and 12.3), 120 of 78 as 960 (12.2 and 15.2; 1024 14.5 and 19.1),
// 416 streams of 500 blocks as one round.
inline int plan_groups(int n_blocks, int streams, int64_t room, int64_t most) {
    constexpr int64_t PART_COST = 2;
    const int64_t total = int64_t(n_blocks) * streams;
    auto waves = [](int64_t blocks) { return (blocks + 3) / 4; };
    const int64_t flat = flat_groups(total, room, most);
    int64_t best = flat;
    int64_t best_cost = waves((total + flat - 1) / flat) * 4 + 4 * PART_COST * (flat + streams - 1) / flat;
    const int64_t most_per_stream = std::max<int64_t>(1, std::min<int64_t>(waves(n_blocks), most / streams));
    for (const int64_t want : {int64_t(1), room / streams, most_per_stream}) {
        const int64_t per_stream = std::max<int64_t>(1, std::min<int64_t>(want, most_per_stream));
        const int64_t groups = per_stream * streams;
        if (groups > most) continue;
        const int64_t rounds = (groups + room - 1) / room;
        const int64_t cost = 4 * rounds * (waves((n_blocks + per_stream - 1) / per_stream) + PART_COST);
        if (cost < best_cost || (cost == best_cost && best == flat)) best = groups, best_cost = cost;
    }
    return int(best);
}

// Workgroups per stream where every stream is split alike, for kernels of which `per_cu` workgroups of four waves fit one of
// `cus` compute units; at least one block per wave, at most `most`; and what that costs by the rule.
// The starting point: about eight blocks to a wave, within two workgroups to a compute unit and 4096 in all.  But the more waves
// a SIMD unit shares, the longer each block takes: with one, two and three workgroups to a compute unit 2.6, 3.4 and 4.2 us
// behind 6, 7 and 9 us of start and end (fused attention, 32 streams of 128 to 1000 blocks, four heads), in units of 2.6 / 16 us below; what is over
// a round of resident workgroups costs its share, and half a workgroup's time at the end.  Where the most workgroups for one, two, .. to a
// compute unit are at least 8 % cheaper they are taken: 32 streams of 1000 blocks 1024 -> 768 workgroups, 66.0 -> 60.8 us; 64 of 300 (three
// heads) 640 -> 768, 45.5 -> 41.1; 40 of 160 (one head) 520 -> 480, 23.7 -> 21.3; 416 of 500 stay.
struct StreamSplits {
    int n;
    int64_t cost;
    bool usual;   // the starting point
};
inline StreamSplits stream_splits(int n_blocks, int streams, int cus, int per_cu, int most) {
    const int64_t most_here = std::max<int64_t>(1, std::min<int64_t>(most, (n_blocks + 3) / 4)), room = int64_t(cus) * per_cu;
    auto with = [&](int64_t want) {
        const int64_t n = std::max<int64_t>(1, std::min(want, most_here)), groups = n * streams, blocks = ((n_blocks + n - 1) / n + 3) / 4;
        const int64_t sharing = std::min<int64_t>((groups + cus - 1) / cus, per_cu), block = 16 + 5 * (sharing - 1), ends = 37 + 9 * (sharing - 1);
        return StreamSplits{int(n), groups <= room ? blocks * block + ends : groups * blocks * block / room + ends + blocks * 8, false};
    };
    const int64_t usual = std::min<int64_t>(std::max<int64_t>(int64_t(n_blocks) * streams / 32, 2 * cus), 16 * cus);
    StreamSplits start = with((usual + streams - 1) / streams);
    start.usual = true;
    StreamSplits best = start;
    for (int64_t sharing = 1; sharing <= per_cu; ++sharing) {
        const StreamSplits s = with(sharing * cus / streams);
        if (s.cost < best.cost) best = s;
    }
    return best.cost * 100 <= start.cost * 92 ? best : start;
}

}  // namespace packkv
