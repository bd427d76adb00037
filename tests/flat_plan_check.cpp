// Host checks of csrc/flat_plan.h, called from test_work_split_plan.py.  Each returns 0 or the number of the check
// that failed.
#include "flat_plan.h"

using namespace packkv;
typedef unsigned __int128 u128;

// x / d for every x with x * d < 2^64 around the multiples of d that matter
extern "C" int check_divisor(uint64_t d, uint64_t x) {
    if (d == 0 || u128(x) * d >= (u128(1) << 64)) return -1;
    return Divisor::of(d).divide(x) == x / d ? 0 : 1;
}

static uint64_t next(uint64_t &s) {
    s ^= s << 13, s ^= s >> 7, s ^= s << 17;
    return s;
}

// All of a plan up to `full` workgroups, a sample of it above.
extern "C" int check_plan(int n_blocks, int batch, int heads, int groups, int full) {
    FlatPlan p = FlatPlan::make(n_blocks, batch, heads);
    p.split(groups);
    const int64_t total = int64_t(n_blocks) * batch * heads, streams = int64_t(batch) * heads;
    if (p.total != total || p.begin(0) != 0 || p.begin(groups) != total) return 1;
    uint64_t seed = 88172645463325252ull;
    const int n = groups <= full ? groups : full;
    int64_t last_row_set = -1;
    for (int i = 0; i < n; ++i) {
        const int w = groups <= full ? i : int(next(seed) % uint64_t(groups));
        const int64_t lo = p.begin(w), hi = p.begin(w + 1);
        if (lo != int64_t(u128(w) * u128(total) / u128(groups))) return 2;
        if (lo >= hi) continue;  // more workgroups than chunks
        for (const int64_t f : {lo, hi - 1, lo + int64_t(next(seed) % uint64_t(hi - lo))})
            if (p.group_of(f) != w) return 3;
        if (groups > full) last_row_set = -1;
        for (int64_t f = lo; f < hi;) {
            const FlatPlan::Segment g = p.segment(f, hi);
            if (g.stream != f / n_blocks || g.b != g.stream / heads || g.h != g.stream % heads) return 4;
            if (g.blk_begin != f % n_blocks || g.blk_end <= g.blk_begin || g.blk_end > n_blocks) return 5;
            if (g.blk_end != n_blocks && f + (g.blk_end - g.blk_begin) != hi) return 6;
            if (w + g.stream <= last_row_set || w + g.stream >= groups + streams) return 7;
            last_row_set = w + g.stream;
            f += g.blk_end - g.blk_begin;
            if (f > hi) return 8;
        }
    }
    // the combine kernels take up to 64 row sets per stream
    if (groups <= 62 * streams) {
        const int64_t some = streams <= full ? streams : full;
        for (int64_t i = 0; i < some; ++i) {
            const int64_t s = streams <= full ? i : int64_t(next(seed) % uint64_t(streams));
            if (p.group_of((s + 1) * n_blocks - 1) - p.group_of(s * n_blocks) + 1 > 64) return 9;
        }
    }
    return 0;
}

extern "C" int uses_estimate(int n_blocks, int batch, int heads, int groups) {
    FlatPlan p = FlatPlan::make(n_blocks, batch, heads);
    p.split(groups);
    return p.by_total.m == 0;
}

extern "C" int groups_for(int n_blocks, int streams, int64_t room, int64_t most) { return plan_groups(n_blocks, streams, room, most); }

// Streams whose first chunk is not the first of a workgroup's range.
extern "C" int crossed_boundaries(int n_blocks, int streams, int groups) {
    FlatPlan p = FlatPlan::make(n_blocks, 1, streams);
    p.split(groups);
    int crossed = 0;
    for (int64_t s = 1; s < streams; ++s) crossed += p.begin(p.group_of(s * n_blocks)) != s * n_blocks;
    return crossed;
}
