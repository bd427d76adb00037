// csrc/flat_plan.h on the host, called from test_stream_splits.py.
#include "flat_plan.h"

extern "C" int splits(int n_blocks, int streams, int cus, int per_cu, int most, int64_t *cost, int *usual) {
    const packkv::StreamSplits s = packkv::stream_splits(n_blocks, streams, cus, per_cu, most);
    *cost = s.cost, *usual = s.usual;
    return s.n;
}
