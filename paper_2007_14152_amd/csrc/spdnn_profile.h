// Host logic of a profiled inference whose launches run several layers each (spdnn_get_profile).
#pragma once

#include <stdint.h>

#include <cstddef>

namespace spdnn {

struct LayerRun {
    int32_t l0, l1;  // one launch: layers l0 .. l1-1
    bool alone;      // a layer's own kernel: it reports the rows on entry to the next layer to the host, not to `rows`
};

// rows[0 .. L]: rows on entry to layer l, as the launches of several layers counted them.  Puts in what the host was told.
inline void take_host_counts(const LayerRun* runs, size_t n, const int* host_counts, int* rows) {
    for (size_t i = 0; i < n; ++i)
        if (runs[i].alone) rows[runs[i].l1] = host_counts[runs[i].l1];
}

}  // namespace spdnn
