// Row patterns: matrices whose rows repeat a few lists of column offsets.
#pragma once

#include "device.hpp"
#include "kernels.hpp"

namespace gko {

// The table in LDS: a lane reads the offsets of its row's pattern, most lanes
// of a wavefront the same ones.
struct pattern_lds {
    alignas(16) int32_t off[kPatternInts];
};

// Copies the table; the caller's next barrier completes it.
template <int T>
__device__ inline void pattern_stage(const row_patterns &p, pattern_lds &L) {
    for (int t = threadIdx.x; t < p.ints; t += T) L.off[t] = p.tab[t];
}

// Columns of slots j .. j + 3 of row i with pattern offsets at `tab` (a
// multiple of 4); negative for padding.
typedef int32_t pattern_quad __attribute__((ext_vector_type(4)));
__device__ inline pattern_quad pattern_cols(const pattern_lds &L, int tab, int64_t j, int32_t i) {
    return *reinterpret_cast<const pattern_quad *>(L.off + tab + j) + i;
}

}  // namespace gko
