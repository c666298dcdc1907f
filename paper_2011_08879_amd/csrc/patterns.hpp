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

// Copies the table in two parts, so that a kernel's other loads are issued in
// between: the table's come first, load, and the barrier after store completes
// the copy.
template <int T>
struct pattern_stage {
    static constexpr int N = (kPatternInts + T - 1) / T;
    int32_t t[N];
    __device__ void load(const row_patterns &p) {
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const int k = threadIdx.x + j * T;
            t[j] = k < p.ints ? p.tab[k] : 0;
        }
    }
    __device__ void store(pattern_lds &L) const {
#pragma unroll
        for (int j = 0; j < N; ++j)
            if (threadIdx.x + j * T < kPatternInts) L.off[threadIdx.x + j * T] = t[j];
    }
};

// Columns of slots j .. j + 3 of row i with pattern offsets at `tab` (a
// multiple of 4); negative for padding.
typedef int32_t pattern_quad __attribute__((ext_vector_type(4)));
__device__ inline pattern_quad pattern_cols(const pattern_lds &L, int tab, int64_t j, int32_t i) {
    return *reinterpret_cast<const pattern_quad *>(L.off + tab + j) + i;
}

}  // namespace gko
