// Block-Jacobi apply of one workgroup's tile of rows, shared by the vector
// kernels that need z = M^-1 r.
#pragma once

#include "device.hpp"

namespace gko {

template <int BS>
constexpr int bj_packed() { return BS * (BS + 1) / 2; }

// LDS of a tile of T rows (nothing without a preconditioner, BS = 0).
template <typename V, int BS, int T>
struct bj_lds {
    V r[T];
    V inv[T / BS * bj_packed<BS>()];
};
template <typename V, int T>
struct bj_lds<V, 0, T> {};

// z_i = sum_j D_b^{-1}[i mod bs][j] r_{b*bs + j}, j ascending, for the tile
// of T rows starting at `base`, with entry (i, j) of a symmetric inverse
// block read from its packed upper triangle (the (min, max) entry).  The
// tile's packed blocks (contiguous because BS divides T) and residuals are
// staged in LDS with coalesced loads.  Slots of a short last block beyond n
// are zero in `inv`.  bj_tile_stage loads the blocks, bj_tile_apply takes the
// residuals and returns z; the barrier between the staged blocks and their
// use is in bj_tile_apply, and another one ends it.
template <typename V, int BS, int T>
__device__ inline void bj_tile_stage(int64_t n, int64_t base, const V *__restrict__ inv,
                                     bj_lds<V, BS, T> &L) {
    constexpr int P = bj_packed<BS>();
    const int64_t nb = (n + BS - 1) / BS;
    const int64_t off = (base / BS) * P;
    for (int t = threadIdx.x; t < (T / BS) * P; t += T)
        L.inv[t] = (off + t < nb * P) ? inv[off + t] : V(0);
}

// bj_tile_stage in two parts: the loads of a tile's blocks, issued while
// another tile is worked on, and their way into LDS.
template <typename V, int BS, int T>
struct bj_ahead {
    static constexpr int P = bj_packed<BS>(), N = (T / BS * P + T - 1) / T;
    V v[N];
    __device__ void load(int64_t n, int64_t base, const V *__restrict__ inv) {
        const int64_t nb = (n + BS - 1) / BS, off = (base / BS) * P;
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const int t = threadIdx.x + j * T;
            v[j] = t < T / BS * P && off + t < nb * P ? load_stream(inv + off + t) : V(0);
        }
    }
    __device__ void store(bj_lds<V, BS, T> &L) const {
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const int t = threadIdx.x + j * T;
            if (t < T / BS * P) L.inv[t] = v[j];
        }
    }
};
template <typename V, int T>
struct bj_ahead<V, 0, T> {};

template <typename V, int BS, int T>
__device__ inline V bj_tile_apply(V ri, bj_lds<V, BS, T> &L) {
    constexpr int P = bj_packed<BS>();
    const int tid = threadIdx.x;
    L.r[tid] = ri;
    __syncthreads();
    V z = V(0);
    const int i = tid % BS, b0 = tid - i;
    const V *D = L.inv + (tid / BS) * P;
    const int row_i = i * BS - i * (i - 1) / 2 - i;  // packed (i, j) = row_i + j, j >= i
#pragma unroll
    for (int j = 0; j < BS; ++j) {
        const int idx = j >= i ? row_i + j : j * BS - j * (j - 1) / 2 - j + i;
        z += D[idx] * L.r[b0 + j];
    }
    __syncthreads();
    return z;
}

}  // namespace gko
