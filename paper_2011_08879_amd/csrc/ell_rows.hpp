// Row sums of ELL SpMV for a thread owning two adjacent rows, shared by the
// plain SpMV and the CG step that fuses p.q into it.
#pragma once

#include "device.hpp"
#include "kernels.hpp"
#include "patterns.hpp"

namespace gko {

// Two adjacent rows per thread: ld is a multiple of 64, so slot j of rows
// 2t and 2t+1 are adjacent and each is fetched with one 16-byte (value) and
// one 8-byte (index) load; rows in [n, ld) are all padding.  Measured on the
// 27-point stencil: 148 us with one row per thread, 140 us with two.
template <typename V> struct ell_pair;
template <> struct ell_pair<double> { typedef double type __attribute__((ext_vector_type(2))); };
template <> struct ell_pair<float> { typedef float type __attribute__((ext_vector_type(2))); };
typedef int32_t ell_cpair __attribute__((ext_vector_type(2)));

// s0, s1 = rows i and i+1 of A x (i even, i < ld); each row stops at its
// first padding slot, the pair when both have reached theirs.
template <typename V>
__device__ inline void ell_pair_rows(int64_t K, int64_t ld, int64_t i,
                                     const int32_t *__restrict__ ecol, const V *__restrict__ eval,
                                     const V *__restrict__ x, V &s0, V &s1) {
    using V2 = typename ell_pair<V>::type;
    const ell_cpair *c = reinterpret_cast<const ell_cpair *>(ecol + i);
    const V2 *v = reinterpret_cast<const V2 *>(eval + i);
    const int64_t ld2 = ld / 2;
    s0 = V(0);
    s1 = V(0);
    for (int64_t j = 0; j < K; j += 4) {
        ell_cpair cc[4];
        V2 vv[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const bool ok = j + u < K;
            cc[u] = ok ? load_stream(c + (j + u) * ld2) : ell_cpair{-1, -1};
            vv[u] = ok ? load_stream(v + (j + u) * ld2) : V2{V(0), V(0)};
        }
        // Padding slots gather x[0] (the matrix has an entry, so x has one)
        // and keep the sum: no branch per gather, so all eight are in flight
        // together instead of one at a time (27-point stencil 138.6 -> 134
        // us).  The same change in the CSR subwarp, merge-path and SELL-P
        // loops measured slower there.
        V x0[4], x1[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            x0[u] = x[cc[u].x >= 0 ? cc[u].x : 0];
            x1[u] = x[cc[u].y >= 0 ? cc[u].y : 0];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const V t0 = s0 + vv[u].x * x0[u], t1 = s1 + vv[u].y * x1[u];
            s0 = cc[u].x >= 0 ? t0 : s0;
            s1 = cc[u].y >= 0 ? t1 : s1;
        }
        if (cc[3].x < 0 && cc[3].y < 0) break;
    }
}

// The same with the columns from the matrix's row patterns, for a wavefront
// whose lanes have consecutive row pairs.  load() issues the loads of the
// first slots, which are on their way while the table comes into LDS; sum()
// follows the barrier.
// FP64: the lane's own two rows, 16-byte value loads, four slots in flight.
typedef uint8_t pattern_pair __attribute__((ext_vector_type(2)));
template <typename V>
struct ell_pattern_pair {
    static constexpr int B = 4;
    using V2 = typename ell_pair<V>::type;
    V2 v[B];
    pattern_pair id;
    __device__ void load_slots(int64_t K, int64_t ld, int64_t i, int64_t j, const V *__restrict__ eval) {
        const V2 *p = reinterpret_cast<const V2 *>(eval + i) + j * (ld / 2);
#pragma unroll
        for (int u = 0; u < B; ++u) v[u] = j + u < K ? load_stream(p + u * (ld / 2)) : V2{V(0), V(0)};
    }
    __device__ void load(int64_t n, int64_t K, int64_t ld, int64_t i, const V *__restrict__ eval,
                         const row_patterns &pat) {
        if (i >= n) return;
        id = *reinterpret_cast<const pattern_pair *>(pat.id + i);
        load_slots(K, ld, i, 0, eval);
    }
    __device__ void sum(int64_t n, int64_t K, int64_t ld, int64_t i, const V *__restrict__ eval,
                        const V *__restrict__ x, const row_patterns &pat, const pattern_lds &L, V &s0,
                        V &s1) {
        s0 = V(0);
        s1 = V(0);
        if (i >= n) return;
        const int tab0 = id.x * pat.stride, tab1 = id.y * pat.stride;
        for (int64_t j = 0; j < K; j += B) {
            if (j > 0) load_slots(K, ld, i, j, eval);
            const pattern_quad q0 = pattern_cols(L, tab0, j, (int32_t)i);
            const pattern_quad q1 = pattern_cols(L, tab1, j, (int32_t)i + 1);
            int32_t c0[B], c1[B];
            V x0[B], x1[B];
#pragma unroll
            for (int u = 0; u < B; ++u) {
                c0[u] = j + u < K ? q0[u] : -1;
                c1[u] = j + u < K ? q1[u] : -1;
                x0[u] = x[c0[u] >= 0 ? c0[u] : 0];
                x1[u] = x[c1[u] >= 0 ? c1[u] : 0];
            }
#pragma unroll
            for (int u = 0; u < B; ++u) {
                const V t0 = s0 + v[u].x * x0[u], t1 = s1 + v[u].y * x1[u];
                s0 = c0[u] >= 0 ? t0 : s0;
                s1 = c1[u] >= 0 ? t1 : s1;
            }
            if (c0[B - 1] < 0 && c1[B - 1] < 0) break;
        }
    }
};

// FP32: lane l sums rows l and l + 64 of the wavefront's 128, so that every
// gather reads 64 neighbouring entries of x (the lane's own two rows: every
// second one of 128), eight slots in flight; then the sums go to their pairs.
// 27-point stencil 128^3 62 -> 46 us.
template <>
struct ell_pattern_pair<float> {
    static constexpr int B = 8;
    float v[2][B];
    int id[2];
    __device__ static int64_t row(int64_t i, int h) {
        const int lane = threadIdx.x % kWave;
        return i - 2 * lane + h * kWave + lane;
    }
    __device__ void load_slots(int64_t n, int64_t K, int64_t ld, int64_t i, int64_t j,
                               const float *__restrict__ eval) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int64_t r = row(i, h);
#pragma unroll
            for (int u = 0; u < B; ++u)
                v[h][u] = r < n && j + u < K ? load_stream(eval + (j + u) * ld + r) : 0.0f;
        }
    }
    __device__ void load(int64_t n, int64_t K, int64_t ld, int64_t i, const float *__restrict__ eval,
                         const row_patterns &pat) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int64_t r = row(i, h);
            id[h] = r < n ? pat.id[r] : -1;
        }
        load_slots(n, K, ld, i, 0, eval);
    }
    __device__ void sum(int64_t n, int64_t K, int64_t ld, int64_t i, const float *__restrict__ eval,
                        const float *__restrict__ x, const row_patterns &pat, const pattern_lds &L,
                        float &s0, float &s1) {
        float s[2] = {0.0f, 0.0f};
        const int tab[2] = {id[0] >= 0 ? id[0] * pat.stride : 0, id[1] >= 0 ? id[1] * pat.stride : 0};
        for (int64_t j = 0; j < K; j += B) {
            if (j > 0) load_slots(n, K, ld, i, j, eval);
            int32_t c[2][B];
            float xs[2][B];
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int u = 0; u < B; u += 4) {
                    const pattern_quad q = j + u < K  // the table has whole quads
                                               ? pattern_cols(L, tab[h], j + u, (int32_t)row(i, h))
                                               : pattern_quad(-1);
#pragma unroll
                    for (int w = 0; w < 4; ++w) c[h][u + w] = id[h] >= 0 && j + u + w < K ? q[w] : -1;
                }
#pragma unroll
            for (int u = 0; u < B; ++u)
#pragma unroll
                for (int h = 0; h < 2; ++h) xs[h][u] = x[c[h][u] >= 0 ? c[h][u] : 0];
#pragma unroll
            for (int u = 0; u < B; ++u)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const float t = s[h] + v[h][u] * xs[h][u];
                    s[h] = c[h][u] >= 0 ? t : s[h];
                }
            if (__all(c[0][B - 1] < 0 && c[1][B - 1] < 0)) break;  // all rows' padding has begun
        }
        // lane l's pair is rows 2l and 2l + 1 of the 128
        const int lane = threadIdx.x % kWave, from = 2 * lane % kWave;
        const float a0 = __shfl(s[0], from), a1 = __shfl(s[0], from + 1);
        const float b0 = __shfl(s[1], from), b1 = __shfl(s[1], from + 1);
        s0 = lane < kWave / 2 ? a0 : b0;
        s1 = lane < kWave / 2 ? a1 : b1;
    }
};

// SELL-P: one row per thread and one slice per wavefront (kSellpSlice ==
// kWave), so the slice's offset and width are wave-uniform: read with scalar
// loads, and the slot loop runs under scalar control.  Slot j of the wave's
// 64 rows is one contiguous 256-byte (index) and 512-byte (value) run, and
// the whole slice is one contiguous block.  Measured on the 27-point stencil
// (128^3): 141 us with two rows per thread (two slices per wave), 135 us
// with one and four slot loads in flight, 133 us with eight; ELL on the same
// matrix 140 us.
struct sellp_slice_of {
    int64_t base;  // first slot of the slice
    int64_t w;     // slice width
    int64_t r;     // the row's position in the slice
};

// The caller must give a wavefront 64 consecutive rows starting at a
// multiple of 64 (rows >= n of the last slice are padding).
__device__ inline sellp_slice_of sellp_slice(int64_t i, const int64_t *__restrict__ sets) {
    static_assert(kWave == kSellpSlice, "one slice per wavefront");
    const int32_t k = __builtin_amdgcn_readfirstlane((int32_t)(i / kSellpSlice));
    const int64_t base = sets[k];
    return {base, (sets[k + 1] - base) / kSellpSlice, i - (int64_t)k * kSellpSlice};
}

// Sum over the slots j0 <= j < j1 of row r of the slice starting at base,
// eight loads in flight; a row stops at its first padding slot.
template <typename V>
__device__ inline V sellp_slots_sum(int64_t base, int64_t r, int64_t j0, int64_t j1,
                                    const int32_t *__restrict__ scol,
                                    const V *__restrict__ sval, const V *__restrict__ x) {
    const int32_t *c = scol + base + r;
    const V *v = sval + base + r;
    V s = V(0);
    for (int64_t j = j0; j < j1; j += 8) {
        int32_t cc[8];
        V vv[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const bool ok = j + u < j1;
            cc[u] = ok ? load_stream(c + (j + u) * kSellpSlice) : -1;
            vv[u] = ok ? load_stream(v + (j + u) * kSellpSlice) : V(0);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (cc[u] >= 0) s += vv[u] * x[cc[u]];
        if (cc[7] < 0) break;  // the row's padding has begun
    }
    return s;
}

// Row i of A x over its whole slice.
template <typename V>
__device__ inline V sellp_row(int64_t i, const int64_t *__restrict__ sets,
                              const int32_t *__restrict__ scol, const V *__restrict__ sval,
                              const V *__restrict__ x) {
    const sellp_slice_of sl = sellp_slice(i, sets);
    return sellp_slots_sum(sl.base, sl.r, 0, sl.w, scol, sval, x);
}

// Row i with the columns from the matrix's row patterns, as ell_pattern_pair.
template <typename V>
struct sellp_pattern_row {
    static constexpr int B = 8;
    const V *p;  // the row's first slot
    int64_t w;
    V v[B];
    int id;
    __device__ void load_slots(int64_t j) {
#pragma unroll
        for (int u = 0; u < B; ++u) v[u] = j + u < w ? load_stream(p + (j + u) * kSellpSlice) : V(0);
    }
    __device__ void load(int64_t i, const int64_t *__restrict__ sets, const V *__restrict__ sval,
                         const row_patterns &pat) {
        id = pat.id[i];
        const sellp_slice_of sl = sellp_slice(i, sets);
        p = sval + sl.base + sl.r;
        w = sl.w;
        load_slots(0);
    }
    __device__ V sum(int64_t i, const V *__restrict__ x, const row_patterns &pat, const pattern_lds &L) {
        const int tab = id * pat.stride;
        V s = V(0);
        for (int64_t j = 0; j < w; j += B) {
            if (j > 0) load_slots(j);
            int32_t c[B];
#pragma unroll
            for (int u = 0; u < B; u += 4) {
                const pattern_quad q = j + u < w ? pattern_cols(L, tab, j + u, (int32_t)i) : pattern_quad(-1);
#pragma unroll
                for (int k = 0; k < 4; ++k) c[u + k] = j + u + k < w ? q[k] : -1;
            }
            V xs[B];
#pragma unroll
            for (int u = 0; u < B; ++u) xs[u] = x[c[u] >= 0 ? c[u] : 0];
#pragma unroll
            for (int u = 0; u < B; ++u) {
                const V t = s + v[u] * xs[u];
                s = c[u] >= 0 ? t : s;
            }
            if (c[B - 1] < 0) break;  // the row's padding has begun
        }
        return s;
    }
};

}  // namespace gko
