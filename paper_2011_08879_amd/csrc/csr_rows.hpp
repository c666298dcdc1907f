// Row sums of CSR SpMV for a subwarp of W lanes owning U consecutive rows,
// shared by the plain SpMV and the CG step that fuses p.q into it.
#pragma once

#include "device.hpp"
#include "offsets.hpp"
#include "patterns.hpp"

namespace gko {

template <int W>
struct csr_shape {
    static constexpr int U = W >= 16 ? 4 : 8;  // rows per subwarp
};

// Rows longer than long_t are left out (their sum is 0 here): a separate
// kernel with a whole workgroup per row handles them.
template <typename V, int W, int U>
__device__ inline void csr_rows_sum(int64_t n, int64_t row0, int lane,
                                    const int32_t *__restrict__ rp,
                                    const int32_t *__restrict__ col, const V *__restrict__ val,
                                    const V *__restrict__ x, V (&s)[U], int32_t long_t) {
    int32_t b[U], e[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const bool ok = row0 + u < n;
        b[u] = ok ? rp[row0 + u] : 0;
        e[u] = ok ? rp[row0 + u + 1] : 0;
        if (e[u] - b[u] > long_t) e[u] = b[u];
    }
    int32_t c[U];
    V v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const entry_steps<W> k(b[u], e[u], lane);
        c[u] = k.more() ? load_stream(col + k.at()) : -1;
        v[u] = k.more() ? load_stream(val + k.at()) : V(0);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) s[u] = c[u] >= 0 ? v[u] * x[c[u]] : V(0);
    // rows longer than W: the rest in strides of 4W, four loads in flight
#pragma unroll
    for (int u = 0; u < U; ++u)
        for (entry_steps<4 * W> k(b[u], e[u], W + lane); k.more(); k.next()) {
            int32_t cc[4];
            V vv[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool ok = j * W < k.left();
                cc[j] = ok ? load_stream(col + k.at() + j * W) : -1;
                vv[j] = ok ? load_stream(val + k.at() + j * W) : V(0);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (cc[j] >= 0) s[u] += vv[j] * x[cc[j]];
        }
#pragma unroll
    for (int u = 0; u < U; ++u) s[u] = subwarp<W>::reduce_sum(s[u]);
}

// Row-per-thread CSR for matrices with short rows (see csr_kernel_width),
// generalised to G lanes per row: a workgroup of T threads owns T / G
// consecutive rows, stages their entries (one contiguous range) through LDS
// in chunks of C with coalesced loads, and the G lanes of a row walk its
// entries in the chunk, lane g taking entries g, g + G, ...; their partial
// sums are added by a xor butterfly.  The x gathers of neighbouring rows then
// hit neighbouring columns for banded and stencil patterns (as in ELL),
// unlike a subwarp reading its row from memory.  Returns the row sum in every
// lane of the row (0 for rows >= n).
// Measured on the 27-point stencil with G = 1: 235 us with a 32-lane subwarp
// per row, 171 us row-per-thread; eight gathers in flight in the walk
// instead of four 170 -> 167 us (banded rows of 24-40 entries 109 -> 105 us),
// sixteen no faster.
constexpr int kRowThreadBlock = 256;
constexpr int kRowThreadChunk = 2048;

// How a kernel takes its columns.  kByColumn: from the matrix.  kByPattern:
// from its row patterns, so that only the values are read.  N > 0: from the
// patterns, all rows with at most N entries (csr_rowwave_sum).
constexpr int kByColumn = 0, kByPattern = -1;

template <typename V, int G, int M>
struct rowthread_lds {
    V val[kRowThreadBlock / kWave][kWave / G * M];
    pattern_lds tab;
};
template <typename V, int G>
struct rowthread_lds<V, G, kByColumn> {
    int32_t col[kRowThreadChunk];
    V val[kRowThreadChunk];
};
template <typename V, int G>
struct rowthread_lds<V, G, kByPattern> {
    V val[kRowThreadChunk];
    pattern_lds tab;
};

// The kernel for G lanes per row.  Measured (FP64 / FP32, us; column indices,
// patterns in chunks, csr_rowwave_sum): 7-point stencil 160^3 (1 lane) 78 /
// 52, 60 / 40, 56 / 33; 27-point stencil 128^3 (4 lanes) 143 / 96, 127 / 88,
// 107 / 63.  FP32 rows of 12 and of 16 entries, four lanes a row, keep the column
// indices: sixteen such rows meet in a few LDS banks, which costs more without
// the columns' loads beside it (column indices, patterns: rows of 16 37 / 42,
// blocks of 16 40 / 46, rows of 12 with one of 1,000 of 40 47 / 57; but rows of
// 13, 14 and 15 47 / 45, 44 / 42 and 44 / 40, FP64 rows of 16 61 / 57).
template <typename V, int G, typename F>
hipError_t with_csr_mode(const row_patterns &p, F launch) {
    // rows of kPatternLongest take one or four lanes (csr_row_lanes)
    static_assert(kPatternLongest < 56, "no rows with patterns take eight lanes");
    if constexpr (G == 1 || G == 4) {
        if (p.id && !(G == 4 && sizeof(V) == 4 && (p.mean == 12 || p.mean == 16))) {
            if constexpr (G == 1) {
                if (p.stride <= 8) return launch(std::integral_constant<int, 8>{});
                if (p.stride <= 12) return launch(std::integral_constant<int, 12>{});
            } else if (p.stride <= 28) {
                return launch(std::integral_constant<int, 28>{});
            }
            return launch(std::integral_constant<int, kByPattern>{});
        }
    }
    return launch(std::integral_constant<int, kByColumn>{});
}

template <typename V, int G, int M>
__device__ inline V csr_chunks_sum(int64_t n, int64_t r0, const int32_t *__restrict__ rp,
                                   const int32_t *__restrict__ col, const V *__restrict__ val,
                                   const V *__restrict__ x, const row_patterns &pat,
                                   rowthread_lds<V, G, M> &L) {
    constexpr bool PAT = M == kByPattern;
    if constexpr (PAT) {
        pattern_stage<kRowThreadBlock> stage;
        stage.load(pat);
        stage.store(L.tab);  // completed by the first chunk's barrier
    }
    constexpr int T = kRowThreadBlock, C = kRowThreadChunk, RT = T / G;
    const int g = threadIdx.x % G;
    const int64_t i = r0 + threadIdx.x / G;
    const int64_t rl = r0 + RT < n ? r0 + RT : n;
    const int32_t kb = rp[r0], ke = rp[rl];
    const int32_t b = i < n ? rp[i] : ke, e = i < n ? rp[i + 1] : ke;
    int tab = 0;
    if constexpr (PAT) tab = i < n ? pat.id[i] * pat.stride : 0;
    V s = V(0);
    for (entry_steps<C> chunk(kb, ke); chunk.more(); chunk.next()) {
        const int32_t c0 = chunk.at(), cn = chunk.count();
        int32_t cc[C / T];
        V vv[C / T];
#pragma unroll
        for (int j = 0; j < C / T; ++j) {
            const int t = threadIdx.x + j * T;
            if constexpr (!PAT) cc[j] = t < cn ? load_stream(col + c0 + t) : 0;
            vv[j] = t < cn ? load_stream(val + c0 + t) : V(0);
        }
#pragma unroll
        for (int j = 0; j < C / T; ++j) {
            const int t = threadIdx.x + j * T;
            if (t < cn) {
                if constexpr (!PAT) L.col[t] = cc[j];
                L.val[t] = vv[j];
            }
        }
        __syncthreads();
        const int32_t lo = (b > c0 ? b : c0) - c0;
        const int32_t hi = (e < c0 + cn ? e : c0 + cn) - c0;
        const auto col_at = [&](int32_t t) -> int64_t {
            if constexpr (PAT) return i + L.tab.off[tab + (c0 - b) + t];
            else return L.col[t];
        };
        int32_t k = lo + g;
        for (; k + 7 * G < hi; k += 8 * G) {  // eight gathers in flight, summed in order
            V xs[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) xs[u] = x[col_at(k + u * G)];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += L.val[k + u * G] * xs[u];
        }
        for (; k + 3 * G < hi; k += 4 * G) {
            const V x0 = x[col_at(k)], x1 = x[col_at(k + G)], x2 = x[col_at(k + 2 * G)],
                    x3 = x[col_at(k + 3 * G)];
            s += L.val[k] * x0;
            s += L.val[k + G] * x1;
            s += L.val[k + 2 * G] * x2;
            s += L.val[k + 3 * G] * x3;
        }
        for (; k < hi; k += G) s += L.val[k] * x[col_at(k)];
        __syncthreads();
    }
    if constexpr (G > 1) s = subwarp<G>::reduce_sum(s);
    return s;
}

// Rows of at most N entries with patterns: a wavefront owns 64 / G consecutive
// rows, whose values (one contiguous range) it takes into LDS with coalesced
// loads that are all in flight together, and with the loads of the pattern
// table.  With the columns known, the lanes walk their rows side by side: lane
// g * (64 / G) + r takes entries g, g + G, ... of row r, so each gather reads
// runs of 64 / G neighbouring entries of x (with the G lanes of a row next to
// each other every gather touches twice the lines).  The G lanes' sums are
// added by a xor butterfly, and row r's sum goes to lanes r G .. r G + G - 1.
template <typename V, int N, int G>
__device__ inline V csr_rowwave_sum(int64_t n, int64_t r0, const int32_t *__restrict__ rp,
                                    const V *__restrict__ val, const V *__restrict__ x,
                                    const row_patterns &pat, rowthread_lds<V, G, N> &L) {
    constexpr int RW = kWave / G, LPL = N / G;  // rows, and loads of a lane
    const int lane = threadIdx.x % kWave, g = lane / RW;
    const int64_t i = r0 + threadIdx.x / kWave * RW + lane % RW;
    V *vals = L.val[threadIdx.x / kWave];
    const int32_t b = rp[i < n ? i : n], e = rp[i < n ? i + 1 : n];
    const int id = i < n ? pat.id[i] : 0;
    pattern_stage<kRowThreadBlock> stage;
    stage.load(pat);
    const int32_t kb = __builtin_amdgcn_readfirstlane(b), cn = __shfl(e, kWave - 1) - kb;
    V vv[LPL];
#pragma unroll
    for (int j = 0; j < LPL; ++j) {
        const int t = lane + j * kWave;
        vv[j] = t < cn ? load_stream(val + kb + t) : V(0);
    }
    stage.store(L.tab);
#pragma unroll
    for (int j = 0; j < LPL; ++j) vals[lane + j * kWave] = vv[j];
    __syncthreads();
    const int32_t *off = L.tab.off + id * pat.stride;
    const V *mine = vals + (b - kb);
    const int32_t len = e - b;
    V s = V(0);
    for (int32_t j = g; j < len; j += 8 * G) {
        V xs[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) xs[u] = x[j + u * G < len ? (int32_t)i + off[j + u * G] : 0];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const V t = s + mine[j + u * G < len ? j + u * G : 0] * xs[u];
            s = j + u * G < len ? t : s;
        }
    }
#pragma unroll
    for (int m = RW; m < kWave; m <<= 1) s += __shfl_xor(s, m);
    return G > 1 ? __shfl(s, lane / G) : s;
}

template <typename V, int G, int M>
__device__ inline V csr_rowthread_sum(int64_t n, int64_t r0, const int32_t *__restrict__ rp,
                                      const int32_t *__restrict__ col, const V *__restrict__ val,
                                      const V *__restrict__ x, const row_patterns &pat,
                                      rowthread_lds<V, G, M> &L) {
    if constexpr (M > 0) return csr_rowwave_sum<V, M, G>(n, r0, rp, val, x, pat, L);
    else return csr_chunks_sum<V, G, M>(n, r0, rp, col, val, x, pat, L);
}

}  // namespace gko
