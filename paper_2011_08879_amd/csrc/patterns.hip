// Row patterns (see row_patterns in kernels.hpp): finding the distinct lists of
// column offsets of a CSR matrix and each row's list.
//
// The rows' lists are hashed and the distinct hashes collected, at most
// kPatternMost of them, each with the first row that has it; the table is built
// from those rows, and every row is compared with its list, so a hash that two
// lists share is found and the matrix is then used without patterns.
#include "patterns.hpp"

#include "offsets.hpp"

namespace gko {

namespace {

constexpr int kPB = 256;
constexpr int kLocalKeys = 512;
static_assert(kPatternMost < kLocalKeys && kPatternMost < kPatternKeys && kPatternMost < 255,
              "open addressing ends, and an index is a byte");

// The key of a row, from the offsets of its entries in order; never zero (an
// empty entry of a table).
struct row_key {
    unsigned long long h;
    __device__ explicit row_key(int32_t len) : h(0x9e3779b97f4a7c15ull * (unsigned)(len + 1)) {}
    __device__ void add(int32_t off) {
        h ^= (unsigned)off;
        h *= 0xff51afd7ed558ccdull;
        h ^= h >> 32;
    }
    __device__ unsigned long long get() const { return h | 1; }
};

// Runs f(j, column) over the entries of the workgroup's rows r0 .. r0 + kPB - 1,
// a thread per row, the columns through LDS in chunks with coalesced loads
// (read from memory by a thread per row, the 27-point stencil on 128^3 took
// 0.5 ms a pass).
constexpr int kColChunk = 4096;
template <typename F>
__device__ inline void each_entry(int64_t n, int64_t r0, const int32_t *__restrict__ rp,
                                  const int32_t *__restrict__ col, int32_t (&L)[kColChunk],
                                  int32_t b, int32_t e, F f) {
    const int32_t kb = rp[r0], ke = rp[r0 + kPB < n ? r0 + kPB : n];
    for (entry_steps<kColChunk> chunk(kb, ke); chunk.more(); chunk.next()) {
        const int32_t c0 = chunk.at(), cn = chunk.count();
        int32_t cc[kColChunk / kPB];
#pragma unroll
        for (int u = 0; u < kColChunk / kPB; ++u) {
            const int t = threadIdx.x + u * kPB;
            cc[u] = t < cn ? load_stream(col + c0 + t) : 0;
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kColChunk / kPB; ++u) L[threadIdx.x + u * kPB] = cc[u];
        __syncthreads();
        const int32_t lo = (b > c0 ? b : c0) - c0, hi = (e < c0 + cn ? e : c0 + cn) - c0;
        for (int32_t t = lo; t < hi; ++t) f(c0 - b + t, L[t]);
    }
}

// Enters key h with the complement of its row into a table of N entries (the
// largest complement stays); false when there is no room.
template <int N>
__device__ inline bool enter(unsigned long long *keys, unsigned *first, unsigned long long h,
                             unsigned inv_row, bool &added) {
    added = false;
    for (int q = 0, t = (int)(h >> 40) % N; q < N; ++q, t = (t + 1) % N) {
        unsigned long long k = keys[t];
        if (k == 0) {
            k = atomicCAS(keys + t, 0ull, h);
            added = k == 0;
        }
        if (k == 0 || k == h) {
            atomicMax(first + t, inv_row);
            return true;
        }
    }
    return false;
}

// A workgroup collects the lists of its rows in LDS and adds them to the
// table at its end: few atomics on the table's entries, which all workgroups
// share.  Matrices without patterns end after the first rows.
__global__ __launch_bounds__(kPB) void pattern_keys_kernel(int64_t n, const int32_t *__restrict__ rp,
                                                           const int32_t *__restrict__ col,
                                                           csr_facts *facts) {
    __shared__ unsigned long long keys[kLocalKeys];
    __shared__ unsigned first[kLocalKeys];
    __shared__ int count;
    __shared__ int32_t C[kColChunk];
    pattern_keys *out = &facts->patterns;
    if (facts->err != 0 || facts->max_len > kPatternLongest) return;
    for (int t = threadIdx.x; t < kLocalKeys; t += kPB) {
        keys[t] = 0;
        first[t] = 0;
    }
    if (threadIdx.x == 0) count = 0;
    __syncthreads();
    for (int64_t base = (int64_t)blockIdx.x * kPB; base < n; base += (int64_t)gridDim.x * kPB) {
        const int64_t i = base + threadIdx.x;
        const int32_t b = i < n ? rp[i] : 0, e = i < n ? rp[i + 1] : 0;
        row_key key(e - b);
        each_entry(n, base, rp, col, C, b, e, [&](int32_t, int32_t c) { key.add(c - (int32_t)i); });
        if (i < n) {
            bool added;
            if (!enter<kLocalKeys>(keys, first, key.get(), ~(unsigned)i, added) || added)
                atomicAdd(&count, 1);
        }
        __syncthreads();
        const int c = count;
        __syncthreads();
        if (c > kPatternMost) {
            if (threadIdx.x == 0) atomicOr(&out->too_many, 1);
            return;
        }
    }
    for (int t = threadIdx.x; t < kLocalKeys; t += kPB)
        if (keys[t] != 0) {
            bool added;
            if (!enter<kPatternKeys>(out->key, out->first, keys[t], first[t], added))
                atomicOr(&out->too_many, 1);
        }
}

__global__ void pattern_table_kernel(int count, int stride, const unsigned *__restrict__ first,
                                     const int32_t *__restrict__ rp, const int32_t *__restrict__ col,
                                     int32_t *__restrict__ tab) {
    const int p = blockIdx.x;  // the last one is all padding
    const int32_t r = p < count ? (int32_t)first[p] : 0;
    const int32_t b = p < count ? rp[r] : 0, e = p < count ? rp[r + 1] : 0;
    for (int j = threadIdx.x; j < stride; j += blockDim.x)
        tab[p * stride + j] = b + j < e ? col[b + j] - r : kPatternPad;
}

// Each row's index in the ascending keys, compared entry by entry with the table.
__global__ __launch_bounds__(kPB) void pattern_ids_kernel(int64_t n, int64_t n_ids, int count,
                                                          int stride,
                                                          const unsigned long long *__restrict__ key,
                                                          const int32_t *__restrict__ tab,
                                                          const int32_t *__restrict__ rp,
                                                          const int32_t *__restrict__ col,
                                                          uint8_t *__restrict__ id, int *wrong) {
    __shared__ unsigned long long keys[kPatternMost];
    __shared__ pattern_lds L;
    __shared__ int32_t C[kColChunk];
    for (int t = threadIdx.x; t < count; t += kPB) keys[t] = key[t];
    for (int t = threadIdx.x; t < (count + 1) * stride; t += kPB) L.off[t] = tab[t];
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kPB, i = base + threadIdx.x;
    const int32_t b = i < n ? rp[i] : 0, e = i < n ? rp[i + 1] : 0;
    row_key rk(e - b);
    if (base < n)
        each_entry(n, base, rp, col, C, b, e, [&](int32_t, int32_t c) { rk.add(c - (int32_t)i); });
    int lo = count;
    if (i < n) {
        const unsigned long long h = rk.get();
        lo = 0;
        for (int hi = count; hi - lo > 1;) {
            const int mid = (lo + hi) / 2;
            if (keys[mid] <= h) lo = mid;
            else hi = mid;
        }
    }
    if (base < n) {
        const int32_t *off = L.off + lo * stride;
        bool same = e - b <= stride && (e - b == stride || i >= n || off[e - b] == kPatternPad);
        each_entry(n, base, rp, col, C, b, e, [&](int32_t j, int32_t c) {
            same = same && j < stride && c - (int32_t)i == off[j];
        });
        if (!same) atomicOr(wrong, 1);
    }
    if (i < n_ids) id[i] = (uint8_t)lo;
}

}  // namespace

hipError_t pattern_collect(hipStream_t s, int64_t n, const int32_t *rp, const int32_t *col,
                           csr_facts *facts) {
    const int64_t g = (n + kPB - 1) / kPB;
    pattern_keys_kernel<<<(unsigned)(g < 1024 ? g : 1024), kPB, 0, s>>>(n, rp, col, facts);
    return hipGetLastError();
}

hipError_t pattern_assign(hipStream_t s, int64_t n, const int32_t *rp, const int32_t *col, int count,
                          int stride, const unsigned long long *key, const unsigned *first,
                          int32_t *tab, uint8_t *id, int *wrong) {
    pattern_table_kernel<<<(unsigned)count + 1, 64, 0, s>>>(count, stride, first, rp, col, tab);
    const int64_t ids = pattern_ids(n);
    pattern_ids_kernel<<<(unsigned)((ids + kPB - 1) / kPB), kPB, 0, s>>>(n, ids, count, stride, key,
                                                                        tab, rp, col, id, wrong);
    return hipGetLastError();
}

}  // namespace gko
