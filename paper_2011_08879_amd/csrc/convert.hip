// Format conversions and structure checks on the device.  All of it is
// integer bookkeeping and copies, so results are bit-exact by construction:
//   CSR -> COO : expand row offsets into row indices.
//   COO -> CSR : row_ptr[i] = first entry with row >= i (binary search).
//   CSR -> ELL : slot (j, i) at j*ld + i = j-th entry of row i, else padding
//                col = -1, val = +0.0.
//   CSR -> HYB : ELL of width K plus a COO tail with entries K.. of each row.
//   CSR -> SELL-P : as ELL, each slice of 64 rows with its own width.
//   ELL/HYB/SELL-P -> CSR : per-row counts, exclusive scan, copy.
#include <climits>
#include <cstdint>

#include "device.hpp"
#include "kernels.hpp"
#include "offsets.hpp"

namespace gko {

static inline unsigned grid_for(int64_t n, int block) { return (unsigned)((n + block - 1) / block); }

// ------------------------------------------------------------------ validation
__global__ void validate_csr_kernel(int64_t n, int64_t m, int64_t nnz, const int32_t *__restrict__ rp,
                                    const int32_t *__restrict__ col, int *err) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i > n) return;
    if (i == 0 && rp[0] != 0) atomicOr(err, 1);
    if (i == n) {
        if ((int64_t)rp[n] != nnz) atomicOr(err, 1);
        return;
    }
    const int32_t b = rp[i], e = rp[i + 1];
    if (e < b || b < 0 || (int64_t)e > nnz) {
        atomicOr(err, 1);
        return;
    }
    int bad = 0;
    for (int32_t k = b; k < e; ++k) {
        const int32_t c = col[k];
        if (c < 0 || (int64_t)c >= m) bad |= 2;
        if (k > b && c <= col[k - 1]) bad |= 4;
    }
    if (bad) atomicOr(err, bad);
}

hipError_t validate_csr(hipStream_t s, int64_t n, int64_t m, int64_t nnz, const int32_t *rp,
                        const int32_t *col, int *err) {
    validate_csr_kernel<<<grid_for(n + 1, 256), 256, 0, s>>>(n, m, nnz, rp, col, err);
    return hipGetLastError();
}

__global__ void narrow_kernel(int64_t n, const int64_t *__restrict__ rp64, int32_t *__restrict__ rp32,
                              int *err) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i > n) return;
    const int64_t v = rp64[i];
    if (v < 0 || v > INT_MAX) atomicOr(err, 1);
    rp32[i] = (int32_t)v;
}

hipError_t narrow_row_ptr(hipStream_t s, int64_t n, const int64_t *rp64, int32_t *rp32, int *err) {
    narrow_kernel<<<grid_for(n + 1, 256), 256, 0, s>>>(n, rp64, rp32, err);
    return hipGetLastError();
}

// ------------------------------------------------------------------ CSR <-> COO
// G lanes per row write consecutive row indices, G about half the mean length:
// a wavefront per row leaves most lanes idle on short rows, a thread per entry
// with a search for its row in LDS was slower on longer ones (200,000 rows of
// 32: 189 -> 210 us for CSR -> COO -> CSR).  Rows of more than 16 G entries are
// left to the whole workgroup: 250,000 lognormal rows took 26 us without.
template <int G>
__global__ __launch_bounds__(256) void csr_rows_kernel(int64_t n, const int32_t *__restrict__ rp,
                                                       int32_t *__restrict__ row) {
    constexpr int R = 256 / G;
    __shared__ int any_long;
    const int64_t r0 = (int64_t)blockIdx.x * R;
    if (threadIdx.x == 0) any_long = 0;
    __syncthreads();
    const int64_t i = r0 + threadIdx.x / G;
    if (i < n) {
        const int32_t b = rp[i], e = rp[i + 1];
        if (e - b > 16 * G) any_long = 1;
        else
            for (entry_steps<G> k(b, e, threadIdx.x % G); k.more(); k.next()) row[k.at()] = (int32_t)i;
    }
    __syncthreads();
    if (!any_long) return;
    for (int64_t r = r0; r < r0 + R && r < n; ++r) {
        const int32_t b = rp[r], e = rp[r + 1];
        if (e - b > 16 * G)
            for (entry_steps<256> k(b, e, threadIdx.x); k.more(); k.next()) row[k.at()] = (int32_t)r;
    }
}

hipError_t csr_rows(hipStream_t s, int64_t n, int64_t nnz, const int32_t *rp, int32_t *row) {
    if (n == 0 || nnz == 0) return hipSuccess;
    const int64_t mean = nnz / n;
    if (mean < 12) csr_rows_kernel<4><<<grid_for(n, 64), 256, 0, s>>>(n, rp, row);
    else if (mean < 48) csr_rows_kernel<16><<<grid_for(n, 16), 256, 0, s>>>(n, rp, row);
    else csr_rows_kernel<kWave><<<grid_for(n, 4), 256, 0, s>>>(n, rp, row);
    return hipGetLastError();
}

__global__ void rows_to_ptr_kernel(int64_t n, int64_t nnz, const int32_t *__restrict__ row,
                                   int32_t *__restrict__ rp) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i > n) return;
    int64_t lo = 0, hi = nnz;  // first k with row[k] >= i
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (row[mid] < i) lo = mid + 1;
        else hi = mid;
    }
    rp[i] = (int32_t)lo;
}

hipError_t rows_to_ptr(hipStream_t s, int64_t n, int64_t nnz, const int32_t *row, int32_t *rp) {
    rows_to_ptr_kernel<<<grid_for(n + 1, 256), 256, 0, s>>>(n, nnz, row, rp);
    return hipGetLastError();
}

// ------------------------------------------------------------------ row lengths
// At most kMaxLenBlocks workgroups, each with one atomic: 65,536 workgroups
// (2^24 rows) queued on the one address for 748 us.
constexpr unsigned kMaxLenBlocks = 512;

__global__ void max_len_kernel(int64_t n, const int32_t *__restrict__ rp, int *maxlen) {
    __shared__ int lds[256 / kWave];
    int v = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        v = max(v, rp[i + 1] - rp[i]);
#pragma unroll
    for (int b = 1; b < kWave; b <<= 1) v = max(v, __shfl_xor(v, b));
    if ((threadIdx.x % kWave) == 0) lds[threadIdx.x / kWave] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 256 / kWave; ++w) v = max(v, lds[w]);
        atomicMax(maxlen, v);
    }
}

hipError_t max_row_len(hipStream_t s, int64_t n, const int32_t *rp, int *maxlen) {
    if (n == 0) return hipSuccess;
    const unsigned g = grid_for(n, 256);
    max_len_kernel<<<g < kMaxLenBlocks ? g : kMaxLenBlocks, 256, 0, s>>>(n, rp, maxlen);
    return hipGetLastError();
}

// Row-length histogram.  Row lengths take few distinct values, so counting
// straight into global memory serialises on a handful of addresses (818 us for
// 250,000 lognormal rows with one of 10,000 entries); each block counts into
// LDS first and adds its nonzero bins once.  Rows too long for the LDS bins,
// few in any matrix, count into global memory.
constexpr int kHistLdsBins = 8192;
constexpr unsigned kHistBlocks = 256;

__global__ void hist_kernel(int64_t n, const int32_t *__restrict__ rp, int *hist, int nbins) {
    __shared__ int lh[kHistLdsBins];
    for (int t = threadIdx.x; t < nbins; t += blockDim.x) lh[t] = 0;
    __syncthreads();
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int l = rp[i + 1] - rp[i];
        atomicAdd(l < nbins ? &lh[l] : hist + l, 1);
    }
    __syncthreads();
    for (int t = threadIdx.x; t < nbins; t += blockDim.x)
        if (lh[t]) atomicAdd(hist + t, lh[t]);
}

hipError_t row_len_hist(hipStream_t s, int64_t n, const int32_t *rp, int *hist, int64_t maxlen) {
    if (n == 0) return hipSuccess;
    const unsigned g = grid_for(n, 256);
    const int bins = (int)(maxlen + 1 < kHistLdsBins ? maxlen + 1 : kHistLdsBins);
    hist_kernel<<<g < kHistBlocks ? g : kHistBlocks, 256, 0, s>>>(n, rp, hist, bins);
    return hipGetLastError();
}

// ------------------------------------------------------------------ column spread
// A workgroup per tile, at most kSpreadTiles of them evenly over the rows, the
// first kSpreadEntries of each row, all in flight together: 8 us, whatever
// the matrix.  The tile's lines are counted by a bit for each line of x in LDS.
constexpr int kSpreadTiles = 256, kSpreadEntries = 16, kSpreadLine = 16;

__global__ __launch_bounds__(256) void column_lines_kernel(int64_t n, int words,
                                                           const int32_t *__restrict__ rp,
                                                           const int32_t *__restrict__ col,
                                                           csr_facts *facts) {
    __shared__ unsigned seen[kSpreadCols / kSpreadLine / 32 + 1];
    __shared__ unsigned sums[3];
    if (facts->err != 0) return;
    for (int t = threadIdx.x; t < words; t += 256) seen[t] = 0;
    if (threadIdx.x < 3) sums[threadIdx.x] = 0;
    __syncthreads();
    const int64_t tiles = (n + 255) / 256, i = blockIdx.x * tiles / gridDim.x * 256 + threadIdx.x;
    unsigned entries = 0, lines = 0, fresh = 0;
    if (i < n) {
        const int32_t b = rp[i], len = rp[i + 1] - b;
        const bool first = threadIdx.x % kWave == 0;
        const int32_t pb = first ? b : rp[i - 1], plen = first ? 0 : b - pb;
        entries = len < kSpreadEntries ? len : kSpreadEntries;
        int32_t own[kSpreadEntries], beside[kSpreadEntries];  // lines, -1: none
#pragma unroll
        for (int k = 0; k < kSpreadEntries; ++k) {
            own[k] = k < len ? col[b + k] / kSpreadLine : -1;
            beside[k] = k < len && k < plen ? col[pb + k] / kSpreadLine : -1;
        }
#pragma unroll
        for (int k = 0; k < kSpreadEntries; ++k)
            if (own[k] != beside[k]) {  // a line of the neighbouring row's is noted by it
                ++lines;
                atomicOr(&seen[own[k] / 32], 1u << own[k] % 32);
            }
    }
    __syncthreads();
    for (int t = threadIdx.x; t < words; t += 256) fresh += __popc(seen[t]);
    const unsigned part[3] = {entries, lines, fresh};
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        unsigned v = part[j];
#pragma unroll
        for (int s = 1; s < kWave; s <<= 1) v += __shfl_xor(v, s);
        if (threadIdx.x % kWave == 0) atomicAdd(&sums[j], v);
    }
    __syncthreads();
    if (threadIdx.x < 3) atomicAdd(&facts->spread[threadIdx.x], sums[threadIdx.x]);
}

hipError_t column_lines(hipStream_t s, int64_t n, int64_t m, const int32_t *rp, const int32_t *col,
                        csr_facts *facts) {
    if (n == 0 || m == 0) return hipSuccess;
    if (m > kSpreadCols) return hipErrorInvalidValue;
    const unsigned g = grid_for(n, 256);
    const int words = (int)((m - 1) / kSpreadLine / 32 + 1);
    column_lines_kernel<<<g < kSpreadTiles ? g : kSpreadTiles, 256, 0, s>>>(n, words, rp, col, facts);
    return hipGetLastError();
}

// ------------------------------------------------------------------ STREAM probe
// Each thread moves one pair of doubles with 16-byte non-temporal loads and
// stores, the access shape that measured fastest on MI355X (about 6.6 TB/s
// for a 1 GiB copy, against 6.2 TB/s with one double per thread); an odd
// last element is handled by the thread of the last pair.  Arrays that are
// not all 16-byte aligned take the one-double-per-thread kernels.
typedef double dpair __attribute__((ext_vector_type(2)));

__global__ void stream_copy1_kernel(int64_t n, const double *__restrict__ a, double *__restrict__ c) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) c[i] = a[i];
}

__global__ void stream_triad1_kernel(int64_t n, const double *__restrict__ a,
                                     const double *__restrict__ b, double sc, double *__restrict__ c) {
#pragma clang fp contract(off)
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) c[i] = a[i] + sc * b[i];
}

__global__ void stream_copy_kernel(int64_t n, const double *__restrict__ a, double *__restrict__ c) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t np = n / 2;
    if (i < np) {
        const dpair v = __builtin_nontemporal_load(reinterpret_cast<const dpair *>(a) + i);
        __builtin_nontemporal_store(v, reinterpret_cast<dpair *>(c) + i);
    }
    if (i == np - (np > 0 ? 1 : 0) && (n & 1)) c[n - 1] = a[n - 1];
}

__global__ void stream_triad_kernel(int64_t n, const double *__restrict__ a,
                                    const double *__restrict__ b, double sc, double *__restrict__ c) {
#pragma clang fp contract(off)
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t np = n / 2;
    if (i < np) {
        const dpair va = __builtin_nontemporal_load(reinterpret_cast<const dpair *>(a) + i);
        const dpair vb = __builtin_nontemporal_load(reinterpret_cast<const dpair *>(b) + i);
        dpair r;
        r.x = va.x + sc * vb.x;
        r.y = va.y + sc * vb.y;
        __builtin_nontemporal_store(r, reinterpret_cast<dpair *>(c) + i);
    }
    if (i == np - (np > 0 ? 1 : 0) && (n & 1)) c[n - 1] = a[n - 1] + sc * b[n - 1];
}

hipError_t stream_op(hipStream_t s, int op, int64_t n, const double *a, const double *b, double sc,
                     double *c) {
    if (n == 0) return hipSuccess;
    const uintptr_t bits = (uintptr_t)a | (uintptr_t)c | (op == 0 ? 0 : (uintptr_t)b);
    if (bits & 15) {
        if (op == 0) stream_copy1_kernel<<<grid_for(n, 256), 256, 0, s>>>(n, a, c);
        else stream_triad1_kernel<<<grid_for(n, 256), 256, 0, s>>>(n, a, b, sc, c);
        return hipGetLastError();
    }
    const int64_t threads = n / 2 > 0 ? n / 2 : 1;
    if (op == 0) stream_copy_kernel<<<grid_for(threads, 256), 256, 0, s>>>(n, a, c);
    else stream_triad_kernel<<<grid_for(threads, 256), 256, 0, s>>>(n, a, b, sc, c);
    return hipGetLastError();
}

// Random-gather probe: y[i] = x[idx[i]].  A wavefront takes 256 consecutive
// elements as two runs of 128, each lane two adjacent elements per run, so
// every index load (8 bytes a lane) and every store (16 bytes a lane) covers
// one contiguous range; the four gathers are issued before any result is
// used.  x is read through a buffer resource of m doubles, so an index
// outside [0, m) reads 0 instead of faulting.  Index and output streams are
// non-temporal, so the L2 holds x the way an SpMV's gathers do.
typedef int32_t probe_i2 __attribute__((ext_vector_type(2)));
typedef double probe_d2 __attribute__((ext_vector_type(2)));
constexpr int kProbeBlock = 256;

__device__ inline double probe_gather(__amdgpu_buffer_rsrc_t rx, int32_t c) {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rx, c * 8, 0, 0));
}

__global__ __launch_bounds__(kProbeBlock) void gather_probe_kernel(
    int64_t n, const double *__restrict__ x, int64_t m, const int32_t *__restrict__ idx,
    double *__restrict__ y) {
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
        (void *)x, (short)0, (int)(m * 8 < INT_MAX ? m * 8 : INT_MAX), 0x00020000);
    const int64_t wave = ((int64_t)blockIdx.x * kProbeBlock + threadIdx.x) / kWave;
    const int lane = threadIdx.x % kWave;
    const int64_t i0 = wave * 256 + 2 * lane, i1 = i0 + 128;
    if (wave * 256 + 256 <= n) {
        const probe_i2 c0 = __builtin_nontemporal_load(reinterpret_cast<const probe_i2 *>(idx + i0));
        const probe_i2 c1 = __builtin_nontemporal_load(reinterpret_cast<const probe_i2 *>(idx + i1));
        probe_d2 v0, v1;
        v0.x = probe_gather(rx, c0.x);
        v0.y = probe_gather(rx, c0.y);
        v1.x = probe_gather(rx, c1.x);
        v1.y = probe_gather(rx, c1.y);
        __builtin_nontemporal_store(v0, reinterpret_cast<probe_d2 *>(y + i0));
        __builtin_nontemporal_store(v1, reinterpret_cast<probe_d2 *>(y + i1));
    } else {
        const int64_t e[4] = {i0, i0 + 1, i1, i1 + 1};
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (e[u] < n) y[e[u]] = probe_gather(rx, idx[e[u]]);
    }
}

hipError_t gather_probe(hipStream_t s, int64_t n, const double *x, int64_t m, const int32_t *idx,
                        double *y) {
    if (n == 0) return hipSuccess;
    const int64_t waves = (n + 255) / 256;  // 256 elements per wavefront
    const int64_t per_block = kProbeBlock / kWave;
    gather_probe_kernel<<<(unsigned)((waves + per_block - 1) / per_block), kProbeBlock, 0, s>>>(
        n, x, m, idx, y);
    return hipGetLastError();
}

// ------------------------------------------------------------------ CSR <-> slots
// ELL, the ELL part of HYB and SELL-P keep the rows' entries in column-major
// slots.  A workgroup converts a tile of 64 rows (SELL-P: one slice), whose CSR
// entries are one contiguous range, through LDS in chunks: the CSR side is read
// or written in its own order, the slot side by wavefronts with a lane per
// row, so both sides are coalesced (a thread per row walking its CSR entries:
// 500,000 rows of 16 entries CSR -> ELL 132 us, ELL -> CSR 255 us).
// A chunk holds few rows of a tile with long ones, and most lanes of a
// wavefront then have none: tiles of more than kSlotWide slots per row are
// converted in blocks of 64 rows and kSlotCols slots instead, by as many
// workgroups as the grid has for a tile.  16M entries, CSR -> ELL / ELL -> CSR
// with the library's host work, chunks and blocks: rows of 65 94 / 147 and 106 /
// 114 us (a third block with one slot), of 80 94 / 167 and 89 / 93, of 256 135 /
// 320 and 77 / 92, of 3,000 4,840 / 21,900 and 98 / 95; a million lognormal rows
// sorted by length in SELL-P 5,520 / 23,800 and 329 / 301.
constexpr int kSlotRows = kWave;
constexpr int kSlotThreads = 256;
constexpr int kSlotChunk = 2048;
constexpr int64_t kSlotWide = 72;
constexpr int kSlotCols = 32;

static_assert(kSlotRows == kSellpSlice, "a SELL-P slice is a tile");

// Slot j of the tile's row r is at start + j stride + r, j < width.
struct slot_tile {
    int64_t start, stride, width;
};

__device__ inline slot_tile slot_tile_of(const slot_layout &S, int64_t tile) {
    if (!S.sets) return {tile * kSlotRows, S.ld, S.K};
    return {S.sets[tile], kSlotRows, (S.sets[tile + 1] - S.sets[tile]) / kSlotRows};
}

// A chunk's entries in LDS, spread so that lanes reading rows of equal length
// do not meet in one bank.
template <typename V>
struct slot_lds {
    int32_t col[kSlotChunk + kSlotChunk / 32];
    V val[kSlotChunk + kSlotChunk / 32];
    __device__ static int at(int t) { return t + (t >> 5); }
};

// The slots of one row (entries b..e) that fall into the chunk of cn entries
// at c0: [lo, hi); and the wavefront's smallest lo and largest hi.
struct slot_span {
    int32_t lo, hi, first, last;
};

__device__ inline slot_span span_of(int32_t b, int32_t e, int64_t width, int32_t c0, int32_t cn) {
    slot_span p;
    const int32_t end = e - b < width ? e : b + (int32_t)width;
    p.lo = (b > c0 ? b : c0) - b;
    p.hi = (end < c0 + cn ? end : c0 + cn) - b;
    p.first = p.lo < p.hi ? p.lo : INT_MAX;
    p.last = p.lo < p.hi ? p.hi : 0;
#pragma unroll
    for (int s = 1; s < kWave; s <<= 1) {
        p.first = min(p.first, __shfl_xor(p.first, s));
        p.last = max(p.last, __shfl_xor(p.last, s));
    }
    p.first = min(p.first, p.last);  // no row in the chunk: an empty range
    return p;
}

template <typename V>
__global__ __launch_bounds__(kSlotThreads) void csr_to_slots_kernel(
    int64_t n, const int32_t *__restrict__ rp, const int32_t *__restrict__ col,
    const V *__restrict__ val, slot_layout S, int32_t *__restrict__ scol, V *__restrict__ sval) {
    __shared__ slot_lds<V> L;
    const int64_t r0 = (int64_t)blockIdx.x * kSlotRows;
    const slot_tile T = slot_tile_of(S, blockIdx.x);
    if (T.width > kSlotWide) return;
    const int lane = threadIdx.x % kWave, wv = threadIdx.x / kWave;
    constexpr int NW = kSlotThreads / kWave, E = kSlotChunk / kSlotThreads;
    const int64_t i = r0 + lane, last = r0 + kSlotRows < n ? r0 + kSlotRows : n;
    const int32_t b = rp[i < n ? i : n], e = rp[i + 1 < n ? i + 1 : n];
    const int32_t kb = rp[r0 < n ? r0 : n], ke = rp[last];
    for (entry_steps<kSlotChunk> chunk(kb, ke); chunk.more(); chunk.next()) {
        const int32_t c0 = chunk.at(), cn = chunk.count();
        const slot_span p = span_of(b, e, T.width, c0, cn);
        if (p.first >= p.last) continue;  // all past their rows' slots (the same in every wavefront)
        int32_t cc[E];
        V vv[E];
#pragma unroll
        for (int u = 0; u < E; ++u) {
            const int t = threadIdx.x + u * kSlotThreads;
            cc[u] = t < cn ? load_stream(col + c0 + t) : 0;
            vv[u] = t < cn ? load_stream(val + c0 + t) : V(0);
        }
#pragma unroll
        for (int u = 0; u < E; ++u) {
            const int t = threadIdx.x + u * kSlotThreads;
            L.col[L.at(t)] = cc[u];
            L.val[L.at(t)] = vv[u];
        }
        __syncthreads();
        for (int32_t j = p.first + wv; j < p.last; j += NW)
            if (j >= p.lo && j < p.hi) {
                const int64_t slot = T.start + j * T.stride + lane;
                const int t = L.at(b + j - c0);
                scol[slot] = L.col[t];
                sval[slot] = L.val[t];
            }
        __syncthreads();
    }
    // padding from the rows' ends on (rows past the last one: all slots)
    const int64_t len = e - b;
    int32_t shortest = e - b;
#pragma unroll
    for (int s = 1; s < kWave; s <<= 1) shortest = min(shortest, __shfl_xor(shortest, s));
    for (int64_t j = shortest + wv; j < T.width; j += NW)
        if (j >= len) {
            const int64_t slot = T.start + j * T.stride + lane;
            scol[slot] = -1;
            sval[slot] = V(0);
        }
}

// rp: the rows' offsets (with a tail: of the whole rows; TAIL leaves the
// places of the tail's entries alone).
template <typename V, bool TAIL>
__global__ __launch_bounds__(kSlotThreads) void slots_to_csr_kernel(
    int64_t n, slot_layout S, const int32_t *__restrict__ scol, const V *__restrict__ sval,
    const int32_t *__restrict__ rp, int32_t *__restrict__ col, V *__restrict__ val) {
    __shared__ slot_lds<V> L;
    const int64_t r0 = (int64_t)blockIdx.x * kSlotRows;
    const slot_tile T = slot_tile_of(S, blockIdx.x);
    if (T.width > kSlotWide) return;
    const int lane = threadIdx.x % kWave, wv = threadIdx.x / kWave;
    constexpr int NW = kSlotThreads / kWave, E = kSlotChunk / kSlotThreads;
    const int64_t i = r0 + lane, last = r0 + kSlotRows < n ? r0 + kSlotRows : n;
    const int32_t b = rp[i < n ? i : n], e = rp[i + 1 < n ? i + 1 : n];
    const int32_t kb = rp[r0], ke = rp[last];
    for (entry_steps<kSlotChunk> chunk(kb, ke); chunk.more(); chunk.next()) {
        const int32_t c0 = chunk.at(), cn = chunk.count();
        const slot_span p = span_of(b, e, T.width, c0, cn);
        if (p.first >= p.last) continue;  // the tail's (the same in every wavefront)
        if constexpr (TAIL) {
            for (int u = 0; u < E; ++u) L.col[L.at(threadIdx.x + u * kSlotThreads)] = -1;
            __syncthreads();
        }
        for (int32_t j = p.first + wv; j < p.last; j += NW)
            if (j >= p.lo && j < p.hi) {
                const int64_t slot = T.start + j * T.stride + lane;
                const int t = L.at(b + j - c0);
                L.col[t] = load_stream(scol + slot);
                L.val[t] = load_stream(sval + slot);
            }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < E; ++u) {
            const int t = threadIdx.x + u * kSlotThreads;
            if (t < cn && (!TAIL || L.col[L.at(t)] >= 0)) {
                col[c0 + t] = L.col[L.at(t)];
                val[c0 + t] = L.val[L.at(t)];
            }
        }
        __syncthreads();
    }
}

// A block of a wide tile in LDS; b and len: the rows' first entry and slots.
template <typename V>
struct slot_block {
    int32_t col[kSlotRows][kSlotCols + 1];
    V val[kSlotRows][kSlotCols + 1];
    int32_t b[kSlotRows], len[kSlotRows];
    __device__ void load_rows(int64_t n, int64_t r0, int64_t width, const int32_t *__restrict__ rp) {
        if (threadIdx.x < kSlotRows) {
            const int64_t i = r0 + threadIdx.x;
            const int32_t first = rp[i < n ? i : n], l = rp[i + 1 < n ? i + 1 : n] - first;
            b[threadIdx.x] = first;
            len[threadIdx.x] = l < width ? l : (int32_t)width;
        }
        __syncthreads();
    }
};

template <typename V>
__global__ __launch_bounds__(kSlotThreads) void csr_to_wide_slots_kernel(
    int64_t n, const int32_t *__restrict__ rp, const int32_t *__restrict__ col,
    const V *__restrict__ val, slot_layout S, int32_t *__restrict__ scol, V *__restrict__ sval) {
    __shared__ slot_block<V> L;
    const slot_tile T = slot_tile_of(S, blockIdx.x);
    if (T.width <= kSlotWide) return;
    constexpr int NR = kSlotThreads / kSlotCols, U = kSlotRows / NR, NW = kSlotThreads / kWave;
    const int lane = threadIdx.x % kWave, wv = threadIdx.x / kWave;
    const int r = threadIdx.x / kSlotCols, q = threadIdx.x % kSlotCols;
    L.load_rows(n, (int64_t)blockIdx.x * kSlotRows, T.width, rp);
    for (int64_t j0 = (int64_t)blockIdx.y * kSlotCols; j0 < T.width; j0 += (int64_t)gridDim.y * kSlotCols) {
        int32_t cc[U];
        V vv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {  // padding where a row has ended
            const int row = r + u * NR;
            const bool ok = j0 + q < L.len[row];
            cc[u] = ok ? load_stream(col + L.b[row] + j0 + q) : -1;
            vv[u] = ok ? load_stream(val + L.b[row] + j0 + q) : V(0);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            L.col[r + u * NR][q] = cc[u];
            L.val[r + u * NR][q] = vv[u];
        }
        __syncthreads();
        for (int k = wv; k < kSlotCols && j0 + k < T.width; k += NW) {
            const int64_t slot = T.start + (j0 + k) * T.stride + lane;
            scol[slot] = L.col[lane][k];
            sval[slot] = L.val[lane][k];
        }
        __syncthreads();
    }
}

template <typename V>
__global__ __launch_bounds__(kSlotThreads) void wide_slots_to_csr_kernel(
    int64_t n, slot_layout S, const int32_t *__restrict__ scol, const V *__restrict__ sval,
    const int32_t *__restrict__ rp, int32_t *__restrict__ col, V *__restrict__ val) {
    __shared__ slot_block<V> L;
    const slot_tile T = slot_tile_of(S, blockIdx.x);
    if (T.width <= kSlotWide) return;
    constexpr int NR = kSlotThreads / kSlotCols, U = kSlotRows / NR, NW = kSlotThreads / kWave;
    const int lane = threadIdx.x % kWave, wv = threadIdx.x / kWave;
    const int r = threadIdx.x / kSlotCols, q = threadIdx.x % kSlotCols;
    L.load_rows(n, (int64_t)blockIdx.x * kSlotRows, T.width, rp);
    int32_t longest = L.len[lane];
#pragma unroll
    for (int s = 1; s < kWave; s <<= 1) longest = max(longest, __shfl_xor(longest, s));
    for (int64_t j0 = (int64_t)blockIdx.y * kSlotCols; j0 < longest; j0 += (int64_t)gridDim.y * kSlotCols) {
        int32_t cc[kSlotCols / NW];
        V vv[kSlotCols / NW];
#pragma unroll
        for (int u = 0; u < kSlotCols / NW; ++u) {
            const int64_t j = j0 + wv + u * NW, slot = T.start + j * T.stride + lane;
            const bool ok = j < L.len[lane];
            cc[u] = ok ? load_stream(scol + slot) : 0;
            vv[u] = ok ? load_stream(sval + slot) : V(0);
        }
#pragma unroll
        for (int u = 0; u < kSlotCols / NW; ++u) {
            L.col[lane][wv + u * NW] = cc[u];
            L.val[lane][wv + u * NW] = vv[u];
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int row = r + u * NR;
            if (j0 + q < L.len[row]) {
                col[L.b[row] + j0 + q] = L.col[row][q];
                val[L.b[row] + j0 + q] = L.val[row][q];
            }
        }
        __syncthreads();
    }
}

// The grid of the wide tiles' kernels: up to 65,536 workgroups over the tiles,
// those of the others end at once.  S.K: the widest tile.
static dim3 wide_grid(unsigned tiles, const slot_layout &S) {
    const int64_t blocks = (S.K + kSlotCols - 1) / kSlotCols, y = 65536 / (int64_t)tiles;
    return dim3(tiles, (unsigned)(y < 1 ? 1 : y < blocks ? y : blocks));
}

// A row's entries are its slots up to the first padding slot, found by
// bisection (reading every slot of 500,000 rows of 34: 24 us).
__global__ void slot_len_kernel(int64_t n, slot_layout S, const int32_t *__restrict__ scol,
                                const int32_t *__restrict__ tail_ptr, int32_t *__restrict__ len) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const slot_tile T = slot_tile_of(S, i / kSlotRows);
    const int32_t *c = scol + T.start + i % kSlotRows;
    int64_t lo = 0, hi = T.width;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (c[mid * T.stride] >= 0) lo = mid + 1;
        else hi = mid;
    }
    len[i] = (int32_t)lo + (tail_ptr ? tail_ptr[i + 1] - tail_ptr[i] : 0);
}

template <typename V>
static hipError_t launch_csr_to_slots(hipStream_t s, int64_t n, const int32_t *rp, const int32_t *col,
                                      const void *val_, const slot_layout &S, int32_t *scol,
                                      void *sval_) {
    const unsigned tiles = grid_for(n, kSlotRows);
    const V *val = static_cast<const V *>(val_);
    V *sval = static_cast<V *>(sval_);
    if (S.sets || S.K <= kSlotWide)
        csr_to_slots_kernel<V><<<tiles, kSlotThreads, 0, s>>>(n, rp, col, val, S, scol, sval);
    if (S.K > kSlotWide)
        csr_to_wide_slots_kernel<V>
            <<<wide_grid(tiles, S), kSlotThreads, 0, s>>>(n, rp, col, val, S, scol, sval);
    return hipGetLastError();
}

hipError_t csr_to_slots(hipStream_t s, vt t, int64_t n, const int32_t *rp, const int32_t *col,
                        const void *val, const slot_layout &S, int32_t *scol, void *sval) {
    if (n == 0 || S.K == 0) return hipSuccess;
    return t == vt::f64 ? launch_csr_to_slots<double>(s, n, rp, col, val, S, scol, sval)
                        : launch_csr_to_slots<float>(s, n, rp, col, val, S, scol, sval);
}

hipError_t slot_lengths(hipStream_t s, int64_t n, const slot_layout &S, const int32_t *scol,
                        const int32_t *tail_ptr, int32_t *len) {
    if (n == 0) return hipSuccess;
    slot_len_kernel<<<grid_for(n, 256), 256, 0, s>>>(n, S, scol, tail_ptr, len);
    return hipGetLastError();
}

template <typename V>
static hipError_t launch_slots_to_csr(hipStream_t s, int64_t n, const slot_layout &S,
                                      const int32_t *scol, const void *sval, bool tail,
                                      const int32_t *rp, int32_t *col, void *val) {
    const unsigned tiles = grid_for(n, kSlotRows);
    const V *from = static_cast<const V *>(sval);
    V *to = static_cast<V *>(val);
    if (S.sets || S.K <= kSlotWide) {
        if (tail)
            slots_to_csr_kernel<V, true><<<tiles, kSlotThreads, 0, s>>>(n, S, scol, from, rp, col, to);
        else
            slots_to_csr_kernel<V, false><<<tiles, kSlotThreads, 0, s>>>(n, S, scol, from, rp, col, to);
    }
    if (S.K > kSlotWide)
        wide_slots_to_csr_kernel<V>
            <<<wide_grid(tiles, S), kSlotThreads, 0, s>>>(n, S, scol, from, rp, col, to);
    return hipGetLastError();
}

hipError_t slots_to_csr(hipStream_t s, vt t, int64_t n, const slot_layout &S, const int32_t *scol,
                        const void *sval, bool tail, const int32_t *rp, int32_t *col, void *val) {
    if (n == 0 || S.K == 0) return hipSuccess;
    return t == vt::f64 ? launch_slots_to_csr<double>(s, n, S, scol, sval, tail, rp, col, val)
                        : launch_slots_to_csr<float>(s, n, S, scol, sval, tail, rp, col, val);
}

// ------------------------------------------------------------------ HYB's tail
__global__ void tail_len_kernel(int64_t n, const int32_t *__restrict__ rp, int64_t K,
                                int32_t *__restrict__ len) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t l = rp[i + 1] - rp[i];
    len[i] = (int32_t)(l > K ? l - K : 0);
}

hipError_t tail_lengths(hipStream_t s, int64_t n, const int32_t *rp, int64_t K, int32_t *len) {
    if (n == 0) return hipSuccess;
    tail_len_kernel<<<grid_for(n, 256), 256, 0, s>>>(n, rp, K, len);
    return hipGetLastError();
}

// The tail's rows (trow, by csr_rows on tail_ptr) say where its entries are in
// CSR: entry q of row r is the (tail_ptr[r + 1] - q)-th from the row's end.  A
// thread per tail entry, so the few long rows that hold most of a tail are as
// parallel as the rest (a wavefront per row: 71 us for 250,000 lognormal rows
// with 3.5M tail entries).
template <typename V>
__global__ void csr_to_tail_kernel(int64_t tnnz, const int32_t *__restrict__ rp,
                                   const int32_t *__restrict__ col, const V *__restrict__ val,
                                   const int32_t *__restrict__ tail_ptr,
                                   const int32_t *__restrict__ trow, int32_t *__restrict__ tcol,
                                   V *__restrict__ tval) {
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= tnnz) return;
    const int32_t r = trow[q];
    const int64_t k = rp[r + 1] - (tail_ptr[r + 1] - q);
    tcol[q] = col[k];
    tval[q] = val[k];
}

hipError_t csr_to_tail(hipStream_t s, vt t, int64_t n, int64_t tnnz, const int32_t *rp,
                       const int32_t *col, const void *val, const int32_t *tail_ptr, int32_t *trow,
                       int32_t *tcol, void *tval) {
    if (tnnz == 0) return hipSuccess;
    const hipError_t e = csr_rows(s, n, tnnz, tail_ptr, trow);
    if (e != hipSuccess) return e;
    if (t == vt::f64)
        csr_to_tail_kernel<double><<<grid_for(tnnz, 256), 256, 0, s>>>(
            tnnz, rp, col, static_cast<const double *>(val), tail_ptr, trow, tcol,
            static_cast<double *>(tval));
    else
        csr_to_tail_kernel<float><<<grid_for(tnnz, 256), 256, 0, s>>>(
            tnnz, rp, col, static_cast<const float *>(val), tail_ptr, trow, tcol,
            static_cast<float *>(tval));
    return hipGetLastError();
}

template <typename V>
__global__ void tail_to_csr_kernel(int64_t tnnz, const int32_t *__restrict__ tail_ptr,
                                   const int32_t *__restrict__ trow, const int32_t *__restrict__ tcol,
                                   const V *__restrict__ tval, const int32_t *__restrict__ rp,
                                   int32_t *__restrict__ col, V *__restrict__ val) {
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= tnnz) return;
    const int32_t r = trow[q];
    const int64_t k = rp[r + 1] - (tail_ptr[r + 1] - q);
    col[k] = tcol[q];
    val[k] = tval[q];
}

hipError_t tail_to_csr(hipStream_t s, vt t, int64_t tnnz, const int32_t *tail_ptr,
                       const int32_t *trow, const int32_t *tcol, const void *tval,
                       const int32_t *rp, int32_t *col, void *val) {
    if (tnnz == 0) return hipSuccess;
    if (t == vt::f64)
        tail_to_csr_kernel<double><<<grid_for(tnnz, 256), 256, 0, s>>>(
            tnnz, tail_ptr, trow, tcol, static_cast<const double *>(tval), rp, col,
            static_cast<double *>(val));
    else
        tail_to_csr_kernel<float><<<grid_for(tnnz, 256), 256, 0, s>>>(
            tnnz, tail_ptr, trow, tcol, static_cast<const float *>(tval), rp, col,
            static_cast<float *>(val));
    return hipGetLastError();
}

// ------------------------------------------------------------------ exclusive scan
// Reduce-then-scan over tiles of 1024 lengths: tile sums, a single-block scan
// of the tile sums, then each tile scans itself from its offset.
constexpr int kScanBlock = 256;
constexpr int kScanItems = 4;
constexpr int kScanTile = kScanBlock * kScanItems;

int64_t scan_tmp_elems(int64_t n) { return (n + kScanTile - 1) / kScanTile + 1; }

__device__ inline int32_t block_excl_scan(int32_t v, int32_t *lds, int32_t *total) {
    // inclusive wave scan, then wave offsets
    const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
    int32_t x = v;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const int32_t u = __shfl_up(x, off);
        if (lane >= off) x += u;
    }
    if (lane == kWave - 1) lds[w] = x;
    __syncthreads();
    int32_t woff = 0, tot = 0;
    for (int j = 0; j < kScanBlock / kWave; ++j) {
        if (j < w) woff += lds[j];
        tot += lds[j];
    }
    __syncthreads();
    *total = tot;
    return woff + x - v;
}

__global__ void scan_tile_sums(int64_t n, const int32_t *__restrict__ len, int32_t *__restrict__ sums) {
    __shared__ int32_t lds[kScanBlock / kWave];
    const int64_t base = (int64_t)blockIdx.x * kScanTile + threadIdx.x * kScanItems;
    int32_t v = 0;
#pragma unroll
    for (int j = 0; j < kScanItems; ++j)
        if (base + j < n) v += len[base + j];
    int32_t tot;
    block_excl_scan(v, lds, &tot);
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

__global__ void scan_sums_kernel(int64_t tiles, int32_t *__restrict__ sums) {
    __shared__ int32_t lds[kScanBlock / kWave];
    int32_t carry = 0;
    for (int64_t base = 0; base < tiles; base += kScanBlock) {
        const int64_t i = base + threadIdx.x;
        const int32_t v = i < tiles ? sums[i] : 0;
        int32_t tot;
        const int32_t ex = block_excl_scan(v, lds, &tot);
        if (i < tiles) sums[i] = carry + ex;
        carry += tot;
        __syncthreads();
    }
    if (threadIdx.x == 0) sums[tiles] = carry;
}

__global__ void scan_tiles_kernel(int64_t n, const int32_t *__restrict__ len,
                                  const int32_t *__restrict__ sums, int32_t *__restrict__ out) {
    __shared__ int32_t lds[kScanBlock / kWave];
    const int64_t base = (int64_t)blockIdx.x * kScanTile + threadIdx.x * kScanItems;
    int32_t v[kScanItems], t = 0;
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
        v[j] = base + j < n ? len[base + j] : 0;
        t += v[j];
    }
    int32_t tot;
    int32_t o = sums[blockIdx.x] + block_excl_scan(t, lds, &tot);
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
        if (base + j < n) out[base + j] = o;
        o += v[j];
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) out[n] = sums[gridDim.x];
}

hipError_t exclusive_scan(hipStream_t s, int64_t n, const int32_t *len, int32_t *out, int32_t *tmp) {
    const int64_t tiles = (n + kScanTile - 1) / kScanTile;
    if (tiles == 0) {
        return hipMemsetAsync(out, 0, sizeof(int32_t), s);
    }
    scan_tile_sums<<<(unsigned)tiles, kScanBlock, 0, s>>>(n, len, tmp);
    scan_sums_kernel<<<1, kScanBlock, 0, s>>>(tiles, tmp);
    scan_tiles_kernel<<<(unsigned)tiles, kScanBlock, 0, s>>>(n, len, tmp, out);
    return hipGetLastError();
}

// ------------------------------------------------------------------ array copies
// Up to three device arrays copied by one launch with 16-byte non-temporal
// loads and stores: bound by memory.  The columns and values of an ELL matrix
// with 18M slots (216 MB, read and written) take 59 us, two of the runtime's
// copies 87 us.  A thread takes 16 bytes; an array's last bytes past a multiple
// of 16 go byte by byte.
typedef uint32_t copy_quad __attribute__((ext_vector_type(4)));

struct copy_args {
    array_copy a[3];
    int64_t units[3];  // 16-byte units of each array, the last one partial
};

__global__ __launch_bounds__(256) void copy_arrays_kernel(copy_args c) {
    int64_t u = (int64_t)blockIdx.x * 256 + threadIdx.x;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        if (u < c.units[k]) {
            const char *src = static_cast<const char *>(c.a[k].src) + u * 16;
            char *dst = static_cast<char *>(c.a[k].dst) + u * 16;
            const int64_t left = c.a[k].bytes - u * 16;
            if (left >= 16)
                __builtin_nontemporal_store(
                    __builtin_nontemporal_load(reinterpret_cast<const copy_quad *>(src)),
                    reinterpret_cast<copy_quad *>(dst));
            else
                for (int64_t q = 0; q < left; ++q) dst[q] = src[q];
            return;
        }
        u -= c.units[k];
    }
}

// What the kernel may write: memory of the current device.  A caller's buffer
// that is on the host or on another device is left to the runtime.
static bool kernel_writable(const void *p) {
    hipPointerAttribute_t at;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || hipPointerGetAttributes(&at, p) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return at.type == hipMemoryTypeDevice && at.device == dev;
}

hipError_t copy_arrays(hipStream_t s, const array_copy &a, const array_copy &b, const array_copy &c) {
    copy_args args{{a, b, c}, {}};
    int64_t units = 0;
    for (int k = 0; k < 3; ++k) {
        array_copy &x = args.a[k];
        if (!x.dst || x.bytes <= 0) x.bytes = 0;
        else if ((((uintptr_t)x.dst | (uintptr_t)x.src) & 15) || !kernel_writable(x.dst)) {
            const hipError_t e = hipMemcpyAsync(x.dst, x.src, x.bytes, hipMemcpyDeviceToDevice, s);
            if (e != hipSuccess) return e;
            x.bytes = 0;
        }
        units += args.units[k] = (x.bytes + 15) / 16;
    }
    if (units == 0) return hipSuccess;
    copy_arrays_kernel<<<grid_for(units, 256), 256, 0, s>>>(args);
    return hipGetLastError();
}

// ------------------------------------------------------------------ casts
template <typename A, typename B>
__global__ void cast_kernel(int64_t n, const A *__restrict__ a, B *__restrict__ b) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) b[i] = (B)a[i];
}

hipError_t cast_values(hipStream_t s, vt from, vt to, int64_t n, const void *src, void *dst) {
    if (n == 0) return hipSuccess;
    const unsigned g = grid_for(n, 256);
    if (from == vt::f64 && to == vt::f32)
        cast_kernel<double, float><<<g, 256, 0, s>>>(n, static_cast<const double *>(src), static_cast<float *>(dst));
    else if (from == vt::f32 && to == vt::f64)
        cast_kernel<float, double><<<g, 256, 0, s>>>(n, static_cast<const float *>(src), static_cast<double *>(dst));
    else
        return hipMemcpyAsync(dst, src, n * vsize(from), hipMemcpyDeviceToDevice, s);
    return hipGetLastError();
}

}  // namespace gko
