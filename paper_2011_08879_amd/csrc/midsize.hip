// Krylov iterations of small and mid-size systems (mid_fits).
//
// Such an iteration is bound by the chain of dependent kernels, not by memory:
// its vectors and the matrix sit in the caches, and a launch costs about as
// much as the work in it.  So an iteration here is as few kernels as the
// recurrence has reductions that must end before the next product or update:
//   CG, flexible CG     2  (product, update)              5 on large systems
//   BiCGSTAB            3  (product, product, update)     9
//   CGS                 2  (product, product)             7
//   pipelined CG        1                                 3
// Two changes make that possible:
//  * the kernel that needs a reduction's totals sums the partials itself (every
//    workgroup, in the same fixed order, so all get the same bits) and applies
//    the scalar step to its own copy of the state; workgroup 0 stores the
//    result for the next kernel.  Each workgroup reads every partial once, and
//    workgroups of 1024 threads keep those reads few.
//  * the vector updates that would come before a product are formed inside it,
//    from the vectors they combine, for every gathered entry (a `view`): twice
//    or three times the gathers, which the caches serve here, but on large
//    systems cost more than the vector pass they save.
// A thread issues the loads of its matrix entries and of all gathered vectors
// before it waits for the totals, so the two latencies overlap.
//
// Vectors that a kernel both gathers and replaces alternate between two
// buffers.  States alternate too: a kernel reads one and workgroup 0 writes
// another, so no workgroup can read a state that is being replaced.
//
// Where a thread has one row the sums take the order of the kernels for large
// systems (partials of 256 threads at the same places, then the finalize
// kernel's tree), so the iterates are theirs bit for bit: BiCGSTAB's can
// magnify a difference in rounding 10^7-fold.  With more rows to a thread a
// workgroup leaves one partial, which is cheaper to sum (CG on 512,000 rows
// 29.6 -> 26.9 us).
// Per iteration, five to nine launches against these (64 iterations, the
// solve's start and the host's polls included, all workgroups of 1024
// threads; kHalfT below has what smaller ones gave on top): CG on the 3D
// Poisson matrix (SELL-P) 16^3 rows 19.4 -> 16.9 us, 48^3 22.8 -> 17.8, 64^3
// 26.5 -> 19.4, 110^3 60.6 -> 51.3; block-Jacobi(8) CG 48^3 24.1 -> 20.1;
// pipelined CG 48^3 18.2 -> 14.6, 110^3 62 -> 48.5; BiCGSTAB on 250^2
// convection-diffusion (ELL) 48.6 -> 33.6, 500^2 57.5 -> 36.4; CGS 250^2 59.6 ->
// 39.1.
#include <cmath>

#include "bj_tile.hpp"
#include "device.hpp"
#include "kernels.hpp"
#include "krylov_ops.hpp"
#include "solver_kernels.hpp"
#include "solver_state.hpp"

namespace gko {

namespace {

// Threads of a workgroup: 1024, and 512 where these still are one round of the
// 256 compute units: 1024 would leave half of them idle.  us per iteration with
// 1024 and with 512: CG 48^3 rows 13.1 / 11.1, 30^3 15.6 / 13.0, 50^3 in CSR
// 16.7 / 14.3; BiCGSTAB 211 x 307 rows 26.2 / 22.2; CGS 200^2 33.0 / 26.4.
constexpr int kT = 1024, kHalfT = 512;
inline bool half_blocks(int64_t threads) { return threads <= 256 * kHalfT; }
constexpr int kPart = 256;        // threads that share one partial
static_assert(kMidRows <= kSpreadCols, "the columns' spread is known");
constexpr int kEntries = 8;       // a row's entries loaded before the totals are waited for

// A grid over n rows: one workgroup for each rows_per_block rows if at most
// `most` are enough, else kMidBlocks / 2 with several rows to a thread.
inline int mid_blocks(int64_t n, int64_t rows_per_block, int most) {
    const int64_t g = (n + rows_per_block - 1) / rows_per_block;
    return (int)(g < 1 ? 1 : g <= most ? g : kMidBlocks / 2);
}

// Partials that a grid leaves for each sum: one per kPart threads that have a
// row (a term), or with several rows to a thread one per workgroup.
inline int mid_parts(int64_t terms, int grid, int terms_per_block) {
    const int64_t g = (terms + kPart - 1) / kPart;
    return (int64_t)grid * terms_per_block < terms ? grid : g < 1 ? 1 : (int)g;
}

// ------------------------------------------------------------ totals
// The totals a kernel's scalar step is for: the partials' loads are issued
// first (load), summed when they are needed (mid_enter), in the order of
// finalize_kernel: 1024 threads' strided sums, wavefront by wavefront, then
// the 16 wavefronts' totals.  A workgroup of T < 1024 threads does the share
// of 1024 / T wavefronts in each of its own.
constexpr int kSumSlots = kFinalizeBlock / kWave;
constexpr int kSumRounds = (kMidBlocks * (kT / kPart) + kFinalizeBlock - 1) / kFinalizeBlock;

// The state k.in comes with them, a word per thread: read by the one thread
// that works on it, after the sums, it was a second wait for memory.
constexpr int kStateWords = sizeof(krylov_scalars) / sizeof(uint64_t);
static_assert(sizeof(krylov_scalars) % sizeof(uint64_t) == 0 && kStateWords <= kWave, "whole words");

template <int T, int NV>
struct mid_totals {
    static constexpr int S = kFinalizeBlock / T;
    double t[NV][S][kSumRounds];
    uint64_t word;  // of the state
    __device__ void load(const scalar_link &k) {
        if (threadIdx.x < kStateWords) word = reinterpret_cast<const uint64_t *>(k.in)[threadIdx.x];
        if (!k.out) return;
#pragma unroll
        for (int j = 0; j < NV; ++j)
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int q = 0; q < kSumRounds; ++q) {
                    const int b = q * kFinalizeBlock + s * T + threadIdx.x;
                    t[j][s][q] = b < k.g ? k.sums[(int64_t)j * k.g + b] : 0.0;
                }
    }
    __device__ void to_slots(double (*slots)[kSumSlots]) const {
#pragma unroll
        for (int j = 0; j < NV; ++j)
#pragma unroll
            for (int s = 0; s < S; ++s) {
                double v = t[j][s][0];
#pragma unroll
                for (int q = 1; q < kSumRounds; ++q) v += t[j][s][q];
                v = wave_total(v);
                if (threadIdx.x % kWave == 0) slots[j][s * (T / kWave) + threadIdx.x / kWave] = v;
            }
    }
};

// The state after the kernel's scalar step, in LDS for the whole workgroup;
// false (alike in all workgroups) when the solve has ended.  One thread works
// on the LDS copy itself: a copy of the state in local variables was moved to
// LDS by the compiler, for every thread of the workgroup (41 KB; the update
// kernel 6 -> 11 us).
template <int T, int NV, typename Step>
__device__ inline bool mid_enter(const scalar_link &k, const mid_totals<T, NV> &totals,
                                 const Step &step, krylov_scalars &st) {
    __shared__ double slots[NV][kSumSlots];
    uint64_t *words = reinterpret_cast<uint64_t *>(&st);
    if (threadIdx.x < kStateWords) words[threadIdx.x] = totals.word;
    if (k.out) totals.to_slots(slots);  // uniform
    __syncthreads();
    if (!k.out) return st.done == 0;
    if (threadIdx.x < kWave) {
        double o[NV] = {};
#pragma unroll
        for (int j = 0; j < NV; ++j)
            o[j] = wave_total(threadIdx.x < kSumSlots ? slots[j][threadIdx.x] : 0.0);
        if (threadIdx.x == 0 && st.done == 0) step(st, o);
    }
    __syncthreads();
    if (blockIdx.x == 0 && threadIdx.x < kStateWords)
        reinterpret_cast<uint64_t *>(k.out)[threadIdx.x] = words[threadIdx.x];
    return st.done == 0;
}

// partials[j * g + p] <- the sums of every kPart threads (four wavefronts, in
// the order of block_sum), or of the whole workgroup where g is the grid's.
// FUSED: sums that the kernels for large systems form in a product; they
// leave their partials in hardware workgroup order.  PAIR: a sum's terms are
// in the even threads, and kPart pairs share a partial.
template <int T, int NV, bool FUSED, bool PAIR>
__device__ inline void mid_store_sums(const double (&acc)[NV], int g, int64_t block,
                                      double *__restrict__ partials) {
    constexpr int NW = PAIR ? T / kWave / 2 : T / kWave, P = NW * kWave / kPart;
    __shared__ double red[NV][T / kWave];
    __shared__ double pairs[PAIR ? NV : 1][PAIR ? T / 2 : 1];
    const int wv = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    if constexpr (PAIR) {
#pragma unroll
        for (int j = 0; j < NV; ++j)
            if (threadIdx.x % 2 == 0) pairs[j][threadIdx.x / 2] = acc[j];
        __syncthreads();
    }
    if (wv < NW) {
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const double s = wave_total(PAIR ? pairs[j][PAIR ? threadIdx.x : 0] : acc[j]);
            if (lane == 0) red[j][wv] = s;
        }
    }
    __syncthreads();
    // (a workgroup of kHalfT threads with one partial has one row to a thread)
    if (P > 1 && g == (int)gridDim.x) {
        if (threadIdx.x < NV) {
            double s = 0.0;
#pragma unroll
            for (int w = 0; w < NW; w += 4) {
                const double *r = &red[threadIdx.x][w];
                s += (r[3] + r[2]) + (r[1] + r[0]);
            }
            partials[(int64_t)threadIdx.x * g + block] = s;
        }
    } else if (threadIdx.x < NV * P) {
        const int j = threadIdx.x / P, q = threadIdx.x % P;
        const double *r = &red[j][4 * q];
        const int64_t p = block * P + q;
        if (p < g)
            partials[(int64_t)j * g + (FUSED ? xcd_block_inverse(p, g) : p)] =
                (r[3] + r[2]) + (r[1] + r[0]);
    }
}

// acc + x y in an even thread, the terms of its row and of the next thread's
// row in this order (ELL's row pairs).
__device__ inline double add_pair(double acc, double x, double y) {
    const double x1 = __shfl_down(x, 1), y1 = __shfl_down(y, 1);
    acc += x * y;
    return acc + x1 * y1;
}

// ------------------------------------------------------------ products
// A row's entries as a strided walk through the column and value arrays, the
// same loop for every format: CSR with G lanes per row (lane g takes entries
// g, g + G, ...), ELL and SELL-P (padding slots have column -1).
struct row_walk {
    int64_t start, stride;
    int32_t count;
};

template <fused_matrix::kind F, int G>
__device__ inline row_walk walk_of(const fused_matrix &A, int64_t i, int g) {
    if constexpr (F == fused_matrix::csr) {
        const int32_t b = A.rp[i] + g, e = A.rp[i + 1];
        return {b, G, e > b ? (e - b + G - 1) / G : 0};
    } else if constexpr (F == fused_matrix::ell) {
        return {i, A.ld, (int32_t)A.K};
    } else {
        const int64_t k = i / kSellpSlice, base = A.sets[k];
        return {base + i - k * kSellpSlice, kSellpSlice, (int32_t)((A.sets[k + 1] - base) / kSellpSlice)};
    }
}

// out = A view, with the view's own vectors updated and its sums left as
// partials.  A view W holds the pointers and says how an entry of the vector
// comes from the RAW vectors it is formed from, and which products x y its NV
// sums are of.
template <fused_matrix::kind F, int G, int T, typename W>
__global__ __launch_bounds__(T) void mid_product_kernel(fused_matrix A, W view, scalar_link k,
                                                         int parts, double *__restrict__ partials) {
    using V = typename W::value_type;
    constexpr int RT = T / G;
    constexpr bool PAIR = F == fused_matrix::ell && W::kFused;
    __shared__ krylov_scalars st;
    const int32_t *__restrict__ col = F == fused_matrix::csr   ? A.col
                                      : F == fused_matrix::ell ? A.ecol
                                                               : A.scol;
    const V *__restrict__ val = static_cast<const V *>(F == fused_matrix::csr   ? A.val
                                                       : F == fused_matrix::ell ? A.eval
                                                                                : A.sval);
    const int g = threadIdx.x % G;
    mid_totals<T, W::Step::NV> totals;
    totals.load(k);
    double acc[W::NV] = {};
    bool entered = false;
    // each XCD takes one contiguous range of rows per round
    const int64_t block = xcd_block(blockIdx.x, gridDim.x);
    for (int64_t r0 = block * RT; r0 < A.n; r0 += (int64_t)gridDim.x * RT) {
        const int64_t i = r0 + threadIdx.x / G;
        row_walk w{0, 0, 0};
        if (i < A.n) w = walk_of<F, G>(A, i, g);
        int32_t c[kEntries];
        V v[kEntries], raw[kEntries][W::RAW];
#pragma unroll
        for (int u = 0; u < kEntries; ++u) {
            const bool ok = u < w.count;
            c[u] = ok ? col[w.start + u * w.stride] : -1;
            v[u] = ok ? val[w.start + u * w.stride] : V(0);
        }
        typename W::own_row own;
        if (i < A.n) view.load_own(i, own);
#pragma unroll
        for (int u = 0; u < kEntries; ++u) view.load(c[u] >= 0 ? c[u] : 0, raw[u]);
        if (!entered) {
            if (!mid_enter<T>(k, totals, view.step, st)) return;
            entered = true;
        }
        V s = V(0);
#pragma unroll
        for (int u = 0; u < kEntries; ++u) {
            const V t = s + v[u] * view.value(st, raw[u]);
            s = c[u] >= 0 ? t : s;
        }
        for (int32_t u0 = kEntries; u0 < w.count; u0 += 4) {
            int32_t cc[4];
            V vv[4], rr[4][W::RAW];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const bool ok = u0 + u < w.count;
                cc[u] = ok ? col[w.start + (u0 + u) * w.stride] : -1;
                vv[u] = ok ? val[w.start + (u0 + u) * w.stride] : V(0);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) view.load(cc[u] >= 0 ? cc[u] : 0, rr[u]);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const V t = s + vv[u] * view.value(st, rr[u]);
                s = cc[u] >= 0 ? t : s;
            }
            if (F != fused_matrix::csr && cc[3] < 0) break;  // the row's padding has begun
        }
        if constexpr (G > 1) s = subwarp<G>::reduce_sum(s);
        double x[W::NV] = {}, y[W::NV] = {};
        if (i < A.n && g == 0) view.finish(st, i, own, s, x, y);
#pragma unroll
        for (int j = 0; j < W::NV; ++j) {
            if constexpr (PAIR) acc[j] = add_pair(acc[j], x[j], y[j]);
            else acc[j] += x[j] * y[j];
        }
    }
    mid_store_sums<T, W::NV, W::kFused, PAIR>(acc, parts, block, partials);
}

// CG: p = z + beta p_old, q = A p, p.q.
template <bool FLEX>
struct cg_beta_step {
    static constexpr int NV = FLEX ? 3 : 2;
    __device__ void operator()(krylov_scalars &s, const double *o) const {
        cg_update_step{FLEX}(s, o);
    }
};

template <typename V, bool FLEX>
struct cg_view {
    // kFused: the sums of a product kernel for large systems
    using value_type = V;
    using Step = cg_beta_step<FLEX>;
    static constexpr int RAW = 2, NV = 1;
    static constexpr bool kFused = true;
    struct own_row {
        V r[RAW];
    };
    const V *z, *p_old;
    V *p, *q;
    Step step;
    __device__ void load(int64_t c, V (&r)[RAW]) const {
        r[0] = z[c];
        r[1] = p_old[c];
    }
    __device__ void load_own(int64_t i, own_row &o) const { load(i, o.r); }
    __device__ V value(const krylov_scalars &s, const V (&r)[RAW]) const {
        return (V)((double)r[0] + s.beta * (double)r[1]);
    }
    __device__ void finish(const krylov_scalars &s, int64_t i, const own_row &o, V out,
                           double (&x)[NV], double (&y)[NV]) const {
        const V pi = value(s, o.r);
        p[i] = pi;
        q[i] = out;
        x[0] = (double)pi;
        y[0] = (double)out;
    }
};

// BiCGSTAB: p = r + beta (p_old - omega v_old), v = A p, rhat.v.
struct bicg_v_view {
    using value_type = double;
    using Step = bicg_update_step;
    static constexpr int RAW = 3, NV = 1;
    static constexpr bool kFused = true;
    struct own_row {
        double r[RAW], rh;
    };
    const double *r, *p_old, *v_old, *rh;
    double *p, *v;
    Step step;
    __device__ void load(int64_t c, double (&o)[RAW]) const {
        o[0] = r[c];
        o[1] = p_old[c];
        o[2] = v_old[c];
    }
    __device__ void load_own(int64_t i, own_row &o) const {
        load(i, o.r);
        o.rh = rh[i];
    }
    __device__ double value(const krylov_scalars &s, const double (&o)[RAW]) const {
        return o[0] + s.beta * (o[1] - s.omega * o[2]);
    }
    __device__ void finish(const krylov_scalars &s, int64_t i, const own_row &o, double out,
                           double (&x)[NV], double (&y)[NV]) const {
        p[i] = value(s, o.r);
        v[i] = out;
        x[0] = o.rh;
        y[0] = out;
    }
};

// BiCGSTAB: s = r - alpha v, t = A s, and s.s, t.s, t.t.
struct bicg_t_view {
    using value_type = double;
    using Step = bicg_alpha_step;
    static constexpr int RAW = 2, NV = 3;
    static constexpr bool kFused = true;
    struct own_row {
        double r[RAW];
    };
    const double *r, *v;
    double *t;
    Step step;
    __device__ void load(int64_t c, double (&o)[RAW]) const {
        o[0] = r[c];
        o[1] = v[c];
    }
    __device__ void load_own(int64_t i, own_row &o) const { load(i, o.r); }
    __device__ double value(const krylov_scalars &s, const double (&o)[RAW]) const {
        return o[0] - s.alpha * o[1];
    }
    __device__ void finish(const krylov_scalars &s, int64_t i, const own_row &o, double out,
                           double (&x)[NV], double (&y)[NV]) const {
        const double si = value(s, o.r);
        t[i] = out;
        x[0] = y[0] = si;
        x[1] = out;
        y[1] = si;
        x[2] = y[2] = out;
    }
};

// CGS: u = r + beta q, p = u + beta (q + beta p_old), t = A p, t.rhat.
struct cgs_t_view {
    using value_type = double;
    using Step = cgs_update_step;
    static constexpr int RAW = 3, NV = 1;
    static constexpr bool kFused = true;
    struct own_row {
        double r[RAW], rh;
    };
    const double *r, *q, *p_old, *rh;
    double *u, *p, *t;
    Step step;
    __device__ void load(int64_t c, double (&o)[RAW]) const {
        o[0] = r[c];
        o[1] = q[c];
        o[2] = p_old[c];
    }
    __device__ void load_own(int64_t i, own_row &o) const {
        load(i, o.r);
        o.rh = rh[i];
    }
    __device__ double value(const krylov_scalars &s, const double (&o)[RAW]) const {
        const double ui = o[0] + s.beta * o[1];
        return ui + s.beta * (o[1] + s.beta * o[2]);
    }
    __device__ void finish(const krylov_scalars &s, int64_t i, const own_row &o, double out,
                           double (&x)[NV], double (&y)[NV]) const {
        u[i] = o.r[0] + s.beta * o.r[1];
        p[i] = value(s, o.r);
        t[i] = out;
        x[0] = o.rh;
        y[0] = out;
    }
};

// CGS: q = u - alpha t, w = u + q, x += alpha w, r -= alpha A w, r.r, r.rhat.
struct cgs_w_view {
    using value_type = double;
    using Step = cgs_alpha_step;
    static constexpr int RAW = 2, NV = 2;
    static constexpr bool kFused = false;
    struct own_row {
        double r[RAW], rh, x, res;
    };
    const double *u, *t, *rh;
    double *q, *sol, *r;
    Step step;
    __device__ void load(int64_t c, double (&o)[RAW]) const {
        o[0] = u[c];
        o[1] = t[c];
    }
    __device__ void load_own(int64_t i, own_row &o) const {
        load(i, o.r);
        o.rh = rh[i];
        o.x = sol[i];
        o.res = r[i];
    }
    __device__ double value(const krylov_scalars &s, const double (&o)[RAW]) const {
        const double qi = o[0] - s.alpha * o[1];
        return o[0] + qi;
    }
    __device__ void finish(const krylov_scalars &s, int64_t i, const own_row &o, double out,
                           double (&x)[NV], double (&y)[NV]) const {
        const double qi = o.r[0] - s.alpha * o.r[1], wi = o.r[0] + qi;
        q[i] = qi;
        sol[i] = o.x + s.alpha * wi;
        const double ri = o.res - s.alpha * out;
        r[i] = ri;
        x[0] = y[0] = x[1] = ri;
        y[1] = o.rh;
    }
};

// Pipelined CG without a preconditioner: n = A w and the whole update;
// gamma = r.r, delta = w.r, r.r.
template <typename V>
struct pipe_view {
    using value_type = V;
    using Step = pipe_update_step;
    static constexpr int RAW = 1, NV = 3;
    static constexpr bool kFused = false;
    struct own_row {
        V w, z, s, p, x, r;
    };
    const V *w_old;
    V *w, *z, *s, *p, *sol, *r;
    Step step;
    __device__ void load(int64_t c, V (&o)[RAW]) const { o[0] = w_old[c]; }
    __device__ void load_own(int64_t i, own_row &o) const {
        o = own_row{w_old[i], z[i], s[i], p[i], sol[i], r[i]};
    }
    __device__ V value(const krylov_scalars &, const V (&o)[RAW]) const { return o[0]; }
    __device__ void finish(const krylov_scalars &k, int64_t i, const own_row &o, V out,
                           double (&x)[NV], double (&y)[NV]) const {
        const V zi = (V)((double)out + k.beta * (double)o.z);
        const V si = (V)((double)o.w + k.beta * (double)o.s);
        const V pi = (V)((double)o.r + k.beta * (double)o.p);
        z[i] = zi;
        s[i] = si;
        p[i] = pi;
        sol[i] = (V)((double)o.x + k.alpha * (double)pi);
        const V ri = (V)((double)o.r - k.alpha * (double)si);
        r[i] = ri;
        const V wi = (V)((double)o.w - k.alpha * (double)zi);
        w[i] = wi;
        x[0] = x[2] = y[0] = y[1] = y[2] = (double)ri;
        x[1] = (double)wi;
    }
};

// ------------------------------------------------------------ updates
// x += alpha p; r -= alpha q; z = M^-1 r; r.z, r.r (and z.(r - r_old)).
// Blocks of 16 rows of doubles always in half-size workgroups, for their LDS.
template <typename V, int BS, bool FLEX, int T>
__global__ __launch_bounds__(T) void mid_cg_update_kernel(
    int64_t n, V *__restrict__ x, V *__restrict__ r, V *__restrict__ z, const V *__restrict__ p,
    const V *__restrict__ q, const V *__restrict__ inv, scalar_link k, int parts,
    double *__restrict__ partials) {
    __shared__ krylov_scalars st;
    __shared__ bj_lds<V, BS, T> L;
    mid_totals<T, 1> totals;
    totals.load(k);
    constexpr int NV = cg_beta_step<FLEX>::NV;
    double acc[NV] = {};
    bool entered = false;
    const int64_t block = xcd_block(blockIdx.x, gridDim.x);
    for (int64_t base = block * T; base < n; base += (int64_t)gridDim.x * T) {
        const int64_t i = base + threadIdx.x;
        const bool ok = i < n;
        const V xi = ok ? x[i] : V(0), pi = ok ? p[i] : V(0);
        const V ro = ok ? r[i] : V(0), qi = ok ? q[i] : V(0);
        if constexpr (BS > 0) bj_tile_stage<V, BS, T>(n, base, inv, L);
        if (!entered) {
            if (!mid_enter<T>(k, totals, cg_alpha_step{}, st)) return;
            entered = true;
        }
        const double alpha = st.alpha;
        const V ri = ok ? (V)((double)ro - alpha * (double)qi) : V(0);
        if (ok) {
            x[i] = (V)((double)xi + alpha * (double)pi);
            r[i] = ri;
        }
        V zi = ri;
        if constexpr (BS > 0) zi = bj_tile_apply<V, BS, T>(ri, L);
        if (ok) {
            if constexpr (BS > 0) z[i] = zi;
            acc[0] += (double)ri * (double)zi;
            acc[1] += (double)ri * (double)ri;
            if constexpr (FLEX) acc[2] += (double)zi * ((double)ri - (double)ro);
        }
    }
    mid_store_sums<T, NV, false, false>(acc, parts, block, partials);
}

// BiCGSTAB: s = r - alpha v; x += alpha p + omega s; r = s - omega t; r.r and
// rhat.r.  At the half step only x += alpha p.
struct bicg_half_step {
    static constexpr int NV = 3;
    __device__ void operator()(krylov_scalars &s, const double *o) const {
        bicg_s_step{}(s, o);
        if (s.done == 0) bicg_omega_step{}(s, o + 1);
    }
};

template <int T>
__global__ __launch_bounds__(T) void mid_bicg_update_kernel(
    int64_t n, double *__restrict__ x, double *__restrict__ r, const double *__restrict__ rh,
    const double *__restrict__ p, const double *__restrict__ v, const double *__restrict__ t,
    scalar_link k, int parts, double *__restrict__ partials) {
    __shared__ krylov_scalars st;
    mid_totals<T, 3> totals;
    totals.load(k);
    double acc[2] = {};
    bool entered = false;
    const int64_t block = xcd_block(blockIdx.x, gridDim.x);
    for (int64_t i = block * T + threadIdx.x; i - threadIdx.x < n; i += (int64_t)gridDim.x * T) {
        const bool ok = i < n;
        const double xi = ok ? x[i] : 0.0, ro = ok ? r[i] : 0.0, rhi = ok ? rh[i] : 0.0;
        const double pi = ok ? p[i] : 0.0, vi = ok ? v[i] : 0.0, ti = ok ? t[i] : 0.0;
        if (!entered) {
            if (!mid_enter<T>(k, totals, bicg_half_step{}, st)) return;
            entered = true;
        }
        if (!ok) continue;
        if (st.half) {
            x[i] = xi + st.alpha * pi;
        } else {
            const double si = ro - st.alpha * vi;
            x[i] = xi + st.alpha * pi + st.omega * si;
            const double ri = si - st.omega * ti;
            r[i] = ri;
            acc[0] += ri * ri;
            acc[1] += rhi * ri;
        }
    }
    mid_store_sums<T, 2, false, false>(acc, parts, block, partials);
}

// The scalar step on the sums that an interval's last kernel left.
template <typename Step>
__global__ __launch_bounds__(kT) void mid_close_kernel(scalar_link k, Step step) {
    __shared__ krylov_scalars st;
    mid_totals<kT, Step::NV> totals;
    totals.load(k);
    (void)mid_enter<kT>(k, totals, step, st);
}

// ------------------------------------------------------------ launches
template <typename W>
hipError_t launch_product(hipStream_t s, const fused_matrix &A, const W &view, const scalar_link &k,
                          const mid_sums &out, int most = kMidBlocks / 2) {
    const int lanes = A.format == fused_matrix::csr ? A.lanes : 1;
    const auto launch = [&](auto threads) {
        constexpr int T = decltype(threads)::value;
        const int g = mid_blocks(A.n, T / lanes, most);
        const bool pair = A.format == fused_matrix::ell && W::kFused;
        const int parts = pair ? mid_parts((A.n + 1) / 2, g, T / 2) : mid_parts(A.n * lanes, g, T);
        *out.parts = parts;
        double *P = out.partials;
        if (A.format == fused_matrix::ell)
            mid_product_kernel<fused_matrix::ell, 1, T, W><<<g, T, 0, s>>>(A, view, k, parts, P);
        else if (A.format == fused_matrix::sellp)
            mid_product_kernel<fused_matrix::sellp, 1, T, W><<<g, T, 0, s>>>(A, view, k, parts, P);
        else if (lanes == 1)
            mid_product_kernel<fused_matrix::csr, 1, T, W><<<g, T, 0, s>>>(A, view, k, parts, P);
        else if (lanes == 4)
            mid_product_kernel<fused_matrix::csr, 4, T, W><<<g, T, 0, s>>>(A, view, k, parts, P);
        else if (lanes == 8)
            mid_product_kernel<fused_matrix::csr, 8, T, W><<<g, T, 0, s>>>(A, view, k, parts, P);
        else if (lanes == 32)
            mid_product_kernel<fused_matrix::csr, 32, T, W><<<g, T, 0, s>>>(A, view, k, parts, P);
        else
            return hipErrorInvalidValue;
        return hipGetLastError();
    };
    return half_blocks(A.n * lanes) ? launch(std::integral_constant<int, kHalfT>{})
                                    : launch(std::integral_constant<int, kT>{});
}

template <typename V, bool FLEX, int BS>
hipError_t launch_cg_update_bs(hipStream_t s, int64_t n, void *x, void *r, void *z, const void *p,
                               const void *q, const void *inv, const scalar_link &k,
                               const mid_sums &out) {
    const auto launch = [&](auto threads) {
        constexpr int T = decltype(threads)::value;
        const int g = mid_blocks(n, T, kMidBlocks / 2), parts = mid_parts(n, g, T);
        *out.parts = parts;
        mid_cg_update_kernel<V, BS, FLEX, T><<<g, T, 0, s>>>(
            n, static_cast<V *>(x), static_cast<V *>(r), static_cast<V *>(z),
            static_cast<const V *>(p), static_cast<const V *>(q), static_cast<const V *>(inv), k,
            parts, out.partials);
        return hipGetLastError();
    };
    constexpr int kMost = BS == 16 && sizeof(V) == 8 ? kHalfT : kT;
    return half_blocks(n) ? launch(std::integral_constant<int, kHalfT>{})
                          : launch(std::integral_constant<int, kMost>{});
}

template <typename V, bool FLEX>
hipError_t launch_cg_update(hipStream_t s, int64_t n, void *x, void *r, void *z, const void *p,
                            const void *q, const void *inv, int bs, const scalar_link &k,
                            const mid_sums &out) {
    switch (bs) {
        case 0: return launch_cg_update_bs<V, FLEX, 0>(s, n, x, r, z, p, q, inv, k, out);
        case 1: return launch_cg_update_bs<V, FLEX, 1>(s, n, x, r, z, p, q, inv, k, out);
        case 2: return launch_cg_update_bs<V, FLEX, 2>(s, n, x, r, z, p, q, inv, k, out);
        case 4: return launch_cg_update_bs<V, FLEX, 4>(s, n, x, r, z, p, q, inv, k, out);
        case 8: return launch_cg_update_bs<V, FLEX, 8>(s, n, x, r, z, p, q, inv, k, out);
        case 16: return launch_cg_update_bs<V, FLEX, 16>(s, n, x, r, z, p, q, inv, k, out);
        default: return hipErrorInvalidValue;
    }
}

template <typename Step>
hipError_t launch_close(hipStream_t s, const scalar_link &k, const Step &step) {
    mid_close_kernel<Step><<<1, kT, 0, s>>>(k, step);
    return hipGetLastError();
}

template <typename V>
hipError_t launch_cg_product(hipStream_t s, const fused_matrix &A, const void *z, const void *p_old,
                             void *p, void *q, bool flexible, const scalar_link &k,
                             const mid_sums &out) {
    const V *Z = static_cast<const V *>(z), *P0 = static_cast<const V *>(p_old);
    V *P = static_cast<V *>(p), *Q = static_cast<V *>(q);
    return flexible ? launch_product(s, A, cg_view<V, true>{Z, P0, P, Q, {}}, k, out)
                    : launch_product(s, A, cg_view<V, false>{Z, P0, P, Q, {}}, k, out);
}

template <typename V>
hipError_t launch_pipe(hipStream_t s, const fused_matrix &A, const void *w_old, void *w,
                       const pipe_vectors &v, const scalar_link &k, const mid_sums &out) {
    const pipe_view<V> view{static_cast<const V *>(w_old), static_cast<V *>(w), static_cast<V *>(v.z),
                            static_cast<V *>(v.s),         static_cast<V *>(v.p), static_cast<V *>(v.x),
                            static_cast<V *>(v.r),         {}};
    return launch_product(s, A, view, k, out);
}

inline const double *cd(const void *p) { return static_cast<const double *>(p); }
inline double *md(void *p) { return static_cast<double *>(p); }

}  // namespace

// A lane walks its share of a row eight entries at a time, then four.  Short
// rows take the lanes that the mean row length asks for (csr_row_lanes); where
// some rows are longer, or the columns scattered, four lanes instead of one,
// while the lanes are one round of the chip.  us per iteration, many launches /
// one lane / four: BiCGSTAB, 30,000 scattered rows of 9 entries 44 / 44 / 30;
// CG, 50,000 rows of 5 with ten of 240 39 / 63 / 31, and above that size 200,000
// such rows 42 / 61 / 39, 800,000 63 / 80 / 78.
int mid_lanes(int64_t n, const mid_shape &m) {
    if (m.nnz > 96 * n) return 32;
    const int lanes = csr_row_lanes(n, m.nnz);
    return lanes == 1 && n <= 65536 && (m.longest > 16 || m.spread.lines > 0.3f) ? 4 : lanes;
}

// Where the gathers of two or three vectors per entry cost less than the
// launches and vector passes they save (us per iteration, many launches
// against these).  By rows and entries: CG 7-point 1.3M rows, 9.3M entries 62 /
// 50; 2.1M rows, 14.6M entries 84 / 69; 3.4M rows, 23M entries 123 / 122 (CSR
// 128 / 148, block-Jacobi 148 / 165); 27-point 0.26M rows, 7M entries (SELL-P)
// 40 / 31; 1M rows, 26M entries 98 / 106; BiCGSTAB 1M rows, 20M entries 274 /
// 303.  FP32 (mixed precision, block-Jacobi): 0.5M rows, 3.6M entries 31.5 /
// 26, 1.3M rows 49.6 / 48, 3.4M rows 95 / 117, so half of both.  ELL and
// SELL-P walk a row by one thread: BiCGSTAB on 50,000 banded rows of 20 entries
// 117 / 100, of 70 entries 184 / 179 (SELL-P 166 / 176), of 120 entries 212 /
// 239, while CSR with 8 or 32 lanes per row takes 155 / 122 and 181 / 152.
// Matrices with row patterns: the kernels for large systems leave out the
// column indices, these do not, so the line lies lower: 7-point 1M rows, 6.9M
// entries 45 / 39 (CSR 46 / 44); 2M rows, 13.6M entries 66 / 70 (CSR 68 / 79,
// block-Jacobi 77 / 107); 5-point 2M rows, 9.8M entries CG 60 / 60, BiCGSTAB 106
// / 112, CGS in CSR 105 / 113; FP32 with block-Jacobi 1M rows, 6.9M entries 35 /
// 33, in CSR 34 / 42.
// All of these gather lines that neighbouring rows share.  Otherwise the
// gathers are what the product waits for, and what they cost is the lines that
// wavefronts ask for and those that are not in the caches yet (column_spread);
// the weights and limits are fitted to CG, BiCGSTAB, CGS and pipelined CG on
// symmetric matrices of 10,000 to 1.6M rows of 5 to 61 entries, columns within
// 16, 200 or 5,000 of the diagonal or anywhere.  CG / BiCGSTAB, speed against
// many launches: 100,000 rows of 9 anywhere 1.07 / 1.00, 200,000 rows of 9 0.84 /
// 0.71 (within 200 1.16 / 1.07), 1M rows of 9 0.46 / 0.40, 400,000 rows of 31
// 0.45 / 0.32 (pipelined CG, which gathers one vector as the others do, 0.88).
// A CSR row that takes a lane more than one round of loads costs more: from 2M
// entries on 0.36M rows of 9 0.92 / 0.81, 0.4M of 3 to 17 within 16 1.04 / 0.87,
// with patterns also rows of 27 on four lanes 0.11M rows 0.95 / 0.83; and a few
// long rows hold up one lane: 800,000 rows of 5 with ten of 60 entries 1.03 /
// 0.98, of 100 0.96 / 0.90.  Long scattered rows walked by one thread in ELL and
// SELL-P: 30,000 rows of 15 BiCGSTAB 0.92, 10,000 of 31 CG 0.94, BiCGSTAB 0.84.
bool mid_fits(const fused_matrix &A, const mid_shape &m, int gathers) {
    const bool f64 = A.t == vt::f64, csr = A.format == fused_matrix::csr;
    const int64_t half = f64 ? 1 : 2;
    int64_t most = 14000000 / half;
    if (A.pat.id) most = f64 ? 8000000 : csr ? 4000000 : 7000000;
    if (A.n > kMidRows / half || m.nnz > most || (!csr && m.nnz > 48 * A.n)) return false;
    const double lines = m.spread.lines, fresh = m.spread.fresh;
    const double cost = (double)m.nnz * half * (0.25 * lines * lines + 0.6 * fresh);
    if (cost > (gathers == 0 ? 1.5e6 : gathers == 1 ? 0.7e6 : 0.42e6)) return false;
    if (csr && A.lanes == 1 && m.longest > (gathers == 0 ? 64 : 40)) return false;
    if (gathers == 0) return true;
    if (csr) return m.nnz * half <= 2000000 || m.longest <= 8 || (A.lanes > 1 && !A.pat.id);
    return lines <= 0.6 || fresh <= 0.05 || m.longest <= (gathers == 1 ? 40 : 24);
}

hipError_t mid_cg_product(hipStream_t s, const fused_matrix &A, const void *z, const void *p_old,
                          void *p, void *q, bool flexible, const scalar_link &k,
                          const mid_sums &out) {
    return A.t == vt::f64 ? launch_cg_product<double>(s, A, z, p_old, p, q, flexible, k, out)
                          : launch_cg_product<float>(s, A, z, p_old, p, q, flexible, k, out);
}

hipError_t mid_cg_update(hipStream_t s, vt t, int64_t n, void *x, void *r, void *z, const void *p,
                         const void *q, const void *inv, int bs, bool flexible,
                         const scalar_link &k, const mid_sums &out) {
    if (flexible)
        return t == vt::f64 ? launch_cg_update<double, true>(s, n, x, r, z, p, q, inv, bs, k, out)
                            : launch_cg_update<float, true>(s, n, x, r, z, p, q, inv, bs, k, out);
    return t == vt::f64 ? launch_cg_update<double, false>(s, n, x, r, z, p, q, inv, bs, k, out)
                        : launch_cg_update<float, false>(s, n, x, r, z, p, q, inv, bs, k, out);
}

hipError_t mid_cg_close(hipStream_t s, bool flexible, const scalar_link &k) {
    return flexible ? launch_close(s, k, cg_beta_step<true>{})
                    : launch_close(s, k, cg_beta_step<false>{});
}

hipError_t mid_pipe(hipStream_t s, const fused_matrix &A, const void *w_old, void *w,
                    const pipe_vectors &v, const scalar_link &k, const mid_sums &out) {
    return A.t == vt::f64 ? launch_pipe<double>(s, A, w_old, w, v, k, out)
                          : launch_pipe<float>(s, A, w_old, w, v, k, out);
}

hipError_t mid_pipe_close(hipStream_t s, const scalar_link &k) {
    return launch_close(s, k, pipe_update_step{});
}

hipError_t mid_bicg_v(hipStream_t s, const fused_matrix &A, const void *r, const void *p_old,
                      const void *v_old, const void *rh, void *p, void *v, const scalar_link &k,
                      const mid_sums &out) {
    if (A.t != vt::f64) return hipErrorInvalidValue;
    return launch_product(s, A, bicg_v_view{cd(r), cd(p_old), cd(v_old), cd(rh), md(p), md(v), {}}, k,
                          out, kMidBlocks);
}

hipError_t mid_bicg_t(hipStream_t s, const fused_matrix &A, const void *r, const void *v, void *t,
                      const scalar_link &k, const mid_sums &out) {
    if (A.t != vt::f64) return hipErrorInvalidValue;
    return launch_product(s, A, bicg_t_view{cd(r), cd(v), md(t), {}}, k, out, kMidBlocks);
}

hipError_t mid_bicg_update(hipStream_t s, int64_t n, void *x, void *r, const void *rh, const void *p,
                           const void *v, const void *t, const scalar_link &k, const mid_sums &out) {
    const auto launch = [&](auto threads) {
        constexpr int T = decltype(threads)::value;
        const int g = mid_blocks(n, T, kMidBlocks), parts = mid_parts(n, g, T);
        *out.parts = parts;
        mid_bicg_update_kernel<T><<<g, T, 0, s>>>(n, md(x), md(r), cd(rh), cd(p), cd(v), cd(t), k,
                                                  parts, out.partials);
        return hipGetLastError();
    };
    return half_blocks(n) ? launch(std::integral_constant<int, kHalfT>{})
                          : launch(std::integral_constant<int, kT>{});
}

hipError_t mid_bicg_close(hipStream_t s, const scalar_link &k) {
    return launch_close(s, k, bicg_update_step{});
}

hipError_t mid_cgs_t(hipStream_t s, const fused_matrix &A, const void *r, const void *q,
                     const void *p_old, const void *rh, void *u, void *p, void *t,
                     const scalar_link &k, const mid_sums &out) {
    if (A.t != vt::f64) return hipErrorInvalidValue;
    return launch_product(s, A, cgs_t_view{cd(r), cd(q), cd(p_old), cd(rh), md(u), md(p), md(t), {}}, k,
                          out, kMidBlocks);
}

hipError_t mid_cgs_w(hipStream_t s, const fused_matrix &A, const void *u, const void *t,
                     const void *rh, void *q, void *x, void *r, const scalar_link &k,
                     const mid_sums &out) {
    if (A.t != vt::f64) return hipErrorInvalidValue;
    return launch_product(s, A, cgs_w_view{cd(u), cd(t), cd(rh), md(q), md(x), md(r), {}}, k, out,
                          kMidBlocks);
}

hipError_t mid_cgs_close(hipStream_t s, const scalar_link &k) {
    return launch_close(s, k, cgs_update_step{});
}

}  // namespace gko
