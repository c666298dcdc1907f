// Restarted GMRES(m), FP64, unpreconditioned (Saad and Schultz 1986; Saad,
// Iterative Methods, Alg. 6.9 with the Givens least-squares update of
// Sec. 6.5.3).
//
// Arnoldi step j with w = A v_j written straight into basis slot j+1:
//   dot         h = V_j^T w and w.w in one pass over the j+1 basis vectors
//   update+dot  w -= V_j h, then h' = V_j^T w and the new w.w, in one pass
//               (each thread re-reads its rows of V_j right after the
//               update, mostly from the caches)
//   update      w -= V_j h' (classical Gram-Schmidt twice) only when the
//               first round shrank w below 1/sqrt(2) of its length (Daniel,
//               Gragg, Kaufman and Stewart's criterion); otherwise the
//               launch returns at once
//   step        (one wavefront; the rotations in series on one lane) the
//               column of H, the earlier rotations, the new Givens rotation,
//               |g_{j+1}| as the residual estimate, the end of the cycle
//   normalise   v_{j+1} = w / h_{j+1,j}
// The basis is column-major with a leading dimension rounded up to 64
// doubles.  The multi-vector passes keep each thread's rows of w in
// registers and read the basis vectors coalesced, one after another; the
// per-vector sums are wave DPP reductions accumulated per wave in LDS, then
// per-block partials summed in block order by a one-block-per-value kernel,
// so every result repeats bitwise.  A cycle ends with the back substitution
// (one workgroup, by column panels) and x += V_k y in one pass.  Up to
// kCompactMaxRows rows the compact passes below take their place.
#include <cmath>

#include "device.hpp"
#include "kernels.hpp"
#include "solver_kernels.hpp"
#include "solver_state.hpp"

namespace gko {

namespace {

constexpr int kG = 256;          // threads per workgroup
constexpr int kGRows = 4;        // rows per thread per chunk
constexpr int kGWaves = kG / kWave;

inline int gmres_blocks(int64_t n) {
    int64_t g = (n + (int64_t)kG * kGRows - 1) / ((int64_t)kG * kGRows);
    if (g > kGmresMaxBlocks) g = kGmresMaxBlocks;
    return g < 1 ? 1 : (int)g;
}

// Phase gates.  mode 0: the passes of an Arnoldi step run only while the
// cycle is open; mode 1: the second Gram-Schmidt round also needs the step
// to have asked for it; mode 2 (cycle start): while the solve runs.
__device__ inline bool gate(const gmres_state *st, int mode) {
    if (mode == 2) return st->done == kRunning;
    return st->cycle_done == 0 && (mode == 0 || st->reorth != 0);
}

// partials[v * gridDim.x + block] <- block sums of V_i . w (v = i < k) and of
// w . w (v = k)
__global__ __launch_bounds__(kG) void gmres_dot_kernel(int64_t n, int k, const double *__restrict__ V,
                                                       int64_t ldv, const double *__restrict__ w,
                                                       const gmres_state *st, int mode,
                                                       double *__restrict__ partials) {
    __shared__ double part[kGmresMaxKrylov + 1][kGWaves];
    if (!gate(st, mode)) return;
    const int lane = threadIdx.x % kWave, wv = threadIdx.x / kWave;
    for (int e = threadIdx.x; e < (k + 1) * kGWaves; e += kG) part[e / kGWaves][e % kGWaves] = 0.0;
    __syncthreads();
    for (int64_t base = (int64_t)blockIdx.x * kG * kGRows; base < n;
         base += (int64_t)gridDim.x * kG * kGRows) {
        double wr[kGRows];
        double ww = 0.0;
#pragma unroll
        for (int r = 0; r < kGRows; ++r) {
            const int64_t l = base + r * kG + threadIdx.x;
            wr[r] = l < n ? w[l] : 0.0;
            ww += wr[r] * wr[r];
        }
        for (int i = 0; i < k; ++i) {
            const double *vi = V + (int64_t)i * ldv;
            double s = 0.0;
#pragma unroll
            for (int r = 0; r < kGRows; ++r) {
                const int64_t l = base + r * kG + threadIdx.x;
                s += (l < n ? vi[l] : 0.0) * wr[r];
            }
            s = wave_total(s);
            if (lane == 0) part[i][wv] += s;
        }
        ww = wave_total(ww);
        if (lane == 0) part[k][wv] += ww;
    }
    __syncthreads();
    for (int v = threadIdx.x; v <= k; v += kG) {
        double s = 0.0;
        for (int q = 0; q < kGWaves; ++q) s += part[v][q];
        partials[(int64_t)v * gridDim.x + blockIdx.x] = s;
    }
}

// w -= sum_i h_i V_i (i ascending), block sums of the new w . w
__global__ __launch_bounds__(kG) void gmres_update_kernel(int64_t n, int k,
                                                          const double *__restrict__ V,
                                                          int64_t ldv, const double *__restrict__ h,
                                                          double *__restrict__ w,
                                                          const gmres_state *st, int mode,
                                                          double *__restrict__ partials) {
    __shared__ double hs[kGmresMaxKrylov];
    __shared__ double red[kGWaves];
    if (!gate(st, mode)) return;
    for (int i = threadIdx.x; i < k; i += kG) hs[i] = h[i];
    __syncthreads();
    double ww = 0.0;
    for (int64_t base = (int64_t)blockIdx.x * kG * kGRows; base < n;
         base += (int64_t)gridDim.x * kG * kGRows) {
        double acc[kGRows];
#pragma unroll
        for (int r = 0; r < kGRows; ++r) {
            const int64_t l = base + r * kG + threadIdx.x;
            acc[r] = l < n ? w[l] : 0.0;
        }
        for (int i = 0; i < k; ++i) {
            const double *vi = V + (int64_t)i * ldv;
            const double hi = hs[i];
#pragma unroll
            for (int r = 0; r < kGRows; ++r) {
                const int64_t l = base + r * kG + threadIdx.x;
                if (l < n) acc[r] = acc[r] - hi * vi[l];
            }
        }
#pragma unroll
        for (int r = 0; r < kGRows; ++r) {
            const int64_t l = base + r * kG + threadIdx.x;
            if (l < n) {
                w[l] = acc[r];
                ww += acc[r] * acc[r];
            }
        }
    }
    ww = block_sum<kG>(ww, red);
    if (threadIdx.x == 0) partials[blockIdx.x] = ww;
}

// The first round's update fused with the second round's dots:
// w -= sum_i h_i V_i, then partials of V_i . w (i < k) and w . w (at k) for
// the new w.  The second read of each V_i[l] follows the first within the
// same thread's chunk, so it mostly hits the caches instead of HBM.
__global__ __launch_bounds__(kG) void gmres_update_dot_kernel(int64_t n, int k,
                                                              const double *__restrict__ V,
                                                              int64_t ldv,
                                                              const double *__restrict__ h,
                                                              double *__restrict__ w,
                                                              const gmres_state *st,
                                                              double *__restrict__ partials) {
    __shared__ double part[kGmresMaxKrylov + 1][kGWaves];
    __shared__ double hs[kGmresMaxKrylov];
    if (!gate(st, 0)) return;
    const int lane = threadIdx.x % kWave, wv = threadIdx.x / kWave;
    for (int e = threadIdx.x; e < (k + 1) * kGWaves; e += kG) part[e / kGWaves][e % kGWaves] = 0.0;
    for (int i = threadIdx.x; i < k; i += kG) hs[i] = h[i];
    __syncthreads();
    for (int64_t base = (int64_t)blockIdx.x * kG * kGRows; base < n;
         base += (int64_t)gridDim.x * kG * kGRows) {
        double acc[kGRows];
#pragma unroll
        for (int r = 0; r < kGRows; ++r) {
            const int64_t l = base + r * kG + threadIdx.x;
            acc[r] = l < n ? w[l] : 0.0;
        }
        for (int i = 0; i < k; ++i) {
            const double *vi = V + (int64_t)i * ldv;
            const double hi = hs[i];
#pragma unroll
            for (int r = 0; r < kGRows; ++r) {
                const int64_t l = base + r * kG + threadIdx.x;
                if (l < n) acc[r] = acc[r] - hi * vi[l];
            }
        }
        double ww = 0.0;
#pragma unroll
        for (int r = 0; r < kGRows; ++r) {
            const int64_t l = base + r * kG + threadIdx.x;
            if (l < n) w[l] = acc[r];
            ww += acc[r] * acc[r];
        }
        // newest vectors first: they were read last, so the most of them are
        // still in the caches (each V_i . w is formed on its own, so the
        // order changes no result)
        for (int i = k - 1; i >= 0; --i) {
            const double *vi = V + (int64_t)i * ldv;
            double sd = 0.0;
#pragma unroll
            for (int r = 0; r < kGRows; ++r) {
                const int64_t l = base + r * kG + threadIdx.x;
                sd += (l < n ? vi[l] : 0.0) * acc[r];
            }
            sd = wave_total(sd);
            if (lane == 0) part[i][wv] += sd;
        }
        ww = wave_total(ww);
        if (lane == 0) part[k][wv] += ww;
    }
    __syncthreads();
    for (int v = threadIdx.x; v <= k; v += kG) {
        double sum = 0.0;
        for (int q = 0; q < kGWaves; ++q) sum += part[v][q];
        partials[(int64_t)v * gridDim.x + blockIdx.x] = sum;
    }
}

// The same for k <= kGRegVecs with one row per thread per chunk: the
// thread's element of every V_i stays in registers between the update and
// the dots, so V is read once (the loops are unrolled to kGRegVecs so the
// register array is indexed statically).
constexpr int kGRegVecs = 32;

__global__ __launch_bounds__(kG) void gmres_update_dot_regs_kernel(int64_t n, int k,
                                                                   const double *__restrict__ V,
                                                                   int64_t ldv,
                                                                   const double *__restrict__ h,
                                                                   double *__restrict__ w,
                                                                   const gmres_state *st,
                                                                   double *__restrict__ partials) {
    __shared__ double part[kGRegVecs + 1][kGWaves];
    __shared__ double hs[kGRegVecs];
    if (!gate(st, 0)) return;
    const int lane = threadIdx.x % kWave, wv = threadIdx.x / kWave;
    for (int e = threadIdx.x; e < (k + 1) * kGWaves; e += kG) part[e / kGWaves][e % kGWaves] = 0.0;
    for (int i = threadIdx.x; i < k; i += kG) hs[i] = h[i];
    __syncthreads();
    for (int64_t base = (int64_t)blockIdx.x * kG; base < n; base += (int64_t)gridDim.x * kG) {
        const int64_t l = base + threadIdx.x;
        const bool ok = l < n;
        double vr[kGRegVecs];
        double acc = ok ? w[l] : 0.0;
#pragma unroll
        for (int i = 0; i < kGRegVecs; ++i) {
            vr[i] = (i < k && ok) ? V[(int64_t)i * ldv + l] : 0.0;
            acc = acc - (i < k ? hs[i] : 0.0) * vr[i];
        }
        if (ok) w[l] = acc;
#pragma unroll
        for (int i = 0; i < kGRegVecs; ++i) {
            if (i < k) {  // uniform
                const double sd = wave_total(vr[i] * acc);
                if (lane == 0) part[i][wv] += sd;
            }
        }
        const double ww = wave_total(acc * acc);
        if (lane == 0) part[k][wv] += ww;
    }
    __syncthreads();
    for (int v = threadIdx.x; v <= k; v += kG) {
        double sum = 0.0;
        for (int q = 0; q < kGWaves; ++q) sum += part[v][q];
        partials[(int64_t)v * gridDim.x + blockIdx.x] = sum;
    }
}

// out[v] <- sum over blocks of partials[v * g + b], block order, one
// workgroup per value
__global__ __launch_bounds__(kG) void gmres_sum_kernel(int g, const double *__restrict__ partials,
                                                       double *__restrict__ out,
                                                       const gmres_state *st, int mode) {
    __shared__ double red[kGWaves];
    if (!gate(st, mode)) return;
    const double *p = partials + (int64_t)blockIdx.x * g;
    double s = 0.0;
    for (int b = threadIdx.x; b < g; b += kG) s += p[b];
    s = block_sum<kG>(s, red);
    if (threadIdx.x == 0) out[blockIdx.x] = s;
}

// After the first round: decide on a second round.  dot1: V^T w and w.w
// before the round; dot2: V^T w and w.w after it.
__global__ void gmres_check_kernel(int j, const double *__restrict__ dot1,
                                   const double *__restrict__ dot2, gmres_state *st) {
    if (st->cycle_done) return;
    // |w_after| < |w_before| / sqrt(2)
    st->reorth = (2.0 * dot2[j + 1] < dot1[j + 1]) ? 1 : 0;
    st->reorths += st->reorth;
    st->ww = dot2[j + 1];
}

// Close step j (every thread of the workgroup; T threads): the column of H
// from the rounds' sums (dot1, and dot2 after a second round), the earlier
// rotations, the new one, the residual estimate, the end of the cycle.  ww is
// the w.w left by the rounds.  The chain of rotations is serial, so one thread
// walks it, but out of LDS: column, cosines and sines are loaded together
// first, and the column is stored by all threads (from global memory the same
// chain took 13 us at j = 30).
struct step_lds {
    double h[kGmresMaxKrylov + 1], cs[kGmresMaxKrylov], sn[kGmresMaxKrylov];
    double beta;  // g_j
    int ok;
};

template <int T>
__device__ inline void close_step(int j, int m, double ww, bool reorth, const double *dot1,
                                  const double *dot2, gmres_state &st, const gmres_work &wk,
                                  step_lds &L) {
    for (int i = threadIdx.x; i <= j; i += T) {
        L.h[i] = reorth ? dot1[i] + dot2[i] : dot1[i];
        if (i < j) {
            L.cs[i] = wk.cs[i];
            L.sn[i] = wk.sn[i];
        }
    }
    if (threadIdx.x == 0) L.beta = wk.g[j];
    __syncthreads();
    if (threadIdx.x == 0) {
        const double hn = sqrt(ww);
        double a = L.h[0];
        for (int i = 0; i < j; ++i) {
            const double c = L.h[i + 1];
            L.h[i] = L.cs[i] * a + L.sn[i] * c;
            a = -L.sn[i] * a + L.cs[i] * c;
        }
        const double d = sqrt(a * a + hn * hn);
        st.iter += 1;
        st.k = j + 1;
        L.ok = d > 0.0;
        if (!(d > 0.0)) {
            st.done = kBreakdown;
            st.cycle_done = 1;
        } else {
            const double c = a / d, sn = hn / d;
            wk.cs[j] = c;
            wk.sn[j] = sn;
            L.h[j] = d;
            const double next = -sn * L.beta;
            wk.g[j + 1] = next;
            wk.g[j] = c * L.beta;
            const double est = fabs(next);
            st.est = est;
            st.hn = hn;
            if (std::isnan(est)) {
                st.done = kBreakdown;
                st.cycle_done = 1;
            } else if (est <= st.stop || hn == 0.0 || st.iter >= st.maxit || j + 1 == m) {
                st.cycle_done = 1;
            }
        }
    }
    __syncthreads();
    if (L.ok)
        for (int i = threadIdx.x; i <= j; i += T) wk.H[(int64_t)i * m + j] = L.h[i];
}

__global__ __launch_bounds__(kWave) void gmres_step_kernel(int j, int m, gmres_state *st,
                                                           gmres_work wk) {
    __shared__ step_lds L;
    if (st->cycle_done) return;
    gmres_state s = *st;
    __syncthreads();  // every thread has read the state that thread 0 stores
    const bool reorth = s.reorth != 0;
    close_step<kWave>(j, m, reorth ? wk.upd2[0] : s.ww, reorth, wk.dot1, wk.dot2, s, wk, L);
    if (threadIdx.x == 0) *st = s;
}

__global__ __launch_bounds__(kG) void gmres_scale_kernel(int64_t n, double *__restrict__ v,
                                                         const gmres_state *st) {
    if (st->cycle_done) return;
    const double hn = st->hn;
    for (int64_t l = (int64_t)blockIdx.x * kG + threadIdx.x; l < n; l += (int64_t)gridDim.x * kG)
        v[l] = v[l] / hn;
}

// Back substitution R y = g over the cycle's k columns, one workgroup.  A
// panel of up to 64 columns is staged in LDS (its diagonal block, loaded
// together), solved column by column by one wavefront (lane l holds row l's
// right-hand side), then subtracted from the rows above it, a thread per row.
// By one thread from global memory, k = 30 took 34 us.
constexpr int kSolvePanel = kWave;

__global__ __launch_bounds__(2 * kWave) void gmres_solve_kernel(int m, const double *__restrict__ H,
                                                                const double *__restrict__ gv,
                                                                double *__restrict__ y,
                                                                const gmres_state *st) {
    __shared__ double R[kSolvePanel][kSolvePanel + 1];
    __shared__ double s[kGmresMaxKrylov];
    if (st->done == kBreakdown) return;
    const int k = st->k, t = threadIdx.x;
    if (t < k) s[t] = gv[t];
    for (int c0 = (k - 1) / kSolvePanel * kSolvePanel; c0 >= 0; c0 -= kSolvePanel) {
        const int c = k - c0 < kSolvePanel ? k - c0 : kSolvePanel;
        for (int e = t; e < c * c; e += 2 * kWave)
            R[e / c][e % c] = H[(int64_t)(c0 + e / c) * m + c0 + e % c];
        __syncthreads();
        if (t < kWave) {
            double v = t < c ? s[c0 + t] : 0.0;
            for (int i = c - 1; i >= 0; --i) {
                const double yi = lane_value(v, i) / R[i][i];
                if (t == i) v = yi;
                else if (t < i) v = v - R[t][i] * yi;
            }
            if (t < c) {
                s[c0 + t] = v;
                y[c0 + t] = v;
            }
        }
        __syncthreads();
        if (t < c0) {
            double v = s[t];
            for (int i = c - 1; i >= 0; --i) v = v - H[(int64_t)t * m + c0 + i] * s[c0 + i];
            s[t] = v;
        }
        __syncthreads();
    }
}

// x += sum_i y_i V_i (i ascending)
__global__ __launch_bounds__(kG) void gmres_xupdate_kernel(int64_t n, const double *__restrict__ V,
                                                           int64_t ldv,
                                                           const double *__restrict__ y,
                                                           double *__restrict__ x,
                                                           const gmres_state *st) {
    __shared__ double ys[kGmresMaxKrylov];
    if (st->done == kBreakdown) return;
    const int k = st->k;
    for (int i = threadIdx.x; i < k; i += kG) ys[i] = y[i];
    __syncthreads();
    for (int64_t l = (int64_t)blockIdx.x * kG + threadIdx.x; l < n; l += (int64_t)gridDim.x * kG) {
        double xl = x[l];
        for (int i = 0; i < k; ++i) xl = xl + ys[i] * V[(int64_t)i * ldv + l];
        x[l] = xl;
    }
}

// Cycle start from v0 = b - A x (unnormalised) and its squared norm rr; the
// scale v0 = r / beta follows.
__device__ inline void open_cycle(double rr, gmres_state &st, double *__restrict__ gv, bool writes) {
    const double beta = sqrt(rr);
    st.beta = beta;
    st.cycle_done = 0;
    st.reorth = 0;
    st.k = 0;
    st.hn = beta;
    if (writes) gv[0] = beta;
    if (std::isnan(beta) || std::isinf(beta)) {
        st.done = kBreakdown;
        st.cycle_done = 1;
    } else if (beta <= st.stop) {
        st.done = kConverged;
        st.cycle_done = 1;
    } else if (st.iter >= st.maxit) {
        st.done = kMaxIter;
        st.cycle_done = 1;
    } else {
        st.cycles += 1;
    }
}

__global__ void gmres_cycle_kernel(const double *__restrict__ rr, gmres_state *st,
                                   double *__restrict__ gv) {
    if (st->done != kRunning) return;
    gmres_state s = *st;
    open_cycle(rr[0], s, gv, true);
    *st = s;
}

// ------------------------------------------------------------ compact passes
// Systems of up to kCompactMaxRows rows are bound by launches and by the chain
// of dependent kernels of a step, not by memory: the basis sits in the caches.
// A step is four launches after the product instead of nine: the sums over
// blocks are formed by the kernel that uses them (every workgroup sums the
// few partials itself, in block order, so all get the same bits) instead of a
// launch of their own, the decision on the second round moves into its update,
// and the step's scalar work into the scaling pass.  One row per thread; the
// workgroup grows with n (256 to 1024 threads) so that the grid stays within
// kCompactMaxBlocks and the partials of a value are two loads per lane.
//   dots      P1 = partials of V_i . w, w . w; a workgroup takes 8 values
//   update    h = sums of P1; w -= V h; P2 = partials of V_i . w, w . w
//   update2   h' = sums of P2; if the first round lost more than 1/sqrt(2):
//             w -= V h', P1 = partials of w . w
//   close     hn from P1 (or P2), v_{j+1} = w / hn; workgroup 0 closes the
//             step and writes the state that the next step reads (the kernel's
//             other workgroups still read this step's)
// GMRES(30) per step, nine passes against these: 22,500 rows 68 -> 30 us,
// 90,000 rows 75 -> 39, 250,000 rows 87 -> 48, 524,176 rows 103 -> 81 us (the
// four kernels themselves take 4, 9, 6 and 4 us at 22,500 rows).  Above
// kCompactMaxRows the partials outgrow eight loads per lane and value.
constexpr int64_t kCompactMaxRows = 524288;
constexpr int kCompactMaxBlocks = 512;
constexpr int kCompactDots = 8;   // values per workgroup of the dots pass

inline int compact_threads(int64_t n) { return n <= 32768 ? 256 : n <= 65536 ? 512 : 1024; }

// out[v] (LDS) = sum over the g blocks of P[v * g + b] for v < nv, by
// wavefronts, up to 32 loads in flight per lane; ends with a barrier.
template <int T, int U, int Q>
__device__ inline void sum_values_q(int nv, int g, const double *__restrict__ P, double *out) {
    constexpr int NW = T / kWave;
    const int lane = threadIdx.x % kWave, wv = threadIdx.x / kWave;
    for (int v0 = wv; v0 < nv; v0 += NW * U) {
        double t[U][Q];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const int v = v0 + u * NW, b = lane + q * kWave;
                t[u][q] = v < nv && b < g ? P[(int64_t)v * g + b] : 0.0;
            }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            double s = t[u][0];
#pragma unroll
            for (int q = 1; q < Q; ++q) s += t[u][q];
            s = wave_total(s);
            if (lane == 0 && v0 + u * NW < nv) out[v0 + u * NW] = s;
        }
    }
    __syncthreads();
}

template <int T>
__device__ inline void sum_values(int nv, int g, const double *__restrict__ P, double *out) {
    static_assert(kCompactMaxBlocks == 8 * kWave, "at most eight partials per lane");
    if constexpr (T < 1024) {  // at most 128 workgroups
        sum_values_q<T, 8, 2>(nv, g, P, out);
    } else {
        if (g <= 2 * kWave) sum_values_q<T, 2, 2>(nv, g, P, out);
        else sum_values_q<T, 2, 8>(nv, g, P, out);
    }
}

// P[(v0 + u) * g + block] = block sums of val[u] over the T threads, u < nv.
template <int T, int U>
__device__ inline void store_sums(const double (&val)[U], int nv, int v0, double (*red)[T / kWave],
                                  double *__restrict__ P) {
    constexpr int NW = T / kWave;
    const int lane = threadIdx.x % kWave, wv = threadIdx.x / kWave;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (u < nv) {  // uniform
            const double s = wave_total(val[u]);
            if (lane == 0) red[u][wv] = s;
        }
    }
    __syncthreads();
    if (threadIdx.x < U && (int)threadIdx.x < nv) {
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < NW; ++q) s += red[threadIdx.x][q];
        P[(int64_t)(v0 + threadIdx.x) * gridDim.x + blockIdx.x] = s;
    }
    __syncthreads();
}

template <int T>
__global__ __launch_bounds__(T) void compact_dots_kernel(int64_t n, int k, const double *__restrict__ V,
                                                         int64_t ldv, const double *__restrict__ w,
                                                         const gmres_state *st, int mode,
                                                         double *__restrict__ P) {
    __shared__ double red[kCompactDots][T / kWave];
    if (!gate(st, mode)) return;
    const int64_t l = (int64_t)blockIdx.x * T + threadIdx.x;
    const int v0 = blockIdx.y * kCompactDots;
    const int nv = k + 1 - v0 < kCompactDots ? k + 1 - v0 : kCompactDots;
    const double wl = l < n ? w[l] : 0.0;
    double s[kCompactDots];
#pragma unroll
    for (int u = 0; u < kCompactDots; ++u)
        s[u] = (v0 + u < k && l < n ? V[(int64_t)(v0 + u) * ldv + l] : wl) * wl;
    store_sums<T>(s, nv, v0, red, P);
}

// w - sum_{i < k} h_i V_i at row l (i ascending), eight loads in flight
__device__ inline double compact_subtract(int k, const double *__restrict__ V, int64_t ldv,
                                          const double *h, int64_t l, double w) {
    for (int i0 = 0; i0 < k; i0 += 8) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = i0 + u < k ? V[(int64_t)(i0 + u) * ldv + l] : 0.0;
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (i0 + u < k) w = w - h[i0 + u] * v[u];
    }
    return w;
}

template <int T>
__global__ __launch_bounds__(T) void compact_update_kernel(int64_t n, int k,
                                                           const double *__restrict__ V, int64_t ldv,
                                                           double *__restrict__ w,
                                                           const gmres_state *st,
                                                           const double *__restrict__ P1,
                                                           double *__restrict__ P2,
                                                           double *__restrict__ dot1) {
    __shared__ double h[kGmresMaxKrylov + 1];
    __shared__ double red[kGRegVecs][T / kWave];
    if (!gate(st, 0)) return;
    const int64_t l = (int64_t)blockIdx.x * T + threadIdx.x;
    const bool ok = l < n;
    double acc = ok ? w[l] : 0.0;
    if (k < kGRegVecs) {
        // the thread's element of every V_i in registers, loaded before the
        // sums of h are waited for
        double vr[kGRegVecs];
#pragma unroll
        for (int i = 0; i < kGRegVecs; ++i) vr[i] = i < k && ok ? V[(int64_t)i * ldv + l] : 0.0;
        sum_values<T>(k + 1, gridDim.x, P1, h);
#pragma unroll
        for (int i = 0; i < kGRegVecs; ++i)
            if (i < k) acc = acc - h[i] * vr[i];
#pragma unroll
        for (int i = 0; i < kGRegVecs; ++i) vr[i] = (i < k ? vr[i] : acc) * acc;
        store_sums<T>(vr, k + 1, 0, red, P2);
    } else {
        sum_values<T>(k + 1, gridDim.x, P1, h);
        if (ok) acc = compact_subtract(k, V, ldv, h, l, acc);
        for (int v0 = 0; v0 <= k; v0 += kCompactDots) {
            const int nv = k + 1 - v0 < kCompactDots ? k + 1 - v0 : kCompactDots;
            double s[kCompactDots];
#pragma unroll
            for (int u = 0; u < kCompactDots; ++u)
                s[u] = (v0 + u < k && ok ? V[(int64_t)(v0 + u) * ldv + l] : acc) * acc;
            store_sums<T>(s, nv, v0, red, P2);
        }
    }
    if (ok) w[l] = acc;
    if (blockIdx.x == 0)
        for (int i = threadIdx.x; i <= k; i += T) dot1[i] = h[i];
}

template <int T>
__global__ __launch_bounds__(T) void compact_update2_kernel(
    int64_t n, int k, const double *__restrict__ V, int64_t ldv, double *__restrict__ w,
    gmres_state *st, const double *__restrict__ P2, double *__restrict__ P1,
    const double *__restrict__ dot1, double *__restrict__ dot2) {
    __shared__ double h[kGmresMaxKrylov + 1];
    __shared__ double red[1][T / kWave];
    if (!gate(st, 0)) return;
    const double before = dot1[k];
    sum_values<T>(k + 1, gridDim.x, P2, h);
    const bool reorth = 2.0 * h[k] < before;  // |w_after| < |w_before| / sqrt(2)
    if (blockIdx.x == 0) {
        for (int i = threadIdx.x; i < k; i += T) dot2[i] = h[i];
        if (threadIdx.x == 0) {  // no workgroup of this kernel reads these fields
            st->reorth = reorth ? 1 : 0;
            st->reorths += reorth ? 1 : 0;
            st->ww = h[k];
        }
    }
    if (!reorth) return;
    const int64_t l = (int64_t)blockIdx.x * T + threadIdx.x;
    double s[1] = {0.0};
    if (l < n) {
        const double acc = compact_subtract(k, V, ldv, h, l, w[l]);
        w[l] = acc;
        s[0] = acc * acc;
    }
    store_sums<T>(s, 1, 0, red, P1);
}

template <int T>
__global__ __launch_bounds__(T) void compact_close_kernel(int64_t n, int j, int m,
                                                          double *__restrict__ w,
                                                          const gmres_state *st, gmres_state *next,
                                                          gmres_work wk) {
    __shared__ double ww;
    __shared__ step_lds L;
    gmres_state s = *st;
    if (s.cycle_done) {
        if (blockIdx.x == 0 && threadIdx.x == 0) *next = s;
        return;
    }
    const bool reorth = s.reorth != 0;
    const int64_t l = (int64_t)blockIdx.x * T + threadIdx.x;
    const double wl = l < n ? w[l] : 0.0;
    if (reorth) sum_values<T>(1, gridDim.x, wk.partials, &ww);
    const double w2 = reorth ? ww : s.ww;
    if (l < n) w[l] = wl / sqrt(w2);
    if (blockIdx.x == 0) {
        close_step<T>(j, m, w2, reorth, wk.dot1, wk.dot2, s, wk, L);
        if (threadIdx.x == 0) *next = s;
    }
}

// Cycle start from v0 = b - A x (unnormalised), P1 = partials of v0 . v0.
template <int T>
__global__ __launch_bounds__(T) void compact_start_kernel(int64_t n, double *__restrict__ v,
                                                          const gmres_state *st, gmres_state *next,
                                                          gmres_work wk) {
    __shared__ double rr;
    gmres_state s = *st;
    if (s.done != kRunning) {
        if (blockIdx.x == 0 && threadIdx.x == 0) *next = s;
        return;
    }
    const int64_t l = (int64_t)blockIdx.x * T + threadIdx.x;
    const double vl = l < n ? v[l] : 0.0;
    sum_values<T>(1, gridDim.x, wk.partials, &rr);
    open_cycle(rr, s, wk.g, blockIdx.x == 0 && threadIdx.x == 0);
    if (l < n && s.cycle_done == 0) v[l] = vl / s.beta;
    if (blockIdx.x == 0 && threadIdx.x == 0) *next = s;
}

template <int T>
hipError_t compact_step(hipStream_t s, int64_t n, int m, int j, double *V, int64_t ldv,
                        gmres_state *st, gmres_state *next, const gmres_work &wk) {
    const unsigned g = (unsigned)((n + T - 1) / T);
    const int k = j + 1;
    double *w = V + (int64_t)k * ldv;
    compact_dots_kernel<T><<<dim3(g, k / kCompactDots + 1), T, 0, s>>>(n, k, V, ldv, w, st, 0,
                                                                       wk.partials);
    compact_update_kernel<T><<<g, T, 0, s>>>(n, k, V, ldv, w, st, wk.partials, wk.partials2, wk.dot1);
    compact_update2_kernel<T><<<g, T, 0, s>>>(n, k, V, ldv, w, st, wk.partials2, wk.partials, wk.dot1,
                                              wk.dot2);
    compact_close_kernel<T><<<g, T, 0, s>>>(n, j, m, w, st, next, wk);
    return hipGetLastError();
}

template <int T>
hipError_t compact_start(hipStream_t s, int64_t n, double *V, gmres_state *st, gmres_state *next,
                         const gmres_work &wk) {
    const unsigned g = (unsigned)((n + T - 1) / T);
    compact_dots_kernel<T><<<g, T, 0, s>>>(n, 0, V, 0, V, st, 2, wk.partials);
    compact_start_kernel<T><<<g, T, 0, s>>>(n, V, st, next, wk);
    return hipGetLastError();
}

// ------------------------------------------------------------ one workgroup
// The whole restarted GMRES(m) of a small CSR system in one launch of one
// 1024-thread workgroup: the same steps, criteria and state as the kernels
// above, without a launch or host poll per step.  Thread t owns rows t,
// t + 1024, ...; w of those rows stays in registers through a step; the
// basis lives in global memory (L2-resident at these sizes); the rotated
// Hessenberg R, g and the rotations in LDS.  Per-vector sums are wave DPP
// sums, then the waves' totals are added in wave order; the small scalar
// work (the column's rotations, the back substitution) runs on thread 0.
constexpr int kSGT = 1024;
constexpr int kSGRows = 4;
constexpr int kSGWaves = kSGT / kWave;

struct small_gmres_lds {
    double red[kSGWaves][kGmresSmallKrylov + 2];
    double R[kGmresSmallKrylov][kGmresSmallKrylov];  // R[i][j], i <= j
    double g[kGmresSmallKrylov + 1], cs[kGmresSmallKrylov], sn[kGmresSmallKrylov];
    double h[kGmresSmallKrylov + 2], h2[kGmresSmallKrylov + 2], y[kGmresSmallKrylov];
    double hcol[kGmresSmallKrylov + 1];
    double hn, est, ww;
    int cycle_done, breakdown;
};

// Vectors taken together by the passes over the basis, so that their loads
// are in flight at once.
constexpr int kSGVecs = 4;

// out[i] = V_i . w for i < k, out[k] = w . w (w: this thread's rows).
__device__ inline void sg_dots(int k, int64_t n, const double *__restrict__ V, int64_t ldv,
                               const double (&w)[kSGRows], double *out, small_gmres_lds &L) {
    const int t = threadIdx.x, lane = t % kWave, wv = t / kWave;
    for (int i0 = 0; i0 <= k; i0 += kSGVecs) {
        double s[kSGVecs];
#pragma unroll
        for (int u = 0; u < kSGVecs; ++u) s[u] = 0.0;
#pragma unroll
        for (int r = 0; r < kSGRows; ++r) {
            const int64_t row = t + (int64_t)r * kSGT;
            if (row < n) {
#pragma unroll
                for (int u = 0; u < kSGVecs; ++u) {
                    const int i = i0 + u;
                    if (i < k) s[u] += V[(int64_t)i * ldv + row] * w[r];
                    else if (i == k) s[u] += w[r] * w[r];
                }
            }
        }
#pragma unroll
        for (int u = 0; u < kSGVecs; ++u) {
            if (i0 + u > k) break;
            const double tot = wave_total(s[u]);
            if (lane == 0) L.red[wv][i0 + u] = tot;
        }
    }
    __syncthreads();
    if (t <= k) {
        double s = 0.0;
        for (int q = 0; q < kSGWaves; ++q) s += L.red[q][t];
        out[t] = s;
    }
    __syncthreads();
}

// w -= sum_{i < k} c_i V_i over this thread's rows, in ascending i, two
// vectors' loads at a time (four would spill).
__device__ inline void sg_subtract(int k, int64_t n, const double *__restrict__ V, int64_t ldv,
                                   const double *c, double (&w)[kSGRows]) {
    constexpr int U = 2;
    const int t = threadIdx.x;
    for (int i0 = 0; i0 < k; i0 += U) {
        double v[U][kSGRows];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int r = 0; r < kSGRows; ++r) {
                const int64_t row = t + (int64_t)r * kSGT;
                v[u][r] = (i0 + u < k && row < n) ? V[(int64_t)(i0 + u) * ldv + row] : 0.0;
            }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i0 + u < k)
#pragma unroll
                for (int r = 0; r < kSGRows; ++r) w[r] = w[r] - c[i0 + u] * v[u][r];
    }
}

// y = A v over this thread's rows (CSR rows from memory), four entries of a
// row in flight.
__device__ inline void sg_spmv(int64_t n, const int32_t *__restrict__ rp,
                               const int32_t *__restrict__ col, const double *__restrict__ val,
                               const double *__restrict__ v, double (&y)[kSGRows]) {
    const int t = threadIdx.x;
#pragma unroll
    for (int r = 0; r < kSGRows; ++r) {
        const int64_t row = t + (int64_t)r * kSGT;
        double s = 0.0;
        if (row < n) {
            const int32_t b = rp[row], e = rp[row + 1];
            int32_t q = b;
            for (; q + 4 <= e; q += 4) {
                const int32_t c0 = col[q], c1 = col[q + 1], c2 = col[q + 2], c3 = col[q + 3];
                const double x0 = v[c0], x1 = v[c1], x2 = v[c2], x3 = v[c3];
                s += val[q] * x0;
                s += val[q + 1] * x1;
                s += val[q + 2] * x2;
                s += val[q + 3] * x3;
            }
            for (; q < e; ++q) s += val[q] * v[col[q]];
        }
        y[r] = s;
    }
}

__global__ __launch_bounds__(kSGT) void gmres_small_kernel(
    int64_t n, int m, const int32_t *__restrict__ rp, const int32_t *__restrict__ col,
    const double *__restrict__ val, const double *__restrict__ b, double *__restrict__ x,
    double *__restrict__ V, int64_t ldv, double stop, int maxit, gmres_state *out) {
    __shared__ small_gmres_lds L;
    const int t = threadIdx.x;
    if (t == 0) L.est = 0.0;  // visible after the first sum's barrier
    int iter = 0, cycles = 0, reorths = 0, done = kRunning, k = 0;
    double beta = 0.0;
    double w[kSGRows];
    for (;;) {
        // cycle start: v0 = b - A x and its norm
        sg_spmv(n, rp, col, val, x, w);
#pragma unroll
        for (int r = 0; r < kSGRows; ++r) {
            const int64_t row = t + (int64_t)r * kSGT;
            w[r] = row < n ? b[row] - w[r] : 0.0;
        }
        sg_dots(0, n, V, ldv, w, L.h, L);
        beta = sqrt(L.h[0]);
        if (std::isnan(beta) || std::isinf(beta)) { done = kBreakdown; break; }
        if (beta <= stop) { done = kConverged; break; }
        if (iter >= maxit) { done = kMaxIter; break; }
        ++cycles;
#pragma unroll
        for (int r = 0; r < kSGRows; ++r) {
            const int64_t row = t + (int64_t)r * kSGT;
            if (row < n) V[row] = w[r] / beta;
        }
        if (t == 0) L.g[0] = beta;
        __syncthreads();
        for (int j = 0; j < m; ++j) {
            // w = A v_j
            sg_spmv(n, rp, col, val, V + (int64_t)j * ldv, w);
            // classical Gram-Schmidt, a second round when the first lost
            // more than 1/sqrt(2) of w
            sg_dots(j + 1, n, V, ldv, w, L.h, L);
            sg_subtract(j + 1, n, V, ldv, L.h, w);
            sg_dots(j + 1, n, V, ldv, w, L.h2, L);
            double ww = L.h2[j + 1];
            const bool reorth = 2.0 * L.h2[j + 1] < L.h[j + 1];
            if (reorth) {
                ++reorths;
                sg_subtract(j + 1, n, V, ldv, L.h2, w);
                sg_dots(0, n, V, ldv, w, &L.ww, L);
                ww = L.ww;
            }
            ++iter;
            k = j + 1;
            if (t == 0) {
                // the column of H, the earlier rotations, the new one
                double *hcol = L.hcol;
                for (int i = 0; i <= j; ++i) hcol[i] = reorth ? L.h[i] + L.h2[i] : L.h[i];
                const double hn = sqrt(ww);
                for (int i = 0; i < j; ++i) {
                    const double a = hcol[i], c = hcol[i + 1];
                    hcol[i] = L.cs[i] * a + L.sn[i] * c;
                    hcol[i + 1] = -L.sn[i] * a + L.cs[i] * c;
                }
                const double a = hcol[j];
                const double d = sqrt(a * a + hn * hn);
                L.hn = hn;
                L.breakdown = 0;
                L.cycle_done = 0;
                if (!(d > 0.0)) {
                    L.breakdown = 1;
                } else {
                    L.cs[j] = a / d;
                    L.sn[j] = hn / d;
                    hcol[j] = d;
                    for (int i = 0; i <= j; ++i) L.R[i][j] = hcol[i];
                    L.g[j + 1] = -L.sn[j] * L.g[j];
                    L.g[j] = L.cs[j] * L.g[j];
                    const double est = fabs(L.g[j + 1]);
                    L.est = est;
                    if (std::isnan(est)) L.breakdown = 1;
                    else if (est <= stop || hn == 0.0 || iter >= maxit || j + 1 == m)
                        L.cycle_done = 1;
                }
            }
            __syncthreads();
            if (L.breakdown) { done = kBreakdown; break; }
            if (L.cycle_done) break;
            const double hn = L.hn;
            double *vn = V + (int64_t)(j + 1) * ldv;
#pragma unroll
            for (int r = 0; r < kSGRows; ++r) {
                const int64_t row = t + (int64_t)r * kSGT;
                if (row < n) vn[row] = w[r] / hn;
            }
            __syncthreads();
        }
        if (done == kBreakdown) break;
        // cycle end: R y = g over the k columns, x += V_k y
        if (t == 0)
            for (int i = k - 1; i >= 0; --i) {
                double s = L.g[i];
                for (int l = i + 1; l < k; ++l) s = s - L.R[i][l] * L.y[l];
                L.y[i] = s / L.R[i][i];
            }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kSGRows; ++r) {
            const int64_t row = t + (int64_t)r * kSGT;
            if (row < n) {
                double xl = x[row];
                for (int i = 0; i < k; ++i) xl = xl + L.y[i] * V[(int64_t)i * ldv + row];
                x[row] = xl;
            }
        }
        __syncthreads();
    }
    if (t == 0) {
        out->iter = iter;
        out->cycles = cycles;
        out->reorths = reorths;
        out->done = done;
        out->est = L.est;
        out->beta = beta;
        out->k = k;
    }
}

}  // namespace

int64_t gmres_ld(int64_t n) { return (n + 63) / 64 * 64; }

int64_t gmres_partial_elems(int64_t n, int m) {
    const int64_t g = gmres_blocks(n);
    return (int64_t)(m + 2) * (gmres_compact(n) && g < kCompactMaxBlocks ? kCompactMaxBlocks : g);
}

bool gmres_compact(int64_t n) { return n <= kCompactMaxRows; }

hipError_t gmres_arnoldi_step(hipStream_t s, int64_t n, int m, int j, double *V, int64_t ldv,
                              gmres_state *st, gmres_state *next, const gmres_work &wk) {
    if (gmres_compact(n)) {
        switch (compact_threads(n)) {
            case 256: return compact_step<256>(s, n, m, j, V, ldv, st, next, wk);
            case 512: return compact_step<512>(s, n, m, j, V, ldv, st, next, wk);
            default: return compact_step<1024>(s, n, m, j, V, ldv, st, next, wk);
        }
    }
    const int g = gmres_blocks(n);
    double *w = V + (int64_t)(j + 1) * ldv;
    const int k = j + 1;
    // first Gram-Schmidt round; its update also forms the second round's dots
    gmres_dot_kernel<<<g, kG, 0, s>>>(n, k, V, ldv, w, st, 0, wk.partials);
    gmres_sum_kernel<<<k + 1, kG, 0, s>>>(g, wk.partials, wk.dot1, st, 0);
    if (k <= kGRegVecs)
        gmres_update_dot_regs_kernel<<<g, kG, 0, s>>>(n, k, V, ldv, wk.dot1, w, st, wk.partials);
    else
        gmres_update_dot_kernel<<<g, kG, 0, s>>>(n, k, V, ldv, wk.dot1, w, st, wk.partials);
    gmres_sum_kernel<<<k + 1, kG, 0, s>>>(g, wk.partials, wk.dot2, st, 0);
    gmres_check_kernel<<<1, 1, 0, s>>>(j, wk.dot1, wk.dot2, st);
    // the second round's update, only when the first lost too much of w
    gmres_update_kernel<<<g, kG, 0, s>>>(n, k, V, ldv, wk.dot2, w, st, 1, wk.partials);
    gmres_sum_kernel<<<1, kG, 0, s>>>(g, wk.partials, wk.upd2, st, 1);
    gmres_step_kernel<<<1, kWave, 0, s>>>(j, m, st, wk);
    gmres_scale_kernel<<<reduction_blocks(n), kG, 0, s>>>(n, w, st);
    return hipGetLastError();
}

hipError_t gmres_cycle_start(hipStream_t s, int64_t n, double *V, gmres_state *st,
                             gmres_state *next, const gmres_work &wk) {
    if (gmres_compact(n)) {
        switch (compact_threads(n)) {
            case 256: return compact_start<256>(s, n, V, st, next, wk);
            case 512: return compact_start<512>(s, n, V, st, next, wk);
            default: return compact_start<1024>(s, n, V, st, next, wk);
        }
    }
    // v0 . v0 through the dot pass with no basis vectors
    const int g = gmres_blocks(n);
    gmres_dot_kernel<<<g, kG, 0, s>>>(n, 0, V, 0, V, st, 2, wk.partials);
    gmres_sum_kernel<<<1, kG, 0, s>>>(g, wk.partials, wk.upd1, st, 2);
    gmres_cycle_kernel<<<1, 1, 0, s>>>(wk.upd1, st, wk.g);
    gmres_scale_kernel<<<reduction_blocks(n), kG, 0, s>>>(n, V, st);
    return hipGetLastError();
}

// us per step, estimated.  One workgroup's time grows with the dots of a step,
// the basis entries it passes over and the entries of its product; the compact
// passes are bound by their launches, whose number grows little with m, and pay
// once per cycle for the start, the update and the host's look at the state.
// Least squares over solves of two and of ten whole cycles, 15 sizes, m = 5 to
// 64; the side taken was at most 7% slower than the other, but for data on which
// the second Gram-Schmidt round is rare.  Two cycles, one workgroup / compact:
// 5-point, 225 rows GMRES(50) 29.5 / 30.0, (64) 36.4 / 32.1; 1,024 rows (30) 24.2
// / 26.5, (50) 35.1 / 30.6; 2,025 rows (20) 25.4 / 29.2, (25) 28.7 / 28.3; 4,096
// rows (10) 29.9 / 35.4, (15) 34.4 / 31.0, (30) 51.5 / 28.4; scattered, 1,500
// rows of 9 (20) 27.4 / 30.3, (30) 32.9 / 29.1, of 21 (15) 34.2 / 31.5; 4,096 of
// 21 (10) 76 / 36.
bool gmres_small_fits(int64_t n, int64_t nnz, int m) {
    if (n < 1 || n > (int64_t)kSGT * kSGRows || m < 1 || m > kGmresSmallKrylov) return false;
    const double one = 12.0 + 0.005 * m * m + 0.00016 * n * m + 0.0006 * nnz;
    return one <= 17.0 + 0.24 * m + 125.0 / m;
}

hipError_t gmres_small(hipStream_t s, int64_t n, int64_t nnz, int m, const int32_t *rp,
                       const int32_t *col, const double *val, const double *b, double *x, double *V,
                       int64_t ldv, double stop, int maxit, gmres_state *out) {
    if (!gmres_small_fits(n, nnz, m)) return hipErrorInvalidValue;
    gmres_small_kernel<<<1, kSGT, 0, s>>>(n, m, rp, col, val, b, x, V, ldv, stop, maxit, out);
    return hipGetLastError();
}

hipError_t gmres_cycle_end(hipStream_t s, int64_t n, int m, const double *V, int64_t ldv, double *x,
                           gmres_state *st, const gmres_work &wk) {
    gmres_solve_kernel<<<1, 2 * kWave, 0, s>>>(m, wk.H, wk.g, wk.y, st);
    gmres_xupdate_kernel<<<reduction_blocks(n), kG, 0, s>>>(n, V, ldv, wk.y, x, st);
    return hipGetLastError();
}

}  // namespace gko
