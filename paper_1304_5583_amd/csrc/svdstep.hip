// The ALM iteration in singular coordinates (FP64).
//
// With A = U diag(d) Qm^T the dictionary's singular value decomposition (r
// triplets), every iterate of the batched ALM lives in fixed r-dimensional
// spaces: Z, J, Y2 in range(A^T) = range(Qm), and X, E, Y1 in range(A) =
// range(U) as far as the observations lie there (for DFC-LRR they are columns of
// A); what lies outside keeps its direction, and its length is one more coordinate
// with d = 0.  Both bases are orthonormal, so the column
// norms of the l2,1 shrinkage and the singular values of the thresholding step
// are those of the coefficients, and the three dictionary products of the
// Z-step (A Q, (I + A A^T)^{-1} T, A^T V) become row scalings by d,
// 1 / (1 + d^2) and d.  What is left of an iteration outside the thresholding
// step is one pass over the columns:
//
//   Q = J - Y2/mu,  T = X - E + Y1/mu,  V = (T - d Q) / (1 + d^2),
//   q = E + V,  Z = Q + d V,  R2 = Z - J = d V - Y2/mu,  Y2' = Y2 + mu R2 = mu d V,
//   E' = f q with the column's shrinkage factor f = (1 - lam / (mu |q|))_+,
//   R1 = q - Y1/mu - E',  Y1' = Y1 + mu R1 = mu (1 - f) q,
//   Y' = Z + Y2'/mu'   (the next thresholding step's input, mu' its penalty).
//
// E and Y1 are both multiples of q, so the pair is kept as q and, per column,
// f and 1 - f.  A pass reads J, X, Y2, q and writes Y2, q, Y: 7 r doubles per
// column, where the general form moves 27 and runs three products.
// q, Y2, Y and the factors alternate between two buffers, so that the residuals
// can be formed again for the few blocks whose stop test needs their max-norm.
//
// The stop test uses max-norms of the full residuals U R1 and Qm R2.  An
// orthonormal basis gives |R e_j|_2 / sqrt(rows) <= |basis R e_j|_inf <=
// |R e_j|_2, which decides nearly every block in nearly every iteration; only
// a block that may have converged has U R1, and then Qm R2, formed.
#include <algorithm>

#include "common.hpp"
#include "kernels.hpp"

namespace lrr {

namespace {

// T = D^{-1} (3 I - D^{-1} G D^{-1}) / 2 with D = diag(G)^{1/2}: C^T T has
// orthonormal columns when the rows of C, G = C C^T, are orthogonal up to a
// small deviation (one Newton-Schulz step on the normalised rows)
__global__ __launch_bounds__(256) void k_rows_factor(const double* __restrict__ G, double* __restrict__ T, int r) {
    const long idx = (long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (long)r * r) return;
    const int i = (int)(idx % r), j = (int)(idx / r);
    const double gi = G[i + (long)i * r], gj = G[j + (long)j * r];
    const double di = gi > 0.0 ? 1.0 / sqrt(gi) : 0.0, dj = gj > 0.0 ? 1.0 / sqrt(gj) : 0.0;
    T[idx] = di * ((i == j ? 1.5 : 0.0) - 0.5 * di * G[idx] * dj);
}

// diagonal of the r x r matrix A (ld) into d, 1 / (1 + d^2) into dinv; stat[0] = max
// off-diagonal entry, stat[1] = max diagonal entry (bit patterns).  A NaN would
// lose every comparison, so it is recorded as infinity.
__global__ __launch_bounds__(256) void k_take_diag(const double* __restrict__ A, int r, long ld, double* __restrict__ d,
                                                    double* __restrict__ dinv, unsigned long long* __restrict__ stat) {
    double off = 0.0, dia = 0.0;
    const int j = blockIdx.x;
    for (int i = threadIdx.x; i < r; i += 256) {
        const double a = A[i + j * ld];
        const double x = a == a ? fabs(a) : INFINITY;
        if (i == j) {
            d[i] = a;
            dinv[i] = 1.0 / (1.0 + a * a);
            dia = x;
        } else {
            off = fmax(off, x);
        }
    }
    off = wave_max(off);
    dia = wave_max(dia);
    if ((threadIdx.x & 63) == 0) {
        atomic_max_nonneg(&stat[0], off);
        atomic_max_nonneg(&stat[1], dia);
    }
}

// largest column 2-norm of A (m x ncols), one wave per column
__global__ __launch_bounds__(256) void k_colnorm_max(const double* __restrict__ A, int m, long ld, int ncols,
                                                      unsigned long long* __restrict__ out) {
    double mx = 0.0;
    for (int j = blockIdx.x * 4 + (threadIdx.x >> 6); j < ncols; j += gridDim.x * 4) {
        double s = 0.0;
        for (int i = threadIdx.x & 63; i < m; i += 64) {
            const double x = A[i + (long)j * ld];
            s += x * x;
        }
        s = wave_sum(s);
        mx = fmax(mx, s == s ? sqrt(s) : INFINITY);
    }
    if ((threadIdx.x & 63) == 0) atomic_max_nonneg(out, mx);
}

// 1 / mu, finite also for the smallest penalties: 0 / mu has to stay 0
__device__ __forceinline__ double inv_mu(double mu) { return fmin(1.0 / mu, 1.7976931348623157e308); }

// sum over the TPC threads (64 or 256) that share a column
template <int TPC>
__device__ __forceinline__ double col_sum(double v, double* red) {
    v = wave_sum(v);
    if (TPC == 64) return v;
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) red[w] = v;
    __syncthreads();
    const double r = (red[0] + red[1]) + (red[2] + red[3]);
    __syncthreads();
    return r;
}

template <bool VEC>
__device__ __forceinline__ void load2(const double* __restrict__ p, int i, int n, double& a, double& b) {
    if (VEC && i + 1 < n) {
        const double2 x = *reinterpret_cast<const double2*>(p + i);
        a = x.x;
        b = x.y;
    } else {
        a = i < n ? p[i] : 0.0;
        b = i + 1 < n ? p[i + 1] : 0.0;
    }
}
template <bool VEC>
__device__ __forceinline__ void store2(double* __restrict__ p, int i, int n, double a, double b) {
    if (VEC && i + 1 < n) {
        *reinterpret_cast<double2*>(p + i) = double2{a, b};
    } else {
        if (i < n) p[i] = a;
        if (i + 1 < n) p[i + 1] = b;
    }
}

// One iteration's column pass (see the top of the file).  TPC threads share a
// column (a wave up to 512 rows, the workgroup beyond); each holds NCH pairs of
// consecutive rows in registers (NCH * 2 * TPC >= r), so that the column norm
// is known before E' and R1 are formed without a second read.  NCH = 0: any r,
// q read again from memory.
template <int TPC, int NCH, bool VEC>
__global__ __launch_bounds__(256) void k_zstep_fused(SvdStep a, BlockState bs, const DevIter* __restrict__ it,
                                                      const double* __restrict__ sched) {
    __shared__ double red[4];
    constexpr int CPW = 256 / TPC;
    const int j = blockIdx.x * CPW + threadIdx.x / TPC;
    if (j >= a.ncols) return;
    const int b = a.colblk[j];
    if (!bs.active[b]) return;
    const bool run = bs.svt_run[b] != 0;
    const int lane = threadIdx.x % TPC, k = it->k, r = a.r;
    const double mu = it->mu, imu = inv_mu(mu);
    const double ratio = k > 0 ? sched[k - 1] / mu : 1.0;   // mu of the stored E, Y1 over mu
    const double fnext = mu / sched[k + 1];
    const double f = a.f0[2 * j], g = a.f0[2 * j + 1];      // E = f q, Y1 = mu g q, g = 1 - f
    const double y1 = ratio * g, ax = y1 - f;               // T = X + ax q, Y1/mu = y1 q
    const long o = (long)j * r, od = (long)b * a.dstride;
    constexpr int N = NCH > 0 ? NCH : 1;
    double qn[N][2], qo[N][2];
    double sq = 0.0, s2 = 0.0, sy = 0.0;
    auto pass = [&](int i, double (&qnew)[2], double (&qold)[2]) {
        double x[2], y2[2], jj[2] = {0.0, 0.0}, d[2], di[2];
        load2<VEC>(a.X + o, i, r, x[0], x[1]);
        load2<VEC>(a.q0 + o, i, r, qold[0], qold[1]);
        load2<VEC>(a.Y20 + o, i, r, y2[0], y2[1]);
        if (run) load2<VEC>(a.J + o, i, r, jj[0], jj[1]);   // J = 0 where nothing was thresholded
        load2<true>(a.d + od, i, r, d[0], d[1]);
        load2<true>(a.dinv + od, i, r, di[0], di[1]);
        double y2n[2], yn[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const double Q = jj[h] - y2[h] * imu;
            const double V = ((x[h] + ax * qold[h]) - d[h] * Q) * di[h];
            const double dv = d[h] * V;
            const double r2 = dv - y2[h] * imu;
            qnew[h] = f * qold[h] + V;
            y2n[h] = mu * dv;
            yn[h] = (jj[h] + r2) + fnext * dv;
            sq += qnew[h] * qnew[h];   // rows past r hold zeros
            s2 += r2 * r2;
            sy += yn[h] * yn[h];
        }
        store2<VEC>(a.Y21 + o, i, r, y2n[0], y2n[1]);
        store2<VEC>(a.Y1 + o, i, r, yn[0], yn[1]);
        store2<VEC>(a.q1 + o, i, r, qnew[0], qnew[1]);
    };
    if (NCH > 0) {
#pragma unroll
        for (int c = 0; c < N; ++c) pass(2 * (c * TPC + lane), qn[c], qo[c]);
    } else {
        for (int i = 2 * lane; i < r; i += 2 * TPC) pass(i, qn[0], qo[0]);
    }
    sq = col_sum<TPC>(sq, red);
    const double nrm = sqrt(sq), thr = a.lam / mu;
    const double g1 = nrm > thr ? thr / nrm : 1.0, f1 = nrm > thr ? 1.0 - thr / nrm : 0.0;
    double s1 = 0.0;
    if (NCH > 0) {
#pragma unroll
        for (int c = 0; c < N; ++c)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const double r1 = g1 * qn[c][h] - y1 * qo[c][h];
                s1 += r1 * r1;
            }
    } else {
        for (int i = 2 * lane; i < r; i += 2 * TPC) {
            double u[2], v[2];
            load2<VEC>(a.q1 + o, i, r, u[0], u[1]);   // this thread's own stores
            load2<VEC>(a.q0 + o, i, r, v[0], v[1]);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const double r1 = g1 * u[h] - y1 * v[h];
                s1 += r1 * r1;
            }
        }
    }
    s1 = col_sum<TPC>(s1, red);
    s2 = col_sum<TPC>(s2, red);
    sy = col_sum<TPC>(sy, red);
    if (lane == 0) {
        a.f1[2 * j] = f1;
        a.f1[2 * j + 1] = g1;
        a.colsq[j] = sy;
        // a NaN would lose every later comparison and meet the stop test
        bs.colr1[j] = s1 == s1 ? sqrt(s1) : INFINITY;
        bs.colr2[j] = s2 == s2 ? sqrt(s2) : INFINITY;
    }
}

// Per block: the largest column 2-norms x1, x2 of the two residuals and what they
// decide (one workgroup per block).  x1 >= sqrt(m) tol or x2 >= sqrt(n) tol: not
// converged, the lower bounds are recorded.  Otherwise, and in the last
// iteration, whose residuals are reported, U R1 is formed (expand1).
__global__ __launch_bounds__(256) void k_svd_decide(const int* __restrict__ boff, BlockState bs,
                                                     unsigned long long* __restrict__ x2max,
                                                     int* __restrict__ expand1, int* __restrict__ expand2, double tol,
                                                     double sqrt_m, double sqrt_n, int n_iter, const DevIter* it) {
    __shared__ double red[8];
    const int b = blockIdx.x;
    if (!bs.active[b]) {
        if (threadIdx.x == 0) expand1[b] = expand2[b] = 0;
        return;
    }
    double m1 = 0.0, m2 = 0.0;
    for (int c = boff[b] + threadIdx.x; c < boff[b + 1]; c += 256) {
        m1 = fmax(m1, bs.colr1[c]);
        m2 = fmax(m2, bs.colr2[c]);
    }
    m1 = wave_max(m1);
    m2 = wave_max(m2);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        red[w] = m1;
        red[4 + w] = m2;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const double x1 = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
        const double x2 = fmax(fmax(red[4], red[5]), fmax(red[6], red[7]));
        const bool last = it->k + 1 >= n_iter;
        const bool open = x1 >= sqrt_m * tol || x2 >= sqrt_n * tol;
        const int e = (!open || last) ? 1 : 0;
        expand1[b] = e;
        expand2[b] = 0;
        x2max[b] = dbl_bits(x2);
        // a lower bound that decides must not round below tol
        bs.r1max[b] = e ? 0ull : dbl_bits(x1 >= sqrt_m * tol ? fmax(x1 / sqrt_m, tol) : x1 / sqrt_m);
        bs.r2max[b] = dbl_bits(x2 < tol ? x2 : (x2 >= sqrt_n * tol ? fmax(x2 / sqrt_n, tol) : x2 / sqrt_n));
    }
}

// After U R1: Qm R2 is formed where its bounds leave the stop test open
__global__ void k_svd_decide2(BlockState bs, const unsigned long long* __restrict__ x2max,
                              const int* __restrict__ expand1, int* __restrict__ expand2, int t, double tol,
                              double sqrt_n, int n_iter, const DevIter* it) {
    const bool last = it->k + 1 >= n_iter;
    for (int b = threadIdx.x; b < t; b += blockDim.x) {
        if (!expand1[b]) continue;
        const double r1 = __longlong_as_double((long long)bs.r1max[b]);
        const double x2 = __longlong_as_double((long long)x2max[b]);
        const int e = (r1 < tol || last) && x2 >= tol && x2 < sqrt_n * tol ? 1 : 0;
        expand2[b] = e;
        if (e) bs.r2max[b] = 0ull;
    }
}

// The coefficient residuals of the flagged blocks, from the pass's two buffers:
// R1 = g1 q' - (Y1/mu) (which = 1) or R2 = Y2'/mu - Y2/mu (which = 2)
__global__ __launch_bounds__(256) void k_svd_resid(SvdStep a, const int* __restrict__ boff,
                                                    const int* __restrict__ expand, double* __restrict__ R, int which,
                                                    const DevIter* __restrict__ it, const double* __restrict__ sched) {
    const int b = blockIdx.y;
    if (!expand[b]) return;
    const int k = it->k, r = a.r;
    const double imu = inv_mu(it->mu), ratio = k > 0 ? sched[k - 1] / it->mu : 1.0;
    for (int j = boff[b] + blockIdx.x * 4 + (threadIdx.x >> 6); j < boff[b + 1]; j += gridDim.x * 4) {
        const long o = (long)j * r;
        const double g1 = a.f1[2 * j + 1], y1 = ratio * a.f0[2 * j + 1];
        for (int i = threadIdx.x & 63; i < r; i += 64)
            R[o + i] = which == 1 ? g1 * a.q1[o + i] - y1 * a.q0[o + i] : a.Y21[o + i] * imu - a.Y20[o + i] * imu;
    }
}

// |x|, a NaN as infinity
__device__ __forceinline__ double abs_or_inf(double x) { return x == x ? fabs(x) : INFINITY; }

// max |A[:, j] + D[:, j] R[r - 1, j]| over the columns of the flagged blocks; D
// (may be null): the directions outside range(U), whose coordinate is the last row
// of the r-row coefficients R
__global__ __launch_bounds__(256) void k_svd_colmax(const double* __restrict__ A, int rows, long ld,
                                                     const int* __restrict__ boff, const int* __restrict__ expand,
                                                     unsigned long long* __restrict__ out,
                                                     const double* __restrict__ D, const double* __restrict__ R,
                                                     int r) {
    const int b = blockIdx.y;
    if (!expand[b]) return;
    double mx = 0.0;
    for (int j = boff[b] + blockIdx.x * 4 + (threadIdx.x >> 6); j < boff[b + 1]; j += gridDim.x * 4) {
        const double w = D ? R[r - 1 + (long)j * r] : 0.0;
        for (int i = threadIdx.x & 63; i < rows; i += 64) {
            const long k = i + (long)j * ld;
            mx = fmax(mx, abs_or_inf(D ? A[k] + D[k] * w : A[k]));
        }
    }
    mx = wave_max(mx);
    if ((threadIdx.x & 63) == 0 && mx > 0.0) atomic_max_nonneg(&out[b], mx);
}

// The expansions for small problems in one launch each, without the coefficient
// and result matrices: max |basis R e_j| over a block's columns, R1 with the left
// basis (which = 1) for the blocks flagged in expand1, then R2 with the right one
// where its bounds leave the stop test open (the test of k_svd_decide2; the
// recorded lower bound is not above the exact value, so the maximum replaces it).
// One wave per column, a lane per row; the coefficients are formed on the way.
template <int WHICH>
__global__ __launch_bounds__(256) void k_svd_expand(SvdStep a, const double* __restrict__ basis, int rows,
                                                     const double* __restrict__ D, const int* __restrict__ boff,
                                                     BlockState bs, const unsigned long long* __restrict__ x2max,
                                                     const int* __restrict__ expand1, double tol, double sqrt_n,
                                                     int n_iter, const DevIter* __restrict__ it,
                                                     const double* __restrict__ sched) {
    const int b = blockIdx.y;
    if (!expand1[b]) return;
    const int k = it->k, r = a.r;
    if (WHICH == 2) {
        const double r1 = __longlong_as_double((long long)bs.r1max[b]);
        const double x2 = __longlong_as_double((long long)x2max[b]);
        if (!((r1 < tol || k + 1 >= n_iter) && x2 >= tol && x2 < sqrt_n * tol)) return;
    }
    const double imu = inv_mu(it->mu), ratio = k > 0 ? sched[k - 1] / it->mu : 1.0;
    double mx = 0.0;
    for (int j = boff[b] + blockIdx.x * 4 + (threadIdx.x >> 6); j < boff[b + 1]; j += gridDim.x * 4) {
        const long o = (long)j * r;
        const double g1 = a.f1[2 * j + 1], y1 = ratio * a.f0[2 * j + 1];
        for (int i = threadIdx.x & 63; i < rows; i += 64) {
            double acc = 0.0, v = 0.0;
            for (int q = 0; q < r; ++q) {
                v = WHICH == 1 ? g1 * a.q1[o + q] - y1 * a.q0[o + q] : a.Y21[o + q] * imu - a.Y20[o + q] * imu;
                acc += basis[i + (long)q * rows] * v;
            }
            if (D) acc += D[i + (long)j * rows] * v;
            mx = fmax(mx, abs_or_inf(acc));
        }
    }
    mx = wave_max(mx);
    if ((threadIdx.x & 63) == 0 && mx > 0.0) atomic_max_nonneg(WHICH == 1 ? &bs.r1max[b] : &bs.r2max[b], mx);
}

// The end of an iteration of a small problem in one launch, one workgroup per block:
// the decision of k_svd_decide, the expansions it asks for, the stop test, and
// ||Y||_F against the next threshold; the last workgroup to finish advances the
// iteration.  Five launches of about 3 us otherwise.
template <int WHICH>
__device__ double expand_max(const SvdStep& a, const double* __restrict__ basis, int rows,
                             const double* __restrict__ D, int c0, int c1, double imu, double ratio, double* red) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, r = a.r;
    double mx = 0.0;
    for (int j = c0 + w; j < c1; j += 16) {
        const long o = (long)j * r;
        const double g1 = a.f1[2 * j + 1], y1 = ratio * a.f0[2 * j + 1];
        for (int i = lane; i < rows; i += 64) {
            double acc = 0.0, v = 0.0;
#pragma unroll 4
            for (int q = 0; q < r; ++q) {
                v = WHICH == 1 ? g1 * a.q1[o + q] - y1 * a.q0[o + q] : a.Y21[o + q] * imu - a.Y20[o + q] * imu;
                acc += basis[i + (long)q * rows] * v;
            }
            if (D) acc += D[i + (long)j * rows] * v;
            mx = fmax(mx, abs_or_inf(acc));
        }
    }
    mx = wave_max(mx);
    __syncthreads();
    if (lane == 0) red[w] = mx;
    __syncthreads();
    for (int q = 0; q < 16; ++q) mx = fmax(mx, red[q]);
    return mx;
}

__global__ __launch_bounds__(1024) void k_svd_tail(SvdStep a, SvdTail z, BlockState bs, DevIter* it,
                                                    const double* __restrict__ sched) {
    __shared__ double red[48];
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int k = it->k;
    const double mu = it->mu, imu = inv_mu(mu), ratio = k > 0 ? sched[k - 1] / mu : 1.0;
    const bool last = k + 1 >= z.n_iter, act = bs.active[b] != 0;
    if (act) {
        const int c0 = z.boff[b], c1 = z.boff[b + 1];
        double x1 = 0.0, x2 = 0.0, fro = 0.0;
        for (int c = c0 + tid; c < c1; c += 1024) {
            x1 = fmax(x1, bs.colr1[c]);
            x2 = fmax(x2, bs.colr2[c]);
            fro += a.colsq[c];
        }
        x1 = wave_max(x1);
        x2 = wave_max(x2);
        fro = wave_sum(fro);
        if (lane == 0) {
            red[w] = x1;
            red[16 + w] = x2;
            red[32 + w] = fro;
        }
        __syncthreads();
        fro = 0.0;
        for (int q = 0; q < 16; ++q) {
            x1 = fmax(x1, red[q]);
            x2 = fmax(x2, red[16 + q]);
            fro += red[32 + q];
        }
        const double tol = z.tol;
        const bool lo1 = x1 >= z.sqrt_m * tol, lo2 = x2 >= z.sqrt_n * tol;
        // lower bounds that decide must not round below tol
        double r1 = lo1 ? fmax(x1 / z.sqrt_m, tol) : x1 / z.sqrt_m;
        double r2 = x2 < tol ? x2 : (lo2 ? fmax(x2 / z.sqrt_n, tol) : x2 / z.sqrt_n);
        if (!(lo1 || lo2) || last) {
            r1 = expand_max<1>(a, z.U, z.m, z.D, c0, c1, imu, ratio, red);
            if ((r1 < tol || last) && x2 >= tol && !lo2)
                r2 = expand_max<2>(a, z.Q, z.n, nullptr, c0, c1, imu, ratio, red);
        }
        if (tid == 0) {
            bs.res1[b] = r1;
            bs.res2[b] = r2;
            bs.iters[b] = k + 1;
            const bool stop = !z.fixed && r1 < tol && r2 < tol;
            if (stop) bs.active[b] = 0;
            else atomicAdd(&z.tick[1], 1);
            // sigma_max <= ||Y||_F, so ||Y||_F <= tau gives J = 0 without a decomposition
            const bool run = !stop && !last && sqrt(fro) > 1.0 / sched[k + 1];
            if (!last) {
                bs.svt_run[b] = run ? 1 : 0;
                if (!stop && !run) bs.rank[b] = 0;
            }
        }
    }
    if (tid == 0) {
        __threadfence();
        if (atomicAdd(&z.tick[0], 1) == (int)gridDim.x - 1) {
            __threadfence();
            *z.n_active = atomicExch(&z.tick[1], 0);
            z.tick[0] = 0;
            it->k = k + 1;
            it->mu = sched[k + 1];
            it->tau = 1.0 / sched[k + 1];
        }
    }
}

// Results of a finished solve, per block from the buffers its last pass wrote
// (iters passes: buffer iters & 1):  what = 0: E = f q;  what = 1: Z = Y - Y2/mu'
// (mu' the penalty after the last iteration).
__global__ __launch_bounds__(256) void k_svd_result(SvdStep a, const int* __restrict__ iters,
                                                     double* __restrict__ out, int what,
                                                     const double* __restrict__ sched) {
    const int j = blockIdx.x;
    const int n = iters[a.colblk[j]];
    const bool odd = (n & 1) != 0;
    const long o = (long)j * a.r;
    const double f = (odd ? a.f1 : a.f0)[2 * j], imu = inv_mu(sched[n]);
    const double* q = odd ? a.q1 : a.q0;
    const double* Y = odd ? a.Y1 : a.Y0;
    const double* Y2 = odd ? a.Y21 : a.Y20;
    for (int i = threadIdx.x; i < a.r; i += 256) out[o + i] = what == 0 ? f * q[o + i] : Y[o + i] - Y2[o + i] * imu;
}

// T (m x c): per column its length into len and its direction into D (zero if T is)
__global__ __launch_bounds__(256) void k_svd_outside(const double* __restrict__ T, int m, int c,
                                                      double* __restrict__ D, double* __restrict__ len) {
    const int j = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (j >= c) return;
    const long o = (long)j * m;
    double s = 0.0;
    for (int i = threadIdx.x & 63; i < m; i += 64) s += T[o + i] * T[o + i];
    const double nrm = sqrt(wave_sum(s)), inv = nrm > 0.0 ? 1.0 / nrm : 0.0;
    for (int i = threadIdx.x & 63; i < m; i += 64) D[o + i] = T[o + i] * inv;
    if ((threadIdx.x & 63) == 0) len[j] = nrm;
}

// X[:, j] (ldx) = the rows values of Xs[:, j] (ld rows), zero beyond
__global__ __launch_bounds__(256) void k_svd_pad_cols(const double* __restrict__ Xs, int rows, double* __restrict__ X,
                                                       int ldx) {
    const long j = blockIdx.x;
    for (int i = threadIdx.x; i < ldx; i += 256) X[i + j * ldx] = i < rows ? Xs[i + j * rows] : 0.0;
}

__global__ __launch_bounds__(256) void k_svd_set_row(double* __restrict__ X, int row, int ld, int c,
                                                      const double* __restrict__ v) {
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j < c) X[row + (long)j * ld] = v[j];
}

// out[:, map(j)] += D[:, j] R[r - 1, j]
__global__ __launch_bounds__(256) void k_svd_add_outside(double* __restrict__ out, long ldo, int m,
                                                          const double* __restrict__ D,
                                                          const double* __restrict__ R, int r,
                                                          const int* __restrict__ map) {
    const int j = blockIdx.x;
    const double w = R[r - 1 + (long)j * r];
    double* o = out + (map ? map[j] : j) * ldo;
    for (int i = threadIdx.x; i < m; i += 256) o[i] += D[i + (long)j * m] * w;
}

// U (rows x L) = the columns of W (L x L) with h > 0, zero elsewhere
__global__ __launch_bounds__(256) void k_svd_left_basis(const double* __restrict__ W, int L,
                                                         const double* __restrict__ h, double* __restrict__ U,
                                                         int rows) {
    const long j = blockIdx.x;
    const bool keep = h[j] > 0.0;
    for (int i = threadIdx.x; i < rows; i += 256) U[i + j * rows] = keep ? W[i + j * L] : 0.0;
}

// J = 0 for the blocks whose last thresholding step kept nothing
__global__ __launch_bounds__(256) void k_svd_zero_J(double* __restrict__ J, int r, const int* __restrict__ colblk,
                                                     const int* __restrict__ rank) {
    const int j = blockIdx.x;
    if (rank[colblk[j]] != 0) return;
    for (int i = threadIdx.x; i < r; i += 256) J[i + (long)j * r] = 0.0;
}

template <int TPC, int NCH>
void launch_fused(const SvdStep& a, const BlockState& bs, const DevIter* it, const double* sched, hipStream_t s) {
    const dim3 grid((a.ncols * TPC + 255) / 256);
    if ((a.r & 1) == 0)
        hipLaunchKernelGGL((k_zstep_fused<TPC, NCH, true>), grid, dim3(256), 0, s, a, bs, it, sched);
    else
        hipLaunchKernelGGL((k_zstep_fused<TPC, NCH, false>), grid, dim3(256), 0, s, a, bs, it, sched);
}

dim3 block_cols_grid(int t, int maxl) { return dim3((unsigned)std::min((maxl + 3) / 4, 64), t); }

}  // namespace

void launch_rows_factor(const double* G, double* T, int r, hipStream_t s) {
    const long nn = (long)r * r;
    hipLaunchKernelGGL(k_rows_factor, dim3((unsigned)((nn + 255) / 256)), dim3(256), 0, s, G, T, r);
}
void launch_take_diag(const double* A, int r, long ld, double* d, double* dinv, unsigned long long* stat, hipStream_t s) {
    hipLaunchKernelGGL(k_take_diag, dim3(r), dim3(256), 0, s, A, r, ld, d, dinv, stat);
}
void launch_colnorm_max(const double* A, int m, long ld, int ncols, unsigned long long* out, hipStream_t s) {
    hipLaunchKernelGGL(k_colnorm_max, dim3(std::min((ncols + 3) / 4, 1024)), dim3(256), 0, s, A, m, ld, ncols, out);
}

void launch_zstep_fused(const SvdStep& a, const BlockState& bs, const DevIter* it, const double* sched,
                        hipStream_t s) {
    // a wave per column while a lane holds it in at most 4 + 4 pairs; then a
    // workgroup per column up to 4096 rows, beyond that q is read again
    if (a.r <= 128) launch_fused<64, 1>(a, bs, it, sched, s);
    else if (a.r <= 256) launch_fused<64, 2>(a, bs, it, sched, s);
    else if (a.r <= 512) launch_fused<64, 4>(a, bs, it, sched, s);
    else if (a.r <= 1024) launch_fused<256, 2>(a, bs, it, sched, s);
    else if (a.r <= 2048) launch_fused<256, 4>(a, bs, it, sched, s);
    else if (a.r <= 4096) launch_fused<256, 8>(a, bs, it, sched, s);
    else launch_fused<256, 0>(a, bs, it, sched, s);
}
void launch_svd_decide(const int* boff, int t, const BlockState& bs, unsigned long long* x2max, int* expand1,
                       int* expand2, double tol, double sqrt_m, double sqrt_n, int n_iter, const DevIter* it,
                       hipStream_t s) {
    hipLaunchKernelGGL(k_svd_decide, dim3(t), dim3(256), 0, s, boff, bs, x2max, expand1, expand2, tol, sqrt_m, sqrt_n,
                       n_iter, it);
}
void launch_svd_decide2(const BlockState& bs, const unsigned long long* x2max, const int* expand1, int* expand2, int t,
                        double tol, double sqrt_n, int n_iter, const DevIter* it, hipStream_t s) {
    hipLaunchKernelGGL(k_svd_decide2, dim3(1), dim3(256), 0, s, bs, x2max, expand1, expand2, t, tol, sqrt_n, n_iter,
                       it);
}
void launch_svd_resid(const SvdStep& a, const int* boff, int t, int maxl, const int* expand, double* R, int which,
                      const DevIter* it, const double* sched, hipStream_t s) {
    hipLaunchKernelGGL(k_svd_resid, block_cols_grid(t, maxl), dim3(256), 0, s, a, boff, expand, R, which, it, sched);
}
void launch_svd_colmax(const double* A, int rows, long ld, const int* boff, int t, int maxl, const int* expand,
                       unsigned long long* out, const double* D, const double* R, int r, hipStream_t s) {
    hipLaunchKernelGGL(k_svd_colmax, block_cols_grid(t, maxl), dim3(256), 0, s, A, rows, ld, boff, expand, out, D, R,
                       r);
}
void launch_svd_expand(const SvdStep& a, int which, const double* basis, int rows, const double* D, const int* boff,
                       int t, int maxl, const BlockState& bs, const unsigned long long* x2max, const int* expand1,
                       double tol, double sqrt_n, int n_iter, const DevIter* it, const double* sched, hipStream_t s) {
    const dim3 grid = block_cols_grid(t, maxl);
    if (which == 1)
        hipLaunchKernelGGL((k_svd_expand<1>), grid, dim3(256), 0, s, a, basis, rows, D, boff, bs, x2max, expand1, tol,
                           sqrt_n, n_iter, it, sched);
    else
        hipLaunchKernelGGL((k_svd_expand<2>), grid, dim3(256), 0, s, a, basis, rows, D, boff, bs, x2max, expand1, tol,
                           sqrt_n, n_iter, it, sched);
}
void launch_svd_tail(const SvdStep& a, const SvdTail& z, int t, const BlockState& bs, DevIter* it,
                     const double* sched, hipStream_t s) {
    hipLaunchKernelGGL(k_svd_tail, dim3(t), dim3(1024), 0, s, a, z, bs, it, sched);
}
void launch_svd_outside(const double* T, int m, int c, double* D, double* len, hipStream_t s) {
    hipLaunchKernelGGL(k_svd_outside, dim3((c + 3) / 4), dim3(256), 0, s, T, m, c, D, len);
}
void launch_svd_pad_cols(const double* Xs, int rows, double* X, int ldx, int cols, hipStream_t s) {
    hipLaunchKernelGGL(k_svd_pad_cols, dim3(cols), dim3(256), 0, s, Xs, rows, X, ldx);
}
void launch_svd_set_row(double* X, int row, int ld, int c, const double* v, hipStream_t s) {
    hipLaunchKernelGGL(k_svd_set_row, dim3((c + 255) / 256), dim3(256), 0, s, X, row, ld, c, v);
}
void launch_svd_add_outside(double* out, long ldo, int m, int c, const double* D, const double* R, int r,
                            const int* map, hipStream_t s) {
    hipLaunchKernelGGL(k_svd_add_outside, dim3(c), dim3(256), 0, s, out, ldo, m, D, R, r, map);
}
void launch_svd_result(const SvdStep& a, const int* iters, double* out, int what, const double* sched, hipStream_t s) {
    hipLaunchKernelGGL(k_svd_result, dim3(a.ncols), dim3(256), 0, s, a, iters, out, what, sched);
}
void launch_svd_left_basis(const double* W, int L, const double* h, double* U, int rows, hipStream_t s) {
    hipLaunchKernelGGL(k_svd_left_basis, dim3(L), dim3(256), 0, s, W, L, h, U, rows);
}
void launch_svd_zero_J(double* J, int r, int ncols, const int* colblk, const int* rank, hipStream_t s) {
    hipLaunchKernelGGL(k_svd_zero_J, dim3(ncols), dim3(256), 0, s, J, r, colblk, rank);
}

}  // namespace lrr
