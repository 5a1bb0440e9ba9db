// Eigen-decompositions of small symmetric matrices (order <= 96), one workgroup
// per matrix, the whole solve in LDS (FP64).
//
// At these orders the launch-per-round solver of jacobi.hip and the refinement of
// refsyev.hip are bound by launches: an iteration of the batched ALM on blocks
// of 32 points made about 55 of them.  Here the matrix and its eigenvectors stay in
// LDS (2 x 96 x 97 doubles = 146 KB of the CU's 160), the products that start and
// end a thresholding step run on the matrix cores out of LDS, and a sweep costs
// two barriers per round instead of two launches:
//   X <- X (3 I - X^T X) / 2   (the previous iteration's eigenvectors),
//   B = X^T G X, first-order corrections or cyclic Jacobi sweeps until nothing exceeds
//   the tolerance of jacobi.hip, X <- X R, one correction of what is below it,  weights
//   from the eigenvalues,  P = X diag(g) X^T.
// Plain LRR of 200 points (order 45): 57 -> 28 ms per solve; 3 blocks of 32 points
// (order 15): 35 -> 9 ms.
#include <algorithm>

#include "common.hpp"
#include "jacobi_rot.hpp"
#include "kernels.hpp"

namespace lrr {

namespace {

constexpr double kRelTol = 1e-15;
constexpr double kAbsFloor = 1e-14;

// op(A) op(B) for E x E operands in LDS (row stride ES), 16 x 16 tiles over the
// waves of the workgroup, results in registers (tile slot u of a wave: tile
// wave + u * waves)
template <int NT, int MT, bool TA, bool TB>
__device__ __forceinline__ void mm_regs(const double* A, const double* B, int E, int ES, dbl4 (&acc)[MT]) {
    const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4, nt = E >> 4;
#pragma unroll
    for (int u = 0; u < MT; ++u) {
        const int t = (threadIdx.x >> 6) + u * (NT / 64);
        acc[u] = dbl4{0.0, 0.0, 0.0, 0.0};
        if (t >= nt * nt) continue;
        const int ti = (t % nt) * 16 + lr, tj = (t / nt) * 16 + lr;
#pragma unroll 2
        for (int k0 = 0; k0 < E; k0 += 4) {
            const int k = k0 + lk;
            const double a = TA ? A[k * ES + ti] : A[ti * ES + k];
            const double b = TB ? B[tj * ES + k] : B[k * ES + tj];
            acc[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc[u], 0, 0, 0);
        }
    }
}
// f(row, column, value) for every element a thread holds
template <int NT, int MT, class F>
__device__ __forceinline__ void each(const dbl4 (&acc)[MT], int E, F&& f) {
    const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4, nt = E >> 4;
#pragma unroll
    for (int u = 0; u < MT; ++u) {
        const int t = (threadIdx.x >> 6) + u * (NT / 64);
        if (t >= nt * nt) continue;
#pragma unroll
        for (int v = 0; v < 4; ++v) f((t % nt) * 16 + lk + 4 * v, (t / nt) * 16 + lr, acc[u][v]);
    }
}

// What a check of B finds (per workgroup, in LDS)
struct Found {
    int above;      // some entry exceeds the tolerance
    int steep;      // some such entry exceeds kLinear of its two eigenvalues' distance
    double sum;     // sum of the squared first-order corrections
    double most;    // largest of them
};
constexpr double kLinear = 0.1;     // largest correction the refinement takes
constexpr double kDone = 1e-13;     // corrections up to which the eigenvectors are final
constexpr double kRounding = 1e-14; // couplings below this part of an eigenvalue don't change it or its vector
constexpr double kSumMax = 0.02;    // and largest sum of their squares
constexpr double kWarmMax = 1e-6;   // |X^T X - I| up to which earlier eigenvectors are used
constexpr double kStepMax = 0.1;    // and above which a correction is given up

// LDS of a small solve: B, X, then these
template <int NT>
struct SmallLds {
    double *B, *X, *cs, *sn, *lam;
    int* pr;
    Found* f;
    double* red;
    __device__ SmallLds(double* lds, int E) {
        B = lds;
        X = B + E * (E + 1);
        cs = X + E * (E + 1);
        sn = cs + 48;
        lam = sn + 48;
        red = lam + 96;
        f = reinterpret_cast<Found*>(red + 32);
        pr = reinterpret_cast<int*>(f + 1);
    }
};
constexpr int kSmallTail = 96 + 96 + 32 + 4 + 24;   // doubles beyond B and X

template <int NT>
__device__ double diag_max(const SmallLds<NT>& m, int e, int ES) {
    double mx = 0.0;
    for (int i = threadIdx.x; i < e; i += NT) mx = fmax(mx, fabs(m.B[i * ES + i]));
    mx = wave_max(mx);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) m.red[threadIdx.x >> 6] = mx;
    __syncthreads();
    for (int w = 0; w < NT / 64; ++w) mx = fmax(mx, m.red[w]);
    return mx;
}

// Whether entry b of B couples two indices with diagonal entries di and dj above the
// tolerance of a rotation, and the first-order correction v = b / (dj - di) it asks for, 0
// where that does not apply.  Corrections don't stop at the rotations' absolute floor: for an
// eigenvalue of 1e-8 of the largest a coupling of 1e-14 is an angle of 1e-6 (m = 72, n =
// 224, replaced columns: Z off by 9e-4 instead of 1e-6).  Below it a coupling matters if the
// larger of its eigenvalues is not far below the squared threshold, and if it is more than
// rounding of that eigenvalue or stands between a kept and a dropped one.
__device__ __forceinline__ bool coupling(double b, double di, double dj, double floor_abs, double tau2, bool& steep,
                                         double& v) {
    const double s = fabs(b), gap = dj - di, big = fmax(di, dj);
    const bool above = s > fmax(kRelTol * sqrt(fabs(di * dj)), floor_abs);
    const bool lin = s <= kLinear * fabs(gap) && gap != 0.0;
    const bool small = big > 0.25 * tau2 && (s > kRounding * big || (di > tau2) != (dj > tau2));
    steep = above && !lin;
    v = lin && (above || small) ? b / gap : 0.0;
    return above;
}

// entries above the tolerance (relative to the two diagonal entries, and floor_abs),
// and whether first-order corrections would resolve what is left
template <int NT>
__device__ Found check(const SmallLds<NT>& m, int e, int ES, double floor_abs, double tau2) {
    const int tid = threadIdx.x;
    __syncthreads();
    if (tid == 0) {
        m.f->above = 0;
        m.f->steep = 0;
    }
    __syncthreads();
    int above = 0, steep = 0;
    double sum = 0.0, most = 0.0;
    for (int idx = tid; idx < e * e; idx += NT) {
        const int i = idx / e, j = idx - i * e;
        if (i >= j) continue;
        bool st;
        double v;
        above |= coupling(m.B[i * ES + j], m.B[i * ES + i], m.B[j * ES + j], floor_abs, tau2, st, v);
        steep |= st;
        sum += 2.0 * v * v;
        most = fmax(most, fabs(v));
    }
    if (above) m.f->above = 1;   // every writer stores 1
    if (steep) m.f->steep = 1;
    sum = wave_sum(sum);
    most = wave_max(most);
    if ((tid & 63) == 0) {
        m.red[tid >> 6] = sum;
        m.red[16 + (tid >> 6)] = most;
    }
    __syncthreads();
    Found f = *m.f;
    f.sum = f.most = 0.0;
    for (int w = 0; w < NT / 64; ++w) {
        f.sum += m.red[w];
        f.most = fmax(f.most, m.red[16 + w]);
    }
    __syncthreads();
    return f;
}

// One cyclic Jacobi sweep on the E x E matrix B in LDS (order e), rotations
// accumulated in X.  A round is two barriers and the latency between them: 0.4 us at
// order 45 (0.9 with the pair indices recomputed by every thread).
template <int NT>
__device__ void sweep(const SmallLds<NT>& m, int e, int ES, double floor_abs) {
    const int tid = threadIdx.x;
    double* const B = m.B;
    double* const X = m.X;
    const int N = (e + 1) & ~1, NP = N / 2;
    // thread layout: QW >= NP lanes over Q, PSTEP rows of threads over P
    constexpr int QW = NT == 256 ? 16 : NT == 512 ? 32 : 64, PSTEP = NT / QW;
    constexpr int NQ = NT == 256 ? 1 : NT == 512 ? 2 : 3;
    const int tq = tid % QW, tp = tid / QW;
    for (int r = 0; r < N - 1; ++r) {
        if (tid < NP) {
            int a, b;
            rr_pair(N, r, tid, a, b);
            const double app = B[a * ES + a], aqq = B[b * ES + b], apq = B[a * ES + b];
            const double thr = fmax(0.999 * kRelTol * __builtin_amdgcn_sqrt(fabs(app * aqq)), floor_abs);
            double c = 1.0, s = 0.0;
            if (b < e && fabs(apq) > thr) jacobi_rotation(app, aqq, apq, c, s);
            m.cs[tid] = c;
            m.sn[tid] = s;
            m.pr[tid] = a | (b << 8);
        }
        __syncthreads();
        // 2 x 2 blocks (P, Q) of the round's pairs: a thread keeps its Q, the rows
        // of threads step through P
        if (tq < NP) {
            const double cQ = m.cs[tq], sQ = m.sn[tq];
            const int vQ = m.pr[tq], aQ = vQ & 255, bQ = vQ >> 8;
#pragma unroll
            for (int u = 0; u < NQ; ++u) {
                const int P = tp + u * PSTEP;
                if (P < NP) {
                    const double cP = m.cs[P], sP = m.sn[P];
                    const int vP = m.pr[P], aP = (vP & 255) * ES, bP = (vP >> 8) * ES;
                    const double s_aa = B[aP + aQ], s_ab = B[aP + bQ];
                    const double s_ba = B[bP + aQ], s_bb = B[bP + bQ];
                    const double t_aa = cQ * s_aa - sQ * s_ab, t_ab = sQ * s_aa + cQ * s_ab;
                    const double t_ba = cQ * s_ba - sQ * s_bb, t_bb = sQ * s_ba + cQ * s_bb;
                    B[aP + aQ] = cP * t_aa - sP * t_ba;
                    B[aP + bQ] = cP * t_ab - sP * t_bb;
                    B[bP + aQ] = sP * t_aa + cP * t_ba;
                    B[bP + bQ] = sP * t_ab + cP * t_bb;
                }
            }
            // the eigenvectors: rows i, columns of pair Q
            if (sQ != 0.0) {
#pragma unroll
                for (int u = 0; u < 2 * NQ; ++u) {
                    const int i = tp + u * PSTEP;
                    if (i < e) {
                        const double xa = X[i * ES + aQ], xb = X[i * ES + bQ];
                        X[i * ES + aQ] = cQ * xa - sQ * xb;
                        X[i * ES + bQ] = sQ * xa + cQ * xb;
                    }
                }
            }
        }
        __syncthreads();
    }
}

// X <- X (3 I - X^T X) / 2 (B is scratch) if max |X^T X - I| is at most limit: a step
// maps a deviation d to about 3 d^2 / 4, and moves away from large ones.  Returns the
// deviation (infinity for a NaN), the same in every thread.
template <int NT, int MT>
__device__ double orthonormalise(const SmallLds<NT>& m, int E, int ES, double limit) {
    dbl4 acc[MT];
    mm_regs<NT, MT, true, false>(m.X, m.X, E, ES, acc);
    double dev = 0.0;
    each<NT, MT>(acc, E, [&](int i, int j, double v) {
        const double x = fabs(v - (i == j ? 1.0 : 0.0));
        dev = fmax(dev, x == x ? x : INFINITY);   // fmax would drop the NaN
        m.B[i * ES + j] = (i == j ? 1.5 : 0.0) - 0.5 * v;
    });
    dev = wave_max(dev);
    if ((threadIdx.x & 63) == 0) m.red[threadIdx.x >> 6] = dev;
    __syncthreads();
    for (int w = 0; w < NT / 64; ++w) dev = fmax(dev, m.red[w]);
    if (!(dev <= limit)) {
        __syncthreads();
        return dev;
    }
    mm_regs<NT, MT, false, false>(m.X, m.B, E, ES, acc);
    __syncthreads();
    each<NT, MT>(acc, E, [&](int i, int j, double v) { m.X[i * ES + j] = v; });
    __syncthreads();
    return dev;
}

// B <- X^T B X
template <int NT, int MT>
__device__ void transform(const SmallLds<NT>& m, int E, int ES) {
    dbl4 acc[MT];
    mm_regs<NT, MT, false, false>(m.B, m.X, E, ES, acc);
    __syncthreads();
    each<NT, MT>(acc, E, [&](int i, int j, double v) { m.B[i * ES + j] = v; });
    __syncthreads();
    mm_regs<NT, MT, true, false>(m.X, m.B, E, ES, acc);
    __syncthreads();
    each<NT, MT>(acc, E, [&](int i, int j, double v) { m.B[i * ES + j] = v; });
    __syncthreads();
}

// First-order correction of the eigenvectors (X orthonormal to rounding, B = X^T G X):
// X <- X (I + E), E_ij = -E_ji = b_ij / (b_jj - b_ii), i < j, for the couplings that the
// caller's check counted (Ogita and Aishima 2018 with X^T X = I), orthonormalised.  B is
// left as scratch, its diagonal in m.lam.  False if X was not orthonormal after all.
template <int NT, int MT>
__device__ bool refine(const SmallLds<NT>& m, int E, int ES, double floor_abs, double tau2, double sum) {
    double* const d = m.lam;
    for (int i = threadIdx.x; i < E; i += NT) d[i] = m.B[i * ES + i];
    __syncthreads();
    // One decision a pair, the check's (upper half): the halves of B differ in the last
    // bits, and an entry that only the lower half puts above the tolerance would be
    // divided by a distance nobody has looked at.  E is then skew-symmetric to the bit.
    for (int idx = threadIdx.x; idx < E * E; idx += NT) {
        const int i = idx / E, j = idx - i * E;
        if (i > j) continue;
        bool steep;
        double v = 0.0;
        if (i != j) coupling(m.B[i * ES + j], d[i], d[j], floor_abs, tau2, steep, v);
        m.B[i * ES + j] = v;
        if (i != j) m.B[j * ES + i] = -v;
    }
    __syncthreads();
    dbl4 acc[MT];
    mm_regs<NT, MT, false, false>(m.X, m.B, E, ES, acc);
    __syncthreads();
    each<NT, MT>(acc, E, [&](int i, int j, double v) { m.X[i * ES + j] += v; });
    __syncthreads();
    // (I + E)^T (I + E) = I - E^2 deviates by at most sum = |E|_F^2; a step squares that
    for (double dev = sum; dev > 1e-16; dev *= dev)
        if (!(orthonormalise<NT, MT>(m, E, ES, kStepMax) <= kStepMax)) return false;
    return true;
}

// Gram matrix of the block Y (nr x l) into B: Y Y^T (left) or Y^T Y, operands from
// global memory (16 rows of 8 bytes or strided columns, L2-resident)
template <int NT, int MT>
__device__ void gram(const SmallEig& d, int E, int ES, double* B) {
    const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4, nt = E >> 4;
    const int K = d.left ? d.l : d.nr, e = d.e;
    const long si = d.left ? 1 : d.nr, sk = d.left ? d.nr : 1;   // strides of the Gram index and of k
#pragma nounroll
    for (int u = 0; u < MT; ++u) {
        const int t = (threadIdx.x >> 6) + u * (NT / 64);
        if (t >= nt * nt) continue;
        const int i = (t % nt) * 16 + lr, j = (t / nt) * 16 + lr;
        const double* pi = d.Y + si * (i < e ? i : 0);
        const double* pj = d.Y + si * (j < e ? j : 0);
        const double mi = i < e ? 1.0 : 0.0, mj = j < e ? 1.0 : 0.0;
        dbl4 acc = {0.0, 0.0, 0.0, 0.0};
        int k0 = 0;   // the same in every lane: a matrix instruction needs the whole wave
        for (; k0 + 16 <= K; k0 += 16) {   // four chunks of loads in flight
            double a[4], b[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                a[c] = pi[sk * (k0 + lk + 4 * c)] * mi;
                b[c] = pj[sk * (k0 + lk + 4 * c)] * mj;
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[c], b[c], acc, 0, 0, 0);
        }
        for (; k0 < K; k0 += 4) {
            const int k = k0 + lk;
            const double a = k < K ? pi[sk * k] * mi : 0.0, b = k < K ? pj[sk * k] * mj : 0.0;
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc, 0, 0, 0);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) B[((t % nt) * 16 + lk + 4 * v) * ES + (t / nt) * 16 + lr] = acc[v];
    }
    __syncthreads();
}

// J = P Y (left) or Y P, P in LDS.  Left: Y and J have nr >= e rows (blocks with
// dictionaries of their own share the largest rank as their row count), of which P
// (E x E) covers the first e; the rows beyond are zero.
template <int NT>
__device__ void rebuild(const SmallEig& d, int E, int ES, const double* P) {
    const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4, e = d.e, nr = d.nr, l = d.l;
    const int tr = (nr + 15) >> 4, tc = (l + 15) >> 4;
    for (int t = threadIdx.x >> 6; t < tr * tc; t += NT / 64) {
        const int i0 = (t % tr) * 16, j0 = (t / tr) * 16;
        const int i = i0 + lr, j = j0 + lr;
        dbl4 acc = {0.0, 0.0, 0.0, 0.0};
        for (int k0 = 0; k0 < E; k0 += 4) {
            const int k = k0 + lk;
            double a, b;
            if (d.left) {
                a = i < E ? P[i * ES + k] : 0.0;   // tr * 16 may exceed E
                b = k < e && j < l ? d.Y[k + (long)j * nr] : 0.0;
            } else {
                a = k < e && i < nr ? d.Y[i + (long)k * nr] : 0.0;
                b = P[k * ES + j];   // tc * 16 = E columns
            }
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc, 0, 0, 0);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int r = i0 + lk + 4 * v;
            if (r < nr && j < l) d.J[r + (long)j * nr] = acc[v];
        }
    }
}

// One block's thresholding step from its Gram matrix (see the top of the file)
template <int NT, int MT>
__global__ __launch_bounds__(NT) void k_small_svt(const SmallEig* __restrict__ descs, BlockState bs,
                                                   const DevIter* __restrict__ it, int max_sweeps) {
    extern __shared__ double lds[];
    const SmallEig d = descs[blockIdx.x];
    if (!d.run[0]) return;
    const int e = d.e, E = (e + 15) & ~15, ES = E + 1, tid = threadIdx.x;
    const long L = d.L;
    const SmallLds<NT> m(lds, E);
    double* const B = m.B;
    double* const X = m.X;
    bool warm = d.warm[0] != 0;
    dbl4 acc[MT];
    auto load_gram = [&] {
        for (int idx = tid; idx < E * E; idx += NT) {
            const int j = idx / E, i = idx - j * E;
            B[i * ES + j] = (i < e && j < e) ? d.G[i + j * L] : 0.0;
        }
        __syncthreads();
    };
    auto identity = [&] {
        for (int idx = tid; idx < E * E; idx += NT) {
            const int j = idx / E, i = idx - j * E;
            X[i * ES + j] = i == j ? 1.0 : 0.0;
        }
        __syncthreads();
    };
    for (int idx = tid; idx < E * E; idx += NT) {
        const int j = idx / E, i = idx - j * E;
        X[i * ES + j] = (warm && i < e && j < e) ? d.X[i + j * L] : (i == j ? 1.0 : 0.0);
    }
    __syncthreads();
    // earlier eigenvectors that are no longer orthonormal (of a step that met an overflow,
    // say) would make X^T G X something else than a similarity: from the identity then
    if (warm && !(orthonormalise<NT, MT>(m, E, ES, kWarmMax) <= kWarmMax)) {
        identity();
        warm = false;
    }
    if (d.Y) {
        // the Gram matrix as well (short rows or columns), kept for the refinement
        gram<NT, MT>(d, E, ES, B);
        for (int idx = tid; idx < e * e; idx += NT) {
            const int j = idx / e, i = idx - j * e;
            d.G[i + j * L] = B[i * ES + j];
        }
        __threadfence_block();
        __syncthreads();
    } else {
        load_gram();
    }
    if (warm) transform<NT, MT>(m, E, ES);
    // Corrections where they resolve everything that is left (6 products, about a
    // quarter of a sweep's time at order 45), a Jacobi sweep otherwise
    const double floor_abs = kAbsFloor * diag_max(m, e, ES), tau = it->tau, tau2 = tau * tau;
    int left = max_sweeps;
    bool linear = true;       // corrections are still tried
    bool fresh = true;        // B is X^T G X, not the sweeps' own update of it
    bool lam_saved = false;   // the eigenvalues are in m.lam, no longer in B
    for (int step = 0; step < 4 * max_sweeps && left > 0; ++step) {
        const Found f = check(m, e, ES, floor_abs, tau2);
        const bool below = !f.above;  // only couplings below the floor are left: one correction of
                                      // them is the last step (the next would meet rounding)
        if (below && (f.most <= kDone || !linear || f.sum > kSumMax)) break;
        if (below && !fresh) {
            load_gram();
            transform<NT, MT>(m, E, ES);
            fresh = true;
        } else if (linear && !f.steep && f.sum <= kSumMax && step < 2 * max_sweeps) {
            linear = refine<NT, MT>(m, E, ES, floor_abs, tau2, f.sum);
            if (linear && below) {
                lam_saved = true;
                break;
            }
            if (!linear) identity();
            load_gram();
            if (linear) transform<NT, MT>(m, E, ES);
            fresh = true;
        } else if (f.above) {
            sweep(m, e, ES, floor_abs);
            --left;
            fresh = false;
        } else {
            break;
        }
    }
    // weights g = (1 - tau / sigma)_+, eigenvectors back, then B = X diag(g)
    int* const flag = m.pr;
    if (tid == 0) *flag = 0;
    if (!lam_saved)
        for (int i = tid; i < E; i += NT) m.lam[i] = i < e ? B[i * ES + i] : 0.0;
    __syncthreads();
    int kept = 0;
    for (int i = tid; i < L; i += NT) {
        const double lam = i < e ? m.lam[i] : 0.0, sig = sqrt(fmax(lam, 0.0));
        const bool keep = sig > tau;
        d.lam[i] = lam;
        d.h[i] = keep ? 1.0 / sig : 0.0;
        kept += keep;
    }
    if (kept) atomicAdd(flag, kept);
    for (int idx = tid; idx < e * e; idx += NT) {
        const int j = idx / e, i = idx - j * e;
        d.X[i + j * L] = X[i * ES + j];
    }
    double* g = m.cs;   // cs and sn are free now: E <= 96 weights
    for (int j = tid; j < E; j += NT) {
        const double sig = j < e ? sqrt(fmax(m.lam[j], 0.0)) : 0.0;
        g[j] = sig > tau ? 1.0 - tau / sig : 0.0;
    }
    __syncthreads();
    for (int idx = tid; idx < E * E; idx += NT) {
        const int i = idx / E, j = idx - i * E;
        B[i * ES + j] = X[i * ES + j] * g[j];
    }
    __syncthreads();
    mm_regs<NT, MT, false, true>(B, X, E, ES, acc);
    if (d.Y) {
        __syncthreads();
        each<NT, MT>(acc, E, [&](int i, int j, double v) { B[i * ES + j] = v; });   // P
        __syncthreads();
        rebuild<NT>(d, E, ES, B);
    } else {
        each<NT, MT>(acc, E, [&](int i, int j, double v) {
            if (i < e && j < e) d.P[i + j * L] = v;
        });
    }
    if (tid == 0) {
        bs.rank[d.block] = *flag;
        d.warm[0] = 1;
    }
}

// Cold eigen-decomposition of one matrix A (order e, ld L): eigenvalues into lam
// (zero beyond e), eigenvectors into W (ld L, identity beyond e)
template <int NT, int MT>
__global__ __launch_bounds__(NT) void k_small_syev(const double* __restrict__ A, double* __restrict__ W,
                                                    double* __restrict__ lam, int e, int L, int max_sweeps,
                                                    double floor_rel) {
    extern __shared__ double lds[];
    const int E = (e + 15) & ~15, ES = E + 1, tid = threadIdx.x;
    const SmallLds<NT> m(lds, E);
    double* const B = m.B;
    double* const X = m.X;
    for (int idx = tid; idx < E * E; idx += NT) {
        const int j = idx / E, i = idx - j * E;
        B[i * ES + j] = (i < e && j < e) ? A[i + (long)j * L] : 0.0;
        X[i * ES + j] = i == j ? 1.0 : 0.0;
    }
    __syncthreads();
    const double floor_abs = floor_rel * diag_max(m, e, ES);
    for (int sw = 0; sw < max_sweeps && check(m, e, ES, floor_abs, INFINITY).above; ++sw) sweep(m, e, ES, floor_abs);
    __syncthreads();
    for (int i = tid; i < L; i += NT) lam[i] = i < e ? B[i * ES + i] : 0.0;
    for (long idx = tid; idx < (long)L * L; idx += NT) {
        const int j = (int)(idx / L), i = (int)(idx - (long)j * L);
        W[idx] = (i < e && j < e) ? X[i * ES + j] : (i == j ? 1.0 : 0.0);
    }
}

size_t lds_bytes(int e) {
    const int E = (e + 15) & ~15;
    return sizeof(double) * (2 * (size_t)E * (E + 1) + kSmallTail);
}

template <class K>
void allow_lds(K* kernel, size_t bytes) {
    LRR_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)bytes));
}

}  // namespace

void small_eig_prepare(void) {
    allow_lds(&k_small_svt<1024, 3>, lds_bytes(kSmallEig));
    allow_lds(&k_small_syev<1024, 3>, lds_bytes(kSmallEig));
}

// 4, 8 or 16 waves: the largest tile count a wave multiplies is 1, 2 and 3
void launch_small_svt(const SmallEig* d, int count, int maxe, BlockState bs, const DevIter* it, int max_sweeps,
                      hipStream_t s) {
    const size_t lds = lds_bytes(maxe);
    if (maxe <= 32) hipLaunchKernelGGL((k_small_svt<256, 1>), dim3(count), dim3(256), lds, s, d, bs, it, max_sweeps);
    else if (maxe <= 64)
        hipLaunchKernelGGL((k_small_svt<512, 2>), dim3(count), dim3(512), lds, s, d, bs, it, max_sweeps);
    else hipLaunchKernelGGL((k_small_svt<1024, 3>), dim3(count), dim3(1024), lds, s, d, bs, it, max_sweeps);
}
void launch_small_syev(const double* A, double* W, double* lam, int e, int L, int max_sweeps, bool floor,
                       hipStream_t s) {
    const size_t lds = lds_bytes(e);
    const double fl = floor ? kAbsFloor : 0.0;
    if (e <= 32) hipLaunchKernelGGL((k_small_syev<256, 1>), dim3(1), dim3(256), lds, s, A, W, lam, e, L,
                                       max_sweeps, fl);
    else if (e <= 64)
        hipLaunchKernelGGL((k_small_syev<512, 2>), dim3(1), dim3(512), lds, s, A, W, lam, e, L,
                                       max_sweeps, fl);
    else hipLaunchKernelGGL((k_small_syev<1024, 3>), dim3(1), dim3(1024), lds, s, A, W, lam, e, L,
                                       max_sweeps, fl);
}

}  // namespace lrr
