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
//   B = X^T G X, cyclic Jacobi sweeps on B until nothing exceeds the tolerance of
//   jacobi.hip, X <- X R,  weights from the eigenvalues,  P = X diag(g) X^T.
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

// Jacobi sweeps on the E x E matrix B in LDS (order e), rotations accumulated in X.
// Returns after a check that finds no entry above the tolerance (relative to the
// two diagonal entries, and floor_rel of the largest one), or max_sweeps.  A round
// is two barriers and the latency between them: 0.4 us at order 45 (0.9 with the
// pair indices recomputed by every thread).
template <int NT>
__device__ void sweeps(double* B, double* X, double* cs, double* sn, int* flag, int e, int E, int ES, int max_sweeps,
                       double floor_rel = kAbsFloor) {
    const int tid = threadIdx.x;
    __shared__ double red[16];
    double mx = 0.0;
    for (int i = tid; i < e; i += NT) mx = fmax(mx, fabs(B[i * ES + i]));
    mx = wave_max(mx);
    if ((tid & 63) == 0) red[tid >> 6] = mx;
    __syncthreads();
    for (int w = 0; w < NT / 64; ++w) mx = fmax(mx, red[w]);
    const double floor_abs = floor_rel * mx;
    const int N = (e + 1) & ~1, NP = N / 2;
    // thread layout: QW >= NP lanes over Q, PSTEP rows of threads over P
    constexpr int QW = NT == 256 ? 16 : NT == 512 ? 32 : 64, PSTEP = NT / QW, NQ = QW / PSTEP > 1 ? (NT == 1024 ? 3 : QW / PSTEP) : 1;
    const int tq = tid % QW, tp = tid / QW;
    int* pr = flag + 2;
    for (int sw = 0; sw < max_sweeps; ++sw) {
        if (tid == 0) *flag = 0;
        __syncthreads();
        int any = 0;
        for (int idx = tid; idx < e * e; idx += NT) {
            const int i = idx / e, j = idx - i * e;
            if (i < j && fabs(B[i * ES + j]) > fmax(kRelTol * sqrt(fabs(B[i * ES + i] * B[j * ES + j])), floor_abs))
                any = 1;
        }
        if (any) *flag = 1;   // every writer stores 1
        __syncthreads();
        if (*flag == 0) break;
        for (int r = 0; r < N - 1; ++r) {
            if (tid < NP) {
                int a, b;
                rr_pair(N, r, tid, a, b);
                const double app = B[a * ES + a], aqq = B[b * ES + b], apq = B[a * ES + b];
                const double thr = fmax(0.999 * kRelTol * __builtin_amdgcn_sqrt(fabs(app * aqq)), floor_abs);
                double c = 1.0, s = 0.0;
                if (b < e && fabs(apq) > thr) jacobi_rotation(app, aqq, apq, c, s);
                cs[tid] = c;
                sn[tid] = s;
                pr[tid] = a | (b << 8);
            }
            __syncthreads();
            // 2 x 2 blocks (P, Q) of the round's pairs: a thread keeps its Q, the rows
            // of threads step through P
            if (tq < NP) {
                const double cQ = cs[tq], sQ = sn[tq];
                const int vQ = pr[tq], aQ = vQ & 255, bQ = vQ >> 8;
#pragma unroll
                for (int u = 0; u < NQ; ++u) {
                    const int P = tp + u * PSTEP;
                    if (P < NP) {
                        const double cP = cs[P], sP = sn[P];
                        const int vP = pr[P], aP = (vP & 255) * ES, bP = (vP >> 8) * ES;
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
    __syncthreads();
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
    double* B = lds;
    double* X = lds + E * ES;
    double* cs = X + E * ES;
    double* sn = cs + 48;
    int* flag = reinterpret_cast<int*>(sn + 48);
    const bool warm = d.warm[0] != 0;
    dbl4 acc[MT];
    for (int idx = tid; idx < E * E; idx += NT) {
        const int j = idx / E, i = idx - j * E;
        X[i * ES + j] = (warm && i < e && j < e) ? d.X[i + j * L] : (i == j ? 1.0 : 0.0);
    }
    __syncthreads();
    if (warm) {
        mm_regs<NT, MT, true, false>(X, X, E, ES, acc);
        each<NT, MT>(acc, E, [&](int i, int j, double v) { B[i * ES + j] = (i == j ? 1.5 : 0.0) - 0.5 * v; });
        __syncthreads();
        mm_regs<NT, MT, false, false>(X, B, E, ES, acc);
        __syncthreads();
        each<NT, MT>(acc, E, [&](int i, int j, double v) { X[i * ES + j] = v; });
    }
    __syncthreads();
    for (int idx = tid; idx < E * E; idx += NT) {
        const int j = idx / E, i = idx - j * E;
        B[i * ES + j] = (i < e && j < e) ? d.G[i + j * L] : 0.0;
    }
    __syncthreads();
    if (warm) {
        mm_regs<NT, MT, false, false>(B, X, E, ES, acc);
        __syncthreads();
        each<NT, MT>(acc, E, [&](int i, int j, double v) { B[i * ES + j] = v; });
        __syncthreads();
        mm_regs<NT, MT, true, false>(X, B, E, ES, acc);
        __syncthreads();
        each<NT, MT>(acc, E, [&](int i, int j, double v) { B[i * ES + j] = v; });
        __syncthreads();
    }
    sweeps<NT>(B, X, cs, sn, flag, e, E, ES, max_sweeps);
    // weights g = (1 - tau / sigma)_+, eigenvectors back, then B = X diag(g)
    const double tau = it->tau;
    if (tid == 0) *flag = 0;
    __syncthreads();
    int kept = 0;
    for (int i = tid; i < L; i += NT) {
        const double lam = i < e ? B[i * ES + i] : 0.0, sig = sqrt(fmax(lam, 0.0));
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
    double* g = cs;   // cs and sn are free now: E <= 96 weights
    for (int j = tid; j < E; j += NT) {
        const double sig = j < e ? sqrt(fmax(B[j * ES + j], 0.0)) : 0.0;
        g[j] = sig > tau ? 1.0 - tau / sig : 0.0;
    }
    __syncthreads();
    for (int idx = tid; idx < E * E; idx += NT) {
        const int i = idx / E, j = idx - i * E;
        B[i * ES + j] = X[i * ES + j] * g[j];
    }
    __syncthreads();
    mm_regs<NT, MT, false, true>(B, X, E, ES, acc);
    each<NT, MT>(acc, E, [&](int i, int j, double v) {
        if (i < e && j < e) d.P[i + j * L] = v;
    });
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
    double* B = lds;
    double* X = lds + E * ES;
    double* cs = X + E * ES;
    double* sn = cs + 48;
    int* flag = reinterpret_cast<int*>(sn + 48);
    for (int idx = tid; idx < E * E; idx += NT) {
        const int j = idx / E, i = idx - j * E;
        B[i * ES + j] = (i < e && j < e) ? A[i + (long)j * L] : 0.0;
        X[i * ES + j] = i == j ? 1.0 : 0.0;
    }
    __syncthreads();
    sweeps<NT>(B, X, cs, sn, flag, e, E, ES, max_sweeps, floor_rel);
    for (int i = tid; i < L; i += NT) lam[i] = i < e ? B[i * ES + i] : 0.0;
    for (long idx = tid; idx < (long)L * L; idx += NT) {
        const int j = (int)(idx / L), i = (int)(idx - (long)j * L);
        W[idx] = (i < e && j < e) ? X[i * ES + j] : (i == j ? 1.0 : 0.0);
    }
}

size_t lds_bytes(int e) {
    const int E = (e + 15) & ~15;
    return sizeof(double) * (2 * (size_t)E * (E + 1) + 96 + 2 + 24);
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
