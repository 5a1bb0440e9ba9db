// Batched two-sided block-Jacobi eigensolver for symmetric FP64 matrices.
//
// This is the "small dense SVD in FP64" of the singular-value thresholding
// step: the SVT of a block Y (n x l) needs the eigen-decomposition of its Gram
// matrix Y^T Y (l x l).  Several matrices (one per DFC block, of different
// orders) are processed by the same launches.
//
// A matrix of padded order L is cut into nb = L / BS blocks of BS indices.  One
// sweep has nb - 1 rounds; in a round the blocks are paired by the circle
// method and every pair (p, q) is handled in two phases, a launch each, or phase B
// of a round and phase A of the next in one launch (k_jacobi_step):
//   phase A  one workgroup per pair applies parallel-Jacobi rotations to the
//            2BS x 2BS sub-matrix B[p u q, p u q] in LDS (every coupling between
//            the two blocks once, those inside them in some of the rounds) and
//            writes the accumulated rotation R_pq (2BS x 2BS);
//   phase B  every tile pair (P, Q), P <= Q, of the round is replaced by
//            R_P^T B[P, Q] R_Q (and its transpose), and the eigenvector
//            accumulator gets W[:, P] <- W[:, P] R_P; the 2BS-square products
//            run on the FP64 matrix cores out of LDS.
// Rounds come from the circle method (a full sweep) or, when the check found
// couplings in only a few index-block pairs, from a host-built schedule of
// perfect matchings that covers just those pairs (EigDesc::sched).
// Pairs of indices whose Gershgorin discs both lie below tau^2 are never
// rotated: the thresholding step discards every eigenvalue of that cluster, so
// only the subspace it spans matters, not a basis of it.
// Convergence: an off-diagonal entry needs a rotation when
// |b_pq| > max(1e-15 sqrt(|b_pp b_qq|), 1e-14 max|diag B|).  The absolute floor
// sits at the rounding level of the matrix: a Gram matrix of a rank-deficient
// block has exactly-zero eigenvalues whose coupling entries are pure rounding
// noise, and rotating them only regenerates noise.  Before each sweep one
// launch checks every off-diagonal entry; pairs whose sub-matrix is already
// diagonal skip their work, and so do the tiles they touch.
#include "common.hpp"
#include "jacobi_rot.hpp"
#include "kernels.hpp"

namespace lrr {

namespace {

constexpr double kRelTol = 1e-15;
constexpr double kAbsFloor = 1e-14;
constexpr int kPairThreads = 512;  // half of them update S, half rotate R

// blocks (p, q) of slot P in a round: the circle method, or the explicit schedule
__device__ __forceinline__ void round_pair(const EigDesc& d, int nb, int round, int P, int sched, int& p, int& q) {
    if (sched) {
        const int v = d.sched[round * (nb / 2) + P];
        p = v & 0xffff;
        q = v >> 16;
    } else {
        rr_pair(nb, round, P, p, q);
    }
}

// LDS of one pair solve.  Row stride PB + 8: the four rows that a wave's 2 x 2
// blocks touch start 8 bank pairs apart, and the diagonal entries fall into
// different ones.
template <int BS>
struct PairLds {
    static constexpr int PB = 2 * BS;
    static constexpr int NBUF = BS == 16 ? 2 : 1;   // 32-wide blocks would not fit twice
    double S[NBUF][PB][PB + 8];
    double R[PB][PB + 1];
    double c[2][BS], s[2][BS];   // rotations of two consecutive steps (SPLIT)
    unsigned long long lo;   // bit i: index i lies below the cut
    int any;                 // 1: a coupling between the two index blocks, 2: inside one
};

// Indices (a < b) of rotation k in step st of a pair solve: steps 0..BS-2 pair the
// indices inside each of the two blocks (circle method, k < BS/2 in the first),
// steps BS-1..2BS-2 pair index k of the first with one of the second.
template <int BS>
__device__ __forceinline__ void step_pair(int st, int k, int& a, int& b) {
    if (st >= BS - 1) {
        a = k;
        b = BS + ((k + st - (BS - 1)) & (BS - 1));
    } else {
        const int o = k < BS / 2 ? 0 : BS;
        rr_pair(BS, st, k & (BS / 2 - 1), a, b);
        a += o;
        b += o;
    }
}

// Phase A for slot P of a round, by the NT threads of a workgroup: one cyclic
// sweep over the couplings between the two index blocks (BS steps) and, in every
// eighth round and in targeted rounds, first over those inside each block (BS - 1
// steps), on the 2BS x 2BS sub-matrix in LDS; the rotation goes to R_P.  Rotating
// inside the blocks in every round, as a full cyclic sweep of the sub-matrix
// does, costs 31 steps instead of 16 and saves no outer sweep (12 from the
// identity at order 512 either way; with it only once per sweep, up to 12 instead
// of 10 at order 208).
// A step is bound by its chain of dependent instructions, not by throughput:
// every lane computes the rotation of pair lane % BS itself (no hand-over through
// LDS), the 2 x 2 block's row rotation comes from another lane, and S alternates
// between two buffers, so that a step has one barrier.  Together with the cheaper
// rotation: 32.7 -> about 15 us a launch (64 pair solves, 4 matrices of order
// 512); a solve with m = 500, n = 2000, t = 4 465 -> 354 ms, plain LRR of 200
// points 352 -> 252 ms.
// wslot spreads the operation counter over its slots.  Every thread returns
// through the same path (the branches depend on LDS values only).
// set: which set of rotation blocks and flags takes the result.  loaded: S is in
// sm.S[0] already (k_jacobi_step); otherwise it is read from B.
template <int BS, int NT>
__device__ void pair_solve(const EigDesc& d, int round, int P, int sched, int wslot, PairLds<BS>& sm, int set = 0,
                           bool loaded = false) {
    constexpr int PB = 2 * BS;
    constexpr int NP = PB / 2;   // rotations per step
    constexpr int NBUF = PairLds<BS>::NBUF;
    constexpr bool SPLIT = NT >= 2 * NP * NP;      // separate waves for S and R
    constexpr int NS = SPLIT ? NP * NP : NT;       // threads on S
    constexpr int NR = SPLIT ? NT - NS : NT;       // threads on R
    static_assert(!SPLIT || NBUF == 2, "the waves on R meet one barrier a step");
    static_assert(64 % NP == 0 && NS % 64 == 0 && (NP * NP) % NS == 0 && (PB * NP) % NR == 0, "thread layout");
    constexpr int IS = NP * NP / NS, IR = PB * NP / NR;
    const int nb = d.L / BS;
    int p, q;
    round_pair(d, nb, round, P, sched, p, q);

    const int tid = threadIdx.x, lane = tid & 63;
    const long L = d.L;
    // every global load is issued before the first use
    constexpr int NV = PB * PB / NT;
    double v[NV];
#pragma unroll
    for (int u = 0; u < NV; ++u) {
        const int idx = tid + u * NT;
        const int i = idx % PB, j = idx / PB;
        const long gi = (i < BS) ? (long)p * BS + i : (long)q * BS + (i - BS);
        const long gj = (j < BS) ? (long)p * BS + j : (long)q * BS + (j - BS);
        v[u] = loaded ? sm.S[0][i][j] : d.B[gi + gj * L];
    }
    const int lo_i = tid < PB ? d.lo[(tid < BS) ? p * BS + tid : q * BS + (tid - BS)] : 0;
    const double floor_abs = kAbsFloor * d.scale[0];
#pragma unroll
    for (int u = 0; u < NV; ++u) {
        const int idx = tid + u * NT;
        const int i = idx % PB, j = idx / PB;
        if (!loaded) sm.S[0][i][j] = v[u];
        sm.R[i][j] = (i == j) ? 1.0 : 0.0;
    }
    if (tid < 64) {
        const unsigned long long m = __ballot(lo_i != 0);
        if (tid == 0) {
            sm.lo = m;
            sm.any = 0;
        }
    }
    __syncthreads();
    const unsigned long long lo = sm.lo;
    // parallel convergence test of the whole sub-matrix
#pragma unroll
    for (int u = 0; u < NV; ++u) {
        const int idx = tid + u * NT;
        const int i = idx % PB, j = idx / PB;
        if (i < j && !((lo >> i) & (lo >> j) & 1ull) &&
            fabs(v[u]) > fmax(kRelTol * sqrt(fabs(sm.S[0][i][i] * sm.S[0][j][j])), floor_abs))
            atomicOr(&sm.any, (i < BS) == (j < BS) ? 2 : 1);
    }
    __syncthreads();
    const int any = sm.any;
    const bool inside = (any & 2) && (sched || (round & 7) == 0), cross = (any & 1) != 0;
    int* const prot = d.prot + set * (nb / 2);
    if (!inside && !cross) {
        if (tid == 0) prot[P] = 0;
        return;
    }
    const int st0 = inside ? 0 : BS - 1, st1 = cross ? 2 * BS - 1 : BS - 1;
    const int k = lane % NP;
    int cur = 0;
    // With separate waves the rotations of R follow one step behind those of S, from
    // LDS: the waves on R then compute no rotations of their own (the redundant ones
    // of every wave on S already fill half of a SIMD's issue slots).
    auto rotate_R = [&](int st) {
        int aQ, bQ;
        step_pair<BS>(st, k, aQ, bQ);
        const double c = sm.c[st & 1][k], s = sm.s[st & 1][k];
#pragma unroll
        for (int u = 0; u < IR; ++u) {
            const int i = (tid - NS + u * NR) / NP;
            const double ra = sm.R[i][aQ], rb = sm.R[i][bQ];
            sm.R[i][aQ] = c * ra - s * rb;
            sm.R[i][bQ] = s * ra + c * rb;
        }
    };
    for (int st = st0; st < st1; ++st) {
        if (SPLIT && tid >= NS) {
            if (st > st0) rotate_R(st - 1);
            __syncthreads();
            if (NBUF == 2) cur ^= 1;
            continue;
        }
        auto& S = sm.S[cur];
        auto& Sn = sm.S[NBUF == 2 ? cur ^ 1 : 0];
        int aQ, bQ;
        step_pair<BS>(st, k, aQ, bQ);
        double c = 1.0, s = 0.0;
        {
            const double app = S[aQ][aQ], aqq = S[bQ][bQ], apq = S[aQ][bQ];
            // a little below the check's threshold, so that what it marks is rotated
            // in spite of the approximate square root
            const double thr =
                fmax(0.999 * kRelTol * __builtin_amdgcn_sqrt(fabs(app * aqq)), floor_abs);
            double cr, sr;
            jacobi_rotation(app, aqq, apq, cr, sr);
            if (!((lo >> aQ) & (lo >> bQ) & 1ull) && fabs(apq) > thr) {
                c = cr;
                s = sr;
            }
        }
        if (SPLIT && tid < NP) {
            sm.c[st & 1][k] = c;
            sm.s[st & 1][k] = s;
        }
        double w[IS][4];
        // the sub-matrix: (P2, Q2) blocks of the step's 2 x 2 index pairs
        {
#pragma unroll
            for (int u = 0; u < IS; ++u) {
                const int P2 = (tid + u * NS) / NP;
                int aP, bP;
                step_pair<BS>(st, P2, aP, bP);
                const double cP = __shfl(c, P2, 64), sP = __shfl(s, P2, 64);
                const double s_aa = S[aP][aQ], s_ab = S[aP][bQ];
                const double s_ba = S[bP][aQ], s_bb = S[bP][bQ];
                // columns: T = S G_Q
                const double t_aa = c * s_aa - s * s_ab, t_ab = s * s_aa + c * s_ab;
                const double t_ba = c * s_ba - s * s_bb, t_bb = s * s_ba + c * s_bb;
                // rows: S' = G_P^T T
                w[u][0] = cP * t_aa - sP * t_ba;
                w[u][1] = cP * t_ab - sP * t_bb;
                w[u][2] = sP * t_aa + cP * t_ba;
                w[u][3] = sP * t_ab + cP * t_bb;
            }
        }
        if (NBUF == 1) __syncthreads();   // one buffer: every read before the first write
        {
#pragma unroll
            for (int u = 0; u < IS; ++u) {
                const int P2 = (tid + u * NS) / NP;
                int aP, bP;
                step_pair<BS>(st, P2, aP, bP);
                Sn[aP][aQ] = w[u][0];
                Sn[aP][bQ] = w[u][1];
                Sn[bP][aQ] = w[u][2];
                Sn[bP][bQ] = w[u][3];
            }
        }
        // the accumulated rotation: row i, columns of pair Q2
        if (!SPLIT) {
#pragma unroll
            for (int u = 0; u < IR; ++u) {
                const int i = (tid + u * NR) / NP;
                const double ra = sm.R[i][aQ], rb = sm.R[i][bQ];
                sm.R[i][aQ] = c * ra - s * rb;
                sm.R[i][bQ] = s * ra + c * rb;
            }
        }
        __syncthreads();
        if (NBUF == 2) cur ^= 1;
    }
    if (SPLIT) {
        if (tid >= NS) rotate_R(st1 - 1);
        __syncthreads();
    }
    if (tid == 0 && d.work) {
        // per step: NP angles (~30 operations), NP^2 2x2 updates (24), PB*NP rotations of R (6)
        const unsigned long long per_step = 30ull * NP + 24ull * NP * NP + 6ull * PB * NP;
        atomicAdd(&d.work[work_slot(0, wslot)], per_step * (st1 - st0));
    }
    double* Rg = d.R + (long)(set * (nb / 2) + P) * PB * PB;
#pragma unroll
    for (int u = 0; u < NV; ++u) {
        const int idx = tid + u * NT;
        const int i = idx % PB, j = idx / PB;
        Rg[i + (long)j * PB] = sm.R[i][j];
    }
    if (tid == 0) prot[P] = 1;
}

template <int BS, int NT>
__global__ __launch_bounds__(NT) void k_jacobi_pairs(const EigDesc* __restrict__ descs, int round, int sched) {
    const EigDesc d = descs[blockIdx.y];
    if (d.run[0] == 0 || d.st[0] != 0) return;
    const int nb = d.L / BS;
    const int P = blockIdx.x;
    if (P >= nb / 2 || round >= nb - 1) return;
    __shared__ PairLds<BS> sm;
    pair_solve<BS, NT>(d, round, P, sched, blockIdx.x + blockIdx.y * gridDim.x, sm);
}

// C (PB x PB, into LDS) = op(A) B for PB x PB operands in LDS (row stride PB + 1),
// on the FP64 matrix cores: the (PB/16)^2 output tiles of 16 x 16 are spread over
// the four waves, each a chain of PB/4 v_mfma_f64_16x16x4f64 (register v of a
// lane holds row lane/16 + 4v, column lane%16 of its tile).  TA: op(A) = A^T.
template <int PB, bool TA>
__device__ __forceinline__ void mm_lds(const double (*A)[PB + 1], const double (*B)[PB + 1], double (*C)[PB + 1],
                                       int tid) {
    constexpr int NTILE = PB / 16;
    const int wave = tid >> 6, lane = tid & 63;
    const int lr = lane & 15, lk = lane >> 4;
    for (int t = wave; t < NTILE * NTILE; t += 4) {
        const int ti = (t % NTILE) * 16, tj = (t / NTILE) * 16;
        dbl4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int kk = 0; kk < PB; kk += 4) {
            const int k = kk + lk;
            const double a = TA ? A[k][ti + lr] : A[ti + lr][k];
            const double b = B[k][tj + lr];
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc, 0, 0, 0);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) C[ti + lk + 4 * v][tj + lr] = acc[v];
    }
}

// LDS of one phase-B item
template <int BS>
struct ApplyLds {
    static constexpr int PB = 2 * BS;
    double X[PB][PB + 1];
    double RP[PB][PB + 1];
    double RQ[PB][PB + 1];
    double T[PB][PB + 1];
};

constexpr int kApplyRows = 64;   // rows of W per phase-B item

template <int BS>
__device__ __forceinline__ int apply_items(int L) {
    const int npair = L / BS / 2;
    return npair * (npair + 1) / 2 + ((L + kApplyRows - 1) / kApplyRows) * npair;
}

// phase B, item `item` of a round (256 threads, tid): a tile pair of B, read from
// src and written to dst (the same buffer, or the other one), or a row chunk of W.
// set: the round's set of rotation blocks and flags.  Two groups of 256 threads of
// one workgroup may each run an item of the same kind: every group meets the same
// barriers, whatever its item needs.
template <int BS>
__device__ void apply_item(const EigDesc& d, int round, int item, int sched, int wslot, ApplyLds<BS>& sm,
                           const double* src, double* dst, int set, int tid, bool live) {
    constexpr int PB = 2 * BS;
    constexpr int RC = kApplyRows;
    const int nb = d.L / BS;
    const int npair = nb / 2;
    const int ntri = npair * (npair + 1) / 2;
    auto& X = sm.X;
    auto& RP = sm.RP;
    auto& RQ = sm.RQ;
    auto& T = sm.T;
    const long L = d.L;
    const int* const prot = d.prot + set * npair;
    const double* const Rset = d.R + (long)set * npair * PB * PB;

    if (item < ntri) {
        // decode upper-triangular index (P <= Q)
        int P = 0, rem = item;
        while (rem >= npair - P) { rem -= npair - P; ++P; }
        const int Q = P + rem;
        const bool rotP = prot[P] != 0, rotQ = prot[Q] != 0, any = rotP || rotQ;
        live = live && (any || src != dst);
        if (live && any && tid == 0 && d.work)   // two PB^3 products
            atomicAdd(&d.work[work_slot(1, wslot)], 4ull * PB * PB * PB);
        int p1, q1, p2, q2;
        round_pair(d, nb, round, P, sched, p1, q1);
        round_pair(d, nb, round, Q, sched, p2, q2);
        const double* RgP = Rset + (long)P * PB * PB;
        const double* RgQ = Rset + (long)Q * PB * PB;
        if (live)
            for (int idx = tid; idx < PB * PB; idx += 256) {
                const int i = idx % PB, j = idx / PB;
                const long gi = (i < BS) ? (long)p1 * BS + i : (long)q1 * BS + (i - BS);
                const long gj = (j < BS) ? (long)p2 * BS + j : (long)q2 * BS + (j - BS);
                X[i][j] = src[gi + gj * L];
                // a pair that did not rotate has R = I (its R block was not written)
                RP[i][j] = rotP ? RgP[i + (long)j * PB] : (i == j ? 1.0 : 0.0);
                RQ[i][j] = rotQ ? RgQ[i + (long)j * PB] : (i == j ? 1.0 : 0.0);
            }
        __syncthreads();
        if (live && any) mm_lds<PB, false>(X, RQ, T, tid);       // T = X R_Q
        __syncthreads();
        if (live && any) mm_lds<PB, true>(RP, T, X, tid);        // X = R_P^T T (X is free after the first product)
        __syncthreads();
        if (!live) return;
        for (int idx = tid; idx < PB * PB; idx += 256) {
            const int i = idx % PB, j = idx / PB;
            const long gi = (i < BS) ? (long)p1 * BS + i : (long)q1 * BS + (i - BS);
            const long gj = (j < BS) ? (long)p2 * BS + j : (long)q2 * BS + (j - BS);
            dst[gi + gj * L] = X[i][j];
        }
        if (P != Q) {
            // the mirrored tile, with consecutive threads on consecutive rows of it; a tile
            // that did not rotate keeps its own (its halves can differ in the last bits)
            for (int idx = tid; idx < PB * PB; idx += 256) {
                const int j = idx % PB, i = idx / PB;
                const long gi = (i < BS) ? (long)p1 * BS + i : (long)q1 * BS + (i - BS);
                const long gj = (j < BS) ? (long)p2 * BS + j : (long)q2 * BS + (j - BS);
                dst[gj + gi * L] = any ? X[i][j] : src[gj + gi * L];
            }
        }
    } else {
        const int w = item - ntri;
        const int P = w % npair, chunk = w / npair;
        live = live && prot[P] != 0;
        if (live && tid == 0 && d.work)   // RC x PB times PB x PB
            atomicAdd(&d.work[work_slot(1, wslot)], 2ull * RC * PB * PB);
        int p1, q1;
        round_pair(d, nb, round, P, sched, p1, q1);
        const double* RgP = Rset + (long)P * PB * PB;
        const int r0 = chunk * RC;
        // reuse X as a RC x PB panel when RC <= PB, else loop in pieces of PB rows
        for (int rr = 0; rr < RC; rr += PB) {
            if (live)
                for (int idx = tid; idx < PB * PB; idx += 256) {
                    const int i = idx % PB, j = idx / PB;
                    const long gi = r0 + rr + i;
                    const long gj = (j < BS) ? (long)p1 * BS + j : (long)q1 * BS + (j - BS);
                    X[i][j] = (gi < L) ? d.W[gi + gj * L] : 0.0;
                    if (rr == 0) RP[i][j] = RgP[i + (long)j * PB];
                }
            __syncthreads();
            if (live) mm_lds<PB, false>(X, RP, T, tid);   // T = W panel R_P
            __syncthreads();
            if (live)
                for (int idx = tid; idx < PB * PB; idx += 256) {
                    const int i = idx % PB, j = idx / PB;
                    const long gi = r0 + rr + i;
                    const long gj = (j < BS) ? (long)p1 * BS + j : (long)q1 * BS + (j - BS);
                    if (gi < L) d.W[gi + gj * L] = T[i][j];
                }
            __syncthreads();
        }
    }
}

template <int BS>
__global__ __launch_bounds__(256) void k_jacobi_apply(const EigDesc* __restrict__ descs, int round, int sched) {
    const EigDesc d = descs[blockIdx.y];
    if (d.run[0] == 0 || d.st[0] != 0) return;
    const int nb = d.L / BS;
    const int item = blockIdx.x;
    if (item >= apply_items<BS>(d.L) || round >= nb - 1) return;
    __shared__ ApplyLds<BS> sm;
    apply_item<BS>(d, round, item, sched, blockIdx.x + blockIdx.y * gridDim.x, sm, d.B, d.B, 0, threadIdx.x, true);
}

// Pairs of round r and tile updates of round r - 1 in one launch (16-wide blocks).
// A round's pair solves need only three 16 x 16 blocks of the matrix that the tile
// updates of the round before are still writing, so each forms those itself from
// the matrix before that round and its rotations (the same products in the same
// order: the same bits), while the other workgroups run the updates into the
// second buffer.  A round then takes the longer of the two phases instead of their
// sum, and one launch instead of two (15.5 + 11 us and two gaps -> about 21 us and
// one, 4 matrices of order 320).
struct AheadLds {
    double X[3][32][33];     // tiles [A, A], [A, C], [C, C] of the previous round, then T
    double RA[32][17], RC[32][17];
    int slot[2];
};

// slot of index block x in round r, for x = p (first) and q (second half of the
// workgroup's search); every thread takes part
__device__ __forceinline__ void find_slots(const EigDesc& d, int nb, int round, int sched, int p, int q, int* slot) {
    for (int k = threadIdx.x; k < nb / 2; k += blockDim.x) {
        int a, b;
        round_pair(d, nb, round, k, sched, a, b);
        if (a == p || b == p) slot[0] = k;
        if (a == q || b == q) slot[1] = k;
    }
    __syncthreads();
}

// S (32 x 32, index blocks p and q of round r) after the updates of round r - 1,
// from src, the matrix before them.  Loads by every thread of the workgroup, products
// by its first four waves.
__device__ void look_ahead(const EigDesc& d, int round, int p, int q, int sched, const double* src, AheadLds& sm,
                           double (*S)[40]) {
    constexpr int BS = 16, PB = 32;
    const int nb = d.L / BS, tid = threadIdx.x, prev = round - 1, set = prev & 1;
    const long L = d.L;
    find_slots(d, nb, prev, sched, p, q, sm.slot);
    const int A = sm.slot[0], C = sm.slot[1];
    int a1, a2, c1, c2;
    round_pair(d, nb, prev, A, sched, a1, a2);
    round_pair(d, nb, prev, C, sched, c1, c2);
    const int hp = p == a1 ? 0 : BS, hq = q == c1 ? 0 : BS;   // halves of p and q in their pairs
    const int* prot = d.prot + set * (nb / 2);
    const bool rotA = prot[A] != 0, rotC = prot[C] != 0;
    const bool still = !rotA && !rotC;   // the mirrored half then is the one in memory
    const double* RgA = d.R + (long)(set * (nb / 2) + A) * PB * PB;
    const double* RgC = d.R + (long)(set * (nb / 2) + C) * PB * PB;
    // the off-diagonal tile as the update forms it: rows of the lower slot
    const bool swap = A > C;
    const int r1 = swap ? c1 : a1, r2 = swap ? c2 : a2, s1 = swap ? a1 : c1, s2 = swap ? a2 : c2;
    for (int idx = tid; idx < PB * PB; idx += blockDim.x) {
        const int i = idx % PB, j = idx / PB;
        const long ai = (i < BS ? a1 * BS : a2 * BS - BS) + i, aj = (j < BS ? a1 * BS : a2 * BS - BS) + j;
        const long ci = (i < BS ? c1 * BS : c2 * BS - BS) + i, cj = (j < BS ? c1 * BS : c2 * BS - BS) + j;
        const long ri = (i < BS ? r1 * BS : r2 * BS - BS) + i, sj = (j < BS ? s1 * BS : s2 * BS - BS) + j;
        sm.X[0][i][j] = src[ai + aj * L];
        sm.X[1][i][j] = src[ri + sj * L];
        sm.X[2][i][j] = src[ci + cj * L];
        if (j < BS) {
            sm.RA[i][j] = rotA ? RgA[i + (long)(hp + j) * PB] : (i == hp + j ? 1.0 : 0.0);
            sm.RC[i][j] = rotC ? RgC[i + (long)(hq + j) * PB] : (i == hq + j ? 1.0 : 0.0);
        }
    }
    __syncthreads();
    // T = X R, the 16 columns wanted: wave w < 3 takes tile w (rows 0..31); then
    // 16 x 16 results R^T T.  Where p and q were a pair already (A = C), wave 3 forms
    // the other half of that tile, which is not the mirror image to the last bit.
    const int w = tid >> 6, lane = tid & 63, lr = lane & 15, lk = lane >> 4;
    dbl4 t0 = {0.0, 0.0, 0.0, 0.0}, t1 = t0, o = t0;
    // tile 1 has rows of the lower slot and columns of the upper one
    const double (*Rr)[17] = w == 0 ? sm.RA : w == 2 ? sm.RC : swap ? sm.RA : sm.RC;   // on the columns
    const double (*Rl)[17] = w == 0 ? sm.RA : w == 2 ? sm.RC : swap ? sm.RC : sm.RA;   // on the rows
    if (w < 3) {
#pragma unroll
        for (int kk = 0; kk < PB; kk += 4) {
            const int k = kk + lk;
            const double b = Rr[k][lr];
            t0 = __builtin_amdgcn_mfma_f64_16x16x4f64(sm.X[w][lr][k], b, t0, 0, 0, 0);
            t1 = __builtin_amdgcn_mfma_f64_16x16x4f64(sm.X[w][16 + lr][k], b, t1, 0, 0, 0);
        }
    }
    __syncthreads();
    if (w < 3) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            sm.X[w][lk + 4 * v][lr] = t0[v];
            sm.X[w][16 + lk + 4 * v][lr] = t1[v];
        }
    }
    __syncthreads();
    const bool other = w == 3 && A == C;
    if (w < 3 || other) {
        const double (*Rw)[17] = other ? sm.RC : Rl;
        const double (*Tw)[33] = other ? sm.X[0] : sm.X[w];
#pragma unroll
        for (int kk = 0; kk < PB; kk += 4) {
            const int k = kk + lk;
            o = __builtin_amdgcn_mfma_f64_16x16x4f64(Rw[k][lr], Tw[k][lr], o, 0, 0, 0);
        }
    }
    __syncthreads();   // S may share the space of sm
    if (w < 3 || other) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int i = lk + 4 * v, j = lr;
            if (w == 0) S[i][j] = o[v];
            else if (w == 2) S[BS + i][BS + j] = o[v];
            else if (w == 3) S[BS + i][j] = o[v];
            else if (!swap) {
                S[i][BS + j] = o[v];
                if (A != C) S[BS + j][i] = still ? src[(long)q * BS + j + ((long)p * BS + i) * L] : o[v];
            } else {
                S[j][BS + i] = still ? src[(long)p * BS + j + ((long)q * BS + i) * L] : o[v];
                S[BS + i][j] = o[v];
            }
        }
    }
    __syncthreads();
}

// Workgroups [0, npair_max) of a matrix: pair solves of round r; then the tile
// updates of round r - 1 (r >= 1), two per workgroup: first the tiles of B, then the
// chunks of W.  rounds: of this pass; the last update writes the matrix back into B.
__global__ __launch_bounds__(kPairThreads) void k_jacobi_step(const EigDesc* __restrict__ descs, int r, int rounds,
                                                               int sched, int npair_max) {
    constexpr int BS = 16;
    const EigDesc d = descs[blockIdx.y];
    if (d.run[0] == 0 || d.st[0] != 0) return;
    __shared__ union {
        ApplyLds<BS> a[2];
        PairLds<BS> p;
        AheadLds h;
    } sm;
    const int nb = d.L / BS, npair = nb / 2;
    const int mine = min(rounds, nb - 1);   // rounds this matrix takes
    const double* src = (r & 1) ? d.B : d.B2;   // the matrix before round r - 1
    if ((int)blockIdx.x < npair_max) {
        const int P = blockIdx.x;
        if (P >= npair || r >= mine) return;
        int p, q;
        round_pair(d, nb, r, P, sched, p, q);
        look_ahead(d, r, p, q, sched, src, sm.h, sm.p.S[0]);
        pair_solve<BS, kPairThreads>(d, r, P, sched, blockIdx.x + blockIdx.y * gridDim.x, sm.p, r & 1, true);
    } else {
        const int half = threadIdx.x >> 8;
        const int ntri = npair * (npair + 1) / 2, ntri2 = (ntri + 1) / 2, all = apply_items<BS>(d.L);
        const int g = blockIdx.x - npair_max;
        const int item = g < ntri2 ? 2 * g + half : ntri + 2 * (g - ntri2) + half;
        if (ntri + 2 * (g - ntri2) >= all || r - 1 >= mine) return;
        const bool live = g < ntri2 ? item < ntri : item < all;
        double* dst = (r == mine || !(r & 1)) ? d.B : d.B2;
        apply_item<BS>(d, r - 1, live ? item : (g < ntri2 ? 0 : ntri), sched, blockIdx.x + blockIdx.y * gridDim.x,
                       sm.a[half], src, dst, (r - 1) & 1, threadIdx.x & 255, live);
    }
}

// start of an eigensolve: reset flags, scale = max |diag|
__global__ __launch_bounds__(256) void k_jacobi_init(const EigDesc* __restrict__ descs) {
    const EigDesc d = descs[blockIdx.x];
    if (d.run[0] == 0) return;
    const bool done = d.done && d.done[0];
    if (done) {
        for (int i = threadIdx.x; i < d.l; i += 256) d.B[i + (long)i * d.L] = d.lam[i];
        __syncthreads();
    }
    double mx = 0.0;
    for (int i = threadIdx.x; i < d.l; i += 256) mx = fmax(mx, fabs(d.B[i + (long)i * d.L]));
    mx = wave_max(mx);
    __shared__ double red[4];
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
        d.scale[0] = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
        d.st[0] = done ? 1 : 0;
        d.st[1] = 0;
    }
}

// one launch per sweep: does any off-diagonal entry still need a rotation?  With
// bs > 0 and need set, the index-block pairs holding such entries are marked.
__global__ __launch_bounds__(256) void k_jacobi_offcheck(const EigDesc* __restrict__ descs, int* n_open, int bs) {
    const EigDesc d = descs[blockIdx.y];
    if (d.run[0] == 0 || d.st[0] != 0) return;
    const long L = d.L;
    const long total = (long)d.l * d.l;
    const double floor_abs = kAbsFloor * d.scale[0];
    int* const mark = (bs > 0) ? d.need : nullptr;
    const int nb = (bs > 0) ? d.L / bs : 0;
    int need = 0;
    for (long idx = (long)blockIdx.x * 256 + threadIdx.x; idx < total; idx += (long)gridDim.x * 256) {
        const int i = (int)(idx % d.l), j = (int)(idx / d.l);
        if (i < j && !(d.lo[i] && d.lo[j])) {
            const double a = d.B[i + j * L];
            if (fabs(a) > fmax(kRelTol * sqrt(fabs(d.B[i + i * L] * d.B[j + j * L])), floor_abs)) {
                need = 1;
                if (mark) mark[(i / bs) * nb + j / bs] = 1;   // every writer stores 1
            }
        }
    }
    __shared__ int any;
    if (threadIdx.x == 0) any = 0;
    __syncthreads();
    if (need) any = 1;
    __syncthreads();
    if (threadIdx.x == 0 && any) atomicOr(&d.st[1], 1);
}

// after the check: a matrix with nothing left to rotate is converged
__global__ void k_jacobi_close(const EigDesc* __restrict__ descs, int count, int* n_open) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= count) return;
    const EigDesc d = descs[b];
    if (d.run[0] == 0 || d.st[0] != 0) return;
    if (d.st[1] == 0) d.st[0] = 1;
    else atomicAdd(n_open, 1);
    d.st[1] = 0;
}

// eigenvalues = diagonal (padding -> 0)
__global__ void k_jacobi_eigvals(const EigDesc* __restrict__ descs) {
    const EigDesc d = descs[blockIdx.x];
    if (d.run[0] == 0) return;
    for (int i = threadIdx.x; i < d.L; i += blockDim.x)
        d.lam[i] = (i < d.l) ? d.B[i + (long)i * d.L] : 0.0;
}

// ---------------------------------------------------------------------------
// Persistent eigensolve: the whole pass loop of the batched block-Jacobi method
// in one launch.  Each pass: Gershgorin flags of every open matrix, the check of
// every off-diagonal entry (marking the index-block pairs that still need a
// rotation), closing converged matrices, and either a targeted pass (rounds of
// perfect matchings covering the marked pairs, planned per matrix on the
// device) or a full circle sweep; then the rounds, each a pair phase and an
// apply phase.  Phases are separated by grid-wide barriers; every workgroup
// takes the same decisions from the same global values, so the control flow
// is uniform across the grid.  The results are those of the launch-per-phase
// kernels above (same device functions, same order of operations).
//
// The grid must fit on the chip at once (the host sizes it from the occupancy
// of this kernel).  Each barrier wait is bounded: a wait that runs out sets
// JacCtl::err and every workgroup leaves at its next barrier, so the kernel
// always ends; the host reports the flag as an error.
// ---------------------------------------------------------------------------
constexpr int kSolveThreads = 256;
constexpr long kSpinLimit = 1L << 23;   // s_sleep(1) waits of one barrier (~0.4 s)
constexpr int kChecksPerMatrix = 64;    // check items per matrix (as the check launch's grid)
constexpr int kPlanMaxNb = 64;          // index blocks the device planner handles (bit masks)

// all workgroups of the grid reach this point; false once any wait ran out
__device__ bool grid_sync(JacCtl* ctl, unsigned nwg, unsigned& gen) {
    __syncthreads();
    __shared__ int bad;
    if (threadIdx.x == 0) {
        const unsigned g = gen;
        const unsigned a = __hip_atomic_fetch_add(&ctl->bar_count, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
        if (a == nwg - 1) {
            __hip_atomic_store(&ctl->bar_count, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&ctl->bar_gen, g + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        } else {
            long spins = 0;
            while (__hip_atomic_load(&ctl->bar_gen, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) == g) {
                __builtin_amdgcn_s_sleep(1);
                if (++spins > kSpinLimit) {
                    __hip_atomic_store(&ctl->err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    break;
                }
                // another workgroup's wait ran out: leave at once
                if ((spins & 1023) == 0 && __hip_atomic_load(&ctl->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                    break;
            }
        }
        gen = g + 1;
        bad = __hip_atomic_load(&ctl->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    return bad == 0;
}

// block b of item `item` given the prefix counts off[0..t]
__device__ __forceinline__ int item_block(const int* __restrict__ off, int t, int item) {
    int b = 0;
    while (b + 1 < t && off[b + 1] <= item) ++b;
    return b;
}

struct PlanLds {
    unsigned short pp[kPlanMaxNb * (kPlanMaxNb - 1) / 2];
    unsigned short qq[kPlanMaxNb * (kPlanMaxNb - 1) / 2];
    unsigned char cov[kPlanMaxNb * (kPlanMaxNb - 1) / 2];
    int cnt[kSolveThreads + 1];
    unsigned long long inner;
};

// Targeted rounds of one matrix (the device form of the host planner
// plan_rounds): the marked pairs p < q in p-major order are covered greedily,
// round by round, each round completed to a perfect matching of the nb index
// blocks (a block marked inside goes with a free partner, preferring another
// such block; the rest pair up in order).  Returns the number of rounds, or -1
// when more than cap would be needed (or nb exceeds the bit masks).
__device__ int plan_device(const int* __restrict__ need, int nb, int cap, int* __restrict__ sched, PlanLds& pl) {
    const int tid = threadIdx.x;
    if (nb > kPlanMaxNb) return -1;
    const int total = nb * nb;
    const int per = (total + kSolveThreads - 1) / kSolveThreads;
    const int i0 = tid * per, i1 = min(total, i0 + per);
    if (tid == 0) pl.inner = 0ull;
    __syncthreads();
    int c = 0;
    unsigned long long inner = 0ull;
    for (int idx = i0; idx < i1; ++idx) {
        const int p = idx / nb, q = idx % nb;
        if (q < p || !need[idx]) continue;
        if (p == q) inner |= 1ull << p;
        else ++c;
    }
    pl.cnt[tid + 1] = c;
    if (inner) atomicOr(&pl.inner, inner);
    __syncthreads();
    if (tid == 0) {
        pl.cnt[0] = 0;
        for (int k = 1; k <= kSolveThreads; ++k) pl.cnt[k] += pl.cnt[k - 1];
    }
    __syncthreads();
    int w = pl.cnt[tid];
    for (int idx = i0; idx < i1; ++idx) {
        const int p = idx / nb, q = idx % nb;
        if (q <= p || !need[idx]) continue;
        pl.pp[w] = (unsigned short)p;
        pl.qq[w] = (unsigned short)q;
        pl.cov[w] = 0;
        ++w;
    }
    __syncthreads();
    const int npend = pl.cnt[kSolveThreads];
    int rounds = 0;
    if (tid == 0) {
        unsigned long long in = pl.inner;
        const unsigned long long all = (nb == 64) ? ~0ull : ((1ull << nb) - 1ull);
        int left = npend;
        if (npend > cap * (nb / 2)) {
            rounds = -1;   // each round covers at most nb / 2 pairs
        } else {
            for (;;) {
                if (left == 0 && in == 0ull) break;
                if (rounds == cap) { rounds = -1; break; }
                int* slot = sched + (long)rounds * (nb / 2);
                int ns = 0;
                unsigned long long used = 0ull;
                for (int e = 0; e < npend; ++e) {
                    if (pl.cov[e]) continue;
                    const int p = pl.pp[e], q = pl.qq[e];
                    const unsigned long long bits = (1ull << p) | (1ull << q);
                    if (used & bits) continue;
                    slot[ns++] = p | (q << 16);
                    used |= bits;
                    in &= ~bits;   // a pair solve also sweeps inside both blocks
                    pl.cov[e] = 1;
                    --left;
                }
                for (int p = 0; p < nb; ++p) {
                    if (!((in >> p) & 1ull) || ((used >> p) & 1ull)) continue;
                    const unsigned long long fr = all & ~used & ~(1ull << p);
                    const unsigned long long fri = fr & in;
                    const int q = fri ? __ffsll((long long)fri) - 1 : __ffsll((long long)fr) - 1;
                    if (q < 0) break;   // cannot happen (nb is even, so a free partner exists)
                    const int a = min(p, q), b = max(p, q);
                    slot[ns++] = a | (b << 16);
                    const unsigned long long bits = (1ull << p) | (1ull << q);
                    used |= bits;
                    in &= ~bits;
                }
                int u = -1;
                for (int x = 0; x < nb; ++x) {
                    if ((used >> x) & 1ull) continue;
                    if (u < 0) u = x;
                    else { slot[ns++] = u | (x << 16); u = -1; }
                }
                ++rounds;
            }
        }
        pl.cnt[0] = rounds;
    }
    __syncthreads();
    rounds = pl.cnt[0];
    __syncthreads();
    return rounds;
}

template <int BS>
__global__ __launch_bounds__(kSolveThreads) void k_jacobi_solve(const EigDesc* __restrict__ descs, int t,
                                                                 const int* __restrict__ offs, int* brounds,
                                                                 JacCtl* ctl, const DevIter* it, int max_sweeps,
                                                                 int max_targeted, int nb_max, int* need_all,
                                                                 long need_total) {
    __shared__ union {
        PairLds<BS> p;
        ApplyLds<BS> a;
        PlanLds pl;
    } sm;
    __shared__ double red[4];
    const unsigned G = gridDim.x;
    const int wg = blockIdx.x, tid = threadIdx.x;
    const int* off_rows = offs;
    const int* off_pairs = offs + (t + 1);
    const int* off_apply = offs + 2 * (t + 1);
    unsigned gen = 0;

    // start of the eigensolve: scale = max |diag|, flags cleared
    for (int b = wg; b < t; b += G) {
        const EigDesc d = descs[b];
        if (d.run[0] == 0) continue;
        const bool done = d.done && d.done[0];
        if (done) {
            for (int i = tid; i < d.l; i += kSolveThreads) d.B[i + (long)i * d.L] = d.lam[i];
            __syncthreads();
        }
        double mx = 0.0;
        for (int i = tid; i < d.l; i += kSolveThreads) mx = fmax(mx, fabs(d.B[i + (long)i * d.L]));
        mx = wave_max(mx);
        if ((tid & 63) == 0) red[tid >> 6] = mx;
        __syncthreads();
        if (tid == 0) {
            d.scale[0] = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
            d.st[0] = done ? 1 : 0;
            d.st[1] = 0;
        }
        __syncthreads();
    }
    if (!grid_sync(ctl, G, gen)) return;

    const double tau = it->tau;
    const int full_all = it->full;
    int full = 0, targeted = 0, pass = 0;
    bool counted = true;
    for (;;) {
        // Gershgorin flags of the open matrices; the marks are cleared
        for (long k = (long)wg * kSolveThreads + tid; k < need_total; k += (long)G * kSolveThreads) need_all[k] = 0;
        for (int item = wg; item < off_rows[t]; item += G) {
            const int b = item_block(off_rows, t, item);
            const EigDesc d = descs[b];
            if (d.run[0] == 0 || d.st[0] != 0) continue;
            const int i = item - off_rows[b];
            const long L = d.L;
            double rs = 0.0;   // column i of the symmetric matrix, contiguous
            for (int j = tid; j < d.l; j += kSolveThreads)
                if (j != i) rs += fabs(d.B[j + i * L]);
            rs = wave_sum(rs);
            if ((tid & 63) == 0) red[tid >> 6] = rs;
            __syncthreads();
            if (tid == 0) {
                const double r = (red[0] + red[1]) + (red[2] + red[3]);
                d.lo[i] = (i >= d.l) ? 1 : (full_all ? 0 : lo_flag(d.B[i + i * L] + r, tau, d.cut[0], d.scale[0]));
                if (i == 0 && counted) d.passes[0] += 1;
            }
            __syncthreads();
        }
        if (!grid_sync(ctl, G, gen)) return;
        // check: does any off-diagonal entry still need a rotation; mark its blocks
        for (int item = wg; item < t * kChecksPerMatrix; item += G) {
            const int b = item / kChecksPerMatrix, part = item % kChecksPerMatrix;
            const EigDesc d = descs[b];
            if (d.run[0] == 0 || d.st[0] != 0) continue;
            const long L = d.L;
            const long total = (long)d.l * d.l;
            const double floor_abs = kAbsFloor * d.scale[0];
            const int nb = d.L / BS;
            int need = 0;
            for (long idx = (long)part * kSolveThreads + tid; idx < total; idx += (long)kChecksPerMatrix * kSolveThreads) {
                const int i = (int)(idx % d.l), j = (int)(idx / d.l);
                if (i < j && !(d.lo[i] && d.lo[j])) {
                    const double a = d.B[i + j * L];
                    if (fabs(a) > fmax(kRelTol * sqrt(fabs(d.B[i + i * L] * d.B[j + j * L])), floor_abs)) {
                        need = 1;
                        d.need[(i / BS) * nb + j / BS] = 1;   // every writer stores 1
                    }
                }
            }
            if (__syncthreads_or(need) && tid == 0) atomicOr(&d.st[1], 1);
        }
        if (!grid_sync(ctl, G, gen)) return;
        // close converged matrices, count the open ones, plan targeted rounds
        for (int b = wg; b < t; b += G) {
            const EigDesc d = descs[b];
            const int nbb = d.L / BS;
            int open = 0;
            if (d.run[0] != 0 && d.st[0] == 0) {
                open = d.st[1] != 0;
                __syncthreads();
                if (tid == 0) {
                    if (!open) d.st[0] = 1;
                    else atomicAdd(&ctl->n_open[pass & 1], 1);
                    d.st[1] = 0;
                }
            }
            int rb = 0;
            if (open && targeted < max_targeted)
                rb = plan_device(d.need, nbb, min((nb_max - 1) / 2, nbb - 1), const_cast<int*>(d.sched), sm.pl);
            if (tid == 0) brounds[b] = rb;
            __syncthreads();
        }
        if (!grid_sync(ctl, G, gen)) return;
        // the same decision in every workgroup
        const int nopen = __hip_atomic_load(&ctl->n_open[pass & 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (wg == 0 && tid == 0) ctl->n_open[(pass + 1) & 1] = 0;
        if (nopen == 0 || full == max_sweeps) break;
        int rounds = targeted < max_targeted ? 0 : -1;
        for (int b = 0; b < t && rounds >= 0; ++b) {
            const int rb = brounds[b];
            rounds = rb < 0 ? -1 : max(rounds, rb);
        }
        int sched;
        if (rounds > 0) {
            // matrices that need fewer rounds get circle rounds (any perfect matching is valid)
            for (int b = wg; b < t; b += G) {
                const EigDesc d = descs[b];
                const int nbb = d.L / BS, np = nbb / 2;
                const int r0 = brounds[b], r1 = min(rounds, nbb - 1);
                int* sc = const_cast<int*>(d.sched);
                for (int k = tid; k < (r1 - r0) * np; k += kSolveThreads) {
                    const int r = r0 + k / np, P = k % np;
                    int a0, b0;
                    rr_pair(nbb, r, P, a0, b0);
                    sc[r * np + P] = a0 | (b0 << 16);
                }
            }
            if (!grid_sync(ctl, G, gen)) return;
            ++targeted;
            counted = false;
            sched = 1;
        } else {
            rounds = nb_max - 1;
            ++full;
            counted = true;
            sched = 0;
        }
        for (int r = 0; r < rounds; ++r) {
            for (int item = wg; item < off_pairs[t]; item += G) {
                const int b = item_block(off_pairs, t, item);
                const EigDesc d = descs[b];
                if (d.run[0] == 0 || d.st[0] != 0 || r >= d.L / BS - 1) continue;
                pair_solve<BS, kSolveThreads>(d, r, item - off_pairs[b], sched, wg, sm.p);
                __syncthreads();
            }
            if (!grid_sync(ctl, G, gen)) return;
            for (int item = wg; item < off_apply[t]; item += G) {
                const int b = item_block(off_apply, t, item);
                const EigDesc d = descs[b];
                if (d.run[0] == 0 || d.st[0] != 0 || r >= d.L / BS - 1) continue;
                apply_item<BS>(d, r, item - off_apply[b], sched, wg, sm.a, d.B, d.B, 0, tid, true);
                __syncthreads();
            }
            if (!grid_sync(ctl, G, gen)) return;
        }
        ++pass;
    }
}

// before each launch; the error flag stays set once raised (the host clears it
// at the start of a solve and reads it with the convergence flags)
__global__ void k_jacobi_ctl_reset(JacCtl* ctl) {
    ctl->bar_count = 0u;
    ctl->bar_gen = 0u;
    ctl->n_open[0] = 0;
    ctl->n_open[1] = 0;
}

}  // namespace

void launch_jacobi_init(const EigDesc* d_descs, int count, hipStream_t s) {
    hipLaunchKernelGGL(k_jacobi_init, dim3(count), dim3(256), 0, s, d_descs);
}

void launch_jacobi_pairs(const EigDesc* d_descs, int count, int maxL, int bs, int round, hipStream_t s,
                         bool sched) {
    const int npair = maxL / bs / 2;
    if (bs == 16)
        hipLaunchKernelGGL((k_jacobi_pairs<16, kPairThreads>), dim3(npair, count), dim3(kPairThreads), 0, s, d_descs,
                           round, (int)sched);
    else
        hipLaunchKernelGGL((k_jacobi_pairs<32, kPairThreads>), dim3(npair, count), dim3(kPairThreads), 0, s, d_descs,
                           round, (int)sched);
}

void launch_jacobi_apply(const EigDesc* d_descs, int count, int maxL, int bs, int round, hipStream_t s,
                         bool sched) {
    const int npair = maxL / bs / 2;
    const int ntri = npair * (npair + 1) / 2;
    const int nchunks = (maxL + 63) / 64;
    if (bs == 16)
        hipLaunchKernelGGL((k_jacobi_apply<16>), dim3(ntri + nchunks * npair, count), dim3(256), 0, s,
                           d_descs, round, (int)sched);
    else
        hipLaunchKernelGGL((k_jacobi_apply<32>), dim3(ntri + nchunks * npair, count), dim3(256), 0, s,
                           d_descs, round, (int)sched);
}

constexpr double kLastLevelCache = 256.0 * 1048576.0;

// compute units of the device (looked up once; outside any stream capture)
static int cu_count() {
    static int cus = 0;
    if (cus == 0) {
        int dev = 0, n = 0;
        LRR_HIP(hipGetDevice(&dev));
        LRR_HIP(hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev));
        cus = std::max(n, 1);
    }
    return cus;
}

void launch_jacobi_rounds(const EigDesc* d_descs, int count, int maxL, int bs, int rounds, hipStream_t s,
                          bool sched) {
    // Both phases in one launch while the pair solves alone do not fill the chip: m =
    // 500, n = 2000, 4 matrices of order 320, 219 -> 201 ms per solve.  With 640 pairs (40
    // matrices of order 512) there is nothing to overlap and the tiles that did not rotate
    // would be copied: 336 -> 341 ms.  And while B, its second buffer and W stay in the
    // last-level cache, as B and W alone do longer: whole eigensolves in two launches a
    // round and in one, order 2016 93 / 79 ms, 3000 243 / 231, 3500 367 / 370, 4000 541 /
    // 691, 5000 1362 / 1485; two matrices of order 2000 142 / 137, three 193 / 205.
    const double bytes = 3.0 * count * (double)maxL * maxL * sizeof(double);
    if (bs != 16 || count * (maxL / bs / 2) >= cu_count() || bytes > kLastLevelCache) {
        for (int r = 0; r < rounds; ++r) {
            launch_jacobi_pairs(d_descs, count, maxL, bs, r, s, sched);
            launch_jacobi_apply(d_descs, count, maxL, bs, r, s, sched);
        }
        return;
    }
    const int npair = maxL / bs / 2;
    const int items = (npair * (npair + 1) / 2 + 1) / 2 + (((maxL + 63) / 64) * npair + 1) / 2;
    launch_jacobi_pairs(d_descs, count, maxL, bs, 0, s, sched);
    for (int r = 1; r <= rounds; ++r) {
        const int np = r < rounds ? npair : 0;
        hipLaunchKernelGGL(k_jacobi_step, dim3(np + items, count), dim3(kPairThreads), 0, s, d_descs, r, rounds,
                           (int)sched, np);
    }
}

void launch_jacobi_check(const EigDesc* d_descs, int count, int maxL, int* d_open, hipStream_t s, int bs) {
    const int blocks = (maxL * maxL + 255) / 256 < 64 ? (maxL * maxL + 255) / 256 : 64;
    hipLaunchKernelGGL(k_jacobi_offcheck, dim3(blocks, count), dim3(256), 0, s, d_descs, d_open, bs);
    hipLaunchKernelGGL(k_jacobi_close, dim3((count + 63) / 64), dim3(64), 0, s, d_descs, count, d_open);
}

int jacobi_solve_grid(int bs) {
    static int grid[2] = {0, 0};
    int& g = grid[bs == 32 ? 1 : 0];
    if (g == 0) {
        int per = 0;
        if (bs == 32)
            LRR_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_jacobi_solve<32>, kSolveThreads, 0));
        else
            LRR_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_jacobi_solve<16>, kSolveThreads, 0));
        if (per < 1) throw HipError("the persistent eigensolve does not fit on a CU");
        // one workgroup per CU: a grid barrier costs each workgroup an L2
        // write-back and invalidation at agent scope (measured 15-24 us with 256
        // workgroups, 67-93 us with 1024)
        g = cu_count();
    }
    return g;
}

void launch_jacobi_solve(const EigDesc* d_descs, int count, const int* d_offs, int* d_brounds, JacCtl* ctl,
                         const DevIter* it, int max_sweeps, int max_targeted, int nb_max, int bs, int* need_all,
                         long need_total, hipStream_t s) {
    hipLaunchKernelGGL(k_jacobi_ctl_reset, dim3(1), dim3(1), 0, s, ctl);
    const dim3 grid(jacobi_solve_grid(bs));
    if (bs == 32)
        hipLaunchKernelGGL((k_jacobi_solve<32>), grid, dim3(kSolveThreads), 0, s, d_descs, count, d_offs, d_brounds,
                           ctl, it, max_sweeps, max_targeted, nb_max, need_all, need_total);
    else
        hipLaunchKernelGGL((k_jacobi_solve<16>), grid, dim3(kSolveThreads), 0, s, d_descs, count, d_offs, d_brounds,
                           ctl, it, max_sweeps, max_targeted, nb_max, need_all, need_total);
}

void launch_jacobi_eigvals(const EigDesc* d_descs, int count, hipStream_t s) {
    hipLaunchKernelGGL(k_jacobi_eigvals, dim3(count), dim3(256), 0, s, d_descs);
}

}  // namespace lrr
