"""The work that a user of the DFC-LRR library has it do, as cases that can be timed and checked.

Every case goes through the public entry points of ``paper_1304_5583_amd.binding``
and ``paper_1304_5583_amd.autograd`` the way a program calls them.  The data are
seeded unions of subspaces with corrupted columns (``paper_1304_5583_amd.datagen``),
in the sizes of the five workloads, of the tests, and between them.

    kind      entry point and what it stands for
    lrr       lrr_solve(M, M): plain LRR of one data set
    dfc       dfc_lrr_solve: Algorithm 1, the library's main call; float64
              buffers, or float32 ones for data that come that way (images) and
              for the reduced-precision forms
    local     dfc_lrr_solve_local: each block its own dictionary
    grad      dfc_lrr and its reverse mode: one step of a program that learns the
              dictionary or the regulariser
    segment   lrr_segment: cluster labels from a coefficient matrix
    slr       lrr_slr_graph: neighbours and edge weights from a coefficient matrix

    recipe    data (Section 4.1.1 generator and the workloads built from it)
    replaced  Gaussian coefficients, some columns replaced by Gaussian vectors
    unit      columns of length one, 5 % of them with 0.3 of noise added
    image     non-negative, clipped to [0, 1], 10 % of the columns with 10 % of
              their entries overwritten
"""
import math

import numpy as np
import torch

from paper_1304_5583_amd import autograd, binding, datagen

ITERS = 190   # iterations of a solve to the default tolerance, for work() only


def _case(kind, recipe, m, k, r, ns, lo, hi, **more):
    """m rows; k subspaces of dimension r with ns points each; blocks of lo..hi columns."""
    c = dict(kind=kind, recipe=recipe, m=m, k=k, r=r, ns=ns, lo=lo, hi=hi, replace=0, lam=0.2,
             dtype="float64", precision=0, tol=1e-8, fixed_iters=0, nk=0)
    c.update(more)
    return c


def listed():
    return [
        # plain LRR of 200 points: one block, latency throughout (workload 1)
        dict(_case("lrr", "replaced", 100, 5, 5, 40, 200, 200, replace=20, lam=0.1), name="lrr_n200"),
        # the smallest DFC call that the tests and the smoke check make
        dict(_case("dfc", "replaced", 48, 3, 3, 32, 28, 36, replace=6, lam=0.3), name="dfc_n96_t3"),
        # an ordinary DFC solve: 2000 unit columns, 4 blocks of 500 (workload 2)
        dict(_case("dfc", "unit", 500, 20, 10, 100, 500, 500), name="dfc_n2000_t4"),
        # the shape of a face data set, 48 x 42 pixels, uneven blocks, in the float32
        # that images come in (workload 3)
        dict(_case("dfc", "image", 2016, 38, 9, 64, 100, 200, lam=0.15, dtype="float32"), name="dfc_faces_t16"),
        # the largest: 20000 points, 40 blocks of 500 (workload 4, the benchmark)
        dict(_case("dfc", "replaced", 512, 100, 20, 200, 500, 500, replace=2000, lam=0.0244), name="dfc_n20000_t40"),
        # the reduced-precision form on float32 buffers, odd sizes
        dict(_case("dfc", "unit", 333, 17, 11, 239, 260, 330, dtype="float32", precision=2), name="dfc_bf16x3_n4063"),
        # forward and reverse mode of the unrolled solve (workload 5's kind of step)
        dict(_case("grad", "unit", 200, 10, 6, 60, 150, 150, fixed_iters=200), name="grad_n600_t4"),
        # every block its own dictionary
        dict(_case("local", "unit", 500, 20, 10, 100, 500, 500), name="local_n2000_t4"),
        # labels of 2000 points, directly, and of 12000 through the range sketch
        dict(_case("segment", "unit", 500, 20, 10, 100, 0, 0), name="segment_n2000"),
        dict(_case("segment", "unit", 512, 60, 8, 200, 0, 0), name="segment_n12000"),
        # the graph with the paper's 500 neighbours, and at scale on data whose
        # replaced columns draw large supports
        dict(_case("slr", "unit", 500, 20, 10, 100, 0, 0, nk=500), name="slr_n2000"),
        dict(_case("slr", "replaced", 512, 50, 20, 200, 0, 0, replace=1000, nk=500), name="slr_n10000"),
    ]


def draw(rng):
    def size(lo, hi):   # spread over the logarithm
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["lrr", "dfc", "dfc", "dfc", "dfc", "local", "grad", "segment", "slr"])
    n = {"lrr": size(96, 600), "dfc": size(90, 9000), "local": size(120, 2000), "grad": size(90, 500),
         "segment": size(200, 9000), "slr": size(300, 6000)}[kind]
    m = size(40, 520) if kind != "lrr" else size(40, n // 2)
    r = rng.randint(3, min(12, m // 5))
    k = max(2, min(m // r - 1, n // (5 * r), rng.randint(3, 30)))
    ns = max(2 * r, n // k)
    n = k * ns
    # drawn solves stop at 1e-6: on data that converge slowly the last decades of
    # the default 1e-8 decide about directions at the rounding level of the result
    c = _case(kind, "unit", m, k, r, ns, n, n, tol=1e-6)
    if kind in ("dfc", "local", "grad"):
        width = min(n // 2, size(28, 500 if kind != "grad" else 150))
        t = min(4 if kind == "local" else 40, max(2, n // width))
        width = n // t
        if width > 520:   # as in the listed cases, a block has at most about 500 columns
            t = -(-n // 500)
            width = n // t
        c.update(lo=max(2, width - width // 7 - 1), hi=width + width // 7 + 2)
    if kind == "dfc":
        form = rng.choice(["unit", "unit", "unit32", "reduced", "image", "replaced"])
        if form == "unit32":
            c.update(dtype="float32")
        elif form == "reduced" and n >= 1000:   # a form for the larger inputs
            c.update(dtype="float32", precision=rng.choice([1, 2]))
        elif form == "image":
            c.update(recipe="image", m=size(100, 2000), dtype="float32", lam=0.15)
        elif form == "replaced":
            # as in workload 4 the subspaces fill the space (k r > m, n > 3 m)
            c.update(k=(3 * m) // (2 * r) + 1)
            c.update(ns=max(2 * r, n // c["k"]))
            n = c["k"] * c["ns"]
            t = max(2, -(-n // min(width, 480)))
            c.update(lo=n // t - n // t // 9 - 1, hi=n // t + n // t // 9 + 2, recipe="replaced", replace=n // 10,
                     lam=0.0, dtype="float32")
    if kind == "grad":
        c.update(fixed_iters=rng.randint(150, 200))
    if kind == "slr":
        c.update(nk=min(n - 1, size(20, 500)))
        if rng.random() < 0.5:
            c.update(recipe="replaced", replace=n // 10)
    return c


# ------------------------------------------------------------------ inputs

def _data(c, seed):
    """M (m x n), perm and offsets of the blocks, as numpy arrays."""
    rng = np.random.default_rng([seed, c["m"], c["k"], c["ns"]])
    m, n = c["m"], c["k"] * c["ns"]
    if c["recipe"] == "image":
        M = np.empty((m, n))
        for i in range(c["k"]):
            B = rng.uniform(0.0, 2.0 / c["r"], size=(m, c["r"]))
            M[:, i * c["ns"]:(i + 1) * c["ns"]] = np.clip(B @ rng.uniform(0.0, 1.0, size=(c["r"], c["ns"])), 0.0, 1.0)
        for j in rng.choice(n, size=n // 10, replace=False):
            rows = rng.choice(m, size=max(1, m // 10), replace=False)
            M[rows, j] = rng.uniform(0.0, 1.0, size=rows.size)
    else:
        M, _, _ = datagen.union_of_subspaces(rng, m=m, k=c["k"], r=c["r"], ns=c["ns"], n_replace=c["replace"])
    if c["recipe"] == "unit":
        M /= np.linalg.norm(M, axis=0, keepdims=True)
        idx = rng.choice(n, size=max(1, n // 20), replace=False)
        g = rng.standard_normal((m, idx.size))
        M[:, idx] += 0.3 * g / np.linalg.norm(g, axis=0, keepdims=True)
    if c["kind"] in ("dfc", "local", "grad"):
        t = max(1, round(2 * n / (c["lo"] + c["hi"])))
        if c["lo"] == c["hi"]:
            perm, offsets = datagen.equal_partition(rng, n, t)
        else:
            perm, offsets = datagen.uneven_partition(rng, n, t, c["lo"], c["hi"])
    else:
        perm, offsets = np.arange(n, dtype=np.int32), np.array([0, n], dtype=np.int32)
    if c["dtype"] == "float32":
        M = M.astype(np.float32).astype(np.float64)
    return M, perm, offsets


def _lam(c, M, perm, offsets):
    """The case's regulariser; 0 asks for three times the value below which some
    block's solution is Z = 0, to three digits (how workload 4's was chosen)."""
    if c["lam"]:
        return c["lam"]
    G, worst = M @ M.T, 0.0
    for b in range(len(offsets) - 1):
        X = M[:, perm[offsets[b]:offsets[b + 1]]]
        X = X / np.linalg.norm(X, axis=0, keepdims=True)
        v = np.ones(X.shape[1])
        for _ in range(60):
            v = X.T @ (G @ (X @ v))
            s = np.linalg.norm(v)
            v /= s
        worst = max(worst, 1.0 / math.sqrt(s))
    return float("%.3g" % (3.0 * worst))


def _coefficients(c, M, seed):
    """A coefficient matrix of the form a solve returns: the shape interaction
    matrix of the data (the closed-form solution on clean data), its singular
    values spread below one as a threshold leaves them."""
    G = torch.from_numpy(M @ M.T)
    lam, W = torch.linalg.eigh(G)
    keep = lam > 1e-10 * lam[-1]
    if c["recipe"] == "unit":   # the clean subspaces only
        keep &= torch.arange(len(lam)) >= len(lam) - c["k"] * c["r"]
    Mt = torch.from_numpy(np.ascontiguousarray(M.T)).cuda()
    V = Mt @ (W[:, keep] / torch.sqrt(lam[keep])).cuda()
    s = torch.from_numpy(np.random.default_rng([seed, 7]).uniform(0.5, 1.0, int(keep.sum()))).cuda()
    return Mt, (V @ (s[:, None] * V.T)).contiguous()


def prepare(c, seed):
    M, perm, offsets = _data(c, seed)
    s = dict(case=c, perm=perm, offsets=offsets)
    if c["kind"] in ("segment", "slr"):
        s["Mt"], s["Zt"] = _coefficients(c, M, seed)
        return s
    s["lam"] = _lam(c, M, perm, offsets)
    s["Mt"] = torch.from_numpy(np.ascontiguousarray(M.T)).cuda()
    if c["dtype"] == "float32":
        s["Mt"] = s["Mt"].float()
    if c["kind"] == "grad":
        W = np.random.default_rng([seed, 5]).uniform(0.0, 1.0, size=(M.shape[1], M.shape[1]))
        s["W2"] = torch.from_numpy(W * W).cuda()
        s["Mt"].requires_grad_(True)
        s["lam"] = torch.tensor(s["lam"], dtype=torch.float64, device="cuda", requires_grad=True)
        s["opts"] = binding.lrr_opts_default(fixed_iters=c["fixed_iters"], checkpoint_every=20)
    else:
        s["opts"] = binding.lrr_opts_default(precision=c["precision"], tol=c["tol"])
    return s


# -------------------------------------------------------------------- calls

def run(s):
    c, kind = s["case"], s["case"]["kind"]
    if kind == "lrr":
        Zt, Et, _ = binding.lrr_solve(s["Mt"], s["Mt"], s["lam"], s["opts"])
        return Zt, Et
    if kind == "dfc":
        Zt, St, _ = binding.dfc_lrr_solve(s["Mt"], s["lam"], s["perm"], s["offsets"], s["opts"])
        return Zt, St
    if kind == "local":
        Zt, St, _ = binding.dfc_lrr_solve_local(s["Mt"], s["lam"], s["perm"], s["offsets"], 0, s["opts"])
        return Zt, St
    if kind == "grad":
        Zt = autograd.dfc_lrr(s["Mt"], s["lam"], s["perm"], s["offsets"], s["opts"])
        Z = Zt.detach()   # the loss sum(W^2 Z^2)
        dM, dlam = torch.autograd.grad(Zt, (s["Mt"], s["lam"]), grad_outputs=2.0 * s["W2"] * Z)
        return Z, dM, dlam
    if kind == "segment":
        n = s["Zt"].shape[0]
        bound = 0 if n <= 4000 else c["k"] * c["r"]
        labels, info = binding.lrr_segment(s["Zt"], c["k"], rank_bound=bound)
        return labels, info["rank"], info["theta_k"]
    nbr, w, obj, _ = binding.lrr_slr_graph(s["Mt"], s["Zt"], c["nk"])
    return nbr, w, obj


def work(c):
    """Inputs read once and outputs written once; per iteration of a solve one
    Gram product and one reconstruction per block (of order min(m, n) x width),
    per reverse step twice that; products of the affinity or of M^T M else."""
    m, n = c["m"], c["k"] * c["ns"]
    e = 4 if c["dtype"] == "float32" else 8
    if c["kind"] == "segment":
        return {"bytes": 8.0 * n * n + 8.0 * n, "flops": 2.0 * n * n * c["k"] * c["r"]}
    if c["kind"] == "slr":
        return {"bytes": 8.0 * (m * n + n * n) + 12.0 * n * c["nk"], "flops": 1.0 * n * n * m}
    width = 0.5 * (c["lo"] + c["hi"])
    flops = 4.0 * min(m, n) * n * width * (c["fixed_iters"] or ITERS)
    if c["kind"] == "grad":
        return {"bytes": 8.0 * (2 * m * n + 2 * n * n), "flops": 3.0 * flops}
    return {"bytes": e * (2.0 * m * n + n * n), "flops": flops}


# ------------------------------------------------- 64-bit values, numpy only

def _alm(A, X, lam, tol):
    """Inexact ALM of Eq. (2): J, Z, E, the last threshold's left basis and weights."""
    n, l = A.shape[1], X.shape[1]
    inv = np.linalg.inv(np.eye(n) + A.T @ A)
    Z, E, Y1, Y2 = np.zeros((n, l)), np.zeros_like(X), np.zeros_like(X), np.zeros((n, l))
    mu = 1e-6
    for _ in range(1000):
        U, sv, Vt = np.linalg.svd(Z + Y2 / mu, full_matrices=False)
        U, sv, Vt = U[:, sv > 1 / mu], sv[sv > 1 / mu] - 1 / mu, Vt[sv > 1 / mu]
        J = (U * sv) @ Vt
        Z = inv @ (A.T @ (X - E + Y1 / mu) + J - Y2 / mu)
        Q = X - A @ Z + Y1 / mu
        nrm = np.linalg.norm(Q, axis=0)
        E = Q * np.where(nrm > lam / mu, 1 - (lam / mu) / np.maximum(nrm, 1e-300), 0.0)
        R1, R2 = X - A @ Z - E, Z - J
        Y1, Y2, mu = Y1 + mu * R1, Y2 + mu * R2, min(1.1 * mu, 1e10)
        if np.abs(R1).max() < tol and np.abs(R2).max() < tol:
            break
    return Z, E, J, U, sv, Vt


def exact(c, seed):
    n = c["k"] * c["ns"]
    # larger ones take the plain iteration minutes; the other kinds return whole
    # numbers, or have no short form
    if c["kind"] not in ("lrr", "dfc", "local") or n > 260 or c["m"] > 260 or c["precision"]:
        return None
    M, perm, offsets = _data(c, seed)
    lam = _lam(c, M, perm, offsets)
    blocks = [perm[offsets[b]:offsets[b + 1]] for b in range(len(offsets) - 1)]
    if c["kind"] == "lrr":
        Z, E = _alm(M, M, lam, c["tol"])[:2]
        return Z.T.copy(), E.T.copy()
    Z, S = np.zeros((n, n)), np.zeros(M.shape)
    if c["kind"] == "dfc":
        U1 = None
        for cols in blocks:
            _, E, J, U, _, _ = _alm(M, M[:, cols], lam, c["tol"])
            U1 = U if U1 is None else U1
            Z[:, cols], S[:, cols] = U1 @ (U1.T @ J), E
        return Z.T.copy(), S.T.copy()
    parts = [_alm(M[:, cols], M[:, cols], lam, c["tol"]) for cols in blocks]
    rank = max(len(p[4]) for p in parts)   # the combine keeps this many triplets over all blocks
    every = np.sort(np.concatenate([p[4] for p in parts]))[::-1]
    cut = every[rank - 1] if rank else np.inf
    for cols, (_, E, _, U, sv, Vt) in zip(blocks, parts):
        keep = sv >= cut
        Z[np.ix_(cols, cols)], S[:, cols] = (U[:, keep] * sv[keep]) @ Vt[keep], E
    return Z.T.copy(), S.T.copy()
