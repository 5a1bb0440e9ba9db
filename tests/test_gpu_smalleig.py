"""The single-workgroup thresholding step of small Gram orders (lrr_diag_small_svt)
against numpy's eigen-decomposition, where it can go wrong: a block of lower rank
beside one of higher rank.

Tolerances: entries of J are differences of O(1) numbers formed from eigenpairs
that are accurate to 1e-14 of the largest eigenvalue; with tau at a tenth of the
largest singular value the weights 1 - tau / sigma amplify that by at most 100, so
1e-11 of the largest entry.
"""
import numpy as np
import pytest

from gpu_util import need_gpu, say

pytestmark = pytest.mark.gpu


def _svt(Y, tau):
    U, s, Vt = np.linalg.svd(Y, full_matrices=False)
    return (U * np.maximum(s - tau, 0.0)) @ Vt, int((s > tau).sum())


@pytest.mark.parametrize("e,nr,l", [(12, 90, 40), (1, 96, 17), (16, 17, 16), (31, 48, 33), (48, 90, 256), (90, 90, 91),
                                    (64, 65, 80)])
def test_rows_beyond_a_blocks_rank_are_zero(e, nr, l):
    """Blocks with dictionaries of their own share the largest rank as their row
    count: J of a block of rank e has exact zeros in the rows from e on."""
    torch = need_gpu()
    from paper_1304_5583_amd import binding as B
    rng = np.random.default_rng(e + nr + l)
    Y = np.zeros((nr, l))
    Y[:e] = rng.standard_normal((e, l))
    tau = 0.1 * np.linalg.norm(Y, 2)
    Jt = torch.full((l, nr), float("nan"), dtype=torch.float64, device="cuda")
    Jt, lam, Xt, rank = B.lrr_diag_small_svt(e, tau, Yt=torch.from_numpy(np.ascontiguousarray(Y.T)).cuda(), Jt=Jt)
    J = Jt.cpu().numpy().T
    ref, k = _svt(Y, tau)
    say(f"[small svt] e={e} nr={nr} l={l} err={np.abs(J - ref).max():.2e}")
    assert np.all(J[e:] == 0.0)
    assert np.abs(J - ref).max() <= 1e-11 * np.abs(ref).max()
    assert rank == k


def test_local_blocks_of_very_different_ranks():
    """Ranks 12, 48 and 90 in one call: the outputs do not depend on what other
    workgroups left in the LDS, so two calls with other work in between agree bit
    for bit, and with full coordinates to the parity bar."""
    need_gpu()
    from paper_1304_5583_amd import binding as B
    rng = np.random.default_rng(12)
    m, widths, ranks = 100, (40, 60, 100), (12, 48, 90)
    M = np.concatenate([rng.standard_normal((m, r)) @ rng.standard_normal((r, w)) for w, r in zip(widths, ranks)], 1)
    M /= np.linalg.norm(M, axis=0)
    offs = np.concatenate([[0], np.cumsum(widths)]).astype(np.int32)
    perm = np.arange(M.shape[1], dtype=np.int32)
    Mt = B.to_device_colmajor(M)

    def solve(coords):
        Zt, St, info = B.dfc_lrr_solve_local(Mt, 0.3, perm, offs, combine_rank=-1, opts=B.lrr_opts_default(coords=coords))
        return B.from_device_colmajor(Zt), B.from_device_colmajor(St), info
    Z, S, a = solve(B.LRR_COORDS_AUTO)
    # other kernels that fill the LDS: a large eigenproblem and a solve of its own
    G = rng.standard_normal((96, 96))
    B.lrr_diag_small_svt(96, 1.0, Gt=B.to_device_colmajor(G @ G.T))
    Z2, S2, _ = solve(B.LRR_COORDS_AUTO)
    assert np.array_equal(Z, Z2) and np.array_equal(S, S2)
    Zf, Sf, f = solve(B.LRR_COORDS_FULL)
    assert a.iters.tolist() == f.iters.tolist() and a.rank.tolist() == f.rank.tolist()
    assert np.linalg.norm(Z - Zf) <= 1e-6 * np.linalg.norm(Zf)
    assert np.linalg.norm(S - Sf) <= 1e-6 * max(np.linalg.norm(Sf), 1.0)


@pytest.mark.parametrize("upper,lower", [(0.99e-14, 1.01e-14), (1.01e-14, 0.99e-14)])
@pytest.mark.parametrize("e", [20, 50, 96])
def test_halves_on_either_side_of_the_tolerance(e, upper, lower):
    """The two halves of X^T G X differ in the last bits.  A pair of equal eigenvalues
    whose coupling lies above the absolute floor (1e-14 of the largest eigenvalue) in
    one half only, beside a coupling that a first-order correction resolves: the pair
    must not be divided by its distance of zero."""
    torch = need_gpu()
    from paper_1304_5583_amd import binding as B
    d = np.linspace(1.0, 0.3, e)
    d[2] = d[3] = 1e-3
    G = np.diag(d)
    G[0, 5] = G[5, 0] = 1e-6
    G[2, 3], G[3, 2] = upper, lower
    tau = 0.01
    # (e, e) tensor of the column-major G: G[i, j] at [j, i]
    Pt, lam, Xt, rank = B.lrr_diag_small_svt(e, tau, Gt=B.to_device_colmajor(G),
                                             X0t=torch.eye(e, dtype=torch.float64, device="cuda"))
    w, V = np.linalg.eigh(0.5 * (G + G.T))
    ref = (V * np.maximum(1.0 - tau / np.sqrt(w), 0.0)) @ V.T
    X = Xt.cpu().numpy().T
    assert rank == e
    assert np.abs(Pt.cpu().numpy() - ref).max() <= 1e-11
    assert np.abs(X.T @ X - np.eye(e)).max() <= 1e-13


@pytest.mark.parametrize("kind", ["exact", "nan", "inf", "zero", "gaussian", "scaled", "one column lost"])
@pytest.mark.parametrize("e", [7, 40, 96])
def test_eigenvectors_of_an_earlier_step_that_are_not_orthonormal(e, kind):
    """A step that starts from eigenvectors which have lost their orthonormality (or
    are not finite) gives what one from the identity gives."""
    need_gpu()
    from paper_1304_5583_amd import binding as B
    rng = np.random.default_rng(e)
    Y = rng.standard_normal((e, 2 * e))
    G = Y @ Y.T
    w, V = np.linalg.eigh(G)
    tau = 0.1 * np.sqrt(w[-1])
    X0 = {"exact": V, "nan": np.full((e, e), np.nan), "inf": np.where(np.eye(e) > 0, np.inf, 0.0),
          "zero": np.zeros((e, e)), "gaussian": rng.standard_normal((e, e)), "scaled": 2.0 * V,
          "one column lost": np.where(np.arange(e) == 2, V[:, [0]], V)}[kind]
    Pt, lam, Xt, rank = B.lrr_diag_small_svt(e, tau, Gt=B.to_device_colmajor(G), X0t=B.to_device_colmajor(X0))
    ref = (V * np.maximum(1.0 - tau / np.sqrt(np.maximum(w, 1e-300)), 0.0)) @ V.T
    X = Xt.cpu().numpy().T
    assert rank == int((np.sqrt(np.maximum(w, 0.0)) > tau).sum())
    assert np.abs(Pt.cpu().numpy() - ref).max() <= 1e-11
    assert np.abs(X.T @ X - np.eye(e)).max() <= 1e-12


@pytest.mark.parametrize("e", [10, 48, 96])
@pytest.mark.parametrize("warm", [False, True])
def test_couplings_below_the_absolute_floor(e, warm):
    """Kept eigenvalues of 1e-7 and 1e-8 of the largest, coupled by 5e-15 of it: less
    than the floor of the Jacobi rotations, but an angle of 5e-8.  The Gram matrix
    consists of 2 x 2 blocks, whose P has a closed form; what a first-order correction
    leaves is the angle's square, and rounding: 1e-12."""
    torch = need_gpu()
    from paper_1304_5583_amd import binding as B
    import math
    tau = math.sqrt(5e-9)
    G, ref, kept = np.zeros((e, e)), np.zeros((e, e)), 0
    for i in range(0, e, 2):
        a, b, s = (1.0, 0.5, 0.0) if i == 0 else (1e-7 * (1.0 + i / e), 1e-8 * (1.0 + i / e), 5e-15)
        G[i:i + 2, i:i + 2] = [[a, s], [s, b]]
        t = 2.0 * s / ((a - b) + math.hypot(a - b, 2.0 * s))      # tan of the angle
        c = 1.0 / math.sqrt(1.0 + t * t)
        V = np.array([[c, -c * t], [c * t, c]])
        g = [max(1.0 - tau / math.sqrt(x), 0.0) for x in (a + s * t, b - s * t)]
        ref[i:i + 2, i:i + 2] = (V * g) @ V.T
        kept += sum(x > 0.0 for x in g)
    X0 = torch.eye(e, dtype=torch.float64, device="cuda") if warm else None
    Pt, lam, Xt, rank = B.lrr_diag_small_svt(e, tau, Gt=B.to_device_colmajor(G), X0t=X0)
    say(f"[small svt] e={e} below the floor: {np.abs(Pt.cpu().numpy() - ref).max():.2e}")
    assert rank == kept
    assert np.abs(Pt.cpu().numpy() - ref).max() <= 1e-12
