"""The iteration in singular coordinates (reduced coordinates with the dictionary
diagonalised) against the FP64 oracle, at the edges of its column pass: a wave
per column up to 512 rows in chunks of 128, a workgroup beyond, odd and even row
counts, and the dictionaries and observations that have to take the dense form.

Tolerances: the parity bar of the solver (1e-6) on Z and S; the primal residual
after a fixed number of iterations, while it is far above the rounding of the
O(1) quantities it is the difference of, to 1e-6 of its value.
"""
import numpy as np
import pytest

from gpu_util import need_gpu, one_thread, rel, say

pytestmark = pytest.mark.gpu


def _run(p, **kw):
    from paper_1304_5583_amd import binding as B
    o = B.lrr_opts_default(coords=B.LRR_COORDS_REDUCED, **kw)
    Zt, St, info = B.dfc_lrr_solve(B.to_device_colmajor(p.M), p.lam, p.perm, p.offsets, opts=o)
    return B.from_device_colmajor(Zt), B.from_device_colmajor(St), info


@pytest.mark.parametrize("m,ns,t", [(127, 48, 5), (128, 48, 5), (129, 48, 5), (257, 96, 9), (512, 180, 17),
                                    (513, 180, 17)])
def test_row_counts_vs_oracle(m, ns, t):
    import oracle
    from paper_1304_5583_amd.datagen import small_problem
    need_gpu()
    # noise on every column makes the rank min(m, n)
    n = 3 * ns
    p = small_problem(900 + m, m=m, k=3, r=4, ns=ns, n_replace=0, t=t, lam=0.2, uneven=(n // t - 3, n // t + 4),
                      normalize=True)
    rng = np.random.default_rng(m)
    p.M[:] += 0.02 / np.sqrt(m) * rng.standard_normal(p.M.shape)
    say(f"[svd rows] m={p.m} n={p.n} t={p.t}")
    Z, S, info = _run(p, max_iter=400)
    with one_thread():
        ref = oracle.dfc_lrr(p.M, p.lam, p.perm, p.offsets)
    assert info.status == 0
    assert info.iters.tolist() == [b.iters for b in ref.blocks]
    assert info.rank.tolist() == [b.rank for b in ref.blocks]
    assert rel(Z, ref.Z) <= 1e-6
    assert rel(S, ref.S) <= 1e-6 or np.linalg.norm(ref.S) == 0.0


@pytest.mark.parametrize("iters", [1, 2, 61, 128])
def test_fixed_iterations_report_the_last_residual(iters):
    from oracle.lrr import ALMOptions, dfc_lrr
    from paper_1304_5583_amd.datagen import small_problem
    need_gpu()
    p = small_problem(77, m=45, k=4, r=3, ns=33, n_replace=5, t=4, lam=0.25, uneven=(28, 40), normalize=True)
    Z, S, info = _run(p, fixed_iters=iters)
    with one_thread():
        ref = dfc_lrr(p.M, p.lam, p.perm, p.offsets, ALMOptions(fixed_iters=iters))
    assert info.iters.tolist() == [iters] * p.t
    np.testing.assert_allclose(info.res_primal, [b.res1 for b in ref.blocks], rtol=1e-6)
    assert np.linalg.norm(Z - ref.Z) <= 1e-6 * max(np.linalg.norm(ref.Z), 1e-300)
    assert np.linalg.norm(S - ref.S) <= 1e-6 * max(np.linalg.norm(ref.S), 1e-300)


def test_more_rows_than_a_wave_holds():
    """1030 and 2050 rows (the workgroup-per-column pass): against full coordinates
    of the same library, whose column kernels are separate."""
    from paper_1304_5583_amd import binding as B
    need_gpu()
    for m in (1030, 2050):
        rng = np.random.default_rng(m)
        n = m + 46
        M = rng.standard_normal((m, 12)) @ rng.standard_normal((12, n)) + 0.05 * rng.standard_normal((m, n))
        M /= np.linalg.norm(M, axis=0)
        offs = np.arange(0, n + 1, n // 12, dtype=np.int32)
        offs[-1] = n
        perm = rng.permutation(n).astype(np.int32)
        Mt = B.to_device_colmajor(M)
        out = {}
        for coords in (B.LRR_COORDS_FULL, B.LRR_COORDS_REDUCED):
            o = B.lrr_opts_default(coords=coords, fixed_iters=130)
            Zt, St, info = B.dfc_lrr_solve(Mt, 0.15, perm, offs, opts=o)
            out[coords] = (B.from_device_colmajor(Zt), B.from_device_colmajor(St), info)
        a, b = out[B.LRR_COORDS_FULL], out[B.LRR_COORDS_REDUCED]
        say(f"[svd rows] m={m} relZ={rel(b[0], a[0]):.2e}")
        assert rel(b[0], a[0]) <= 1e-6 and rel(b[1], a[1]) <= 1e-6
        assert b[2].rank.tolist() == a[2].rank.tolist()
        np.testing.assert_allclose(b[2].res_primal, a[2].res_primal, rtol=1e-6)


def test_observations_outside_the_dictionary_range():
    """lrr_solve with X partly outside range(A): one more coordinate carries that part."""
    from oracle.lrr import lrr_alm
    from paper_1304_5583_amd import binding as B
    need_gpu()
    rng = np.random.default_rng(5)
    A = rng.standard_normal((40, 6)) @ rng.standard_normal((6, 90))
    A /= np.linalg.norm(A, axis=0)
    X = A[:, :30] + 0.1 * rng.standard_normal((40, 30)) / np.sqrt(40)
    Zt, Et, info = B.lrr_solve(B.to_device_colmajor(A), B.to_device_colmajor(X), 0.3)
    with one_thread():
        ref = lrr_alm(X, A, 0.3)
    assert info.iters[0] == ref.iters
    assert rel(B.from_device_colmajor(Zt), ref.Z) <= 1e-6
    assert rel(B.from_device_colmajor(Et), ref.E) <= 1e-6


def test_wide_singular_spread_vs_full_coordinates():
    """Singular values over six decades, all above the rank cut."""
    from paper_1304_5583_amd import binding as B
    need_gpu()
    rng = np.random.default_rng(9)
    m, n = 48, 120
    U, _ = np.linalg.qr(rng.standard_normal((m, m)))
    V, _ = np.linalg.qr(rng.standard_normal((n, m)))
    M = (U * np.logspace(0, -6, m)) @ V.T
    offs, perm = np.array([0, 40, 80, 120], dtype=np.int32), rng.permutation(n).astype(np.int32)
    out = []
    for coords in (B.LRR_COORDS_FULL, B.LRR_COORDS_REDUCED):
        o = B.lrr_opts_default(coords=coords, fixed_iters=110)
        Zt, St, info = B.dfc_lrr_solve(B.to_device_colmajor(M), 0.5, perm, offs, opts=o)
        out.append((B.from_device_colmajor(Zt), B.from_device_colmajor(St)))
    assert rel(out[1][0], out[0][0]) <= 1e-6 and rel(out[1][1], out[0][1]) <= 1e-6


@pytest.mark.parametrize("tail,reduced", [(0.0, True), (1e-9, False)])
def test_auto_keeps_full_coordinates_where_reduced_ones_drop_data(tail, reduced):
    """m < n < 2m: AUTO gives the reduced form's result bit for bit where the basis
    holds the data to rounding, the full form's where directions of 1e-9 of the
    data would be dropped."""
    from paper_1304_5583_amd import binding as B
    need_gpu()
    rng = np.random.default_rng(21)
    m, n = 60, 90
    M = rng.standard_normal((m, 20)) @ rng.standard_normal((20, n))
    M /= np.linalg.norm(M, axis=0)
    M += tail * rng.standard_normal((m, n))
    perm, offs = rng.permutation(n).astype(np.int32), np.array([0, 30, 60, 90], dtype=np.int32)
    out = {}
    for coords in (B.LRR_COORDS_AUTO, B.LRR_COORDS_FULL, B.LRR_COORDS_REDUCED):
        Zt, St, _ = B.dfc_lrr_solve(B.to_device_colmajor(M), 0.3, perm, offs, opts=B.lrr_opts_default(coords=coords))
        out[coords] = (B.from_device_colmajor(Zt), B.from_device_colmajor(St))
    same = B.LRR_COORDS_REDUCED if reduced else B.LRR_COORDS_FULL
    assert np.array_equal(out[B.LRR_COORDS_AUTO][0], out[same][0])
    assert np.array_equal(out[B.LRR_COORDS_AUTO][1], out[same][1])
    assert rel(out[B.LRR_COORDS_REDUCED][0], out[B.LRR_COORDS_FULL][0]) <= 1e-6


@pytest.mark.parametrize("r", [1, 16, 17, 32, 33, 64, 65, 96, 97])
@pytest.mark.parametrize("wide", [True, False])
def test_small_gram_orders_vs_oracle(r, wide):
    """Gram orders around the tile and workgroup sizes of the in-LDS eigensolver (up
    to 96) and the first order beyond it, as Y Y^T (blocks wider than the rank) and
    as Y^T Y (blocks of r columns)."""
    import oracle
    from paper_1304_5583_amd import binding as B
    need_gpu()
    rng = np.random.default_rng(300 + r)
    rank, n = (r, 3 * r + 3) if wide else (2 * r + 1, 5 * r + 3)
    M = rng.standard_normal((rank + 2, rank)) @ rng.standard_normal((rank, n))
    M /= np.linalg.norm(M, axis=0)
    width = (n + 1) // 2 if wide else r
    offs = np.append(np.arange(0, n, width), n).astype(np.int32)
    perm = rng.permutation(n).astype(np.int32)
    o = B.lrr_opts_default(coords=B.LRR_COORDS_REDUCED)
    Zt, St, info = B.dfc_lrr_solve(B.to_device_colmajor(M), 0.4, perm, offs, opts=o)
    with one_thread():
        ref = oracle.dfc_lrr(M, 0.4, perm, offs)
    say(f"[gram order {r} wide={wide}] iters {info.iters.tolist()} oracle {[b.iters for b in ref.blocks]}")
    assert info.iters.tolist() == [b.iters for b in ref.blocks]
    assert info.rank.tolist() == [b.rank for b in ref.blocks]
    assert info.batch_iters == max(b.iters for b in ref.blocks)
    assert np.linalg.norm(B.from_device_colmajor(Zt) - ref.Z) <= 1e-6 * max(np.linalg.norm(ref.Z), 1e-300)
    assert np.linalg.norm(B.from_device_colmajor(St) - ref.S) <= 1e-6 * max(np.linalg.norm(ref.S), 1e-300)


def test_small_gram_orders_same_in_every_mode():
    """The four ways of issuing an iteration, and reads of the flags every 1 or 5
    iterations, give the same bits on blocks that the in-LDS eigensolver takes."""
    from paper_1304_5583_amd import binding as B
    from paper_1304_5583_amd.datagen import small_problem
    need_gpu()
    p = small_problem(31, m=50, k=3, r=4, ns=40, n_replace=9, t=3, lam=0.3, uneven=(36, 44))
    Mt = B.to_device_colmajor(p.M)
    first = None
    for kw in (dict(use_graph=0), dict(use_graph=1), dict(use_graph=2), dict(use_graph=3),
               dict(use_graph=1, check_every=5)):
        Zt, St, info = B.dfc_lrr_solve(Mt, p.lam, p.perm, p.offsets, opts=B.lrr_opts_default(**kw))
        got = (B.from_device_colmajor(Zt), B.from_device_colmajor(St), info.iters.tolist())
        every = kw.get("check_every", 1)
        assert info.batch_iters == -(-max(info.iters) // every) * every
        if first is None:
            first = got
        assert np.array_equal(got[0], first[0]) and np.array_equal(got[1], first[1]) and got[2] == first[2]


@pytest.mark.parametrize("m,widths,ranks", [
    (40, (17, 30, 1), (3, 5, 1)),            # rank below width, one single point
    (24, (31, 60, 25), (4, 24, 9)),          # wider than tall; one block of full row rank
    (150, (130, 97, 140), (130, 97, 140)),   # full column rank: the other Gram side, over 96 points
    (150, (170, 97, 260), (131, 20, 101)),   # odd row count, over 96 rows
])
def test_local_dictionaries_vs_full_coordinates(m, widths, ranks):
    """Every block in the singular coordinates of its own points (ranks of the blocks
    differ, rows beyond a block's rank stay zero) against the same solve in full
    coordinates, which factor I + C C^T instead."""
    from paper_1304_5583_amd import binding as B
    need_gpu()
    rng = np.random.default_rng(m + len(widths) + widths[0])
    M = np.concatenate([rng.standard_normal((m, r)) @ rng.standard_normal((r, w)) for w, r in zip(widths, ranks)], 1)
    M /= np.linalg.norm(M, axis=0)
    M[:, 0] *= 3.0
    offs = np.concatenate([[0], np.cumsum(widths)]).astype(np.int32)
    n = int(offs[-1])
    perm = rng.permutation(n).astype(np.int32)
    Mp = np.empty_like(M)
    Mp[:, perm] = M
    Mt = B.to_device_colmajor(Mp)
    out = []
    for coords in (B.LRR_COORDS_AUTO, B.LRR_COORDS_FULL):
        Zt, St, info = B.dfc_lrr_solve_local(Mt, 0.3, perm, offs, combine_rank=-1,
                                             opts=B.lrr_opts_default(coords=coords))
        out.append((B.from_device_colmajor(Zt), B.from_device_colmajor(St), info))
    (Z, S, a), (Zf, Sf, f) = out
    say(f"[local svd] m={m} relZ={rel(Z, Zf):.2e} iters={a.iters.tolist()} {f.iters.tolist()} rank={a.rank.tolist()}")
    assert a.status == 0 and f.status == 0
    assert a.iters.tolist() == f.iters.tolist()
    assert a.rank.tolist() == f.rank.tolist() and a.combine_rank == f.combine_rank
    assert rel(Z, Zf) <= 1e-6
    assert rel(S, Sf) <= 1e-6 or np.linalg.norm(Sf) <= 1e-6


@pytest.mark.parametrize("m,ns,t", [(140, 160, 2), (260, 150, 3)])
def test_launch_forms_agree_above_the_small_orders(m, ns, t):
    """Gram orders above 96, where the Jacobi rounds run pair solves and tile updates
    in one launch: the same bits as the persistent eigensolve (use_graph 2), whose
    rounds take the two phases one after the other."""
    from paper_1304_5583_amd import binding as B
    from paper_1304_5583_amd.datagen import small_problem
    need_gpu()
    p = small_problem(40 + m, m=m, k=3, r=4, ns=ns, n_replace=ns // 2, t=t, lam=0.25, normalize=True)
    Mt = B.to_device_colmajor(p.M)
    out = [B.dfc_lrr_solve(Mt, p.lam, p.perm, p.offsets, opts=B.lrr_opts_default(use_graph=g, check_every=4))
           for g in (1, 2)]
    assert out[0][2].iters.tolist() == out[1][2].iters.tolist()
    assert (out[0][0] == out[1][0]).all() and (out[0][1] == out[1][1]).all()


@pytest.mark.parametrize("m,n,cond", [(40, 100, 5.0), (130, 300, 6.0), (130, 200, 6.0)])
def test_full_row_rank_with_small_singular_values(m, n, cond):
    """Full row rank with singular values over many decades: the left basis spans the
    whole space, so observations have no part outside it and no coordinate may be
    added for one; against full coordinates of the same solve."""
    from paper_1304_5583_amd import binding as B
    need_gpu()
    rng = np.random.default_rng(m + n)
    U, _ = np.linalg.qr(rng.standard_normal((m, m)))
    V, _ = np.linalg.qr(rng.standard_normal((n, m)))
    M = (U * np.logspace(0.0, -cond, m)) @ V.T * 10.0
    perm = rng.permutation(n).astype(np.int32)
    offs = np.array([0, n // 2, n], dtype=np.int32)
    out = []
    for coords in (B.LRR_COORDS_AUTO, B.LRR_COORDS_REDUCED, B.LRR_COORDS_FULL):
        Zt, _, info = B.dfc_lrr_solve(B.to_device_colmajor(M), 0.5, perm, offs,
                                      opts=B.lrr_opts_default(coords=coords, tol=1e-7))
        assert info.status == 0
        out.append(B.from_device_colmajor(Zt))
    say(f"[full row rank] m={m} n={n} auto {rel(out[0], out[2]):.2e} reduced {rel(out[1], out[2]):.2e}")
    assert rel(out[0], out[2]) <= 1e-6 and rel(out[1], out[2]) <= 1e-6


# 16: the whole end of an iteration in one launch; 60: one launch per expansion;
# 300: expansions by products
SMALLEST_PENALTY = [(16, 40, 20), (60, 130, 100), (300, 700, 400)]


def _smallest_penalty(m, n, l, coords):
    from paper_1304_5583_amd import binding as B
    need_gpu()
    A = np.random.default_rng(m).standard_normal((m, n))
    A /= np.linalg.norm(A, axis=0)
    Zt, Et, info = B.lrr_solve(B.to_device_colmajor(A), B.to_device_colmajor(A[:, :l]), 0.3,
                               B.lrr_opts_default(coords=coords, mu0=1e-310, rho=10.0))
    return B.from_device_colmajor(Zt), B.from_device_colmajor(Et), info


@pytest.mark.parametrize("m,n,l", SMALLEST_PENALTY)
def test_a_solve_that_meets_nan_does_not_converge(m, n, l):
    """A penalty whose reciprocal overflows: whatever becomes of the iterates, LRR_OK is
    not returned with anything but finite numbers."""
    from paper_1304_5583_amd import binding as B
    Z, E, info = _smallest_penalty(m, n, l, B.LRR_COORDS_REDUCED)
    assert info.status != 0 or (np.isfinite(Z).all() and np.isfinite(E).all())


@pytest.mark.parametrize("m,n,l", SMALLEST_PENALTY)
def test_smallest_penalties_vs_full_coordinates(m, n, l):
    """... and the solve is that of full coordinates, which divide by the penalty."""
    from paper_1304_5583_amd import binding as B
    Z, E, info = _smallest_penalty(m, n, l, B.LRR_COORDS_REDUCED)
    Zf, Ef, full = _smallest_penalty(m, n, l, B.LRR_COORDS_FULL)
    assert info.status == 0 and full.status == 0
    assert info.iters.tolist() == full.iters.tolist()
    assert rel(Z, Zf) <= 1e-6 and np.linalg.norm(E - Ef) <= 1e-6 * max(np.linalg.norm(Ef), 1.0)


def test_float32_buffers_drop_nothing_of_the_dictionary():
    """m < n < 2m with float32 buffers: data rounded to float32 hold directions of 1e-8
    of their size, below the rank cut of the bases; AUTO keeps them (full coordinates,
    bit for bit), as it does for the same numbers in float64 buffers."""
    from paper_1304_5583_amd import binding as B
    need_gpu()
    rng = np.random.default_rng(21)
    m, n = 60, 90
    M = rng.standard_normal((m, 20)) @ rng.standard_normal((20, n))
    M /= np.linalg.norm(M, axis=0)
    perm, offs = rng.permutation(n).astype(np.int32), np.array([0, 30, 60, 90], dtype=np.int32)
    Mt = B.to_device_colmajor(M).float()
    for X in (Mt, Mt.double()):
        auto, full = (B.dfc_lrr_solve(X, 0.3, perm, offs, opts=B.lrr_opts_default(coords=c))
                      for c in (B.LRR_COORDS_AUTO, B.LRR_COORDS_FULL))
        assert (auto[0] == full[0]).all() and (auto[1] == full[1]).all()


@pytest.mark.parametrize("kw,reduced", [(dict(fixed_iters=60), False), (dict(fixed_iters=128), True), (dict(max_iter=127), False),
                                        (dict(rho=1.5), False), (dict(), True)])
def test_short_solves_do_without_a_basis(kw, reduced):
    """m < n < 2m, and a dictionary per block: AUTO builds a basis only where the limits
    and the penalty schedule leave enough iterations for it; the result then is the
    explicit form's bit for bit."""
    from paper_1304_5583_amd import binding as B
    need_gpu()
    rng = np.random.default_rng(22)
    m, n = 60, 90
    M = rng.standard_normal((m, 20)) @ rng.standard_normal((20, n))
    M /= np.linalg.norm(M, axis=0)
    perm, offs = rng.permutation(n).astype(np.int32), np.array([0, 30, 60, 90], dtype=np.int32)
    Mt = B.to_device_colmajor(M)
    same = B.LRR_COORDS_REDUCED if reduced else B.LRR_COORDS_FULL
    auto, form = (B.dfc_lrr_solve(Mt, 0.3, perm, offs, opts=B.lrr_opts_default(coords=c, **kw))
                  for c in (B.LRR_COORDS_AUTO, same))
    assert (auto[0] == form[0]).all() and (auto[1] == form[1]).all()
    auto, full = (B.dfc_lrr_solve_local(Mt, 0.3, perm, offs, combine_rank=-1, opts=B.lrr_opts_default(coords=c, **kw))
                  for c in (B.LRR_COORDS_AUTO, B.LRR_COORDS_FULL))
    assert bool((auto[0] == full[0]).all()) != reduced
    # (the two forms stop in the same iteration, or a fixed one)
    assert auto[2].iters.tolist() == full[2].iters.tolist()


@pytest.mark.parametrize("m,kind,reduced", [(999, "rounded", False), (1000, "rounded", True), (1000, "decades", True),
                                            (1000, "exact rank", True), (999, "exact rank", True)])
def test_directions_below_the_rank_cut_are_kept(m, kind, reduced):
    """m < n < 2m from 1000 rows on: what the first basis leaves of the dictionary (the
    rounding of float32 data; singular values over 12 decades) gets a basis of its own;
    below, such a solve runs in full coordinates, bit for bit."""
    from paper_1304_5583_amd import binding as B
    need_gpu()
    rng = np.random.default_rng(m)
    n = m + 56
    if kind == "decades":
        U = np.linalg.qr(rng.standard_normal((m, 200)))[0]
        V = np.linalg.qr(rng.standard_normal((n, 200)))[0]
        M = 20.0 * (U * np.logspace(0.0, -12.0, 200)) @ V.T
    else:
        M = rng.standard_normal((m, 30)) @ rng.standard_normal((30, n))
        M /= np.linalg.norm(M, axis=0)
        if kind == "rounded":
            M = M.astype(np.float32).astype(np.float64)
    offs = np.array([0, n // 4, n // 2, n // 2 + 100, n], dtype=np.int32)
    perm = rng.permutation(n).astype(np.int32)
    Mt = B.to_device_colmajor(M)
    (Z, S, a), (Zf, Sf, f) = (B.dfc_lrr_solve(Mt, 0.3, perm, offs, opts=B.lrr_opts_default(coords=c))
                              for c in (B.LRR_COORDS_AUTO, B.LRR_COORDS_FULL))
    assert bool((Z == Zf).all()) != reduced
    Z, S, Zf, Sf = (B.from_device_colmajor(x) for x in (Z, S, Zf, Sf))
    say(f"[stages] m={m} {kind} relZ={rel(Z, Zf):.2e} |Z|={np.linalg.norm(Zf):.2e}")
    assert np.linalg.norm(Zf) > 1.0
    assert a.rank.tolist() == f.rank.tolist() and a.iters.tolist() == f.iters.tolist()
    assert rel(Z, Zf) <= 1e-6 and np.linalg.norm(S - Sf) <= 1e-6 * max(np.linalg.norm(Sf), 1.0)
