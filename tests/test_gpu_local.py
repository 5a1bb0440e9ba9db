"""GPU parity of the footnote variant of Section 2.2 (dfc_lrr_solve_local).

Every block solves Eq. (1) with its own columns as dictionary, all blocks in the
same batched launches; the C step keeps the k largest singular triplets of
diag(J_1, ..., J_t).  Against the oracle's dfc_lrr_local on the same inputs:
||Z - Z_oracle||_F / ||Z_oracle||_F <= 1e-6 in FP64 (iteration counts within
one); for the reduced-precision forms the bounds the precision tests state for
their worst input class, 1e-4 (FP32) and 5e-4 (split BF16; 1.35e-4 measured on
the case below); the same per-block ranks, the same combine rank, and exact
zeros outside the diagonal blocks.  The full-size workload 2 is compared with
the stored oracle fingerprint.
"""
import json
import os

import numpy as np
import pytest

from gpu_util import need_gpu, one_thread, rel, say

pytestmark = pytest.mark.gpu

GOLD = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden")


def _small(seed, **kw):
    from paper_1304_5583_amd.datagen import small_problem
    return small_problem(seed, **kw)


def _inside(p):
    n = p.n
    mask = np.zeros((n, n), dtype=bool)
    for i in range(len(p.offsets) - 1):
        cols = p.perm[p.offsets[i]:p.offsets[i + 1]]
        mask[np.ix_(cols, cols)] = True
    return mask


CASES = [
    # seed, problem kwargs, combine rank, precision, tolerance
    (51, dict(m=40, k=3, r=3, ns=30, n_replace=6, t=1), -1, 0, 1e-6),
    (52, dict(m=48, k=4, r=3, ns=25, n_replace=10, t=3, uneven=(28, 38)), 0, 0, 1e-6),
    (53, dict(m=64, k=3, r=4, ns=40, n_replace=8, t=4, lam=0.3), 7, 0, 1e-6),
    (54, dict(m=30, k=3, r=2, ns=30, n_replace=6, t=2, lam=0.35), -1, 0, 1e-6),
    (55, dict(m=64, k=3, r=4, ns=40, n_replace=8, t=3, lam=0.3), 0, 1, 1e-4),
    (55, dict(m=64, k=3, r=4, ns=40, n_replace=8, t=3, lam=0.3), 0, 2, 5e-4),
]


@pytest.mark.parametrize("seed,kw,rank,prec,tol", CASES)
def test_local_matches_oracle(seed, kw, rank, prec, tol):
    need_gpu()
    import oracle
    from paper_1304_5583_amd import binding as B
    p = _small(seed, **kw)
    o = B.lrr_opts_default(precision=prec)
    Zt, St, info = B.dfc_lrr_solve_local(B.to_device_colmajor(p.M), p.lam, p.perm, p.offsets,
                                         combine_rank=rank, opts=o)
    Zg, Sg = B.from_device_colmajor(Zt), B.from_device_colmajor(St)
    with one_thread():
        ref = oracle.dfc_lrr_local(p.M, p.lam, p.perm, p.offsets, rank=rank)
    it_o = np.array([b.iters for b in ref.blocks])
    rk_o = np.array([b.rank for b in ref.blocks])
    ez, es = rel(Zg, ref.Z), rel(Sg, ref.S)
    say(f"[local s{seed}] t={p.t} widths={np.diff(p.offsets).tolist()} k={info.combine_rank}/{ref.combine_rank} "
        f"relZ={ez:.2e} relS={es:.2e} iters gpu={info.iters.tolist()} oracle={it_o.tolist()} "
        f"rank gpu={info.rank.tolist()} oracle={rk_o.tolist()}")
    assert info.status == 0
    assert ez <= tol and es <= tol
    assert np.array_equal(info.rank, rk_o)
    assert info.combine_rank == ref.combine_rank
    if prec == 0:
        assert np.all(np.abs(info.iters - it_o) <= 1)
    assert np.all(Zg[~_inside(p)] == 0.0)


def test_local_single_block_equals_plain_lrr():
    """t = 1, no truncation: the local variant is plain LRR of M with M as its own
    dictionary, i.e. J of lrr_solve(X = M, A = M), up to the point order."""
    need_gpu()
    from paper_1304_5583_amd import binding as B
    p = _small(56, m=40, k=3, r=3, ns=25, n_replace=5, t=1)
    Mt = B.to_device_colmajor(p.M)
    Zt, _, info = B.dfc_lrr_solve_local(Mt, p.lam, p.perm, p.offsets, combine_rank=-1)
    Zd, _, _ = B.dfc_lrr_solve(Mt, p.lam, np.arange(p.n), np.array([0, p.n]))
    assert rel(B.from_device_colmajor(Zt), B.from_device_colmajor(Zd)) <= 1e-9


def test_local_errors():
    need_gpu()
    from paper_1304_5583_amd import binding as B
    p = _small(57, m=20, k=2, r=2, ns=15, n_replace=2, t=2)
    Mt = B.to_device_colmajor(p.M)
    with pytest.raises(B.LRRError) as e:
        B.dfc_lrr_solve_local(Mt, p.lam, p.perm, p.offsets, opts=B.lrr_opts_default(save_for_backward=1,
                                                                                       fixed_iters=5))
    assert e.value.status == B.LRR_EINVAL
    with pytest.raises(B.LRRError) as e:
        B.dfc_lrr_solve_local(Mt, -1.0, p.perm, p.offsets)
    assert e.value.status == B.LRR_EINVAL


def test_workload2_local_matches_stored_oracle():
    """Workload 2 at full size (t = 4 blocks of 500 columns, each its own
    dictionary) against the stored oracle fingerprint: Z at probe vectors and
    positions, norms, iterations within one, ranks and combine rank."""
    need_gpu()
    from paper_1304_5583_amd import binding as B
    from paper_1304_5583_amd.datagen import make_config
    path = os.path.join(GOLD, "workload2_local_oracle.json")
    g = json.load(open(path))
    p = make_config(2)
    Zt, St, info = B.dfc_lrr_solve_local(B.to_device_colmajor(p.M), p.lam, p.perm, p.offsets)
    Zg = B.from_device_colmajor(Zt)
    rng = np.random.default_rng(4242)
    W = rng.standard_normal((p.n, 2))
    idx = rng.integers(0, p.n, size=(512, 2))
    ezw = rel((Zg @ W).T, np.array(g["Zw"]))
    zat = np.array([Zg[i, j] for i, j in idx])
    ezat = float(np.abs(zat - np.array(g["Z_at"])).max() / np.abs(Zg).max())
    say(f"[local wl2] relZw={ezw:.2e} maxZat={ezat:.2e} iters gpu={info.iters.tolist()} oracle={g['iters']} "
        f"rank gpu={info.rank.tolist()} oracle={g['rank']} k={info.combine_rank}/{g['combine_rank']}")
    assert info.status == 0
    assert ezw <= 1e-6 and ezat <= 1e-6
    assert abs(np.linalg.norm(Zg) - g["Z_fro"]) <= 1e-6 * g["Z_fro"]
    assert np.all(np.abs(info.iters - np.array(g["iters"])) <= 1)
    assert info.rank.tolist() == g["rank"]
    assert info.combine_rank == g["combine_rank"]


def test_local_reduced_and_tuned_calls_take_the_automatic_form(tmp_path):
    """coords REDUCED is AUTO where every block has its own dictionary, and the schedule
    table, measured with the common dictionary, does not set coords: the same bits."""
    torch = need_gpu()
    from paper_1304_5583_amd import binding as B
    p = _small(58, m=64, k=3, r=4, ns=40, n_replace=8, t=3, lam=0.3)
    Mt = B.to_device_colmajor(p.M)
    ctx = B.Context(0)

    def solve(**kw):
        return B.dfc_lrr_solve_local(Mt, p.lam, p.perm, p.offsets, combine_rank=-1, opts=B.lrr_opts_default(**kw),
                                     ctx=ctx)
    auto, full = solve(), solve(coords=B.LRR_COORDS_FULL)
    assert not torch.equal(auto[0], full[0])     # two forms
    assert rel(auto[0].cpu().numpy(), full[0].cpu().numpy()) <= 1e-6
    red = solve(coords=B.LRR_COORDS_REDUCED)
    assert torch.equal(red[0], auto[0]) and torch.equal(red[1], auto[1])
    maxl = int(np.diff(p.offsets).max())
    for co in (1, 2):
        path = tmp_path / f"table{co}.txt"
        path.write_text(f"{p.m} {p.n} {p.t} {maxl} 0 16 0 4 {co}\n")
        B.lrr_tune_load(str(path), ctx=ctx)
        tuned = solve(tune=1)
        assert torch.equal(tuned[0], auto[0]) and torch.equal(tuned[1], auto[1])
