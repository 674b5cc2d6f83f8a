"""Which form an FP64 Jacobi solve takes (a workgroup or a cluster of workgroups per column,
or the streaming sweeps), and the ways through the on-chip forms that few columns and one
launch do not reach.

Tolerance against the oracle: both solve to ||r|| <= 1e-12 ||b|| by the same iteration; with
the potentials here (V >= 2000) lambda_min ||x|| >= 1e-2 ||b||, so 1e-9 of max |x| bounds the
difference with a margin.  Columns with equal data give equal bits whichever cluster, range or
launch they fall into.
"""
import os

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _binding():
    import torch  # noqa: F401

    from paper_2605_25149_amd import binding

    binding.load_library()
    return binding


class _Env:
    def __init__(self, **kw):
        self.kw = kw

    def __enter__(self):
        self.old = {k: os.environ.get(k) for k in self.kw}
        os.environ.update(self.kw)

    def __exit__(self, *a):
        for k, v in self.old.items():
            os.environ.pop(k, None)
            if v is not None:
                os.environ[k] = v


def _problem(n, N, seed=7):
    ng = int(np.prod(n))
    rng = np.random.default_rng(seed)
    V = 2000.0 * (1.0 + rng.random(ng))
    base = rng.standard_normal((3, ng))
    return ng, V, np.asfortranarray(base[np.arange(N) % 3].T)


def _launches(s):
    d = s.profile_data()
    return d["cg_f64"]["launches"], d["sweep1_f64"]["launches"] + d["sweep2_f64"]["launches"]


@pytest.mark.parametrize("n", [(32, 32), (128, 64), (20, 20, 20), (91, 90), (128, 128), (199, 199),
                               (64, 64, 33), (64, 64, 128)])
def test_solve_stays_on_chip(n):
    B = _binding()
    ng, V, Bm = _problem(n, 3)
    with B.Solver(len(n), n, 3, pcg_tol=1e-10) as s:
        s.set_potential(V)
        s.profile(True)
        s.solve(B.as_block(Bm))
        cg, sweeps = _launches(s)
    assert cg == 1 and sweeps == 0


@pytest.mark.parametrize("n,N", [((128, 128), 130), ((150, 160), 90), ((64, 64, 128), 33)],
                         ids=["workgroup-per-column", "second-column", "ranges"])
def test_many_columns(oracle_mod, n, N):
    """More columns than clusters (one workgroup per column where that fits, several columns
    per cluster elsewhere) and more than eight per cluster (several launches)."""
    B = _binding()
    dim = len(n)
    ng, V, Bm = _problem(n, N)
    Xr, itr, _, _ = oracle_mod.Problem(dim, n, V).solve(np.asfortranarray(Bm[:, :3]), tol=1e-12,
                                                        variant=0)
    with B.Solver(dim, n, N, pcg_tol=1e-12) as s:
        s.set_potential(V)
        s.profile(True)
        X, it = s.solve(B.as_block(Bm))
        cg, sweeps = _launches(s)
        X = B.to_numpy(X)
    assert sweeps == 0 and cg == (2 if n == (64, 64, 128) else 1)
    for j in range(N):
        assert np.array_equal(X[:, j], X[:, j % 3]) and it[j] == it[j % 3]
    assert np.max(np.abs(X[:, :3] - Xr)) <= 1e-9 * np.max(np.abs(Xr))
    assert np.all(np.abs(it[:3] - itr) <= 2)


@pytest.mark.parametrize("n", [(17, 19, 23), (33, 31, 9), (64, 64, 33)])
def test_continued_3d(n):
    B = _binding()
    ng, V, Bm = _problem(n, 3)
    X0 = np.asfortranarray(1e-3 * np.random.default_rng(1).standard_normal((3, ng)).T)
    out = []
    for env in ({}, {"QO_COL_CHUNK": "3"}):
        with _Env(**env), B.Solver(3, n, 3, pcg_tol=1e-10) as s:
            s.set_potential(V)
            s.profile(True)
            for start in (None, X0):
                X, it = s.solve(B.as_block(Bm), None if start is None else B.as_block(start))
                out.append((B.to_numpy(X), it))
            assert _launches(s)[1] == 0
    for a, b in zip(out[:2], out[2:]):
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])


@pytest.mark.parametrize("n,onchip", [((100, 90), True), ((199, 199), False), ((40, 40, 40), False)])
@pytest.mark.parametrize("warm", [False, True])
def test_wait_given_up(oracle_mod, capfd, n, onchip, warm):
    """Every wait between the workgroups made to run out: all of them leave, and the solve and the handle's later ones take one workgroup per column where
    that fits and the streaming sweeps elsewhere, with one message."""
    B = _binding()
    dim = len(n)
    ng, V, Bm = _problem(n, 3)
    X0 = np.asfortranarray(1e-3 * np.random.default_rng(1).standard_normal((3, ng)).T) if warm else None
    Xr, itr, _, _ = oracle_mod.Problem(dim, n, V).solve(Bm, X0=X0, tol=1e-12, variant=0)
    with _Env(QO_CLU_GIVE_UP="1"):
        s = B.Solver(dim, n, 3, pcg_tol=1e-12)
    with s:
        s.set_potential(V)
        for again in range(2):
            s.profile(True)
            X, it = s.solve(B.as_block(Bm), None if X0 is None else B.as_block(X0))
            cg, sweeps = _launches(s)
            assert (sweeps == 0) == onchip
            assert cg == (1 if onchip else 0) + (1 if again == 0 else 0)
            assert np.max(np.abs(B.to_numpy(X) - Xr)) <= 1e-9 * np.max(np.abs(Xr))
            assert np.all(np.abs(it - itr) <= 2)
    assert capfd.readouterr().err.count("not resident together") == 1
