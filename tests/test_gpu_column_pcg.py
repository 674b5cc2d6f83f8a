"""The FP64 Jacobi-PCG forms that keep a column on the chip, one workgroup or a cluster of
workgroups per column, against the oracle's PCG, at the edges of their point counts and
thread shapes.

Tolerance: both solve to ||r|| <= 1e-12 ||b|| by the same iteration; x differs by at most
about 2e-12 ||b|| / lambda_min, and lambda_min ||x|| >= 1e-2 ||b|| is checked for the random
right-hand sides here, so 1e-9 of max |x| bounds the difference with a margin.  Iteration
counts come from a floating-point test and may differ by one (two late in a solve).
"""
import os

import numpy as np
import pytest

from paper_2605_25149_amd import inputs

pytestmark = pytest.mark.gpu


def _binding():
    import torch  # noqa: F401

    from paper_2605_25149_amd import binding

    binding.load_library()
    return binding


GRIDS = [(2, (1, 2)), (2, (5, 1)), (2, (32, 32)), (2, (25, 41)), (2, (1024, 2)), (2, (64, 33)),
         (2, (128, 32)), (2, (17, 241)), (2, (128, 64)), (2, (113, 73)), (2, (128, 128)),
         (3, (8, 8, 16)), (3, (7, 13, 12)), (3, (16, 16, 16)), (3, (3, 5, 300)), (3, (20, 20, 20)),
         (3, (21, 23, 17)), (3, (16, 32, 32)), (3, (25, 25, 26)), (3, (1, 1, 9)),
         # several workgroups per column: two, a ragged last one, planes larger than a range's
         # half, many (slabs of less than a plane), the most a column takes
         (2, (91, 90)), (2, (129, 127)), (2, (199, 199)), (3, (33, 31, 9)), (3, (75, 77, 5)),
         (3, (64, 64, 33)), (3, (70, 70, 40)), (3, (64, 64, 128))]


@pytest.mark.parametrize("dim,n", GRIDS, ids=["x".join(map(str, n)) for _, n in GRIDS])
def test_column_solve(oracle_mod, dim, n):
    B = _binding()
    ng = int(np.prod(n))
    N = min(3, ng - 1)
    rng = np.random.default_rng(ng)
    L = (1.0, 1.3, 0.8)[:dim]
    V = 30.0 * rng.random(ng)
    prob = oracle_mod.Problem(dim, n, V, L=L)
    Bm = np.asfortranarray(rng.standard_normal((N, ng)).T)
    X0 = np.asfortranarray(0.01 * rng.standard_normal((N, ng)).T)
    with B.Solver(dim, n, N, L=L, pcg_tol=1e-12) as s:
        s.set_potential(V)
        for start in (None, X0):
            Xr, itr, st, _ = prob.solve(Bm, X0=start, tol=1e-12, variant=0)
            X, it = s.solve(B.as_block(Bm), None if start is None else B.as_block(start))
            Xg = B.to_numpy(X)
            assert np.max(np.abs(Xg - Xr)) <= 1e-9 * np.max(np.abs(Xr))
            assert np.all(np.abs(it - itr) <= 2), (it, itr)
        zero = np.asfortranarray(np.zeros((ng, N)))
        X, it = s.solve(B.as_block(zero))
        assert not X.any() and not it.any()


@pytest.mark.parametrize("n", [(20, 17), (100, 90), (150, 160)])
def test_column_solve_continued_and_limits(n):
    """A solve cut into launches of three iterations gives the same bits as one launch; the
    iteration limit and non-finite input are reported."""
    B = _binding()
    ng, N = n[0] * n[1], 3
    rng = np.random.default_rng(5)
    V = inputs.harmonic(n, 100.0)
    Bm = B.as_block(np.asfortranarray(rng.standard_normal((N, ng)).T))
    out = []
    for chunk in (None, "3"):
        old = os.environ.pop("QO_COL_CHUNK", None)
        try:
            if chunk:
                os.environ["QO_COL_CHUNK"] = chunk
            s = B.Solver(2, n, N, pcg_tol=1e-10)
        finally:
            os.environ.pop("QO_COL_CHUNK", None)
            if old is not None:
                os.environ["QO_COL_CHUNK"] = old
        with s:
            s.set_potential(V)
            X, it = s.solve(Bm)
            out.append((B.to_numpy(X), it))
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
    with B.Solver(2, n, N, pcg_tol=1e-10, pcg_maxit=3) as s:
        s.set_potential(V)
        with pytest.raises(B.QOError) as e:
            s.solve(Bm)
        assert e.value.status == B.QO_ERR_PCG_NOCONV
        bad = Bm.clone()
        bad[1, ng // 2] = float("nan")
        with pytest.raises(B.QOError) as e:
            s.solve(bad)
        assert e.value.status == B.QO_ERR_NONFINITE and "column 1" in str(e.value)


def test_concurrent_handles():
    """Two handles on two streams, driven by two threads at once, give the bits they give
    alone (clusters of workgroups wait for one another inside a launch)."""
    import threading

    import torch

    B = _binding()
    n, N = (40, 40, 40), 24
    rng = np.random.default_rng(3)
    V = 30.0 * rng.random(n[0] * n[1] * n[2])
    blocks = [B.as_block(np.asfortranarray(rng.standard_normal((N, V.size)).T)) for _ in range(2)]
    torch.cuda.synchronize()
    solvers = []
    for _ in range(2):
        s = B.Solver(3, n, N, pcg_tol=1e-10, stream=torch.cuda.Stream())
        s.set_potential(V)
        solvers.append(s)
    alone = [B.to_numpy(s.solve(b)[0]) for s, b in zip(solvers, blocks)]
    got = [[], []]

    def work(i):
        with torch.cuda.stream(solvers[i].stream):
            for _ in range(4):
                X = torch.zeros_like(blocks[i])
                solvers[i].stream.synchronize()
                got[i].append(solvers[i].solve(blocks[i], X)[0])

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for i in range(2):
        for X in got[i]:
            assert np.array_equal(B.to_numpy(X), alone[i])
        solvers[i].close()
