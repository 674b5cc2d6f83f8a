"""The fast-Poisson operator Z = M^{-1} R at the edges of its row and plane passes: 2-D slabs
of 32 rows, every width class of the row pass, rows that are not whole 16-byte groups (the
last group is read past the row's end and masked), one-column-wide grids.

Tolerance: six FP16 roundings plus the spectral scaling per column, independent: about
sqrt(7) 2^-11 = 1.3e-3 relative in the 2-norm; 4e-3 allowed.  In the mixed solve the inverse
pass also forms the search direction: solutions meet the tolerance of the solve.
"""
import numpy as np
import pytest

from paper_2605_25149_amd import inputs

pytestmark = pytest.mark.gpu

GRIDS = [(5, 31), (8, 32), (33, 33), (7, 65), (63, 97), (95, 20), (97, 64), (129, 63), (161, 34),
         (199, 199), (225, 40), (255, 256), (256, 33), (1, 40), (2, 3), (9, 11, 10), (61, 15, 33),
         (31, 130, 4), (1, 5, 6), (150, 140, 3)]


@pytest.mark.parametrize("n", GRIDS, ids=["x".join(map(str, n)) for n in GRIDS])
def test_precond_edges(oracle_mod, n):
    import torch  # noqa: F401

    from paper_2605_25149_amd import binding as B

    dim, N = len(n), 3
    V = inputs.gaussian_wells(n, seed=2) + 25.0
    prob = oracle_mod.Problem(dim, n, V)
    R = inputs.random_block(prob.ng, N, seed=11)
    ref = prob.precond_apply(R)
    with B.Solver(dim, n, N, precond="fast_poisson") as s:
        s.set_potential(V)
        Zt, rz = s.precond(B.as_block(R))
        Z = B.to_numpy(Zt)
    err = np.linalg.norm(Z - ref, axis=0) / np.linalg.norm(ref, axis=0)
    assert np.all(err <= 4e-3), err
    rz_ref = np.einsum("ij,ij->j", R, ref)
    assert np.all(np.abs(rz - rz_ref) <= 4e-3 * np.abs(rz_ref))
    for precision in ("fp64", "mixed"):
        with B.Solver(dim, n, N, precond="fast_poisson", precision=precision,
                      pcg_tol=1e-10) as s:
            s.set_potential(V)
            Xt, it = s.solve(B.as_block(R))
            res = R - B.to_numpy(s.apply(Xt))
        rel = np.linalg.norm(res, axis=0) / np.linalg.norm(R, axis=0)
        assert np.all(rel <= 2e-10), (precision, rel)
        assert np.all(it <= 40), (precision, it)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n,slabs", [((20, 18, 16), 16), ((24, 50, 16), 16), ((21, 100, 16), 16),
                                     ((20, 140, 16), 16), ((33, 256), 8)],
                         ids=lambda n: "x".join(map(str, n)) if isinstance(n, tuple) else "")
def test_fused_scalars_bitwise(n, slabs, precision):
    """Up to 4096 workgroups the plane passes form the scales and beta themselves, with one
    column more launches of their own do, adding in the same order: the columns of both
    solves are the same bits."""
    from paper_2605_25149_amd import binding as B

    C = 4096 // slabs
    V = inputs.gaussian_wells(n, seed=2) + 25.0
    R = B.as_block(inputs.random_block(int(np.prod(n)), C + 1, seed=7))
    with B.Solver(len(n), n, C + 1, precond="fast_poisson", precision=precision,
                  pcg_tol=1e-10) as s:
        s.set_potential(V)
        X0, it0 = s.solve(R[:C])
        X1, it1 = s.solve(R)
        assert np.array_equal(it0, it1[:C])
        assert np.array_equal(B.to_numpy(X0), B.to_numpy(X1)[:, :C])
