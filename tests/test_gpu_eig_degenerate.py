"""The device eigensolver on matrices with bitwise equal diagonal entries and couplings far
below the square root of the smallest double, against SciPy on the same data.

Tolerance as for the other read-out tests: backward stable, cond(S) < 20, bounded by 1e-11 of
max |lambda|.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TINY = (1e-140, 1e-155, 1e-165, 1e-250)


@pytest.mark.parametrize("N", [19, 98, 99, 120])  # one workgroup up to 98, one launch per round above
def test_equal_diagonals_tiny_couplings(N):
    import scipy.linalg

    import torch  # noqa: F401

    from paper_2605_25149_amd import binding as B

    n, sigma = (18, 17, 16), 0.25
    ng = n[0] * n[1] * n[2]
    rng = np.random.default_rng(N)
    V = 5.0 * rng.standard_normal(ng) + 40.0
    a = np.sqrt(ng)
    U = np.zeros((ng, N))
    # spikes four points apart along x and y, in planes of their own
    spikes = iter([x + n[0] * (y + n[1] * z) for z in (2, 6) for y in (2, 6, 10, 14)
                   for x in (2, 6, 10, 14)])
    free = np.ones(ng, bool)
    free.reshape(n[::-1])[:9] = False
    V[~free] = 40.0
    for k, eps in enumerate(TINY):
        # U_0 and U_1: equal norms, <U_0, U_1> = eps
        i, j = next(spikes), next(spikes)
        U[i, 4 * k] = U[j, 4 * k + 1] = a
        U[j, 4 * k] = eps
        # <U_2, U_3> = 0, <U_2, H U_3> of order eps, equal <U, HU>
        i, j = next(spikes), next(spikes)
        U[i, 4 * k + 2] = U[j, 4 * k + 3] = a
        U[i + 1, 4 * k + 3] = eps
    U[free, 16:] = rng.standard_normal((int(free.sum()), N - 16)) * np.sqrt(ng / free.sum())
    with B.Solver(3, n, N, sigma=sigma) as s:
        s.set_potential(V)
        s.set_state(U)
        S, K = s.gram()
        for k, eps in enumerate(TINY):
            assert S[4 * k, 4 * k] == S[4 * k + 1, 4 * k + 1] and S[4 * k, 4 * k + 1] != 0.0
            c = 4 * k + 2
            assert K[c, c] == K[c + 1, c + 1] and S[c, c + 1] == 0.0 and K[c, c + 1] != 0.0
        lam, vec = s.eigenpairs("ritz", vectors=True)
        ref = scipy.linalg.eigh(0.5 * (K + K.T), S, eigvals_only=True) - sigma
        assert np.max(np.abs(lam - ref)) <= 1e-11 * np.max(np.abs(ref))
        w = 1.0 / np.prod([m + 1.0 for m in n])
        X = vec.cpu().numpy()
        assert np.max(np.abs(w * (X @ X.T) - np.eye(N))) <= 1e-11
