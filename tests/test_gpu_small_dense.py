"""FP64 Gram matrices and the device eigensolver at the edges of their tilings, against
NumPy / SciPy on the same data.

Tolerances: a Gram entry is a sum of ng products; split sums round it to about
sqrt(ng) eps relative to the diagonal, far below 1e-13 for these sizes.  The Jacobi
iteration is backward stable: eigenvalues within a modest multiple of n eps cond(S) of
max |lambda| (n <= 131, cond(S) < 20 here), bounded by 1e-11.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _mods():
    import torch

    from paper_2605_25149_amd import binding

    return torch, binding


@pytest.mark.parametrize("ncols,ng", [(1, 1), (1, 17), (7, 15), (8, 16), (8, 255), (9, 257),
                                      (24, 4097), (31, 1000), (32, 4096), (33, 65537),
                                      (48, 40001), (65, 3000), (100, 70001)])
def test_gram_edges(ncols, ng):
    torch, B = _mods()
    rng = np.random.default_rng(ncols * 1000003 + ng)
    X, Y = rng.standard_normal((2, ncols, ng))
    w = 1.0 / ng
    Z = np.concatenate([X, Y])
    ref = w * (Z @ Z.T)
    for pad in (0, 1):  # 16-byte aligned columns where ng is even, and odd strides
        bx = torch.zeros((ncols, ng + pad), dtype=torch.float64, device="cuda")
        by = torch.zeros_like(bx)
        bx[:, :ng] = torch.from_numpy(X)
        by[:, :ng] = torch.from_numpy(Y)
        G = torch.full((4 * ncols * ncols,), float("nan"), dtype=torch.float64, device="cuda")
        B.gram_pair_noalloc(bx[:, :ng], by[:, :ng], w, G)
        g = G.cpu().numpy().reshape(2 * ncols, 2 * ncols)
        assert np.max(np.abs(g - ref)) <= 1e-13 * np.max(np.abs(ref))
        assert np.array_equal(g, g.T)


@pytest.mark.parametrize("N", [1, 2, 3, 16, 33, 97, 98, 99, 100, 131])
def test_eigenpairs_sizes(N):
    import scipy.linalg

    torch, B = _mods()
    n = (12, 10, 11)
    ng = n[0] * n[1] * n[2]
    rng = np.random.default_rng(N)
    with B.Solver(3, n, N, sigma=0.25) as s:
        s.set_potential(5.0 * rng.standard_normal(ng) + 40.0)
        s.set_state(rng.standard_normal((ng, N)))
        S, K = s.gram()
        lam, vec = s.eigenpairs("ritz", vectors=True)
        ref = scipy.linalg.eigh(0.5 * (K + K.T), S, eigvals_only=True) - 0.25
        assert np.max(np.abs(lam - ref)) <= 1e-11 * np.max(np.abs(ref))
        assert np.all(np.diff(lam) >= 0.0)
        HV = s.apply(vec)
        w = 1.0 / np.prod([m + 1.0 for m in n])
        V = vec.cpu().numpy()
        T = w * (V @ HV.cpu().numpy().T)
        assert np.max(np.abs(w * (V @ V.T) - np.eye(N))) <= 1e-11
        assert np.max(np.abs(T - np.diag(ref + 0.25))) <= 1e-11 * np.max(np.abs(ref))
