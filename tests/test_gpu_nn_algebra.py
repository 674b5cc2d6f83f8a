"""N x N algebra of the step, of batches and of the reverse mode at the edges of its
dispatch: 16, 32, 64 and 128 columns of [A | B] per register form of the Gauss-Jordan solve,
64 rows, and the column counts from which an instance's matrices no longer all fit the LDS
(batch: 35, reverse mode: 28).

Tolerances: the systems are solved by backward stable eliminations (cond(S) < 20, n <= 66, so
n eps cond is below 1e-12 with its constant); 1e-11 of the largest entry.  States of two
solver paths differ by their PCG tolerance (1e-12) times a small factor: 1e-9.
"""
import numpy as np
import pytest

from paper_2605_25149_amd import inputs

pytestmark = pytest.mark.gpu

GRID = (12, 10, 11)
SIZES = [1, 2, 8, 9, 16, 17, 32, 33, 35, 36, 64, 65]


def _mods():
    import torch

    from paper_2605_25149_amd import binding

    return torch, binding


def _problem(N, n=GRID):
    V = inputs.harmonic(n, 60.0) + inputs.gaussian_wells(n, seed=3, depth=(1.0, 4.0))
    return V, inputs.random_block(int(np.prod(n)), N, seed=N)


@pytest.mark.parametrize("N", SIZES)
def test_predictor_matrices(N):
    _, B = _mods()
    V, U0 = _problem(N)
    tau = 6.0
    with B.Solver(3, GRID, N, sigma=0.3, pcg_tol=1e-12, precond="fast_poisson") as s:
        s.set_potential(V)
        s.set_state(U0)
        s.step(tau)
        S, M, R, X, Y = (s.get_matrix(k) for k in "SMRXY")
    eye, a = np.eye(N), 0.5 * tau
    K = np.block([[eye - a * M, -a * S], [a * R, eye + a * M.T]])
    sol = np.linalg.solve(K, np.vstack([S, -M.T]))
    Yr, Xr = tau * sol[:N], eye + tau * sol[N:]
    assert np.max(np.abs(X - Xr)) <= 1e-11 * np.max(np.abs(Xr))
    assert np.max(np.abs(Y - Yr)) <= 1e-11 * np.max(np.abs(Yr))


def test_batch_sizes():
    _, B = _mods()
    n, tau = (24, 20), 6.0
    cfg = dict(dim=2, n=n, sigma=0.3, pcg_tol=1e-12, precond="fast_poisson")
    b = B.Batch([dict(cfg, N=N, pcg_maxit=40) for N in SIZES])
    try:
        probs = [_problem(N, n) for N in SIZES]
        for i, (V, U0) in enumerate(probs):
            b.set_potential(i, V)
            b.set_state(i, U0)
        st = b.step([tau] * len(SIZES))
        for i, (V, U0) in enumerate(probs):
            with B.Solver(2, n, SIZES[i], sigma=0.3, pcg_tol=1e-12, pcg_check=1,
                          precond="fast_poisson") as s:
                s.set_potential(V)
                s.set_state(U0)
                r = s.step(tau)
                Ur = B.to_numpy(s.get_state())
            assert abs(st[i]["energy"] - r["energy"]) <= 1e-10 * abs(r["energy"]), SIZES[i]
            U = b.get_state(i)
            assert np.max(np.abs(U - Ur)) <= 1e-9 * np.max(np.abs(Ur)), SIZES[i]
    finally:
        b.close()


@pytest.mark.parametrize("N", [1, 28, 29, 64, 65])
def test_reverse_mode_sizes(oracle_mod, N):
    _, B = _mods()
    V, U0 = _problem(N)
    prob = oracle_mod.Problem(3, GRID, V, sigma=0.3)
    Lr, gVr, gUr = oracle_mod.steps_loss_grad(prob, U0, 6.0, 1, "energy")
    with B.Solver(3, GRID, N, sigma=0.3, pcg_tol=1e-13, pcg_check=1,
                  precond="fast_poisson") as s:
        s.set_potential(V)
        s.set_state(U0)
        L = s.tape_forward(6.0, 1, "energy")
        gV, gU = s.tape_backward()
        gV, gU = gV.cpu().numpy(), B.to_numpy(gU)
    assert abs(L - Lr) <= 1e-11 * abs(Lr)
    assert np.max(np.abs(gV - gVr)) <= 1e-9 * np.max(np.abs(gVr))
    assert np.max(np.abs(gU - gUr)) <= 1e-9 * np.max(np.abs(gUr))
