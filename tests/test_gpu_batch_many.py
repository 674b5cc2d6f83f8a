"""Grouped batches of many small instances, whose Grams have few partials each, and of few
instances (many partials) against single FP64 handles on the same problems.

Tolerance: both solve to ||r|| <= 1e-11 ||b|| and take the same two steps in FP64; states agree
to a small multiple of the solves' tolerance (conditioning of the 16 x 16 operator about 50),
bounded by 1e-8 of max |U|, energies by 1e-9.
"""
import numpy as np
import pytest

from paper_2605_25149_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count,n,N", [(300, (16, 16), 1), (300, (16, 16), 4), (270, (17, 15), 7),
                                       (260, (16, 16), 33), (2, (64, 64), 5), (3, (96, 64), 33),
                                       (9, (64, 60), 12)])
def test_many_instances(count, n, N):
    import torch  # noqa: F401

    from paper_2605_25149_amd import binding as B

    ng = n[0] * n[1]
    rng = np.random.default_rng(count + N)
    V = [inputs.harmonic(n, 50.0 + 10.0 * i) for i in range(3)]
    U = [np.asfortranarray(rng.standard_normal((N, ng)).T) for _ in range(3)]
    kw = dict(pcg_tol=1e-11, pcg_maxit=60, precond="fast_poisson")
    tau = [3.0, 3.5, 4.0]
    with B.Batch([dict(dim=2, n=n, N=N, **kw) for _ in range(count)]) as b:
        for i in range(count):
            b.set_potential(i, V[i % 3])
            b.set_state(i, U[i % 3])
        stats = b.step([tau[i % 3] for i in range(count)], 2)
        got = {i: b.get_state(i) for i in range(count) if i < 3 or i >= count - 3}
    for j in range(min(3, count)):
        with B.Solver(2, n, N, **kw) as s:
            s.set_potential(V[j])
            s.set_state(U[j])
            st = s.step(tau[j], 2)
            ref = B.to_numpy(s.get_state())
        for i, X in got.items():
            if i % 3 == j:
                assert np.max(np.abs(X - ref)) <= 1e-8 * np.max(np.abs(ref))
        for i in range(j, count, 3):
            assert abs(stats[i]["energy"] - st["energy"]) <= 1e-9 * abs(st["energy"])
            assert abs(stats[i]["orth_err_fro"] - st["orth_err_fro"]) <= 1e-8 * (1 + st["orth_err_fro"])
