"""Batch steps whose fixed iteration counts ask for more launches than one graph may hold
(pcg_maxit until counts are observed): enqueued directly, same results as without graphs."""
import numpy as np
import pytest

from paper_2605_25149_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,precond,maxit", [("fp64", "jacobi", 15000),
                                                     ("fp64", "fast_poisson", 5000),
                                                     ("mixed", "jacobi", 2500)])
def test_long_first_step(precision, precond, maxit):
    import torch  # noqa: F401

    from paper_2605_25149_amd import binding as B

    n, N = (16, 12), 2
    ng = n[0] * n[1]
    U = np.asfortranarray(np.random.default_rng(2).standard_normal((N, ng)).T)
    out = []
    for graph in (True, False):
        with B.Batch([dict(dim=2, n=n, N=N, pcg_tol=1e-10, pcg_maxit=maxit, precond=precond,
                           precision=precision)]) as b:
            b.set_potential(0, inputs.harmonic(n, 50.0))
            b.set_state(0, U)
            for _ in range(4):  # the first at pcg_maxit, the rest at the observed counts
                st = b.step([3.0], 1, use_graph=graph)
            out.append((b.get_state(0), st[0]["energy"], st[0]["pcg_iters"]))
    assert np.max(np.abs(out[0][0] - out[1][0])) <= 1e-9 * np.max(np.abs(out[1][0]))
    assert abs(out[0][1] - out[1][1]) <= 1e-10 * abs(out[1][1])
    assert np.all(np.abs(np.subtract(out[0][2], out[1][2])) <= 1)
