"""FP64 Gram matrices at the edges of their tilings, against NumPy on the same data.

Tolerance: a Gram entry is a sum of ng products; split sums round it to about sqrt(ng) eps
relative to the diagonal, far below 1e-13 for these sizes.
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
