"""FP64 Gram matrices of more than 256 columns, where a wavefront works a tile alone, at the
edges of its rule (tiles trimmed up to six a side, whole from seven), against NumPy.

Tolerance: an entry is a sum of ng products; split sums round it to about sqrt(ng) eps relative
to the diagonal, far below 1e-13 for these sizes.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ncols,ng", [(129, 1000), (160, 15), (192, 3001), (193, 4096), (201, 17),
                                      (224, 4111), (225, 2050), (256, 20001), (300, 257)])
def test_gram_many_columns(ncols, ng):
    import torch

    from paper_2605_25149_amd import binding as B

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
