"""Backward pass of the project-first neighbour sum by source: every width / base-count class of its dispatch (lanes per
row, bases per lane, chunks of bases, the dot products alone), sources with no edge, one edge, more than one chunk of 64
edges and more than one unit of 256.

Tolerances: fp32 as in the split-product tests; bf16 messages 2e-2 of the largest element (P and dP are rounded to bf16,
2^-9 each, and enter sums of up to a few hundred terms)."""
import numpy as np
import pytest

from test_gpu_split_products import TOL, layer, model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("msg", [0, 1])
@pytest.mark.parametrize("do,B", [(8, 1), (8, 17), (32, 9), (40, 3), (64, 8), (72, 2), (128, 5), (128, 40), (136, 1), (136, 3),
                                  (200, 7), (200, 11), (256, 13), (256, 20)])
def test_every_class_of_shapes(do, B, msg):
    n, R, di = 61, 5, 16
    H0, dH, V, a, W0 = model(do + B, n, R, di, do, B)
    got, want = layer(n, R, 60 * n, di, do, B, 0, H0, dH, V, a, W0, msg)
    for k in want:
        tol = 2e-2 if msg else 10 * TOL
        assert np.abs(got[k] - want[k]).max() <= tol * np.abs(want[k]).max(), k


def test_long_edge_lists():
    n, R, di, do, B = 3, 2, 16, 36, 3          # a source with more edges than one unit holds
    H0, dH, V, a, W0 = model(1, n, R, di, do, B)
    got, want = layer(n, R, 1500, di, do, B, 0, H0, dH, V, a, W0)
    for k in want:
        assert np.abs(got[k] - want[k]).max() <= 10 * TOL * np.abs(want[k]).max(), k


# an infinity in a gradient row: the dot products with it are infinite, also at widths that leave lanes of a row idle
@pytest.mark.parametrize("do,B,msg", [(8, 2, 0), (12, 2, 0), (40, 3, 0), (72, 3, 0), (132, 2, 0), (200, 10, 0), (256, 3, 0),
                                      (200, 10, 1), (96, 40, 1), (160, 33, 1)])
def test_infinite_gradients_stay_infinite(do, B, msg):
    n, R, di = 40, 3, 16
    H0, dH, V, a, W0 = model(do, n, R, di, do, B)
    H0, V = np.abs(H0), np.abs(V)               # P > 0: every term with the infinity has its sign
    dH[7, 1] = np.inf
    got, want = layer(n, R, 20 * n, di, do, B, 0, H0, dH, V, a, W0, msg)
    hit = np.isinf(want["da"])
    assert hit.any() and not np.isnan(want["da"]).any()
    np.testing.assert_array_equal(got["da"][hit], want["da"][hit].astype(np.float32))
    assert np.isfinite(got["da"][~hit]).all()
