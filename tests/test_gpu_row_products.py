"""fp32 layers of 100 to 160 columns in the relation-weight order, whose products with rows run on the fp16 matrix cores: edges
of the classes of widths, tiles that end inside their rows, rows and matrices of very different size, operands that are not
finite.  Tolerance of ordinary operands as in the split-product tests (4e-6 of the largest element)."""
import numpy as np
import pytest

from oracle import oracle as orc
from test_gpu_split_products import TOL, layer, model

pytestmark = pytest.mark.gpu


def takes(n, R, di, do):
    """The rule that takes the forward products and the transposed ones to these kernels, from the graph that `layer` draws."""
    rng = np.random.default_rng(n + di)
    head, tail = rng.integers(0, n, 8 * n).astype(np.int32), rng.integers(0, n, 8 * n).astype(np.int32)
    head[:n] = np.arange(n)
    runs = orc.build_partition(head, rng.integers(0, R, 8 * n).astype(np.int32), tail, n, R)["n_seg"] >= 256 * 2 * R
    return runs and 100 <= di <= 160 and do <= 128, runs and 100 <= do <= 160 and di <= 128


def run(n, R, di, do, B, change=None, reach=True):
    if reach:
        assert any(takes(n, R, di, do)), "the graph is too small for these kernels"
    H0, dH, V, a, W0 = model(n + di, n, R, di, do, B)
    if change:
        change(H0, dH, V, a, W0)
    return layer(n, R, 8 * n, di, do, B, 2, H0, dH, V, a, W0)


@pytest.mark.parametrize("n,R", [(130, 1), (257, 2), (261, 1), (613, 2), (1500, 3)])       # the first two stay with the tiled product
@pytest.mark.parametrize("di,do", [(100, 4), (112, 32), (116, 36), (128, 128), (132, 64), (160, 100), (4, 128), (96, 112)])
def test_widths(n, R, di, do):
    assert any(takes(n, R, di, do)) == (n > 257)
    got, want = run(n, R, di, do, 2, reach=False)
    for k in want:
        assert np.abs(got[k] - want[k]).max() <= TOL * np.abs(want[k]).max(), k


def close_by_rows(got, want, tol):
    """Every row against its own size."""
    size = np.abs(want).max(axis=1)
    assert (np.abs(got - want).max(axis=1) <= tol * size + 1e-37).all()


@pytest.mark.parametrize("exponent", [-60, -20, 20, 60])
def test_every_input_row_at_its_own_size(exponent):
    """No edge joins the scaled vertices to others' rows: W_r is zero, so an output row is its vertex's own product."""
    n, scaled = 600, slice(100, 200)

    def change(H0, dH, V, a, W0):
        H0[scaled] *= np.float32(2.0 ** exponent); dH[scaled] *= np.float32(2.0 ** exponent)
        a[:] = 0
    got, want = run(n, 1, 128, 128, 1, change)
    close_by_rows(got["out"], want["out"], 8e-6)
    close_by_rows(got["dH0"], want["dH0"], 8e-6)


@pytest.mark.parametrize("gap", [24, 30, 70])
@pytest.mark.parametrize("what", ["rows", "entries", "one number"])
def test_sums_that_rest_on_small_numbers(what, gap):
    """Large numbers that meet zeros do not cost the small ones beside them any bits: every column of the results against its own
    size.  Random rounding errors of an fp32 sum of 128 terms, the largest of some thousand: 4e-6 of its largest element."""
    n, d, half, big = 600, 128, 64, np.float32(2.0 ** gap)
    columns = slice(0, half)

    def change(H0, dH, V, a, W0):
        if what == "rows":                             # a column of the rows is large where the matrices' first half is zero
            H0[:, 70] *= big; dH[:, 70] *= big
            for W in (V[0], V[1], W0):
                W[70, columns] = 0; W[columns, 70] = 0
        elif what == "entries":                        # an entry of every row and column is large, where the rows are zero
            H0[:, half:] = 0; dH[:, half:] = 0
            for W in (V[0], V[1], W0):
                W[np.arange(d), (np.arange(d) + half) % d] *= big
        else:                                          # a row of its own has one number that matters, far below the others
            H0[5::7, 70:] *= big; dH[5::7, 70:] *= big
            H0[5::7, :69] = 0; dH[5::7, :69] = 0
            for W in (V[0], V[1], W0):
                W[70:, columns] = 0; W[columns, 70:] = 0
    got, want = run(n, 1, d, d, 2, change)
    for k in ("out", "dH0"):
        size = np.abs(want[k][:, columns]).max(axis=0)
        assert (np.abs(got[k] - want[k])[:, columns].max(axis=0) <= TOL * size).all(), k


@pytest.mark.parametrize("alone", [False, True])
@pytest.mark.parametrize("what", ["column", "row", "matrix", "huge"])
def test_matrices_that_are_not_split(what, alone):
    """A column or row far below the rest, or entries near the ends of the range: plain fp32 products.  Alone: the self-loop's
    matrix is all there is, and every column of its products is held to its own size."""
    def change(H0, dH, V, a, W0):
        if alone: a[:] = 0
        if what == "column": W0[:, 5] *= np.float32(2.0 ** -40)
        elif what == "row": W0[7] *= np.float32(2.0 ** -30)
        elif what == "matrix": W0 *= np.float32(2.0 ** -110)
        else: W0 *= np.float32(2.0 ** 105)
    got, want = run(300, 1, 112, 104, 2, change)
    for k in ("out", "dH0"):
        assert np.abs(got[k] - want[k]).max() <= 2 * TOL * np.abs(want[k]).max(), k
        if alone:
            assert (np.abs(got[k] - want[k]).max(axis=0) <= 2 * TOL * np.abs(want[k]).max(axis=0)).all(), k
    if what == "column":                          # the column's own sums: only the self-loop's part is tiny, the runs' is not
        assert np.abs(got["out"][:, 5] - want["out"][:, 5]).max() <= 2 * TOL * np.abs(want["out"][:, 5]).max()


@pytest.mark.parametrize("bad", [np.inf, np.nan])
@pytest.mark.parametrize("where", ["H0", "dH", "W0", "V"])
def test_numbers_that_are_not_finite(bad, where):
    """They reach exactly the results that they reach in the oracle, and the others stay as they are."""
    def change(H0, dH, V, a, W0):
        a[:] = np.abs(a) + np.float32(0.1)
        dict(H0=H0, dH=dH, W0=W0, V=V[0])[where][3, 2] = bad
    assert all(takes(300, 1, 128, 112))
    got, want = run(300, 1, 128, 112, 2, change)
    for k in ("out", "dH0"):
        finite = np.isfinite(want[k])
        assert np.array_equal(np.isfinite(got[k]), finite), k
        if finite.any():
            scale = np.abs(want[k][finite]).max()
            assert np.abs(got[k][finite] - want[k][finite]).max() <= 2 * TOL * scale, k
