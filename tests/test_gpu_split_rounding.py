"""Products of short sums on the bf16 matrix cores: nothing averages out, so what the three bf16 parts of an operand and
the six of their nine products leave out shows in full.

With parts rounded to nearest |x - x1| <= 2^-8 |x| (x1 the leading part, and so on), so what the three products left out can
add up to is 2 x 2^-8 2^-17 |x y| = 2^-24 |x y| (parts that are cut off instead: 7.8 x 2^-24, all of one sign).  A sum of four
products then passes through six matrix-core additions, of which only the last is as large as the result: cut off to 24
bits, at most 2^-23 of it.  Together 3 x 2^-24 of the sum of the terms' magnitudes; 4 x allowed."""
import numpy as np
import pytest

from test_gpu_split_products import layer

pytestmark = pytest.mark.gpu
BOUND = 4 * 2.0 ** -24


# the mantissa for which cut-off parts leave out most, the one for which rounded parts do, and random ones
def operands(kind, *shapes):
    rng = np.random.default_rng(11)
    if kind == "cut":
        return [np.full(s, 1 + 2.0 ** -7 - 2.0 ** -23, np.float32) for s in shapes]
    if kind == "tie":
        return [np.full(s, 1 + 2.0 ** -8 + 2.0 ** -17 + 2.0 ** -23, np.float32) for s in shapes]
    return [(rng.uniform(1, 2, s) * rng.choice([-1, 1], s)).astype(np.float32) for s in shapes]


def off(got, x, y):
    """largest |got - x y| over the terms' magnitudes"""
    x, y = x.astype(np.float64), y.astype(np.float64)
    return (np.abs(got - x @ y) / (np.abs(x) @ np.abs(y))).max()


@pytest.mark.parametrize("kind", ["cut", "tie", "random"])
def test_layer_products_of_four_terms(kind):
    """No messages (V = 0): the layer's products are H W_0, G W_0^T and H^T G alone, over 4 columns and 4 vertices."""
    n, di, do = 4, 4, 4
    H0, dH, W0 = operands(kind, (n, di), (n, do), (di, do))
    got, _ = layer(n, 1, 8, di, do, 1, 0, H0, dH, np.zeros((1, di, do), np.float32), np.zeros((2, 1), np.float32), W0)
    assert off(got["out"], H0, W0) <= BOUND
    assert off(got["dH0"], dH, W0.T) <= BOUND
    assert off(got["dW0"], H0.T, dH) <= BOUND


@pytest.mark.parametrize("kind", ["cut", "tie", "random"])
def test_scores_of_four_terms(kind):
    import torch
    from paper_2201_02791_amd import binding as kb
    n, d, n_test = 64, 4, 20
    H, = operands(kind, (n, d))
    ids = np.random.default_rng(5).integers(0, n, (2, n_test)).astype(np.int32)
    t = lambda x: torch.from_numpy(x).cuda()  # noqa: E731
    scores, answer = kb.eval_debug_scores(t(H), t(np.ones((1, d), np.float32)), t(ids[0]), t(np.zeros(n_test, np.int32)), t(ids[1]))
    fixed, true = np.concatenate([ids[0], ids[1]]), np.concatenate([ids[1], ids[0]])
    s = scores.cpu().numpy()
    assert off(s, H[fixed], H.T) <= BOUND
    np.testing.assert_array_equal(s[np.arange(2 * n_test), true], answer.cpu().numpy())


def test_small_numbers_lose_no_more_than_the_smallest_bf16():
    """Parts below 2^-133, the smallest bf16 number, round away: at most half of that per number."""
    n, di, do = 4, 4, 4
    H0, dH, W0 = operands("random", (n, di), (n, do), (di, do))
    for e in (-100, -112, -120, -126):
        small, big = H0 * np.float32(2.0 ** e), W0 * np.float32(2.0 ** 90)
        got, _ = layer(n, 1, 8, di, do, 1, 0, small, dH, np.zeros((1, di, do), np.float32), np.zeros((2, 1), np.float32), big)
        x, y = small.astype(np.float64), big.astype(np.float64)
        lost = BOUND * (np.abs(x) @ np.abs(y)) + 2.0 ** -134 * np.abs(y).sum(0)
        assert (np.abs(got["out"] - x @ y) <= lost).all(), e
