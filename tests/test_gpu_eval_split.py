"""The evaluation's scores from two fp16 parts per number, and where three bf16 parts take their place: widths around the
change, rows of very different size, numbers near fp16's and fp32's limits, ragged tiles.  Against 64 bits.

Bound on a score: every term q_k h_k is known to 2^-21 of itself (each factor keeps 23 of its 24 bits or more, 2^-23 each,
and the product of the two second parts is left out, 2^-22), and every addition into the accumulator (six per 16 terms at
most) rounds at 2^-23 of a partial sum, which is at most S = sum |q_k h_k|.  Columns of a row that are tiny against the row's largest
add up to 2^-25 of the scaled sizes, 2^-39 of the largest numbers' product per term."""
import sys

import numpy as np
import pytest

from oracle import eval_oracle as ev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def kb():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2201_02791_amd import binding
    binding.load()
    return binding


def check(kb, H, M, n, R, n_test, seed):
    import torch
    rng = np.random.default_rng(seed)
    th, tr, tt = (rng.integers(0, hi, n_test).astype(np.int32) for hi in (n, R, n))
    th[:3], tt[:3] = n - 1, 0
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    scores, ans = kb.eval_debug_scores(dev(H), dev(M), dev(th), dev(tr), dev(tt))
    fixed, rel, true, _ = ev.queries_of(th, tr, tt)
    picked = scores[torch.arange(2 * n_test, device="cuda"), dev(true)]
    assert torch.equal(picked.view(torch.int32), ans.view(torch.int32))       # the two kernels agree on a pair's bits
    Q = dev(H[fixed] * M[rel]).double()                                         # the query vectors are fp32 products
    H64 = dev(H).double()
    want, size = Q @ H64.T, Q.abs() @ H64.abs().T
    d = H.shape[1]
    tiny = d * 2.0 ** -39 * float(Q.abs().max()) * float(H64.abs().max())
    bound = (2.0 ** -21 + 6 * -(-d // 16) * 2.0 ** -23) * size + tiny
    assert bool(((scores.double() - want).abs() <= bound).all())
    # counts are those of the scores themselves
    hi, eq = kb.eval_rank_all(dev(H), dev(M), dev(th), dev(tr), dev(tt))
    others = torch.ones_like(scores, dtype=torch.bool)
    others[torch.arange(2 * n_test, device="cuda"), dev(true)] = False
    assert torch.equal(hi.long(), ((scores > ans[:, None]) & others).sum(1))
    assert torch.equal(eq.long(), ((scores == ans[:, None]) & others).sum(1))


def two_parts(n, n_test, d):
    """Whether an evaluation of that size is one that two fp16 parts are for."""
    return d >= 80 and 2 * n_test * n * d * d >= 3.4e11


def model(n, R, d, seed):
    rng = np.random.default_rng(seed)
    H, M = rng.normal(size=(n, d)).astype(np.float32), rng.normal(size=(R, d)).astype(np.float32)
    H[n // 2] = H[n // 3]                               # equal scores, and a row of zeros
    H[1] = 0.0
    return H, M


@pytest.mark.parametrize("n,n_test", [(700, 90), (17001, 520)])       # 128 x 128 and 256 x 256 tiles, ragged both ways
@pytest.mark.parametrize("d", [76, 80, 84, 200, 1024])
def test_widths(kb, n, n_test, d):
    print("[case] widths", n, n_test, d, file=sys.stderr, flush=True)
    H, M = model(n, 3, d, 51)
    check(kb, H, M, n, 3, n_test, 52)


@pytest.mark.parametrize("n,n_test,d,two", [(30001, 890, 80, True), (30001, 880, 80, False), (30001, 810, 84, True), (9001, 480, 200, True),
                                            (9001, 470, 200, False), (3001, 70, 1024, True), (700, 90, 1024, False)])
def test_sizes_around_the_change(kb, n, n_test, d, two):
    """Evaluations just large enough for two parts and just not, tiles of 128 x 128 and of 256 x 256."""
    print("[case] around the change", n, n_test, d, file=sys.stderr, flush=True)
    assert two_parts(n, n_test, d) == two
    H, M = model(n, 3, d, 59)
    check(kb, H, M, n, 3, n_test, 60)


@pytest.mark.parametrize("n,n_test", [(700, 90), (17001, 640)])          # three parts, two where the numbers allow them
@pytest.mark.parametrize("what,scale", [("row", 2.0 ** -13), ("row", 2.0 ** -16), ("row", 2.0 ** -40), ("column", 2.0 ** -30),
                                        ("all", 2.0 ** -23), ("all", 2.0 ** -26), ("all", 2.0 ** 23), ("all", 2.0 ** 30),
                                        ("relation", 2.0 ** -20)])
def test_sizes(kb, what, scale, n, n_test):
    """Rows, columns, relations and whole tensors far from the rest in size."""
    print("[case] sizes", what, scale, n, file=sys.stderr, flush=True)
    R, d = 3, 128
    assert two_parts(n, n_test, d) == (n > 700)
    H, M = model(n, R, d, 53)
    if what == "row": H[n - 1] *= scale; H[5] *= scale
    elif what == "column": H[:, 7] *= scale
    elif what == "all": H *= scale
    else: M[1] *= scale
    check(kb, H, M, n, R, n_test, 54)


def far_apart(what, gap, n, R, d):
    """Models whose scores rest, for some queries or all, on numbers 2^gap below the largest ones."""
    rng = np.random.default_rng(57)
    H, M = rng.normal(size=(n, d)).astype(np.float32), rng.normal(size=(R, d)).astype(np.float32)
    low = np.float32(2.0 ** -gap)
    if what in ("column", "relations"):                  # a column of H above the rest, which all or one of the relations do not read
        H *= np.float32(2.0 ** -20)
        H[:, 5] /= low
        M[slice(None) if what == "column" else 0, 5] = 0.0
    elif what == "tiny":                                 # ... or read by next to nothing
        H *= np.float32(2.0 ** -20)
        H[:, 5] /= low
        M[:, 5] *= low * low
    elif what == "kinds":                                # two kinds of rows, and relations that read the columns of either
        H[0::2, : d // 2] *= low
        H[1::2, d // 2:] *= low
        M[0, : d // 2] = 0.0
        M[1, d // 2:] = 0.0
    elif what == "sizes":                                # rows and relations of many sizes, one of zeros
        H *= (2.0 ** (-gap * (np.arange(n) % 5) / 4)).astype(np.float32)[:, None]
        M[1] *= low
        H[n // 2] = 0.0
    return H, M


@pytest.mark.parametrize("n,n_test,d", [(700, 90, 100), (9001, 520, 200), (17001, 1010, 100)])     # three parts; two, tiles of either size
@pytest.mark.parametrize("what,gap", [("column", 20), ("column", 24), ("column", 30), ("relations", 26), ("tiny", 24), ("kinds", 20),
                                      ("kinds", 40), ("sizes", 14), ("sizes", 30)])
def test_scores_far_below_the_largest_numbers(kb, what, gap, n, n_test, d):
    """A score is as accurate as its own terms allow, and as accurate as the answer's where that is larger: the sides of the
    answer's score are what is counted.  2^-20 of the terms' sizes: an fp32 sum of 100 terms has rounding errors of 2^-24 of
    its partial sums, some 50 of random sign."""
    import torch
    print("[case] far apart", what, gap, n, n_test, file=sys.stderr, flush=True)
    R = 3
    assert two_parts(n, n_test, d) == (n > 700)
    H, M = far_apart(what, gap, n, R, d)
    rng = np.random.default_rng(58)
    th, tr, tt = (rng.integers(0, hi, n_test).astype(np.int32) for hi in (n, R, n))
    th[:3], tt[:3] = n - 1, n // 2
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    scores, ans = kb.eval_debug_scores(dev(H), dev(M), dev(th), dev(tr), dev(tt))
    fixed, rel, true, _ = ev.queries_of(th, tr, tt)
    rows = torch.arange(2 * n_test, device="cuda")
    assert torch.equal(scores[rows, dev(true)].view(torch.int32), ans.view(torch.int32))
    Q = dev(H[fixed] * M[rel]).double()
    H64 = dev(H).double()
    want, size = Q @ H64.T, Q.abs() @ H64.abs().T
    assert bool(((scores.double() - want).abs() <= 2.0 ** -20 * (size + size[rows, dev(true)][:, None])).all())
    known = [np.concatenate([x, rng.integers(0, hi, 4000)]).astype(np.int32) for x, hi in ((th, n), (tr, R), (tt, n))]
    hi, eq = kb.eval_rank_all(dev(H), dev(M), dev(th), dev(tr), dev(tt), kb.EvalFilter(*known, n, R))
    gone = np.zeros((2 * n_test, n), bool)               # what the filter removes, and the answer itself
    tails, heads = {}, {}
    for h, r, t in zip(*known):
        tails.setdefault((h, r), []).append(t)
        heads.setdefault((t, r), []).append(h)
    for i in range(2 * n_test):
        gone[i, (tails if i < n_test else heads).get((fixed[i], rel[i]), [])] = True
        gone[i, true[i]] = True
    left = ~dev(gone)
    assert torch.equal(hi.long(), ((scores > ans[:, None]) & left).sum(1))
    assert torch.equal(eq.long(), ((scores == ans[:, None]) & left).sum(1))


@pytest.mark.parametrize("n,n_test", [(5000, 300), (20001, 950)])
def test_whole_numbers_are_exact(kb, n, n_test):
    print("[case] whole numbers", n, file=sys.stderr, flush=True)
    import torch
    R, d = 2, 96
    rng = np.random.default_rng(55)
    H = rng.integers(-9, 10, (n, d)).astype(np.float32); M = rng.integers(-3, 4, (R, d)).astype(np.float32)
    th, tr, tt = (rng.integers(0, hi, n_test).astype(np.int32) for hi in (n, R, n))
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    hi, eq = kb.eval_rank_all(dev(H), dev(M), dev(th), dev(tr), dev(tt))
    whi, weq = ev.filtered_counts(H, M, th, tr, tt)
    assert weq.max() > 0
    np.testing.assert_array_equal(hi.cpu().numpy(), whi)
    np.testing.assert_array_equal(eq.cpu().numpy(), weq)


def test_counts_of_many_queries(kb):
    """Mean reciprocal rank and shares of ranks up to k from given counts, extreme ones among them."""
    print("[case] metrics", file=sys.stderr, flush=True)
    import torch
    rng = np.random.default_rng(56)
    for n in (1, 1023, 8193, 30000):
        hi, eq = rng.integers(0, 40, n).astype(np.int32), rng.integers(0, 4, n).astype(np.int32)
        hi[: n // 9], eq[0] = 2**31 - 1, 2**31 - 1
        ks = (1, 3, 10, 2**31 - 1)
        got = kb.eval_metrics(torch.from_numpy(hi).cuda(), torch.from_numpy(eq).cuda(), ks).cpu().numpy()
        rank = 1.0 + hi.astype(np.float64) + 0.5 * eq
        np.testing.assert_allclose(got, [np.mean(1.0 / rank)] + [np.mean(rank <= k) for k in ks], rtol=1e-12)


def test_reciprocals_round_correctly(kb):
    """The sum of reciprocal ranks to the last bit: 1024 sums in the order of the queries, 64 of them halved six times over and
    the 16 results in order."""
    print("[case] reciprocals", file=sys.stderr, flush=True)
    import torch
    lane = np.arange(64)
    for n in (1, 3, 1025, 30000):
        rng = np.random.default_rng(n)
        for top in (50, 10**6, 2**31 - 1):
            hi, eq = rng.integers(0, top, n).astype(np.int32), rng.integers(0, 4, n).astype(np.int32)
            x = np.zeros(-(-n // 1024) * 1024)
            x[:n] = 1.0 / (1.0 + hi.astype(np.float64) + 0.5 * eq)
            s = np.zeros(1024)
            for row in x.reshape(-1, 1024):
                s = s + row
            s = s.reshape(16, 64)
            for off in (32, 16, 8, 4, 2, 1):
                s = s + s[:, lane ^ off]
            want = 0.0
            for w in range(16):
                want = want + s[w, 0]
            got = kb.eval_metrics(torch.from_numpy(hi).cuda(), torch.from_numpy(eq).cuda(), (1,)).cpu().numpy()[0]
            assert got == want / n
