"""fp32 products on the bf16 matrix cores (three bf16 parts per operand): edges of the 128 x 128 x 16 tiles, operands
that are not finite, and the evaluation's scores, whose bits must agree between the kernel that counts over all
entities and the one that scores the filtered pairs.

Tolerance of the layer results: a product of the parts is off by less than 2^-24 of it and a sum of K terms by about
sqrt(K) fp32 roundings, K <= 4096 here: 64 * 2^-24 = 4e-6 of the result's size, relative to the largest element."""
import numpy as np
import pytest

from oracle import eval_oracle as ev
from oracle import oracle as orc

pytestmark = pytest.mark.gpu
TOL = 4e-6


def layer(n, R, m, di, do, B, order, H0, dH, V, a, W0, msg=0, a_at=0):
    import torch
    from paper_2201_02791_amd import binding as kb
    rng = np.random.default_rng(n + di)
    head, tail = rng.integers(0, n, m).astype(np.int32), rng.integers(0, n, m).astype(np.int32)
    head[:n] = np.arange(n)
    rel = rng.integers(0, R, m).astype(np.int32)
    part, opart = kb.build_partition(head, rel, tail, n, R), orc.build_partition(head, rel, tail, n, R)
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    coeff = torch.empty(a.size + a_at, device="cuda")[a_at:].view(a.shape).copy_(t(a))
    lay = [dict(V=t(V), a=coeff, W0=t(W0), act=kb.ACT_IDENTITY, order=order)]
    ws = torch.zeros(kb.workspace_bytes(part, lay, msg), dtype=torch.uint8, device="cuda")
    H, G, out, dH0 = t(H0), t(dH), torch.empty(n, do, device="cuda"), torch.empty(n, di, device="cuda")
    grads = [{k: torch.empty_like(lay[0][k[1:]]) for k in ("dV", "da", "dW0")}]
    kb.rgcn_forward(part, lay, H, ws, out, msg)
    kb.rgcn_backward(part, lay, H, ws, G, grads, dH0, msg)
    torch.cuda.synchronize()
    got = dict(out=out.cpu().numpy(), dH0=dH0.cpu().numpy(), **{k: v.cpu().numpy() for k, v in grads[0].items()})
    with np.errstate(all="ignore"):
        pre, h = orc.layer_forward(opart, V, a, W0, 0, H0)
        want = orc.layer_backward(opart, V, a, W0, 0, H0, pre, dH)
    return got, dict(out=h, dH0=want["dH"], dV=want["dV"], da=want["da"], dW0=want["dW0"])


def model(seed, n, R, di, do, B):
    rng = np.random.default_rng(seed)
    f = lambda *s: rng.standard_normal(s).astype(np.float32)  # noqa: E731
    return f(n, di), f(n, do), f(B, di, do) / np.float32(np.sqrt(di)), f(2 * R, B), f(di, do) / np.float32(np.sqrt(di))


# widths around the tile edges (16 deep, 32 and 128 wide), one row, one past a tile of rows, a relation of few runs
@pytest.mark.parametrize("order", [0, 2])
@pytest.mark.parametrize("n,R,di,do,B", [(1, 1, 4, 4, 1), (129, 1, 16, 128, 2), (300, 7, 20, 132, 3), (257, 2, 128, 36, 2),
                                         (400, 30, 200, 200, 5), (131, 1, 256, 256, 1), (90, 40, 36, 64, 15),
                                         (60, 3, 32, 32, 64), (40, 500, 256, 256, 20), (40, 501, 256, 256, 132)])
def test_tile_edges(n, R, di, do, B, order):
    H0, dH, V, a, W0 = model(n, n, R, di, do, B)
    got, want = layer(n, R, 4 * n, di, do, B, order, H0, dH, V, a, W0)
    for k in want:
        assert np.abs(got[k] - want[k]).max() <= TOL * np.abs(want[k]).max(), k


# the coefficients may lie at any multiple of 4 bytes; the basis gradient's product reads them in pairs
@pytest.mark.parametrize("a_at", [1, 2, 3])
def test_coefficients_at_any_float(a_at):
    n, R, di, do, B = 40, 60, 256, 256, 20
    H0, dH, V, a, W0 = model(n, n, R, di, do, B)
    got, want = layer(n, R, 4 * n, di, do, B, 2, H0, dH, V, a, W0, a_at=a_at)
    for k in want:
        assert np.abs(got[k] - want[k]).max() <= TOL * np.abs(want[k]).max(), k


# the parts of an infinity or a NaN are no use: such results come from fp32 products, and no other result changes
@pytest.mark.parametrize("order", [0, 2])
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan, 1.5e38, 3.4e38])
def test_values_that_do_not_split(bad, order):
    n, R, di, do = 200, 2, 36, 132
    H0, dH, V, a, W0 = model(3, n, R, di, do, 1)
    dH, W0, V = dH * np.float32(1e-3), W0 * np.float32(1e-3), V * np.float32(1e-3)
    H0[70, 5] = bad
    got, want = layer(n, R, 4 * n, di, do, 1, order, H0, dH, V, a, W0)
    for k in want:
        x, y = got[k], want[k]
        np.testing.assert_array_equal(np.isfinite(x), np.isfinite(y), err_msg=k)
        if k == "dW0":         # a product alone; the neighbour sums may turn an infinity into NaN (they pad with 0 * row)
            np.testing.assert_array_equal(x[~np.isfinite(y)], y[~np.isfinite(y)].astype(np.float32))
        # what the value enters is compared at its own size, everything else at the size of everything else
        for part in (np.isfinite(y) & (np.abs(y) > 1e20), np.isfinite(y) & (np.abs(y) <= 1e20)):
            scale = 0.0 if not part.any() else np.abs(y[part]).max() if np.abs(y[part]).max() > 1e20 else np.median(np.abs(y[part]))
            assert np.abs(x[part].astype(np.float64) - y[part]).max(initial=0.0) <= 40 * TOL * max(scale, 1e-30), k


# integer embeddings (every score exact): counts bit for bit, with lists of known answers longer than a block's share
@pytest.mark.parametrize("n,R,d,n_test,hub", [(600, 3, 36, 40, 500), (300, 2, 4, 9, 33), (129, 1, 260, 70, 120), (40, 5, 16, 1, 0)])
def test_filtered_counts_of_hubs(n, R, d, n_test, hub):
    import torch
    from paper_2201_02791_amd import binding as kb
    rng = np.random.default_rng(n)
    H = rng.integers(-2, 3, (n, d)).astype(np.float32)
    M = rng.integers(-1, 2, (R, d)).astype(np.float32)
    H[n // 2] = np.inf                      # one entity whose scores are infinite or not a number
    test = [rng.integers(0, hi, n_test).astype(np.int32) for hi in (n, R, n)]
    test[0][: n_test // 2] = 7
    test[1][: n_test // 2] = 0
    known = [np.concatenate([np.full(hub, 7), rng.integers(0, n, 200)]).astype(np.int32),
             np.concatenate([np.zeros(hub), rng.integers(0, R, 200)]).astype(np.int32),
             np.concatenate([rng.permutation(n)[:hub], rng.integers(0, n, 200)]).astype(np.int32)]
    t = lambda x: torch.from_numpy(x).cuda()  # noqa: E731
    hi, eq = kb.eval_rank_all(t(H), t(M), t(test[0]), t(test[1]), t(test[2]), kb.EvalFilter(*known, n, R))
    with np.errstate(all="ignore"):
        want = ev.filtered_counts(H, M, *test, known)
    finite = np.array([np.isfinite(H[f]).all() and np.isfinite(H[x]).all() for f, x in
                       zip(np.concatenate([test[0], test[2]]), np.concatenate([test[2], test[0]]))])
    np.testing.assert_array_equal(hi.cpu().numpy()[finite], want[0][finite])
    np.testing.assert_array_equal(eq.cpu().numpy()[finite], want[1][finite])
    out = kb.eval_metrics(hi, eq, (1, 3, 10)).cpu().numpy()
    rank = 1.0 + hi.cpu().numpy() + 0.5 * eq.cpu().numpy()
    assert np.allclose(out, [np.mean(1 / rank)] + [np.mean(rank <= k) for k in (1, 3, 10)], rtol=1e-12)
