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


# few bases, narrow rows and many edges per relation of a source: the lane groups share the edges (every width / base-count
# class of that form; 200 or 600 edges per source, the latter in units of 256), an infinity among them as above
@pytest.mark.parametrize("msg", [0, 1])
@pytest.mark.parametrize("n,do,B", [(30, 8, 1), (10, 16, 2), (30, 24, 3), (10, 32, 4), (30, 40, 1), (10, 56, 2), (30, 64, 4), (1, 8, 2)])
def test_edges_shared_by_lane_groups(n, do, B, msg):
    R, di = 2, 16
    H0, dH, V, a, W0 = model(do + B, n, R, di, do, B)
    m = 100 * n if n == 30 else 600 * n
    got, want = layer(n, R, m, di, do, B, 0, H0, dH, V, a, W0, msg)
    for k in want:
        tol = 2e-2 if msg else 10 * TOL
        assert np.abs(got[k] - want[k]).max() <= tol * np.abs(want[k]).max(), k
    if n > 1:
        dH[n // 2, 1] = np.inf
        got, want = layer(n, R, m, di, do, B, 0, np.abs(H0), dH, np.abs(V), a, W0, msg)
        hit = np.isinf(want["da"])
        assert hit.any()
        np.testing.assert_array_equal(got["da"][hit], want["da"][hit].astype(np.float32))


@pytest.mark.parametrize("d,B", [(16, 2), (36, 3), (64, 1)])
def test_shared_edges_on_a_batch_s_sub_graph(orc, d, B):
    """One positive: of the 100 edges per relation of a source, the last layer takes those into two vertices."""
    from paper_2201_02791_amd import synth
    from gpu_util import assert_step_close, gpu_step, oracle_step
    n, R, m = 60, 2, 6000
    spec = synth.scaled(synth.WORKLOADS[0], name="dense", seed=3, n_entities=n, n_relations=R, n_triples=m, d=d, n_bases=B,
                        n_pos=1, n_neg=0, n_parts=1, part_id=0, acts=[0, 0])
    rng = np.random.default_rng(d)
    head, rel, tail = (rng.integers(0, k, m).astype(np.int32) for k in (n, R, n))
    gp, ts, params, pos = gpu_step(spec, head, rel, tail, cone=True)
    op, res = oracle_step(orc, spec, head, rel, tail, params, pos)
    assert_step_close(ts, res, 1e-5, 1e-4, batch_rows=orc.batch_vertices(op, pos, res["neg_ent"]))
