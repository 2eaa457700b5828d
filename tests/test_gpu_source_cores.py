"""Backward pass of the project-first neighbour sum on the matrix cores (nine bases or more, or fewer where sources have many
relations): every class of widths and their edges, 16 bases and remainders, sources whose groups fill, miss or overflow a
tile of 16, more than one page of 64 edges and one unit of 256, infinities.  Tolerances as for the vector form."""
import numpy as np
import pytest

from test_gpu_split_products import TOL, layer, model

pytestmark = pytest.mark.gpu


def compare(n, R, m, do, B, msg, inf=False):
    di = 16
    H0, dH, V, a, W0 = model(do + B, n, R, di, do, B)
    if inf:
        H0, V = np.abs(H0), np.abs(V)
        dH[n // 2, 1] = np.inf
    got, want = layer(n, R, m, di, do, B, 0, H0, dH, V, a, W0, msg)
    if inf:
        hit = np.isinf(want["da"])
        assert hit.any() and not np.isnan(want["da"]).any()
        np.testing.assert_array_equal(got["da"][hit], want["da"][hit].astype(np.float32))
        assert np.isfinite(got["da"][~hit]).all()
        return
    for k in want:
        tol = 2e-2 if msg else 10 * TOL
        assert np.abs(got[k] - want[k]).max() <= tol * np.abs(want[k]).max(), k


@pytest.mark.parametrize("msg", [0, 1])
@pytest.mark.parametrize("do,B", [(40, 9), (64, 16), (64, 1), (72, 9), (128, 5), (128, 17), (136, 16), (200, 5), (208, 12),
                                  (216, 9), (256, 33)])
def test_widths_and_bases(do, B, msg):
    compare(61, 30, 60 * 61, do, B, msg)


@pytest.mark.parametrize("do,B", [(36, 10), (100, 6), (204, 16), (252, 9)])
def test_fp32_widths_that_end_inside_a_block_of_columns(do, B):
    compare(47, 40, 50 * 47, do, B, 0)


@pytest.mark.parametrize("n,R,m", [(500, 3, 700), (200, 9, 1700), (40, 300, 3000), (3, 2, 1500), (2, 400, 900)])
@pytest.mark.parametrize("do,B", [(64, 9), (128, 12), (200, 10)])
def test_fill_of_the_tiles(n, R, m, do, B):
    """Sources with one or two groups, about 16, more than a page's 64, edge lists of several units."""
    compare(n, R, m, do, B, 0)


@pytest.mark.parametrize("do,B,msg", [(40, 9, 0), (104, 10, 1), (200, 16, 0), (216, 9, 0)])
def test_infinite_gradients_stay_infinite(do, B, msg):
    compare(40, 3, 800, do, B, msg, inf=True)


@pytest.mark.parametrize("d,B", [(64, 9), (136, 12)])
def test_a_batch_s_sub_graph_takes_some_of_the_edges(orc, d, B):
    from paper_2201_02791_amd import synth
    from gpu_util import assert_step_close, gpu_step, oracle_step
    n, R, m = 80, 6, 6000
    spec = synth.scaled(synth.WORKLOADS[0], name="part", seed=3, n_entities=n, n_relations=R, n_triples=m, d=d, n_bases=B,
                        n_pos=3, n_neg=1, n_parts=1, part_id=0, acts=[0, 0])
    rng = np.random.default_rng(d)
    head, rel, tail = (rng.integers(0, k, m).astype(np.int32) for k in (n, R, n))
    gp, ts, params, pos = gpu_step(spec, head, rel, tail, cone=True)
    op, res = oracle_step(orc, spec, head, rel, tail, params, pos)
    assert_step_close(ts, res, 1e-5, 1e-4, batch_rows=orc.batch_vertices(op, pos, res["neg_ent"]))


@pytest.mark.parametrize("d,B", [(64, 9), (128, 12), (200, 10), (256, 16)])
def test_dot_products_in_short_chains(d, B):
    """One edge per relation and numbers of one sign: a coefficient's gradient is one dot product of d terms.  In u = 2^-24, a
    rounding moves a sum by 0.4 u (rms); 16 chains of at most 16 terms, two sums of pairs and d / 64 - 1 more leave about
    0.4 sqrt(16 / 3 / 4 + 1 + 1 + 1) u = 0.8 u, and the terms' own errors (six bf16 products each, 2 u) another 2 u / sqrt(d).
    Chains of d / 2 terms: 0.4 sqrt(d / 6) u, 2.3 u at 200."""
    import torch
    from paper_2201_02791_amd import binding as kb
    print("[case] chains", d, B, flush=True)
    n, R, di = 3000, 1500, 16
    ids = np.arange(R, dtype=np.int32)
    part = kb.build_partition(ids, ids, ids + R, n, R, 1, 0, 2)
    assert part.n_edge == 2 * R and part.n_vert == n
    gen = torch.Generator(device="cuda").manual_seed(d)
    t = lambda *s: torch.rand(s, generator=gen, device="cuda") + 0.5  # noqa: E731
    lay = dict(V=t(B, di, d), a=t(2 * R, B), W0=t(di, d), act=kb.ACT_IDENTITY, order=kb.ORDER_PROJECT_FIRST)
    H0, G = t(n, di), t(n, d)
    ws = torch.empty(kb.workspace_bytes(part, [lay], 0), dtype=torch.uint8, device="cuda")
    grads = [{k: torch.empty_like(lay[k[1:]]) for k in ("dV", "da", "dW0")}]
    kb.rgcn_forward(part, [lay], H0, ws, torch.empty_like(G), 0)
    kb.rgcn_backward(part, [lay], H0, ws, G, grads, torch.empty_like(H0), 0)
    src = torch.from_numpy(part.export("col_src").astype(np.int64)).cuda()          # one run per edge, in relation order
    dst = torch.from_numpy(part.export("seg_dst").astype(np.int64)).cuda()
    want = torch.stack([((H0.double() @ lay["V"][b].double())[src] * G.double()[dst]).sum(1) for b in range(B)], 1)
    off = (grads[0]["da"].double() / want - 1.0) * 2.0 ** 24
    rms = float(off.square().mean().sqrt())
    print("rms error in 2^-24:", rms, flush=True)
    assert rms <= 1.4
