"""The products of an fp32 layer in the relation-weight order, several in one launch: blocks that belong to one product or the
next, widths below and above a tile, graphs of one edge, layers without an input gradient.  Tolerance as in the
split-product tests (4e-6 of the largest element)."""
import numpy as np
import pytest

from oracle import oracle as orc
from test_gpu_split_products import TOL, model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("need_in", [True, False])
@pytest.mark.parametrize("n,R,m,di,do", [(1, 1, 1, 4, 4), (5, 2, 1, 132, 252), (40, 3, 30, 200, 36), (129, 1, 129, 32, 32),
                                         (1000, 10, 5000, 32, 32), (700, 200, 1500, 64, 200), (3000, 4, 20000, 256, 72)])
def test_products_of_a_layer(n, R, m, di, do, need_in):
    import torch
    from paper_2201_02791_amd import binding as kb
    rng = np.random.default_rng(n + m)
    head, rel, tail = (rng.integers(0, hi, m).astype(np.int32) for hi in (n, R, n))
    part, opart = kb.build_partition(head, rel, tail, n, R), orc.build_partition(head, rel, tail, n, R)
    n = part.n_vert
    H0, dH, V, a, W0 = model(n, n, R, di, do, 3)
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    lay = [dict(V=t(V), a=t(a), W0=t(W0), act=kb.ACT_IDENTITY, order=kb.ORDER_RELATION_WEIGHTS)]
    ws = torch.empty(kb.workspace_bytes(part, lay, 0), dtype=torch.uint8, device="cuda")
    H, out = t(H0), torch.empty(n, do, device="cuda")
    dH0 = torch.empty(n, di, device="cuda") if need_in else None
    grads = [{k: torch.empty_like(lay[0][k[1:]]) for k in ("dV", "da", "dW0")}]
    kb.rgcn_forward(part, lay, H, ws, out, 0)
    kb.rgcn_backward(part, lay, H, ws, t(dH), grads, dH0, 0)
    torch.cuda.synchronize()
    pre, h = orc.layer_forward(opart, V, a, W0, 0, H0)
    want = orc.layer_backward(opart, V, a, W0, 0, H0, pre, dH)
    got = dict(grads[0], out=out, **({"dH": dH0} if need_in else {}))
    want["out"] = h
    for k, v in got.items():
        assert np.abs(v.cpu().numpy() - want[k]).max() <= TOL * max(np.abs(want[k]).max(), 1e-30), k
