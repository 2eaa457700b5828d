"""The atomic-free scoring call where its gather can go wrong: four, some and 64 entities per block, entities whose
occurrences fall to several wavefronts of a block (a hub that is the head of half the batch), blocks without any
occurrence, more than 64 negatives, rows wider than a wavefront's 64 x 4 columns; batches on both sides of the index
that one launch builds (4096 occurrences, 16,384 entities).

Tolerance: a row of dH is an fp32 sum of up to 5000 terms: sqrt(5000) * 2^-24 = 4e-6 of the largest element; scores and
loss 1e-5."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,n_pos,n_neg,hub", [(50, 4, 3, 0, False), (900, 36, 700, 1, True), (20000, 200, 1500, 10, True),
                                                 (140000, 16, 5000, 3, True), (140001, 256, 3000, 70, False),
                                                 (300, 300, 40, 65, True), (131072, 8, 20, 1, False),
                                                 (16384, 8, 1, 0, False), (16384, 8, 128, 30, True), (16385, 8, 64, 30, True),
                                                 (700, 8, 4096 // 7, 5, True), (700, 8, 1366, 1, False)])
def test_scoring_against_fp64(n, d, n_pos, n_neg, hub):
    import torch
    from paper_2201_02791_amd import binding as kb
    rng = np.random.default_rng(n + d)
    R, m = 7, n + n_pos
    head, tail = rng.integers(0, n, m).astype(np.int32), rng.integers(0, n, m).astype(np.int32)
    head[:n] = np.arange(n)
    if hub:
        head[n:n + n_pos // 2] = 5
    rel = rng.integers(0, R, m).astype(np.int32)
    part = kb.build_partition(head, rel, tail, n, R)
    H = torch.randn(n, d, device="cuda") * 0.3
    M = torch.randn(R, d, device="cuda") * 0.3
    idx = np.concatenate([np.arange(n, n + n_pos // 2), rng.integers(0, m, n_pos - n_pos // 2)]).astype(np.int32)
    pos = torch.from_numpy(idx).cuda()
    ent = torch.zeros((n_pos, max(n_neg, 1)), dtype=torch.int32, device="cuda")
    side = torch.zeros((n_pos, max(n_neg, 1)), dtype=torch.uint8, device="cuda")
    kb.sample_negatives(part, pos, n_neg, kb.NEG_HEAD_OR_TAIL, 3, 4, ent, side)
    out = []
    for _ in range(2):
        scores, loss = torch.full((n_pos, 1 + n_neg), 9.0, device="cuda"), torch.zeros(1, device="cuda")
        dH, dM = torch.full((n, d), 9.0, device="cuda"), torch.full((R, d), 9.0, device="cuda")
        kb.distmult_score_loss(part, H, M, pos, ent, side, n_neg, scores, loss, dH, dM, index=kb.ScoreIndex(part, n_pos, n_neg, d))
        out.append((scores, loss, dH, dM))
    torch.cuda.synchronize()
    scores, loss, dH, dM = out[0]
    assert torch.equal(dH, out[1][2]) and torch.equal(loss, out[1][1])         # repeats bit for bit
    h, r, t = (torch.from_numpy(x[idx].astype(np.int64)).cuda()[:, None] for x in (head, rel, tail))
    e, sd = ent[:, :n_neg].long(), side[:, :n_neg].bool()
    s, o = torch.cat([h, torch.where(sd, e, h)], 1), torch.cat([t, torch.where(sd, t, e)], 1)
    H64, M64, T = H.double(), M.double(), n_pos * (1 + n_neg)
    g = (H64[s] * M64[r] * H64[o]).sum(2)
    y = torch.zeros_like(g)
    y[:, 0] = 1
    delta = ((torch.sigmoid(g) - y) / T)[:, :, None]
    want_dH, want_dM = torch.zeros_like(H64), torch.zeros_like(M64)
    want_dH.index_add_(0, s.flatten(), (delta * M64[r] * H64[o]).flatten(0, 1))
    want_dH.index_add_(0, o.flatten(), (delta * M64[r] * H64[s]).flatten(0, 1))
    want_dM.index_add_(0, r.flatten(), (delta * H64[s] * H64[o]).sum(1))
    want_loss = torch.nn.functional.softplus(torch.where(y > 0, -g, g)).sum() / T
    err = lambda x, w: float((x.double() - w).abs().max() / w.abs().max())  # noqa: E731
    assert err(scores, g) < 1e-5 and abs(float(loss) - float(want_loss)) < 1e-5 * float(want_loss)
    assert err(dH, want_dH) < 4e-6 and err(dM, want_dM) < 1e-5
    assert part.bad_ids() == 0
