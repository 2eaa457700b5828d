"""The calls whose speed this repository is held to: inputs, one pass, its work and its exact result.

Every case goes through `paper_2201_02791_amd.binding` or `TrainStep`, with the shapes of the five benchmark
workloads of `synth.py` (a tiny graph, the 14,541-entity knowledge graph whole and as one of eight partitions, the
citation-shaped graph, the large many-relation graph) and of the evaluation that `bench.py` runs.  Graphs are drawn
on the GPU with the same degree and relation statistics (power-law heads, bounded Zipf relations), so that a case is
made in well under a second.

Kinds of case:
  step    one training step of Algorithm 1: negatives, sub-graph of the batch, encoder forward, score and loss,
          encoder backward (two layers, ReLU then identity)
  layer   one RGCN layer, forward and backward, on the whole partition
  score   DistMult scores, cross-entropy loss and their gradients for a batch of positives and negatives
  rank    filtered link-prediction ranks against all entities, with MRR and Hits@k
  cand    ranks against a given list of candidates per query
  adam    the optimizer step on an entity table of which a batch read some rows
"""
import math

import numpy as np
import torch

DEV = "cuda"
MASK32 = 0xFFFFFFFF


# ------------------------------------------------------------------------------------------------ cases

def listed():
    return [
        # the smallest call: a whole step in which every kernel takes microseconds
        dict(name="step-tiny", kind="step", n_ent=1000, n_rel=10, n_tri=5000, heads="uniform", tails="uniform", zipf=1.1,
             parts=1, d=32, bases=4, order="relation", cone=True, dropout=0.0, n_pos=1024, n_neg=1, both=False),
        # the paper's mid-size knowledge graph as one partition, fp32, on the batch's sub-graph
        dict(name="step-mid", kind="step", n_ent=14541, n_rel=237, n_tri=272115, heads="power", tails="uniform", zipf=1.0,
             parts=1, d=200, bases=10, order="relation", cone=True, dropout=0.0, n_pos=30000, n_neg=10, both=True),
        # one of eight partitions of it, in the order the step is usually written in (TrainStep's default)
        dict(name="step-part-project", kind="step", n_ent=14541, n_rel=237, n_tri=272115, heads="power", tails="uniform",
             zipf=1.0, parts=8, d=200, bases=10, order="project", cone=False, dropout=0.0, n_pos=8192, n_neg=10, both=True),
        # a layer of the citation-shaped graph at its full size: 2.9 M vertices, 60 M message edges, one relation
        dict(name="layer-citation", kind="layer", n_ent=2900000, n_rel=1, n_tri=30000000, heads="power", tails="power",
             zipf=0.0, parts=16, d_in=128, d_out=128, bases=2, dtype="f32", order="relation", dropout=0.0, dh0=True),
        # the paper's large-graph hyper-parameters (fixed 128-wide features to 32, dropout 0.2) on a tenth of that graph
        dict(name="layer-features", kind="layer", n_ent=290001, n_rel=1, n_tri=3000000, heads="power", tails="power",
             zipf=0.0, parts=4, d_in=128, d_out=32, bases=2, dtype="f32", order="relation", dropout=0.2, dh0=False),
        # a layer of the large many-relation graph at its full size, bf16 messages
        dict(name="layer-bigkg-bf16", kind="layer", n_ent=1000000, n_rel=1000, n_tri=20000000, heads="power", tails="uniform",
             zipf=1.1, parts=4, d_in=256, d_out=256, bases=64, dtype="bf16", order="relation", dropout=0.0, dh0=True),
        # bf16 messages in the project-first order, at a twentieth of that size
        dict(name="layer-kg-bf16-project", kind="layer", n_ent=50021, n_rel=237, n_tri=1000003, heads="power", tails="uniform",
             zipf=1.1, parts=1, d_in=128, d_out=128, bases=16, dtype="bf16", order="project", dropout=0.0, dh0=True),
        # the scoring call of the large graph: 65,536 positives, 64 negatives each
        dict(name="score-bigkg", kind="score", n_ent=1000000, n_rel=1000, n_tri=2000000, d=256, n_pos=65536, n_neg=64, both=True),
        # evaluation of the mid-size graph: the size of FB15k-237's test split, training triples filtered
        dict(name="rank-mid", kind="rank", n_ent=14541, n_rel=237, n_known=272115, n_test=20466, d=200),
        # evaluation against a million entities
        dict(name="rank-big", kind="rank", n_ent=1000000, n_rel=1000, n_known=2000000, n_test=10000, d=256),
        # the citation graph's evaluation: 1000 given negative targets per query
        dict(name="cand-citation", kind="cand", n_ent=2900000, n_rel=1, n_query=20000, n_cand=1000, d=128),
        # Adam on the large graph's entity table, most of whose rows a batch's sub-graph reads
        dict(name="adam-table", kind="adam", n_rows=1000000, d=256, read=0.9),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi, mult):
    return max(mult, _log(rng, lo, hi) // mult * mult)


def draw(rng):
    kind = rng.choice(["step", "step", "layer", "layer", "layer", "score", "rank", "rank", "cand", "adam"])
    if kind == "step":
        n = _log(rng, 500, 40000)
        m, parts = n * rng.randint(4, 20) + rng.randint(0, 63), rng.choice([1, 1, 4, 8])
        return dict(kind=kind, n_ent=n, n_rel=_log(rng, 1, 300), n_tri=m, heads=rng.choice(["uniform", "power"]),
                    tails="uniform", zipf=rng.choice([1.0, 1.1]), parts=parts, d=_width(rng, 16, 256, 4),
                    bases=rng.randint(1, 12), order=rng.choice(["relation", "relation", "project"]), cone=rng.random() < 0.7,
                    dropout=rng.choice([0.0, 0.0, 0.2]), n_pos=min(_log(rng, 500, 30000), m // (2 * parts)),
                    n_neg=rng.choice([1, 1, 4, 10, 16]), both=rng.random() < 0.7)
    if kind == "layer":
        dtype = rng.choice(["f32", "f32", "bf16"])
        order = rng.choice(["relation", "relation", "relation", "project"])
        n = _log(rng, 5000, 1000000 if order == "relation" else 100000)
        many = rng.random() < 0.6
        return dict(kind=kind, n_ent=n, n_rel=_log(rng, 8, 1000) if many else rng.randint(1, 4),
                    n_tri=min(n * rng.randint(4, 20), 8000000) + rng.randint(0, 63), heads="power",
                    tails="uniform" if many else "power", zipf=1.1, parts=rng.choice([1, 4, 16]),
                    d_in=_width(rng, 32, 256, 8), d_out=_width(rng, 32, 256, 8),
                    bases=rng.randint(2, 64 if many and order == "relation" else 16), dtype=dtype, order=order,
                    dropout=rng.choice([0.0, 0.0, 0.2]), dh0=rng.random() < 0.8)
    if kind == "score":
        n = _log(rng, 5000, 1000000)
        return dict(kind=kind, n_ent=n, n_rel=_log(rng, 1, 1000), n_tri=2 * n + 70000, d=_width(rng, 32, 256, 4),
                    n_pos=_log(rng, 4000, 65536), n_neg=rng.choice([1, 4, 10, 16, 32, 64]), both=rng.random() < 0.7)
    if kind == "rank":
        n = _log(rng, 5000, 500000)
        return dict(kind=kind, n_ent=n, n_rel=_log(rng, 1, 1000), n_known=min(20 * n, 1000000), n_test=_log(rng, 500, 20000),
                    d=_width(rng, 32, 256, 4))
    if kind == "cand":
        return dict(kind=kind, n_ent=_log(rng, 20000, 2900000), n_rel=rng.randint(1, 20), n_query=_log(rng, 1000, 20000),
                    n_cand=rng.randint(50, 1000), d=_width(rng, 32, 256, 4))
    return dict(kind=kind, n_rows=_log(rng, 10000, 1000000), d=_width(rng, 32, 256, 4), read=round(rng.uniform(0.2, 1.0), 2))


# ------------------------------------------------------------------------------------------------ inputs

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _rand(shape, gen, std):
    return torch.randn(shape, generator=gen, device=DEV, dtype=torch.float32) * std


def _glorot(shape, gen):
    lim = math.sqrt(6.0 / (shape[-2] + shape[-1]))
    return (torch.rand(shape, generator=gen, device=DEV, dtype=torch.float32) * 2 - 1) * lim


def _entities(kind, n, m, gen, exponent):
    u = torch.rand(m, generator=gen, device=DEV, dtype=torch.float64)
    if kind == "uniform":
        return (u * n).long().clamp_(max=n - 1)
    # power law: entity x has weight min((x / n)^-a, cap), a = 1 / (exponent - 1); drawn by the inverse of the weight's
    # integral, then spread over the ids by a multiplicative permutation
    a, cap = 1.0 / (exponent - 1.0), min(1e4, max(8.0, n / 15.0))
    knee = cap ** (-1.0 / a)
    flat = cap * knee
    if abs(a - 1.0) < 1e-9:
        total = flat - math.log(knee)
        x = torch.where(u * total < flat, u * total / cap, knee * torch.exp(u * total - flat))
    else:
        total = flat + (1.0 - knee ** (1 - a)) / (1 - a)
        x = torch.where(u * total < flat, u * total / cap,
                        (knee ** (1 - a) + (1 - a) * (u * total - flat)).clamp_(min=1e-300) ** (1.0 / (1 - a)))
    mult = int(n * 0.6180339887) | 1
    while math.gcd(mult, n) != 1:
        mult += 2
    return ((x * n).long().clamp_(0, n - 1) * mult) % n


def _relations(n_rel, m, zipf, gen):
    if n_rel == 1:
        return torch.zeros(m, dtype=torch.int64, device=DEV)
    w = (np.arange(n_rel) + 1.0) ** -zipf
    cdf = torch.from_numpy(np.cumsum(w / w.sum())).to(DEV)
    return torch.searchsorted(cdf, torch.rand(m, generator=gen, device=DEV, dtype=torch.float64)).clamp_(max=n_rel - 1)


def _part_of(head, parts):
    return (((head * 0x9E3779B1) & MASK32) >> 8) % parts


def _graph(case, seed):
    gen = _gen(seed * 7 + 1)
    n, m = case["n_ent"], case["n_tri"]
    exponent = 2.0 if case.get("tails") == "power" else 2.1
    head = _entities(case.get("heads", "power"), n, m, gen, exponent)
    tail = _entities(case.get("tails", "uniform"), n, m, gen, exponent)
    rel = _relations(case["n_rel"], m, case.get("zipf", 1.1), gen)
    # an entity is there because a triple names it, and two hops from partition 0 reach nearly all of them: here each
    # is a head once, with a tail that partition 0 owns, so that every seed gives a partition of n_ent vertices
    ids = torch.arange(n, device=DEV)
    owned = ids[_part_of(ids, case.get("parts", 1)) == 0]
    head[:n] = ids
    tail[:n] = owned[(torch.rand(n, generator=gen, device=DEV, dtype=torch.float64) * len(owned)).long().clamp_(max=len(owned) - 1)]
    return head, rel, tail


def _host(x):
    return x.to(torch.int32).cpu().numpy()


def _inputs(case, seed):
    """Everything but the graph that is drawn: parameters, layer input, upstream gradients (float32, on the GPU)."""
    gen = _gen(seed * 7 + 2)
    k = case["kind"]
    if k == "step":
        d, B = case["d"], case["bases"]
        return dict(V=[_glorot((B, d, d), gen) for _ in range(2)], a=[_glorot((2 * case["n_rel"], B), gen) for _ in range(2)],
                    W0=[_glorot((d, d), gen) for _ in range(2)], M=_rand((case["n_rel"], d), gen, 0.1),
                    H0=_rand((case["n_ent"], d), gen, 0.1))
    if k == "layer":
        di, do, B = case["d_in"], case["d_out"], case["bases"]
        return dict(V=_glorot((B, di, do), gen), a=_glorot((2 * case["n_rel"], B), gen), W0=_glorot((di, do), gen),
                    H0=_rand((case["n_ent"], di), gen, 1.0 if case["n_rel"] == 1 else 0.1),
                    dH=_rand((case["n_ent"], do), gen, 1e-3))
    if k == "adam":
        n, d = case["n_rows"], case["d"]
        return dict(p=_rand((n, d), gen, 0.1), g=_rand((n, d), gen, 1e-3), m=_rand((n, d), gen, 1e-3),
                    v=_rand((n, d), gen, 1e-3).square_(),
                    mask=(torch.rand(n, generator=gen, device=DEV) < case["read"]).to(torch.uint8))
    out = dict(H=_rand((case["n_ent"], case["d"]), gen, 0.3), M=_rand((case["n_rel"], case["d"]), gen, 0.3))
    ints = lambda hi, *shape: torch.randint(0, hi, shape, generator=gen, device=DEV, dtype=torch.int32)  # noqa: E731
    if k == "rank":
        n, m = case["n_ent"], case["n_known"]
        known = (_entities("power", n, m, gen, 2.1), _relations(case["n_rel"], m, 1.1, gen), _entities("uniform", n, m, gen, 2.1))
        t = case["n_test"]
        out.update(known=known, th=_entities("power", n, t, gen, 2.1).int(), tr=_relations(case["n_rel"], t, 1.1, gen).int(), tt=ints(n, t))
    elif k == "cand":
        q = case["n_query"]
        out.update(fixed=ints(case["n_ent"], q), rel=ints(case["n_rel"], q), answer=ints(case["n_ent"], q),
                   cand=ints(case["n_ent"], q, case["n_cand"]))
    return out


def _batch(n_core, n_pos, seed):
    return torch.randperm(n_core, generator=torch.Generator().manual_seed(int(seed) * 7 + 3))[:n_pos].to(torch.int32)


def _order(kb, case):
    return kb.ORDER_RELATION_WEIGHTS if case["order"] == "relation" else kb.ORDER_PROJECT_FIRST


def prepare(case, seed):
    from paper_2201_02791_amd import binding as kb
    k, s = case["kind"], dict(case=dict(case), kb=kb)
    x = _inputs(case, seed)
    if k in ("step", "layer", "score"):
        head, rel, tail = (_host(v) for v in _graph(case, seed))
        s["part"] = part = kb.build_partition(head, rel, tail, case["n_ent"], case["n_rel"], case.get("parts", 1), 0, 2)
    if k == "step":
        from paper_2201_02791_amd.step import TrainStep
        params = {n: [t.cpu().numpy() for t in x[n]] for n in ("V", "a", "W0")}
        params.update(M=x["M"].cpu().numpy(), H0=x["H0"].cpu().numpy())
        ts = TrainStep(part, params, [kb.ACT_RELU, kb.ACT_IDENTITY], cone=case["cone"], order=_order(kb, case),
                       dropout=case["dropout"])
        ts.set_batch(_batch(part.n_core, case["n_pos"], seed).numpy(), case["n_neg"])
        s.update(ts=ts, mode=kb.NEG_HEAD_OR_TAIL if case["both"] else kb.NEG_TAIL, seed=1000 + seed)
    elif k == "layer":
        layer = dict(V=x["V"], a=x["a"], W0=x["W0"], act=kb.ACT_IDENTITY, order=_order(kb, case), dropout=case["dropout"],
                     drop_seed=1000 + seed, drop_step=5)
        msg = kb.MSG_BF16 if case["dtype"] == "bf16" else kb.MSG_F32
        H0, dH = x["H0"], x["dH"]
        s.update(layers=[layer], msg=msg, H0=H0, dH=dH, H=torch.empty_like(dH),
                 ws=torch.empty(kb.workspace_bytes(part, [layer], msg), dtype=torch.uint8, device=DEV),
                 grads=[dict(dV=torch.empty_like(x["V"]), da=torch.empty_like(x["a"]), dW0=torch.empty_like(x["W0"]))],
                 dH0=torch.empty_like(H0) if case["dh0"] else None)
    elif k == "score":
        n_pos, n_neg, d = case["n_pos"], case["n_neg"], case["d"]
        pos = _batch(part.n_core, n_pos, seed).to(DEV)
        ent = torch.empty((n_pos, n_neg), dtype=torch.int32, device=DEV)
        side = torch.empty((n_pos, n_neg), dtype=torch.uint8, device=DEV)
        kb.sample_negatives(part, pos, n_neg, kb.NEG_HEAD_OR_TAIL if case["both"] else kb.NEG_TAIL, 1000 + seed, 5, ent, side)
        H = x["H"]
        s.update(H=H, M=x["M"], pos=pos, ent=ent, side=side, scores=torch.empty((n_pos, 1 + n_neg), device=DEV),
                 loss=torch.zeros(1, device=DEV), dH=torch.empty_like(H), dM=torch.empty_like(x["M"]),
                 index=kb.ScoreIndex(part, n_pos, n_neg, d))
    elif k == "rank":
        s.update({n: x[n] for n in ("H", "M", "th", "tr", "tt")})
        s["filt"] = kb.EvalFilter(*(_host(v) for v in x["known"]), case["n_ent"], case["n_rel"])
        s["ws"] = torch.empty(kb.eval_workspace_bytes(2 * case["n_test"], case["d"]), dtype=torch.uint8, device=DEV)
    elif k == "cand":
        s.update({n: x[n] for n in ("H", "M", "fixed", "rel", "answer", "cand")})
        s["ws"] = torch.empty(kb.eval_workspace_bytes(case["n_query"], case["d"]), dtype=torch.uint8, device=DEV)
    else:
        s.update(x, t=0)
    return s


# ------------------------------------------------------------------------------------------------ one pass

def run(s):
    case, kb = s["case"], s["kb"]
    k = case["kind"]
    if k == "step":
        ts = s["ts"]
        ts.run(s["mode"], s["seed"], 5)
        out = dict(scores=ts.scores, loss=ts.loss, dM=ts.dM, dH0=ts.dH0)
        for l, g in enumerate(ts.grads):
            out.update({"%s_%d" % (n, l): g[n] for n in ("dV", "da", "dW0")})
        return out
    if k == "layer":
        kb.rgcn_forward(s["part"], s["layers"], s["H0"], s["ws"], s["H"], s["msg"])
        kb.rgcn_backward(s["part"], s["layers"], s["H0"], s["ws"], s["dH"], s["grads"], s["dH0"], s["msg"])
        return dict(H=s["H"], dH0=s["dH0"], **s["grads"][0])
    if k == "score":
        kb.distmult_score_loss(s["part"], s["H"], s["M"], s["pos"], s["ent"], s["side"], case["n_neg"], s["scores"], s["loss"],
                               s["dH"], s["dM"], index=s["index"])
        return dict(scores=s["scores"], loss=s["loss"], dH=s["dH"], dM=s["dM"])
    if k == "rank":
        higher, equal = kb.eval_rank_all(s["H"], s["M"], s["th"], s["tr"], s["tt"], s["filt"], s["ws"])
        # the mean position over the ties, as a program reports it: two scores within fp32 rounding of each other may
        # change places, so the counts themselves are whole numbers only up to such pairs
        return dict(position=torch.add(higher.float(), equal, alpha=0.5), metrics=kb.eval_metrics(higher, equal))
    if k == "cand":
        higher, equal = kb.eval_rank_candidates(s["H"], s["M"], s["fixed"], s["rel"], s["answer"], s["cand"], s["ws"])
        return dict(higher=higher, equal=equal, metrics=kb.eval_metrics(higher, equal))
    s["t"] += 1
    kb.optimizer_step(kb.OPT_ADAM, s["p"], s["g"], s["m"], s["v"], t=s["t"], rows=True, row_mask=s["mask"])
    return dict(p=s["p"], m=s["m"], v=s["v"])


# ------------------------------------------------------------------------------------------------ work and tolerance

def _layer_work(n, m, n_rel, di, do, B, order, dh0):
    """One layer, forward and backward: the edge list, the parameters and each vertex's rows once."""
    E = 2.0 * m
    runs = min(E, 2.0 * n_rel * n)
    mult = min(runs, float(n) * B) if order == "relation" else float(n) * B
    passes = 3.0 if dh0 else 2.0
    return dict(bytes=E * 12 + n * 4.0 * (di * (2 if dh0 else 1) + 2 * do) + 8.0 * ((B + 1) * di * do + 2 * n_rel * B),
                flops=passes * 2.0 * di * do * (mult + n) + passes * 2.0 * E * min(di, do))


def work(case):
    k = case["kind"]
    if k == "step":
        d, B, n = case["d"], case["bases"], case["n_ent"]
        w = _layer_work(n, case["n_tri"], case["n_rel"], d, d, B, case["order"], True)
        n_pos = case["n_pos"]
        return dict(bytes=2 * w["bytes"] + n_pos * (1.0 + case["n_neg"]) * 9 + 8.0 * case["n_rel"] * d,
                    flops=2 * w["flops"] + n_pos * (1.0 + case["n_neg"]) * 8 * d)
    if k == "layer":
        return _layer_work(case["n_ent"], case["n_tri"], case["n_rel"], case["d_in"], case["d_out"], case["bases"],
                           case["order"], case["dh0"])
    if k == "score":
        t = case["n_pos"] * (1.0 + case["n_neg"])
        return dict(bytes=8.0 * case["n_ent"] * case["d"] + 8.0 * case["n_rel"] * case["d"] + t * 9, flops=t * 8 * case["d"])
    if k == "rank":
        return dict(bytes=4.0 * case["n_ent"] * case["d"] + 2.0 * case["n_test"] * 12, flops=4.0 * case["n_test"] * case["n_ent"] * case["d"])
    if k == "cand":
        rows = case["n_query"] * (case["n_cand"] + 2.0)
        return dict(bytes=4.0 * case["n_ent"] * case["d"] + rows * 4, flops=rows * 2 * case["d"])
    return dict(bytes=case["n_rows"] * (1.0 + 28.0 * case["d"] * case["read"]), flops=case["n_rows"] * case["read"] * case["d"] * 12)


def tolerance(case):
    k = case["kind"]
    if k == "step":
        # fp32 sums in another order move a pre-activation across the ReLU's kink now and then, and with it whole
        # terms of the first layer's gradients; everything else agrees to 1e-6
        return dict(rel=4e-3, max=0.5)
    if k == "layer":
        return dict(rel=1e-2) if case["dtype"] == "bf16" else dict(rel=1e-5)
    if k == "rank":
        return dict(rel=4e-5, max=2e-3)
    if k == "cand":
        return dict(rel=1e-4, differ=1e-3)
    return dict(rel=1e-5)


# ------------------------------------------------------------------------------------------------ exact results

def _philox(c, key):
    """Philox4x32-10 (Salmon et al., SC'11) on int64 tensors that hold 32-bit words."""
    c, (k0, k1) = list(c), key
    for _ in range(10):
        p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57
        c = [((p1 >> 32) & MASK32) ^ c[1] ^ k0, p1 & MASK32, ((p0 >> 32) & MASK32) ^ c[3] ^ k1, p0 & MASK32]
        k0, k1 = (k0 + 0x9E3779B9) & MASK32, (k1 + 0xBB67AE85) & MASK32
    return c


def _local(case, graph):
    """The partition in local ids: core triples, message edges with their 1/c, and the candidates for negatives."""
    head, rel, tail = graph
    n, R = case["n_ent"], case["n_rel"]
    parts = case.get("parts", 1)
    core = (_part_of(head, parts) == 0).nonzero().flatten()
    seen = torch.zeros(n, dtype=torch.bool, device=DEV)
    seen[head[core]] = True
    seen[tail[core]] = True
    ends = seen.clone()
    src, dst, r2 = torch.cat([head, tail]), torch.cat([tail, head]), torch.cat([rel, rel + R])
    for _ in range(2):
        keep = seen[dst]
        nxt = seen.clone()
        nxt[src[keep]] = True
        seen = nxt
    src, dst, r2 = src[keep], dst[keep], r2[keep]
    lid = torch.cumsum(seen.long(), 0) - 1
    src, dst, N = lid[src], lid[dst], n
    order = torch.argsort(r2 * N + dst)
    src, dst, r2 = src[order], dst[order], r2[order]
    _, run, count = torch.unique_consecutive(r2 * N + dst, return_inverse=True, return_counts=True)
    ptr = [0] + torch.cumsum(torch.bincount(r2, minlength=2 * R), 0).tolist()
    return dict(src=src, dst=dst, w=1.0 / count.double()[run], ptr=ptr, h=lid[head[core]], r=rel[core], t=lid[tail[core]],
                cand=lid[ends.nonzero().flatten()])


def _drop(x, case, seed, layer):
    if case["dropout"] == 0.0:
        return torch.ones_like(x)
    p = float(np.float32(case["dropout"]))
    i = torch.arange(x.shape[0], device=DEV)[:, None]
    j = torch.arange(x.shape[1] // 4, device=DEV)[None, :]
    z = torch.zeros_like(i + j)
    words = _philox([i + z, j + z, z + 5, z], (seed & MASK32, (layer + 1) ^ (seed >> 32)))
    keep = torch.stack(words, 2).reshape(x.shape) >= int(p * 2.0 ** 32)
    return keep.double() / (1.0 - p)


def _chunks(ptr, most):
    for r in range(len(ptr) - 1):
        for b in range(ptr[r], ptr[r + 1], most):
            yield r, slice(b, min(b + most, ptr[r + 1]))


def _layer_forward(g, H, V, a, W0):
    W = (a @ V.flatten(1)).view(-1, *V.shape[1:])
    out = H @ W0
    for r, e in _chunks(g["ptr"], 1 << 21):
        out.index_add_(0, g["dst"][e], (H[g["src"][e]] * g["w"][e, None]) @ W[r])
    return out


def _layer_backward(g, H, V, a, W0, G):
    W = (a @ V.flatten(1)).view(-1, *V.shape[1:])
    dW, dH = torch.zeros_like(W), G @ W0.T
    for r, e in _chunks(g["ptr"], 1 << 21):
        x, y, w = H[g["src"][e]], G[g["dst"][e]], g["w"][e, None]
        dW[r] += (x * w).T @ y
        dH.index_add_(0, g["src"][e], (y @ W[r].T) * w)
    dW = dW.flatten(1)
    return dict(dV=(a.T @ dW).view_as(V), da=dW @ V.flatten(1).T, dW0=H.T @ G), dH


def _negatives(g, case, seed, pos):
    n_neg = case["n_neg"]
    slot = torch.arange(n_neg, device=DEV)[None, :]
    c = pos.long()[:, None] + torch.zeros_like(slot)
    z = torch.zeros_like(c)
    x = _philox([c, slot + z, z + 5, z], ((1000 + seed) & MASK32, (1000 + seed) >> 32))
    ent = g["cand"][(x[0] * len(g["cand"])) >> 32]
    return ent, (x[1] >= 1 << 31) if case["both"] else torch.zeros_like(ent, dtype=torch.bool)


def _score(g, case, seed, H, M, pos):
    pos = pos.long()
    T = pos.numel() * (1.0 + case["n_neg"])
    dH, dM, loss, scores = torch.zeros_like(H), torch.zeros_like(M), 0.0, []
    for p in pos.split(max(1, (1 << 27) // ((1 + case["n_neg"]) * H.shape[1]))):
        ent, side = _negatives(g, case, seed, p)
        h, r, t = (g[n][p][:, None] for n in "hrt")
        s = torch.cat([h, torch.where(side, ent, h)], 1)
        o = torch.cat([t, torch.where(side, t, ent)], 1)
        hs, ho, m = H[s], H[o], M[r]
        q = (hs * m * ho).sum(2)
        y = torch.zeros_like(q)
        y[:, 0] = 1.0
        loss = loss + torch.nn.functional.softplus(torch.where(y > 0, -q, q)).sum() / T
        delta = ((torch.sigmoid(q) - y) / T)[:, :, None]
        dH.index_add_(0, s.flatten(), (delta * m * ho).flatten(0, 1))
        dH.index_add_(0, o.flatten(), (delta * m * hs).flatten(0, 1))
        dM.index_add_(0, r.flatten(), (delta * hs * ho).sum(1))
        scores.append(q)
    return dict(scores=torch.cat(scores), loss=loss.reshape(1), dH=dH, dM=dM)


def _mean_ranks(higher, equal):
    rank = 1.0 + higher.double() + 0.5 * equal.double()
    return torch.stack([(1.0 / rank).mean()] + [(rank <= k).double().mean() for k in (1, 3, 10)])


def exact(case, seed):
    k, x = case["kind"], _inputs(case, seed)
    f64 = lambda t: t.double()  # noqa: E731
    if k == "step":
        g = _local(case, _graph(case, seed))
        V, a, W0 = ([f64(t) for t in x[n]] for n in ("V", "a", "W0"))
        H, M = f64(x["H0"]), f64(x["M"])
        pos = _batch(g["h"].numel(), case["n_pos"], seed).to(DEV)
        keep = [_drop(H, case, 1000 + seed, l) for l in range(2)]
        X0 = H * keep[0]
        X1 = torch.relu(_layer_forward(g, X0, V[0], a[0], W0[0])) * keep[1]
        s = _score(g, case, seed, _layer_forward(g, X1, V[1], a[1], W0[1]), M, pos)
        top, _ = _layer_backward(g, X1, V[1], a[1], W0[1], s.pop("dH"))
        # the first layer's gradients jump where a pre-activation is within rounding of the ReLU's kink: no value
        # in 64 bits is theirs alone
        out = dict(s, dH0=None)
        for n in ("dV", "da", "dW0"):
            out.update({n + "_0": None, n + "_1": top[n]})
        return out
    if k == "layer":
        g = _local(case, _graph(case, seed))
        H, V, a, W0 = f64(x["H0"]), f64(x["V"]), f64(x["a"]), f64(x["W0"])
        keep = _drop(H, case, 1000 + seed, 0)
        H *= keep
        out = _layer_forward(g, H, V, a, W0)
        grads, dH0 = _layer_backward(g, H, V, a, W0, f64(x["dH"]))
        return dict(H=out, dH0=dH0 * keep if case["dh0"] else None, **grads)
    if k == "score":
        g = _local(case, _graph(case, seed))
        pos = _batch(g["h"].numel(), case["n_pos"], seed).to(DEV)
        return _score(g, case, seed, f64(x["H"]), f64(x["M"]), pos)
    if k == "rank":
        H, M, n, R = f64(x["H"]), f64(x["M"]), case["n_ent"], case["n_rel"]
        kh, kr, kt = x["known"]
        h, r, t = x["th"].long(), x["tr"].long(), x["tt"].long()
        higher, equal = [], []
        for fixed, answer, keys, others in ((h, t, kh * R + kr, kt), (t, h, kt * R + kr, kh)):
            pairs = torch.unique(keys * n + others)
            keys, others = pairs // n, pairs % n
            q = fixed * R + r
            beg, end = torch.searchsorted(keys, q), torch.searchsorted(keys, q, right=True)
            for b in range(0, len(q), 512):
                e = slice(b, min(b + 512, len(q)))
                s = (H[fixed[e]] * M[r[e]]) @ H.T
                top = s.gather(1, answer[e, None])
                num = end[e] - beg[e]                      # known answers of these queries, as (row, entity) pairs
                row = torch.repeat_interleave(torch.arange(len(num), device=DEV), num)
                at = torch.arange(len(row), device=DEV) - (torch.cumsum(num, 0) - num)[row] + beg[e][row]
                s[row, others[at]] = -math.inf
                s.scatter_(1, answer[e, None], -math.inf)
                higher.append((s > top).sum(1))
                equal.append((s == top).sum(1))
        higher, equal = torch.cat(higher), torch.cat(equal)
        return dict(position=higher.double() + 0.5 * equal, metrics=_mean_ranks(higher, equal))
    if k == "cand":
        H, M, cand = f64(x["H"]), f64(x["M"]), x["cand"].long()
        higher, equal = [], []
        for b in range(0, case["n_query"], 500):
            e = slice(b, min(b + 500, case["n_query"]))
            q = H[x["fixed"][e].long()] * M[x["rel"][e].long()]
            ans = x["answer"][e].long()
            s = (H[cand[e]] * q[:, None]).sum(2)
            top = (H[ans] * q).sum(1, keepdim=True)
            s[cand[e] == ans[:, None]] = -math.inf
            higher.append((s > top).sum(1))
            equal.append((s == top).sum(1))
        higher, equal = torch.cat(higher).int(), torch.cat(equal).int()
        return dict(higher=higher, equal=equal, metrics=_mean_ranks(higher, equal))
    p, g, m, v = (f64(x[n]) for n in "pgmv")
    on = x["mask"].bool()[:, None]
    lr, b1, b2, eps = (float(np.float32(c)) for c in (0.01, 0.9, 0.999, 1e-8))
    m1, v1 = b1 * m + (1 - b1) * g, b2 * v + (1 - b2) * g * g
    step = lr * (m1 / (1 - b1)) / (torch.sqrt(v1 / (1 - b2)) + eps)
    return dict(p=torch.where(on, p - step, p), m=torch.where(on, m1, m), v=torch.where(on, v1, v))
