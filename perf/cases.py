"""The cases by which the speed of this library is measured: what users of it run, through its public calls.

Four kinds of program use the library:

  train     a training loop: one stx_train_step per batch, each call naming the batch after it, negatives drawn on
            the way, tables updated in place.  The loop walks the full batches of a graph, one after the other.
  calls     a loop that wants the gradients in hand (an optimiser of its own, a gradient check): the separate calls
            stx_sample_negatives, stx_build_incidence, stx_forward, stx_backward, stx_sgd_step on each batch.
  rank      an evaluation: stx_rank of held-out triplets against every entity, tail side and head side.
  semiring  DistMult / ComplEx / RotatE scoring rows for a loss of the user's: stx_spmm_semiring, then
            stx_spmm_semiring_t for the gradient of that loss.

Inputs are those of paper_2502_16949_amd/workloads.py (Zipf graphs, uniform tables), drawn on the GPU here.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2502_16949_amd import binding as B

DEV = "cuda:0"
KINDS = {"distmult": B.STX_DISTMULT, "complex": B.STX_COMPLEX, "rotate": B.STX_ROTATE}


def _train(name, model, dist, n_ent, n_rel, dim, batch, n_neg, n_batches, margin, lr, zipf_ent, zipf_rel, rel_dim=0, op="train"):
    return {"name": name, "op": op, "model": model, "dist": dist, "n_ent": n_ent, "n_rel": n_rel, "dim": dim,
            "rel_dim": rel_dim or dim, "batch": batch, "n_neg": n_neg, "n_batches": n_batches, "margin": margin, "lr": lr,
            "zipf_ent": zipf_ent, "zipf_rel": zipf_rel}


def _rank(name, model, dist, n_ent, n_rel, dim, queries, zipf_ent, zipf_rel, rel_dim=0):
    return {"name": name, "op": "rank", "model": model, "dist": dist, "n_ent": n_ent, "n_rel": n_rel, "dim": dim,
            "rel_dim": rel_dim or dim, "queries": queries, "zipf_ent": zipf_ent, "zipf_rel": zipf_rel}


def listed():
    return [
        # the smallest step: a small graph trained with small batches, where launches and the host count
        _train("train_tiny", "transe", "l2", 1_000, 20, 32, 1_024, 1, 9, 1.0, 0.01, 0.0, 0.0),
        # the ordinary step, and the shape of the headline benchmark: an FB15k-sized graph, 32,768 positives
        _train("train_transe", "transe", "l1", 15_000, 1_350, 128, 32_768, 1, 14, 1.0, 0.01, 1.1, 1.3),
        # the same graph with relation hyperplanes
        _train("train_transh", "transh", "l2", 15_000, 1_350, 128, 32_768, 1, 14, 1.0, 0.01, 1.1, 1.3),
        # an FB15k-237-sized graph with a projection matrix per relation: bf16 products on the matrix cores
        _train("train_transr", "transr", "l2", 14_500, 237, 128, 16_384, 1, 16, 1.0, 0.0004, 1.1, 1.3),
        # the largest table: 4 M entities, four negatives per positive, nothing fits a cache
        _train("train_toruse_4m", "toruse", "torus_l1", 4_000_000, 1_000, 128, 262_144, 4, 20, 1.0, 0.01, 1.05, 1.2),
        # the widest rows and the largest batch: the paper's own training shape
        _train("train_wide", "transe", "l2", 14_951, 1_345, 1_024, 393_216, 1, 2, 0.5, 0.0004, 1.1, 1.3),
        # gradients in hand, at sizes that fit nothing evenly: five negatives, an odd batch, rows of 50 float4
        _train("calls_ragged", "toruse", "torus_l2", 40_559, 19, 200, 9_999, 5, 7, 1.0, 0.01, 1.05, 1.2, op="calls"),
        # evaluation of the ordinary model: a test split of FB15k's size against all entities
        _rank("rank_transe", "transe", "l1", 15_000, 1_350, 128, 59_071, 1.1, 1.3),
        # evaluation of the wide model during training: a sample of the test split
        _rank("rank_wide", "transe", "l2", 14_951, 1_345, 1_024, 4_096, 1.1, 1.3),
        # evaluation with projection matrices: a test split of FB15k-237's size, a table projected per relation
        _rank("rank_transr", "transr", "l2", 14_500, 237, 128, 20_466, 1.1, 1.3),
        # a few queries against the largest table, as a link-prediction service asks them
        _rank("rank_few_4m", "toruse", "torus_l1", 4_000_000, 1_000, 128, 256, 1.05, 1.2),
        # ComplEx on the ordinary graph: product and gradient of one batch
        {"name": "semiring_complex", "op": "semiring", "kind": "complex", "n_ent": 15_000, "n_rel": 1_350, "dim": 128,
         "batch": 32_768, "n_neg": 1, "zipf_ent": 1.1, "zipf_rel": 1.3},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["train", "train", "train", "calls", "calls", "rank", "rank", "semiring"])
    model = rng.choice(["transe", "transe", "toruse", "transh", "transr"]) if op != "semiring" else "transe"
    dist = rng.choice({"toruse": ["torus_l1", "torus_l2"], "transe": ["l1", "l2", "l2_sq"]}.get(model, ["l1", "l2"]))
    c = {"op": op, "zipf_ent": rng.choice([0.0, 1.05, 1.1]), "zipf_rel": rng.choice([0.0, 1.2, 1.3]),
         "n_ent": _log_int(rng, 1_000, 4_000_000), "n_rel": _log_int(rng, 11, 1_350)}
    if model == "transr":                       # projections come in 32-wide tiles, up to 256
        c["n_ent"] = _log_int(rng, 1_000, 200_000)
        c["dim"], c["rel_dim"] = rng.choice([32, 64, 96, 128, 192, 256]), rng.choice([32, 64, 128, 256])
    else:
        c["dim"] = 4 * _log_int(rng, 4, 256)
        c["rel_dim"] = c["dim"]
    width = max(c["dim"], c["rel_dim"])
    if op == "rank":
        # at most a third of the steps of the largest listed evaluation, after what a step costs for the kind
        steps = 4.0e10 / (2.5 if model == "toruse" else 2.0 if model in ("transh", "transr") else 1.0)
        most = int(steps / (c["n_ent"] * width))
        if model == "transr":                   # one projected table per relation that occurs
            c["n_rel"] = max(1, min(c["n_rel"], int(2.0e11 / (c["n_ent"] * c["dim"] * c["rel_dim"]))))
        c.update(model=model, dist=dist, queries=_log_int(rng, 1, max(2, min(59_071, most))))
        return c
    c["n_neg"] = rng.choice([1, 1, 1, 2, 3, 4, 5, 8])
    rows = int(4.0e8 / (3 if model in ("transh", "transr") or op == "semiring" else 1) / width)   # a step's rows, by memory traffic
    c["batch"] = min(_log_int(rng, 512, 393_216), min(rows, 1_310_720) // (1 + c["n_neg"]))
    if op == "semiring":
        c["kind"] = rng.choice(sorted(KINDS))
        del c["rel_dim"]
        return c
    c.update(model=model, dist=dist, n_batches=rng.choice([2, 3, 5]), margin=rng.choice([0.5, 1.0]), lr=0.01)
    if model == "transr":                       # a matrix takes the sum of its rows' rank-one terms
        c["lr"] = round(min(0.0004, 6.5 / c["batch"]), 8)
    if dist == "l2_sq":                         # the gradient grows with y: the mean keeps hot columns stable
        c["mean"] = True
    return c


# ---- inputs ---------------------------------------------------------------------------------------------------

def _zipf(n_items, s, size, gen):
    """size ids with P(rank j) proportional to j**-s over a random order of the items; s == 0: uniform."""
    if s == 0.0:
        return torch.randint(0, n_items, (size,), generator=gen, device=DEV, dtype=torch.int32)
    cdf = torch.cumsum(torch.arange(1, n_items + 1, device=DEV, dtype=torch.float64) ** (-s), 0)
    u = torch.rand(size, generator=gen, device=DEV, dtype=torch.float64) * cdf[-1]
    rank = torch.searchsorted(cdf, u, right=True).clamp_(max=n_items - 1)
    return torch.randperm(n_items, generator=gen, device=DEV)[rank].to(torch.int32)


def _triplets(c, m, gen):
    return (_zipf(c["n_ent"], c["zipf_ent"], m, gen), _zipf(c["n_rel"], c["zipf_rel"], m, gen),
            _zipf(c["n_ent"], c["zipf_ent"], m, gen))


def _uniform(rows, cols, gen):
    a = 6.0 / math.sqrt(cols)
    return torch.empty(rows, cols, device=DEV).uniform_(-a, a, generator=gen)


def _tables(c, model, gen):
    if model in ("transe", "toruse"):
        x = _uniform(c["n_ent"] + c["n_rel"], c["dim"], gen)
        if model == "toruse":
            x = x - torch.floor(x)
            x[x >= 1.0] = 0.0
        return B.Params(x)
    ent, rel = _uniform(c["n_ent"], c["dim"], gen), _uniform(c["n_rel"], c["rel_dim"], gen)
    if model == "transh":
        w = torch.randn(c["n_rel"], c["dim"], generator=gen, device=DEV)
        return B.Params(ent, rel, w=w / w.norm(dim=1, keepdim=True))
    m = torch.randn(c["n_rel"], c["rel_dim"], c["dim"], generator=gen, device=DEV) * math.sqrt(1.0 / c["dim"])
    return B.Params(ent, rel, proj=m)


class _State:
    pass


def prepare(case, seed):
    """Tables, triplets, a context with its workspace and the output arrays, as a program holds them."""
    c, s = case, _State()
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    s.op = c["op"]
    model = c.get("model", "transe")
    flags = {"transh": B.STX_FLAG_RENORM_W, "transr": B.STX_FLAG_BF16_PROJ}.get(model, 0)
    s.params = _tables(c, model, gen)
    i32 = dict(dtype=torch.int32, device=DEV)
    f32 = dict(dtype=torch.float32, device=DEV)
    if s.op == "rank":
        nq = c["queries"]
        s.ctx = B.Context(B.make_config(model, c["dist"], c["n_ent"], c["n_rel"], c["dim"], 8, 1, rel_dim=c["rel_dim"],
                                        flags=flags), DEV)
        s.h, s.r, s.t = _triplets(c, nq, gen)
        need = B.stx_rank_work_bytes(s.ctx, nq)
        s.work = torch.empty(need + 256, dtype=torch.uint8, device=DEV) if need else None
        s.score, s.less, s.equal = torch.zeros(2, nq, **f32), torch.zeros(2, nq, **i32), torch.zeros(2, nq, **i32)
        return s
    b, k = c["batch"], c["n_neg"]
    s.n_neg, s.neg_seed = k, 3000 + int(seed)
    s.m = b * c.get("n_batches", 1)
    cfg = B.make_config(model, c.get("dist", "l2"), c["n_ent"], c["n_rel"], c["dim"], b, k, rel_dim=c.get("rel_dim", 0),
                        margin=c.get("margin", 1.0), reduce=B.STX_MEAN if c.get("mean") else B.STX_SUM, flags=flags)
    s.ctx = B.Context(cfg, DEV)
    s.inc = B.Incidence(s.ctx)
    s.inc.at_touched_cols.zero_()               # only the touched columns' part is written
    s.inc.at_seg_ptr.zero_()
    h, r, t = _triplets(c, s.m, gen)
    s.batches = [(h[i:i + b], r[i:i + b], t[i:i + b], i) for i in range(0, s.m, b)]
    s.neg_h, s.neg_t = torch.zeros(b * k, **i32), torch.zeros(b * k, **i32)
    s.at = 0
    if s.op == "semiring":
        s.kind = KINDS[c["kind"]]
        s.grads = B.Grads(s.ctx)
        s.grads.rows.zero_()
        B.stx_sample_negatives(s.ctx, h, r, t, k, s.neg_seed, 0, s.m, 0, s.neg_h, s.neg_t)
        B.stx_build_incidence(s.ctx, h, r, t, s.neg_h, s.neg_t, k, s.inc)
        rows = s.inc.n_rows
        s.z, s.work = torch.empty(rows, c["dim"], **f32), torch.empty(3 * rows * c["dim"], **f32)
        s.gz = torch.rand(rows, c["dim"], generator=gen, device=DEV) - 0.5
        return s
    s.lr = c["lr"]
    s.scores, s.loss = torch.zeros(b * (1 + k), **f32), torch.zeros(1, **f32)
    s.grads = None
    if s.op == "calls":
        s.grads = B.Grads(s.ctx)
        for g in (s.grads.rows, s.grads.w_rows, s.grads.proj):
            if g is not None:
                g.zero_()                       # only the touched rows' part is written
    else:
        s.blocks = B.link_batches([B.make_batch(hb, rb, tb, k, s.neg_seed, 0, s.m, i, s.neg_h, s.neg_t)
                                   for hb, rb, tb, i in s.batches], cyclic=True)
    return s


# ---- one pass -------------------------------------------------------------------------------------------------

def _updated(s):
    p, inc = s.params, s.inc
    return {"tables": [x for x in (p.ent, p.rel, p.w, p.proj) if x is not None], "scores": s.scores, "loss": s.loss,
            "negatives": [s.neg_h, s.neg_t],
            "transpose": [inc.at_touched_cols, inc.at_seg_ptr, inc.at_row_idx, inc.at_sign, inc.at_seg_id, inc.n_touched],
            "incidence": [inc.a_rowptr, inc.a_colidx, inc.a_vals]}


def run(s):
    if s.op == "rank":
        B.stx_rank(s.ctx, s.params, s.h, s.r, s.t, B.STX_TAIL, s.score[0], s.less[0], s.equal[0], s.work)
        B.stx_rank(s.ctx, s.params, s.h, s.r, s.t, B.STX_HEAD, s.score[1], s.less[1], s.equal[1], s.work)
        return s.score, s.less, s.equal
    if s.op == "semiring":
        B.stx_spmm_semiring(s.ctx, s.inc, s.params, s.kind, s.z)
        B.stx_spmm_semiring_t(s.ctx, s.inc, s.params, s.kind, s.gz, s.work, s.grads)
        return s.z, s.grads.rows
    i = s.at
    s.at = (i + 1) % len(s.batches)
    if s.op == "train":
        B.stx_train_step(s.ctx, s.blocks[i], s.inc, s.params, None, s.lr, s.scores, s.loss)
        return _updated(s)
    h, r, t, offset = s.batches[i]
    B.stx_sample_negatives(s.ctx, h, r, t, s.n_neg, s.neg_seed, 0, s.m, offset, s.neg_h, s.neg_t)
    B.stx_build_incidence(s.ctx, h, r, t, s.neg_h, s.neg_t, s.n_neg, s.inc)
    B.stx_forward(s.ctx, s.inc, s.params, s.scores, s.loss)
    B.stx_backward(s.ctx, s.inc, s.params, s.grads)
    B.stx_sgd_step(s.ctx, s.params, s.inc, s.grads, s.lr)
    out = _updated(s)
    out["gradients"] = [g for g in (s.grads.rows, s.grads.w_rows, s.grads.proj) if g is not None]
    return out


# ---- what a pass cannot do without ------------------------------------------------------------------------------

def _distinct(n_items, s, draws):
    """Expected number of distinct items among that many draws."""
    if n_items <= 0 or draws <= 0:
        return 0.0
    if s == 0.0:
        return float(n_items * -np.expm1(-draws / n_items))
    p = np.arange(1, n_items + 1, dtype=np.float64) ** (-s)
    return float(-np.expm1(-draws * p / p.sum()).sum())


def work(case):
    """Every table row a pass needs read once, every row it changes written once, the index arrays and results the
    calls return written once; the arithmetic of the products, distances and sums."""
    c = case
    d, n = c["dim"], c["n_ent"]
    if c["op"] == "rank":
        nq, k = c["queries"], c["rel_dim"]
        per = {"l1": 2, "l2": 3, "l2_sq": 3, "torus_l1": 5, "torus_l2": 6}[c["dist"]] + (4 if c["model"] == "transh" else 0)
        rels = _distinct(c["n_rel"], c["zipf_rel"], nq)
        table = 4.0 * (n * d + rels * (k + (k * d if c["model"] == "transr" else d if c["model"] == "transh" else 0)))
        flops = 2.0 * nq * n * k * per + (2.0 * rels * n * d * k * 2 if c["model"] == "transr" else 0.0)
        return {"bytes": 2 * (table + nq * (12.0 + 12.0)), "flops": flops}
    b, neg = c["batch"], c["n_neg"]
    rows = b * (1 + neg)
    # entities: the graph's heads and tails, and the uniform ones that replace one of them in every negative
    ent = _distinct(n, c["zipf_ent"], 2 * b)
    ent = ent + (n - ent) * -math.expm1(-float(b * neg) / n)
    rel = _distinct(c["n_rel"], c["zipf_rel"], b)
    if c["op"] == "semiring":
        rowb = 4.0 * d
        return {"bytes": (ent + rel) * rowb * 3 + rows * (12.0 * 2 + rowb * 2) + 3 * rows * 4.0,
                "flops": rows * d * (6.0 + 15.0)}
    model = c["model"]
    k = c["rel_dim"]
    params = ent * d + rel * (k + (d if model == "transh" else k * d if model == "transr" else 0))
    calls = c["op"] == "calls"
    index = 12.0 * b + 8.0 * b * neg + rows * (4 + 24 + 3 * (4 + 1 + 4)) + (ent + rel) * 8 + rows * 4.0
    flops = rows * ({"transr": 6.0 * d * k}.get(model, 0.0) + d * {"transh": 30.0}.get(model, 14.0))
    return {"bytes": 4.0 * params * (3 if calls else 2) + index, "flops": flops}


def tolerance(case):
    op = case["op"]
    if op == "rank":
        # the order of every sum is part of the interface, so scores have fixed bits and the counts follow from them
        return "exact"
    if op == "semiring":
        return {"rel": 1e-5, "max": 1e-3}       # products have fixed bits; 32-bit sums over thousands of terms
    if case["model"] == "transr":
        return {"rel": 1e-2, "max": 0.5} if op == "calls" else {"rel": 1e-4, "max": 1e-2}   # gradients of bf16 operands; tables that move by lr of them
    # 32-bit sums.  The L1 kinds' subgradient jumps: where y is within rounding of a jump, an element may take the
    # other sign and move by 2 lr
    return {"rel": 1e-5, "max": 0.1 if case["dist"] in ("l1", "torus_l1") else 1e-3}
