"""The filtered sweeps of stx_rank (one large call) against the plain sweep, which small calls take: the same queries
128 at a time must give the same true scores and the same counts, bit for bit.  The plain sweep itself is held against
the oracle in test_gpu_rank.py."""
import numpy as np
import pytest
import torch

from paper_2502_16949_amd import binding as B
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

FILTER_STEPS = 6e8       # queries (padded to 128) x entities x dim below which no call is filtered


def _rank(ctx, p, h, r, t, side, work=None):
    nq = len(h)
    ts = torch.empty(nq, dtype=torch.float32, device=G.DEV)
    less = torch.empty(nq, dtype=torch.int32, device=G.DEV)
    equal = torch.empty_like(less)
    B.stx_rank(ctx, p, h, r, t, side, ts, less, equal, work)
    return ts, less, equal


def _sweeps_filtered(ctx, *args):
    """The counts, and how many filtered sweeps the call made."""
    B.stx_profile_kernel(ctx, "k_rank_pairs", 256)
    got = _rank(ctx, *args)
    n = B.stx_profile_read(ctx)[1]
    B.stx_profile_kernel(ctx, None, 0)
    return got, n


def _ms(f):
    a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    torch.cuda.synchronize()
    a.record()
    f()
    b.record()
    torch.cuda.synchronize()
    return a.elapsed_time(b)


CASES = [
    # (sizes at which the rule that compares both sweeps' times takes the filter)
    # dist, n_ent, dim, nq: row widths at and around the pieces of 8 and 16 elements, ragged tiles and query blocks
    ("l1", 60_001, 16, 8_000), ("l1", 4_097, 128, 1_300), ("l1", 2_050, 260, 1_250), ("l1", 1_100, 1024, 700),
    ("torus_l1", 40_000, 36, 700), ("torus_l1", 3_000, 200, 1_290), ("torus_l1", 1_500, 1000, 513),
    ("l2", 60_001, 16, 4_000), ("l2", 30_000, 44, 600), ("l2", 4_129, 128, 1_300), ("l2", 9_000, 196, 385),
    ("l2_sq", 2_050, 260, 1_250), ("l2", 1_300, 700, 800), ("l2", 1_100, 1024, 700),
    ("l2", 500_000, 100, 33), ("l1", 200_000, 60, 5),     # few queries, several segments of candidates
    # L2 kinds above 256 floats: the counts of steps that are not above, ragged; several segments
    ("l2", 4_001, 388, 700), ("l2_sq", 2_050, 512, 1_250), ("l2", 2_050, 768, 900), ("l2", 40_001, 500, 200),
]


@pytest.mark.parametrize("odd_rows", [False, True])
@pytest.mark.parametrize("dist,n_ent,dim,nq", CASES)
def test_filtered_counts_equal_the_plain_sweep(dist, n_ent, dim, nq, odd_rows):
    assert -(-nq // 128) * 128.0 * n_ent * dim >= FILTER_STEPS
    n_rel = 5
    rng = np.random.default_rng(dim + n_ent)
    X = rng.uniform(-1, 1, (n_ent + n_rel, dim)).astype(np.float32)
    if odd_rows:                                          # rows the bounds cannot cover, and exact ties
        X[7] = 1e30
        X[8, dim // 2] = np.inf
        X[9, 0] = np.nan
        X[10] *= 1e-22
        X[11] = 0.0
        X[12] *= 300.0
        X[13:13 + n_ent // 8] = X[n_ent - n_ent // 8:n_ent]
    h = rng.integers(0, n_ent, nq).astype(np.int32)
    t = rng.integers(0, n_ent, nq).astype(np.int32)
    if odd_rows:
        h[:4], t[:4] = [7, 9, 10, 11], [8, 20, 10, 12]
    r = rng.integers(0, n_rel, nq).astype(np.int32)
    hd, rd, td = G.dev_i32(h), G.dev_i32(r), G.dev_i32(t)
    cfg = B.make_config("toruse" if dist.startswith("torus") else "transe", dist, n_ent, n_rel, dim, 8, 1)
    ctx, p = B.Context(cfg, G.DEV), B.Params(G.dev_f32(X))
    step = 128 if 128.0 * n_ent * dim < FILTER_STEPS else 0
    for side in (B.STX_TAIL, B.STX_HEAD):
        got, sweeps = _sweeps_filtered(ctx, p, hd, rd, td, side)
        assert sweeps > 0
        got = [x.cpu().numpy() for x in got]
        if step:
            assert _sweeps_filtered(ctx, p, hd[:step].clone(), rd[:step].clone(), td[:step].clone(), side)[1] == 0
            parts = [_rank(ctx, p, hd[i:i + step].clone(), rd[i:i + step].clone(), td[i:i + step].clone(), side)
                     for i in range(0, nq, step)]
            want = [torch.cat([x[k] for x in parts]).cpu().numpy() for k in range(3)]
        else:                                             # entities in ranges small enough for the plain sweep
            want = _by_ranges(cfg, X, h, r, t, side, n_ent, n_rel, dim, dist)
        for g, w in zip(got, want):
            assert np.array_equal(g, w, equal_nan=True)
    assert B.stx_check_indices(ctx) == 0


# Which kernel sweeps: bytes above 256 floats, fp16 up to there; launches: one per chunk of queries and segment of candidates.
@pytest.mark.parametrize("n_ent,dim,nq,segments", [(8_193, 256, 700, 1), (8_193, 260, 700, 1), (4_001, 388, 700, 1), (4_001, 512, 700, 1),
                                                   (4_001, 516, 700, 1), (4_001, 1024, 700, 1), (40_001, 500, 200, 2)])
def test_kernel_of_wide_rows(n_ent, dim, nq, segments):
    rng = np.random.default_rng(dim)
    ctx = B.Context(B.make_config("transe", "l2", n_ent, 3, dim, 8, 1), G.DEV)
    p = B.Params(G.dev_f32(rng.uniform(-1, 1, (n_ent + 3, dim))))
    h, r, t = (G.dev_i32(rng.integers(0, n, nq)) for n in (n_ent, 3, n_ent))
    seen = {}
    for kernel in ("k_rank_wide", "k_rank_mfma"):
        B.stx_profile_kernel(ctx, kernel, 64)
        _rank(ctx, p, h, r, t, B.STX_TAIL)
        seen[kernel] = B.stx_profile_read(ctx)[1]
    B.stx_profile_kernel(ctx, None, 0)
    wide, other = ("k_rank_wide", "k_rank_mfma") if dim > 256 else ("k_rank_mfma", "k_rank_wide")
    assert seen[wide] >= segments and (segments > 1) == (seen[wide] > 1) and seen[other] == 0, seen


# Zero query points against whole tiles (32 candidates) of zero rows: every sum is exactly zero and so is every rounding.
@pytest.mark.parametrize("dist", ["l2", "l2_sq"])
@pytest.mark.parametrize("n_ent,dim,n_zero", [(4_129, 128, 1_000), (2_050, 260, 33), (4_129, 128, 4_129)])
def test_zero_queries_tie_with_zero_rows(n_ent, dim, n_zero, dist):
    nq, n_rel = 1_300, 3
    assert -(-nq // 128) * 128.0 * n_ent * dim >= FILTER_STEPS
    rng = np.random.default_rng(n_zero)
    X = rng.uniform(-1, 1, (n_ent + n_rel, dim)).astype(np.float32)
    X[:n_zero] = 0.0
    X[n_ent:] = 0.0                                       # (the relations)
    h, t = (rng.integers(0, n_zero, nq).astype(np.int32) for _ in range(2))
    r = rng.integers(0, n_rel, nq).astype(np.int32)
    ctx = B.Context(B.make_config("transe", dist, n_ent, n_rel, dim, 8, 1), G.DEV)
    p = B.Params(G.dev_f32(X))
    for side in (B.STX_TAIL, B.STX_HEAD):
        ts, less, equal = (x.cpu().numpy() for x in _rank(ctx, p, G.dev_i32(h), G.dev_i32(r), G.dev_i32(t), side))
        assert not ts.any() and not less.any() and np.all(equal == n_zero)


@pytest.mark.parametrize("dist", ["l2", "l2_sq"])
def test_transr_zero_projections_tie(dist):
    # relation 0: a zero matrix, all candidates tie; relation 1: the rows of 70 zero entities do; relation 2: no zero
    n_ent, dim, k, n_zero, nq = 1_000, 64, 32, 70, 300
    rng = np.random.default_rng(4)
    E = rng.uniform(-1, 1, (n_ent, dim)).astype(np.float32)
    E[:n_zero] = 0.0
    M = rng.uniform(-1, 1, (3, k, dim)).astype(np.float32)
    M[0] = 0.0
    R = np.zeros((3, k), np.float32)
    R[2] = 1.0
    h, t = (rng.integers(0, n_zero, nq).astype(np.int32) for _ in range(2))
    r = (np.arange(nq) % 3).astype(np.int32)
    ctx = B.Context(B.make_config("transr", dist, n_ent, 3, dim, 8, 1, rel_dim=k, flags=B.STX_FLAG_BF16_PROJ), G.DEV)
    p = B.Params(G.dev_f32(E), G.dev_f32(R), proj=G.dev_f32(M))
    work = torch.empty(B.stx_rank_work_bytes(ctx, nq) + 256, dtype=torch.uint8, device=G.DEV)
    for side in (B.STX_TAIL, B.STX_HEAD):
        ts, less, equal = (x.cpu().numpy() for x in _rank(ctx, p, G.dev_i32(h), G.dev_i32(r), G.dev_i32(t), side, work))
        for rel, tied in ((0, n_ent), (1, n_zero)):
            assert not ts[r == rel].any() and not less[r == rel].any() and np.all(equal[r == rel] == tied)
        # zero rows all score |r|^2 = k (or its root)
        assert np.all(equal[r == 2] == n_zero)
        assert np.allclose(ts[r == 2], k if dist == "l2_sq" else np.sqrt(k), rtol=1e-6)


# Sums in the subnormal range: there a step is off by up to half of 2^-149 whatever the sum.  Odd multiples of 2^-75 have
# squares halfway between two subnormal numbers, which round to the even sum, so that rows of the same values in other orders
# (of those and of any others, which make odd sums) have other sums.  A zero query point: the sums of the squares.
@pytest.mark.parametrize("dist", ["l2", "l2_sq"])
@pytest.mark.parametrize("largest", [3, 12, 60])
def test_order_of_subnormal_sums(dist, largest):
    n_ent, dim, nq, n_tiny = 4_129, 128, 1_300, 64
    rng = np.random.default_rng(11)
    X = rng.uniform(-1, 1, (n_ent + 1, dim)).astype(np.float32)
    X[n_ent] = 0.0
    row = np.concatenate([rng.integers(0, largest, dim // 2), rng.uniform(0, largest, dim // 2)]).astype(np.float32) * np.float32(2.0**-75)
    X[:n_tiny] = [rng.permutation(row) for _ in range(n_tiny)]
    X[100] = 0.0
    h, t = (rng.integers(200, n_ent, nq).astype(np.int32) for _ in range(2))
    h[:n_tiny], t[:n_tiny] = 100, np.arange(n_tiny)
    hd, rd, td = G.dev_i32(h), G.dev_i32(np.zeros(nq)), G.dev_i32(t)
    ctx = B.Context(B.make_config("transe", dist, n_ent, 1, dim, 8, 1), G.DEV)
    p = B.Params(G.dev_f32(X))
    got = _rank(ctx, p, hd, rd, td, B.STX_TAIL)
    parts = [_rank(ctx, p, hd[i:i + 128].clone(), rd[i:i + 128].clone(), td[i:i + 128].clone(), B.STX_TAIL)
             for i in range(0, nq, 128)]
    for g, w in zip(got, zip(*parts)):
        assert torch.equal(g, torch.cat(w))
    assert (got[1][:n_tiny] > 1).any()                    # (their order is decided by those roundings)


# More undecided pairs than the list of a sweep holds: the plain sweep does the chunk.  In the first chunk of queries or in
# a later one, over one segment of candidates or several, with the queries before and after it decided as usual.
@pytest.mark.parametrize("dist,n_ent,dim,nq,equal", [
    ("l1", 15_000, 128, 59_071, 15_000), ("l1", 4_097, 128, 9_000, 3_000), ("torus_l1", 40_000, 36, 700, 40_000),
    ("l2", 4_129, 128, 9_000, 4_000), ("l2_sq", 2_050, 260, 5_250, 2_050), ("l2", 60_001, 16, 4_000, 50_000),
    ("l2", 500_000, 100, 33, 400_000)])
def test_tables_of_equal_rows(dist, n_ent, dim, nq, equal):
    n_rel = 5
    rng = np.random.default_rng(equal)
    X = rng.uniform(0, 1, (n_ent + n_rel, dim)).astype(np.float32)
    X[:equal] = X[n_ent - 1]
    X[n_ent:] = X[n_ent]
    h, t = (rng.integers(0, n_ent, nq).astype(np.int32) for _ in range(2))
    if nq > 4_000 and equal < n_ent:                      # the first queries decide against the equal rows
        h[:2_000] = rng.integers(equal, n_ent - 1, 2_000)
        t[:2_000] = rng.integers(equal, n_ent - 1, 2_000)
    r = rng.integers(0, n_rel, nq).astype(np.int32)
    cfg = B.make_config("toruse" if dist.startswith("torus") else "transe", dist, n_ent, n_rel, dim, 8, 1)
    ctx, p = B.Context(cfg, G.DEV), B.Params(G.dev_f32(X))
    hd, rd, td = G.dev_i32(h), G.dev_i32(r), G.dev_i32(t)
    assert _sweeps_filtered(ctx, p, hd, rd, td, B.STX_TAIL)[1] > 0
    parts = [(hd[i:i + 128].clone(), rd[i:i + 128].clone(), td[i:i + 128].clone()) for i in range(0, nq, 128)]
    for side in (B.STX_TAIL, B.STX_HEAD):
        got = _rank(ctx, p, hd, rd, td, side)
        if 128.0 * n_ent * dim < FILTER_STEPS:
            want = [torch.cat(x) for x in zip(*(_rank(ctx, p, *q, side) for q in parts))]
        else:
            want = [torch.from_numpy(x).to(G.DEV) for x in _by_ranges(cfg, X, h, r, t, side, n_ent, n_rel, dim, dist)]
        for g, w in zip(got, want):
            assert torch.equal(g, w)
    if nq < 4_000 or 128.0 * n_ent * dim >= FILTER_STEPS:
        return
    # and at the plain sweep's pace (pair by pair, such a table took tens of times as long)
    one = min(_ms(lambda: _rank(ctx, p, hd, rd, td, B.STX_TAIL)) for _ in range(3))
    many = min(_ms(lambda: [_rank(ctx, p, *q, B.STX_TAIL) for q in parts]) for _ in range(3))
    assert one < 2 * many, (one, many)


# One row far outside the others' range, among the queries' rows or not, is left undecided by itself: the bounds and the
# steps of the other rows stay as they are (they did not: 2 to 60 times the time).
@pytest.mark.parametrize("dist,n_ent,dim,nq", [("l1", 15_000, 128, 59_071), ("torus_l1", 400_000, 128, 256)])
def test_one_row_far_out(dist, n_ent, dim, nq):
    n_rel = 5
    rng = np.random.default_rng(1)
    X = rng.uniform(0, 1, (n_ent + n_rel, dim)).astype(np.float32)
    h, t = (rng.integers(0, n_ent, nq).astype(np.int32) for _ in range(2))
    r = rng.integers(0, n_rel, nq).astype(np.int32)
    free = np.setdiff1d(np.arange(n_ent), np.concatenate([h, t]))
    hd, rd, td = G.dev_i32(h), G.dev_i32(r), G.dev_i32(t)
    cfg = B.make_config("toruse" if dist.startswith("torus") else "transe", dist, n_ent, n_rel, dim, 8, 1)
    ctx, ms = B.Context(cfg, G.DEV), []
    for row, value in ((0, None), (int(free[0]) if len(free) else 777, 1e13), (int(h[0]), 1e13), (int(h[0]), 3e4)):
        Y = X.copy()
        if value:
            Y[row] = value
        p = B.Params(G.dev_f32(Y))
        got = _rank(ctx, p, hd, rd, td, B.STX_TAIL)
        pick = np.unique(np.concatenate([np.arange(3), rng.integers(0, nq, 30)]))   # too few for the filter at these sizes
        want = [_rank(ctx, p, hd[i:i + 1].clone(), rd[i:i + 1].clone(), td[i:i + 1].clone(), B.STX_TAIL)
                for i in pick] if 128.0 * n_ent * dim < FILTER_STEPS else []
        for i, w in zip(pick, want):
            assert all(torch.equal(a[i:i + 1], b) for a, b in zip(got, w))
        ms.append(min(_ms(lambda: _rank(ctx, p, hd, rd, td, B.STX_TAIL)) for _ in range(5)))
    assert max(ms[1:]) < 1.5 * ms[0], ms


def test_transr_relations_of_equal_rows():
    # relations 1, 4, 7, ... map all entities to one point; they share launches with others that do not
    n_ent, dim, k, n_rel, nq = 6_000, 64, 32, 40, 30_000
    rng = np.random.default_rng(6)
    M = rng.uniform(-1, 1, (n_rel, k, dim)).astype(np.float32)
    M[1::3] = 0.0
    R = rng.uniform(-1, 1, (n_rel, k)).astype(np.float32)
    p = B.Params(G.dev_f32(rng.uniform(-1, 1, (n_ent, dim))), G.dev_f32(R), proj=G.dev_f32(M))
    h, t = (rng.integers(0, n_ent, nq).astype(np.int32) for _ in range(2))
    r = np.where(rng.random(nq) < 0.3, 1, rng.integers(0, n_rel, nq)).astype(np.int32)   # relation 1 has a launch of its own
    ctx = B.Context(B.make_config("transr", "l2", n_ent, n_rel, dim, 8, 1, rel_dim=k, flags=B.STX_FLAG_BF16_PROJ), G.DEV)
    work = torch.empty(B.stx_rank_work_bytes(ctx, nq) + 256, dtype=torch.uint8, device=G.DEV)
    hd, rd, td = G.dev_i32(h), G.dev_i32(r), G.dev_i32(t)
    for side in (B.STX_TAIL, B.STX_HEAD):
        ts, less, equal = (x.cpu().numpy() for x in _rank(ctx, p, hd, rd, td, side, work))
        flat = r % 3 == 1
        assert not less[flat].any() and np.all(equal[flat] == n_ent)
        for rel in (0, 2, 39):                            # the others as they come out in calls of their own
            i = np.nonzero(r == rel)[0]
            one = [x.cpu().numpy() for x in _rank(ctx, p, hd[i].clone(), rd[i].clone(), td[i].clone(), side, work)]
            for a, b in zip((ts[i], less[i], equal[i]), one):
                assert np.array_equal(a, b)
            assert equal[i].max() <= 3


# The scratch of the filtered sweeps is optional: without it the sweeps are plain, with the same results.
def test_without_scratch_of_the_filter(monkeypatch):
    n_ent, dim, nq, n_rel = 4_129, 128, 1_300, 3
    rng = np.random.default_rng(3)
    p = B.Params(G.dev_f32(rng.uniform(-1, 1, (n_ent + n_rel, dim))))
    h, r, t = (G.dev_i32(rng.integers(0, n, nq)) for n in (n_ent, n_rel, n_ent))
    cfg = B.make_config("transe", "l2", n_ent, n_rel, dim, 8, 1)
    core = B.stx_workspace_bytes(B.make_config("transe", "torus_l2", n_ent, n_rel, dim, 8, 1))
    assert core < B.stx_workspace_bytes(cfg)
    full = B.Context(cfg, G.DEV)
    monkeypatch.setattr(B, "stx_workspace_bytes", lambda c: core)
    small = B.Context(cfg, G.DEV)
    (one, n_one), (two, n_two) = (_sweeps_filtered(c, p, h, r, t, B.STX_HEAD) for c in (full, small))
    assert n_one > 0 and n_two == 0 and all(torch.equal(a, b) for a, b in zip(one, two))
    monkeypatch.setattr(B, "stx_workspace_bytes", lambda c: core - 256)
    with pytest.raises(B.StxError) as e:
        B.Context(cfg, G.DEV)
    assert e.value.status == B.STX_ERR_WORKSPACE


def test_transr_without_scratch_of_the_filter():
    n_ent, dim, k, nq, n_rel = 1_000, 64, 32, 3_000, 5
    rng = np.random.default_rng(3)
    p = B.Params(G.dev_f32(rng.uniform(-1, 1, (n_ent, dim))), G.dev_f32(rng.uniform(-1, 1, (n_rel, k))),
                 proj=G.dev_f32(rng.uniform(-1, 1, (n_rel, k, dim))))
    h, r, t = (G.dev_i32(rng.integers(0, n, nq)) for n in (n_ent, n_rel, n_ent))
    ctx = {d: B.Context(B.make_config("transr", d, n_ent, n_rel, dim, 8, 1, rel_dim=k, flags=B.STX_FLAG_BF16_PROJ), G.DEV)
           for d in ("l1", "l2")}
    plain, full = (B.stx_rank_work_bytes(ctx[d], nq) for d in ("l1", "l2"))
    assert plain < full
    work = torch.empty(full + 512, dtype=torch.uint8, device=G.DEV)
    work = work[-work.data_ptr() % 256:]
    want = _rank(ctx["l2"], p, h, r, t, B.STX_TAIL, work[:full])
    for size in (full - 256, plain):
        got, n = _sweeps_filtered(ctx["l2"], p, h, r, t, B.STX_TAIL, work[:size])
        assert n == 0 and all(torch.equal(a, b) for a, b in zip(got, want))
    with pytest.raises(B.StxError) as e:
        _rank(ctx["l2"], p, h, r, t, B.STX_TAIL, work[:plain - 256])
    assert e.value.status == B.STX_ERR_WORKSPACE


# More undecided pairs in one sweep than an int32 counts (every candidate ties): a chunk of fixed-point queries is
# never smaller than 32, and a TransR relation is swept in one piece.
def test_more_undecided_pairs_than_an_int32_counts():
    n_ent, dim, nq = 68_000_000, 4, 32
    assert nq * n_ent > 2**31
    p = B.Params(torch.full((n_ent + 1, dim), 0.25, device=G.DEV))
    ctx = B.Context(B.make_config("transe", "l1", n_ent, 1, dim, 8, 1), G.DEV)
    q = torch.arange(nq, dtype=torch.int32, device=G.DEV)
    _, less, equal = _rank(ctx, p, q, torch.zeros_like(q), q + 7, B.STX_TAIL)
    assert not less.any() and bool((equal == n_ent).all())


def test_more_undecided_pairs_than_an_int32_counts_transr():
    n_ent, dim, nq = 125_000, 32, 17_500
    assert nq * n_ent > 2**31
    E = torch.rand(n_ent, dim, device=G.DEV)
    p = B.Params(E, torch.zeros(1, dim, device=G.DEV), proj=torch.zeros(1, dim, dim, device=G.DEV))
    ctx = B.Context(B.make_config("transr", "l2", n_ent, 1, dim, 8, 1, rel_dim=dim, flags=B.STX_FLAG_BF16_PROJ), G.DEV)
    work = torch.empty(B.stx_rank_work_bytes(ctx, nq) + 256, dtype=torch.uint8, device=G.DEV)
    q = torch.arange(nq, dtype=torch.int32, device=G.DEV)
    _, less, equal = _rank(ctx, p, q, torch.zeros_like(q), q + 7, B.STX_TAIL, work)
    assert not less.any() and bool((equal == n_ent).all())


def _by_ranges(cfg, X, h, r, t, side, n_ent, n_rel, dim, dist):
    """The counts of long tables from plain sweeps over tables of a part of the entities each, to which the entities
    of the queries are added (and subtracted again)."""
    nq, size = len(h), int(FILTER_STEPS / 128 / dim / 2)
    own = np.concatenate([h, t])
    less, equal, ts = np.zeros(nq, np.int64), np.zeros(nq, np.int64), None

    def run(rows):
        n = len(rows)
        ctx = B.Context(B.make_config(cfg.model, cfg.dist, n, n_rel, dim, 8, 1), G.DEV)
        p = B.Params(G.dev_f32(np.concatenate([X[rows], X[n_ent:]])))
        q = np.arange(nq, dtype=np.int32)
        return [x.cpu().numpy() for x in _rank(ctx, p, G.dev_i32(q), G.dev_i32(r), G.dev_i32(q + nq), side)]

    ts, less0, equal0 = run(own)
    for lo in range(0, n_ent, size):
        part = np.arange(lo, min(lo + size, n_ent))
        _, l, e = run(np.concatenate([own, part]))
        less += l - less0
        equal += e - equal0
    return ts, less.astype(np.int32), equal.astype(np.int32)
