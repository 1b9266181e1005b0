"""TransR's L2 kinds swept over the entity table itself against plain sweeps over projected tables (which a call gets that
leaves the filter's scratch out): the same scores and counts, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2502_16949_amd import binding as B
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

CASES = [
    # dist, n_ent, n_rel, dim, rel_dim, nq: every compiled number of steps, one and two halves of the outputs, ragged tiles of
    # entities, blocks of one query and of 32, several sweeps (the last)
    ("l2", 1_999, 300, 32, 32, 900),
    ("l2_sq", 3_001, 200, 64, 96, 700),
    ("l2", 2_113, 150, 96, 256, 301),
    ("l2", 4_097, 120, 128, 128, 1_500),
    ("l2_sq", 2_500, 90, 160, 64, 333),
    ("l2", 1_025, 220, 224, 160, 400),
    ("l2", 2_049, 60, 256, 256, 97),
    ("l2", 60_001, 90, 64, 32, 350),
]


def _run(ctx, p, ids, side, work, kernel="k_rr_sweep"):
    nq = len(ids[0])
    ts = torch.empty(nq, dtype=torch.float32, device=G.DEV)
    less, equal = (torch.empty(nq, dtype=torch.int32, device=G.DEV) for _ in range(2))
    B.stx_profile_kernel(ctx, kernel, 256)
    B.stx_rank(ctx, p, *ids, side, ts, less, equal, work)
    n = B.stx_profile_read(ctx)[1]
    B.stx_profile_kernel(ctx, None, 0)
    return (ts, less, equal), n


def _compare(dist, n_ent, n_rel, dim, k, nq, E, R, M, ids, sides=(B.STX_TAIL, B.STX_HEAD), launches=()):
    """launches: (kernel, least number of them) of the call with all its scratch."""
    ctx = {d: B.Context(B.make_config("transr", d, n_ent, n_rel, dim, 8, 1, rel_dim=k, flags=B.STX_FLAG_BF16_PROJ), G.DEV)
           for d in ("l1", dist)}
    p = B.Params(G.dev_f32(E), G.dev_f32(R), proj=G.dev_f32(M))
    plain, full = (B.stx_rank_work_bytes(ctx[d], nq) for d in ("l1", dist))
    work = torch.empty(full + 256, dtype=torch.uint8, device=G.DEV)
    work = work[-work.data_ptr() % 256:]
    for side in sides:
        want, none = _run(ctx[dist], p, ids, side, work[:plain])
        work.random_(0, 255)                               # nothing is expected of the scratch
        got, n = _run(ctx[dist], p, ids, side, work[:full])
        assert none == 0 and n > 0
        for a, b, what in zip(got, want, ("score", "less", "equal")):
            assert torch.equal(a.view(torch.int32), b.view(torch.int32)), (what, side)
        for kernel, least in launches:
            again, n = _run(ctx[dist], p, ids, side, work[:full], kernel)
            assert n >= least, (kernel, n)
            assert all(torch.equal(a.view(torch.int32), b.view(torch.int32)) for a, b in zip(again, want)), (kernel, side)


def _inputs(seed, n_ent, n_rel, dim, k, nq):
    rng = np.random.default_rng(seed)
    E = rng.uniform(-1, 1, (n_ent, dim)).astype(np.float32)
    R = rng.uniform(-1, 1, (n_rel, k)).astype(np.float32)
    M = (rng.standard_normal((n_rel, k, dim)) / np.sqrt(dim)).astype(np.float32)
    ids = [G.dev_i32(x) for x in (rng.integers(0, n_ent, nq), rng.integers(0, n_rel, nq) ** 2 // n_rel, rng.integers(0, n_ent, nq))]
    return E, R, M, ids


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_counts_equal_the_plain_sweep(case):
    dist, n_ent, n_rel, dim, k, nq = case
    _compare(*case, *_inputs(dim + k, n_ent, n_rel, dim, k, nq))


# Values that no bound covers (infinities, NaN, rows and matrices far out or close to zero) are decided one by one; ties by
# the bits of the sums.
def test_odd_values():
    dist, n_ent, n_rel, dim, k, nq = case = CASES[3]
    E, R, M, ids = _inputs(3, n_ent, n_rel, dim, k, nq)
    E[100, 5], E[200, 7], E[300], E[400] = np.inf, np.nan, 1e9, 0.0
    E[401:420] = E[500]                                    # ties of whole rows
    E[1000:1032] *= 1e-9                                   # a tile near zero
    M[3], M[5, 2, 2], M[7], M[9] = 0.0, np.inf, 1e8, 1e-12
    M[11, 40, 3] = np.nan
    R[4] = 1e6
    h, r, t = (x.cpu().numpy() for x in ids)
    r[:40], t[40:60], h[60:64], h[64], h[65] = np.repeat([3, 5, 7, 9, 11], 8), 410, 100, 200, 300
    _compare(*case, E, R, M, [G.dev_i32(x) for x in (h, r, t)])


# More undecided pairs than their list has places: every entity scores alike for all relations but a few.
def test_more_undecided_pairs_than_places():
    dist, n_ent, n_rel, dim, k, nq = case = ("l2", 6_001, 400, 64, 64, 3_000)
    E, R, M, ids = _inputs(4, n_ent, n_rel, dim, k, nq)
    E[:] = E[0]
    E[1::1000] *= 1.5
    _compare(*case, E, R, M, ids)


def test_indices_out_of_range_are_counted():
    dist, n_ent, n_rel, dim, k, nq = CASES[0]
    E, R, M, ids = _inputs(5, n_ent, n_rel, dim, k, nq)
    ids[0][3], ids[1][4], ids[2][5] = -1, n_rel, n_ent + 7
    _compare(dist, n_ent, n_rel, dim, k, nq, E, R, M, ids)


# More relations than a batch of them holds operands for: 206 at these sizes, of 300 or so that occur.
def _batches_case():
    dist, n_ent, n_rel, dim, k, nq = case = ("l2", 60_001, 400, 64, 32, 1_000)
    E, R, M, ids = _inputs(6, n_ent, n_rel, dim, k, nq)
    r = np.random.default_rng(7).permutation(np.r_[np.arange(300), np.random.default_rng(8).integers(0, 300, nq - 300)])
    ids[1] = G.dev_i32(r + 50)
    return case, E, R, M, ids


def test_several_batches_of_relations():
    case, E, R, M, ids = _batches_case()
    _compare(*case, E, R, M, ids, launches=[("k_rr_pack", 2), ("k_rr_norms", 2)])


# ... the first of which leaves more pairs undecided than there are places: its matrices are zero.
def test_a_batch_of_relations_behind_one_that_stopped():
    case, E, R, M, ids = _batches_case()
    M[50:250], R[50:250] = 0.0, 0.0
    _compare(*case, E, R, M, ids, launches=[("k_rr_pack", 2)])


# One relation with more queries than pay without a table (7,410 at these sizes), and many that have few: both ways in one
# call, the second's scratch over the first's.
def test_both_ways_in_one_call():
    dist, n_ent, n_rel, dim, k, nq = case = ("l2", 2_049, 61, 256, 256, 10_500)
    E, R, M, ids = _inputs(9, n_ent, n_rel, dim, k, nq)
    rng = np.random.default_rng(10)
    r = rng.permutation(np.r_[np.full(9_000, 17), rng.choice([x for x in range(n_rel) if x != 17], nq - 9_000)])
    ids[1] = G.dev_i32(r)
    _compare(*case, E, R, M, ids, launches=[("k_rr_sweep", 1), ("k_rank_mfma", 1)])


# A buffer that holds the scratch of one way alone: that way runs.  (The first two relations' tables take less than the
# entities' operands, the others' tables more.)
@pytest.mark.parametrize("case,share,kernel", [(("l2", 60_000, 2, 256, 256, 300), 0.8, "k_rank_mfma"),
                                               (("l2_sq", 9_000, 200, 64, 64, 1_000), 0.8, "k_rr_sweep")])
def test_scratch_of_one_way(case, share, kernel):
    dist, n_ent, n_rel, dim, k, nq = case
    E, R, M, ids = _inputs(11, n_ent, n_rel, dim, k, nq)
    cfg = lambda d: B.make_config("transr", d, n_ent, n_rel, dim, 8, 1, rel_dim=k, flags=B.STX_FLAG_BF16_PROJ)
    ctx, p = B.Context(cfg(dist), G.DEV), B.Params(G.dev_f32(E), G.dev_f32(R), proj=G.dev_f32(M))
    plain, full = B.stx_rank_work_bytes(B.Context(cfg("l1"), G.DEV), nq), B.stx_rank_work_bytes(ctx, nq)
    some = plain + int(share * (full - plain)) // 256 * 256
    work = torch.empty(full + 256, dtype=torch.uint8, device=G.DEV)
    work = work[-work.data_ptr() % 256:]
    want, none = _run(ctx, p, ids, B.STX_TAIL, work[:plain], kernel)
    work.random_(0, 255)
    got, n = _run(ctx, p, ids, B.STX_TAIL, work[:some], kernel)
    assert none == 0 and n > 0
    assert all(torch.equal(a.view(torch.int32), b.view(torch.int32)) for a, b in zip(got, want))
    other = {"k_rank_mfma": "k_rr_sweep", "k_rr_sweep": "k_rank_mfma"}[kernel]
    assert _run(ctx, p, ids, B.STX_TAIL, work[:some], other)[1] == 0


# Calls that cannot gain by it keep no scratch for the sweep without tables.
def test_no_scratch_for_few_queries():
    cfg = lambda dist, n_rel: B.make_config("transr", dist, 9_951, n_rel, 64, 8, 1, rel_dim=64, flags=B.STX_FLAG_BF16_PROJ)
    more = {n_rel: B.stx_rank_work_bytes(B.Context(cfg("l2", n_rel), G.DEV), 3) - B.stx_rank_work_bytes(B.Context(cfg("l1", n_rel), G.DEV), 3)
            for n_rel in (32, 1_000)}
    assert more[32] == more[1_000]                         # (the tables' filter: 32 tables at most)
