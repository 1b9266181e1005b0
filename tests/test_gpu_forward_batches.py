"""The forward kernel that fetches a positive's rows once, at numbers of negatives around the batches it holds at a time
(four, two for rows of more than two float4 per lane), and the transposed product's stitching of runs that cross
chunks, at few columns; against the oracle at the bars of the step test."""
import numpy as np
import pytest
import torch

from oracle import stxo
from paper_2502_16949_amd import binding as B
from tests import gpu_util as G
from tests.test_gpu_stacked import _check_step, _problem

pytestmark = pytest.mark.gpu


# (Rows of 12 floats at least: table values reach 6 / sqrt(dim), and past 2 their last place, 2^-22, is more than the
# absolute term 2^-23 of the step test's bar.)
@pytest.mark.parametrize("k", [2, 3, 4, 5, 8, 9])
@pytest.mark.parametrize("model,dist,dim", [("transe", "l2", 12), ("toruse", "torus_l1", 60), ("transe", "l1", 200),
                                            ("transe", "l2", 260), ("toruse", "torus_l2", 516), ("transe", "l1", 1020)])
def test_batches_of_negatives(model, dist, dim, k):
    wl, tabs, bt = _problem(model, dist, 300, 7, 203, k, dim, seed=dim + k, zipf=1.1)
    _check_step(wl, tabs, bt, model, dim, B.STX_SUM)
    # the last negative of the last positive alone is of a kind that the kernel does not cover
    nh, nt = bt.nh.copy(), bt.nt.copy()
    nh[-1], nt[-1] = (bt.h[-1] + 1) % wl.n_ent, (bt.t[-1] + 1) % wl.n_ent
    _check_step(wl, tabs, stxo.Batch(bt.h, bt.r, bt.t, nh, nt), model, dim, B.STX_SUM)
    # every third positive has negatives of that kind only, so that both ways of fetching meet in a wavefront
    own = np.repeat(np.arange(len(bt.h)) % 3 == 0, k)
    nh, nt = np.where(own, (bt.nh + 1) % wl.n_ent, bt.nh), np.where(own, (bt.nt + 1) % wl.n_ent, bt.nt)
    _check_step(wl, tabs, stxo.Batch(bt.h, bt.r, bt.t, nh.astype(np.int32), nt.astype(np.int32)), model, dim, B.STX_SUM)


# A caller's own negatives need three rows each where the sampler's need one (out of the caches here): 1.15 times the
# time measured, 2.15 when every such batch went through two kernels.
def test_own_negatives_cost_one_pass():
    n_ent, n_rel, dim, b, k = 15_000, 1_350, 128, 16_384, 5
    rng = np.random.default_rng(5)
    ctx = B.Context(B.make_config("transe", "l2", n_ent, n_rel, dim, b, k), G.DEV)
    inc, p = B.Incidence(ctx), B.Params(G.dev_f32(rng.uniform(-0.5, 0.5, (n_ent + n_rel, dim))))
    ids = lambda n, m: G.dev_i32(rng.integers(0, n, m))
    h, r, t, nh, nt = ids(n_ent, b), ids(n_rel, b), ids(n_ent, b), ids(n_ent, b * k), ids(n_ent, b * k)
    scores, loss = torch.zeros(b * (1 + k), device=G.DEV), torch.zeros(1, device=G.DEV)
    ms = []
    for own in (True, False):
        if not own:
            B.stx_sample_negatives(ctx, h, r, t, k, 7, 0, b, 0, nh, nt)
        B.stx_build_incidence(ctx, h, r, t, nh, nt, k, inc)
        best = 1e9
        for _ in range(5):
            e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            e0.record()
            for _ in range(50):
                B.stx_forward(ctx, inc, p, scores, loss)
            e1.record()
            torch.cuda.synchronize()
            best = min(best, e0.elapsed_time(e1))
        ms.append(best)
    assert ms[0] < 1.6 * ms[1], ms


# rows of 8, 16, 32 and 64 lanes; two entities: runs over many chunks and tiles; more: runs that end at
# any place
@pytest.mark.parametrize("dim", [32, 64, 128, 256])
@pytest.mark.parametrize("n_ent,n_rel,b", [(2, 1, 700), (3, 2, 411), (40, 3, 1_025)])
def test_runs_across_chunks(n_ent, n_rel, b, dim):
    wl, tabs, bt = _problem("transe", "l2", n_ent, n_rel, b, 1, dim, seed=dim + b)
    rng = np.random.default_rng(b)
    h, t = (rng.integers(0, n_ent, b).astype(np.int32) for _ in range(2))
    bt = stxo.Batch(h, bt.r, t, np.roll(h, 1), t)
    _check_step(wl, tabs, bt, "transe", dim, B.STX_SUM)
