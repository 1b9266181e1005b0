"""Batches whose rows of dL/dx stx_train_step forms where they are summed (from 192 MiB of them on, 384 below 256 floats a
row; few columns), with the same bits as the separate calls, which store them."""
import numpy as np
import pytest
import torch

from paper_2502_16949_amd import binding as B
from paper_2502_16949_amd import workloads as W
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

FORMED_BYTES = {True: 192 << 20, False: 384 << 20}       # dim >= 256
CASES = [
    # model, dist, n_ent, n_rel, b, k, dim: rows of 16 slices of 16 float4, a ragged last slice, an odd last tile
    ("transe", "l2", 3000, 7, 24_667, 1, 1024),
    ("transe", "l2_sq", 900, 5, 10_001, 5, 852),
    ("toruse", "torus_l2", 20_000, 300, 130_001, 3, 200),
    ("transe", "l2", 3000, 7, 401_000, 1, 128),
    ("transe", "l2", 5_000, 11, 49_000, 1, 516),          # one float4 in the last slice
]


def _setup(model, dist, n_ent, n_rel, b, k, dim):
    assert b * (1 + k) * dim * 4 >= FORMED_BYTES[dim >= 256] and dim >= 128
    wl = W.Workload("formed", 21, model, dist, n_ent, n_rel, b, dim, dim, b, k, 1.0, 0.01, 1, 1.1, 1.1)
    tabs = W.make_tables(wl)
    tabs["rel_weight"] = np.linspace(0.5, 1.5, n_rel).astype(np.float32)
    rng = np.random.default_rng(8)
    hd, td = (G.dev_i32(rng.integers(0, n_ent, b) ** 2 // n_ent) for _ in range(2))
    rd = G.dev_i32(rng.integers(0, n_rel, b))
    neg = [torch.zeros(b * k, dtype=torch.int32, device=G.DEV) for _ in range(2)]
    return wl, tabs, hd, rd, td, neg


def _forward(m, hd, rd, td, k, neg):
    b = len(hd)
    B.stx_sample_negatives(m.ctx, hd, rd, td, k, 5, 0, b, 0, neg[0], neg[1])
    B.stx_build_incidence(m.ctx, hd, rd, td, neg[0], neg[1], k, m.inc)
    m.forward()


@pytest.mark.parametrize("odd_rows", [False, True])
@pytest.mark.parametrize("model,dist,n_ent,n_rel,b,k,dim", CASES)
def test_step_of_formed_rows_equals_the_separate_calls(model, dist, n_ent, n_rel, b, k, dim, odd_rows):
    wl, tabs, hd, rd, td, neg = _setup(model, dist, n_ent, n_rel, b, k, dim)
    if odd_rows:                                          # products that are NaN also where the pair is inactive
        tabs["ent"][n_ent // 2, 3] = np.inf
        tabs["ent"][n_ent // 3, dim - 1] = np.nan
    # l2_sq gradients grow with y: a small rate keeps the second step finite
    lr = 1e-5 if dist == "l2_sq" else 0.01
    ma, mb, mc = (G.GpuModel(wl, tabs) for _ in range(3))
    for step in range(2):
        _forward(ma, hd, rd, td, k, neg)
        ma.backward()
        ma.sgd(lr)
        _forward(mc, hd, rd, td, k, neg)
        mc.backward_sgd(lr)
        batch = B.make_batch(hd, rd, td, k, 5, 0, b, 0, neg[0], neg[1])
        B.stx_train_step(mb.ctx, batch, mb.inc, mb.params, None, lr, mb.scores, mb.loss)
        want = ma.params.ent.view(torch.int32)
        if odd_rows:                                      # (a NaN's bits are nobody's promise)
            assert torch.isnan(ma.params.ent).any()
            want = torch.nan_to_num(ma.params.ent, nan=7.0)
        for m in (mb, mc):
            got = torch.nan_to_num(m.params.ent, nan=7.0) if odd_rows else m.params.ent.view(torch.int32)
            assert torch.equal(got, want), step
        assert torch.equal(ma.scores.view(torch.int32), mb.scores.view(torch.int32))


def test_gradients_are_those_of_the_tables_the_forward_pass_saw():
    wl, tabs, hd, rd, td, neg = _setup(*CASES[0])
    m = G.GpuModel(wl, tabs)
    _forward(m, hd, rd, td, 1, neg)
    m.backward()
    cols, want = m.grad_rows_numpy()
    _forward(m, hd, rd, td, 1, neg)
    m.params.ent.mul_(1.5)
    m.grads.rows.zero_()
    m.backward()
    assert np.array_equal(m.grad_rows_numpy()[1], want)


@pytest.mark.parametrize("mean", [False, True])
@pytest.mark.parametrize("model,dist,n_ent,n_rel,b,k,dim", CASES)
def test_sliced_forward_pass_against_64_bits(model, dist, n_ent, n_rel, b, k, dim, mean):
    wl, tabs, hd, rd, td, neg = _setup(model, dist, n_ent, n_rel, b, k, dim)
    reduce = B.STX_MEAN if mean else B.STX_SUM
    ma, mb = (G.GpuModel(wl, tabs, reduce=reduce) for _ in range(2))
    _forward(ma, hd, rd, td, k, neg)
    ma.backward_sgd(1e-5)
    x = mb.params.ent.clone()
    batch = B.make_batch(hd, rd, td, k, 5, 0, b, 0, neg[0], neg[1])
    B.stx_train_step(mb.ctx, batch, mb.inc, mb.params, None, 1e-5, mb.scores, mb.loss)
    assert torch.equal(ma.loss, mb.loss) and torch.equal(ma.params.ent, mb.params.ent)
    rows = mb.inc.n_rows
    scores = mb.scores[:rows].double()
    want = torch.empty_like(scores)
    weight = mb.params.rel_weight.double()
    for c in torch.arange(rows, device=G.DEV).split(1 << 16):
        col = mb.inc.a_colidx[:3 * rows].view(rows, 3)[c].long()
        y = (x[col[:, 0]] + x[col[:, 1]]) - x[col[:, 2]]  # (rounded as the library rounds it, and so is the torus' fraction)
        if model == "toruse":
            f = y - torch.floor(y)
            y = torch.minimum(f, 1.0 - f)
        s = y.double().square().sum(1)
        want[c] = weight[col[:, 1] - n_ent] * (s if dist == "l2_sq" else s.sqrt())
    # 32-bit sums of non-negative terms: at most dim roundings of 2^-24 each, and those of the term, the root and the weight
    assert torch.all((scores - want).abs() <= (dim + 4) * 2.0 ** -24 * want)
    pos, n = scores[:b].float().repeat_interleave(k), scores[b:].float()
    hinge = ((wl.margin + pos) - n).clamp(min=0.0).double().sum() / (b * k if mean else 1)
    assert hinge > 0 and abs(mb.loss.double().item() - hinge.item()) <= 1e-6 * hinge.item()
