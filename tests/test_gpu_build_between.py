"""A program may build its next batch's incidence between the forward and the backward pass of this one: the gradients are
those of the forward pass that was stored, bit for bit."""
import pytest
import torch

from paper_2502_16949_amd import binding as B
from paper_2502_16949_amd import workloads as W
from tests import gpu_util as G
from tests.util import oracle_batch

pytestmark = pytest.mark.gpu

# model, dist, dim, rel_dim, negatives.  TransR: the kernel that holds whole positives (few relations: lists above its 64
# entries, dL/dy stored as one sum per positive) and the separate ones (negatives that do not fit 64, wide rows)
CASES = [("transe", "l2", 64, 64, 2), ("toruse", "torus_l1", 128, 128, 1), ("transh", "l2", 128, 128, 3),
         ("transr", "l2", 128, 128, 1), ("transr", "l1", 64, 128, 3), ("transr", "l2", 64, 64, 2), ("transr", "l2", 192, 64, 1)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_another_incidence_is_built_between_forward_and_backward(case):
    model, dist, dim, k, n_neg = case
    b = 700
    wl = W.Workload("case", 7, model, dist, 500, 3, 2 * b, dim, k, b, n_neg, 1.0, 0.01, 1, 1.1, 1.1, model == "transr")
    h, r, t = W.make_graph(wl)
    flags = B.STX_FLAG_BF16_PROJ if model == "transr" else 0
    m = G.GpuModel(wl, W.make_tables(wl), flags=flags, max_batch=2 * b)
    other = B.Incidence(m.ctx)
    nxt = oracle_batch(wl, h, r, t, b, 2 * b)

    def grads(between):
        m.build(oracle_batch(wl, h, r, t, 0, b))
        m.forward()
        if between:
            inc, m.inc = m.inc, other
            m.build(nxt)
            m.inc = inc
        for g in (m.grads.rows, m.grads.w_rows, m.grads.proj):
            if g is not None:
                g.zero_()
        m.backward()
        return [g.clone() for g in (m.grads.rows, m.grads.w_rows, m.grads.proj) if g is not None]

    want, got = grads(False), grads(True)
    for a, c in zip(want, got):
        assert float(a.abs().max()) > 0 and torch.equal(a.view(torch.int32), c.view(torch.int32))
    m.forward()                                            # the other incidence's own pass follows as usual
    with pytest.raises(B.StxError) as e:
        B.stx_backward(m.ctx, other, m.params, m.grads)
    assert e.value.status == B.STX_ERR_STATE
