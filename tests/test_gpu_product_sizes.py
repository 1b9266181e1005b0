"""The sort's 16-bit tile histograms and the two chunk lengths of the transposed product, at the sizes where they change."""
import numpy as np
import pytest
import torch

from paper_2502_16949_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _build(ctx, inc, h, r, t, nh, nt, k):
    dev = [torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).to(DEV) for a in (h, r, t, nh, nt)]
    B.stx_build_incidence(ctx, *dev, k, inc)
    torch.cuda.synchronize()


# 1,024 entries a tile: 1 tile, the tables that are added up in one go (448 tiles), in two (449, 512), two levels (beyond, 4,096 a
# tile), and a last tile of one entry
@pytest.mark.parametrize("entries", [3, 1024 * 3, 448 * 1024, 449 * 1024, 511 * 1024 + 1, 512 * 1024, 512 * 1024 + 3, 33 * 4096 * 8])
@pytest.mark.parametrize("skew", ["one column", "spread"])
def test_sorted_transpose_of_full_tiles(entries, skew):
    b, n_ent, n_rel = entries // 3, 70_000, 3
    rng = np.random.default_rng(entries)
    if skew == "one column":                                # every tile's keys fall on two digits, 65,536 of them in 64 tiles
        h, t, r = np.full(b, 65_000), np.full(b, 65_000), np.zeros(b)
        h[-1] = 5
    else:
        h, t, r = rng.integers(0, n_ent, b), rng.integers(0, n_ent, b), rng.integers(0, n_rel, b)
    ctx = B.Context(B.make_config("transe", "l2", n_ent, n_rel, 4, b, 1), DEV)
    inc = B.Incidence(ctx)
    _build(ctx, inc, h, r, t, np.zeros(0), np.zeros(0), 0)
    cols = np.stack([h, n_ent + r, t], 1).reshape(-1).astype(np.int64)
    order = np.argsort(cols, kind="stable")
    nnz = 3 * b
    assert np.array_equal(inc.at_row_idx[:nnz].cpu().numpy(), order // 3)
    assert np.array_equal(inc.at_sign[:nnz].cpu().numpy(), np.where(order % 3 == 2, -1, 1))
    u = int(inc.n_touched.item())
    want, start = np.unique(cols, return_index=False), np.flatnonzero(np.diff(cols[order], prepend=-1))
    assert u == len(want) and np.array_equal(inc.at_touched_cols[:u].cpu().numpy(), want)
    assert np.array_equal(inc.at_seg_ptr[:u + 1].cpu().numpy(), np.append(start, nnz))


# 3,600 tiles of the short chunks: 64 entries each at more than 128 floats a row, 128 at 65 to 128; both sides of the line, and of
# a million entries for the dense kinds
@pytest.mark.parametrize("dist,dim,rows", [("l1", 200, 3600 * 64 // 3), ("l1", 200, 3600 * 64 // 3 + 2), ("l1", 128, 3600 * 128 // 3),
                                           ("l1", 128, 3600 * 128 // 3 + 2), ("l1", 520, 3600 * 64 // 3 + 2), ("l1", 1024, 3600 * 64 // 3 + 2),
                                           ("l2", 200, (1 << 20) // 3 - 1), ("l2", 200, (1 << 20) // 3 + 1), ("l2", 128, (1 << 20) // 3 + 1)])
def test_product_on_both_sides_of_the_chunk_lines(dist, dim, rows):
    b, n_ent, n_rel = rows // 2, 30_000, 7
    gen = torch.Generator(device=DEV)
    gen.manual_seed(rows + dim)
    x = torch.rand(n_ent + n_rel, dim, generator=gen, device=DEV) - 0.5
    idx = [torch.randint(0, hi, (b,), generator=gen, device=DEV, dtype=torch.int32) for hi in (n_ent, n_rel, n_ent, n_ent)]
    idx[0][: b // 3] = 11                                   # one entity owns a sixth of its side's entries
    p = B.Params(x)
    ctx = B.Context(B.make_config("transe", dist, n_ent, n_rel, dim, b, 1, margin=1.0), DEV)
    inc, grads = B.Incidence(ctx), B.Grads(ctx)
    scores, loss = torch.zeros(2 * b, device=DEV), torch.zeros(1, device=DEV)
    B.stx_build_incidence(ctx, idx[0], idx[1], idx[2], idx[3], idx[2], 1, inc)
    B.stx_forward(ctx, inc, p, scores, loss)
    B.stx_backward(ctx, inc, p, grads)
    torch.cuda.synchronize()
    cols = inc.a_colidx[: 6 * b].view(2 * b, 3).long()
    y = x[cols[:, 0]] + x[cols[:, 1]]
    y = (y - x[cols[:, 2]]).double()                        # (the roundings of the library's x, whose signs the L1 kind takes)
    norm = y.norm(dim=1) if dist == "l2" else y.abs().sum(1)
    # scores are 32-bit sums of non-negative terms: at most dim roundings of 2^-24 each
    assert torch.all((scores.double() - norm).abs() <= (dim + 4) * 2.0 ** -24 * norm)
    active = ((1.0 + scores[:b]) - scores[b:] > 0).double()
    coef = torch.cat([active, -active])
    g = y * (coef / norm)[:, None] if dist == "l2" else torch.sign(y) * coef[:, None]
    u = int(inc.n_touched.item())
    touched = inc.at_touched_cols[:u].long()
    want = torch.zeros(n_ent + n_rel, dim, dtype=torch.float64, device=DEV)
    size = torch.zeros_like(want)
    for s, sign in ((0, 1.0), (1, 1.0), (2, -1.0)):
        want.index_add_(0, cols[:, s], sign * g)
        size.index_add_(0, cols[:, s], g.abs())
    # each term is off by its distance's and its own roundings, each sum by one rounding a level and entry of a chunk and of the
    # partial rows: 1e-5 of the terms' magnitudes, as everywhere
    assert torch.all((grads.rows[:u, :dim].double() - want[touched]).abs() <= 1e-5 * size[touched] + 1e-30)
