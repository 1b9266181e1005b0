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


# columns, entries, and what the sort does with them: bits of a digit, entries a tile, levels of its tables, and rounds of rows that a
# workgroup adds two counts a word before it takes them apart (one level)
SORTS = [(70_003, 3, 6, 1024, 1, 1), (70_003, 1024 * 3, 6, 1024, 1, 1), (70_003, 512 * 1024 - 2, 6, 1024, 1, 1),
         (40_003, 448 * 1024 - 1, 8, 1024, 1, 1), (40_003, 448 * 1024 + 2, 8, 1024, 1, 2), (40_003, 512 * 1024 - 2, 8, 1024, 1, 2),
         (40_003, 512 * 1024 + 1, 8, 4096, 1, 3), (40_003, 512 * 4096 - 2, 8, 4096, 1, 8), (70_003, 33 * 4096 * 8, 6, 4096, 1, 2),
         (40_003, 512 * 4096 + 1, 8, 4096, 2, 0), (40_003, 1024 * 4096 + 2, 8, 4096, 2, 0), (70_003, 1025 * 4096 + 1, 6, 4096, 2, 0),
         (3, 512 * 4096 + 1, 2, 4096, 2, 0), (3, 300 * 1024, 2, 1024, 1, 0)]


def _sort_of(cols, nnz):
    bits = max(1, (cols - 1).bit_length())
    passes = -(-bits // 8)
    digit = -(-bits // passes)
    tile = 1024 if nnz <= 1 << 19 else 4096
    tiles, parts = -(-nnz // tile), 256 // max(1, (1 << digit) // 8)
    levels = 2 if tiles > 512 else 1
    rows = 65535 // tile // 8 * 8 * parts
    return digit, tile, levels, -(-tiles // rows) if levels == 1 and digit > 2 else 0


@pytest.mark.parametrize("n_cols,entries,digit,tile,levels,rounds", SORTS)
@pytest.mark.parametrize("skew", ["one digit", "spread"])
def test_sorted_transpose_of_full_tiles(n_cols, entries, digit, tile, levels, rounds, skew):
    b, n_rel = entries // 3, 3 if n_cols > 3 else 1
    n_ent = n_cols - n_rel
    assert 3 * b == entries and _sort_of(n_cols, entries) == (digit, tile, levels, rounds)
    rng = np.random.default_rng(entries)
    if skew == "one digit":                                 # all of a tile's keys fall on one first digit, as many as a count can be
        h, t, r = np.full(b, max(0, n_ent - (1 << digit))), np.full(b, max(0, n_ent - (2 << digit))), np.zeros(b)
        h[-1] = 5 % n_ent
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
    want, start = np.unique(cols), np.flatnonzero(np.diff(cols[order], prepend=-1))
    assert u == len(want) and np.array_equal(inc.at_touched_cols[:u].cpu().numpy(), want)
    assert np.array_equal(inc.at_seg_ptr[:u + 1].cpu().numpy(), np.append(start, nnz))


# 300,000 entries of the exact sums (of the L1 kinds), divided by the slices of 256 floats that a row has, and a million of the
# others: both sides of the lines, and the lengths of a lane group's walk on either side at 32 and 64 lanes
@pytest.mark.parametrize("dist,dim,rows", [("l1", 200, 100_000), ("l1", 200, 100_002), ("l1", 128, 100_000), ("l1", 128, 100_002),
                                           ("l1", 520, 33_332), ("l1", 520, 33_334), ("l1", 1024, 25_000), ("l1", 1024, 25_002),
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


# Sums that round are added in one order up to a million entries, also where the exact ones change theirs (more than 300,000
# entries) or once did (460,800 of 65 to 128 floats, 230,400 of more): a column that sorts first and has the same entries in a
# batch on either side gets the same bits.  The mean's scale is halved by twice the pairs, exactly.
@pytest.mark.parametrize("model,dist,dim,mean,weights,b_small,b_large", [
    ("transe", "l1", 200, False, True, 38_000, 76_000), ("transe", "l1", 200, True, False, 29_000, 58_000),
    ("toruse", "torus_l1", 128, False, True, 49_000, 98_000), ("toruse", "torus_l1", 128, True, False, 40_000, 80_000),
    ("transe", "l1", 520, False, True, 24_000, 48_000), ("transe", "l2", 200, False, False, 38_000, 76_000)])
def test_sums_that_round_keep_their_order(model, dist, dim, mean, weights, b_small, b_large):
    n_ent, n_rel, hot = 30_000, 7, 9_000
    gen = torch.Generator(device=DEV)
    gen.manual_seed(dim)
    rand = lambda *shape: torch.rand(*shape, generator=gen, device=DEV) - 0.5
    p = B.Params(rand(n_ent + n_rel, dim), rel_weight=torch.rand(n_rel, generator=gen, device=DEV) + 0.3 if weights else None)
    if model == "toruse":
        p.ent.copy_(p.ent - torch.floor(p.ent))
    ints = lambda lo, hi: torch.randint(lo, hi, (b_large,), generator=gen, device=DEV, dtype=torch.int32)
    h, r, t, nh = ints(1, n_ent), ints(0, n_rel), ints(1, n_ent), ints(1, n_ent)
    h[torch.randperm(b_small, generator=gen, device=DEV)[:hot]] = 0
    got = []
    for b in (b_small, b_large):
        ctx = B.Context(B.make_config(model, dist, n_ent, n_rel, dim, b, 1, margin=1000.0,   # every pair is active
                                      reduce=B.STX_MEAN if mean else B.STX_SUM), DEV)
        inc, grads = B.Incidence(ctx), B.Grads(ctx)
        scores, loss = torch.zeros(2 * b, device=DEV), torch.zeros(1, device=DEV)
        B.stx_build_incidence(ctx, h[:b], r[:b], t[:b], nh[:b], t[:b], 1, inc)
        B.stx_forward(ctx, inc, p, scores, loss)
        B.stx_backward(ctx, inc, p, grads)
        torch.cuda.synchronize()
        assert int(inc.at_touched_cols[0]) == 0 and int(inc.at_seg_ptr[1]) == hot
        got.append(grads.rows[0, :dim] * (b / b_small if mean else 1.0))
    assert torch.equal(got[0].view(torch.int32), got[1].view(torch.int32))


# The semiring gradient: short chunks up to 2,304 tiles of them (147,456 entries; 294,912 at 128 floats), and up to 360,000 entries where
# long ones fill the chip unevenly (162,000 entries: 2.47 workgroups a unit, and three times that at 520 floats; 180,000: 2.75;
# 195,000: 2.98; 294,915: 4.50)
@pytest.mark.parametrize("kind", [B.STX_DISTMULT, B.STX_COMPLEX, B.STX_ROTATE])
@pytest.mark.parametrize("dim", [128, 200, 520])
@pytest.mark.parametrize("b", [54_000, 60_000, 65_000, 98_305, 120_001])
def test_semiring_gradient_on_both_sides_of_its_line(kind, dim, b):
    n_ent, n_rel = 9_000, 7
    gen = torch.Generator(device=DEV)
    gen.manual_seed(dim + b)
    x = torch.rand(n_ent + n_rel, dim, generator=gen, device=DEV) - 0.5
    h, r, t = (torch.randint(0, hi, (b,), generator=gen, device=DEV, dtype=torch.int32) for hi in (n_ent, n_rel, n_ent))
    h[: b // 3] = 11
    ctx = B.Context(B.make_config("transe", "l2", n_ent, n_rel, dim, b, 0), DEV)
    inc, grads = B.Incidence(ctx), B.Grads(ctx)
    none = torch.zeros(0, dtype=torch.int32, device=DEV)
    B.stx_build_incidence(ctx, h, r, t, none, none, 0, inc)
    gz, work = torch.rand(b, dim, generator=gen, device=DEV) - 0.5, torch.empty(3 * b * dim, device=DEV)
    B.stx_spmm_semiring_t(ctx, inc, B.Params(x), kind, gz, work, grads)
    torch.cuda.synchronize()
    cols = [c.long() for c in (h, r + n_ent, t)]
    leaves = [x.double()[c].requires_grad_() for c in cols]
    if kind == B.STX_DISTMULT:
        z = leaves[0] * leaves[1] * leaves[2]
    else:
        ch, cr, ct = (torch.view_as_complex(v.view(b, dim // 2, 2)) for v in leaves)
        z = torch.view_as_real(ch * cr * ct.conj() if kind == B.STX_COMPLEX else ch * cr - ct).reshape(b, dim)
    g = torch.autograd.grad(z, leaves, gz.double())
    u = int(inc.n_touched.item())
    touched = inc.at_touched_cols[:u].long()
    want = torch.zeros(n_ent + n_rel, dim, dtype=torch.float64, device=DEV)
    size = torch.zeros_like(want)
    # (the roundings of a ComplEx term are of the products it is the sum of: at most twice their larger ones, gz and two factors of 1/2)
    for c, v in zip(cols, g):
        want.index_add_(0, c, v)
        size.index_add_(0, c, v.abs() + 2.0 ** -3)
    assert torch.all((grads.rows[:u, :dim].double() - want[touched]).abs() <= 1e-5 * size[touched])


# TransR's rows of dL/dx and dL/dy, on both sides of 3,600 tiles of 128 and of 64 entries: a batch's gradient is the sum of its
# halves', which lie on the short side.
@pytest.mark.parametrize("dim,line", [(128, 3600 * 128), (256, 3600 * 64)])
@pytest.mark.parametrize("beyond", [0, 2])
def test_transr_product_on_both_sides_of_its_line(dim, line, beyond):
    b, n_ent, n_rel = line // 6 + beyond, 5_000, 7
    gen = torch.Generator(device=DEV)
    gen.manual_seed(dim + b)
    rand = lambda *shape: torch.rand(*shape, generator=gen, device=DEV) - 0.5
    p = B.Params(rand(n_ent, dim), rand(n_rel, dim), proj=rand(n_rel, dim, dim))
    h, r, t, nh = (torch.randint(0, hi, (b,), generator=gen, device=DEV, dtype=torch.int32) for hi in (n_ent, n_rel, n_ent, n_ent))
    h[: b // 3] = 11

    def gradient(part):
        n = len(h[part])
        ctx = B.Context(B.make_config("transr", "l2", n_ent, n_rel, dim, n, 1, rel_dim=dim, margin=1000.0, flags=B.STX_FLAG_BF16_PROJ), DEV)
        inc, grads = B.Incidence(ctx), B.Grads(ctx)
        scores, loss = torch.zeros(2 * n, device=DEV), torch.zeros(1, device=DEV)
        B.stx_build_incidence(ctx, h[part], r[part], t[part], nh[part], t[part], 1, inc)
        B.stx_forward(ctx, inc, p, scores, loss)
        B.stx_backward(ctx, inc, p, grads)
        torch.cuda.synchronize()
        u = int(inc.n_touched.item())
        out = torch.zeros(n_ent + n_rel, dim, dtype=torch.float64, device=DEV)
        out[inc.at_touched_cols[:u].long()] = grads.rows[:u, :dim].double()
        return out

    got, want = gradient(slice(0, b)), gradient(slice(0, b // 2)) + gradient(slice(b // 2, b))
    # the terms' magnitudes: |dL/dy| is one (L2, weight one), so |dL/dx| is at most the largest |M_r|, row by row
    bound = torch.cat([p.proj.norm(dim=1).max().expand(n_ent), torch.ones(n_rel, device=DEV)]).double()[:, None]
    count = torch.bincount(torch.cat([h, nh, t, t, r + n_ent, r + n_ent]).cpu().long(), minlength=n_ent + n_rel).to(DEV)
    assert torch.all((got - want).abs() <= 1e-5 * bound * count[:, None])
