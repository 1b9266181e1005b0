"""What stx_rank assumes about the roundings of two matrix-core instructions: the bound of the filtered L2 sweep, and the
fused multiply-adds of TransR's projection, which are part of the interface (every sum in index order)."""
import ctypes as C
import os

import numpy as np
import pytest
import torch

from paper_2502_16949_amd import binding as B
from paper_2502_16949_amd.build import build_probe
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

N = 96
libm = C.CDLL("libm.so.6")
libm.fmaf.restype, libm.fmaf.argtypes = C.c_float, [C.c_float] * 3
fmaf = np.frompyfunc(libm.fmaf, 3, 1)


def _probe(name, a, b, c):
    so = os.path.join(os.path.dirname(os.path.abspath(__file__)), "libmfma_probe.so")
    lib = C.CDLL(so if os.path.exists(so) else build_probe())
    a, b, c = (torch.from_numpy(x).to(G.DEV) for x in (a, b, c))
    d = torch.full_like(c, float("nan"))
    args = [C.c_void_p(x.data_ptr()) for x in (a, b, c, d)] + [C.c_int(len(c)), C.c_void_p(torch.cuda.current_stream().cuda_stream)]
    assert getattr(lib, name)(*args) == 0
    torch.cuda.synchronize()
    return d.cpu().numpy()


def _f16(kind, rng):
    if kind.startswith("spread"):                         # products of one size and of many
        s = int(kind[6:])
        return tuple((rng.uniform(-1, 1, (N, 32, 16)) * 2.0 ** rng.integers(-s, s + 1, (N, 32, 16)) * 8).astype(np.float16)
                     for _ in range(2))
    if kind == "one":                                     # one product far larger than the rest
        size = 2.0 ** -rng.uniform(8, 13, (N, 1, 1))
        a, b = np.ones((N, 32, 16)) * size, rng.uniform(0.6, 1, (N, 32, 16)) * size
        at = rng.integers(0, 16, N)
        a[np.arange(N), :, at], b[np.arange(N), :, at] = 1.0, rng.uniform(1, 2, (N, 32))
        return a.astype(np.float16), b.astype(np.float16)
    # fp16 subnormals, as small elements of a scaled row are
    return (rng.uniform(-6e-5, 6e-5, (N, 32, 16)).astype(np.float16), rng.uniform(-128, 128, (N, 32, 16)).astype(np.float16))


@pytest.mark.parametrize("kind", ["spread0", "spread2", "spread6", "spread10", "one", "subnormal"])
def test_f16_product_error_bound(kind):
    # |computed - exact| <= 2^-24 (2.5 |c| + 10 sum |p|).  (Two groups of eight products each; in a group what lies below
    # 2^-24 of the largest is cut off, up to seven times, and each group's sum is rounded once into the accumulator: 2 |c| +
    # 9 sum |p|.)
    rng = np.random.default_rng(len(kind))
    a, b = _f16(kind, rng)
    p = np.einsum("nik,njk->nijk", a.astype(np.float64), b.astype(np.float64))   # (exact)
    total = np.abs(p).sum(-1)
    for scale in (0.0, 1e-3, 0.3, 1.0, 30.0, 1e4, None):
        if scale is None:
            c = -p.sum(-1).astype(np.float32)             # what is left of the sum is its roundings
        else:
            c = (total * scale * rng.uniform(-1, 1, (N, 32, 32))).astype(np.float32)
        got = _probe("probe_f16", a, b, c)
        err = np.abs(got.astype(np.float64) - (p.sum(-1) + c))
        used = err / (2.0**-24 * (2.5 * np.abs(c) + 10.0 * total) + 1e-300)
        print(f"{kind}, |c| about {scale} of the products: {used.max():.2f} of the bound")
        assert used.max() <= 1.0


@pytest.mark.parametrize("spread", [0, 4, 30])
def test_f32_product_is_a_chain_of_fused_multiply_adds(spread):
    rng = np.random.default_rng(spread)
    a, b = ((rng.uniform(-1, 1, (N // 4, 32, 2)) * 2.0 ** rng.integers(-spread, spread + 1, (N // 4, 32, 2))).astype(np.float32) for _ in range(2))
    c = (rng.uniform(-1, 1, (N // 4, 32, 32)) * 2.0 ** rng.integers(-2 * spread, 2 * spread + 1, (N // 4, 32, 32))).astype(np.float32)
    got = _probe("probe_f32", a, b, c)
    want = c
    for k in range(2):
        want = fmaf(a[:, :, None, k], b[:, None, :, k], want).astype(np.float32)
    assert np.array_equal(got.view(np.int32), want.view(np.int32))


@pytest.mark.parametrize("dim,k,spread", [(32, 32, 0), (96, 64, 4), (128, 160, 12)])
def test_transr_scores_are_index_order_sums(dim, k, spread):
    n_ent, n_rel, nq = 140, 3, 24
    rng = np.random.default_rng(dim)
    wide = lambda *s: (rng.uniform(-1, 1, s) * 2.0 ** rng.integers(-spread, spread + 1, s)).astype(np.float32)
    E, R, M = wide(n_ent, dim), wide(n_rel, k), wide(n_rel, k, dim)
    h, t = (rng.integers(0, n_ent, nq).astype(np.int32) for _ in range(2))
    r = rng.integers(0, n_rel, nq).astype(np.int32)
    ctx = B.Context(B.make_config("transr", "l2_sq", n_ent, n_rel, dim, 8, 1, rel_dim=k, flags=B.STX_FLAG_BF16_PROJ), G.DEV)
    p = B.Params(G.dev_f32(E), G.dev_f32(R), proj=G.dev_f32(M))
    work = torch.empty(B.stx_rank_work_bytes(ctx, nq) + 256, dtype=torch.uint8, device=G.DEV)
    ph, pt = (np.zeros((nq, k), np.float32) for _ in range(2))
    for j in range(dim):
        ph = fmaf(E[h, j][:, None], M[r, :, j], ph).astype(np.float32)
        pt = fmaf(E[t, j][:, None], M[r, :, j], pt).astype(np.float32)
    for side, y in ((B.STX_TAIL, (ph + R[r]) - pt), (B.STX_HEAD, ph - (pt - R[r]))):
        ts = torch.empty(nq, dtype=torch.float32, device=G.DEV)
        cnt = [torch.empty(nq, dtype=torch.int32, device=G.DEV) for _ in range(2)]
        B.stx_rank(ctx, p, G.dev_i32(h), G.dev_i32(r), G.dev_i32(t), side, ts, *cnt, work)
        want = np.zeros(nq, np.float32)
        for a in range(k):
            want = fmaf(y[:, a], y[:, a], want).astype(np.float32)
        assert np.array_equal(ts.cpu().numpy().view(np.int32), want.view(np.int32))
