// The three-entry product under the semirings of SparseTransX Appendix D, and its backward.
//
// Appendix D keeps the incidence matrix (a head, a relation and a tail column per row) and swaps the
// operators of the sparse-dense product: the row's entries are multiplied instead of added, with real
// products for DistMult (h r t), complex ones for ComplEx (h r conj(t)) and RotatE (h r - t).  A table
// row of a complex kind holds dim/2 numbers as (re, im) pairs, so a lane's float4 is two of them.
// Every real product and sum is rounded once, in the order written in cmul() and below.
//
// Backward for a real loss, given G = dL/dZ: every entry of a row receives G times the (conjugated)
// product of the row's other two factors.  The transposed product (stx_backward.hip) forms that where it
// sums the entries of a column.
#include "stx_semiring_ops.h"

namespace stx {

template <int KIND>
__device__ inline float4 product(float4 h, float4 r, float4 t)
{
    if (KIND == SR_DISTMULT) return mul4(mul4(h, r), t);
    const float2 p0 = cmul(lo2(h), lo2(r)), p1 = cmul(hi2(h), hi2(r));
    if (KIND == SR_COMPLEX) return join(cmul(p0, conj2(lo2(t))), cmul(p1, conj2(hi2(t))));
    return make_float4(p0.x - t.x, p0.y - t.y, p1.x - t.z, p1.y - t.w);
}

template <int LPR, int ITERS, int KIND>
__global__ __launch_bounds__(kThreads) void k_semiring(const int32_t *__restrict__ colidx, const float *__restrict__ X,
                                                       int64_t n_rows, int dim, float *__restrict__ Z)
{
    const int lig = threadIdx.x % LPR;
    const int64_t row = ((int64_t)blockIdx.x * kThreads + threadIdx.x) / LPR;
    if (row >= n_rows) return;
    const int d4 = dim / 4;
    const float *ph = X + (int64_t)colidx[3 * row] * dim, *pr = X + (int64_t)colidx[3 * row + 1] * dim;
    const float *pt = X + (int64_t)colidx[3 * row + 2] * dim;
    float4 h[ITERS], r[ITERS], t[ITERS];
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {   // all loads first
        const int j = min(lig + it * LPR, d4 - 1);
        h[it] = ld4(ph + 4 * j); r[it] = ld4(pr + 4 * j); t[it] = ld4(pt + 4 * j);
    }
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
        const int j = lig + it * LPR;
        if (j < d4) st4_stream(Z + row * dim + 4 * j, product<KIND>(h[it], r[it], t[it]));
    }
}

template <int LPR, int ITERS>
static void semiring_go(stx_ctx *c, const stx_incidence *inc, const stx_params *p, int kind, float *out)
{
    const int64_t threads = inc->n_rows * LPR;
    const dim3 grid((unsigned)((threads + kThreads - 1) / kThreads)), block(kThreads);
    const int dim = c->cfg.dim;
    ProfScope prof(c, "k_semiring");
#define STX_SR(K)                                                                                               \
    hipLaunchKernelGGL((k_semiring<LPR, ITERS, K>), grid, block, 0, c->stream, inc->a_colidx, p->ent, inc->n_rows, dim, out)
    if (kind == SR_DISTMULT) STX_SR(SR_DISTMULT);
    else if (kind == SR_COMPLEX) STX_SR(SR_COMPLEX);
    else STX_SR(SR_ROTATE);
#undef STX_SR
}

stx_status launch_semiring(stx_ctx *c, const stx_incidence *inc, const stx_params *p, int kind, float *z_out)
{
    if (inc->n_rows == 0) return STX_OK;
    Launch L = row_launch(c->cfg.dim);
    STX_DISPATCH_ROW(L, semiring_go, c, inc, p, kind, z_out);
    return hip_ok(hipGetLastError());
}

}  // namespace stx
