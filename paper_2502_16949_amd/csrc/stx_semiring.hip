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
#include <mutex>

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

// Scratch of stx_spmm_semiring_t_static for gradient rows that share memory with what the product reads.  Every GPU the
// library runs on holds its own copy of the array, at its own address, until the process ends.  In host code the
// array's name is only a handle for the symbol look-up below, never an address.
static __device__ __align__(256) unsigned char scratch[STX_STATIC_WORK_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices];   // device address of `scratch` on each GPU, null until first asked for
}  // namespace

static stx_status static_work(float **out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return STX_ERR_HIP;
    if (dev < 0 || dev >= kMaxDevices) return STX_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return STX_ERR_HIP;
        g_scratch_ptr[dev] = ptr;
    }
    *out = static_cast<float *>(g_scratch_ptr[dev]);
    return STX_OK;
}

// Gradient rows of the touched columns from where they were formed to where the caller wants them.
__global__ __launch_bounds__(kThreads) void k_copy_touched(const float4 *__restrict__ src, const int32_t *__restrict__ n_touched,
                                                           int row4, float4 *__restrict__ dst)
{
    const int64_t n = (int64_t)*n_touched * row4;
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kThreads) dst[i] = src[i];
}

static bool overlap(const float *a, int64_t na, const float *b, int64_t nb)
{
    const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
    return x < y + (uintptr_t)nb * 4 && y < x + (uintptr_t)na * 4;
}

// The product reads dL/dZ and the table while other workgroups store gradient rows.  A caller may hand over gradient
// rows that share memory with either (dL/dZ replaced in place): they are formed in `work` then, and copied.
stx_status launch_semiring_t(stx_ctx *c, const stx_incidence *inc, const stx_params *p, int kind, const float *gz,
                             float *work, float *out_rows)
{
    if (inc->n_rows == 0) return STX_OK;
    const int64_t dim = c->cfg.dim, cols = c->cfg.n_ent + c->cfg.n_rel, n_out = (inc->nnz < cols ? inc->nnz : cols) * c->ld;
    if (!overlap(out_rows, n_out, gz, inc->n_rows * dim) && !overlap(out_rows, n_out, p->ent, cols * dim))
        return launch_semiring_product_t(c, inc, p, kind, gz, out_rows);
    if (!work) {
        const stx_status s = static_work(&work);
        if (s != STX_OK) return s;
    }
    const stx_status s = launch_semiring_product_t(c, inc, p, kind, gz, work);
    if (s != STX_OK) return s;
    const int64_t blocks = (n_out / 4 + kThreads - 1) / kThreads;
    hipLaunchKernelGGL(k_copy_touched, dim3((unsigned)(blocks < 2048 ? blocks : 2048)), dim3(kThreads), 0, c->stream,
                       (const float4 *)work, inc->n_touched, c->ld / 4, (float4 *)out_rows);
    return hip_ok(hipGetLastError());
}

}  // namespace stx
