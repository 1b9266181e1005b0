// Forward product C = A.X and the fused TransE / TorusE forward step.
//
// Every row of the incidence matrix A has exactly three entries (SparseTransX Sec. 4.2.2, Appendix B),
// so the sparse-dense product is a three-row gather: x_i = (X[h] + X[n_ent + r]) - X[t], with the `ht`
// form (Sec. 4.2.1) dropping the middle term.  A sub-wavefront group of LPR lanes owns one row and
// moves it as float4 per lane, so a 128-wide fp32 row is one 512-byte coalesced access by 32 lanes.
//
// The fused forward kernel gives one group a positive row and its k negatives: it computes the
// distances (Sec. 4.3, 4.6), the margin-ranking hinge (Sec. 5.3) and writes dL/dx of each of those
// rows straight away, so x itself never goes to memory.
#include "stx_emit_body.h"
#include "stx_forward_body.h"

namespace stx {

template <int LPR, int ITERS, bool HRT>
__global__ __launch_bounds__(kThreads) void k_spmm(const int32_t *__restrict__ colidx, const float *__restrict__ X,
                                                   int64_t n_rows, int dim, int32_t rel_off, float *__restrict__ C)
{
    const int lig = threadIdx.x % LPR;
    const int64_t row = ((int64_t)blockIdx.x * kThreads + threadIdx.x) / LPR;
    if (row >= n_rows) return;
    const int d4 = dim / 4;
    int32_t c0 = colidx[3 * row], c1 = colidx[3 * row + 1] - rel_off, c2 = colidx[3 * row + 2];
    RowVec<ITERS> x;
    gather_row<LPR, ITERS, HRT>(X, dim, d4, lig, c0, c1, c2, x);
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
        int j = lig + it * LPR;
        if (j < d4) st4(C + row * dim + 4 * j, x.v[it]);
    }
}

__global__ __launch_bounds__(kThreads) void k_finish_loss(const float *__restrict__ partials, int n, float scale,
                                                          float *__restrict__ loss)
{
    finish_loss_body(partials, n, scale, loss);
}

// (torus L2: six wavefronts per SIMD, as its terms take 76 to 79 registers; held to the 64 of eight, it spilled eleven of them:
// 20,000 positives and as many negatives, 256 floats a row: 29.0 us, with six 18.1)
template <int LPR, int ITERS, int DIST>
__global__ __launch_bounds__(kThreads, ITERS > 1 ? 1 : DIST == STX_TORUS_L2 ? 6 : 8) void k_forward_y(ForwardArgs a)
{
    forward_y_body<LPR, ITERS, DIST>((int)blockIdx.x, a);
}

// (rows of one float4 per lane: 64 registers, every workgroup of a large batch resident at once; wider rows hold
// four rows of ITERS float4 per lane)
template <int LPR, int ITERS, int DIST, bool PACKED, int NB, bool MORE, bool CHECK>
__global__ __launch_bounds__(kThreads, ITERS == 1 ? (NB == 1 || (PACKED && !MORE && !CHECK) ? 8 : PACKED && !(MORE && CHECK) ? 6 : 5) : ITERS == 2 ? (NB > 1 ? 3 : 4) : 2) void k_forward_stacked(ForwardArgs a)
{
    if (a.stream_rows) forward_body<LPR, ITERS, DIST, PACKED, NB, MORE, CHECK, true>((int)blockIdx.x, a);
    else if (!PACKED && LPR >= 32 && a.slice_sums) forward_body<LPR, ITERS, DIST, PACKED, NB, MORE, CHECK, false, !PACKED && LPR >= 32>((int)blockIdx.x, a);
    else forward_body<LPR, ITERS, DIST, PACKED, NB, MORE, CHECK, false>((int)blockIdx.x, a);
}

// The two parts of the sliced forward pass.  The slices are dealt to the dies, each of which keeps its own in its L2 cache.
// 393,216 positives, d = 1024, 16,296 rows of table: whole rows 404 us, the two parts 290 + 10.
template <int DIST, int NB, bool MORE, int PP>
__global__ __launch_bounds__(kThreads, 8) void k_forward_slices(ForwardArgs a, int nblocks, int nslices)
{
    const uint32_t total = (uint32_t)nblocks * (uint32_t)nslices, per = (total + 7u) / 8u;
    const uint32_t work = (blockIdx.x & 7u) * per + (blockIdx.x >> 3);
    if ((blockIdx.x >> 3) >= per || work >= total) return;
    forward_slice_body<DIST, NB, MORE, PP>((int)(work % (uint32_t)nblocks), (int)(work / (uint32_t)nblocks), a);
}
template <int DIST>
__global__ __launch_bounds__(kThreads) void k_forward_combine(ForwardArgs a, int nslices, int per)
{
    forward_combine_body<DIST>((int)blockIdx.x, nslices, per, a);
}

// TransR in stx_train_step: the first kernel of the next batch's build (which also counts the rows per relation)
// rides with the distances over the rows of y; nothing after this launch reads the A arrays it overwrites.
template <int LPR, int ITERS, int DIST>
__global__ __launch_bounds__(kThreads) void k_forward_y_emit(ForwardArgs a, EmitAhead ea)
{
    if ((int)blockIdx.x < ea.ntiles) emit_body<kSortItems, true, true, true>((int)blockIdx.x, ea.ntiles, ea.args);
    else forward_y_body<LPR, ITERS, DIST>((int)blockIdx.x - ea.ntiles, a);
}

__global__ void k_zero_loss(float *loss) { loss[0] = 0.f; }

__global__ __launch_bounds__(kThreads) void k_copy_f32(float *__restrict__ dst, const float *__restrict__ src, int64_t n4)
{
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n4; i += (int64_t)gridDim.x * kThreads)
        st4(dst + 4 * i, ld4(src + 4 * i));
}

stx_status launch_copy_f32(stx_ctx *c, float *dst, const float *src, int64_t n)
{
    if (n == 0) return STX_OK;
    int64_t n4 = n / 4, blocks = (n4 + kThreads - 1) / kThreads;
    if (blocks > 16384) blocks = 16384;
    hipLaunchKernelGGL(k_copy_f32, dim3((unsigned)blocks), dim3(kThreads), 0, c->stream, dst, src, n4);
    return hip_ok(hipGetLastError());
}

// Scattered reads of known volume: thread i reads the 32 bytes at the start of slot (i * 40503) mod n_slots (an
// odd multiplier, so a power-of-two number of slots is visited once each when n_reads == n_slots), `slot_bytes`
// apart: like the sign records the transposed product fetches, one memory sector per lane with no two lanes of a
// wavefront in one line when slot_bytes >= 128.  The sums go to `sink` so that the loads are kept.
__global__ __launch_bounds__(kThreads) void k_read_sectors(const char *__restrict__ src, int64_t n_slots, int slot_bytes,
                                                           int64_t n_reads, float *__restrict__ sink)
{
    float acc = 0.f;
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n_reads; i += (int64_t)gridDim.x * kThreads) {
        const int64_t slot = (i * 40503) % n_slots;
        const float *q = reinterpret_cast<const float *>(src + slot * slot_bytes);
        const float4 a = ld4(q), b = ld4(q + 4);
        acc += (a.x + a.y + a.z + a.w) + (b.x + b.y + b.z + b.w);
    }
    if (acc == 12345.678f) sink[blockIdx.x] = acc;   // practically never: the loads must only be kept
}

stx_status launch_read_sectors(stx_ctx *c, const void *src, int64_t n_slots, int slot_bytes, int64_t n_reads, float *sink)
{
    if (n_reads == 0) return STX_OK;
    int64_t blocks = (n_reads + kThreads - 1) / kThreads;
    if (blocks > 16384) blocks = 16384;
    hipLaunchKernelGGL(k_read_sectors, dim3((unsigned)blocks), dim3(kThreads), 0, c->stream, static_cast<const char *>(src),
                       n_slots, slot_bytes, n_reads, sink);
    return hip_ok(hipGetLastError());
}

stx_status launch_finish_loss(stx_ctx *c, int n_partials, float scale, float *loss)
{
    if (n_partials <= 0) hipLaunchKernelGGL(k_zero_loss, dim3(1), dim3(1), 0, c->stream, loss);
    else {
        ProfScope prof(c, "k_finish_loss");
        hipLaunchKernelGGL(k_finish_loss, dim3(1), dim3(kThreads), 0, c->stream, c->loss_partials, n_partials, scale,
                           loss);
    }
    return hip_ok(hipGetLastError());
}

// ---- dispatch --------------------------------------------------------------------------------------
template <int LPR, int ITERS>
static void spmm_go(stx_ctx *c, const stx_incidence *inc, const stx_params *p, float *out, bool hrt)
{
    int64_t threads = inc->n_rows * LPR;
    dim3 grid((unsigned)((threads + kThreads - 1) / kThreads));
    if (hrt)
        hipLaunchKernelGGL((k_spmm<LPR, ITERS, true>), grid, dim3(kThreads), 0, c->stream, inc->a_colidx, p->ent,
                           inc->n_rows, c->cfg.dim, 0, out);
    else
        hipLaunchKernelGGL((k_spmm<LPR, ITERS, false>), grid, dim3(kThreads), 0, c->stream, inc->a_colidx, p->ent,
                           inc->n_rows, c->cfg.dim, 0, out);
}

stx_status launch_spmm(stx_ctx *c, const stx_incidence *inc, const stx_params *p, float *out)
{
    if (inc->n_rows == 0) return STX_OK;
    Launch L = row_launch(c->cfg.dim);
    bool hrt = c->cfg.model == STX_TRANSE || c->cfg.model == STX_TORUSE;
    STX_DISPATCH_ROW(L, spmm_go, c, inc, p, out, hrt);
    return hip_ok(hipGetLastError());
}

// The forward pass of a step that forms its rows of dL/dx; returns the number of loss partials.
static int forward_slices_go(stx_ctx *c, const stx_incidence *inc, const stx_params *p, float *scores, float scale)
{
    const FormedRows fr = formed_buffers(c, inc->n_rows);
    const ForwardArgs fa{inc->a_colidx, p->ent, inc->b, inc->k, c->cfg.dim, c->cfg.margin, scale, scores, nullptr, 0,
                         c->loss_partials, p->rel_weight, (int32_t)c->cfg.n_ent, 0, 1, fr.coefs, fr.sums};
    const int nslices = (c->cfg.dim + 63) / 64, per = kThreads / row_launch(c->cfg.dim).lpr;
#define STX_SLICES(D, NB, MORE, PP)                                                                             \
    do {                                                                                                        \
        const int nblocks = (inc->b + kThreads / 16 * PP - 1) / (kThreads / 16 * PP);                           \
        hipLaunchKernelGGL((k_forward_slices<D, NB, MORE, PP>), dim3(((unsigned)nblocks * (unsigned)nslices + 7u) / 8u * 8u), \
                           dim3(kThreads), 0, c->stream, fa, nblocks, nslices);                                 \
    } while (0)
#define STX_FWD(D)                                                                                              \
    do {                                                                                                        \
        {                                                                                                       \
            ProfScope prof(c, "k_forward_slices");                                                              \
            if (inc->k <= 1) STX_SLICES(D, 1, false, 2);                                                        \
            else if (inc->k <= 4) STX_SLICES(D, 4, false, 1);                                                   \
            else STX_SLICES(D, 4, true, 1);                                                                     \
        }                                                                                                       \
        ProfScope prof(c, "k_forward_combine");                                                                 \
        hipLaunchKernelGGL((k_forward_combine<D>), dim3((inc->b + kThreads - 1) / kThreads), dim3(kThreads), 0, c->stream, \
                           fa, nslices, per);                                                                   \
    } while (0)
    if (c->cfg.dist == STX_L2) STX_FWD(STX_L2);
    else if (c->cfg.dist == STX_L2_SQ) STX_FWD(STX_L2_SQ);
    else STX_FWD(STX_TORUS_L2);
#undef STX_FWD
#undef STX_SLICES
    return (inc->b + per - 1) / per;
}

template <int LPR, int ITERS>
static void forward_go(stx_ctx *c, const stx_incidence *inc, const stx_params *p, float *scores, float *loss,
                       float scale, bool from_y, int width)
{
    constexpr int GROUPS = kThreads / LPR;
    dim3 grid((unsigned)((inc->b + GROUPS - 1) / GROUPS));
    const ForwardArgs fa{inc->a_colidx, p->ent, inc->b, inc->k, width, c->cfg.margin, scale, scores, c->gbuf[0],
                         packed_stride(c->cfg.dim), c->loss_partials, from_y ? nullptr : p->rel_weight,
                         (int32_t)c->cfg.n_ent, from_y ? 0 : big_tables(c),
                         !from_y && formed_rows(c, inc->n_rows) ? 1 : 0, nullptr, nullptr};
    // (the next batch's first build kernel, if one is due and counts rows per relation as TransR's do)
    EmitAhead ea{};
    if (from_y && c->ahead.armed && !c->ahead.emit_done && c->ahead.args.rc.cur) ea = take_emit_ahead(c);
    const dim3 grid_e(grid.x + (unsigned)ea.ntiles);
    // Negatives that the library's sampler drew in this build need no check of their kind.
    const bool sampled = c->sampled_inc == inc;
#define STX_ROWS2(D, P, NB, MORE)                                                                               \
    do {                                                                                                        \
        if (sampled)                                                                                            \
            hipLaunchKernelGGL((k_forward_stacked<LPR, ITERS, D, P, NB, MORE, false>), grid, dim3(kThreads), 0, c->stream, fa); \
        else                                                                                                    \
            hipLaunchKernelGGL((k_forward_stacked<LPR, ITERS, D, P, NB, MORE, true>), grid, dim3(kThreads), 0, c->stream, fa); \
    } while (0)
#define STX_ROWS(D, P)                                                                                          \
    do {                                                                                                        \
        if (inc->k <= 1) STX_ROWS2(D, P, fast_batch(ITERS, true), false);                                       \
        else if (inc->k <= 4) STX_ROWS2(D, P, fast_batch(ITERS, false), (ITERS > 2));                           \
        else STX_ROWS2(D, P, fast_batch(ITERS, false), true);                                                   \
    } while (0)
#define STX_FWD(D)                                                                                              \
    do {                                                                                                        \
        ProfScope prof(c, "k_forward_stacked");                                                                 \
        if (!from_y) STX_ROWS(D, is_sign_kind(D));                                                              \
        else if (ea.ntiles) hipLaunchKernelGGL((k_forward_y_emit<LPR, ITERS, D>), grid_e, dim3(kThreads), 0, c->stream, fa, ea); \
        else hipLaunchKernelGGL((k_forward_y<LPR, ITERS, D>), grid, dim3(kThreads), 0, c->stream, fa);          \
    } while (0)
    switch (c->cfg.dist) {
    case STX_L1: STX_FWD(STX_L1); break;
    case STX_L2: STX_FWD(STX_L2); break;
    case STX_TORUS_L1: STX_FWD(STX_TORUS_L1); break;
    case STX_L2_SQ: STX_FWD(STX_L2_SQ); break;
    default: STX_FWD(STX_TORUS_L2); break;
    }
#undef STX_FWD
#undef STX_ROWS
#undef STX_ROWS2
    if (c->defer_finish) { c->fin_n = (int)grid.x; c->fin_scale = scale; c->fin_loss = loss; }
    else launch_finish_loss(c, (int)grid.x, scale, loss);
}

stx_status launch_forward_stacked(stx_ctx *c, const stx_incidence *inc, const stx_params *p, float *scores,
                                  float *loss)
{
    if (inc->n_rows == 0) return launch_finish_loss(c, 0, 1.0f, loss);
    float scale = 1.0f;
    if (c->cfg.reduce == STX_MEAN && inc->k > 0) scale = 1.0f / (float)((int64_t)inc->b * inc->k);
    if (c->form_rows) {
        const int n = forward_slices_go(c, inc, p, scores, scale);
        if (c->defer_finish) { c->fin_n = n; c->fin_scale = scale; c->fin_loss = loss; }
        else launch_finish_loss(c, n, scale, loss);
        return hip_ok(hipGetLastError());
    }
    Launch L = row_launch(c->cfg.dim);
    STX_DISPATCH_ROW(L, forward_go, c, inc, p, scores, loss, scale, false, c->cfg.dim);
    return hip_ok(hipGetLastError());
}

// Distances, hinge and dL/dy over rows of y already stored in gbuf[0] (row width = out_dim).
stx_status launch_forward_from_y(stx_ctx *c, const stx_incidence *inc, const stx_params *p, float *scores,
                                 float *loss)
{
    float scale = 1.0f;
    if (c->cfg.reduce == STX_MEAN && inc->k > 0) scale = 1.0f / (float)((int64_t)inc->b * inc->k);
    Launch L = row_launch(c->out_dim);
    STX_DISPATCH_ROW(L, forward_go, c, inc, p, scores, loss, scale, true, c->out_dim);
    return hip_ok(hipGetLastError());
}

}  // namespace stx
