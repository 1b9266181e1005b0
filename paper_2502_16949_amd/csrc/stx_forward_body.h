// Device-side bodies of the fused TransE / TorusE forward step and of the final loss sum, shared by the
// kernels that run them alone (stx_forward.hip) and by the launches that run them beside another,
// independent piece of work (stx_step.hip).
#pragma once

#include "stx_rowops.h"

namespace stx {

// Packed dL/dy row of an L1-kind distance: record `row` of gs = coefficient (fp32), then the sign bytes.
template <int LPR, int ITERS, int DIST>
__device__ inline void write_grad_row_packed(uint8_t *__restrict__ gs, int gstride, float *__restrict__ coefs,
                                             int64_t row, int d4, int lig, const RowVec<ITERS> &x, float coef)
{
    uint8_t *rec = gs + row * gstride;
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
        int j = lig + it * LPR;
        if (j < d4) rec[j] = (uint8_t)sign_bits<DIST>(x.v[it]);
    }
    if (lig == 0) coefs[row] = coef;
}

template <int LPR, int ITERS, int DIST>
__device__ inline void write_grad_row(float *__restrict__ g, int d4, int lig, const RowVec<ITERS> &x, float coef,
                                      float dist)
{
    const float cs = coef_scale<DIST>(coef, dist);
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
        int j = lig + it * LPR;
        if (j < d4)
            st4(g + 4 * j, make_float4(dterm<DIST>(x.v[it].x, cs), dterm<DIST>(x.v[it].y, cs),
                                       dterm<DIST>(x.v[it].z, cs), dterm<DIST>(x.v[it].w, cs)));
    }
}

// The coefficient of a row that is formed again where it is summed.  +0 there means that the row adds nothing and is
// not fetched; an inactive row with an infinity or a NaN in it keeps -0, as its stored products would be NaN.
template <int DIST>
__device__ inline float formed_coef(float coef, float dist)
{
    const float cs = coef_scale<DIST>(coef, dist);
    return cs != 0.f ? cs : fabsf(dist) < __builtin_inff() ? 0.f : -0.f;
}

// Sum of the per-workgroup loss partials in a fixed order (one workgroup, after the forward kernel).
// ARENA: the body's LDS array lives in the kFinishLds bytes at `lds` (8-byte aligned) instead of its own.
template <bool ARENA = false>
__device__ inline void finish_loss_body(const float *__restrict__ partials, int n, float scale,
                                        float *__restrict__ loss, unsigned char *lds = nullptr)
{
    double *s_acc;
    if constexpr (ARENA) {
        s_acc = reinterpret_cast<double *>(lds);
    } else {
        __shared__ double o_acc[kThreads];
        s_acc = o_acc;
    }
    const int tid = threadIdx.x;
    double a = 0.0;
    int i = tid;
    for (; i + 7 * kThreads < n; i += 8 * kThreads) {   // eight loads in flight, added in index order
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = partials[i + u * kThreads];
#pragma unroll
        for (int u = 0; u < 8; ++u) a += (double)v[u];
    }
    for (; i < n; i += kThreads) a += (double)partials[i];
    s_acc[tid] = a;
    __syncthreads();
    for (int off = kThreads / 2; off >= 1; off >>= 1) {
        if (tid < off) s_acc[tid] += s_acc[tid + off];
        __syncthreads();
    }
    if (tid == 0) loss[0] = (float)(s_acc[0] * (double)scale);
}

// The forward step for batches whose negatives come from the sampler (Sec. 5.3: every negative keeps the relation
// and one entity of its positive).  One group per positive: its lanes fetch the 3 + 3 NB column ids of the positive
// and its first NB negatives in ONE load (id j in lane j; two loads when the group has fewer lanes) and share them by
// shuffles; then the positive's three rows and the ONE row in which each negative differs are requested together
// (3 + k table rows instead of 3 + 3k), so a wavefront pays two dependent memory round trips.  Further negatives
// follow NB at a time, their ids requested a batch ahead, so each batch costs one more.
// x is formed by the same two roundings in the same order as a full gather would: the bits are those of
// forward_any_rows.
// MORE: the batch may have more than NB negatives per positive (the loop costs registers).
// CHECK: the negatives may be a caller's own.  false is returned, by all lanes of the group, when one of another kind
// turns up: what was written until then is to be written again (forward_any_rows).
// STREAM: the table is far larger than the caches, and a row used once does not displace the others.
// SLICES: distances are summed as the sliced pass sums them (forward_slice_body).
template <int LPR, int ITERS, int DIST, bool PACKED, int NB, bool MORE, bool CHECK, bool STREAM, bool SLICES>
__device__ inline bool forward_fast_rows(const int32_t i, const int lig, const ForwardArgs &a, float &hinge_sum)
{
    constexpr int NI = (3 + 3 * NB + LPR - 1) / LPR;       // column ids per lane
    const int32_t *__restrict__ colidx = a.colidx;
    const float *__restrict__ X = a.X;
    const int32_t b = a.b, k = a.k;
    const int dim = a.dim, d4 = dim / 4, gstride = a.gstride;
    float *__restrict__ scores = a.scores;
    const int32_t row0 = b + i * k;
    int32_t mine[NI];                                  // id j of (positive, negatives of the batch) in lane j % LPR
#pragma unroll
    for (int u = 0; u < NI; ++u) {
        const int j = lig + u * LPR;
        mine[u] = 0;
        if (j < 3 + 3 * min(k, NB)) mine[u] = colidx[j < 3 ? 3 * (int64_t)i + j : 3 * (int64_t)row0 + (j - 3)];
    }
    auto id = [&](int j) { return __shfl(mine[j / LPR], j % LPR, LPR); };
    const int32_t c0 = id(0), c1 = id(1), c2 = id(2);
    const float wr = a.rel_weight ? a.rel_weight[c1 - a.n_ent] : 1.0f;
    // (lanes past the row's width hold its last float4 again, see load_vec: every reduction leaves them out)
    RowVec<ITERS> hr, pr, pt, xp;
    load_vec<LPR, ITERS>(X + (int64_t)c0 * dim, d4, lig, hr);
    load_vec<LPR, ITERS>(X + (int64_t)c1 * dim, d4, lig, pr);
    load_vec<LPR, ITERS>(X + (int64_t)c2 * dim, d4, lig, pt);
    uint8_t *recs = reinterpret_cast<uint8_t *>(a.G);
    float *gcoef = PACKED ? reinterpret_cast<float *>(recs + packed_coef_offset((int64_t)b * (1 + k), gstride)) : nullptr;
    bool shared = true;
    int n_active = 0;
    float npos = 0.f, dpos = 0.f;
    for (int q0 = 0; q0 == 0 || (MORE && q0 < k); q0 += NB) {
        int32_t ce[NB];
        unsigned tail_mask = 0;
#pragma unroll
        for (int q = 0; q < NB; ++q) {
            const int32_t nh = id(3 + 3 * q), nr = id(4 + 3 * q), nt = id(5 + 3 * q);
            const bool ts = nh == c0;
            ce[q] = ts ? nt : nh;
            tail_mask |= ts ? 1u << q : 0u;
            if (CHECK && q0 + q < k) shared = shared && nr == c1 && (ts || nt == c2);
        }
        if (CHECK && !shared) return false;
        RowVec<ITERS> e[NB];
#pragma unroll
        for (int q = 0; q < NB; ++q)
            if (q0 + q < k) load_vec<LPR, ITERS, STREAM>(X + (int64_t)ce[q] * dim, d4, lig, e[q]);
        if (MORE && q0 + NB < k) {                     // the next batch's ids, in the places of this one's
#pragma unroll
            for (int u = 0; u < NI; ++u) {
                const int j = lig + u * LPR;
                if (j >= 3 && j < 3 + 3 * min(k - q0 - NB, NB)) mine[u] = colidx[3 * (int64_t)(row0 + q0 + NB) + (j - 3)];
            }
        }
        if (q0 == 0) {
#pragma unroll
            for (int it = 0; it < ITERS; ++it) {
                hr.v[it] = add4(hr.v[it], pr.v[it]);
                xp.v[it] = sub4(hr.v[it], pt.v[it]);
            }
            npos = row_distance<LPR, ITERS, DIST, SLICES>(xp, d4, lig);
            dpos = wr * npos;
            if (lig == 0) scores[i] = dpos;
        }
#pragma unroll
        for (int q = 0; q < NB; ++q)
            if (q0 + q < k) {
                RowVec<ITERS> x;
#pragma unroll
                for (int it = 0; it < ITERS; ++it)
                    x.v[it] = (tail_mask >> q & 1u) ? sub4(hr.v[it], e[q].v[it]) : sub4(add4(e[q].v[it], pr.v[it]), pt.v[it]);
                const float nneg = row_distance<LPR, ITERS, DIST, SLICES>(x, d4, lig);
                const float dneg = wr * nneg;
                const float arg = (a.margin + dpos) - dneg;
                const bool active = arg > 0.f;
                const int32_t row = row0 + q0 + q;
                if (lig == 0) scores[row] = dneg;
                if (active) { hinge_sum += arg; ++n_active; }
                if (PACKED)
                    write_grad_row_packed<LPR, ITERS, DIST>(recs, gstride, gcoef, row, d4, lig, x, active ? -a.scale * wr : 0.f);
                else
                    write_grad_row<LPR, ITERS, DIST>(a.G + (int64_t)row * dim, d4, lig, x, active ? -a.scale * wr : 0.f, nneg);
            }
    }
    if (PACKED)
        write_grad_row_packed<LPR, ITERS, DIST>(recs, gstride, gcoef, i, d4, lig, xp, (float)n_active * a.scale * wr);
    else
        write_grad_row<LPR, ITERS, DIST>(a.G + (int64_t)i * dim, d4, lig, xp, (float)n_active * a.scale * wr, npos);
    return true;
}

// One group per positive i: rows i and b + i*k + kk (kk < k).
// FROM_Y = false: the translated vector of a row is gathered from the stacked table X (TransE/TorusE).
// FROM_Y = true : it is row `row` of the dense buffer G (TransR: y = M_r (h - t) + r was put there by
//                 the projection kernel), and dL/dy overwrites it in place; every row is read and then
//                 written by one group only.
// PACKED (L1 kinds, gathered rows only): dL/dx is written as records of gstride bytes at G (sign bytes), the
// rows' coefficients behind the records of the batch.
// K1: at most one negative per positive (the benchmarks' shape): no registers are kept for a batch of them, and
// more wavefronts fit (same arithmetic in the same order, so the same bits).
template <int LPR, int ITERS, int DIST, bool FROM_Y, bool PACKED, bool K1, bool SLICES = false>
__device__ inline void forward_any_rows(const int64_t i, const int lig, const ForwardArgs &a, float &hinge_sum)
{
    const int32_t *__restrict__ colidx = a.colidx;
    const float *__restrict__ X = a.X;
    const int32_t b = a.b, k = a.k;
    const int dim = a.dim, gstride = a.gstride;
    const float margin = a.margin, scale = a.scale;
    float *__restrict__ scores = a.scores;
    float *G = a.G;
    float *gcoef = PACKED ? reinterpret_cast<float *>(reinterpret_cast<uint8_t *>(a.G) +
                                                      packed_coef_offset((int64_t)b * (1 + k), gstride))
                          : nullptr;
    static_assert(!PACKED || (is_sign_kind(DIST) && !FROM_Y), "packed rows need an L1-kind distance");
    const int d4 = dim / 4;
    // Negatives are taken NB at a time so that the kernel pays two memory round trips per batch (all
    // column ids, then all table rows) instead of two per row; the positive rides with the first batch.
    constexpr int NB = K1 ? 1 : (ITERS <= 2 ? 4 : 2);
    RowVec<ITERS> xp;
    float dpos = 0.f, npos = 0.f;   // the positive's score and its norm (they differ by the relation's weight)
    int n_active = 0;
    int32_t cp[3] = {0, 0, 0};
    if (!FROM_Y) { cp[0] = colidx[3 * i]; cp[1] = colidx[3 * i + 1]; cp[2] = colidx[3 * i + 2]; }
    // Table 2, TransM row: a fixed weight per relation multiplies the norm (1 when there is none; the
    // negatives of a positive keep its relation).  Multiplying by 1 changes no bit.
    const float wr = (!FROM_Y && a.rel_weight) ? a.rel_weight[cp[1] - a.n_ent] : 1.0f;
    for (int kk0 = 0; kk0 < k || kk0 == 0; kk0 += NB) {
        const int nb = min(NB, k - kk0);
        const int64_t row0 = (int64_t)b + i * k + kk0;
        int32_t cn[NB][3];
        RowVec<ITERS> xn[NB];
        if (!FROM_Y) {
#pragma unroll
            for (int q = 0; q < NB; ++q) {
                const int64_t rr = q < nb ? row0 + q : i;   // past the end: re-read the positive's ids
                cn[q][0] = colidx[3 * rr]; cn[q][1] = colidx[3 * rr + 1]; cn[q][2] = colidx[3 * rr + 2];
            }
        }
        if (kk0 == 0) {
            if (FROM_Y) load_vec<LPR, ITERS>(G + i * dim, d4, lig, xp);
            else gather_row<LPR, ITERS, true>(X, dim, d4, lig, cp[0], cp[1], cp[2], xp);
        }
#pragma unroll
        for (int q = 0; q < NB; ++q) {
            if (q < nb) {
                if (FROM_Y) load_vec<LPR, ITERS>(G + (row0 + q) * dim, d4, lig, xn[q]);
                else gather_row<LPR, ITERS, true>(X, dim, d4, lig, cn[q][0], cn[q][1], cn[q][2], xn[q]);
            }
        }
        if (kk0 == 0) {
            npos = row_distance<LPR, ITERS, DIST, SLICES>(xp, d4, lig);
            dpos = wr * npos;
            if (lig == 0) scores[i] = dpos;
        }
#pragma unroll
        for (int q = 0; q < NB; ++q) {
            if (q < nb) {
                const int64_t row = row0 + q;
                const float nneg = row_distance<LPR, ITERS, DIST, SLICES>(xn[q], d4, lig);
                const float dneg = wr * nneg;
                const float arg = (margin + dpos) - dneg;
                const bool active = arg > 0.f;
                if (lig == 0) scores[row] = dneg;
                if (active) { hinge_sum += arg; ++n_active; }
                if (PACKED)
                    write_grad_row_packed<LPR, ITERS, DIST>(reinterpret_cast<uint8_t *>(G), gstride, gcoef, row, d4,
                                                            lig, xn[q], active ? -scale * wr : 0.f);
                else
                    write_grad_row<LPR, ITERS, DIST>(G + row * dim, d4, lig, xn[q], active ? -scale * wr : 0.f,
                                                     nneg);
            }
        }
    }
    if (PACKED)
        write_grad_row_packed<LPR, ITERS, DIST>(reinterpret_cast<uint8_t *>(G), gstride, gcoef, i, d4, lig, xp,
                                                (float)n_active * scale * wr);
    else
        write_grad_row<LPR, ITERS, DIST>(G + i * dim, d4, lig, xp, (float)n_active * scale * wr, npos);
}

// Sum of the groups' hinge terms of workgroup `block` (of those of the forward pass; the launch may hold others).
template <int GROUPS>
__device__ inline void forward_loss(const int block, const int lig, const int grp, float hinge_sum, const ForwardArgs &a)
{
    __shared__ float s_loss[GROUPS];
    if (lig == 0) s_loss[grp] = hinge_sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        float sum = 0.f;
#pragma unroll
        for (int g = 0; g < GROUPS; ++g) sum += s_loss[g];
        a.loss_partials[block] = sum;
    }
}

// The distances over rows of y (TransR).
template <int LPR, int ITERS, int DIST>
__device__ inline void forward_y_body(const int block, const ForwardArgs &a)
{
    constexpr int GROUPS = kThreads / LPR;
    const int lig = threadIdx.x % LPR, grp = threadIdx.x / LPR;
    const int64_t i = (int64_t)block * GROUPS + grp;
    float hinge_sum = 0.f;
    if (i < a.b) forward_any_rows<LPR, ITERS, DIST, true, false, false>(i, lig, a, hinge_sum);   // (uniform within the group)
    forward_loss<GROUPS>(block, lig, grp, hinge_sum, a);
}

// Gathered rows.  CHECK: a positive whose negatives are a caller's own, of a kind that forward_fast_rows does not cover,
// takes three table rows for each, in the same kernel: in a launch of its own behind a fast one, whose groups had then
// loaded and stored for nothing, such batches took 1.4 to 1.7 times as long.
template <int LPR, int ITERS, int DIST, bool PACKED, int NB, bool MORE, bool CHECK, bool STREAM, bool SLICES = false>
__device__ inline void forward_body(const int block, const ForwardArgs &a)
{
    constexpr int GROUPS = kThreads / LPR;
    const int lig = threadIdx.x % LPR, grp = threadIdx.x / LPR;
    const int64_t i = (int64_t)block * GROUPS + grp;
    float hinge_sum = 0.f;
    if (i < a.b && !forward_fast_rows<LPR, ITERS, DIST, PACKED, NB, MORE, CHECK, STREAM, SLICES>((int32_t)i, lig, a, hinge_sum) && CHECK) {
        hinge_sum = 0.f;
        forward_any_rows<LPR, ITERS, DIST, false, PACKED, NB == 1, SLICES>(i, lig, a, hinge_sum);
    }
    forward_loss<GROUPS>(block, lig, grp, hinge_sum, a);
}

// Negatives that forward_fast_rows holds at a time, for k of them per positive: as many rows in flight as the
// registers allow (rows of ITERS float4 per lane, the positive's three beside them).
// (Eight at a time, in one batch for up to eight: 35.6 us for 9,999 positives x 5 at d = 200, four waves per SIMD and
// spills, against 27.0 with four at a time and five waves.)
constexpr int fast_batch(int iters, bool k1) { return k1 ? 1 : iters <= 2 ? 4 : 2; }

// The forward step inside the launches of stx_train_step, whose negatives are the sampler's.  K1: the launch was
// chosen for at most one negative per positive.
template <int LPR, int ITERS, int DIST, bool PACKED, bool K1>
__device__ inline void forward_step_body(const int block, const ForwardArgs &fa)
{
    forward_body<LPR, ITERS, DIST, PACKED, fast_batch(ITERS, K1), !K1, false, false>(block, fa);
}

// The forward pass of a batch whose rows of dL/dx are formed where they are summed (formed_rows), first part: the share of one
// 64-float slice of the columns in every row's distance.  Such a batch reads the table many times over, and whole rows of it
// come from the last-level cache (8 TB/s for random rows of 64 MB); a slice of the whole table stays in a die's L2, which gives
// 30 TB/s in float4 loads of 16 lanes a row (18 in single floats of 64 lanes).  Sixteen lanes per positive, PP positives side by
// side in each group; sums[slice][row].  The second part (k_forward_combine) adds a row's shares in order.
template <int DIST, int NB, bool MORE, int PP>
__device__ inline void forward_slice_body(const int block, const int slice, const ForwardArgs &a)
{
    constexpr int LPR = 16, GROUPS = kThreads / LPR, SPAN = LPR / PP;   // SPAN: lanes that hold a positive's column ids
    static_assert(3 + 3 * NB <= SPAN && (PP == 1 || !MORE), "a lane for each column id");
    const int lig = threadIdx.x % LPR, grp = threadIdx.x / LPR;
    const int32_t b = a.b, k = a.k;
    const int dim = a.dim, c4 = slice * LPR, n4 = min(LPR, dim / 4 - c4);   // float4 of the slice
    const float *__restrict__ X = a.X + 4 * c4;
    const int32_t *__restrict__ colidx = a.colidx;
    float *__restrict__ sums = a.sums + (int64_t)slice * b * (1 + k);
    const int32_t i0 = (block * GROUPS + grp) * PP;
    if (i0 >= b) return;
    const int mp = min(lig / SPAN, PP - 1), mj = lig % SPAN;
    const int32_t mi = min(i0 + mp, b - 1);                // (a positive past the last one: the last one again, not stored)
    int32_t mine = 0;
    if (mj < 3 + 3 * min(k, NB)) mine = colidx[mj < 3 ? 3 * (int64_t)mi + mj : 3 * ((int64_t)b + (int64_t)mi * k) + (mj - 3)];
    auto id = [&](int p, int j) { return __shfl(mine, p * SPAN + j, LPR); };
    RowVec<1> hr[PP], pr[PP], pt[PP];
    int32_t c0[PP];
#pragma unroll
    for (int p = 0; p < PP; ++p) {
        c0[p] = id(p, 0);
        load_vec<LPR, 1>(X + (int64_t)c0[p] * dim, n4, lig, hr[p]);
        load_vec<LPR, 1>(X + (int64_t)id(p, 1) * dim, n4, lig, pr[p]);
        load_vec<LPR, 1>(X + (int64_t)id(p, 2) * dim, n4, lig, pt[p]);
    }
    for (int q0 = 0; q0 == 0 || (MORE && q0 < k); q0 += NB) {
        RowVec<1> e[PP][NB];
        unsigned tail_mask[PP];
#pragma unroll
        for (int p = 0; p < PP; ++p) {
            tail_mask[p] = 0;
#pragma unroll
            for (int q = 0; q < NB; ++q) {
                const int32_t nh = id(p, 3 + 3 * q), nt = id(p, 5 + 3 * q);
                const bool ts = nh == c0[p];
                tail_mask[p] |= ts ? 1u << q : 0u;
                if (q0 + q < k) load_vec<LPR, 1>(X + (int64_t)(ts ? nt : nh) * dim, n4, lig, e[p][q]);
            }
        }
        if (MORE && q0 + NB < k && mj >= 3 && mj < 3 + 3 * min(k - q0 - NB, NB))   // the next batch's ids
            mine = colidx[3 * ((int64_t)b + (int64_t)mi * k + q0 + NB) + (mj - 3)];
#pragma unroll
        for (int p = 0; p < PP; ++p) {
            if (q0 == 0) {
                hr[p].v[0] = add4(hr[p].v[0], pr[p].v[0]);
                const float s = sum16(lig < n4 ? sum_terms<DIST>(sub4(hr[p].v[0], pt[p].v[0])) : 0.f);
                if (lig == 0 && i0 + p < b) sums[i0 + p] = s;
            }
#pragma unroll
            for (int q = 0; q < NB; ++q)
                if (q0 + q < k) {
                    const float4 x = (tail_mask[p] >> q & 1u) ? sub4(hr[p].v[0], e[p][q].v[0]) : sub4(add4(e[p][q].v[0], pr[p].v[0]), pt[p].v[0]);
                    const float s = sum16(lig < n4 ? sum_terms<DIST>(x) : 0.f);
                    if (lig == 0 && i0 + p < b) sums[(int64_t)b + (int64_t)(i0 + p) * k + q0 + q] = s;
                }
        }
    }
}

// ... second part: a thread per positive adds the shares of its rows, slice by slice, and does the rest of the forward step.
// per: positives to a loss partial, as the kernel for whole rows has them.
template <int DIST>
__device__ inline void forward_combine_body(const int block, const int nslices, const int per, const ForwardArgs &a)
{
    __shared__ float s_hinge[kThreads];
    const int32_t b = a.b, k = a.k, i = block * kThreads + (int)threadIdx.x;
    const int64_t rows = (int64_t)b * (1 + k);
    float hinge_sum = 0.f;
    if (i < b) {
        auto distance = [&](int64_t row) {
            float sum = 0.f;
#pragma unroll 8
            for (int s = 0; s < nslices; ++s) sum += a.sums[s * rows + row];
            return finish<DIST>(fabsf(sum));
        };
        const float wr = a.rel_weight ? a.rel_weight[a.colidx[3 * (int64_t)i + 1] - a.n_ent] : 1.0f;
        const float npos = distance(i), dpos = wr * npos;
        a.scores[i] = dpos;
        int n_active = 0;
        for (int q = 0; q < k; ++q) {
            const int64_t row = (int64_t)b + (int64_t)i * k + q;
            const float nneg = distance(row), dneg = wr * nneg;
            const float arg = (a.margin + dpos) - dneg;
            const bool active = arg > 0.f;
            a.scores[row] = dneg;
            if (active) { hinge_sum += arg; ++n_active; }
            a.coefs[row] = formed_coef<DIST>(active ? -a.scale * wr : 0.f, nneg);
        }
        a.coefs[i] = formed_coef<DIST>((float)n_active * a.scale * wr, npos);
    }
    s_hinge[threadIdx.x] = hinge_sum;
    __syncthreads();
    const int at = (int)threadIdx.x * per;
    if (at < kThreads && block * kThreads + at < b) {
        float sum = 0.f;
        for (int g = 0; g < per; ++g) sum += s_hinge[at + g];
        a.loss_partials[(block * kThreads + at) / per] = sum;
    }
}

}  // namespace stx
