// What the kernels of link prediction share (stx_rank.hip, stx_rank_filter.hip): their arguments, the rows of a
// query, and one step of a distance sum.
#pragma once

#include "stx_rowops.h"

namespace stx {

// One step of the distance sum (Sec. 4.3, 4.6), index order.  The L2 kinds use a fused multiply-add.
template <int DIST>
__device__ inline float rank_step(float acc, float y)
{
    if (DIST == STX_L1) return acc + fabsf(y);
    if (DIST == STX_L2 || DIST == STX_L2_SQ) return __builtin_fmaf(y, y, acc);
    const float f = __builtin_amdgcn_fractf(y);            // fractional part, always below 1
    const float m = fminf(f, 1.0f - f);
    return DIST == STX_TORUS_L1 ? acc + m : __builtin_fmaf(m, m, acc);
}

constexpr int kRankTables = 32;        // TransR: relations per launch
constexpr int kRankBig = 1024;         // ... those with more queries than this get a launch of their own
struct RankIds {                       // (an argument of its own: indexed inside the struct that kernels copy and narrow,
    int32_t g[kRankTables];            // it would put that copy in memory)
};
struct RankArgs {
    const float *X;                    // TransE / TorusE: [E;R]; TransH: E.  Rows of dim floats
    const float *D, *W;                // TransH: d_r and w_r, n_rel rows each
    const int32_t *h, *r, *t;          // [nq]; r may be null: every query has relation 0
    int64_t nq;
    int32_t n_ent, n_rel;
    int dim;
    int32_t slice;                     // candidates per blockIdx.y, a multiple of kRankE
    float *true_score;                 // [nq]: the true entity's sum until k_rank_finish
    int32_t *n_less, *n_equal;         // [nq], cleared by k_rank_true
    int32_t *bad;                      // counter of out-of-range indices
    // TransR: blockIdx.z is one of up to kRankTables relations (RankIds); relation g owns the grouped queries
    // [grp_offsets[g], + grp_counts[g]) (h, t and the outputs are grouped arrays) and table number blockIdx.z.
    const int32_t *grp_counts, *grp_offsets;
    int64_t table_stride;              // floats between the tables of consecutive blockIdx.z
    const int32_t *gate;               // k_rank: nothing is done while this is zero; null: no such condition
};

// Narrows the arguments to the relation of this workgroup.
__device__ inline void rank_group(RankArgs &a, const RankIds &ids)
{
    if (!a.grp_counts) return;
    const int32_t g = ids.g[blockIdx.z];
    const int32_t n = a.grp_counts[g];
    const int64_t off = a.grp_offsets[g];
    a.X += (int64_t)blockIdx.z * a.table_stride;
    a.h += off; a.t += off;
    a.true_score += off; a.n_less += off; a.n_equal += off;
    a.nq = n;
}

// Clamped table rows of one query: q = h + r (tail side) or t - r (head side); the true entity is t or h.
struct RankRows {
    const float *pa, *pr, *ptrue;
    int32_t itrue;
    bool bad;
};
template <bool HEAD>
__device__ inline RankRows rank_rows(const RankArgs &a, int64_t qi)
{
    int32_t ih = a.h[qi], ir = a.r ? a.r[qi] : 0, it = a.t[qi];
    const bool bad = ih < 0 || ih >= a.n_ent || it < 0 || it >= a.n_ent || ir < 0 || ir >= a.n_rel;
    ih = min(max(ih, 0), a.n_ent - 1);
    it = min(max(it, 0), a.n_ent - 1);
    ir = min(max(ir, 0), a.n_rel - 1);
    return {a.X + (int64_t)(HEAD ? it : ih) * a.dim, a.X + ((int64_t)a.n_ent + ir) * a.dim,
            a.X + (int64_t)(HEAD ? ih : it) * a.dim, HEAD ? ih : it, bad};
}

// Counts of the active lanes' pairs.  A query that decides nothing brings many at once, and 400,000 additions to one
// counter, one by one, take 5 ms: the pairs of the first lane's query are added together, then those of the first lane that
// is left, TRIES times; what is then left (the usual mixture of queries) costs less in single additions.
template <int TRIES>
__device__ inline void rank_count(int32_t *n_less, int32_t *n_equal, uint32_t q, bool less, bool equal)
{
#pragma unroll 1
    for (int i = 0; i < TRIES; ++i) {
        const bool mine = q == (uint32_t)__builtin_amdgcn_readfirstlane((int)q);
        const int nl = __builtin_popcountll(__ballot(mine && less)), ne = __builtin_popcountll(__ballot(mine && equal));
        const uint64_t on = __ballot(true);
        if (__builtin_amdgcn_mbcnt_hi((uint32_t)(on >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)on, 0u)) == 0) {
            if (nl) atomicAdd(&n_less[q], nl);
            if (ne) atomicAdd(&n_equal[q], ne);
        }
        if (mine) return;
    }
    if (less) atomicAdd(&n_less[q], 1);
    if (equal) atomicAdd(&n_equal[q], 1);
}

// ---- stx_rank_transr.hip ------------------------------------------------------------------------------
struct RrBlock {
    int32_t rel, slot, first, count;   // up to 32 queries of a relation: their first grouped position; slot: number of the
};                                     // relation among those that occur
struct RankGroups {                    // queries grouped by relation
    const int32_t *h, *t;              // clamped
    float *score;
    int32_t *less, *equal;
    const RrBlock *blocks;             // [nq / 32 + relations]
    const int32_t *occ;                // relations that occur with at most `most` queries, in order; the blocks are theirs
    int32_t most;
};
// TransR's L2 kinds: true sums and counts of grouped queries (not the final square roots), given the queries per relation
// on the host, of the relations with at most `most` of them.  tables: relations that a launch over projected tables would
// take.  false: it would be slower than that, nothing launched.
bool rank_transr(stx_ctx *, const stx_params *, int64_t nq, int side, const RankGroups &, int tables, void *work, size_t bytes, const int32_t *counts);
int32_t rank_transr_most(const stx_config &);
size_t rank_transr_bytes(const stx_config &, int64_t nq, int tables);             // 0: a call that never takes this way

// ---- stx_rank_filter.hip ------------------------------------------------------------------------------
// Scratch of a filtered sweep: packed queries with their thresholds; packed candidates (matrix-core kinds).  Sweeps
// of more queries or candidates than fit go chunk by chunk.
struct RankScratch {
    char *q, *e;
    size_t q_bytes, e_bytes;
    float *q32;                        // TransR: fp32 query points of all grouped queries (else part of q)
};
// Whether one table's sweep of these sizes is faster filtered than plain, given q_bytes of query scratch.
bool rank_filter_pays(int dist, int64_t queries, int64_t n_ent, int width, size_t q_bytes);
size_t rank_filter_q_bytes(int dist, int width, int64_t queries);                 // 0: a kind without a filtered sweep
size_t rank_filter_e_bytes(int dist, int width, int64_t candidates, int tables);
// True scores and counts (not the final square roots) through the filter.  nz: 0, or the number of relations of a
// TransR launch (blockIdx.z), which must fit the scratch in one piece; queries: all of theirs.  false: not for this kind,
// nothing launched.
bool rank_filtered(stx_ctx *, const RankArgs &, int side, const RankScratch &, int nz, const RankIds &, int64_t queries);

// ---- stx_rank.hip -------------------------------------------------------------------------------------
// The plain sweep of queries [q0, q0 + nq) (TransR: of nz relations; q0 = 0), whose true sums are there and whose counters
// are cleared, done on the GPU only where *gate is not zero by then.
void rank_plain_behind(stx_ctx *, const RankArgs &, int side, int64_t q0, int64_t nq, int nz, const RankIds &, const int32_t *gate);

// ---- what the filtered sweeps share -------------------------------------------------------------------------------
constexpr float kUnit = 5.9604645e-8f; // 2^-24
constexpr float kWideMax = 32639.f;    // largest 16-bit number whose high byte, the low one being signed, fits

// Elements j .. j + 7 of a row, zeros past its end.
__device__ inline void load8(const float *p, int j, int dim, float (&v)[8])
{
    const float4 x = j < dim ? ld4(p + j) : make_float4(0.f, 0.f, 0.f, 0.f);
    const float4 y = j + 4 < dim ? ld4(p + j + 4) : make_float4(0.f, 0.f, 0.f, 0.f);
    v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w; v[4] = y.x; v[5] = y.y; v[6] = y.z; v[7] = y.w;
}
// Sixteen elements scaled and rounded to 16-bit fixed point, as high and (signed) low bytes; adds the squares of the scaled
// values, of the roundings and of the low bytes.
__device__ inline void wide_piece(const float *v, float sc, uint4 &hi, uint4 &lo, float &n2, float &d2, float &l2)
{
    uint32_t h[4], l[4];
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        h[w] = l[w] = 0u;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float x = v[4 * w + i] * sc;
            const float k = fminf(fmaxf(rintf(x), -kWideMax), kWideMax);
            const float d = x - k;
            n2 = __builtin_fmaf(x, x, n2);
            d2 = __builtin_fmaf(d, d, d2);
            const int n = (int)k, b = (int)(int8_t)n;
            l2 += (float)(b * b);
            l[w] |= ((uint32_t)b & 0xffu) << (8 * i);
            h[w] |= ((uint32_t)((n - b) >> 8) & 0xffu) << (8 * i);
        }
    }
    hi = make_uint4(h[0], h[1], h[2], h[3]);
    lo = make_uint4(l[0], l[1], l[2], l[3]);
}

// One kilobyte from global memory straight into LDS (16 bytes per lane, in lane order).  Completion is counted by
// vmcnt like any load; the waits are placed by hand where they are used.  The compiler cannot be told that m0 is written (a reserved
// register): it finds it as it left it.
__device__ inline void load_lds_1k(const uint4 *g, uint32_t lds)
{
    uint32_t m0;
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off\n\ts_mov_b32 m0, %0"
                 : "=&s"(m0) : "v"(g), "s"(__builtin_amdgcn_readfirstlane(lds)) : "memory");
}

__device__ inline void load_lds_256(const float *g, uint32_t lds)             // ... 256 bytes, four per lane
{
    uint32_t m0;
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %1, off\n\ts_mov_b32 m0, %0"
                 : "=&s"(m0) : "v"(g), "s"(__builtin_amdgcn_readfirstlane(lds)) : "memory");
}
__device__ inline uint32_t lds_at(const void *p) { return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void *)p; }

}  // namespace stx
