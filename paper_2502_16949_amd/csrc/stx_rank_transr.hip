// Link prediction with projection matrices (TransR, Sec. 4.4), L2 kinds, without a projected table.
//
// The score of candidate e is dist(q - M_r e) (or dist(M_r e - q), the same number), q = M_r h + r or M_r t - r, and
// its counts are defined by fp32 sums: P = M_r e with fused multiply-adds in index order, then the distance sum of q - P in
// index order.  Projecting every entity for every relation that way runs at the rate of the fp32 matrix cores, and took half
// of the call; packing what came out for the sweep read it all once more.  But
//     |q - M e|^2 = |q|^2 - 2 (M^T q).e + |M e|^2,
// so the sweep can run over the entity table itself, packed once for all relations, with v = M^T q in the query's place,
// if |M e|^2 is known for the relation and entity: a number each, formed on the fp16 matrix cores from operands split in two
// (22 bits).  All of this has a bound on its distance from the sums that count, most of it those sums' own rounding; the pairs
// it leaves undecided (about one in 500 at d = k = 128) are projected and summed exactly as written there, 64 pairs of one
// relation at a time.
//
//   k_rr_pack    entity table and matrices as operands, 32 rows a tile
//   k_rr_query   blocks of 32 queries of one relation: their points and true sums (exact), v, its operands and bounds
//   k_rr_norms   |M_r e|^2 for all entities, relation by relation
//   k_rr_sweep   the decisions
//   k_rr_pairs   undecided pairs, exactly
//   k_rr_behind  all pairs exactly, where a sweep found too many of them; returns at once otherwise
//
// 20,466 queries of 237 relations x 14,500 entities, d = k = 128, both sides: 5,330 us with projected tables, 1,690 now, of
// which a side's norms take 274, sweep 250, pairs 220, queries 57.  Relations with many queries keep a table (rank_transr_most).
#include <algorithm>
#include <new>

#include "stx_rank.h"

namespace stx {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef int intx4 __attribute__((ext_vector_type(4)));
typedef int intx16 __attribute__((ext_vector_type(16)));

constexpr int kPairBlock = 64;         // undecided pairs of one relation that are projected together
constexpr int kAux = 64;               // floats that go with a tile of 32 entities: of the table, and of a relation

struct RrState {
    uint32_t n_blocks;                 // pair blocks begun, cleared by k_rr_query
    int32_t pad[31];
    int32_t full;                      // there were too many, in this sweep or one before it in the call
    int32_t skip;                      // `full` as it was before this sweep
};
struct RrArgs {
    const float *E, *M, *R;
    int32_t n_ent, dim, k;
    int head;                          // side: q = M t - r instead of M h + r
    const int32_t *gh, *gt;            // grouped queries: clamped head and tail
    float *gts;                        // ... the true entity's sum
    int32_t *gless, *gequal;
    const RrBlock *blocks;
    const int32_t *occ;                // relations that occur, in order
    int32_t b0, b1;                    // blocks of this sweep
    int32_t slot0, slots;              // relations of this batch
    float *q32;                        // [grouped position][k]: the query's point
    uint4 *qf;                         // [block][step][lane]: v as high and low bytes
    float4 *qpar;                      // [block * 32 + i][2]
    uint4 *ew;                         // entities as high and low bytes ...
    float *eaux;                       // ... [tile][kAux]: scale, largest norm, largest rounding, largest norm of the low bytes; scale of `es`
    uint4 *es, *ms;                    // entities and this batch's matrices as fp16 pairs: [tile][step][two][lane]
    float *maux;                       // [tile of ms]: 1 / scale^2, infinite where the tile is out of range
    float *nn;                         // [slot][tile of 32][kAux]: |M e|^2, then the root of the largest
    uint2 *pairs;                      // [pair block][kPairBlock]: entity, grouped position
    int2 *heads;                       // [pair block]: relation, pairs
    int32_t pair_blocks;
    RrState *st;
    int32_t first;                     // the call's first sweep
};

// ---- operands -------------------------------------------------------------------------------------------------
// Eight elements as fp16 and the fp16 of what that leaves: 22 bits.
__device__ inline void rr_split(const float (&v)[8], float sc, uint4 &hi, uint4 &lo)
{
    half8 h, l;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const float x = v[i] * sc;                         // exact: sc is a power of two
        h[i] = (_Float16)x;
        l[i] = (_Float16)(x - (float)h[i]);
    }
    hi = __builtin_bit_cast(uint4, h);
    lo = __builtin_bit_cast(uint4, l);
}
// Tiles of 32 rows, eight threads a row.  The first `etiles` workgroups: entities; the others: 32 rows of a matrix of this
// batch each.  Bound by the bytes read and written.
template <int KS>
__global__ __launch_bounds__(kThreads) void k_rr_pack(RrArgs f, int etiles)
{
    __shared__ float s_r[4], s_n[32], s_d[32], s_l[32];
    const int tid = threadIdx.x, u = tid >> 3, l8 = tid & 7, dim = f.dim;
    const bool ent = (int)blockIdx.x < etiles;
    const int tile = ent ? (int)blockIdx.x : (int)blockIdx.x - etiles;
    bool in = true;
    const float *p;
    if (ent) {
        const int64_t e = (int64_t)tile * 32 + u;
        in = e < f.n_ent;
        p = f.E + min(e, (int64_t)f.n_ent - 1) * dim;
    } else {
        const int kt = f.k / 32, slot = tile / kt;
        p = f.M + ((int64_t)f.occ[f.slot0 + slot] * f.k + (tile - slot * kt) * 32 + u) * dim;
    }
    float mx = 0.f;
    bool nan = false;
    for (int j = l8 * 4; j < dim; j += 32) {
        const float4 v = ld4(p + j);
        mx = fmaxf(fmaxf(fmaxf(mx, fabsf(v.x)), fmaxf(fabsf(v.y), fabsf(v.z))), fabsf(v.w));
        nan = nan || v.x != v.x || v.y != v.y || v.z != v.z || v.w != v.w;
    }
    if (nan) mx = __builtin_inff();
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) mx = fmaxf(mx, __shfl_xor(mx, m, 64));
    if ((tid & 63) == 0) s_r[tid >> 6] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(s_r[0], s_r[1]), fmaxf(s_r[2], s_r[3]));
    // (products of these stay far from the ends of the fp32 range; nothing is decided by what does not)
    const bool ok = mx == 0.f || (mx > 1e-6f && mx < 1e6f);
    const float sp = ok && mx != 0.f ? ldexpf(1.f, 6 - ilogbf(mx)) : 1.f;      // largest element: [64, 128)
    uint4 *ds = (ent ? f.es : f.ms) + (int64_t)tile * KS * 128;
    for (int q = l8; q < 2 * KS; q += 8) {
        float v[8];
        uint4 hi, lo;
        load8(p, q * 8, dim, v);
        rr_split(v, ok ? sp : 0.f, hi, lo);
        if (!in) hi = lo = make_uint4(0u, 0u, 0u, 0u);
        ds[(q >> 1) * 128 + u + 32 * (q & 1)] = hi;
        ds[(q >> 1) * 128 + 64 + u + 32 * (q & 1)] = lo;
    }
    if (!ent) {
        if (tid == 0) f.maux[tile] = ok ? 1.f / (sp * sp) : __builtin_inff();
        return;
    }
    const float sw = ok && mx != 0.f ? kWideMax / mx : 1.f;
    float n2 = 0.f, d2 = 0.f, l2 = 0.f;
    uint4 *dw = f.ew + (int64_t)tile * KS * 64;
    for (int q = l8; q < KS; q += 8) {                     // sixteen elements
        float v[16];
        uint4 hi, lo;
        load8(p, q * 16, dim, *(float (*)[8])v);
        load8(p, q * 16 + 8, dim, *(float (*)[8])(v + 8));
        wide_piece(v, ok ? sw : 0.f, hi, lo, n2, d2, l2);
        if (!in) hi = lo = make_uint4(0u, 0u, 0u, 0u);
        dw[(q >> 1) * 128 + u + 32 * (q & 1)] = hi;
        dw[(q >> 1) * 128 + 64 + u + 32 * (q & 1)] = lo;
    }
    n2 = group_sum<8>(n2);
    d2 = group_sum<8>(d2);
    l2 = group_sum<8>(l2);
    if (l8 == 0) { s_n[u] = n2; s_d[u] = d2; s_l[u] = l2; }
    __syncthreads();
    if (tid >= 32) return;
    n2 = s_n[tid]; d2 = s_d[tid]; l2 = s_l[tid];
#pragma unroll
    for (int m = 16; m >= 1; m >>= 1) {
        n2 = fmaxf(n2, __shfl_xor(n2, m, 32));
        d2 = fmaxf(d2, __shfl_xor(d2, m, 32));
        l2 = fmaxf(l2, __shfl_xor(l2, m, 32));
    }
    if (tid) return;
    float *aux = f.eaux + (int64_t)tile * kAux;
    const float en = ok ? sqrtf(n2) * 1.0001f : __builtin_inff();
    st4(aux, make_float4(sw, en, sqrtf(d2) * 1.002f + 1.01f * kUnit * en, sqrtf(l2) * 1.001f));
    aux[4] = sp;
}

// ---- exact rows -----------------------------------------------------------------------------------------------
// P = M_r e of the 64 entities s_id, all k outputs, in registers: acc[c][u][i] is output 128 c + 32 wave + (lane & 31) of row
// 32 u + (i & 3) + 8 (i >> 2) + 4 (lane >> 5).  v_mfma_f32_32x32x2_f32 performs the fused multiply-adds of an index-order
// loop, as in k_rr_project.  lds: kStageLds bytes.
constexpr int kLdM = 132, kLdE = 68;
constexpr int kStageLds = 32 * (kLdM + kLdE) * 4;
template <int A>
__device__ inline void rr_project(const RrArgs &f, int32_t rel, const int32_t *s_id, float *lds, floatx16 (&acc)[A][2])
{
    float (*s_m)[kLdM] = reinterpret_cast<float (*)[kLdM]>(lds);
    float (*s_e)[kLdE] = reinterpret_cast<float (*)[kLdE]>(lds + 32 * kLdM);
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, l31 = lane & 31, wa = (tid >> 6) * 32;
    const int cm = tid & 127, jm = (tid >> 7) * 4, ce = tid & 63, je = (tid >> 6) * 4, dim = f.dim;
    const float *pe = f.E + (int64_t)s_id[ce] * dim + je;
#pragma unroll
    for (int c = 0; c < A; ++c) {
        const float *pm = f.M + ((int64_t)rel * f.k + min(128 * c + cm, f.k - 1)) * dim + jm;
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[c][u][i] = 0.f;
        float4 vm[4], ve[2];
#pragma unroll
        for (int i = 0; i < 4; ++i) vm[i] = ld4(pm + 8 * i);
#pragma unroll
        for (int i = 0; i < 2; ++i) ve[i] = ld4(pe + 16 * i);
        for (int j0 = 0; j0 < dim; j0 += 32) {
            __syncthreads();
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int jj = jm + 8 * i;
                s_m[jj][cm] = vm[i].x; s_m[jj + 1][cm] = vm[i].y; s_m[jj + 2][cm] = vm[i].z; s_m[jj + 3][cm] = vm[i].w;
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int jj = je + 16 * i;
                s_e[jj][ce] = ve[i].x; s_e[jj + 1][ce] = ve[i].y; s_e[jj + 2][ce] = ve[i].z; s_e[jj + 3][ce] = ve[i].w;
            }
            __syncthreads();
            if (j0 + 32 < dim) {
#pragma unroll
                for (int i = 0; i < 4; ++i) vm[i] = ld4(pm + j0 + 32 + 8 * i);
#pragma unroll
                for (int i = 0; i < 2; ++i) ve[i] = ld4(pe + j0 + 32 + 16 * i);
            }
            if (128 * c + wa >= f.k) continue;             // (uniform over the wavefront)
#pragma unroll
            for (int jj = 0; jj < 32; jj += 2) {
                const float mv = s_m[jj + half][wa + l31];
#pragma unroll
                for (int u = 0; u < 2; ++u)
                    acc[c][u] = __builtin_amdgcn_mfma_f32_32x32x2f32(s_e[jj + half][32 * u + l31], mv, acc[c][u], 0, 0, 0);
            }
        }
    }
    __syncthreads();                                       // (the caller may write over lds)
}
// ... into LDS: s_p[output * kLdP + row].
constexpr int kLdP = 65;
template <int A>
__device__ inline void rr_spread(const RrArgs &f, const floatx16 (&acc)[A][2], float *s_p)
{
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, wa = (tid >> 6) * 32;
#pragma unroll
    for (int c = 0; c < A; ++c) {
        const int a = 128 * c + wa + (lane & 31);
        if (a < f.k)
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int i = 0; i < 16; ++i) s_p[a * kLdP + 32 * u + (i & 3) + 8 * (i >> 2) + 4 * half] = acc[c][u][i];
    }
    __syncthreads();
}
static size_t rr_exact_lds(int k) { return std::max((size_t)kStageLds, (size_t)k * kLdP * 4); }
static size_t rr_query_lds(int dim, int k) { return rr_exact_lds(k) + (size_t)32 * (dim + 1) * 4; }

// ---- queries --------------------------------------------------------------------------------------------------
// A block of 32 queries: rows 0 .. 31 are their own entities, 32 .. 63 the true ones.  Then v = M^T q and what its sums
// against candidates can be off by.  In units scaled by v's scale s and the candidate tile's, over 256, with t = q.P_fl -
// |P_fl|^2/2 - tau, tau = (|q|^2 - S_true)/2 (P_fl: as the index-order loop rounds it, f = |M|_F), a candidate is below the true
// entity when t > 0, and what is computed differs by
//   the fixed-point roundings       |v| |de| + |dv| (|e| + |de|); the low bytes' own product: at most that of their norms
//   v and q.P_fl                    the loops' roundings: u sum_j |partial sum j|, the partial sums bounded by the absolute ones,
//                                   so that element j counts (length - j) times: |q| |e| u (g + h), g and h the norms of
//                                   M's elements times those counts along either index
//   |M e|^2                         (2 |P| + eps) eps / 2, eps = |e| (u g + f (7.5 steps + 30) u): the loop's rounding, 22-bit
//                                   operands, the matrix cores' sums (at most 2^-24 (2.5 |C| + 10 sum |p|) an instruction, as
//                                   tests/test_gpu_mfma_rounding.py checks), and the sum of its squares
//   norms, tau, thresholds          a few fp32 roundings, chains of k / 8; the index-order sums (k + 8) u S_true / 2
template <int KS, int A, bool HEAD>
__global__ __launch_bounds__(kThreads, 2) void k_rr_query(RrArgs f)
{
    extern __shared__ __align__(16) unsigned char s_dyn[];
    __shared__ int32_t s_id[64];
    __shared__ float s_st[32], s_sum[3][4];
    const int tid = threadIdx.x, dim = f.dim, k = f.k;
    if (blockIdx.x == 0 && tid == 0) {
        const int32_t full = f.first ? 0 : f.st->full;
        f.st->n_blocks = 0u;
        f.st->skip = full;
        if (f.first) f.st->full = 0;
    }
    const RrBlock blk = f.blocks[f.b0 + blockIdx.x];
    if (tid < 64) {
        const int q = blk.first + min(tid & 31, blk.count - 1);
        s_id[tid] = (tid >= 32) != HEAD ? f.gt[q] : f.gh[q];             // own: head (tail side) or tail; true: the other
    }
    __syncthreads();
    float *s_p = reinterpret_cast<float *>(s_dyn);
    float *s_v = s_p + (kStageLds / 4 > k * kLdP ? kStageLds / 4 : k * kLdP);
    constexpr int LD = kLdP;
    {
        floatx16 acc[A][2];
        rr_project<A>(f, blk.rel, s_id, s_p, acc);
        rr_spread<A>(f, acc, s_p);
    }
    const float *rvec = f.R + (int64_t)blk.rel * k;
    for (int i = tid; i < 32 * k; i += kThreads) {
        const int a = i % k, row = i / k;
        const float p = s_p[a * LD + row], q = HEAD ? p - rvec[a] : p + rvec[a];
        s_p[a * LD + row] = q;
        if (row < blk.count) f.q32[(int64_t)(blk.first + row) * k + a] = q;
    }
    __syncthreads();
    if (tid < 32) {                                        // the true entity's sum, index order
        float acc = 0.f;
        for (int a0 = 0; a0 < k; a0 += 32) {
            float y[32];
#pragma unroll
            for (int a = 0; a < 32; ++a) {
                const float q = s_p[(a0 + a) * LD + tid], e = s_p[(a0 + a) * LD + 32 + tid];
                y[a] = HEAD ? e - q : q - e;
            }
#pragma unroll
            for (int a = 0; a < 32; ++a) acc = rank_step<STX_L2>(acc, y[a]);
        }
        s_st[tid] = acc;
        if (tid < blk.count) {
            f.gts[blk.first + tid] = acc;
            f.gless[blk.first + tid] = 0;
            f.gequal[blk.first + tid] = 0;
        }
    }
    // v on the fp32 matrix cores too, 32 columns a wavefront: rows are queries; and M's norms
    float f2 = 0.f, g2 = 0.f, h2 = 0.f;
    for (int j0 = (tid >> 6) * 32; j0 < dim; j0 += 128) {
        const int lane = tid & 63, half = lane >> 5, j = j0 + (lane & 31);
        const float *pm = f.M + ((int64_t)blk.rel * k + half) * dim + j;
        floatx16 acc;
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = 0.f;
        const float wj = (float)(dim - j + 1);
        for (int a0 = 0; a0 < k; a0 += 32) {
            float m[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) m[i] = pm[(int64_t)(a0 + 2 * i) * dim];
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int a = a0 + 2 * i + half;
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(s_p[a * LD + (lane & 31)], m[i], acc, 0, 0, 0);
                const float wg = m[i] * wj, wh = m[i] * (float)(k - a + 1);
                f2 = __builtin_fmaf(m[i], m[i], f2);
                g2 = __builtin_fmaf(wg, wg, g2);
                h2 = __builtin_fmaf(wh, wh, h2);
            }
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) s_v[((i & 3) + 8 * (i >> 2) + 4 * half) * (dim + 1) + j] = acc[i];
    }
    f2 = group_sum<64>(f2);
    g2 = group_sum<64>(g2);
    h2 = group_sum<64>(h2);
    if ((tid & 63) == 0) { s_sum[0][tid >> 6] = f2; s_sum[1][tid >> 6] = g2; s_sum[2][tid >> 6] = h2; }
    __syncthreads();
    const int u = tid >> 3, l8 = tid & 7;
    float q2 = 0.f;
    for (int a = l8; a < k; a += 8) { const float q = s_p[a * LD + u]; q2 = __builtin_fmaf(q, q, q2); }
    q2 = group_sum<8>(q2);
    const float *v = s_v + u * (dim + 1);
    float mx = 0.f;
    bool nan = false;
    for (int i = l8; i < dim; i += 8) { mx = fmaxf(mx, fabsf(v[i])); nan = nan || v[i] != v[i]; }
    if (nan) mx = __builtin_inff();
#pragma unroll
    for (int m = 4; m >= 1; m >>= 1) mx = fmaxf(mx, __shfl_xor(mx, m, 8));
    const bool ok = mx == 0.f || (mx > 1e-12f && mx < 1e12f);
    const float sc = ok && mx != 0.f ? kWideMax / mx : 1.f;
    float n2 = 0.f, d2 = 0.f, l2 = 0.f;
    uint4 *dst = f.qf + (int64_t)(f.b0 + blockIdx.x) * KS * 64;
    for (int p = l8; p < KS; p += 8) {
        float x[16];
        uint4 hi, lo;
#pragma unroll
        for (int i = 0; i < 16; ++i) x[i] = p * 16 + i < dim ? v[p * 16 + i] : 0.f;
        wide_piece(x, ok ? sc : 0.f, hi, lo, n2, d2, l2);
        dst[(p >> 1) * 128 + u + 32 * (p & 1)] = hi;
        dst[(p >> 1) * 128 + 64 + u + 32 * (p & 1)] = lo;
    }
    n2 = group_sum<8>(n2);
    d2 = group_sum<8>(d2);
    l2 = group_sum<8>(l2);
    if (l8) return;
    f2 = s_sum[0][0] + s_sum[0][1] + s_sum[0][2] + s_sum[0][3];
    g2 = s_sum[1][0] + s_sum[1][1] + s_sum[1][2] + s_sum[1][3];
    h2 = s_sum[2][0] + s_sum[2][1] + s_sum[2][2] + s_sum[2][3];
    const float fm = sqrtf(f2) * 1.0001f, gm = sqrtf(g2) * 1.0001f, hm = sqrtf(h2) * 1.0001f;
    const float s = sc * (1.f / 256.f), st = s_st[u], qn = sqrtf(q2) * 1.0001f, vn = sqrtf(n2) * 1.0001f;
    const float dv = sqrtf(d2) * 1.002f + 1.01f * kUnit * vn;
    const float kap = 0.5f * kUnit * (float)(k / 8 + 24);
    float4 p0, p1;
    p0.x = (dv * 1.001f + 6.f * kUnit * vn) * (1.f / 256.f) + s * qn * 1.01f * kUnit * (gm + hm);   // times the tile's largest norm
    p0.y = vn * (1.f / 256.f);                             // times its largest rounding
    p0.z = 0.5f * (q2 - st) * s;                           // tau, times its scale
    p0.w = s * (kap * (q2 + st) + 0.51f * (float)(k + 8) * kUnit * st) + 8.f * kUnit * fabsf(p0.z);   // times its scale
    p1.x = s;
    p1.y = sqrtf(l2) * 1.001f * (1.f / 256.f);             // times its largest norm of the low bytes
    p1.z = 1.01f * kUnit * (gm + fm * (7.5f * (float)KS + 30.f));              // eps for a norm of 1
    p1.w = 0.f;
    if (!ok || !(p0.w < 1e30f) || !(p1.z < 1e30f)) p0.w = __builtin_inff();
    if (u >= blk.count) { p0 = make_float4(0.f, 0.f, 3e37f, 0.f); p1.x = 1.f; p1.y = p1.z = 0.f; }
    float4 *par = f.qpar + ((int64_t)(f.b0 + blockIdx.x) * 32 + u) * 2;
    par[0] = p0;
    par[1] = p1;
}

// ---- |M e|^2 --------------------------------------------------------------------------------------------------
// A wavefront keeps EF tiles of 32 entities in registers and its workgroup streams matrices past them, 32 outputs a chunk:
// rows of the product are outputs, columns (lanes) entities, so that the squares add up in the lane.  Three products of
// split operands (the low ones' own is left out).  Bound by the matrix cores and the LDS reads that feed them.
template <int KS, int EF>
__global__ __launch_bounds__(kThreads, KS == 16 ? 1 : 2) void k_rr_norms(RrArgs f, int slice)
{
    constexpr int CK = 2 * KS, NB = 3, LW = CK / 4;        // kilobytes of a chunk, chunks in LDS, a wavefront's loads
    __shared__ __align__(1024) uint4 s_ring[NB][CK][64];
    const int lane = threadIdx.x & 63, half = lane >> 5, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if (f.st->skip) return;
    const int tiles = (f.n_ent + 31) / 32, kt = f.k / 32;
    const int s0 = (int)blockIdx.y * slice, s1 = min(s0 + slice, f.slots), chunks = (s1 - s0) * kt;
    const int et = ((int)blockIdx.x * 4 + wave) * EF;
    half8 eh[EF][KS], el[EF][KS];
    float inv[EF];
#pragma unroll
    for (int q = 0; q < EF; ++q) {
        const int t = min(et + q, tiles - 1);
        const uint4 *p = f.es + (int64_t)t * KS * 128 + lane;
#pragma unroll
        for (int i = 0; i < KS; ++i) {
            eh[q][i] = __builtin_bit_cast(half8, p[i * 128]);
            el[q][i] = __builtin_bit_cast(half8, p[i * 128 + 64]);
        }
        const float sp = f.eaux[(int64_t)t * kAux + 4];
        inv[q] = 1.f / (sp * sp);
    }
    // (they arrive here: waited for inside the loop they would hold up the chunks ahead, which the compiler does not count)
#pragma unroll
    for (int q = 0; q < EF; ++q) {
        asm volatile("" : "+v"(inv[q]));
#pragma unroll
        for (int i = 0; i < KS; ++i) asm volatile("" : "+v"(eh[q][i]), "+v"(el[q][i]));
    }
    const uint4 *src = f.ms + (int64_t)s0 * kt * KS * 128 + wave * LW * 64 + lane;
    const uint32_t ring = lds_at(&s_ring[0][0][0]);
    auto fetch = [&](int c, int slot) {                    // (past the end: the last chunk once more)
        const uint4 *g = src + (int64_t)min(c, chunks - 1) * CK * 64;
#pragma unroll
        for (int i = 0; i < LW; ++i) load_lds_1k(g + i * 64, ring + (uint32_t)((slot * CK + wave * LW + i) * 1024));
    };
#pragma unroll
    for (int c = 0; c < NB - 1; ++c) fetch(c, c);
    const STX_CONST_AS float *maux = (const STX_CONST_AS float *)(f.maux + (int64_t)s0 * kt);
    int c = 0;
    for (int s = s0; s < s1; ++s) {
        float sum[EF];
#pragma unroll
        for (int q = 0; q < EF; ++q) sum[q] = 0.f;
        for (int a = 0; a < kt; ++a, ++c) {
            const float scale = maux[c];
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"((NB - 2) * LW) : "memory");
            __builtin_amdgcn_sched_barrier(0);
            fetch(c + NB - 1, (c + NB - 1) % NB);
            const uint4 (*chunk)[64] = s_ring[c % NB];
            floatx16 acc[EF];
#pragma unroll
            for (int q = 0; q < EF; ++q)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[q][i] = 0.f;
#pragma unroll
            for (int i = 0; i < KS; ++i) {
                const half8 mh = __builtin_bit_cast(half8, chunk[2 * i][lane]), ml = __builtin_bit_cast(half8, chunk[2 * i + 1][lane]);
#pragma unroll
                for (int q = 0; q < EF; ++q) {
                    acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_f16(mh, el[q][i], acc[q], 0, 0, 0);
                    acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ml, eh[q][i], acc[q], 0, 0, 0);
                    acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_f16(mh, eh[q][i], acc[q], 0, 0, 0);
                }
            }
#pragma unroll
            for (int q = 0; q < EF; ++q) {
                float x = 0.f;
#pragma unroll
                for (int i = 0; i < 16; ++i) x = __builtin_fmaf(acc[q][i], acc[q][i], x);
                sum[q] = __builtin_fmaf(x, scale, sum[q]);
            }
        }
#pragma unroll
        for (int q = 0; q < EF; ++q) {
            if (et + q >= tiles) continue;
            const float n = (sum[q] + __shfl_xor(sum[q], 32, 64)) * inv[q];
            const bool in = (et + q) * 32 + (lane & 31) < f.n_ent;
            float mx = in ? (n < 1e30f ? n : __builtin_inff()) : 0.f;          // (NaN too)
#pragma unroll
            for (int m = 16; m >= 1; m >>= 1) mx = fmaxf(mx, __shfl_xor(mx, m, 32));
            float *out = f.nn + ((int64_t)s * tiles + et + q) * kAux;
            // past the table's end: never below
            __builtin_nontemporal_store(half ? sqrtf(mx) * 1.001f : in ? n : 3e37f, out + lane);
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" : : : "memory");     // (loads into LDS still in flight must not outlive the workgroup)
}

// ---- sweep ----------------------------------------------------------------------------------------------------
// As k_rank_wide, with a relation's |M e|^2 beside the candidates: the stream of candidates is shared by the workgroup's
// four blocks of queries, and every wavefront fetches its own relation's numbers along.  A wavefront's undecided pairs are
// of one relation and leave in blocks for k_rr_pairs.
template <int KS>
__global__ __launch_bounds__(kThreads, KS <= 4 ? 1 : 2) void k_rr_sweep(RrArgs f, int slice)
{
    constexpr int TPC = KS >= 12 ? 1 : KS >= 6 ? 2 : 16 / KS, CK = TPC * KS, NB = 4, LW = CK / 4, LA = TPC > 4 ? TPC / 4 : 1;
    static_assert(CK % 4 == 0, "whole chunks");
    constexpr int S = KS / 2;                              // steps of 32 elements, two kilobytes each
    __shared__ __align__(1024) uint4 s_ring[NB][CK][64];
    __shared__ __align__(256) float s_aux[NB][TPC][kAux];
    __shared__ __align__(256) float s_nn[NB][4][TPC][kAux];
    __shared__ uint2 s_list[4][2 * kPairBlock];
    const int lane = threadIdx.x & 63, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int b = f.b0 + (int)blockIdx.x * 4 + wave;
    const bool works = b < f.b1;                           // (the others only fetch)
    const RrBlock blk = f.blocks[works ? b : f.b0];
    const int32_t skip = f.st->skip;
    const int tiles = (f.n_ent + 31) / 32;
    const int t0 = (int)blockIdx.y * slice, t1 = min(t0 + slice, tiles), chunks = (t1 - t0 + TPC - 1) / TPC;
    intx4 qh[S], ql[S];
    {
        const uint4 *qs = f.qf + (int64_t)(works ? b : f.b0) * KS * 64 + lane;
#pragma unroll
        for (int i = 0; i < S; ++i) {
            qh[i] = __builtin_bit_cast(intx4, qs[i * 128]);
            ql[i] = __builtin_bit_cast(intx4, qs[i * 128 + 64]);
        }
    }
    const float4 *par = f.qpar + ((int64_t)(works ? b : f.b0) * 32 + (lane & 31)) * 2;
    float4 p0 = par[0], p1 = par[1];
    // (they arrive here: see k_rr_norms)
#pragma unroll
    for (int i = 0; i < S; ++i) asm volatile("" : "+v"(qh[i]), "+v"(ql[i]));
    asm volatile("" : "+v"(p0.x), "+v"(p0.y), "+v"(p0.z), "+v"(p0.w), "+v"(p1.x), "+v"(p1.y), "+v"(p1.z));
    const int slot = __builtin_amdgcn_readfirstlane(blk.slot) - f.slot0, rel = __builtin_amdgcn_readfirstlane(blk.rel);
    const int first = __builtin_amdgcn_readfirstlane(blk.first), count = __builtin_amdgcn_readfirstlane(blk.count);
    const uint4 *src = f.ew + (int64_t)t0 * KS * 64 + wave * LW * 64 + lane;
    const float *aux = f.eaux + (int64_t)t0 * kAux + lane, *nn = f.nn + ((int64_t)slot * tiles + t0) * kAux + lane;
    const uint32_t ring = lds_at(&s_ring[0][0][0]), ring_aux = lds_at(&s_aux[0][0][0]), ring_nn = lds_at(&s_nn[0][0][0][0]);
    const int last = t1 - t0 - 1;
    auto fetch = [&](int c, int at) {                      // (past the end: the last chunk or tile once more)
        const uint4 *g = src + (int64_t)min(c, chunks - 1) * CK * 64;
#pragma unroll
        for (int i = 0; i < LW; ++i) load_lds_1k(g + i * 64, ring + (uint32_t)((at * CK + wave * LW + i) * 1024));
#pragma unroll
        for (int i = 0; i < LA; ++i) {
            const int tile = (wave + 4 * i) % TPC;
            load_lds_256(aux + (int64_t)min(c * TPC + tile, last) * kAux, ring_aux + (uint32_t)((at * TPC + tile) * kAux * 4));
        }
#pragma unroll
        for (int i = 0; i < TPC; ++i)
            load_lds_256(nn + (int64_t)min(c * TPC + i, last) * kAux, ring_nn + (uint32_t)(((at * 4 + wave) * TPC + i) * kAux * 4));
    };
    int less = 0, cnt = 0;
    bool listing = true;                                   // until there are too many undecided pairs
    auto flush = [&] {
        int at = 0;
        if (lane == 0) {
            at = (int)min(atomicAdd(&f.st->n_blocks, 1u), (uint32_t)f.pair_blocks);
            if (at == f.pair_blocks) __hip_atomic_store(&f.st->full, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            else f.heads[at] = make_int2(rel, min(cnt, kPairBlock));
        }
        at = __builtin_amdgcn_readfirstlane(at);
        if (at == f.pair_blocks) listing = false;
        else if (lane < cnt) f.pairs[(int64_t)at * kPairBlock + lane] = s_list[wave][lane];
        cnt -= kPairBlock;
        if (lane < cnt) s_list[wave][lane] = s_list[wave][kPairBlock + lane];
    };
#pragma unroll
    for (int c = 0; c < NB - 1; ++c) fetch(c, c);
    if (skip) {
        asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
        return;
    }
    const float half_k = (0.25f * (float)f.k + 16.f) * kUnit;
    for (int c = 0; c < chunks; ++c) {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"((NB - 2) * (LW + LA + TPC)) : "memory");
        __builtin_amdgcn_sched_barrier(0);
        fetch(c + NB - 1, (c + NB - 1) % NB);
        if (!works) continue;
#pragma unroll 1
        for (int tt = 0; tt < TPC; ++tt) {
            const int t = t0 + c * TPC + tt;
            if (t >= t1) break;
            const uint4 (*tile)[64] = s_ring[c % NB] + tt * KS;
            const float *tn = s_nn[c % NB][wave][tt];
            const float4 ea = ld4(s_aux[c % NB][tt]);      // scale, largest norm, rounding, low bytes
            intx16 hh, mid;
#pragma unroll
            for (int i = 0; i < 16; ++i) hh[i] = mid[i] = 0;
#pragma unroll
            for (int i = 0; i < S; ++i) {
                const intx4 eh = __builtin_bit_cast(intx4, tile[2 * i][lane]), el = __builtin_bit_cast(intx4, tile[2 * i + 1][lane]);
                hh = __builtin_amdgcn_mfma_i32_32x32x32_i8(eh, qh[i], hh, 0, 0, 0);
                mid = __builtin_amdgcn_mfma_i32_32x32x32_i8(el, qh[i], mid, 0, 0, 0);
                mid = __builtin_amdgcn_mfma_i32_32x32x32_i8(eh, ql[i], mid, 0, 0, 0);
            }
            const float pm = tn[32], sse = p1.x * ea.x, eps = p1.z * (ea.y / ea.x);
            float w = __builtin_fmaf(p0.x, ea.y, __builtin_fmaf(p0.y, ea.z, __builtin_fmaf(p0.w, ea.x, p1.y * ea.w)));
            w = __builtin_fmaf(sse, __builtin_fmaf(eps, pm + eps, half_k * (pm * pm)), w);
            w = __builtin_fmaf(w, 1.0001f, 1e-37f);        // (never zero: exact ties are undecided)
            const float tau = p0.z * ea.x, hs = 0.5f * sse;
            uint32_t neg = 0, near = 0;                    // signs of t and of |t| - w
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const float4 n4 = ld4(tn + 8 * g + 4 * half);
                const float nv[4] = {n4.x, n4.y, n4.z, n4.w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    // (at most 256 steps of up to 127 127 256 and twice 127 128: below 2^31)
                    const float v = (float)(hh[4 * g + i] * 256 + mid[4 * g + i]) - __builtin_fmaf(nv[i], hs, tau);
                    neg = __builtin_amdgcn_alignbit(neg, __float_as_uint(v), 31);
                    near = __builtin_amdgcn_alignbit(near, __float_as_uint(fabsf(v) - w), 31);
                }
            }
            if (!(w < 1e37f)) near = 0xffffu;              // no bound: nothing is decided
            less += 16 - __builtin_popcount(neg | near);
            uint32_t und = near << 16;                     // the lane's undecided sums: bit 31 - i
            while (__any(und != 0) && listing) {
                const int i = __builtin_clz(und | 1u);
                const int e = t * 32 + (i & 3) + 8 * ((i >> 2) & 3) + 4 * half, q = lane & 31;
                const bool mine = und != 0 && e < f.n_ent && q < count;
                const uint64_t m = __ballot(mine);
                und &= ~(0x80000000u >> i);
                if (mine) s_list[wave][cnt + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] =
                    make_uint2((uint32_t)e, (uint32_t)(first + q));
                cnt += __builtin_popcountll(m);
                if (cnt >= kPairBlock) flush();
            }
        }
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" : : : "memory");   // (loads into LDS still in flight must not outlive the workgroup)
    if (!works) return;
    if (cnt > 0 && listing) flush();
    const int n = less + __shfl_xor(less, 32, 64);
    if (lane < count && n) atomicAdd(&f.gless[first + lane], n);
}

// ---- exact pairs ----------------------------------------------------------------------------------------------
// A block of undecided pairs at a time: their entities are projected together, then a thread walks each pair's sum.  Bound by
// the fp32 matrix cores.  Where the sweep stopped, what it counted is cleared instead, for k_rr_behind.
template <int A>
__global__ __launch_bounds__(kThreads, A == 1 ? 4 : 2) void k_rr_pairs(RrArgs f)
{
    extern __shared__ __align__(16) unsigned char s_dyn[];
    __shared__ int32_t s_id[kPairBlock];
    const int tid = threadIdx.x, k = f.k;
    if (f.st->full) {
        for (int b = f.b0 + (int)blockIdx.x * 8 + (tid >> 5); b < f.b1; b += (int)gridDim.x * 8) {
            const RrBlock blk = f.blocks[b];
            if ((tid & 31) < blk.count) f.gless[blk.first + (tid & 31)] = f.gequal[blk.first + (tid & 31)] = 0;
        }
        return;
    }
    float *s_p = reinterpret_cast<float *>(s_dyn);
    const int n = (int)min(f.st->n_blocks, (uint32_t)f.pair_blocks);
    for (int b = blockIdx.x; b < n; b += gridDim.x) {
        const int2 head = f.heads[b];
        const uint2 pr = f.pairs[(int64_t)b * kPairBlock + min(tid & (kPairBlock - 1), head.y - 1)];
        __syncthreads();                                   // (the block before this one has been walked)
        if (tid < kPairBlock) s_id[tid] = (int32_t)pr.x;
        __syncthreads();
        floatx16 acc[A][2];
        rr_project<A>(f, head.x, s_id, s_p, acc);
        rr_spread<A>(f, acc, s_p);
        if (tid < head.y) {
            const float *q = f.q32 + (int64_t)pr.y * k;
            const float st = f.gts[pr.y];
            float s = 0.f;
            for (int a = 0; a < k; a += 8) {
                const float4 x = ld4(q + a), y = ld4(q + a + 4);
                const float v[8] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
#pragma unroll
                for (int i = 0; i < 8; ++i) s = rank_step<STX_L2>(s, v[i] - s_p[(a + i) * kLdP + tid]);
            }
            rank_count<4>(f.gless, f.gequal, pr.y, s < st, s == st);
        }
    }
}

// All pairs of the sweep's queries, where it stopped: 64 entities of a relation are projected at a time and every thread
// walks the sums of one against the relation's queries.
template <int A>
__global__ __launch_bounds__(kThreads, A == 1 ? 4 : 2) void k_rr_behind(RrArgs f)
{
    if (!f.st->full) return;
    extern __shared__ __align__(16) unsigned char s_dyn[];
    __shared__ int32_t s_id[64];
    float *s_p = reinterpret_cast<float *>(s_dyn);
    constexpr int LD = kLdP;
    const int tid = threadIdx.x, k = f.k, row = tid & 63;
    const int part = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int e = (int)blockIdx.x * 64 + row;
    if (tid < 64) s_id[tid] = min(e, f.n_ent - 1);
    for (int b = f.b0 + (int)blockIdx.y; b < f.b1;) {      // (a relation's blocks follow one another; the first to see it takes them)
        const RrBlock blk = f.blocks[b];
        const int rel = __builtin_amdgcn_readfirstlane(blk.rel);
        if (b > f.b0 && f.blocks[b - 1].rel == rel) { b += (int)gridDim.y; continue; }
        int e_b = b + 1;
        while (e_b < f.b1 && f.blocks[e_b].rel == rel) ++e_b;
        const int q0 = __builtin_amdgcn_readfirstlane(blk.first), q1 = __builtin_amdgcn_readfirstlane(f.blocks[e_b - 1].first + f.blocks[e_b - 1].count);
        __syncthreads();
        floatx16 acc[A][2];
        rr_project<A>(f, rel, s_id, s_p, acc);
        rr_spread<A>(f, acc, s_p);
        for (int q = q0 + part * 4; q < q1; q += 16) {      // four queries a wavefront at a time, their points through scalar loads
            float s[4] = {0.f, 0.f, 0.f, 0.f};
            const STX_CONST_AS float *qp[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) qp[i] = (const STX_CONST_AS float *)(f.q32 + (int64_t)min(q + i, q1 - 1) * k);
            for (int a = 0; a < k; a += 4)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float p = s_p[(a + j) * LD + row];
#pragma unroll
                    for (int i = 0; i < 4; ++i) s[i] = rank_step<STX_L2>(s[i], qp[i][a + j] - p);
                }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (q + i >= q1) break;
                const float st = f.gts[q + i];
                const int nl = __builtin_popcountll(__ballot(e < f.n_ent && s[i] < st)), ne = __builtin_popcountll(__ballot(e < f.n_ent && s[i] == st));
                if ((tid & 63) == 0) {
                    if (nl) atomicAdd(&f.gless[q + i], nl);
                    if (ne) atomicAdd(&f.gequal[q + i], ne);
                }
            }
        }
        b += (int)gridDim.y;
    }
}

// ---- host -----------------------------------------------------------------------------------------------------
// 16-element steps of a row: the compiled counts, the rest is padded with zeros.
static int rr_steps(int dim)
{
    static const int kSteps[] = {2, 4, 6, 8, 12, 16};
    for (int s : kSteps)
        if (16 * s >= dim) return s;
    return 16;
}
struct RrPlan {
    size_t q32, qf, qpar, ew, eaux, es, ms, maux, nn, pairs, heads, state, total;
    int64_t max_blocks, slots, pair_blocks;
};
static RrPlan rr_plan(const stx_config &cfg, int64_t nq)
{
    const int ks = rr_steps(cfg.dim);
    const int64_t tiles = (cfg.n_ent + 31) / 32, occ = std::min((int64_t)cfg.n_rel, nq);
    RrPlan p{};
    size_t off = 0;
    auto take = [&](size_t bytes) { const size_t o = off; off = (off + bytes + 255) / 256 * 256; return o; };
    p.max_blocks = nq / 32 + occ;
    // relations in batches of at most 96 MiB of operands and |M e|^2
    const int64_t slot_bytes = (int64_t)(cfg.rel_dim / 32) * (ks * 2048 + 4) + tiles * kAux * 4;
    p.slots = std::max((int64_t)1, std::min(occ, ((int64_t)96 << 20) / slot_bytes));
    // undecided pairs: room for one in 128 of the pairs and the blocks that wavefronts leave partly filled, 64 MiB at most
    const int64_t blocks = (int64_t)((double)nq * (double)cfg.n_ent / (128. * kPairBlock)) + p.max_blocks * 2 + 5120;
    p.pair_blocks = std::min(blocks, ((int64_t)64 << 20) / (kPairBlock * (int64_t)sizeof(uint2)));
    p.q32 = take((size_t)nq * cfg.rel_dim * 4);
    p.qf = take((size_t)p.max_blocks * ks * 1024);
    p.qpar = take((size_t)p.max_blocks * 32 * 32);
    p.ew = take((size_t)(tiles + 16) * ks * 1024);         // (reads past the last tile)
    p.eaux = take((size_t)tiles * kAux * 4);
    p.es = take((size_t)tiles * ks * 2048);
    p.ms = take((size_t)p.slots * (cfg.rel_dim / 32) * ks * 2048);
    p.maux = take((size_t)p.slots * (cfg.rel_dim / 32) * 4);
    p.nn = take((size_t)p.slots * tiles * kAux * 4);
    p.pairs = take((size_t)p.pair_blocks * kPairBlock * sizeof(uint2));
    p.heads = take((size_t)p.pair_blocks * sizeof(int2));
    p.state = take(sizeof(RrState));
    p.total = off;
    return p;
}
template <int KS, int A>
static void rr_go(stx_ctx *c, RrArgs f, const RrPlan &p, const int32_t *counts, int32_t n_rel, int32_t most)
{
    const int tiles = (f.n_ent + 31) / 32, kt = f.k / 32;
    const size_t lds_q = rr_query_lds(f.dim, f.k), lds_x = rr_exact_lds(f.k);
    // (more than 64 KB of LDS has to be asked for, on every device that runs the kernels)
    auto lds_limit = [](const void *k, size_t bytes) { (void)hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes); };
    if (f.head) lds_limit(reinterpret_cast<const void *>(&k_rr_query<KS, A, true>), lds_q);
    else lds_limit(reinterpret_cast<const void *>(&k_rr_query<KS, A, false>), lds_q);
    lds_limit(reinterpret_cast<const void *>(&k_rr_pairs<A>), lds_x);
    lds_limit(reinterpret_cast<const void *>(&k_rr_behind<A>), lds_x);
    constexpr int EF = KS <= 8 ? 2 : 1;
    // a sweep covers at most as many pairs as one undecided in 200 of them, in blocks two thirds full, has places for
    const double span = (double)p.pair_blocks * kPairBlock * (2. / 3.) * 200.;
    const int per_sweep = (int)std::max(4., std::min(span / f.n_ent / 32., 1e9));
    int32_t r = 0, slot = 0, block = 0;
    f.first = 1;
    while (r < n_rel) {
        f.slot0 = slot;
        const int32_t b_begin = block;
        for (; r < n_rel && slot - f.slot0 < p.slots; ++r)
            if (counts[r] && counts[r] <= most) { ++slot; block += (counts[r] + 31) / 32; }
        if (slot == f.slot0) break;
        f.slots = slot - f.slot0;
        const int etiles = f.first ? tiles : 0;
        {
            ProfScope prof(c, "k_rr_pack");
            hipLaunchKernelGGL((k_rr_pack<KS>), dim3((unsigned)(etiles + f.slots * kt)), dim3(kThreads), 0, c->stream, f, etiles);
        }
        for (f.b0 = b_begin; f.b0 < block; f.b0 = f.b1) {
            f.b1 = block - f.b0 > per_sweep ? f.b0 + per_sweep : block;
            const int nb = f.b1 - f.b0;
            {
                ProfScope prof(c, "k_rr_query");
                if (f.head) hipLaunchKernelGGL((k_rr_query<KS, A, true>), dim3((unsigned)nb), dim3(kThreads), lds_q, c->stream, f);
                else hipLaunchKernelGGL((k_rr_query<KS, A, false>), dim3((unsigned)nb), dim3(kThreads), lds_q, c->stream, f);
            }
            if (f.b0 == b_begin) {
                const int64_t gx = (tiles + 4 * EF - 1) / (4 * EF), want = std::max((int64_t)1, (1024 + gx - 1) / gx);
                const int slice = (int)((f.slots + want - 1) / want);
                ProfScope prof(c, "k_rr_norms");
                hipLaunchKernelGGL((k_rr_norms<KS, EF>), dim3((unsigned)gx, (unsigned)((f.slots + slice - 1) / slice)), dim3(kThreads), 0,
                                   c->stream, f, slice);
            }
            {
                // Two rounds of the workgroups that fit the chip; 32 tiles each at least, as a wavefront's last pairs take a block of
                // their own (50 queries x 200,000 at d = 256 in slices of eight: 3,128 blocks for 20,000 pairs)
                const int64_t gx = (nb + 3) / 4, want = std::max((int64_t)1, (1024 + gx - 1) / gx);
                const int slice = (int)std::max((int64_t)32, (tiles + want - 1) / want);
                ProfScope prof(c, "k_rr_sweep");
                hipLaunchKernelGGL((k_rr_sweep<KS>), dim3((unsigned)gx, (unsigned)((tiles + slice - 1) / slice)), dim3(kThreads), 0,
                                   c->stream, f, slice);
            }
            {
                ProfScope prof(c, "k_rank_pairs");
                const int64_t most = (int64_t)nb * 32 * f.n_ent / (kPairBlock * 128) + 64;
                hipLaunchKernelGGL((k_rr_pairs<A>), dim3((unsigned)std::min(most, (int64_t)(A == 1 ? 1024 : 512))), dim3(kThreads), lds_x, c->stream, f);
            }
            {
                ProfScope prof(c, "k_rr_behind");
                hipLaunchKernelGGL((k_rr_behind<A>), dim3((unsigned)((f.n_ent + 63) / 64), (unsigned)std::min(nb, 16)), dim3(kThreads), lds_x, c->stream, f);
            }
            f.first = 0;
        }
    }
}

// The rule between this and projected tables, in us as measured at 50 sizes (1,000 to 200,000 entities, widths of 32 to 256,
// 1 to 1,350 relations, 1 to 59,071 queries): what a relation costs as a table, projected and packed, or as |M e|^2; what a
// query costs more without a table (more pairs are undecided, and they are dearer); launches and dependent passes.
// One relation, 20,000 queries x 14,500 entities, d = k = 128: 697 us with a table, 1,043 without; 237 relations: 5,222 and
// 1,674; 4 queries of 4 relations x 9,028 at 96 x 256: 239 and 308, at 133,311 entities: 579 and 353.
static double rr_table_us(const stx_config &c) { return (double)c.n_ent * c.rel_dim * (2. * c.dim / 90e6 + 10. / 5e6); }
static double rr_norms_us(const stx_config &c) { return (double)c.n_ent * c.rel_dim * 16. * rr_steps(c.dim) * 6. / 500e6; }
static double rr_query_us(const stx_config &c) { return 0.0008 + 0.4 * (double)c.n_ent / 500. * c.dim * c.rel_dim * 2. / 65e6; }
static double rr_fixed_us(const stx_config &c) { return 55. + 0.0008 * c.dim * c.rel_dim + (double)c.n_ent * c.dim * 10. / 4e6; }
constexpr double kRrLaunchUs = 28.;    // of a set of launches over projected tables
int32_t rank_transr_most(const stx_config &c)
{
    const double most = (kRrLaunchUs + rr_table_us(c) - rr_norms_us(c)) / rr_query_us(c);
    return (int32_t)std::max(0., std::min(most, 2e9));
}
// No scratch where the rule cannot come out on this side, whatever the relations of the queries: as many of them as there
// can be, one query each and the most launches.  (Such calls do not list blocks of queries either: k_rr_scan takes 2.3 us
// without, 4.0 with it, of calls of 80.)
size_t rank_transr_bytes(const stx_config &cfg, int64_t nq, int tables)
{
    if ((cfg.dist != STX_L2 && cfg.dist != STX_L2_SQ) || rank_transr_most(cfg) == 0) return 0;
    const double rels = (double)std::min((int64_t)cfg.n_rel, nq), big = std::min(rels, floor((double)nq / (kRankBig + 1)));
    const double gain = (big + ceil(rels / tables)) * kRrLaunchUs +
                        std::max(0., rels * (rr_table_us(cfg) - rr_norms_us(cfg) - rr_query_us(cfg))) - rr_fixed_us(cfg);
    return gain > 0. ? rr_plan(cfg, nq).total : 0;
}

bool rank_transr(stx_ctx *c, const stx_params *p, int64_t nq, int side, const RankGroups &g, int tables, void *work, size_t bytes, const int32_t *counts)
{
    const RrPlan pl = rr_plan(c->cfg, nq);
    double rels = 0., queries = 0., big = 0.;
    for (int64_t r = 0; r < c->cfg.n_rel; ++r)
        if (counts[r] && counts[r] <= g.most) {
            rels += 1.;
            queries += counts[r];
            big += counts[r] > kRankBig ? 1. : 0.;         // (launches of its own)
        }
    const double with_tables = (big + ceil((rels - big) / tables)) * kRrLaunchUs + rels * rr_table_us(c->cfg);
    const double without = rr_fixed_us(c->cfg) + rels * rr_norms_us(c->cfg) + queries * rr_query_us(c->cfg);
    if (bytes < pl.total || without >= with_tables) return false;
    char *w = (char *)work;
    RrArgs f{};
    f.E = p->ent; f.M = p->proj; f.R = p->rel;
    f.n_ent = (int32_t)c->cfg.n_ent; f.dim = c->cfg.dim; f.k = c->cfg.rel_dim;
    f.head = side;
    f.gh = g.h; f.gt = g.t; f.gts = g.score; f.gless = g.less; f.gequal = g.equal;
    f.blocks = (const RrBlock *)g.blocks; f.occ = g.occ;
    f.q32 = (float *)(w + pl.q32); f.qf = (uint4 *)(w + pl.qf); f.qpar = (float4 *)(w + pl.qpar);
    f.ew = (uint4 *)(w + pl.ew); f.eaux = (float *)(w + pl.eaux); f.es = (uint4 *)(w + pl.es); f.ms = (uint4 *)(w + pl.ms);
    f.maux = (float *)(w + pl.maux); f.nn = (float *)(w + pl.nn);
    f.pairs = (uint2 *)(w + pl.pairs); f.heads = (int2 *)(w + pl.heads); f.pair_blocks = (int32_t)pl.pair_blocks;
    f.st = (RrState *)(w + pl.state);
    const bool two = c->cfg.rel_dim > 128;
#define STX_RR(KS)                                                                                              \
    case KS: if (two) rr_go<KS, 2>(c, f, pl, counts, (int32_t)c->cfg.n_rel, g.most); else rr_go<KS, 1>(c, f, pl, counts, (int32_t)c->cfg.n_rel, g.most); break
    switch (rr_steps(c->cfg.dim)) {
        STX_RR(2);
        STX_RR(4);
        STX_RR(6);
        STX_RR(8);
        STX_RR(12);
        STX_RR(16);
    }
#undef STX_RR
    return true;
}

}  // namespace stx
