// Link prediction through a filter: most candidates are ordered against the true entity by a cheap sum of known
// error, and only those too close to it are summed exactly.
//
// The counts of stx_rank are defined by the fp32 sums of k_rank (index order, every step rounded as written there),
// so they must come out as if every candidate had been summed that way.  A sum S' with a bound |S' - S| <= W on its
// distance from the exact-order sum S decides the candidate whenever |S' - S_true| > W; with W about a thousandth of
// the spread of the scores, one candidate in about a thousand is left, and those are recomputed in index order.  So the
// result is that of the exhaustive fp32 sweep, bit for bit.  Wherever a bound is not finite (values out of range, infinities, NaN) the
// candidate counts as undecided.
//
// Undecided pairs go to a list that k_rank_pairs works through; when it is full they are summed inside the sweep, one per
// lane, at 20 to 130 times what a pair costs the plain sweep.  How many there are depends on the values: a sweep that
// finds more than that can pay for (many equal rows, rows far outside the others' range) stops, and the plain sweep, which
// is always launched behind it and otherwise returns at once, does the whole chunk.  59,071 queries x 15,000 equal rows at
// d = 128 (L1) took 180 ms a side without that; the plain sweep takes 4.2.
//
// The plain sweep's rate is that of the vector ALU (two fp32 operations per element, five for the torus kind):
// 59,071 queries x 15,000 entities at d = 128 (L1) took 3.85 ms a side and take 1.95; 256 x 4,000,000 (torus-L1) 10.2
// and 4.2; 4,096 x 14,951 at d = 1024 (L2) 2.7 and 0.41.
//
//   L1, torus-L1   k_rank_sad: rows as 16-bit fixed point, two elements per vector operation (v_sad_u16 sums two
//                  absolute differences; the torus kind wraps the difference by a 32-bit subtraction first).  The
//                  bound is the sum of the roundings actually made in each row.
//   L2, squared L2 k_rank_mfma: S = |q|^2 + |e|^2 - 2 q.e with q.e on the matrix cores, rows rounded to fp16 after
//                  scaling by a power of two.  The bound is |q| |de| + |dq| |e| with the norms of the roundings made.
//                  Rows of more than 256 floats: k_rank_wide, the same with 16-bit fixed point in two bytes.
#include <algorithm>

#include "stx_rank.h"

namespace stx {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int kSadGroup = 16;          // queries per group of k_rank_sad: one accumulator each
constexpr int kSadThreads = 512;
constexpr int kNoQuery = -(1 << 30);   // threshold of the places past the last query
constexpr int kListCap = 128;          // undecided pairs a wavefront collects before it recomputes them

struct FilterState {
    unsigned long long n_pairs;        // undecided pairs found (a sweep may find up to 2^31 x 2^31), cleared by k_rank_prep
    int32_t pad[30];                   // (the wavefronts that read the rest do not wait for those that count)
    int32_t full;                      // there were too many, in this sweep or one before it in the call
    int32_t skip;                      // `full` as it was before this sweep, the same for all of its wavefronts
};
struct FilterArgs {
    RankArgs a;
    int32_t q_first;                   // first query of this chunk (relations: 0)
    int32_t q_cap;                     // queries per chunk and blockIdx.z, a multiple of 32
    int32_t e_first, e_count;          // segment of candidates
    int np;                            // 8-element pieces of a row: 2 per matrix-core step, the last may be padding
    int nqb;                           // k_rank_prep: blocks (of 32) that prepare queries; the rest prepare candidates
    float *q32;                        // [query]: its point, fp32
    uint32_t *qt;                      // fixed point: [group][piece][dword][16 queries], two elements per dword
    int2 *thr;                         // ... [query]: (sum below which a candidate is surely below, ... surely above)
    float *scale;                      // ... [1]
    uint4 *qf, *ef;                    // matrix cores: operand fragments [tile of 32 rows][step][lane]
    float4 *qpar;                      // ... [query]: bound factors and threshold, see k_rank_prep
    float *qscale;                     // ... [query]
    float *qlow;                       // ... [query], wide rows: norm of the low bytes
    float *eaux;                       // ... [tile of 32][64]: half the candidates' squared norms, scaled; then, from 32 on,
                                       //     the tile's scale, largest norm, largest rounding, squared-norm term; wide rows:
                                       //     largest norm of the low bytes
    int32_t slice;                     // sweeps: candidates (mfma) or query groups (sad) per blockIdx.y
    int head;                          // side: q = t - r instead of h + r
    FilterState *st;
    int32_t first;                     // the first sweep of the call, and its k_rank_prep
    int32_t tables;                    // relations of a TransR launch, else 1
    uint2 *pairs;                      // undecided pairs: (candidate | table << z_shift, position in the query arrays)
    int32_t pair_cap;                  // places of the list
    unsigned long long pair_limit;     // undecided pairs beyond which the sweep stops
    int z_shift;                       // 32: one table
};

// Lane `lane`'s place among the set bits of a wavefront mask.
__device__ inline int mask_rank(uint64_t m)
{
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// ---- exact treatment of undecided pairs -------------------------------------------------------------------
struct PairRows {
    const float *pq, *pe;
    uint32_t e;
    int64_t q;
    float st;
};
__device__ inline PairRows pair_rows(const FilterArgs &f, uint2 pr)
{
    RankArgs a = f.a;
    uint32_t e = pr.x;
    if (f.z_shift < 32) {
        a.X += (int64_t)(e >> f.z_shift) * a.table_stride;
        e &= (1u << f.z_shift) - 1u;
    }
    PairRows p;
    p.e = e;
    p.q = pr.y;
    p.pq = f.q32 + (p.q - f.q_first) * a.dim;
    p.pe = a.X + (int64_t)e * a.dim;
    p.st = a.true_score[p.q];
    return p;
}
// One term's difference as k_rank forms it (the factor +-1 is exact).
__device__ inline float pair_diff(float sg, float qv, float ev) { return sg * (qv - ev); }

// The index-order sum of one pair per lane.
template <int DIST>
__device__ inline void pair_exact(const FilterArgs &f, uint2 pr)
{
    const PairRows p = pair_rows(f, pr);
    const float sg = f.head ? -1.f : 1.f;
    const int dim = f.a.dim;
    float acc = 0.f;
    for (int j0 = 0; j0 < dim; j0 += 16) {
        float4 vq[4], ve[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int j = min(j0 + 4 * u, dim - 4);
            vq[u] = ld4(p.pq + j); ve[u] = ld4(p.pe + j);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (j0 + 4 * u < dim) {
                acc = rank_step<DIST>(acc, pair_diff(sg, vq[u].x, ve[u].x));
                acc = rank_step<DIST>(acc, pair_diff(sg, vq[u].y, ve[u].y));
                acc = rank_step<DIST>(acc, pair_diff(sg, vq[u].z, ve[u].z));
                acc = rank_step<DIST>(acc, pair_diff(sg, vq[u].w, ve[u].w));
            }
    }
    rank_count<64>(f.a.n_less, f.a.n_equal, (uint32_t)p.q, acc < p.st, acc == p.st);
}

// Eight lanes per pair, the same sum (1: below the true entity's, 2: equal, else 0): a lane adds the four terms it holds of 32 to what the lane before it hands on.  Every
// lane goes through all eight turns and only one of them counts, which is five times the instructions of a sum in any
// order; but such a sum has a bound of its own, a thousandth of the pairs stay within it at d = 1024, and walking
// those one per lane behind the others took longer than all the rest (4,096 x 14,951 at d = 1024: 290 us a side, now 125).
template <int DIST>
__device__ inline int pair_ordered(const FilterArgs &f, uint2 pr, int lane)
{
    const PairRows p = pair_rows(f, pr);
    const float sg = f.head ? -1.f : 1.f;
    const int dim = f.a.dim;
    float acc = 0.f;                                       // (of the lane whose turn is next)
    for (int j0 = 0; j0 < dim; j0 += 128) {
        float4 vq[4], ve[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int j = min(j0 + 32 * u + (lane & 7) * 4, dim - 4);
            vq[u] = ld4(p.pq + j); ve[u] = ld4(p.pe + j);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int j = j0 + 32 * u;
            if (j >= dim) break;
            float y[4] = {pair_diff(sg, vq[u].x, ve[u].x), pair_diff(sg, vq[u].y, ve[u].y), pair_diff(sg, vq[u].z, ve[u].z), pair_diff(sg, vq[u].w, ve[u].w)};
            if (j + (lane & 7) * 4 >= dim) y[0] = y[1] = y[2] = y[3] = 0.f;   // (adds nothing)
            if (DIST != STX_L2) {
#pragma unroll
                for (int i = 0; i < 4; ++i) y[i] = rank_step<DIST>(0.f, y[i]);   // the term by itself
            }
#pragma unroll
            for (int turn = 0; turn < 8; ++turn) {
#pragma unroll
                for (int i = 0; i < 4; ++i) acc = DIST == STX_L2 ? __builtin_fmaf(y[i], y[i], acc) : acc + y[i];
                // to the next lane (row_shr:1), from the last to the first (row_shl:7)
                const int v = __float_as_int(acc);
                acc = __int_as_float(turn < 7 ? __builtin_amdgcn_update_dpp(v, v, 0x111, 0xf, 0xf, false) : __builtin_amdgcn_update_dpp(v, v, 0x107, 0xf, 0xf, false));
            }
        }
    }
    acc = __shfl(acc, 0, 8);
    return acc < p.st ? 1 : acc == p.st ? 2 : 0;
}

// All undecided pairs of a sweep, many wavefronts in flight: bound by the latency and the bytes of the rows it reads.
template <int DIST>
__global__ __launch_bounds__(kThreads) void k_rank_pairs(FilterArgs f, RankIds ids)
{
    if (f.st->full) {                                      // what the chunk's sweeps counted is not used
        const RankArgs &a = f.a;
        for (int z = 0; z < f.tables; ++z) {
            const int64_t q0 = a.grp_counts ? a.grp_offsets[ids.g[z]] : f.q_first;
            const int64_t nq = a.grp_counts ? a.grp_counts[ids.g[z]] : min(a.nq - f.q_first, (int64_t)f.q_cap);
            for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < nq; i += (int64_t)gridDim.x * kThreads)
                a.n_less[q0 + i] = a.n_equal[q0 + i] = 0;
        }
        return;
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = (int)min(f.st->n_pairs, (unsigned long long)f.pair_cap), step = (int)gridDim.x * 32;
    for (int i0 = ((int)blockIdx.x * 4 + wave) * 8; i0 < n;) {
        uint32_t q = 0u;                                   // eight turns' results, one a lane, are counted together
        int res = 0;
#pragma unroll 1
        for (int u = 0; u < 8 && i0 < n; ++u, i0 += step) {
            const int i = i0 + (lane >> 3);
            const uint2 pr = f.pairs[min(i, n - 1)];
            const int got = pair_ordered<DIST>(f, pr, lane);
            if ((lane & 7) == u) { q = pr.y; res = i < n ? got : 0; }
        }
        if (res) rank_count<4>(f.a.n_less, f.a.n_equal, q, res == 1, res == 2);
    }
}

// A wavefront's collected pairs move to the list of the sweep; when that is full they are treated here, one per lane.
// false: the sweep has found too many, nothing it counts is used any more.
template <int DIST>
__device__ inline bool flush_pairs(const FilterArgs &f, const uint2 *list, int cnt, int lane)
{
    int base = 0;                                          // first place, pair_cap: none left, beyond: stop
    if (lane == 0) {
        const unsigned long long n = atomicAdd(&f.st->n_pairs, (unsigned long long)cnt);
        base = n > f.pair_limit ? f.pair_cap + 1 : (int)min(n, (unsigned long long)f.pair_cap);
    }
    base = __builtin_amdgcn_readfirstlane(base);
    if (base > f.pair_cap) {
        if (lane == 0) __hip_atomic_store(&f.st->full, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return false;
    }
    for (int i = lane; i < cnt; i += 64) {
        if (i < f.pair_cap - base) f.pairs[base + i] = list[i];
        else pair_exact<DIST>(f, list[i]);
    }
    return true;
}
__device__ inline float max_group8(float v)
{
#pragma unroll
    for (int m = 4; m >= 1; m >>= 1) v = fmaxf(v, __shfl_xor(v, m, 8));
    return v;
}
// The power of two that brings `mx` to [64, 128); 1 for zero.  ok: mx lies where squares and products of rows stay
// far from the ends of the fp32 range (elsewhere the bounds below would not hold, and nothing is decided by them).
__device__ inline float pow2_scale(float mx, bool &ok)
{
    ok = mx == 0.f || (mx > 1e-12f && mx < 1e12f);
    if (!ok || mx == 0.f) return 1.f;
    return ldexpf(1.f, 6 - ilogbf(mx));
}
// Relative error of half a squared norm formed by eight lanes, and of the few roundings around it.
__device__ inline float norm_slack(int np) { return 0.5f * kUnit * (float)(np + 24); }
// Eight elements scaled and rounded to fp16; adds the squares of the scaled values and of the roundings.
__device__ inline uint4 half_piece(const float (&v)[8], float sc, float &n2, float &d2)
{
    half8 h;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const float x = v[i] * sc;                         // exact: sc is a power of two
        h[i] = (_Float16)x;
        const float d = x - (float)h[i];                   // exact
        n2 = __builtin_fmaf(x, x, n2);
        d2 = __builtin_fmaf(d, d, d2);
    }
    return __builtin_bit_cast(uint4, h);
}
// The scale that brings `mx` to kWideMax, as pow2_scale.
__device__ inline float wide_scale(float mx, bool &ok)
{
    ok = mx == 0.f || (mx > 1e-12f && mx < 1e12f);
    return ok && mx != 0.f ? kWideMax / mx : 1.f;
}
// One element as 16-bit fixed point; adds the rounding made (in units of the last place).
template <bool TORUS>
__device__ inline uint32_t fixed16(float v, float sc, bool upper_q, float &res)
{
    if (TORUS) {
        // the phase; a difference of unwrapped values as fp32 forms it is off by at most 2^-24 (|q| + |e|), the
        // fractional part itself by 2^-24.  The upper half of a query's dword loses the borrow of the lower half's
        // subtraction, 0 or 1 units: it is stored half a unit up and half a unit is added to its rounding.
        const float x = __builtin_amdgcn_fractf(v) * 65536.f + (upper_q ? 0.5f : 0.f);
        const float k = rintf(x);
        res += fabsf(x - k) + 0.02f + fabsf(v) * (65536.f * 1.01f * kUnit) + (upper_q ? 0.5f : 0.f);
        return (uint32_t)(int)k & 0xffffu;
    }
    const float k = fminf(fmaxf(rintf(v * sc), -32768.f), 32767.f);
    res += fabsf(__builtin_fmaf(v, sc, -k)) * 1.0001f;
    return (uint32_t)((int)k + 32768);
}

// ---- scale of the L1 kind ---------------------------------------------------------------------------------
// Up to 128 queries' points and true entities are looked at.  The largest element sets the range of the fixed-point numbers
// (elements beyond it are clamped; what that loses is part of their row's bound), but where few rows lie far outside the
// others' range, leaving those undecided costs less than the coarser steps of all: of the rows' largest elements the one
// is taken at which the share of rows beyond it, and of pairs that its steps leave undecided (about one in 2,000 where
// it is the median), add up to the least.  One workgroup.
template <bool HEAD>
__global__ __launch_bounds__(1024) void k_rank_scale(RankArgs a, float *scale)
{
    __shared__ float s_mx[128], s_med, s_best[2][2];
    const int u = (int)threadIdx.x >> 3, l8 = (int)threadIdx.x & 7;
    const int64_t q = a.nq <= 128 ? u % a.nq : (int64_t)u * (a.nq / 128);
    const RankRows rw = rank_rows<HEAD>(a, q);
    float mx = 0.f;
    for (int j = l8 * 4; j < a.dim; j += 32) {
        const float4 va = ld4(rw.pa + j), vr = ld4(rw.pr + j), ve = ld4(rw.ptrue + j);
        const float4 q4 = HEAD ? sub4(va, vr) : add4(va, vr);
        mx = fmaxf(fmaxf(fmaxf(mx, fabsf(q4.x)), fmaxf(fabsf(q4.y), fabsf(q4.z))), fabsf(q4.w));
        mx = fmaxf(fmaxf(fmaxf(mx, fabsf(ve.x)), fmaxf(fabsf(ve.y), fabsf(ve.z))), fabsf(ve.w));
    }
    mx = max_group8(mx);
    if (l8 == 0) s_mx[u] = mx;
    __syncthreads();
    const int me = (int)threadIdx.x;
    int above = 0, before = 0;
    if (me < 128) {
        mx = s_mx[me];
#pragma unroll 16
        for (int i = 0; i < 128; ++i) {
            const float o = s_mx[i];
            above += o > mx;
            before += o < mx || (o == mx && i < me);
        }
        if (before == 64) s_med = mx;
    }
    __syncthreads();
    if (me < 128) {
        const float med = s_med > 1e-12f ? s_med : mx;
        const bool usable = mx > 1e-12f && mx < 1e12f;
        float cost = usable ? (float)above * (1.f / 128.f) + 5e-4f * (mx / med) : __builtin_inff(), best = usable ? mx : 32767.f;
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) {
            const float oc = __shfl_xor(cost, m, 64), ob = __shfl_xor(best, m, 64);
            if (oc < cost) { cost = oc; best = ob; }
        }
        if ((me & 63) == 0) { s_best[me >> 6][0] = cost; s_best[me >> 6][1] = best; }
    }
    __syncthreads();
    if (me == 0) *scale = 32767.f / (s_best[1][0] < s_best[0][0] ? s_best[1][1] : s_best[0][1]);   // none usable: 1
}

// ---- preparation ------------------------------------------------------------------------------------------
// Blocks of 32 queries: the true entity's sum in index order (one lane per query walks the terms out of LDS), cleared
// counters, and the packed query with its thresholds.  Matrix-core kinds: further blocks of 32 candidates each.
// Eight threads per row.  Bound by the latency of its few dependent passes; the rows come from the caches.
template <int DIST, bool HEAD, bool WIDE = false>
__global__ __launch_bounds__(kThreads) void k_rank_prep(FilterArgs f, RankIds ids)
{
    constexpr bool SAD = DIST == STX_L1 || DIST == STX_TORUS_L1, TORUS = DIST == STX_TORUS_L1;
    RankArgs a = f.a;
    if (blockIdx.x == 0 && blockIdx.z == 0 && threadIdx.x == 0) {
        const int32_t full = f.first ? 0 : f.st->full;
        f.st->n_pairs = 0ull;
        f.st->skip = full;
        if (f.first) f.st->full = 0;
    }
    rank_group(a, ids);
    __shared__ float s_y[32][65];
    __shared__ float s_t[32];
    __shared__ float s_r[8];
    const int tid = threadIdx.x, u = tid >> 3, l8 = tid & 7, dim = a.dim;
    const int z = (int)blockIdx.z;
    if ((int)blockIdx.x < f.nqb) {
        const int64_t ql = (int64_t)blockIdx.x * 32 + u;       // within the chunk
        const int64_t q = f.q_first + ql;
        const int64_t nq = min(a.nq - f.q_first, (int64_t)f.q_cap);
        if ((int64_t)blockIdx.x * 32 >= nq) return;            // (uniform)
        const RankRows rw = rank_rows<HEAD>(a, min(q, a.nq - 1));
        if (rw.bad && l8 == 0 && ql < nq) atomicAdd(a.bad, 1);
        float mx = 0.f, acc = 0.f;
        float *q32 = f.q32 + (ql + (a.true_score - f.a.true_score)) * dim;
        for (int j0 = 0; j0 < dim; j0 += 64) {
            float va[8], vr[8], ve[8];
            const int j = j0 + l8 * 8;
            load8(rw.pa, j, dim, va);
            load8(rw.pr, j, dim, vr);
            load8(rw.ptrue, j, dim, ve);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float qv = HEAD ? va[i] - vr[i] : va[i] + vr[i];
                mx = fmaxf(mx, fabsf(qv));
                s_y[u][l8 * 8 + i] = HEAD ? ve[i] - qv : qv - ve[i];
                va[i] = qv;
            }
            if (ql < nq) {
                if (j < dim) st4(q32 + j, make_float4(va[0], va[1], va[2], va[3]));
                if (j + 4 < dim) st4(q32 + j + 4, make_float4(va[4], va[5], va[6], va[7]));
            }
            __syncthreads();
            if (tid < 32) {
                const int n = min(64, dim - j0);
                if (n == 64) {
#pragma unroll 16
                    for (int jj = 0; jj < 64; ++jj) acc = rank_step<DIST>(acc, s_y[tid][jj]);
                } else {
                    for (int jj = 0; jj < n; ++jj) acc = rank_step<DIST>(acc, s_y[tid][jj]);
                }
            }
            __syncthreads();
        }
        if (tid < 32) {
            s_t[tid] = acc;
            const int64_t qq = f.q_first + (int64_t)blockIdx.x * 32 + tid;
            if ((int64_t)blockIdx.x * 32 + tid < nq) {
                a.true_score[qq] = acc;
                a.n_less[qq] = 0;
                a.n_equal[qq] = 0;
            }
        }
        __syncthreads();
        const float st = s_t[u];
        if (SAD) {
            const float sc = TORUS ? 65536.f : *f.scale;
            const int64_t grp = ql >> 4;
            float res = 0.f;
            for (int p = l8; p < f.np; p += 8) {
                float va[8], vr[8];
                load8(rw.pa, p * 8, dim, va);
                load8(rw.pr, p * 8, dim, vr);
                uint32_t k[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    // (past the row's end query and candidate hold the same number and add nothing, rounding aside)
                    k[i] = fixed16<TORUS>(HEAD ? va[i] - vr[i] : va[i] + vr[i], sc, (i & 1) != 0, res);
                    if (TORUS) k[i] ^= 0x8000u;                // half a turn up: the sweep measures from there
                }
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    f.qt[((grp * f.np + p) * 4 + i) * kSadGroup + (ql & 15)] = k[2 * i] | k[2 * i + 1] << 16;
            }
            res = group_sum<8>(res);
            if (l8 == 0) {
                int2 thr = make_int2(kNoQuery, kNoQuery);  // past the last query: nothing is below, nothing undecided
                if (ql < nq) {
                    // the index-order sum is within (dim + 8) 2^-24 of the sum of its terms' exact values
                    const double t = (double)st * (double)sc, rel = 1.02 * (dim + 8) * (double)kUnit;
                    const double lo = t * (1.0 - rel) - (double)res * 1.001, hi = t * (1.0 + rel) + (double)res * 1.001;
                    thr.x = lo > -1e8 && lo < 5e8 ? (int)floor(lo) - 1 : -(1 << 29);
                    thr.y = hi > -1e8 && hi < 5e8 ? (int)ceil(hi) + 1 : 1 << 29;
                    if (thr.y == 1 << 29) thr.x = -(1 << 29);
                }
                f.thr[ql] = thr;
            }
            return;
        }
        bool ok;
        mx = max_group8(mx);
        float n2 = 0.f, d2 = 0.f;
        uint4 *dst = f.qf + ((int64_t)z * (f.q_cap / 32) + blockIdx.x) * (f.np / 2) * 64;
        if constexpr (WIDE) {
            const float sc = wide_scale(mx, ok);
            float l2 = 0.f;
            for (int p = l8; p < f.np / 2; p += 8) {           // sixteen elements a piece
                float va[16], vr[16];
                load8(rw.pa, p * 16, dim, *(float (*)[8])va);
                load8(rw.pa, p * 16 + 8, dim, *(float (*)[8])(va + 8));
                load8(rw.pr, p * 16, dim, *(float (*)[8])vr);
                load8(rw.pr, p * 16 + 8, dim, *(float (*)[8])(vr + 8));
#pragma unroll
                for (int i = 0; i < 16; ++i) va[i] = HEAD ? va[i] - vr[i] : va[i] + vr[i];
                uint4 hi, lo;
                wide_piece(va, sc, hi, lo, n2, d2, l2);
                dst[(p >> 1) * 128 + u + 32 * (p & 1)] = hi;
                dst[(p >> 1) * 128 + 64 + u + 32 * (p & 1)] = lo;
            }
            n2 = group_sum<8>(n2);
            d2 = group_sum<8>(d2);
            l2 = group_sum<8>(l2);
            if (l8 == 0) {
                // As below, in units scaled by sc / 256 (and by the candidate tile's scale).  The sums of the matrix cores are
                // exact here.  What is computed differs by
                //   the fixed-point roundings |q| |de| + |dq| (|e| + |de|), and 2^-24 of either row where it is scaled
                //   the low bytes' product    at most the product of their norms
                //   a few fp32 roundings      of the sum, of |e|^2/2 and of tau
                //   the norms and tau, the index-order sums: as below
                const float eps = 4.f * kUnit, kap = norm_slack(f.np) + 4.f * kUnit;
                const float qn = sqrtf(n2) * 1.0001f, dq = sqrtf(d2) * 1.002f + 1.01f * kUnit * qn, qq = n2 / sc, un = 1.f / 256.f;
                float4 par;
                par.x = (dq * 1.001f + 6.f * kUnit * qn) * un;
                par.y = qn * un;
                par.z = 0.5f * (qq - st * sc) * un;
                par.w = (kap * (qq + st * sc) + 0.51f * (float)(dim + 8) * kUnit * (st * sc)) * un + eps * fabsf(par.z);
                if (!ok || !(par.w < 1e30f)) par.w = __builtin_inff();
                if (ql >= nq) par = make_float4(0.f, 0.f, 3e37f, 0.f);
                const int64_t i = (int64_t)z * f.q_cap + ql;
                f.qpar[i] = par;
                f.qscale[i] = sc * un;
                f.qlow[i] = sqrtf(l2) * 1.001f * un;
            }
            return;
        }
        const float sc = pow2_scale(mx, ok);
        for (int p = l8; p < f.np; p += 8) {
            float va[8], vr[8], q8[8];
            load8(rw.pa, p * 8, dim, va);
            load8(rw.pr, p * 8, dim, vr);
#pragma unroll
            for (int i = 0; i < 8; ++i) q8[i] = HEAD ? va[i] - vr[i] : va[i] + vr[i];
            dst[(p >> 1) * 64 + u + 32 * (p & 1)] = half_piece(q8, sc, n2, d2);
        }
        n2 = group_sum<8>(n2);
        d2 = group_sum<8>(d2);
        if (l8 == 0) {
            // In units scaled by sc (and, in the sweep, by the candidate tile's scale), with t = q.e - |e|^2/2 - tau and
            // tau = (|q|^2 - S_true)/2, a candidate is below the true entity when t > 0.  What is computed differs by
            //   the fp16 roundings        |q| |de| + |dq| (|e| + |de|)
            //   the fp32 sums of the matrix cores: one instruction at most 2^-24 (2.5 |C| + 10 sum |p|) (it cuts off what lies
            //                             below 2^-24 of the largest of eight products; nine tenths of that measured, and
            //                             tested), |C| up to |e|^2/2 + |tau| + |q| |e|, all the |p| up to |q| |e|
            //   the norms and tau         fp32 sums of |q|^2 and |e|^2 in chains of dim / 8, a few more roundings
            //   the index-order sums      (dim + 8) 2^-24 S_true / 2
            const float eps = 2.5f * kUnit * (float)(f.np / 2 + 2), kap = norm_slack(f.np);
            float4 par;
            const float qn = sqrtf(n2) * 1.0001f, dq = sqrtf(d2) * 1.002f;
            const float qq = n2 / sc;                          // sc |q|^2 in true units
            par.x = dq * 1.001f + (eps + 5.f * kUnit) * qn;                    // times the tile's largest norm
            par.y = qn;                                        // times the tile's largest rounding
            par.z = 0.5f * (qq - st * sc);                     // tau
            par.w = kap * (qq + st * sc) + eps * fabsf(par.z) + 0.51f * (float)(dim + 8) * kUnit * (st * sc);
            if (!ok || !(par.w < 1e30f)) par.w = __builtin_inff();
            if (ql >= nq) par = make_float4(0.f, 0.f, 3e37f, 0.f);
            f.qpar[(int64_t)z * f.q_cap + ql] = par;
            f.qscale[(int64_t)z * f.q_cap + ql] = sc;
        }
        return;
    }
    if (SAD || (!f.first && f.st->full)) return;
    // ---- 32 candidates: tile number et of the segment -----------------------------------------------------
    const int et = (int)blockIdx.x - f.nqb;
    const int64_t e = (int64_t)f.e_first + (int64_t)et * 32 + u;
    const int64_t tiles = ((int64_t)f.e_count + 31) / 32;
    const bool in = e < a.n_ent;
    const float *pe = a.X + min(e, (int64_t)a.n_ent - 1) * dim;
    float mx = 0.f;
    for (int j = l8 * 4; j < dim; j += 32) {
        const float4 v = ld4(pe + j);
        mx = fmaxf(fmaxf(fmaxf(mx, fabsf(v.x)), fmaxf(fabsf(v.y), fabsf(v.z))), fabsf(v.w));
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) mx = fmaxf(mx, __shfl_xor(mx, m, 64));
    if ((tid & 63) == 0) s_r[tid >> 6] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(s_r[0], s_r[1]), fmaxf(s_r[2], s_r[3]));
    bool ok;
    const float sc = WIDE ? wide_scale(mx, ok) : pow2_scale(mx, ok);
    float n2 = 0.f, d2 = 0.f, l2 = 0.f;
    uint4 *dst = f.ef + ((int64_t)z * tiles + et) * (f.np / 2) * 64;
    if constexpr (WIDE) {
        for (int p = l8; p < f.np / 2; p += 8) {
            float v[16];
            load8(pe, p * 16, dim, *(float (*)[8])v);
            load8(pe, p * 16 + 8, dim, *(float (*)[8])(v + 8));
            uint4 hi, lo;
            wide_piece(v, sc, hi, lo, n2, d2, l2);
            if (!in) hi = lo = make_uint4(0u, 0u, 0u, 0u);
            dst[(p >> 1) * 128 + u + 32 * (p & 1)] = hi;
            dst[(p >> 1) * 128 + 64 + u + 32 * (p & 1)] = lo;
        }
        l2 = group_sum<8>(l2);
    } else for (int p = l8; p < f.np; p += 8) {
        float v[8];
        load8(pe, p * 8, dim, v);
        uint4 h = half_piece(v, sc, n2, d2);
        if (!in) h = make_uint4(0u, 0u, 0u, 0u);
        dst[(p >> 1) * 64 + u + 32 * (p & 1)] = h;
    }
    n2 = group_sum<8>(n2);
    d2 = group_sum<8>(d2);
    if (l8 == 0) {
        s_t[u] = n2;
        s_y[0][u] = d2;
        s_y[1][u] = l2;
        f.eaux[((int64_t)z * tiles + et) * 64 + u] = in ? 0.5f * n2 / sc : 3e37f;   // past the end: never below
    }
    __syncthreads();
    if (tid < 32) {
        float m2 = s_t[tid], dd = s_y[0][tid], ll = s_y[1][tid];
        bool fin = m2 < 1e30f && dd < 1e30f;                   // (false for NaN)
#pragma unroll
        for (int m = 16; m >= 1; m >>= 1) {
            m2 = fmaxf(m2, __shfl_xor(m2, m, 32));
            dd = fmaxf(dd, __shfl_xor(dd, m, 32));
            ll = fmaxf(ll, __shfl_xor(ll, m, 32));
        }
        fin = (__ballot(fin) & 0xffffffffull) == 0xffffffffull;
        if (tid == 0) {
            const float kap = norm_slack(f.np) + (WIDE ? 8.f * kUnit : 1.25f * kUnit * (float)(f.np / 2 + 2));
            float4 t = make_float4(sc, sqrtf(m2) * 1.0001f, sqrtf(dd) * 1.002f, kap * m2 / sc);
            if (WIDE) t.z += 1.01f * kUnit * t.y;
            if (!fin || !ok) t.y = t.z = t.w = __builtin_inff();
            float *aux = f.eaux + ((int64_t)z * tiles + et) * 64;
            st4(aux + 32, t);
            aux[36] = sqrtf(ll) * 1.001f;
        }
    }
}

// ---- L1 kinds: fixed point ----------------------------------------------------------------------------------
// A workgroup keeps 64 C candidates (C per lane) in LDS as 16-bit pairs; its wavefronts walk groups of 16 queries,
// whose packed values are wavefront-uniform and come through scalar loads, so the inner step is one vector operation
// per two elements (two for the torus kind) with one 16-byte LDS read per 64 C of them.  Bound by the rate of
// v_sad_u16 (half that of an fp32 addition: 36 against 62 T lane-operations per second measured).
template <int DIST, int C>
__global__ __launch_bounds__(kSadThreads) void k_rank_sad(FilterArgs f)
{
    constexpr bool TORUS = DIST == STX_TORUS_L1;
    constexpr int NE = 64 * C, NW = kSadThreads / 64;
    extern __shared__ __align__(16) unsigned char s_arena[];
    const RankArgs &a = f.a;
    const int np = f.np;
    const int32_t full = f.st->full;                       // (tested below: the load travels beside those of the staging)
    uint4 *s_e = reinterpret_cast<uint4 *>(s_arena);                           // [piece][candidate]
    uint2 *s_list = reinterpret_cast<uint2 *>(s_e + (size_t)np * NE);          // [wavefront][kListCap]
    uint64_t *s_mask = reinterpret_cast<uint64_t *>(s_list + NW * kListCap);   // [wavefront][16 C]
    float *s_res = reinterpret_cast<float *>(s_mask + NW * kSadGroup * C);     // [candidate]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t e0 = (int64_t)blockIdx.x * NE;
    const float sc = TORUS ? 65536.f : *f.scale;
    if (tid < NE) s_res[tid] = 0.f;
    __syncthreads();
    // staging: four pieces (128 bytes) of a row per four consecutive threads
    for (int i = tid; i < ((np + 3) / 4) * 4 * NE; i += kSadThreads) {
        const int c = (i >> 2) & (NE - 1), p = (i / (4 * NE)) * 4 + (i & 3);
        if (p >= np) continue;
        float v[8], res = 0.f;
        load8(a.X + min(e0 + c, (int64_t)a.n_ent - 1) * a.dim, p * 8, a.dim, v);
        uint32_t k[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) k[q] = fixed16<TORUS>(v[q], sc, false, res);
        s_e[p * NE + c] = make_uint4(k[0] | k[1] << 16, k[2] | k[3] << 16, k[4] | k[5] << 16, k[6] | k[7] << 16);
        atomicAdd(&s_res[c], res);
    }
    __syncthreads();
    // The largest rounding of the tile's candidates, in whole units.  Candidates with far larger ones (clamped rows, infinities,
    // NaN) do not count: they are left undecided one by one instead of widening the bound for all.  (Elements inside the
    // range are off by half a unit each; four times the smallest: the torus kind's unwrapped rows are all off by more.)
    uint64_t valid[C], out[C];
    float least = __builtin_inff();
#pragma unroll
    for (int c = 0; c < C; ++c) least = fminf(least, s_res[c * 64 + lane]);
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) least = fminf(least, __shfl_xor(least, m, 64));
    const float far = fminf(fmaxf(0.55f * 8.f * (float)np + 1.f, 4.f * least), 1e8f);
    float res = 0.f;
    bool any_out = false;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const float r = s_res[c * 64 + lane];
        const uint64_t in = __ballot(e0 + c * 64 + lane < a.n_ent);
        out[c] = __ballot(!(r <= far)) & in;
        valid[c] = in & ~out[c];
        any_out = any_out || out[c] != 0ull;
        if (r <= far) res = fmaxf(res, r);
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) res = fmaxf(res, __shfl_xor(res, m, 64));
    const int er = __builtin_amdgcn_readfirstlane((int)ceilf(res * 1.001f) + 1);

    const int64_t ngroups = ((int64_t)min(a.nq - f.q_first, (int64_t)f.q_cap) + kSadGroup - 1) / kSadGroup;
    const int64_t g_end = min((int64_t)(blockIdx.y + 1) * f.slice, ngroups);
    uint2 *list = s_list + wave * kListCap;
    uint64_t *masks = s_mask + wave * kSadGroup * C;
    int cnt = 0;
    if (full) return;                                      // (no barrier from here on)
    for (int64_t g = (int64_t)blockIdx.y * f.slice + wave; g < g_end; g += NW) {
        const STX_CONST_AS uint32_t *qp = (const STX_CONST_AS uint32_t *)(f.qt + g * np * (4 * kSadGroup));
        uint32_t acc[C][kSadGroup];
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
            for (int q = 0; q < kSadGroup; ++q) acc[c][q] = 0u;
        for (int p = 0; p < np; ++p) {
            uint4 ev[C];
#pragma unroll
            for (int c = 0; c < C; ++c) ev[c] = s_e[p * NE + c * 64 + lane];
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int q = 0; q < kSadGroup; ++q) {
                    const uint32_t qv = qp[(p * 4 + k) * kSadGroup + q];
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        const uint32_t e = k == 0 ? ev[c].x : k == 1 ? ev[c].y : k == 2 ? ev[c].z : ev[c].w;
                        if (TORUS) acc[c][q] = __builtin_amdgcn_sad_u16(qv - e, 0x80008000u, acc[c][q]);
                        else acc[c][q] = __builtin_amdgcn_sad_u16(qv, e, acc[c][q]);
                    }
                }
        }
        const STX_CONST_AS int2 *thr = (const STX_CONST_AS int2 *)(f.thr + g * kSadGroup);
        int lessv = 0;
        uint32_t dirty = 0;
#pragma unroll
        for (int q = 0; q < kSadGroup; ++q) {
            const int lo = thr[q].x - er, hi = thr[q].y + er;
            int n = 0;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const uint64_t lm = __ballot((int)acc[c][q] < lo) & valid[c];
                const uint64_t um = __ballot((int)acc[c][q] <= hi) & valid[c] & ~lm;
                n += __builtin_popcountll(lm);
                if (um) {
                    masks[q * C + c] = um;
                    dirty |= 1u << (q * C + c);
                }
            }
            lessv = lane == q ? n : lessv;
        }
        if (any_out) {
#pragma unroll 1
            for (int i = 0; i < kSadGroup * C; ++i) {
                const uint64_t o = C == 2 && (i & 1) ? out[C - 1] : out[0];
                if (!o || thr[i / C].y == kNoQuery) continue;
                masks[i] = o | (dirty >> i & 1u ? masks[i] : 0ull);
                dirty |= 1u << i;
            }
        }
        const int64_t q0 = f.q_first + g * kSadGroup;
        if (lane < kSadGroup && lessv) atomicAdd(&a.n_less[q0 + lane], lessv);
        while (dirty) {
            const int i = __builtin_ctz(dirty);
            dirty &= dirty - 1;
            const uint64_t m = masks[i];
            if (m >> lane & 1) list[cnt + mask_rank(m)] = make_uint2((uint32_t)(e0 + (i % C) * 64 + lane), (uint32_t)(q0 + i / C));
            cnt += __builtin_popcountll(m);
            if (cnt > kListCap - 64) {
                if (!flush_pairs<DIST>(f, list, cnt, lane)) return;
                cnt = 0;
            }
        }
    }
    if (cnt) flush_pairs<DIST>(f, list, cnt, lane);
}

// ---- L2 kinds: matrix cores -----------------------------------------------------------------------------------
// A wavefront keeps QF blocks of 32 queries (all KS steps of their rows) in registers; its workgroup's four wavefronts
// share a stream of candidates, 32 to a tile, in operand order: a step of a tile is one contiguous kilobyte.  The
// stream goes to LDS by direct loads, a chunk of CK kilobytes at a time, each wavefront fetching a quarter, NB - 1
// chunks ahead (one barrier per chunk): with every wavefront reading the stream into its own registers the sweep waited
// for memory most of the time.  Rows of at most 256 floats; 3,000 queries x 100,951 at d = 128 take 210 us.
// v_mfma_f32_32x32x16_f16: rows are candidates, columns (lanes) queries; the accumulator starts at
// -(|e|^2/2 + tau), so its sign is the decision.
template <int QF, int KS, int WPE>
__global__ __launch_bounds__(kThreads, WPE) void k_rank_mfma(FilterArgs f, RankIds ids)
{
    constexpr int CK = 32 % KS == 0 ? 32 : 24, NB = 2;     // kilobytes per chunk, chunks in LDS (64 KB at most: two workgroups per compute unit)
    constexpr int LW = CK / 4, TPC = CK / KS;              // kilobytes a wavefront fetches, tiles per chunk
    static_assert(CK % KS == 0, "whole tiles");
    constexpr int LA = TPC > 4 ? TPC / 4 : 1;              // auxiliary loads per wavefront and chunk
    __shared__ __align__(1024) uint4 s_ring[NB][CK][64];
    __shared__ __align__(256) float s_aux[NB][TPC][64];
    __shared__ uint2 s_list[4][kListCap];
    RankArgs a = f.a;
    rank_group(a, ids);
    const int lane = threadIdx.x & 63, half = lane >> 5, z = (int)blockIdx.z;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int nq = (int)min(a.nq - f.q_first, (int64_t)f.q_cap);
    if ((int)blockIdx.x * 4 * QF * 32 >= nq) return;
    const int32_t skip = f.first ? 0 : f.st->skip;
    const int q_base = f.q_first + (int)(a.true_score - f.a.true_score);       // position of the chunk in the query arrays
    const uint32_t zbits = f.z_shift < 32 ? (uint32_t)z << f.z_shift : 0u;
    // Wavefronts with queries of their own: four, or two or one where the workgroup's queries are few; the others take
    // the same queries and every second or fourth tile of a chunk.
    const int left = (nq - (int)blockIdx.x * 128 * QF + 32 * QF - 1) / (32 * QF), wq = left > 2 ? 4 : left > 1 ? 2 : 1;
    const int parts = 4 / wq, part = wave / wq;
    const int qb = ((int)blockIdx.x * 4 + wave % wq) * QF;                     // first block of 32 queries
    const bool works = qb * 32 < nq;
    const int tiles = (f.e_count + 31) / 32;
    const int t0 = (int)blockIdx.y * f.slice, t1 = min(t0 + f.slice, tiles);
    const uint4 *src = f.ef + ((int64_t)z * tiles + t0) * KS * 64 + wave * LW * 64 + lane;
    const int chunks = ((t1 - t0) * KS + CK - 1) / CK;
    const uint32_t ring = lds_at(&s_ring[0][0][0]);
    const uint32_t ring_aux = lds_at(&s_aux[0][0][0]);
    const float *aux = f.eaux + ((int64_t)z * tiles + t0) * 64 + lane;
    auto fetch = [&](int c, int slot) {                                        // (past the end: the last chunk once more)
        const uint4 *g = src + (int64_t)min(c, chunks - 1) * CK * 64;
#pragma unroll
        for (int i = 0; i < LW; ++i) load_lds_1k(g + i * 64, ring + (uint32_t)((slot * CK + wave * LW + i) * 1024));
        const float *ga = aux + (int64_t)min(c, chunks - 1) * TPC * 64;
#pragma unroll
        for (int i = 0; i < LA; ++i) {                                         // (fewer tiles than wavefronts: some fetch the same)
            const int tile = (wave + 4 * i) % TPC;
            load_lds_256(ga + tile * 64, ring_aux + (uint32_t)((slot * TPC + tile) * 256));
        }
    };
    half8 qf[QF][KS];
    float p_x[QF], p_y[QF], p_z[QF], p_w[QF], p_s[QF];
#pragma unroll
    for (int q = 0; q < QF; ++q) {
        const int blk = min(qb + q, (nq + 31) / 32 - 1);                       // past the end: repeated, made to count nothing
        const uint4 *qs = f.qf + ((int64_t)z * (f.q_cap / 32) + blk) * KS * 64 + lane;
#pragma unroll
        for (int k = 0; k < KS; ++k) qf[q][k] = __builtin_bit_cast(half8, qs[k * 64]);
        const int64_t qi = (int64_t)z * f.q_cap + blk * 32 + (lane & 31);
        float4 par = f.qpar[qi];
        p_s[q] = f.qscale[qi];
        if (qb + q > blk) { par = make_float4(0.f, 0.f, 3e37f, 0.f); p_s[q] = 1.f; }
        p_x[q] = par.x; p_y[q] = par.y; p_z[q] = par.z; p_w[q] = par.w;
    }
    // (the operands arrive here: waited for where they are used, inside the loop, they would hold up the chunks ahead each
    // time, whose loads the compiler does not count)
#pragma unroll
    for (int q = 0; q < QF; ++q)
#pragma unroll
        for (int k = 0; k < KS; ++k) asm volatile("" : "+v"(qf[q][k]));
#pragma unroll
    for (int q = 0; q < QF; ++q) asm volatile("" : "+v"(p_x[q]), "+v"(p_y[q]), "+v"(p_z[q]), "+v"(p_w[q]), "+v"(p_s[q]));
    int less[QF];
#pragma unroll
    for (int q = 0; q < QF; ++q) less[q] = 0;
    int cnt = 0, t = t0;
    bool listing = true;                                   // until there are too many undecided pairs
    floatx16 acc[QF];
    float w[QF];
    auto begin_tile = [&](const float *ta) {
        const float4 et = ld4(ta + 32);
        float4 cn[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) cn[g] = ld4(ta + half * 4 + 8 * g);
#pragma unroll
        for (int q = 0; q < QF; ++q) {
            // (never zero: a zero query's sums against a tile of zero rows are exactly zero, and such ties are undecided)
            w[q] = __builtin_fmaf(__builtin_fmaf(p_x[q], et.y, __builtin_fmaf(p_y[q], et.z, __builtin_fmaf(p_w[q], et.x, p_s[q] * et.w))), 1.0001f, 1e-37f);
            const float tau = -p_z[q] * et.x, ns = -p_s[q];
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                acc[q][4 * g] = __builtin_fmaf(cn[g].x, ns, tau);
                acc[q][4 * g + 1] = __builtin_fmaf(cn[g].y, ns, tau);
                acc[q][4 * g + 2] = __builtin_fmaf(cn[g].z, ns, tau);
                acc[q][4 * g + 3] = __builtin_fmaf(cn[g].w, ns, tau);
            }
        }
    };
    auto end_tile = [&] {
        uint32_t und = 0;                                                      // the lane's undecided sums: bit 31 - 16 q - i
#pragma unroll
        for (int q = QF - 1; q >= 0; --q) {
            uint32_t neg = 0, near = 0;                                        // signs of t and of |t| - w
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const float v = acc[q][i];
                neg = __builtin_amdgcn_alignbit(neg, __float_as_uint(v), 31);
                near = __builtin_amdgcn_alignbit(near, __float_as_uint(fabsf(v) - w[q]), 31);
            }
            if (!(w[q] < 1e37f)) near = 0xffffu;                               // no bound: nothing is decided
            less[q] += 16 - __builtin_popcount(neg | near);
            und |= near << (16 * (1 - q));
        }
        while (__any(und != 0) && listing) {
            const int i = __builtin_clz(und | 1u);
            const int e = f.e_first + t * 32 + (i & 3) + 8 * ((i >> 2) & 3) + 4 * half, q = (qb + i / 16) * 32 + (lane & 31);
            const uint64_t m = __ballot(und != 0 && e < a.n_ent && q < nq);
            und &= ~(0x80000000u >> i);
            if (m >> lane & 1) s_list[wave][cnt + mask_rank(m)] = make_uint2((uint32_t)e | zbits, (uint32_t)(q_base + q));
            cnt += __builtin_popcountll(m);
            if (cnt > kListCap - 64) {
                listing = flush_pairs<STX_L2>(f, s_list[wave], cnt, lane);
                cnt = 0;
            }
        }
    };
#pragma unroll
    for (int c = 0; c < NB - 1; ++c) fetch(c, c);
    if (skip) {
        asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
        return;
    }
    for (int c = 0; c < chunks; ++c) {
        // this wavefront's quarter of chunk c has landed when at most the later NB - 2 chunks' loads are outstanding
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"((NB - 2) * (LW + LA)) : "memory");
        __builtin_amdgcn_sched_barrier(0);
        fetch(c + NB - 1, (c + NB - 1) % NB);              // over the chunk that every wavefront is done with
        if (!works) continue;
        const uint4 (*chunk)[64] = s_ring[c % NB];
#pragma unroll 1
        for (int tt = part; tt < TPC; tt += parts) {
            t = t0 + c * TPC + tt;
            if (t >= t1) break;
            begin_tile(s_aux[c % NB][tt]);
#pragma unroll
            for (int k = 0; k < KS; ++k) {
                const half8 e8 = __builtin_bit_cast(half8, chunk[tt * KS + k][lane]);
#pragma unroll
                for (int q = 0; q < QF; ++q)
                    acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_f16(e8, qf[q][k], acc[q], 0, 0, 0);
            }
            end_tile();
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" : : : "memory");     // (loads into LDS still in flight must not outlive the workgroup)
    if (!works) return;
    if (cnt && listing) flush_pairs<STX_L2>(f, s_list[wave], cnt, lane);
#pragma unroll
    for (int q = 0; q < QF; ++q) {
        const int n = less[q] + __shfl_xor(less[q], 32, 64);
        const int qi = (qb + q) * 32 + lane;
        if (lane < 32 && qi < nq && n) atomicAdd(&a.n_less[f.q_first + qi], n);
    }
}

// Wide rows.  Fp16 leaves one pair in a hundred undecided at d = 1024 (a rounding of 2^-12 a side against scores that differ
// by a few per cent), and summing those took twice the sweep's time.  Here rows are 16-bit fixed point, as high and low
// bytes: three byte products (v_mfma_i32_32x32x32_i8, exact, twice fp16's rate) leave out only the low bytes' own, and one
// pair in 400 is undecided at the same bytes per row, most of them for the index-order sum's own rounding.
// The queries' operands stay in registers, which d = 1024 would fill: every LDS read then waited for its use (5 times the
// matrix cores' time).  So the steps of a row are dealt to KH wavefronts (even and odd ones), and each holds 128 registers
// of them; a tile's halves are exchanged through LDS, behind the next chunk's barrier, and each decides half the candidates.
template <int KS, int KH>
__global__ __launch_bounds__(kThreads * KH, 2) void k_rank_wide(FilterArgs f, RankIds ids)
{
    typedef int intx4 __attribute__((ext_vector_type(4)));
    typedef int intx16 __attribute__((ext_vector_type(16)));
    constexpr int CK = KS / 2, NB = 4, CPT = KS / CK, NW = 4 * KH, LW = CK / NW;   // as in k_rank_mfma
    constexpr int S = KS / 2 / KH, SC = CK / 2 / KH;       // steps of 32 elements (two kilobytes) a wavefront takes of a tile, of a chunk
    constexpr int NV = 16 / KH;                            // sums of a tile a lane decides
    static_assert(CK % NW == 0 && KS % CK == 0 && CK / 2 % KH == 0, "whole chunks");
    __shared__ __align__(1024) uint4 s_ring[NB][CK][64];
    __shared__ __align__(256) float s_aux[NB][64];
    __shared__ uint2 s_list[NW][kListCap];
    __shared__ int s_half[KH > 1 ? NW : 1][KH > 1 ? NV : 1][64];
    RankArgs a = f.a;
    rank_group(a, ids);
    const int lane = threadIdx.x & 63, half = lane >> 5, z = (int)blockIdx.z;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), kh = wave >> 2;
    const int nq = (int)min(a.nq - f.q_first, (int64_t)f.q_cap);
    if ((int)blockIdx.x * 128 >= nq) return;
    const int32_t skip = f.first ? 0 : f.st->skip;
    const int q_base = f.q_first + (int)(a.true_score - f.a.true_score);       // position of the chunk in the query arrays
    const uint32_t zbits = f.z_shift < 32 ? (uint32_t)z << f.z_shift : 0u;
    const int qb = (int)blockIdx.x * 4 + (wave & 3);                           // block of 32 queries
    const bool works = qb * 32 < nq;                                           // (the others only fetch)
    const int tiles = (f.e_count + 31) / 32;
    const int t0 = (int)blockIdx.y * f.slice, t1 = min(t0 + f.slice, tiles);
    const uint4 *src = f.ef + ((int64_t)z * tiles + t0) * KS * 64 + wave * LW * 64 + lane;
    const int chunks = (t1 - t0) * CPT;
    const uint32_t ring = lds_at(&s_ring[0][0][0]);
    const uint32_t ring_aux = lds_at(&s_aux[0][0]);
    const float *aux = f.eaux + ((int64_t)z * tiles + t0) * 64 + lane;
    auto fetch = [&](int c, int slot) {                                        // (past the end: the last chunk once more)
        const int at = min(c, chunks - 1);
        const uint4 *g = src + (int64_t)at * CK * 64;
#pragma unroll
        for (int i = 0; i < LW; ++i) load_lds_1k(g + i * 64, ring + (uint32_t)((slot * CK + wave * LW + i) * 1024));
        load_lds_256(aux + (int64_t)(at / CPT) * 64, ring_aux + (uint32_t)(slot * 256));
    };
    intx4 qh[S], ql[S];
    {
        const int blk = works ? qb : 0;
        const uint4 *qs = f.qf + ((int64_t)z * (f.q_cap / 32) + blk) * KS * 64 + lane;
#pragma unroll
        for (int i = 0; i < S; ++i) {
            qh[i] = __builtin_bit_cast(intx4, qs[(KH * i + kh) * 128]);
            ql[i] = __builtin_bit_cast(intx4, qs[(KH * i + kh) * 128 + 64]);
        }
    }
    // (they arrive here: waited for where they are used, inside the loop, they would hold up the chunks ahead each time,
    // whose loads the compiler does not count)
#pragma unroll
    for (int i = 0; i < S; ++i) asm volatile("" : "+v"(qh[i]), "+v"(ql[i]));
    const int64_t qi0 = (int64_t)z * f.q_cap + (works ? qb : 0) * 32 + (lane & 31);
    float4 par = f.qpar[qi0];
    float p_s = f.qscale[qi0], p_l = f.qlow[qi0];
    asm volatile("" : "+v"(par.x), "+v"(par.y), "+v"(par.z), "+v"(par.w), "+v"(p_s), "+v"(p_l));
    int less = 0, cnt = 0;
    bool listing = true;                                   // until there are too many undecided pairs
    float thr[NV], w = 0.f;                                // of the tile at hand: its sums are held against thr, give or take w
    int mine[NV];
    auto decide = [&](int t) {
        uint32_t neg = 0, near = 0;                        // signs of t and of |t| - w
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const float v = (KH > 1 ? (float)mine[i] + (float)s_half[wave ^ 4][i][lane] : (float)mine[i]) - thr[i];
            neg = __builtin_amdgcn_alignbit(neg, __float_as_uint(v), 31);
            near = __builtin_amdgcn_alignbit(near, __float_as_uint(fabsf(v) - w), 31);
        }
        if (!(w < 1e37f)) near = (1u << NV) - 1u;          // no bound: nothing is decided
        less += NV - __builtin_popcount(neg | near);
        uint32_t und = near << (32 - NV);                  // the lane's undecided sums: bit 31 - i
        while (__any(und != 0) && listing) {
            const int b = __builtin_clz(und | 1u), i = b + kh * NV;
            const int e = f.e_first + t * 32 + (i & 3) + 8 * ((i >> 2) & 3) + 4 * half, q = qb * 32 + (lane & 31);
            const uint64_t m = __ballot(und != 0 && e < a.n_ent && q < nq);
            und &= ~(0x80000000u >> b);
            if (m >> lane & 1) s_list[wave][cnt + mask_rank(m)] = make_uint2((uint32_t)e | zbits, (uint32_t)(q_base + q));
            cnt += __builtin_popcountll(m);
            if (cnt > kListCap - 64) {
                listing = flush_pairs<STX_L2>(f, s_list[wave], cnt, lane);
                cnt = 0;
            }
        }
    };
#pragma unroll
    for (int c = 0; c < NB - 1; ++c) fetch(c, c);
    if (skip) {
        asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
        return;
    }
    intx16 hh, mid;
    for (int c0 = 0; c0 < chunks; c0 += CPT) {
        const int t = t0 + c0 / CPT;
#pragma unroll
        for (int cc = 0; cc < CPT; ++cc) {
            const int c = c0 + cc;
            // this wavefront's part of chunk c has landed when at most the later NB - 2 chunks' loads are outstanding
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"((NB - 2) * (LW + 1)) : "memory");
            __builtin_amdgcn_sched_barrier(0);
            fetch(c + NB - 1, (c + NB - 1) % NB);          // over the chunk that every wavefront is done with
            if (!works) continue;
            const uint4 (*chunk)[64] = s_ring[c % NB];
            if (cc == 0) {
                if (KH > 1 && c0 > 0) decide(t - 1);       // the tile before: the other half's sums lie in LDS now
                const float *ta = s_aux[c % NB];
                const float4 et = ld4(ta + 32);
                w = __builtin_fmaf(par.x, et.y, __builtin_fmaf(par.y, et.z, __builtin_fmaf(par.w, et.x, p_s * et.w)));
                w = __builtin_fmaf(__builtin_fmaf(p_l, ta[36], w), 1.0001f, 1e-37f);   // (never zero: exact ties are undecided)
                const float tau = par.z * et.x;
#pragma unroll
                for (int i = 0; i < NV; ++i) {
                    const int j = i + kh * NV;
                    thr[i] = __builtin_fmaf(ta[(j & 3) + 8 * (j >> 2) + 4 * half], p_s, tau);
                }
#pragma unroll
                for (int i = 0; i < 16; ++i) hh[i] = mid[i] = 0;
            }
            // (two LDS reads ahead of the three products that use them)
            __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
            for (int k = 0; k < SC; ++k) {
                __builtin_amdgcn_sched_group_barrier(0x008, 3, 0);
                if (k + 2 < SC) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                const intx4 eh = __builtin_bit_cast(intx4, chunk[(KH * k + kh) * 2][lane]), el = __builtin_bit_cast(intx4, chunk[(KH * k + kh) * 2 + 1][lane]);
                hh = __builtin_amdgcn_mfma_i32_32x32x32_i8(eh, qh[cc * SC + k], hh, 0, 0, 0);
                mid = __builtin_amdgcn_mfma_i32_32x32x32_i8(el, qh[cc * SC + k], mid, 0, 0, 0);
                mid = __builtin_amdgcn_mfma_i32_32x32x32_i8(eh, ql[cc * SC + k], mid, 0, 0, 0);
            }
        }
        if (!works) continue;
        // (at most 512 steps of up to 127 127 256 and twice 127 128: below 2^31)
        if constexpr (KH > 1) {
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                const int lo = hh[i] * 256 + mid[i], up = hh[NV + i] * 256 + mid[NV + i];
                mine[i] = kh ? up : lo;
                s_half[wave][i][lane] = kh ? lo : up;
            }
        } else {
#pragma unroll
            for (int i = 0; i < NV; ++i) mine[i] = hh[i] * 256 + mid[i];
            decide(t);
        }
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" : : : "memory");   // (loads into LDS still in flight must not outlive the workgroup)
    if (KH > 1) {
        __syncthreads();
        if (works && chunks > 0) decide(t1 - 1);
    }
    if (!works) return;
    if (cnt && listing) flush_pairs<STX_L2>(f, s_list[wave], cnt, lane);
    const int n = less + __shfl_xor(less, 32, 64), qi = qb * 32 + lane;
    if (lane < 32 && qi < nq && n) atomicAdd(&a.n_less[f.q_first + qi], n);
}

// ---- host ---------------------------------------------------------------------------------------------------
static bool sad_kind(int dist) { return dist == STX_L1 || dist == STX_TORUS_L1; }
static bool mfma_kind(int dist) { return dist == STX_L2 || dist == STX_L2_SQ; }
static int sad_pieces(int width) { return (width + 7) / 8; }
// Matrix-core steps of a row: the compiled counts, rows in between are padded with zeros.
static int mfma_steps(int width)
{
    static const int kSteps[] = {1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64};
    for (int s : kSteps)
        if (16 * s >= width) return s;
    return 64;
}
static bool mfma_wide(int ks) { return ks >= 24; }
static size_t mfma_query_bytes(int ks) { return (size_t)ks * 32 + sizeof(float4) + 2 * sizeof(float); }
static size_t mfma_tile_bytes(int ks) { return (size_t)ks * 1024 + 256; }
constexpr size_t kMfmaSlack = 32 * 1024 + 32 * 256;            // reads past the last tile

size_t rank_filter_q_bytes(int dist, int width, int64_t queries)
{
    const int64_t q = (queries + 31) / 32 * 32;
    size_t each = 0;
    if (sad_kind(dist)) each = sad_pieces(width) * 16 + sizeof(int2);
    else if (mfma_kind(dist)) each = mfma_query_bytes(mfma_steps(width));
    else return 0;
    each += (size_t)width * 4;
    const size_t b = (q * each + 2048) * 3 / 2;               // and half as much again for the list of undecided pairs
    return b > (size_t)4 << 20 ? b : (size_t)4 << 20;
}
// Both sides as measured at 230 sizes over rows of 16 to 1,000 floats, tables of 1,000 to 1,500,000 entities and 1 to
// 59,071 queries, in us a side; the rule took the slower filter at none of them.  Rows above 256 floats were measured with
// fp16 operands; k_rank_wide takes about half of that, so the rule still takes no slower filter there, but leaves calls of
// few queries and long tables plain that would gain (128 queries x 150,001 at d = 400: 460 plain, 290 filtered).
// The plain sweep: a serial walk of the row by the kernel of the true sums, then its steps, padded to
// 128 queries and 32 floats.  The filter: launches and dependent passes for every chunk of queries that its scratch
// holds, a little per query, then its steps; the matrix-core kinds also pack the table, which few queries do not repay
// once it is past the caches (128 queries x 700,000 at d = 544: 2,010 plain, 2,245 filtered; 20 x 300,001 at d = 400: 680
// and 465), and a small table gives
// the fixed-point sweep too few candidates to share a query's load (8,000 x 1,000 at d = 256, L1: 177 plain, 597
// filtered; 59,071 x 15,000 at d = 128: 3,850 and 1,950).
bool rank_filter_pays(int dist, int64_t queries, int64_t n_ent, int width, size_t q_bytes)
{
    if (!q_bytes || (!sad_kind(dist) && !mfma_kind(dist))) return false;
    const double q = (double)queries, n = (double)n_ent, w32 = (width + 31) / 32 * 32;
    const double padded = (double)((queries + 127) / 128 * 128);
    if (padded * n * width < 6e8) return false;                // a plain sweep of at most about 20 us
    const bool narrow = width <= 32;
    const double per_query = (double)rank_filter_q_bytes(dist, width, 1 << 20) / (1 << 20);   // the list's share included
    double chunks = ceil(q * per_query / (double)q_bytes), pass = 25. + 0.1 * width, sweep;
    if (sad_kind(dist)) {
        const double listed = ceil(q * n / ((double)(q_bytes / 3 / sizeof(uint2)) * 1000.));   // as rank_filtered cuts them
        if (chunks < listed) chunks = listed;
        if (narrow) pass = 60.;
        sweep = q * (n > 4096. ? n : 4096.) * w32 / (narrow ? 38e6 : dist == STX_TORUS_L1 ? 25e6 : 41e6);
    } else {
        const double wp = 16. * mfma_steps(width);
        sweep = n * wp * (3.8e-6 + 0.018e-6 * (q < 128. ? q : 128.)) + n * (narrow ? 0.8e-6 * q : 0.012e-6 * wp * (q > 128. ? q - 128. : 0.));
    }
    const double filtered = chunks * pass + 0.003 * q + sweep;
    const double plain = 0.6 * width + padded * n * w32 / (dist == STX_TORUS_L1 ? 12e6 : 28e6);
    return filtered < plain;
}
size_t rank_filter_e_bytes(int dist, int width, int64_t candidates, int tables)
{
    return mfma_kind(dist) ? (size_t)((candidates + 31) / 32) * tables * mfma_tile_bytes(mfma_steps(width)) + kMfmaSlack : 0;
}

template <int QF, int KS, int WPE>
static void go_mfma(stx_ctx *c, FilterArgs &f, int64_t nq, int nz, const RankIds &ids)
{
    const unsigned gx = (unsigned)((nq + 128 * QF - 1) / (128 * QF));
    const int tiles = (f.e_count + 31) / 32;
    // One round of the workgroups that fit the chip (starting one costs a few microseconds of dependent loads), up to
    // four when a workgroup then still streams 256 steps: the last round is partly empty.
    const int64_t slots = 256 * WPE, blocks = (int64_t)gx * nz;
    int64_t rounds = (int64_t)tiles * KS * blocks / (slots * 256);
    rounds = rounds < 1 ? 1 : rounds > 4 ? 4 : rounds;
    int64_t slices = (slots * rounds + blocks - 1) / blocks;
    int slice = (int)((tiles + slices - 1) / slices);
    if (slice < 4) slice = 4;
    slices = (tiles + slice - 1) / slice;
    f.slice = slice;
    ProfScope prof(c, "k_rank_mfma");
    hipLaunchKernelGGL((k_rank_mfma<QF, KS, WPE>), dim3(gx, (unsigned)slices, (unsigned)nz), dim3(kThreads), 0, c->stream, f, ids);
}
template <int QF, int KS, int WPE>
static void go_mfma_q(stx_ctx *c, FilterArgs &f, int64_t nq, int nz, const RankIds &ids)
{
    if (nq <= 128) go_mfma<1, KS, WPE>(c, f, nq, nz, ids);
    else go_mfma<QF, KS, WPE>(c, f, nq, nz, ids);
}
template <int KS, int KH>
static void go_wide(stx_ctx *c, FilterArgs &f, int64_t nq, int nz, const RankIds &ids)
{
    const unsigned gx = (unsigned)((nq + 127) / 128);
    const int tiles = (f.e_count + 31) / 32;
    const int64_t slots = 256 * 2 / KH, blocks = (int64_t)gx * nz;             // rounds as in go_mfma
    int64_t rounds = (int64_t)tiles * KS * blocks / (slots * 256);
    rounds = rounds < 1 ? 1 : rounds > 4 ? 4 : rounds;
    int64_t slices = (slots * rounds + blocks - 1) / blocks;
    int slice = (int)((tiles + slices - 1) / slices);
    if (slice < 4) slice = 4;
    slices = (tiles + slice - 1) / slice;
    f.slice = slice;
    ProfScope prof(c, "k_rank_wide");
    hipLaunchKernelGGL((k_rank_wide<KS, KH>), dim3(gx, (unsigned)slices, (unsigned)nz), dim3(kThreads * KH), 0, c->stream, f, ids);
}
template <int DIST, int C>
static void go_sad(stx_ctx *c, FilterArgs &f, int64_t nq)
{
    const size_t lds = (size_t)f.np * 64 * C * 16 + (kSadThreads / 64) * ((size_t)kListCap * 8 + kSadGroup * C * 8) + 64 * C * 4;
    // (more than 64 KB of LDS has to be asked for, on every device that runs the kernel)
    (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&k_rank_sad<DIST, C>), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    const int64_t groups = (nq + kSadGroup - 1) / kSadGroup;
    const int64_t gx = ((int64_t)f.a.n_ent + 64 * C - 1) / (64 * C);
    int64_t slices = (4096 + gx - 1) / gx;
    int64_t slice = (groups + slices - 1) / slices;
    const int64_t waves = kSadThreads / 64;
    if (slice < 4 * waves) slice = 4 * waves;                  // staging pays off over a few groups per wavefront
    slice = (slice + waves - 1) / waves * waves;
    slices = (groups + slice - 1) / slice;
    f.slice = (int32_t)slice;
    ProfScope prof(c, "k_rank_sad");
    hipLaunchKernelGGL((k_rank_sad<DIST, C>), dim3((unsigned)gx, (unsigned)slices), dim3(kSadThreads), lds, c->stream, f);
}

bool rank_filtered(stx_ctx *c, const RankArgs &a, int side, const RankScratch &ws, int nz, const RankIds &ids,
                   int64_t queries)
{
    const int dist = c->cfg.dist, width = a.dim;
    const bool sad = sad_kind(dist) && nz == 0;
    if (!sad && !mfma_kind(dist)) return false;
    const int tables = nz > 0 ? nz : 1;
    FilterArgs f{};
    f.a = a;
    f.head = side;
    size_t q_each = ws.q32 ? 0 : (size_t)width * 4;
    if (sad) {
        f.np = sad_pieces(width);
        q_each += (size_t)f.np * 16 + sizeof(int2);
    } else {
        f.np = 2 * mfma_steps(width);
        q_each += mfma_query_bytes(f.np / 2);
    }
    // the list of undecided pairs takes a third of the query scratch; about one pair in a thousand to three hundred is
    // undecided in tables of ordinary values, so one table's sweep covers at most 1,000 pairs per place (fixed point; 32
    // queries at least) or 300 (matrix cores).  Beyond the list, and TransR's sweeps cover any number of pairs, they are
    // treated inside the sweep.
    f.pair_cap = (int32_t)std::min(ws.q_bytes / 3 / sizeof(uint2), (size_t)1 << 30);
    f.tables = tables;
    f.z_shift = 32;
    if (nz > 0) {
        f.z_shift = 26;
        if (a.n_ent >= 1 << 26 || nz > kRankTables) return false;
    }
    const int64_t span = (int64_t)f.pair_cap * (sad ? 1000 : 300);
    int64_t cap = (int64_t)((ws.q_bytes - (size_t)f.pair_cap * sizeof(uint2) - 1024) / q_each / tables) / 32 * 32;
    if (sad && cap > span / a.n_ent / 32 * 32) cap = span / a.n_ent / 32 * 32;
    if (sad && cap < 32) cap = 32;
    if (cap > (a.nq + 31) / 32 * 32) cap = (a.nq + 31) / 32 * 32;
    if (cap < 32 || (nz > 0 && cap < a.nq)) return false;
    f.q_cap = (int32_t)cap;
    char *q = ws.q;
    f.st = (FilterState *)q;
    f.pairs = (uint2 *)(q + 256);
    q += 256 + (size_t)f.pair_cap * sizeof(uint2);
    q += -(uintptr_t)q & 255u;
    f.q32 = ws.q32;
    if (!f.q32) {
        f.q32 = (float *)q;
        q += (size_t)cap * width * 4;
    }
    if (sad) {
        f.scale = (float *)q;
        f.thr = (int2 *)(q + 256);
        f.qt = (uint32_t *)(f.thr + cap);
    } else {
        f.qf = (uint4 *)q;
        f.qpar = (float4 *)(f.qf + (size_t)cap * tables * (f.np / 2) * 2);
        f.qscale = (float *)(f.qpar + (size_t)cap * tables);
        f.qlow = f.qscale + (size_t)cap * tables;
    }
    int64_t seg = a.n_ent;                                     // candidates per segment (matrix cores)
    if (!sad) {
        int64_t tiles = (int64_t)((ws.e_bytes - kMfmaSlack) / mfma_tile_bytes(f.np / 2)) / tables;
        const int64_t all = ((int64_t)a.n_ent + 31) / 32;
        if (tiles < 1 || (nz > 0 && tiles < all)) return false;
        if (tiles > all) tiles = all;
        if (nz == 0 && tiles > span / cap / 32) tiles = span / cap / 32 > 0 ? span / cap / 32 : 1;
        seg = tiles * 32;
        f.ef = (uint4 *)ws.e;
        f.eaux = (float *)(ws.e + (size_t)tiles * tables * (f.np / 2) * 1024 + 32 * 1024);
    }
    int64_t swept = 0;                                         // pairs of the sweep at hand
    auto limit = [&](int64_t nq) {
        swept = (nz > 0 ? queries : nq) * (sad ? a.n_ent : f.e_count);
        // (inside the sweep a pair costs 42 times what it costs the plain one at d = 128, L1; 13 to 23 times with the L2 kinds)
        f.pair_limit = (unsigned long long)f.pair_cap + (unsigned long long)swept / (sad ? 256 : 128);
    };
    auto pairs = [&] {
        ProfScope prof(c, "k_rank_pairs");
        // up to eight workgroups per compute unit, 32 pairs each at a time, for one pair in 256
        const dim3 grid((unsigned)std::min(std::max(swept / 8192, (int64_t)64), (int64_t)2048));
        if (dist == STX_L1) hipLaunchKernelGGL((k_rank_pairs<STX_L1>), grid, dim3(kThreads), 0, c->stream, f, ids);
        else if (dist == STX_TORUS_L1) hipLaunchKernelGGL((k_rank_pairs<STX_TORUS_L1>), grid, dim3(kThreads), 0, c->stream, f, ids);
        else hipLaunchKernelGGL((k_rank_pairs<STX_L2>), grid, dim3(kThreads), 0, c->stream, f, ids);
    };
    // (a call whose pairs all fit the list needs none)
    auto behind = [&](int64_t q0, int64_t nq) {
        if ((unsigned long long)swept > f.pair_limit || seg < a.n_ent) rank_plain_behind(c, a, side, q0, nq, tables, ids, &f.st->full);
    };
    auto prep = [&](int nqb, int neb) {
        f.nqb = nqb;
        f.first = f.q_first == 0 && f.e_first == 0;
        const dim3 grid((unsigned)(nqb + neb), 1, (unsigned)tables);
        ProfScope prof(c, "k_rank_prep");
#define STX_PREP(D, W)                                                                                        \
    if (side) hipLaunchKernelGGL((k_rank_prep<D, true, W>), grid, dim3(kThreads), 0, c->stream, f, ids);      \
    else hipLaunchKernelGGL((k_rank_prep<D, false, W>), grid, dim3(kThreads), 0, c->stream, f, ids);
        if (dist == STX_L1) { STX_PREP(STX_L1, false) }
        else if (dist == STX_TORUS_L1) { STX_PREP(STX_TORUS_L1, false) }
        else if (mfma_wide(f.np / 2)) { STX_PREP(STX_L2, true) }
        else { STX_PREP(STX_L2, false) }
#undef STX_PREP
    };
    if (sad && dist == STX_L1) {
        if (side) hipLaunchKernelGGL((k_rank_scale<true>), dim3(1), dim3(1024), 0, c->stream, a, f.scale);
        else hipLaunchKernelGGL((k_rank_scale<false>), dim3(1), dim3(1024), 0, c->stream, a, f.scale);
    }
    for (int64_t q0 = 0; q0 < a.nq; q0 += cap) {
        const int64_t nq = a.nq - q0 < cap ? a.nq - q0 : cap;
        const int nqb = (int)((nq + 31) / 32);
        f.q_first = (int32_t)q0;
        if (sad) {
            limit(nq);
            prep(nqb, 0);
            const bool narrow = width <= 256;                  // two candidates per lane while their tile leaves LDS for two workgroups
            if (dist == STX_L1) { if (narrow) go_sad<STX_L1, 2>(c, f, nq); else go_sad<STX_L1, 1>(c, f, nq); }
            else { if (narrow) go_sad<STX_TORUS_L1, 2>(c, f, nq); else go_sad<STX_TORUS_L1, 1>(c, f, nq); }
            pairs();
            behind(q0, nq);
            continue;
        }
        for (int64_t e0 = 0; e0 < a.n_ent; e0 += seg) {
            f.e_first = (int32_t)e0;
            f.e_count = (int32_t)(a.n_ent - e0 < seg ? a.n_ent - e0 : seg);
            const bool packed = q0 > 0 && seg >= a.n_ent;      // a table of one segment stays packed for the later chunks
            // (packed and no queries cannot both hold: the first segment of a chunk always has queries to prepare)
            const int nb_q = e0 == 0 ? nqb : 0, nb_e = packed ? 0 : (f.e_count + 31) / 32;
            limit(nq);
            prep(nb_q, nb_e);
            switch (f.np / 2) {
            case 1: go_mfma_q<2, 1, 1>(c, f, nq, tables, ids); break;
            case 2: go_mfma_q<2, 2, 2>(c, f, nq, tables, ids); break;
            case 3: go_mfma_q<2, 3, 2>(c, f, nq, tables, ids); break;
            case 4: go_mfma_q<2, 4, 2>(c, f, nq, tables, ids); break;
            case 6: go_mfma_q<2, 6, 2>(c, f, nq, tables, ids); break;
            case 8: go_mfma_q<2, 8, 2>(c, f, nq, tables, ids); break;
            case 12: go_mfma_q<2, 12, 2>(c, f, nq, tables, ids); break;
            case 16: go_mfma_q<2, 16, 2>(c, f, nq, tables, ids); break;
            case 24: go_wide<24, 1>(c, f, nq, tables, ids); break;
            case 32: go_wide<32, 1>(c, f, nq, tables, ids); break;
            case 48: go_wide<48, 2>(c, f, nq, tables, ids); break;
            default: go_wide<64, 2>(c, f, nq, tables, ids); break;
            }
            pairs();
        }
        behind(q0, nq);
    }
    return true;
}

}  // namespace stx
