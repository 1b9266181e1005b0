// Transposed product A^T.G without atomics, and the sparse SGD update.
//
// SparseTransX Appendix G: for C = A.X the gradient is dL/dX = A^T.dL/dC, itself a sparse-dense
// product.  A^T arrives sorted by column (see stx_build.hip), so the gradient row of column c is the
// signed sum of the G rows named by one contiguous run ("segment") of sorted entries.  Power-law graphs
// make segment lengths wildly uneven (one entity can own >10% of all entries), so work is split by
// entries, not by segments:
//
//   k_seg_reduce   each workgroup owns a tile of consecutive sorted entries, each of its lane groups a
//                  chunk of LPR of them.  A group walks its chunk in order, adding signed G rows into
//                  registers and closing a run whenever an entry is flagged as a segment head.  Runs that
//                  lie inside the chunk are stored to the output directly.  A chunk's first / last run
//                  may continue in a neighbouring chunk; those go to LDS, are stitched in chunk order by
//                  one group, and the (at most two) runs that cross the workgroup's own borders are
//                  stored as partial rows.
//   k_seg_fixup    the workgroup in which a border-crossing run ends adds up that run's partial rows,
//                  in tile order, and stores the result.
//
// Every output row is written exactly once and every sum has a fixed association order, so results are
// bitwise reproducible from run to run.
//
// FUSED variants of both kernels apply the SGD update in place of the store: wherever a gradient row
// would be written they write table[column] - lr * gradient (and wrap it for TorusE) instead, with the
// same two roundings as k_sgd_rows, so the gradient rows never travel to memory and back.  The table
// row of a run is fetched together with the run's first source row, so closing a run costs no extra
// memory round trip.
//
// In stx_train_step the launches of both kernels carry more (template parameter RIDE): the product reads the
// sorted keys and payloads of the build itself, so that the build's last kernel and the sum of the loss run
// as extra workgroups of its launch, and one stage of the next batch's build rides in each launch; with TransR
// the dL/dM_r product (stx_transr_dm_body.h) rides in the product's launch and the sums of its partial matrices
// in the fix-up's.  All parts of a launch share one block of LDS.
#include <algorithm>
#include <type_traits>

#include "stx_emit_body.h"
#include "stx_forward_body.h"
#include "stx_rowops.h"
#include "stx_segw_body.h"
#include "stx_semiring_ops.h"
#include "stx_sort_body.h"
#include "stx_transr_dm_body.h"

namespace stx {

// Work that rides in the launches of the transposed product, as workgroups with the low block indices: the last
// kernel of this batch's build and the sum of the loss (SegWriteRide), and one stage of the next batch's build
// per launch (EmitAhead, ScatterAhead, HistAhead).
struct SegWriteRide {
    SegWriteArgs args;
    int ntiles;
    int use_map;
    // a final sum of the loss that waits for a launch (fin_n > 0: one more workgroup)
    const float *fin_partials;
    int fin_n;
    float fin_scale;
    float *fin_loss;
};

// A value of lane j of each group of LPR lanes, in all lanes of the group.  Groups of whole wavefronts read it into scalar
// registers: what follows from it is then the wavefront's own.
template <int LPR>
__device__ inline int32_t of_lane(int32_t v, int j)
{
    if constexpr (LPR == 64) return __builtin_amdgcn_readlane(v, j);
    else return __shfl(v, j & (LPR - 1), LPR);
}
// The index of a thread's group in the workgroup.
template <int LPR>
__device__ inline int group_index()
{
    const int g = (int)threadIdx.x / LPR;
    return LPR == 64 ? __builtin_amdgcn_readfirstlane(g) : g;
}

enum { HAS_FIRST = 1, FIRST_CONT = 2, HAS_LAST = 4 };

template <int ITERS>
struct Acc {
    float4 v[ITERS];
    __device__ inline void zero()
    {
#pragma unroll
        for (int it = 0; it < ITERS; ++it) v[it] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    __device__ inline void add(const Acc &o)
    {
#pragma unroll
        for (int it = 0; it < ITERS; ++it) {
            v[it].x += o.v[it].x; v[it].y += o.v[it].y; v[it].z += o.v[it].z; v[it].w += o.v[it].w;
        }
    }
};

// STREAM: a row of a table far larger than the caches, read once and rewritten: fetched past them.  (Lanes past the row's width
// load its last float4 again, see load_vec.)
template <int LPR, int ITERS, bool STREAM = false>
__device__ inline void load_row(const float *__restrict__ p, int d4, int lig, Acc<ITERS> &a)
{
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
        const int j = min(lig + it * LPR, d4 - 1);
        a.v[it] = STREAM ? ld4_stream(p + 4 * j) : ld4(p + 4 * j);
    }
}
template <int LPR, int ITERS>
__device__ inline void store_row_stream(float *__restrict__ p, int d4, int lig, const Acc<ITERS> &a)
{
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
        int j = lig + it * LPR;
        if (j < d4) st4_stream(p + 4 * j, a.v[it]);
    }
}
template <int LPR, int ITERS>
__device__ inline void store_row(float *__restrict__ p, int d4, int lig, const Acc<ITERS> &a)
{
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
        int j = lig + it * LPR;
        if (j < d4) st4(p + 4 * j, a.v[it]);
    }
}

struct FusedArgs {             // the update that replaces the store of a gradient row (FUSED kernels)
    float *table;              // rows of 4*d4 floats: row c for column c < n_split
    float *table_b;            // ... and row c - n_split of this one for the other columns
    int32_t n_split;
    const int32_t *touched_cols;
    const int32_t *cols_sorted;  // column of every sorted entry, or null: then it is looked up through the segment
    float lr;
    int mode;                  // 0 plain, 1 keep the fractional part (TorusE, Sec. 4.6), 2 rescale to unit length
    int stream;                // tables far larger than the caches: updated rows bypass them on the way out
};
__device__ inline float *fused_row(const FusedArgs &fu, int32_t col, int ld_tab)
{
    // (unsigned 32 x 32 -> 64 bit product: one instruction, where signed 64-bit operands take six)
    const bool first = col < fu.n_split;
    const uint32_t r = (uint32_t)(first ? col : col - fu.n_split);
    return (first ? fu.table : fu.table_b) + (uint64_t)r * (uint32_t)ld_tab;
}

// A second, independent transposed product that shares the launch (TransH: the sums of gw over the
// relation columns beside the sums of gx / gy over all columns).  Workgroups from `first_block` on work
// on it; all of its entries read `src`.
struct SegSecond {
    int first_block;           // INT_MAX: no second product
    int32_t e_begin, e_end;
    const float *src;
    float *out_rows, *partials;
    float *fused_table;        // FUSED: its columns all lie at or above n_split and update this table ...
    int fused_mode;            // ... in this mode
    int32_t n_pos;             // > 0: in the relation columns, of both products, only rows below this are stored (and not zero)
};

// Entries whose source row is not stored but formed where it is summed (template parameter SRC of k_seg_reduce).
// SRC_SEMIRING + kind: dL/dZ row and the rows of the entry's two other columns (semiring_term).  Storing the three
// terms of every matrix row for the product to read took a launch and ten row transfers per matrix row where this takes
// nine: 47 + 6 us at 65,536 rows of 128 floats (ComplEx) as two kernels and the fix-up.
enum { SRC_STORED = 0, SRC_SEMIRING = 1 };
struct SrcArgs {
    const int32_t *colidx;     // A's column ids, three per row
    const float *X, *G;        // table and per-row rows, d4 float4 each
};

// table row <- x - lr * g, each product and difference rounded once, as in k_sgd_rows.  UNIT: mode 2 may be asked for.
template <int LPR, int ITERS, bool UNIT = true>
__device__ inline void apply_update(float *__restrict__ row, int d4, int lig, const Acc<ITERS> &x, const Acc<ITERS> &g,
                                    float lr, int mode, int stream)
{
    Acc<ITERS> o;
    float ss = 0.f;
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
        const float *xv = &x.v[it].x, *gv = &g.v[it].x;
        float *ov = &o.v[it].x;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float step = lr * gv[q];
            float nv = xv[q] - step;
            if (mode == 1) {
                nv = nv - floorf(nv);
                if (nv >= 1.0f) nv = 0.0f;
            }
            ov[q] = nv;
            ss += lig + it * LPR < d4 ? nv * nv : 0.f;
        }
    }
    if (UNIT && mode == 2) {   // all lanes of the group are here together
        ss = group_sum<LPR>(ss);
        if (ss > 0.f) {
            const float inv = 1.0f / sqrtf(ss);
#pragma unroll
            for (int it = 0; it < ITERS; ++it) {
                o.v[it].x *= inv; o.v[it].y *= inv; o.v[it].z *= inv; o.v[it].w *= inv;
            }
        }
    }
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
        const int j = lig + it * LPR;
        if (j < d4) {
            if (stream) st4_stream(row + 4 * j, o.v[it]);
            else st4(row + 4 * j, o.v[it]);   // a small table is read again by the next step's forward pass
        }
    }
}

// Stitches the chunk-crossing runs of a tile of GROUPS chunks, each in chunk order and by a group of its own: the group in
// whose chunk a run ends adds up its pieces, from the chunk in which the run began (or from the tile's first, for a run that
// came in from an earlier workgroup).  One group walking all chunks took 250 cycles per chunk, 8,000 at 32 groups.
// s_x, s_col_last (FUSED): table row and column of the run that leaves each chunk to the right.
// OWN: the group holds its chunk's flags (own_info); else they are read back from s_info, as the flags of the others are.
template <int LPR, int ITERS, int GROUPS, bool FUSED, bool OWN>
__device__ inline void stitch_runs(const int own_info, const float (*s_part)[2][ITERS * LPR * 4], const int32_t *s_info, const int32_t *s_seg_last,
                                   const float (*s_x)[FUSED ? ITERS * LPR * 4 : 4], const int32_t *s_col_last, float *my_part,
                                   float *out_rows, int ld_out, int d4, int ld_tab, const FusedArgs &fu)
{
    const int lig = threadIdx.x % LPR, grp = threadIdx.x / LPR;
    const int linfo = (int)(threadIdx.x & 63) < GROUPS ? s_info[threadIdx.x & 63] : 0, info = OWN ? own_info : s_info[grp];
    const uint64_t m_cont = __ballot((linfo & FIRST_CONT) != 0), m_last = __ballot((linfo & HAS_LAST) != 0);
    // pieces of the run that reaches chunk g, oldest first; returns the chunk it began in, -1: an earlier workgroup's
    auto run_sum = [&](int g, uint64_t before, Acc<ITERS> &cur) {
        const uint64_t m = m_last & before;
        const int s0 = m ? 63 - __clzll(m) : -1;
#pragma unroll
        for (int it = 0; it < ITERS; ++it) cur.v[it] = ld4(&s_part[s0 < 0 ? 0 : s0][s0 < 0 ? 0 : 1][(lig + it * LPR) * 4]);
        for (int h = s0 < 0 ? 1 : s0 + 1; h <= g; ++h) {
            Acc<ITERS> p;
#pragma unroll
            for (int it = 0; it < ITERS; ++it) p.v[it] = ld4(&s_part[h][0][(lig + it * LPR) * 4]);
            cur.add(p);
        }
        return s0;
    };
    if ((info & HAS_FIRST) && !(info & FIRST_CONT)) {      // a run ends inside this group's chunk
        Acc<ITERS> cur;
        const int s0 = run_sum(grp, (1ull << grp) - 1ull, cur);
        if (s0 < 0) {
            store_row<LPR, ITERS>(my_part, d4, lig, cur);
        } else if constexpr (FUSED) {
            Acc<ITERS> x;
#pragma unroll
            for (int it = 0; it < ITERS; ++it) x.v[it] = ld4(&s_x[s0][(lig + it * LPR) * 4]);
            apply_update<LPR, ITERS>(fused_row(fu, s_col_last[s0], ld_tab), d4, lig, x, cur, fu.lr, fu.mode, fu.stream);
        } else {
            store_row<LPR, ITERS>(out_rows + (int64_t)s_seg_last[s0] * ld_out, d4, lig, cur);
        }
    }
    // the run that goes on into the next tile (then the tile is full); taken by a group that seldom has another
    if (grp == 0 && ((m_cont | m_last) >> (GROUPS - 1) & 1)) {
        Acc<ITERS> cur;
        const int s0 = run_sum(GROUPS - 1, (1ull << (GROUPS - 1) << 1) - 1ull, cur);
        store_row<LPR, ITERS>(my_part + (s0 < 0 ? 0 : ld_out), d4, lig, cur);
    }
}

struct alignas(64) FormedRecord {
    uint32_t a[8], b[8], coef[8], flags[8];
};
// What 64 sorted entries (four chunks of 16) bring to the formed product: worked out once here, read by the wavefronts
// that sum the 64 entries of each slice.
struct alignas(64) FormedHead {
    uint64_t heads;            // entries that head a segment
    uint64_t events;           // positions at which a sum is closed (q: behind entry q - 1): chunk borders and heads ...
    uint64_t to_lds, left;     // ... into LDS; as the run that entered its chunk from the left (else: that leaves it to the right)
    int32_t seg, n_active;     // segment of the first entry; entries of active pairs
    uint32_t info;             // the chunks' flags, a byte each
    uint32_t last;             // the sum closed behind the last entry: 1 into LDS, 2 left
    uint32_t pad[4];
};
// The entries of active pairs (of the others, whose coefficient is +0, nothing is added), in order, from the place of the
// first of 64 on, eight to a record: the byte offsets of the table rows of the matrix row's columns other than the entry's
// own, in row order; its coefficient; 1 tail entry | 2 a sum is closed before this entry | position << 2.  Up to a multiple
// of eight: row 0.
__global__ __launch_bounds__(kThreads) void k_seg_records(const int32_t *__restrict__ packed, const int32_t *__restrict__ seg_id,
                                                          const int32_t *__restrict__ colidx, const float *__restrict__ coefs,
                                                          int32_t nnz, int32_t split, uint32_t row_bytes,
                                                          FormedRecord *__restrict__ recs, FormedHead *__restrict__ hds,
                                                          SegWriteRide fin)
{
    // (the sum of the loss comes along as the first workgroup: 18 us at 98,304 partials as a launch of its own)
    const int fins = fin.fin_n > 0 ? 1 : 0;
    if ((int)blockIdx.x < fins) {                          // uniform in the workgroup
        finish_loss_body(fin.fin_partials, fin.fin_n, fin.fin_scale, fin.fin_loss);
        return;
    }
    const int lane = threadIdx.x & 63;
    const int32_t e0 = (((int32_t)blockIdx.x - fins) * kThreads + (int32_t)threadIdx.x) & ~63;
    if (e0 >= nnz) return;
    const int n = min(64, nnz - e0);
    uint4 rc = make_uint4(0u, 0u, 0u, 0u);
    uint32_t m = 0u;
    if (lane < n) {
        m = (uint32_t)packed[e0 + lane];
        const uint32_t row = m >> 2;
        rc.z = __float_as_uint(coefs[row]);
        if (rc.z != 0u) {                                  // (of the others nothing more is needed)
            const int32_t *cx = colidx + 3 * (int64_t)row;
            const uint32_t c0 = (uint32_t)cx[0] * row_bytes, c1 = (uint32_t)cx[1] * row_bytes, c2 = (uint32_t)cx[2] * row_bytes;
            const bool tail = m & 1u, rel = e0 + lane >= split;
            rc.x = tail || rel ? c0 : c1;
            rc.y = tail ? c1 : c2;
        }
    }
    const bool right_head = e0 + n >= nnz || (packed[e0 + n] & 2);
    const int32_t seg = seg_id[e0];
    const uint64_t heads = __ballot((m & 2u) != 0), active = __ballot(rc.z != 0u);
    const uint64_t events = (heads | 0x0001000100010001ull) & (n < 64 ? (1ull << n) - 1ull : ~0ull) & ~1ull;
    auto from_left = [&](int q) {                          // (no head from the chunk's first entry to entry q - 1)
        const int s = (q - 1) & ~15;
        return e0 + s > 0 && (heads & ((1ull << (q - 1)) * 2ull - 1ull) >> s << s) == 0ull;
    };
    const bool fl = lane > 0 && from_left(max(lane, 1));
    const uint64_t left = __ballot(fl), to_lds = __ballot(fl || ((lane & 15) == 0 && !(heads >> lane & 1ull)));
    uint32_t info = 0u;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int s = 16 * c, t = min(s + 16, n);
        if (s >= n) break;
        const bool first = e0 + s > 0 && !(heads >> s & 1ull), right = t == n ? !right_head : !(heads >> t & 1ull);
        const bool inner = (heads >> s & 0xfffeull) != 0ull;
        info |= (uint32_t)((first ? HAS_FIRST | (!inner && right ? FIRST_CONT : 0) : 0) | (right && (!first || inner) ? HAS_LAST : 0)) << (8 * c);
    }
    const int n_active = __builtin_popcountll(active);
    const bool last_left = from_left(n);
    if (lane == 0)
        hds[e0 >> 6] = FormedHead{heads, events, to_lds, left, seg, n_active, info, (last_left || !right_head ? 1u : 0u) | (last_left ? 2u : 0u), {}};
    const uint64_t upto = (1ull << lane) * 2ull - 1ull, before = active & (upto >> 1);
    const uint64_t since = before ? ~((1ull << (63 - __builtin_clzll(before))) * 2ull - 1ull) : ~0ull;
    const int rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(active >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)active, 0u));
    rc.w = (m & 1u) | ((events & since & upto) ? 2u : 0u) | (uint32_t)lane << 2;
    const bool on = active >> lane & 1ull;
    if (!on) rc = make_uint4(0u, 0u, 0u, 0u);
    const int place = on ? rank : n_active + lane - rank;
    if (on || lane - rank < ((8 - n_active) & 7)) {
        FormedRecord &rec = recs[(e0 + place) >> 3];
        rec.a[place & 7] = rc.x; rec.b[place & 7] = rc.y; rec.coef[place & 7] = rc.z; rec.flags[place & 7] = rc.w;
    }
}

// The transposed product over rows that are formed where they are summed (formed_rows): an active entry's term is
// x = (h + r) - t, from the table row of its own column, which a run keeps in a register, and two others, times the row's
// coefficient through the distance's derivative.  Work is cut as k_seg_reduce<16, 1, false, 16> cuts stored rows, and
// the sums have its bits: tiles of 16 chunks of 16 sorted entries, in 64-float slices.  A wavefront takes four chunks of one
// slice with one float per lane.  Everything but the arithmetic on floats is then the same for the whole wavefront: it
// comes through scalar loads and runs on the scalar unit, and an active entry takes two 256-byte loads and four vector
// instructions.  Bound by the L2 caches' rate for such rows (16 TB/s when every pair is active).  With 16 lanes of a float4
// per entry, four entries side by side and their columns and flags broadcast by shuffles, the vector units were busy three
// quarters of the time with everything but the sums.  This kernel at 393,216 positives, d = 1024, from a fresh table on: 1,197
// us before and 1,112 now while every pair is active; 1,054 and 615 as the mean of the first 30 steps; 926 and 412 in the
// 120th.
// The slices are dealt to the eight dies, each of which keeps its own one or two in its L2 cache.
template <int DIST>
__global__ __launch_bounds__(kThreads, 8) void k_seg_formed(const FormedRecord *__restrict__ recs, const FormedHead *__restrict__ hds,
                                                            const int32_t *__restrict__ touched_cols, int32_t nnz, int ntiles,
                                                            int nslices, const float *__restrict__ X, uint32_t x_bytes, int dim,
                                                            float *__restrict__ out_rows, int ld_out, float *__restrict__ partials)
{
    constexpr int CHUNKS = 16, CPW = CHUNKS / (kThreads / 64), LPR = 16;
    __shared__ float s_part[CHUNKS][2][64];
    __shared__ int32_t s_info[CHUNKS], s_seg_last[CHUNKS];
    // workgroups are dealt to the dies in turn
    const uint32_t total = (uint32_t)ntiles * (uint32_t)nslices, per = (total + 7u) / 8u;
    const uint32_t work = (blockIdx.x & 7u) * per + (blockIdx.x >> 3);
    if (work >= total) return;                             // (uniform)
    const int slice = (int)(work / (uint32_t)ntiles), block = (int)(work - (uint32_t)slice * (uint32_t)ntiles);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int col = slice * 64 + lane;
    // (a row's offset is wavefront-uniform and stays in a scalar register, which a buffer load adds by itself)
    const __amdgpu_buffer_rsrc_t xs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(X), 0, (int)x_bytes, 0x00027000);
    const int lane_off = min(col, dim - 1) * 4;
    auto row_at = [&](uint32_t off) {
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(xs, lane_off, (int)off, 0));
    };
    const int e0 = (block * CHUNKS + wave * CPW) * 16;
    if (e0 >= nnz) {
        if (lane < CPW) s_info[wave * CPW + lane] = 0;
    } else {
        const STX_CONST_AS FormedHead *hd = (const STX_CONST_AS FormedHead *)(hds + (e0 >> 6));
        const STX_CONST_AS FormedRecord *rp = (const STX_CONST_AS FormedRecord *)(recs + (e0 >> 3));
        const STX_CONST_AS int32_t *tc = (const STX_CONST_AS int32_t *)touched_cols;
        const uint64_t heads = hd->heads, to_lds = hd->to_lds, left = hd->left;
        uint64_t waiting = hd->events;                     // events not yet reached
        const int n_active = hd->n_active;
        int32_t cur_seg = hd->seg;
        if (lane < CPW) {
            const uint64_t upto = (1ull << (16 * lane + 15)) * 2ull - 2ull;
            s_info[wave * CPW + lane] = (int)(hd->info >> (8 * lane) & 0xffu);
            s_seg_last[wave * CPW + lane] = cur_seg + __builtin_popcountll(heads & upto);   // (of the chunk's last entry)
        }
        // the rows of this run's column and of the next one's
        const uint32_t row_bytes = (uint32_t)dim * 4u;
        float own = row_at((uint32_t)tc[cur_seg] * row_bytes), next_own = 0.f, acc = 0.f;
        if (heads & ~1ull) next_own = row_at((uint32_t)tc[cur_seg + 1] * row_bytes);
        auto close = [&](int q, bool lds, bool slot0) {
            if (lds) s_part[wave * CPW + ((q - 1) >> 4)][slot0 ? 0 : 1][lane] = acc;
            else if (col < dim) __builtin_nontemporal_store(acc, out_rows + (int64_t)cur_seg * ld_out + col);
            acc = 0.f;
        };
        auto close_until = [&](int p) {                    // the sums whose end lies at or before position p
#pragma unroll 1
            while (waiting & ((1ull << p) * 2ull - 1ull)) {
                const int q = __builtin_ctzll(waiting);
                waiting &= waiting - 1ull;
                close(q, to_lds >> q & 1ull, left >> q & 1ull);
                if (heads >> q & 1ull) {
                    ++cur_seg;
                    own = next_own;
                    if (heads & ~((1ull << q) * 2ull - 1ull)) next_own = row_at((uint32_t)tc[cur_seg + 1] * row_bytes);
                }
            }
        };
        // NB entries at a time, all their rows in flight together
        auto batch = [&](auto nb, int j, int cnt) {
            constexpr int NB = decltype(nb)::value;
            const STX_CONST_AS FormedRecord &rec = rp[j >> 3];
            float va[NB], vb[NB];
#pragma unroll
            for (int u = 0; u < NB; ++u) {
                va[u] = row_at(rec.a[u]);
                vb[u] = row_at(rec.b[u]);
            }
            typedef uint32_t u16x __attribute__((ext_vector_type(16)));
            u16x cf = *(const STX_CONST_AS u16x *)&rec.coef[0];
            asm volatile("" : "+s"(cf));                   // (here, beside the rows' loads, and not one by one where they are used)
#pragma unroll
            for (int u = 0; u < NB; ++u) {
                if (u < cnt) {
                    const uint32_t fl = cf[8 + u];
                    if (fl & 2u) close_until((int)(fl >> 2));
                    // x rounded as the forward pass rounds it (a sum has the same bits either way round); then the derivative
                    // times the coefficient, as write_grad_row would have stored it
                    const float c = __uint_as_float(cf[u]);
                    if (fl & 1u) acc -= dterm<DIST>((va[u] + vb[u]) - own, c);
                    else acc += dterm<DIST>((own + va[u]) - vb[u], c);
                }
            }
        };
        int j = 0;
        for (; j + 8 <= n_active; j += 8) batch(std::integral_constant<int, 8>{}, j, 8);
        if (n_active - j > 4) batch(std::integral_constant<int, 8>{}, j, n_active - j);
        else if (j < n_active) batch(std::integral_constant<int, 4>{}, j, n_active - j);
        close_until(63);
        close(min(64, nnz - e0), hd->last & 1u, hd->last & 2u);
    }
    __syncthreads();
    const int c4 = slice * LPR;
    stitch_runs<LPR, 1, CHUNKS, false, false>(0, s_part, s_info, s_seg_last, nullptr, nullptr, partials + (int64_t)block * 2 * ld_out + 4 * c4,
                                       out_rows + 4 * c4, ld_out, min(LPR, dim / 4 - c4), dim, FusedArgs{});
}

// PACKED: the source rows are records of ld_src bytes at src_a (dim/4 sign bytes) with their coefficients in
// src_b, as the forward pass of an L1-kind distance stores them; values and summation order are the same as with
// dense rows, so both forms give the same bits.
// RAW: `packed` and `seg_id` are the sorted payloads and keys of the build instead (a lane derives its entry's
// row, sign, column and whether it heads a segment from them), and the first sw.ntiles workgroups run the
// build's last kernel, whose arrays nothing reads before the fix-up launch.
// RIDE: 0 none of this; 1 RAW; 2 RAW, and the first kernel of the next batch's build comes along; 3 RAW, and the
// first scatter pass of the next batch's sort comes along; 4 as 2, and that kernel counts the rows per relation;
// 5 as 3, and TransR's dL/dM_r product comes along (its 128 registers still leave four workgroups on a CU, more
// than such a batch gives this product).
// THREADS: threads of a workgroup; with LPR it makes the number of chunks in a tile, and so the order of the sums.
// SUMS: relation columns are summed from rows of positives alone (SegSecond::n_pos); a kernel of its own, as the test for it
// costs the others 2 per cent.
template <int LPR, int ITERS, bool PACKED, int CHUNK, bool FUSED, int RIDE, int SRC = SRC_STORED, int THREADS = kThreads, bool SUMS = false>
__global__ __launch_bounds__(THREADS, RIDE == 5 ? 4 : (ITERS == 1 && FUSED && RIDE != 4 && !SUMS) ? (PACKED ? 8 : 7) : 1) void k_seg_reduce(const int32_t *__restrict__ packed,
                                                         const int32_t *__restrict__ seg_id, int32_t e_begin,
                                                         int32_t e_end, const float *__restrict__ src_a,
                                                         const float *__restrict__ src_b, int32_t split,
                                                         int ld_src, int d4, float *__restrict__ out_rows,
                                                         int ld_out, float *__restrict__ partials, FusedArgs fu,
                                                         SegSecond sec, SegWriteRide sw, EmitAhead ea,
                                                         ScatterAhead sca, DmRide dm, SrcArgs sr = SrcArgs{})
{
    constexpr bool RAW = RIDE != 0;
    static_assert(SRC == SRC_STORED || (!RAW && !PACKED && ITERS == 1 && !FUSED), "formed rows: the plain product");
    constexpr bool SEMI = SRC != SRC_STORED;
    // One block of LDS for whichever part a workgroup plays (the parts' own arrays would add up and cost the
    // launch wavefronts per CU): the product's arrays below, or those of a body that rides.
    static_assert(THREADS == kThreads || RIDE == 0, "the bodies that ride have kThreads threads");
    constexpr int GROUPS_ = THREADS / LPR, ROWF_ = ITERS * LPR * 4;
    constexpr int OWN_LDS = (GROUPS_ * 2 * ROWF_ + (FUSED ? GROUPS_ * ROWF_ : 4) + 3 * GROUPS_) * 4;
    constexpr int RIDE_LDS = RIDE == 0 ? 0
                             : (RIDE == 3 || RIDE == 5) ? kScatterLds
                             : (RIDE == 2 || RIDE == 4) ? emit_lds(true, RIDE == 4)
                                                         : (kFinishLds > kSegWriteLds ? kFinishLds : kSegWriteLds);
    constexpr int ARENA_LDS = OWN_LDS > RIDE_LDS ? OWN_LDS : RIDE_LDS;
    static_assert(kFinishLds <= OWN_LDS || RIDE == 0 || kFinishLds <= RIDE_LDS, "the loss sum fits the block");
    __shared__ __align__(16) unsigned char s_arena[ARENA_LDS];
    int block = (int)blockIdx.x;
    // The arguments that say which part a workgroup plays, and those the product begins with, in one wait: loaded where they
    // are first used, one behind the other, they were 0.8 us of every workgroup of the product.
    if constexpr (RAW) STX_TOGETHER(sw.ntiles, sw.fin_n);
    if constexpr (RIDE == 2 || RIDE == 4) STX_TOGETHER(ea.ntiles);
    if constexpr (RIDE == 3 || RIDE == 5) STX_TOGETHER(sca.ntiles);
    if constexpr (RIDE == 5) STX_TOGETHER(dm.blocks);
    STX_TOGETHER(sec.first_block, gridDim.y, packed, seg_id, e_begin, e_end, src_a, src_b, split, ld_src, d4, partials, ld_out);
    if constexpr (FUSED) STX_TOGETHER(fu.table, fu.table_b, fu.n_split, fu.lr, fu.mode, fu.stream);
    if constexpr (RAW) {
        static_assert(FUSED, "the segment of an entry is not known here");
        static_assert(kSegWriteLds <= ARENA_LDS && kFinishLds <= ARENA_LDS, "riders fit the block of LDS");
        if (block < sw.ntiles) {      // uniform in the workgroup
            if (sw.use_map) seg_write_body<true, true>(block, sw.ntiles, sw.args, s_arena);
            else seg_write_body<false, true>(block, sw.ntiles, sw.args, s_arena);
            return;
        }
        block -= sw.ntiles;
        if (sw.fin_n > 0) {
            if (block == 0) {
                finish_loss_body<true>(sw.fin_partials, sw.fin_n, sw.fin_scale, sw.fin_loss, s_arena);
                return;
            }
            --block;
        }
    }
    if constexpr (RIDE == 2 || RIDE == 4) {
        if (block < ea.ntiles) {      // uniform in the workgroup
            emit_body<kSortItems, true, true, RIDE == 4, true>(block, ea.ntiles, ea.args, s_arena);
            return;
        }
        block -= ea.ntiles;
    }
    if constexpr (RIDE == 5) {
        if (block < dm.blocks) {      // uniform in the workgroup
            transr_dm_body(block, 0, dm.args);
            return;
        }
        block -= dm.blocks;
    }
    if constexpr (RIDE == 3 || RIDE == 5) {
        if (block < sca.ntiles) {
            scatter_body<true, false, kSortItems, true>(block, sca.args, s_arena);
            return;
        }
        block -= sca.ntiles;
    }
    int32_t sums_from = split;                             // SUMS: entries from here on
    if (block >= sec.first_block) {   // uniform in the workgroup
        block -= sec.first_block;
        e_begin = sec.e_begin; e_end = sec.e_end;
        sums_from = e_begin;
        src_a = src_b = sec.src; split = sec.e_end;
        out_rows = sec.out_rows; partials = sec.partials;
        fu.table_b = sec.fused_table; fu.mode = sec.fused_mode;
    }
    // A row wider than the lanes of a group cover at once can be cut into slices of LPR float4, one per
    // blockIdx.y: every pointer moves to the slice's first column and the width shrinks to the slice.
    const int ld_tab = d4 * 4;                             // floats per table row (fused update)
    int pk_off = 0;                                        // packed records: sign byte of the slice's first float4
    if (gridDim.y > 1) {
        const int c4 = (int)blockIdx.y * LPR;
        d4 = min(LPR, d4 - c4);
        if (PACKED) pk_off = c4;
        else if (SRC == SRC_STORED) { src_a += 4 * c4; src_b += 4 * c4; }
        else { sr.X += 4 * c4; sr.G += 4 * c4; }
        if (out_rows) out_rows += 4 * c4;
        partials += 4 * c4;
        if (fu.table) fu.table += 4 * c4;
        if (fu.table_b) fu.table_b += 4 * c4;
    }
    constexpr int GROUPS = THREADS / LPR;
    // rows in flight per lane: dense rows cost 4*ITERS registers each; packed rows are a byte and a float,
    // so a whole chunk is fetched at once and the kernel pays one memory latency per chunk
    constexpr int UNROLL = SRC != SRC_STORED ? 4 : PACKED ? (FUSED ? 4 : (CHUNK < 8 ? CHUNK : 8)) : (ITERS == 1 ? (FUSED ? 4 : 8) : (ITERS == 2 ? 4 : 2));
    constexpr int TILE = GROUPS * CHUNK;    // sorted entries per workgroup
    static_assert(CHUNK <= LPR && CHUNK % UNROLL == 0, "one entry per lane per chunk");
    constexpr int VROWS = PACKED ? 1 : UNROLL;
    constexpr int ROWF = ITERS * LPR * 4;   // floats per staged row in LDS
    static_assert(GROUPS == GROUPS_ && ROWF == ROWF_, "sizes of the block of LDS");
    float (*s_part)[2][ROWF] = reinterpret_cast<float (*)[2][ROWF]>(s_arena);
    // FUSED: table row and column of the run that leaves each chunk to the right
    float (*s_x)[FUSED ? ROWF : 4] = reinterpret_cast<float (*)[FUSED ? ROWF : 4]>(s_arena + GROUPS * 2 * ROWF * 4);
    int32_t *s_small = reinterpret_cast<int32_t *>(s_arena + (GROUPS * 2 * ROWF + (FUSED ? GROUPS * ROWF : 4)) * 4);
    int32_t *s_info = s_small, *s_seg_last = s_small + GROUPS, *s_col_last = s_small + 2 * GROUPS;

    const int lig = threadIdx.x % LPR, grp = group_index<LPR>();
    const int pk_sh = PACKED ? 31 - __clz(ld_src) : 0;
    const int32_t tile0 = e_begin + block * TILE;
    const int32_t ec0 = tile0 + grp * CHUNK;
    const int32_t ec1 = min(ec0 + CHUNK, e_end);

    int info = 0;
    if (ec0 < e_end) {
        const int n = ec1 - ec0;
        int32_t meta = 0;                                  // 0: row 0, a safe address
        int32_t colv = 0;                                  // FUSED: the column of this lane's entry
        bool right_head = true;                            // the entry after the chunk heads a segment
        if constexpr (RAW) {
            if (lig < CHUNK && ec0 + lig < ec1) {
                const int32_t e = ec0 + lig;
                const int32_t pos = packed[e], kc = seg_id[e], kp = e > 0 ? seg_id[e - 1] : -1;
                const int32_t row = pos / 3;
                meta = (row << 2) | (kc != kp ? 2 : 0) | (pos - 3 * row == 2 ? 1 : 0);
                colv = kc;
            }
            if (ec1 < e_end) right_head = seg_id[ec1] != seg_id[ec1 - 1];
        } else {
            if (lig < CHUNK && ec0 + lig < ec1) meta = packed[ec0 + lig];
            if (FUSED && lig < CHUNK && ec0 + lig < ec1)
                colv = fu.cols_sorted ? fu.cols_sorted[ec0 + lig] : fu.touched_cols[seg_id[ec0 + lig]];
            if (ec1 < e_end) right_head = (packed[ec1] & 2) != 0;
        }
        int32_t o1 = 0, o2 = 0;                            // SRC: the other two columns of this lane's entry's row
        if constexpr (SEMI) {
            if (lig < CHUNK && ec0 + lig < ec1) {
                const int32_t *cx = sr.colidx + 3 * (int64_t)((uint32_t)meta >> 2);
                const int32_t c0 = cx[0], c1 = cx[1], c2 = cx[2];
                const bool rel = ec0 + lig >= split;
                o1 = (meta & 1) || rel ? c0 : c1;
                o2 = (meta & 1) ? c1 : c2;
            }
        }
        const bool skip = SUMS && ec0 + lig >= sums_from && (meta >> 2) >= sec.n_pos;   // (no source row is stored)
        const int32_t my_row = skip ? sec.n_pos - 1 : meta >> 2;   // (... for loads without a branch: the last one that is)
        // (groups of whole wavefronts: each lane fetches its own entry's; the others a batch's at a time, as a shuffle for each
        // entry would keep the LDS units busier than those loads keep the caches)
        constexpr bool LANE_COEF = PACKED && LPR == 64;
        float my_coef = 0.f;
        if (LANE_COEF) my_coef = src_b[my_row];
        Acc<ITERS> xcur;                                   // FUSED: table row of the run that is being summed
        int at = 0;                                        // ... and the entry of the chunk it begins with
        xcur.zero();
        // entries of the chunk that head a segment, and tail entries
        const int gsh = (int)(threadIdx.x & 63) & ~(LPR - 1);
        const uint64_t b_head = __ballot((meta & 2) != 0), b_tail = __ballot((meta & 1) != 0);
        using Bits = std::conditional_t<(CHUNK > 32), uint64_t, uint32_t>;
        const Bits heads = (Bits)(b_head >> gsh), tails = (Bits)(b_tail >> gsh);
        // SUMS: ... and those whose source row is stored
        const Bits stored = SUMS ? (Bits)(__ballot(!skip) >> gsh) : 0;
        const bool first_open = (ec0 > e_begin) && !(heads & 1u);
        const bool right_open = (ec1 < e_end) && !right_head;
        int32_t cur_seg = RAW ? 0 : seg_id[ec0];
        int nflush = 0;
        Acc<ITERS> acc;
        acc.zero();

        auto flush = [&](bool last_run) {
            const bool open_left = (nflush == 0) && first_open;
            const bool open_right = last_run && right_open;
            if (!open_left && !open_right) {
                if constexpr (FUSED)
                    apply_update<LPR, ITERS, SUMS>(fused_row(fu, of_lane<LPR>(colv, at), ld_tab), d4, lig, xcur, acc, fu.lr, fu.mode, fu.stream);
                else
                    store_row_stream<LPR, ITERS>(out_rows + (int64_t)cur_seg * ld_out, d4, lig, acc);
            } else {
                const int slot = open_left ? 0 : 1;
#pragma unroll
                for (int it = 0; it < ITERS; ++it)
                    st4(&s_part[grp][slot][(lig + it * LPR) * 4], acc.v[it]);
                if (open_left) {
                    info |= HAS_FIRST | (open_right ? FIRST_CONT : 0);
                } else {
                    info |= HAS_LAST;
                    if (lig == 0) s_seg_last[grp] = cur_seg;
                    if constexpr (FUSED) {   // the run began in this chunk: its table row is already here
#pragma unroll
                        for (int it = 0; it < ITERS; ++it) st4(&s_x[grp][(lig + it * LPR) * 4], xcur.v[it]);
                        if (lig == (at & (LPR - 1))) s_col_last[grp] = colv;
                    }
                }
            }
            ++nflush;
        };

        auto walk = [&](auto stream) {
        constexpr bool STREAM = decltype(stream)::value;
        for (int j0 = 0; j0 < n; j0 += UNROLL) {
            Acc<ITERS> v[VROWS];
            Acc<ITERS> va[SRC != SRC_STORED ? UNROLL : 1], vb[SRC != SRC_STORED ? UNROLL : 1];
            Acc<ITERS> xr[FUSED ? UNROLL : 1];
            const Bits hb = heads >> j0, tb = tails >> j0;
            uint8_t sb[UNROLL][ITERS];
            float cf[UNROLL];
            // all loads of the batch go out together: entries past the end of the chunk carry meta 0, i.e. row 0
            if constexpr (FUSED) {   // a run begins here: its table row comes along with its first source row
                int32_t cu[UNROLL];
#pragma unroll
                for (int u = 0; u < UNROLL; ++u) cu[u] = of_lane<LPR>(colv, j0 + u);
#pragma unroll
                for (int u = 0; u < UNROLL; ++u)
                    // (a row of a table beyond the caches is read once here and rewritten: past them)
                    if (hb >> u & 1) load_row<LPR, ITERS, STREAM>(fused_row(fu, cu[u], ld_tab), d4, lig, xr[u]);
            }
            if (!SUMS || (stored >> j0 & (((Bits)1 << UNROLL) - 1))) {
                uint32_t row[UNROLL];
#pragma unroll
                for (int u = 0; u < UNROLL; ++u) row[u] = (uint32_t)of_lane<LPR>(my_row, j0 + u);
#pragma unroll
                for (int u = 0; u < UNROLL; ++u) {
                    if constexpr (PACKED) {
                        // (records of 1 << pk_sh bytes: a shift and an add give the address)
                        const uint8_t *pb = reinterpret_cast<const uint8_t *>(src_a) + pk_off + ((uint64_t)row[u] << pk_sh);
#pragma unroll
                        for (int it = 0; it < ITERS; ++it) sb[u][it] = pb[min(lig + it * LPR, d4 - 1)];
                        if (!LANE_COEF) cf[u] = src_b[row[u]];
                    } else if constexpr (SEMI) {
                        const int32_t c1 = of_lane<LPR>(o1, j0 + u), c2 = of_lane<LPR>(o2, j0 + u);
                        load_row<LPR, ITERS, true>(sr.G + (uint64_t)row[u] * (uint32_t)ld_tab, d4, lig, v[u]);
                        load_row<LPR, ITERS>(sr.X + (uint64_t)(uint32_t)c1 * (uint32_t)ld_tab, d4, lig, va[u]);
                        if (SRC != SRC_SEMIRING + SR_ROTATE)
                            load_row<LPR, ITERS>(sr.X + (uint64_t)(uint32_t)c2 * (uint32_t)ld_tab, d4, lig, vb[u]);
                    } else {   // entries before `split` read src_a, the rest src_b (entity vs relation columns)
                        load_row<LPR, ITERS>((ec0 + j0 + u < split ? src_a : src_b) + (uint64_t)row[u] * (uint32_t)ld_src, d4, lig, v[u]);
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) {
                const int jj = j0 + u;
                if (jj < n) {
                    if (hb >> u & 1) {
                        if (jj > 0) {
                            flush(false);
                            ++cur_seg;
                            acc.zero();
                        }
                        if constexpr (FUSED) { xcur = xr[u]; at = jj; }
                    }
                    if constexpr (PACKED) {
                        // the dense row the forward pass would have stored is +c, -c or 0 per element, and a tail
                        // entry subtracts it: one fused multiply-add per element with the element's sign
                        const float m = LANE_COEF ? __int_as_float(of_lane<LPR>(__float_as_int(my_coef), jj)) : cf[u];
                        const float c = (tb >> u & 1) ? -m : m;
#pragma unroll
                        for (int it = 0; it < ITERS; ++it) {
                            const unsigned b = sb[u][it];   // (shift up, arithmetic shift down: sign-extends two bits)
                            acc.v[it].x = __builtin_fmaf(c, (float)((int)(b << 30) >> 30), acc.v[it].x);
                            acc.v[it].y = __builtin_fmaf(c, (float)((int)(b << 28) >> 30), acc.v[it].y);
                            acc.v[it].z = __builtin_fmaf(c, (float)((int)(b << 26) >> 30), acc.v[it].z);
                            acc.v[it].w = __builtin_fmaf(c, (float)((int)(b << 24) >> 30), acc.v[it].w);
                        }
                    } else if constexpr (SEMI) {
                        Acc<ITERS> tm;
                        tm.v[0] = semiring_term<SRC - SRC_SEMIRING>(v[u].v[0], va[u].v[0], vb[u].v[0], (tb >> u & 1) != 0);
                        acc.add(tm);
                    } else if (!SUMS || (stored >> jj & 1)) {
                        // (a sum or a difference, rounded once either way)
                        const float sg = (tb >> u & 1) ? -1.0f : 1.0f;
#pragma unroll
                        for (int it = 0; it < ITERS; ++it) {
                            acc.v[it].x = __builtin_fmaf(sg, v[u].v[it].x, acc.v[it].x); acc.v[it].y = __builtin_fmaf(sg, v[u].v[it].y, acc.v[it].y);
                            acc.v[it].z = __builtin_fmaf(sg, v[u].v[it].z, acc.v[it].z); acc.v[it].w = __builtin_fmaf(sg, v[u].v[it].w, acc.v[it].w);
                        }
                    }
                }
            }
        }
        };
        // (the choice lies outside the loop: beside each load it made every head wait for all loads before it)
        if constexpr (FUSED) {
            if (fu.stream) walk(std::true_type{});
            else walk(std::false_type{});
        } else {
            walk(std::false_type{});
        }
        flush(true);
    }
    if (lig == 0) s_info[grp] = info;
    __syncthreads();

    stitch_runs<LPR, ITERS, GROUPS, FUSED, true>(info, s_part, s_info, s_seg_last, s_x, s_col_last, partials + (int64_t)block * 2 * ld_out,
                                           out_rows, ld_out, d4, ld_tab, fu);
}

// RIDE: 1 the first scatter pass of the next batch's sort comes along, 2 its histogram pass of the second digit,
// 3 as 2, and the sums of TransR's partial dL/dM_r matrices come along, 4 the first kernel of the next batch's
// build when that sort is a large one (nothing after this launch reads the A arrays it overwrites).
// MANY: a workgroup takes column slices of LPR float4 in turn, from blockIdx.y on: most tiles end no crossing run, so a
// workgroup for each of a wide row's slices mostly starts to find that out once more (16 slices of 9,216 tiles: 105 us as 16
// workgroups a tile, 65 as four).  A kernel of its own: the loop costs the others registers (four float4 per lane: 102 and 132
// with the update fused, four and three wavefronts per SIMD; 65 and 110 without, seven and four).
// Bound to eight wavefronts per SIMD, and without the wait for all arguments at the start, as most of its workgroups only look at
// a few words and end: 260,000 positives and as many negatives, d = 200: 34.3 us, with seven 40.0.
template <int LPR, int ITERS, int CHUNK, bool FUSED, int RIDE, bool MANY = false>
__global__ __launch_bounds__(kThreads, MANY && !FUSED ? 8 : 1) void k_seg_fixup(const int32_t *__restrict__ packed,
                                                        const int32_t *__restrict__ seg_id,
                                                        const int32_t *__restrict__ seg_ptr, int32_t e_begin,
                                                        int32_t e_end, int d4, float *__restrict__ out_rows,
                                                        int ld_out, const float *__restrict__ partials, FusedArgs fu,
                                                        SegSecond sec, ScatterAhead sa, HistAhead ha, DmRide dm,
                                                        EmitAhead ea)
{
    int block = (int)blockIdx.x;
    if constexpr (!MANY) STX_TOGETHER(ha.ntiles, sa.ntiles, dm.blocks, sec.first_block, gridDim.x, gridDim.y, packed, seg_id, seg_ptr, e_begin, e_end, d4, ld_out, partials);
    if constexpr (RIDE == 4) {
        if (block < ea.ntiles) {      // uniform in the workgroup
            emit_body<kBigSortItems, false, true, false>(block, ea.ntiles, ea.args);
            return;
        }
        block -= ea.ntiles;
    }
    if constexpr (RIDE == 3) {
        if (block < dm.blocks) {      // uniform in the workgroup
            const int slices = (dm.args.k * dm.args.d + kDmFixupSlice - 1) / kDmFixupSlice;
            transr_dm_fixup_body(block / slices, block % slices, dm.args);
            return;
        }
        block -= dm.blocks;
    }
    if constexpr (RIDE == 1) {
        if (block < sa.ntiles) {      // uniform in the workgroup
            scatter_body<true, false, kSortItems>(block, sa.args);
            return;
        }
        block -= sa.ntiles;
    }
    if constexpr (RIDE == 2 || RIDE == 3) {
        if (block < ha.ntiles) {
            hist_body<kSortItems>(block, ha.args.keys, ha.args.nnz, ha.args.shift, ha.args.radix, ha.args.table);
            return;
        }
        block -= ha.ntiles;
    }
    // The tiles are taken from the last one down: the relation columns sort last and own the longest runs (one
    // relation has a fifth of a batch's rows), whose closing workgroups add up the most partial rows; started
    // last, after the other workgroups have come and gone, their chains would set the time of the launch.
    block = ((int)gridDim.x - (RIDE == 1 ? sa.ntiles : RIDE == 2 ? ha.ntiles : RIDE == 3 ? ha.ntiles + dm.blocks
                               : RIDE == 4 ? ea.ntiles : 0)) - 1 - block;
    if (block >= sec.first_block) {   // uniform in the workgroup
        block -= sec.first_block;
        e_begin = sec.e_begin; e_end = sec.e_end;
        out_rows = sec.out_rows; partials = sec.partials;
        fu.table_b = sec.fused_table; fu.mode = sec.fused_mode;
    }
    const int ld_tab = d4 * 4;
    // (Launches with a ride hold whole rows, but a step of 1,024 positives at d = 32 takes 19.47 us without this test in them
    // and 19.31 with it; of 262,144 x 5 at d = 128, ride 4, 569.5 without and 570.6 with it.)
    if (RIDE != 0 && RIDE != 4 && gridDim.y > 1) {
        const int c4 = (int)blockIdx.y * LPR;
        d4 = min(LPR, d4 - c4);
        if (out_rows) out_rows += 4 * c4;
        partials += 4 * c4;
        if (fu.table) fu.table += 4 * c4;
        if (fu.table_b) fu.table_b += 4 * c4;
    }
    constexpr int GROUPS = kThreads / LPR;
    constexpr int ROWF = ITERS * LPR * 4;
    constexpr int TILE = GROUPS * CHUNK;
    static_assert(TILE <= kThreads, "one thread per entry of the tile in the head search");
    __shared__ float s_sum[GROUPS][ROWF];
    const int32_t j = block;
    if (j == 0) return;                                         // tile 0 never ends a crossing run
    const int32_t tile0 = e_begin + j * TILE;
    if (tile0 >= e_end) return;
    const int32_t tile1 = min(tile0 + TILE, e_end);
    const int32_t e = tile0 + (int32_t)threadIdx.x;
    // everything the decision needs is fetched in one round trip
    const int32_t m_first = packed[tile0];
    const int32_t m_mine = (e > tile0 && e < tile1) ? packed[e] : 0;
    const int32_t m_next = tile1 < e_end ? packed[tile1] : 2;
    const int32_t seg = seg_id[tile0];
    if (m_first & 2) return;                                    // the tile starts a new segment: nothing crosses in
    const int any_head = __syncthreads_or((m_mine >> 1) & 1);
    const bool closes = any_head || (m_next & 2);
    if (!closes) return;                                        // the run goes on; a later tile finishes it

    const int lig = threadIdx.x % LPR, grp = threadIdx.x / LPR;
    const int32_t col = FUSED ? fu.touched_cols[seg] : 0;
    const int32_t j0 = (seg_ptr[seg] - e_begin) / TILE;         // tile in which the run began
    const int n = j - j0 + 1;                                   // partial rows: (j0, slot 1), (j0+1 .. j, slot 0)
    auto sum_row = [&](const FusedArgs &fa, float *rows, const float *part, int width4) {
        Acc<ITERS> xrow;                                        // FUSED: the table row, fetched beside the partial rows
        if (FUSED && grp == 0) {
            if (fa.stream) load_row<LPR, ITERS, true>(fused_row(fa, col, ld_tab), width4, lig, xrow);
            else load_row<LPR, ITERS>(fused_row(fa, col, ld_tab), width4, lig, xrow);
        }
        const int per = (n + GROUPS - 1) / GROUPS;
        const int lo = min(grp * per, n), hi = min(lo + per, n);
        Acc<ITERS> acc;
        acc.zero();
        constexpr int FU = ITERS == 1 ? 8 : 2;
        // NB partial rows in flight, added in tile order (past the last one: it again, not added)
        auto rows_at = [&](auto nb, int q) {
            constexpr int NB = decltype(nb)::value;
            Acc<ITERS> v[NB];
#pragma unroll
            for (int u = 0; u < NB; ++u) {
                const int t = min(q + u, hi - 1);
                load_row<LPR, ITERS>(part + ((int64_t)(j0 + t) * 2 + (t == 0 ? 1 : 0)) * ld_out, width4, lig, v[u]);
            }
#pragma unroll
            for (int u = 0; u < NB; ++u)
                if (q + u < hi) acc.add(v[u]);
        };
        int q = lo;
        for (; q + FU <= hi; q += FU) {
            Acc<ITERS> v[FU];
#pragma unroll
            for (int u = 0; u < FU; ++u)
                load_row<LPR, ITERS>(part + ((int64_t)(j0 + q + u) * 2 + (q + u == 0 ? 1 : 0)) * ld_out, width4, lig, v[u]);
#pragma unroll
            for (int u = 0; u < FU; ++u) acc.add(v[u]);
        }
        if (hi - q > 2) rows_at(std::integral_constant<int, FU>{}, q);
        else if (hi - q == 2) rows_at(std::integral_constant<int, 2>{}, q);
        else if (hi > q) rows_at(std::integral_constant<int, 1>{}, q);
#pragma unroll
        for (int it = 0; it < ITERS; ++it) st4(&s_sum[grp][(lig + it * LPR) * 4], acc.v[it]);
        __syncthreads();
        if (grp == 0) {
            const int used = (n + per - 1) / per;               // groups that had at least one row
            for (int g = 1; g < used; ++g) {
                Acc<ITERS> v;
#pragma unroll
                for (int it = 0; it < ITERS; ++it) v.v[it] = ld4(&s_sum[g][(lig + it * LPR) * 4]);
                acc.add(v);
            }
            if constexpr (FUSED) apply_update<LPR, ITERS>(fused_row(fa, col, ld_tab), width4, lig, xrow, acc, fa.lr, fa.mode, fa.stream);
            else store_row<LPR, ITERS>(rows + (int64_t)seg * ld_out, width4, lig, acc);
        }
    };
    if constexpr (MANY) {
        static_assert(ITERS == 1 && RIDE == 0, "slices of one float4 per lane");
        for (int c4 = (int)blockIdx.y * LPR; c4 < d4; c4 += (int)gridDim.y * LPR) {
            FusedArgs fa = fu;
            if (fa.table) fa.table += 4 * c4;
            if (fa.table_b) fa.table_b += 4 * c4;
            if (c4 != (int)blockIdx.y * LPR) __syncthreads();   // the slice before this one has been read out of LDS
            sum_row(fa, out_rows + 4 * c4, partials + 4 * c4, min(LPR, d4 - c4));
        }
    } else {
        if (RIDE == 0 && gridDim.y > 1) {                       // column slices, as in k_seg_reduce
            const int c4 = (int)blockIdx.y * LPR;
            d4 = min(LPR, d4 - c4);
            if (out_rows) out_rows += 4 * c4;
            partials += 4 * c4;
            if (fu.table) fu.table += 4 * c4;
            if (fu.table_b) fu.table_b += 4 * c4;
        }
        sum_row(fu, out_rows, partials, d4);
    }
}

// Row update for every segment s (column c = touched_cols[s]):
//   c <  n_split : table_a row c            -= lr * grad_rows[s]   (width 4*d4_a, mode_a)
//   c >= n_split : table_b row c - n_split  -= lr * grad_rows[s]   (width 4*d4_b, mode 0), if table_b
//                  table_w row c - n_split  -= lr * w_rows[s]      (width 4*d4_a, mode_w), if table_w
// Each product and each difference is rounded once.  mode 1: then keep the fractional part (TorusE,
// Sec. 4.6).  mode 2: then rescale the row to unit length (TransH normals).
template <int LPR, int ITERS>
__device__ inline void sgd_row(float *__restrict__ row, const float *__restrict__ grad, int d4, int lig, float lr,
                               int mode)
{
    Acc<ITERS> x, g;
    load_row<LPR, ITERS>(row, d4, lig, x);
    load_row<LPR, ITERS>(grad, d4, lig, g);
    float ss = 0.f;
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
        float *xv = &x.v[it].x;
        const float *gv = &g.v[it].x;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float step = lr * gv[q];
            float nv = xv[q] - step;
            if (mode == 1) {
                nv = nv - floorf(nv);
                if (nv >= 1.0f) nv = 0.0f;
            }
            xv[q] = nv;
            ss += lig + it * LPR < d4 ? nv * nv : 0.f;
        }
    }
    if (mode == 2) {
        ss = group_sum<LPR>(ss);
        if (ss > 0.f) {
            const float inv = 1.0f / sqrtf(ss);
#pragma unroll
            for (int it = 0; it < ITERS; ++it) {
                x.v[it].x *= inv; x.v[it].y *= inv; x.v[it].z *= inv; x.v[it].w *= inv;
            }
        }
    }
    store_row<LPR, ITERS>(row, d4, lig, x);
}

template <int LPR, int ITERS>
__global__ __launch_bounds__(kThreads) void k_sgd_rows(const int32_t *__restrict__ touched_cols,
                                                       const int32_t *__restrict__ n_touched,
                                                       float *__restrict__ table_a, int d4_a, int mode_a,
                                                       int32_t n_split, float *__restrict__ table_b, int d4_b,
                                                       float *__restrict__ table_w, int mode_w,
                                                       const float *__restrict__ grad_rows,
                                                       const float *__restrict__ w_rows, int ld, float lr, int stream)
{
    constexpr int GROUPS = kThreads / LPR;
    const int lig = threadIdx.x % LPR, grp = threadIdx.x / LPR;
    const int32_t U = n_touched[0];
    if (!table_b && !table_w) {
        // One table (TransE / TorusE): a group takes four consecutive segments per turn so that the four
        // column ids, then the eight rows (table + gradient), are in flight together.
        constexpr int UB = ITERS <= 2 ? 4 : 2;
        auto walk = [&](auto past) {
        constexpr bool STREAM = decltype(past)::value;
        for (int64_t s0 = ((int64_t)blockIdx.x * GROUPS + grp) * UB; s0 < U; s0 += (int64_t)gridDim.x * GROUPS * UB) {
            int32_t col[UB];
#pragma unroll
            for (int u = 0; u < UB; ++u) col[u] = touched_cols[min(s0 + u, (int64_t)U - 1)];
            Acc<ITERS> x[UB], g[UB];
#pragma unroll
            for (int u = 0; u < UB; ++u) {
                load_row<LPR, ITERS, STREAM>(table_a + (int64_t)col[u] * d4_a * 4, d4_a, lig, x[u]);
                load_row<LPR, ITERS, true>(grad_rows + min(s0 + u, (int64_t)U - 1) * ld, d4_a, lig, g[u]);
            }
#pragma unroll
            for (int u = 0; u < UB; ++u) {
                if (s0 + u < U && col[u] < n_split) {
#pragma unroll
                    for (int it = 0; it < ITERS; ++it) {
                        float *xv = &x[u].v[it].x;
                        const float *gv = &g[u].v[it].x;
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            float step = lr * gv[q];
                            float nv = xv[q] - step;
                            if (mode_a == 1) {
                                nv = nv - floorf(nv);
                                if (nv >= 1.0f) nv = 0.0f;
                            }
                            xv[q] = nv;
                        }
                    }
                    float *pr = table_a + (int64_t)col[u] * d4_a * 4;
#pragma unroll
                    for (int it = 0; it < ITERS; ++it) {
                        const int j = lig + it * LPR;
                        if (j < d4_a) {
                            if (STREAM) st4_stream(pr + 4 * j, x[u].v[it]);
                            else st4(pr + 4 * j, x[u].v[it]);
                        }
                    }
                }
            }
        }
        };
        if (stream) walk(std::true_type{});
        else walk(std::false_type{});
        return;
    }
    for (int64_t s = (int64_t)blockIdx.x * GROUPS + grp; s < U; s += (int64_t)gridDim.x * GROUPS) {
        const int32_t col = touched_cols[s];
        if (col < n_split) {
            sgd_row<LPR, ITERS>(table_a + (int64_t)col * d4_a * 4, grad_rows + s * ld, d4_a, lig, lr, mode_a);
        } else {
            const int64_t r = col - n_split;
            if (table_b) sgd_row<LPR, ITERS>(table_b + r * d4_b * 4, grad_rows + s * ld, d4_b, lig, lr, 0);
            if (table_w) sgd_row<LPR, ITERS>(table_w + r * d4_a * 4, w_rows + s * ld, d4_a, lig, lr, mode_w);
        }
    }
}

// ---- dispatch --------------------------------------------------------------------------------------
// A product is cut into short chunks of 16 entries a lane group (the serial walk of every group is short: latency) or long ones
// (fewer partial rows, more rows of a run per sum: bandwidth; with fewer than 32 lanes a group there is one length).  The same
// line for every way of calling, as it decides the order of the sums.
//
// Sums that round (dense rows; the L1 kinds' when a mean over a number of pairs that is no power of two, or weights of relations,
// scale them) keep short chunks up to a million entries: a training run that adds in another order soon decides some hinge the
// other way.  TransR's round as well, but its rows come out of products of bfloat16 operands, whose roundings are 2^15 times
// larger: its line is 3,600 tiles, 460,800 entries of up to 128 floats and 230,400 of more.  Whole steps with short and with long
// chunks, three negatives, 1,000 relations: d = k = 128: 189 and 188 us at 300,000 entries, 243 and 241 at 420,000, 272 and 269 at
// 510,000, 416 and 413 at 900,000; d = k = 256: 506 and 509 at 180,000, 609 and 609 at 240,000, 726 and 719 at 360,000, 1,446 and
// 1,429 at 900,000; relation columns in a product of their own, d = 128, k = 256: 334 and 340 at 60,000, 699 and 693 at 180,000,
// 845 and 834 at 240,000, 1,635 and 1,608 at 510,000.
// Exact sums have the same bits either way.  us of an L1 step with short and with long chunks, 30,000 entities: d = 128: 63.4 and
// 64.2 at 300,000 entries, 78.1 and 76.1 at 420,000, 111.8 and 108.1 at 720,000; d = 200: 71.7 and 74.6 at 240,000, 82.2 and 82.2 at
// 300,000, 104.1 and 98.9 at 420,000, 178 and 164 at 900,000; two slices a row, d = 512: 82.5 and 85.4 at 120,000, 103 and 98.5 at
// 180,000; four, d = 1024: 85.9 and 89.2 at 60,000, 127 and 123 at 120,000.  (Products alone, without the last kernel of the build
// in their launch, meet their line at half as many entries: d = 200: 14.2 and 16.5 at 120,000, 17.9 and 17.2 at 180,000.)
static bool short_chunks(const stx_ctx *c, SegRows kind, int64_t n, int slices, int tile)
{
    if (kind == SegRows::packed_exact) return n * slices <= 300000;
    return n <= (c->cfg.model == STX_TRANSR ? 3600 * tile : 1 << 20);
}

template <int LPR, int ITERS>
static void seg_go(stx_ctx *c, const stx_incidence *inc, int32_t e_begin, int32_t e_end, const float *src_a,
                   const float *src_b, int32_t split, int ld_src, int width, float *out_rows, int ld_out,
                   SegRows kind, const FusedArgs *fused, const SegSecondHost *second)
{
    const bool packed_src = kind != SegRows::dense;
    constexpr int CH_LONG = LPR == 64 ? 64 : (LPR < 32 ? LPR : 32), CH_SHORT = LPR < 16 ? LPR : 16;
    constexpr int GROUPS = kThreads / LPR;
    const bool small = short_chunks(c, kind, e_end - e_begin, ITERS, GROUPS * CH_SHORT);
    const int tile = GROUPS * (small ? CH_SHORT : CH_LONG);
    const int ntiles1 = (e_end - e_begin + tile - 1) / tile;
    SegSecond sec{0x7fffffff, 0, 0, nullptr, nullptr, nullptr, nullptr, 0, 0};
    int ntiles = ntiles1;
    if (second) sec.n_pos = second->n_pos;
    if (second && second->e_end > second->e_begin) {
        sec = SegSecond{ntiles1, second->e_begin, second->e_end, second->src, second->out_rows,
                        c->partials + (int64_t)ntiles1 * 2 * ld_out, second->fused_table, second->fused_mode, second->n_pos};
        ntiles += (second->e_end - second->e_begin + tile - 1) / tile;
    }
    const FusedArgs fu = fused ? *fused : FusedArgs{nullptr, nullptr, 0, nullptr, nullptr, 0.f, 0, 0};
    // The last kernel of this batch's build, when it was left waiting (stx_train_step), runs in the launch of a
    // fused product of one float4 per lane, and so does the sum of the loss; a product that cannot take them runs
    // after them.  The stages of the next batch's build that are due ride too, one per launch.
    const bool raw_now = fused && ITERS == 1 && c->segw.armed && c->sorted_inc == inc;
    if (c->segw.armed && !raw_now) launch_seg_write_late(c);
    const SegWriteRide no_segw{};
    const SegWriteRide segw = raw_now ? SegWriteRide{c->segw.args, c->segw.ntiles, c->segw.use_map ? 1 : 0,
                                                     c->loss_partials, c->fin_n, c->fin_scale, c->fin_loss}
                                      : no_segw;
    const int segw_blocks = segw.ntiles + (segw.fin_n > 0 ? 1 : 0);
    if (raw_now) { c->segw.armed = false; c->fin_n = 0; }
    EmitAhead r_emit{};
    ScatterAhead r_scat{}, f_scat{};
    HistAhead f_hist{};
    if (raw_now) {
        // (the scatter pass writes one of the sort's buffers: not in this launch if that is the one this product
        // reads, as after a sort of one or three passes; the fix-up launch reads neither)
        if (!c->ahead.scatter_ok || c->ahead.sargs.keys_out != segw.args.keys) r_scat = take_scatter_ahead(c);
        if (r_scat.ntiles == 0) r_emit = take_emit_ahead(c);
        if (ntiles > 1) {   // a fix-up launch follows
            f_hist = take_hist_ahead(c);
            if (f_hist.ntiles == 0) f_scat = take_scatter_ahead(c);
        }
    }
    // TransR's dL/dM_r product, left by the backward pass: along with the launch that also takes the scatter pass
    // (the steady state of stx_train_step), its sums along with the fix-up launch; ahead of any other launch.
    DmRide r_dm{}, f_dm{};
    bool dm_fixup_after = false;
    if (c->dm_ride.armed) {
        if (raw_now && r_scat.ntiles && !packed_src && LPR <= 32) {
            c->dm_ride.armed = false;
            r_dm = DmRide{c->dm_ride.args, c->dm_ride.items};
            if (c->dm_ride.fixup) {
                const DmArgs &da = c->dm_ride.args;
                if (ntiles > 1 && f_hist.ntiles)
                    f_dm = DmRide{da, da.n_fix * ((da.k * da.d + kDmFixupSlice - 1) / kDmFixupSlice)};
                else
                    dm_fixup_after = true;
            }
        } else {
            launch_transr_dm_late(c);
        }
    }
    // the first kernel of a large next build: in the fix-up launch, the last one of the step
    EmitAhead f_emit{};
    if (fused && ITERS == 1 && ntiles > 1 && c->ahead.armed && c->ahead.late_only) f_emit = take_emit_ahead(c, true);
    const int r_blocks = r_emit.ntiles + r_scat.ntiles + r_dm.blocks,
              f_blocks = f_scat.ntiles + f_hist.ntiles + f_dm.blocks + f_emit.ntiles;
    // Wide rows (more than one float4 per lane) run as column slices of the one-float4 kernels: more rows in
    // flight per lane and ITERS times the workgroups.  The unit-length rescale needs whole rows.
    const bool sums = sec.n_pos > 0 && !packed_src;        // (TransH, TransR)
    const bool whole_rows = fused && (fu.mode == 2 || sec.fused_mode == 2);
    if (ITERS > 1 && !whole_rows) {
        const dim3 grid((unsigned)ntiles, (unsigned)ITERS);
#define STX_SLICED_R(P, CH, F, S)                                                                               \
    hipLaunchKernelGGL((k_seg_reduce<LPR, 1, P, CH, F, 0, SRC_STORED, kThreads, S>), grid, dim3(kThreads), 0, c->stream, \
                       inc->at_packed, inc->at_seg_id, e_begin, e_end, src_a, src_b, split, ld_src, width / 4,  \
                       out_rows, ld_out, c->partials, fu, sec, no_segw, r_emit, r_scat, r_dm)
#define STX_SLICED(P, CH, F)                                                                                    \
    do {                                                                                                        \
        {                                                                                                       \
            ProfScope prof(c, "k_seg_reduce");                                                                  \
            if (sums) STX_SLICED_R(P, CH, F, !P); else STX_SLICED_R(P, CH, F, false);                           \
        }                                                                                                       \
        if (ntiles > 1) {                                                                                       \
            ProfScope prof(c, "k_seg_fixup");                                                                   \
            hipLaunchKernelGGL((k_seg_fixup<LPR, 1, CH, F, 0>), grid, dim3(kThreads), 0, c->stream,             \
                               inc->at_packed, inc->at_seg_id, inc->at_seg_ptr, e_begin, e_end, width / 4,      \
                               out_rows, ld_out, c->partials, fu, sec, f_scat, f_hist, f_dm, f_emit);           \
        }                                                                                                       \
    } while (0)
#define STX_SLICED2(P, CH) do { if (fused) STX_SLICED(P, CH, true); else STX_SLICED(P, CH, false); } while (0)
        if (packed_src) { if (small) STX_SLICED2(true, CH_SHORT); else STX_SLICED2(true, CH_LONG); }
        else            { if (small) STX_SLICED2(false, CH_SHORT); else STX_SLICED2(false, CH_LONG); }
#undef STX_SLICED2
#undef STX_SLICED
#undef STX_SLICED_R
        return;
    }
#define STX_SEG_R(P, CH, F, R)                                                                                  \
    do { if (sums) STX_SEG_RS(P, CH, F, R, !P); else STX_SEG_RS(P, CH, F, R, false); } while (0)
#define STX_SEG_RS(P, CH, F, R, S)                                                                              \
    hipLaunchKernelGGL((k_seg_reduce<LPR, ITERS, P, CH, F, (F && ITERS == 1 && !(R == 5 && (P || LPR > 32))) ? R : 0, SRC_STORED, kThreads, S>), \
                       dim3(ntiles + segw_blocks + r_blocks), dim3(kThreads), 0, c->stream, segw.args.pay,      \
                       segw.args.keys, e_begin, e_end, src_a, src_b, split, ld_src, width / 4,        \
                       out_rows, ld_out, c->partials, fu, sec, segw, r_emit, r_scat, r_dm)
#define STX_SEG_0(P, CH, F, S)                                                                                  \
    hipLaunchKernelGGL((k_seg_reduce<LPR, ITERS, P, CH, F, 0, SRC_STORED, kThreads, S>), dim3(ntiles), dim3(kThreads), 0, \
                       c->stream, inc->at_packed, inc->at_seg_id, e_begin, e_end, src_a, src_b, split, ld_src,  \
                       width / 4, out_rows, ld_out, c->partials, fu, sec, no_segw, r_emit, r_scat, r_dm)
#define STX_SEG_F(CH, F, R)                                                                                     \
    hipLaunchKernelGGL((k_seg_fixup<LPR, ITERS, CH, F, (F && ITERS == 1 && !(R == 3 && LPR > 32)) ? R : 0>), dim3(ntiles + f_blocks), \
                       dim3(kThreads), 0, c->stream, inc->at_packed, inc->at_seg_id, inc->at_seg_ptr, e_begin,  \
                       e_end, width / 4, out_rows, ld_out, c->partials, fu, sec, f_scat, f_hist, f_dm, f_emit)
#define STX_SEG(P, CH, F)                                                                                       \
    do {                                                                                                        \
        {                                                                                                       \
            ProfScope prof(c, "k_seg_reduce");                                                                  \
            if (F && ITERS == 1 && raw_now && r_scat.ntiles && r_dm.blocks) STX_SEG_R(P, CH, F, 5);             \
            else if (F && ITERS == 1 && raw_now && r_scat.ntiles) STX_SEG_R(P, CH, F, 3);                       \
            else if (F && ITERS == 1 && raw_now && r_emit.ntiles && r_emit.args.rc.cur) STX_SEG_R(P, CH, F, 4); \
            else if (F && ITERS == 1 && raw_now && r_emit.ntiles) STX_SEG_R(P, CH, F, 2);                       \
            else if (F && ITERS == 1 && raw_now) STX_SEG_R(P, CH, F, 1);                                        \
            else if (sums) STX_SEG_0(P, CH, F, !P);                                                             \
            else STX_SEG_0(P, CH, F, false);                                                                    \
        }                                                                                                       \
        if (ntiles > 1) {                                                                                       \
            ProfScope prof(c, "k_seg_fixup");                                                                   \
            if (F && ITERS == 1 && f_hist.ntiles && f_dm.blocks) STX_SEG_F(CH, F, 3);                           \
            else if (F && ITERS == 1 && f_hist.ntiles) STX_SEG_F(CH, F, 2);                                     \
            else if (F && ITERS == 1 && f_scat.ntiles) STX_SEG_F(CH, F, 1);                                     \
            else if (F && ITERS == 1 && f_emit.ntiles) STX_SEG_F(CH, F, 4);                                     \
            else STX_SEG_F(CH, F, 0);                                                                           \
        }                                                                                                       \
    } while (0)
#define STX_SEG2(P, CH) do { if (fused) STX_SEG(P, CH, true); else STX_SEG(P, CH, false); } while (0)
    if (packed_src) { if (small) STX_SEG2(true, CH_SHORT); else STX_SEG2(true, CH_LONG); }
    else            { if (small) STX_SEG2(false, CH_SHORT); else STX_SEG2(false, CH_LONG); }
    if (dm_fixup_after) launch_transr_dm_fixup_late(c);
#undef STX_SEG2
#undef STX_SEG
#undef STX_SEG_F
#undef STX_SEG_0
#undef STX_SEG_RS
#undef STX_SEG_R
}

template <int LPR, int ITERS>
static void sgd_go(stx_ctx *c, const stx_incidence *inc, const SgdTables &T, const float *grad_rows,
                   const float *w_rows, float lr)
{
    constexpr int GROUPS = kThreads / LPR;
    int64_t cap = inc->nnz < c->cfg.n_ent + c->cfg.n_rel ? inc->nnz : c->cfg.n_ent + c->cfg.n_rel;
    int64_t blocks = (cap + GROUPS - 1) / GROUPS;
    if (!T.table_b && !T.table_w) blocks = (blocks + 3) / 4;   // that path takes four segments per group and turn
    if (blocks > 8192) blocks = 8192;   // grid-stride beyond this (measured faster than one segment per group)
    if (blocks < 1) blocks = 1;
    ProfScope prof(c, "k_sgd_rows");
    hipLaunchKernelGGL((k_sgd_rows<LPR, ITERS>), dim3((unsigned)blocks), dim3(kThreads), 0, c->stream,
                       inc->at_touched_cols, inc->n_touched, T.table_a, T.width_a / 4, T.mode_a, (int32_t)T.n_split,
                       T.table_b, T.width_b / 4, T.table_w, T.mode_w, grad_rows, w_rows, c->ld, lr, big_tables(c));
}

// Stored rows of a batch that stx_train_step would form (formed_rows): the tiles of launch_seg_formed, so that the sums
// have the same bits.  Its slices of 16 lanes too where rows are whole memory lines (393,216 positives at d = 1024: 1,605 us,
// 1,631 in slices of 64 lanes); other rows' short slices would begin and end inside lines that two of them then fetch
// (131,072 at d = 516: 383 us against 332), and go in slices of 64 lanes, sixteen groups all the same.
static void seg_slices(stx_ctx *c, const stx_incidence *inc, const float *src, int width, float *out_rows, int ld_out,
                       const FusedArgs *fused)
{
    constexpr int LPR = 16, CH = 16, TILE = kThreads / LPR * CH;
    const int32_t nnz = (int32_t)inc->nnz;
    const int d4 = width / 4, ntiles = (nnz + TILE - 1) / TILE;
    const dim3 grid((unsigned)ntiles, (unsigned)((d4 + LPR - 1) / LPR)), wide((unsigned)ntiles, (unsigned)((d4 + 63) / 64));
    const FusedArgs fu = fused ? *fused : FusedArgs{};
    const SegSecond sec{0x7fffffff, 0, 0, nullptr, nullptr, nullptr, nullptr, 0, 0};
#define STX_SLICES_R(F, L, T, GRID)                                                                             \
    hipLaunchKernelGGL((k_seg_reduce<L, 1, false, CH, F, 0, SRC_STORED, T>), GRID, dim3(T), 0, c->stream,       \
                       inc->at_packed, inc->at_seg_id, 0, nnz, src, src, nnz, width, d4, out_rows, ld_out,      \
                       c->partials, fu, sec, SegWriteRide{}, EmitAhead{}, ScatterAhead{}, DmRide{})
#define STX_SLICES(F)                                                                                           \
    do {                                                                                                        \
        {                                                                                                       \
            ProfScope prof(c, "k_seg_reduce");                                                                  \
            if (width % 32 == 0) STX_SLICES_R(F, LPR, kThreads, grid);                                          \
            else STX_SLICES_R(F, 64, 64 * (kThreads / LPR), wide);                                              \
        }                                                                                                       \
        ProfScope prof(c, "k_seg_fixup");                                                                       \
        hipLaunchKernelGGL((k_seg_fixup<LPR, 1, CH, F, 0, true>), dim3(grid.x, std::min(grid.y, 4u)), dim3(kThreads), 0, c->stream, \
                           inc->at_packed, inc->at_seg_id, inc->at_seg_ptr, 0, nnz, d4, out_rows, ld_out, c->partials, fu, sec, \
                           ScatterAhead{}, HistAhead{}, DmRide{}, EmitAhead{});                                 \
    } while (0)
    if (fused) STX_SLICES(true);
    else STX_SLICES(false);
#undef STX_SLICES
#undef STX_SLICES_R
}

stx_status launch_seg_reduce(stx_ctx *c, const stx_incidence *inc, int64_t e_begin, int64_t e_end,
                             const float *src_a, const float *src_b, int64_t split, int ld_src, int width,
                             float *out_rows, int ld_out, SegRows kind, const SegFusedHost *fh,
                             const SegSecondHost *second)
{
    if (e_end <= e_begin) return STX_OK;
    Launch L = row_launch(width);
    // the sorted keys of the last build on this context are the columns of the sorted entries
    FusedArgs fu{nullptr, nullptr, 0, inc->at_touched_cols, c->sorted_inc == inc ? c->sorted_keys : nullptr, 0.f, 0,
                 big_tables(c)};
    if (fh) { fu.table = fh->table; fu.table_b = fh->table_b; fu.n_split = fh->n_split; fu.lr = fh->lr; fu.mode = fh->mode; }
    const FusedArgs *fused = fh ? &fu : nullptr;
    if (formed_rows(c, inc->n_rows)) {
        seg_slices(c, inc, src_a, width, out_rows, ld_out, fused);
        return hip_ok(hipGetLastError());
    }
    STX_DISPATCH_ROW(L, seg_go, c, inc, (int32_t)e_begin, (int32_t)e_end, src_a, src_b, (int32_t)split, ld_src, width,
                     out_rows, ld_out, kind, fused, second);
    return hip_ok(hipGetLastError());
}

template <int LPR, int ITERS>
static void semiring_t_go(stx_ctx *c, const stx_incidence *inc, const float *X, int kind, const float *gz, float *out_rows)
{
    constexpr int CH_LONG = LPR == 64 ? 64 : (LPR < 32 ? LPR : 32), CH_SHORT = LPR < 16 ? LPR : 16;
    constexpr int GROUPS = kThreads / LPR;
    const int32_t nnz = (int32_t)inc->nnz;
    // Short chunks (see short_chunks) up to 2,304 tiles of them, a little above what the chip holds at once (147,456 entries of more than
    // 128 floats, 294,912 of up to 128), and up to 360,000 entries where long ones would leave the 256 compute units with uneven
    // numbers of workgroups: an eighth more in the fullest than in the mean, a sixteenth where rows have several slices.
    // ComplEx, us with short and with long ones at 120,000, 162,000, 240,000, 330,000 and 390,000 entries, which are 1.83, 2.47, 3.66,
    // 5.04 and 5.95 long workgroups a unit: d = 200: 42.5 and 43.3, 53.5 and 55.7, 75.1 and 72.5, 101 and 103, 116 and 108; d = 128:
    // 26.1 and 27.2, 32.1 and 34.6, 45.3 and 44.1 (196,608 of a power law: 43.5 and 43.7), 59.6 and 60.8, 67.2 and 64.0; two slices a
    // row, d = 512, 180,000, 195,000, 240,000 and 255,000 entries (5.50, 5.95, 7.32 and 7.79): 126 and 128, 135 and 132, 164 and 166,
    // 174 and 168; 232,474 entities, d = 368, 317,196 entries (9.69): 237 and 231 for product and gradient.
    constexpr int CUS = 256;
    const int n_long = (nnz + GROUPS * CH_LONG - 1) / (GROUPS * CH_LONG) * ITERS, fullest = (n_long + CUS - 1) / CUS;
    const bool small = nnz <= 2304 * GROUPS * CH_SHORT || (nnz <= 360000 && 32 * CUS * fullest > (ITERS > 1 ? 34 : 36) * n_long);
    const int tile = GROUPS * (small ? CH_SHORT : CH_LONG), ntiles = (nnz + tile - 1) / tile;
    const dim3 grid((unsigned)ntiles, (unsigned)ITERS);    // wide rows: column slices of one float4 per lane
    const int d4 = c->cfg.dim / 4;
    const FusedArgs fu{};
    const SegSecond sec{0x7fffffff, 0, 0, nullptr, nullptr, nullptr, nullptr, 0, 0};
    const SrcArgs sr{inc->a_colidx, X, gz};
#define STX_SR_T(K, CH)                                                                                         \
    hipLaunchKernelGGL((k_seg_reduce<LPR, 1, false, CH, false, 0, SRC_SEMIRING + K>), grid, dim3(kThreads), 0,  \
                       c->stream, inc->at_packed, inc->at_seg_id, 0, nnz, nullptr, nullptr,                     \
                       (int32_t)(2 * inc->n_rows), 0, d4, out_rows, c->ld, c->partials, fu, sec,             \
                       SegWriteRide{}, EmitAhead{}, ScatterAhead{}, DmRide{}, sr)
#define STX_SR_T2(K) do { if (small) STX_SR_T(K, CH_SHORT); else STX_SR_T(K, CH_LONG); } while (0)
    {
        ProfScope prof(c, "k_seg_reduce");
        if (kind == SR_DISTMULT) STX_SR_T2(SR_DISTMULT);
        else if (kind == SR_COMPLEX) STX_SR_T2(SR_COMPLEX);
        else STX_SR_T2(SR_ROTATE);
    }
#undef STX_SR_T2
#undef STX_SR_T
    if (ntiles <= 1) return;
    ProfScope prof(c, "k_seg_fixup");
#define STX_SR_F(CH)                                                                                            \
    hipLaunchKernelGGL((k_seg_fixup<LPR, 1, CH, false, 0>), grid, dim3(kThreads), 0, c->stream, inc->at_packed, \
                       inc->at_seg_id, inc->at_seg_ptr, 0, nnz, d4, out_rows, c->ld, c->partials, fu, sec,      \
                       ScatterAhead{}, HistAhead{}, DmRide{}, EmitAhead{})
    if (small) STX_SR_F(CH_SHORT);
    else STX_SR_F(CH_LONG);
#undef STX_SR_F
}

stx_status launch_seg_formed(stx_ctx *c, const stx_incidence *inc, const stx_params *p, float *out_rows, int ld_out)
{
    constexpr int LPR = 16, CH = 16, TILE = kThreads / LPR * CH;
    const int32_t nnz = (int32_t)inc->nnz, split = (int32_t)(2 * inc->n_rows);
    const FormedRows fr = formed_buffers(c, inc->n_rows);
    {
        ProfScope prof(c, "k_seg_records");
        SegWriteRide fin{};
        fin.fin_partials = c->loss_partials; fin.fin_n = c->fin_n; fin.fin_scale = c->fin_scale; fin.fin_loss = c->fin_loss;
        hipLaunchKernelGGL(k_seg_records, dim3((unsigned)((nnz + kThreads - 1) / kThreads + (c->fin_n > 0 ? 1 : 0))), dim3(kThreads), 0, c->stream,
                           inc->at_packed, inc->at_seg_id, inc->a_colidx, fr.coefs, nnz, split, (uint32_t)c->cfg.dim * 4u,
                           (FormedRecord *)fr.recs, (FormedHead *)fr.heads, fin);
        c->fin_n = 0;
    }
    const int d4 = c->cfg.dim / 4, ntiles = (nnz + TILE - 1) / TILE, nslices = (d4 + LPR - 1) / LPR;
    const dim3 grid((unsigned)ntiles, (unsigned)nslices);
    const FusedArgs fu{};
    const SegSecond sec{0x7fffffff, 0, 0, nullptr, nullptr, nullptr, nullptr, 0, 0};
    const uint32_t x_bytes = (uint32_t)(c->cfg.n_ent + c->cfg.n_rel) * (uint32_t)c->cfg.dim * 4u;   // (formed_rows: 96 MiB at most)
#define STX_FORMED(D)                                                                                           \
    hipLaunchKernelGGL((k_seg_formed<D>), dim3(((unsigned)ntiles * (unsigned)nslices + 7u) / 8u * 8u), dim3(kThreads), 0, \
                       c->stream, (const FormedRecord *)fr.recs, (const FormedHead *)fr.heads, inc->at_touched_cols, nnz, ntiles, nslices, p->ent, x_bytes, \
                       c->cfg.dim, out_rows, ld_out, c->partials)
    {
        ProfScope prof(c, "k_seg_reduce");
        if (c->cfg.dist == STX_L2) STX_FORMED(STX_L2);
        else if (c->cfg.dist == STX_L2_SQ) STX_FORMED(STX_L2_SQ);
        else STX_FORMED(STX_TORUS_L2);
    }
#undef STX_FORMED
    if (ntiles > 1) {
        ProfScope prof(c, "k_seg_fixup");
        hipLaunchKernelGGL((k_seg_fixup<LPR, 1, CH, false, 0, true>), dim3(grid.x, std::min(grid.y, 4u)), dim3(kThreads), 0, c->stream,
                           inc->at_packed, inc->at_seg_id, inc->at_seg_ptr, 0, nnz, d4, out_rows, ld_out, c->partials, fu, sec,
                           ScatterAhead{}, HistAhead{}, DmRide{}, EmitAhead{});
    }
    return hip_ok(hipGetLastError());
}

stx_status launch_semiring_product_t(stx_ctx *c, const stx_incidence *inc, const stx_params *p, int kind, const float *gz,
                                     float *out_rows)
{
    Launch L = row_launch(c->cfg.dim);
    STX_DISPATCH_ROW(L, semiring_t_go, c, inc, p->ent, kind, gz, out_rows);
    return hip_ok(hipGetLastError());
}

stx_status launch_sgd_rows(stx_ctx *c, const stx_incidence *inc, const SgdTables &T, const float *grad_rows,
                           const float *w_rows, float lr)
{
    if (inc->n_rows == 0) return STX_OK;
    Launch L = row_launch(T.width_a > T.width_b ? T.width_a : T.width_b);
    STX_DISPATCH_ROW(L, sgd_go, c, inc, T, grad_rows, w_rows, lr);
    return hip_ok(hipGetLastError());
}

}  // namespace stx
