// Device-side bodies of the radix-sort passes over the column ids of A (see stx_build.hip), shared by the
// kernels that run them alone and by the launches that run them beside another, independent piece of
// work (stx_step.hip).
#pragma once

#include "stx_device.h"
#include "stx_internal.h"

namespace stx {

// Tile histograms of the digit at `shift` for the later passes.
template <int ITEMS>
__device__ inline void hist_body(const int block, const int32_t *__restrict__ keys, int32_t nnz, int shift,
                                 int radix, uint16_t *__restrict__ table)
{
    __shared__ int32_t s_hist[256];
    const int tid = threadIdx.x;
    s_hist[tid] = 0;
    __syncthreads();
    const int32_t base = block * (kThreads * ITEMS);
    int32_t kv[ITEMS];                                   // all loads first, so that they are in flight together
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const int32_t e = base + it * kThreads + tid;
        kv[it] = keys[min(e, nnz - 1)];
    }
    // The lanes of a wavefront that hold the same digit are found by a ballot per bit, and one of them adds their
    // number: power-law keys put many lanes on one counter, and LDS serialises atomics on one address.
    const int bits = 31 - __clz(radix), lane = tid & 63;
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const int32_t e = base + it * kThreads + tid;
        const bool valid = e < nnz;
        const int dgt = (kv[it] >> shift) & (radix - 1);
        const uint64_t m = digit_class_mask(dgt, valid, bits);
        if (valid && ((m >> lane) >> 1) == 0) atomicAdd(&s_hist[dgt], (int32_t)__popcll(m));   // highest lane of its class
    }
    __syncthreads();
    if (tid < radix) table[block * radix + tid] = (uint16_t)s_hist[tid];
}

// Stable scatter of one tile by the digit at `shift`.  Element order inside a tile is
// (wavefront, iteration, lane): wavefront w owns the contiguous span [w*512, (w+1)*512) of the tile.
// The rank of a key among equal digits is
//   (count in earlier wavefronts) + (count in earlier iterations of this wavefront) + (equal lanes below),
// the last term from a ballot match over the digit's bits.  The base offset of a (digit, tile) is the
// number of keys with a smaller digit anywhere plus those with the same digit in earlier tiles: read
// derived here from the raw tile counts: directly when there are few tiles (TWO_LEVEL false), through
// the group sums of k_super_sums otherwise.
// `block` is the tile (the index of the workgroup among those of the scatter; the launch may hold others).
// ARENA: the body's LDS arrays live in the kScatterLds bytes at `lds` instead of arrays of its own.
template <bool FIRST, bool TWO_LEVEL, int ITEMS, bool ARENA = false>
__device__ inline void scatter_body(const int block, const ScatterArgs &a, unsigned char *lds = nullptr)
{
    const int32_t *__restrict__ keys_in = a.keys_in;
    const int32_t *__restrict__ pay_in = a.pay_in;
    int32_t *__restrict__ keys_out = a.keys_out;
    int32_t *__restrict__ pay_out = a.pay_out;
    const int32_t nnz = a.nnz;
    const int shift = a.shift, bits = a.bits, ntiles = a.ntiles;
    const uint16_t *__restrict__ table = a.table;
    const int32_t *__restrict__ super = a.super;
    int32_t *s_goff, (*s_hist)[256], *s_tot, *s_bel;
    if constexpr (ARENA) {
        int32_t *p = reinterpret_cast<int32_t *>(lds);
        s_goff = p; s_hist = reinterpret_cast<int32_t (*)[256]>(p + 256); s_tot = p + 1280; s_bel = p + 2304;
    } else {
        __shared__ int32_t o_goff[256];
        __shared__ int32_t o_hist[4][256];
        s_goff = o_goff; s_hist = o_hist;
        // (a large sort's tile is put in order in the same place later)
        __shared__ int32_t o_tot[ITEMS > kSortItems ? kThreads * ITEMS : 1024], o_bel[ITEMS > kSortItems ? kThreads * ITEMS : 1024];
        s_tot = o_tot; s_bel = o_bel;
    }
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int radix = 1 << bits;
    for (int i = tid; i < 4 * 256; i += kThreads) (&s_hist[0][0])[i] = 0;
    int32_t key[ITEMS], pay[ITEMS], rank[ITEMS];
    const int32_t wave_base = block * (kThreads * ITEMS) + w * (64 * ITEMS);
    const uint64_t lanes_below = (1ull << lane) - 1ull;
    auto load_items = [&]() {
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {             // all loads at once, so that they are in flight together
            const int32_t e = wave_base + it * 64 + lane;
            const int32_t f = min(e, nnz - 1);           // (past the end: the last one again, without a branch)
            key[it] = keys_in[f];
            pay[it] = FIRST ? e : pay_in[f];
        }
    };
    // The tile's keys are requested before the offsets are derived from the histogram tables, so that the two waits overlap.
    load_items();
    if (TWO_LEVEL) {
        int32_t below = 0, total = 0;
        const int me = block, g_me = me / kSuperTile, ngroups = (ntiles + kSuperTile - 1) / kSuperTile;
        if (radix >= 8) {
            // A thread owns eight neighbouring digits and every `parts`-th row, of the groups' sums and of the tiles of its own
            // group; four in flight, so that 32 groups of 32 tiles cost two round trips.  (A thread per digit walked
            // the rows eight at a time, eight round trips one behind the other; a step of 3.9 M entries, three passes: 558 -> 553 us.)
            constexpr int U = 4;
            const int r8 = radix >> 3, sh = 31 - __clz(r8), parts = kThreads >> sh, d8 = tid & (r8 - 1), q = tid >> sh;
            int32_t tot[8], bel[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) tot[u] = bel[u] = 0;
            const int first = g_me * kSuperTile;
            for (int g0 = q; g0 < ngroups; g0 += U * parts) {
                int4 v[U][2];
#pragma unroll
                for (int u = 0; u < U; ++u) {              // (a row past the last one: the last one again, not added)
                    const int32_t *ps = super + min(g0 + u * parts, ngroups - 1) * radix + 8 * d8;
                    v[u][0] = *reinterpret_cast<const int4 *>(ps);
                    v[u][1] = *reinterpret_cast<const int4 *>(ps + 4);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int g = g0 + u * parts;
                    const int32_t sv[8] = {v[u][0].x, v[u][0].y, v[u][0].z, v[u][0].w, v[u][1].x, v[u][1].y, v[u][1].z, v[u][1].w};
#pragma unroll
                    for (int d = 0; d < 8; ++d) {
                        tot[d] += g < ngroups ? sv[d] : 0;
                        bel[d] += g < g_me ? sv[d] : 0;
                    }
                }
            }
            for (int t0 = first + q; t0 < me; t0 += U * parts) {
                uint4 v[U];
#pragma unroll
                for (int u = 0; u < U; ++u) v[u] = *reinterpret_cast<const uint4 *>(table + min(t0 + u * parts, me) * radix + 8 * d8);
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const uint32_t tv[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
                    for (int d = 0; d < 8; ++d) bel[d] += t0 + u * parts < me ? (int32_t)(d & 1 ? tv[d / 2] >> 16 : tv[d / 2] & 0xffffu) : 0;
                }
            }
            for (int m = r8; m < 64; m <<= 1) {            // the parts that share a wavefront
#pragma unroll
                for (int u = 0; u < 8; ++u) { tot[u] += __shfl_xor(tot[u], m, 64); bel[u] += __shfl_xor(bel[u], m, 64); }
            }
            if (lane < r8) {
                int32_t *pt = &s_tot[w * radix + 8 * d8], *pb = &s_bel[w * radix + 8 * d8];
#pragma unroll
                for (int u = 0; u < 8; ++u) { pt[u] = tot[u]; pb[u] = bel[u]; }
            }
            __syncthreads();
            if (tid < radix) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    total += s_tot[u * radix + tid];
                    below += s_bel[u * radix + tid];
                }
            }
        } else if (tid < radix) {   // two or four bins only
            for (int g = 0; g < ngroups; ++g) {
                const int32_t v = super[g * radix + tid];
                total += v;
                below += g < g_me ? v : 0;
            }
            for (int t = g_me * kSuperTile; t < me; ++t) below += table[t * radix + tid];
        }
        int32_t base = block_exclusive_scan(total, nullptr);
        s_goff[tid] = base + below;
    } else {
        // All 256 threads share the table: a thread owns eight neighbouring digits (one 16-byte load per tile row: a tile's
        // counts fit 16 bits) and every `parts`-th tile, eight loads in flight.  Two counts a word are added at a time, for as
        // many rows as cannot carry from one into the other.  (With counts of 32 bits the scan of 192 rows was 3.9 us of a
        // scatter pass's 9.1.)
        const int me = block;
        int32_t below = 0, total = 0;
        if (radix >= 8) {
            // (rows added two counts a word before they are taken apart: the tables of most batches of small tiles in one go,
            // as the sums of 32 bits that would wait meanwhile are registers that lower the occupancy of the launches this
            // body shares with others)
            constexpr int SCAN = 8, TILE = kThreads * ITEMS, ROWS = 65535 / TILE / SCAN * SCAN;
            static_assert(ROWS >= SCAN, "no carry between the two counts of a word");
            const int r8 = radix >> 3, sh = 31 - __clz(r8), parts = kThreads >> sh, d8 = tid & (r8 - 1), q = tid >> sh;
            for (int t1 = 0; t1 < ntiles; t1 += ROWS * parts) {
                uint4 s4 = make_uint4(0u, 0u, 0u, 0u), b4 = s4;
                for (int t0 = t1 + q; t0 < min(ntiles, t1 + ROWS * parts); t0 += SCAN * parts) {
                    uint4 v[SCAN];
#pragma unroll
                    for (int u = 0; u < SCAN; ++u)         // (a row past the last one: the last one again, not added)
                        v[u] = *reinterpret_cast<const uint4 *>(table + min(t0 + u * parts, ntiles - 1) * radix + 8 * d8);
#pragma unroll
                    for (int u = 0; u < SCAN; ++u) {
                        const int t = t0 + u * parts;
                        if (t < ntiles) { s4.x += v[u].x; s4.y += v[u].y; s4.z += v[u].z; s4.w += v[u].w; }
                        if (t < me) { b4.x += v[u].x; b4.y += v[u].y; b4.z += v[u].z; b4.w += v[u].w; }
                    }
                }
                int32_t tot[8] = {(int32_t)(s4.x & 0xffffu), (int32_t)(s4.x >> 16), (int32_t)(s4.y & 0xffffu), (int32_t)(s4.y >> 16),
                                  (int32_t)(s4.z & 0xffffu), (int32_t)(s4.z >> 16), (int32_t)(s4.w & 0xffffu), (int32_t)(s4.w >> 16)};
                int32_t bel[8] = {(int32_t)(b4.x & 0xffffu), (int32_t)(b4.x >> 16), (int32_t)(b4.y & 0xffffu), (int32_t)(b4.y >> 16),
                                  (int32_t)(b4.z & 0xffffu), (int32_t)(b4.z >> 16), (int32_t)(b4.w & 0xffffu), (int32_t)(b4.w >> 16)};
                for (int m = r8; m < 64; m <<= 1) {        // the parts that share a wavefront
#pragma unroll
                    for (int u = 0; u < 8; ++u) { tot[u] += __shfl_xor(tot[u], m, 64); bel[u] += __shfl_xor(bel[u], m, 64); }
                }
                if (lane < r8) {
                    int32_t *pt = &s_tot[w * radix + 8 * d8], *pb = &s_bel[w * radix + 8 * d8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        pt[u] = t1 == 0 ? tot[u] : pt[u] + tot[u];
                        pb[u] = t1 == 0 ? bel[u] : pb[u] + bel[u];
                    }
                }
            }
            __syncthreads();
            if (tid < radix) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    total += s_tot[u * radix + tid];
                    below += s_bel[u * radix + tid];
                }
            }
        } else if (tid < radix) {   // two or four bins only
            for (int t = 0; t < ntiles; ++t) {
                const int32_t v = table[t * radix + tid];
                total += v;
                below += t < me ? v : 0;
            }
        }
        int32_t base = block_exclusive_scan(total, nullptr);
        s_goff[tid] = base + below;
    }
    __syncthreads();

#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        int32_t e = wave_base + it * 64 + lane;
        bool valid = e < nnz;
        int dgt = (key[it] >> shift) & (radix - 1);
        const uint64_t m = digit_class_mask(dgt, valid, bits);
        int32_t prior = s_hist[w][dgt];
        rank[it] = prior + __popcll(m & lanes_below);
        bool leader = valid && ((m >> lane) >> 1) == 0;   // highest lane of its digit class
        if (leader) s_hist[w][dgt] = prior + __popcll(m);
    }
    __syncthreads();
    int32_t tile_count = 0;                              // keys of the tile with digit `tid`
    if (tid < radix) {
#pragma unroll
        for (int w2 = 0; w2 < 4; ++w2) {
            int32_t c = s_hist[w2][tid];
            s_hist[w2][tid] = tile_count;
            tile_count += c;
        }
    }
    // Large sorts (tiles of kBigSortItems keys per thread): the tile is put in order in LDS first and written from
    // there, so that neighbouring lanes write neighbouring addresses and a digit's keys of one tile (16 on
    // average with 256 digits: 64 bytes) fill whole sectors; written straight from the registers every key is a
    // partial write of its own, and the pass moves 2.5 times the bytes it has to.
    constexpr bool LOCAL = ITEMS > kSortItems && !ARENA;
    if constexpr (LOCAL) {
        __shared__ int32_t s_dstart[256];
        int32_t *s_k = s_tot, *s_p = s_bel;                // (read out before the barriers of the scans)
        s_dstart[tid] = block_exclusive_scan(tile_count, nullptr);   // (its barriers also publish s_hist)
        __syncthreads();
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
            const int32_t e = wave_base + it * 64 + lane;
            if (e < nnz) {
                const int dgt = (key[it] >> shift) & (radix - 1);
                const int32_t lp = s_dstart[dgt] + s_hist[w][dgt] + rank[it];
                s_k[lp] = key[it];
                s_p[lp] = pay[it];
            }
        }
        __syncthreads();
        const int32_t tile_n = min(kThreads * ITEMS, nnz - block * (kThreads * ITEMS));
        for (int32_t i = tid; i < tile_n; i += kThreads) {
            const int32_t kv = s_k[i];
            const int dgt = (kv >> shift) & (radix - 1);
            const int32_t pos = s_goff[dgt] + (i - s_dstart[dgt]);
            keys_out[pos] = kv;
            pay_out[pos] = s_p[i];
        }
    } else {
        __syncthreads();
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
            int32_t e = wave_base + it * 64 + lane;
            if (e < nnz) {
                int dgt = (key[it] >> shift) & (radix - 1);
                int32_t pos = s_goff[dgt] + s_hist[w][dgt] + rank[it];
                keys_out[pos] = key[it];
                pay_out[pos] = pay[it];
            }
        }
    }
}

}  // namespace stx
