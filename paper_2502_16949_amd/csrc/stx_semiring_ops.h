// Arithmetic of the semiring products (SparseTransX Appendix D), shared by the products themselves
// (stx_semiring.hip) and by the transposed product that forms their backward terms (stx_backward.hip).
#pragma once

#include "stx_rowops.h"

namespace stx {

enum { SR_DISTMULT = 0, SR_COMPLEX = 1, SR_ROTATE = 2 };

// (a.x + i a.y)(b.x + i b.y)
__device__ inline float2 cmul(float2 a, float2 b)
{
    const float ac = a.x * b.x, bd = a.y * b.y, ad = a.x * b.y, bc = a.y * b.x;
    return make_float2(ac - bd, ad + bc);
}
__device__ inline float2 conj2(float2 a) { return make_float2(a.x, -a.y); }
__device__ inline float2 lo2(float4 v) { return make_float2(v.x, v.y); }
__device__ inline float2 hi2(float4 v) { return make_float2(v.z, v.w); }
__device__ inline float4 join(float2 a, float2 b) { return make_float4(a.x, a.y, b.x, b.y); }
__device__ inline float4 mul4(float4 a, float4 b) { return make_float4(a.x * b.x, a.y * b.y, a.z * b.z, a.w * b.w); }
__device__ inline float4 neg4(float4 a) { return make_float4(-a.x, -a.y, -a.z, -a.w); }

// One entry's share of the backward of a row's product, for a real loss with dL/dZ = g: g times the conjugated product
// of the other two factors, a before b in the row (tail: of the head entry and relation entry), as the transposed
// product adds it.  Head and relation entries (tail false): dL/dh = (g conj(r)) t, dL/dr = (g conj(h)) t; tail
// entries: -(-dL/dt), with dL/dt = (conj(g) h) r for ComplEx, g h r for DistMult and -g for RotatE.
template <int KIND>
__device__ inline float4 semiring_term(float4 g, float4 a, float4 b, bool tail)
{
    if (KIND == SR_DISTMULT) return mul4(mul4(g, a), b);
    if (KIND == SR_ROTATE) {
        if (tail) return neg4(g);
        return join(cmul(lo2(g), conj2(lo2(a))), cmul(hi2(g), conj2(hi2(a))));
    }
    if (tail) return join(cmul(cmul(conj2(lo2(g)), lo2(a)), lo2(b)), cmul(cmul(conj2(hi2(g)), hi2(a)), hi2(b)));
    return join(cmul(cmul(lo2(g), conj2(lo2(a))), lo2(b)), cmul(cmul(hi2(g), conj2(hi2(a))), hi2(b)));
}

}  // namespace stx
