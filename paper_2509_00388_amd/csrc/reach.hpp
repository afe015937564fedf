// The filter pass's 32-bit test of the bounds: which of a key's dots with 16 sources make an edge that reaches the
// source's bound.  Plain C++, so that it can be compiled and tested on the host.
#pragma once
#include <float.h>
#include <math.h>
#include <stdint.h>

namespace gkv {

// What dot / |k_j| must reach for the edge to be listed: the source's bound, lowered by twice the slack, divided by
// 1/|k_i| (inv).  Impossible bounds and rows past the last source (there: false) ask for +infinity, which nothing
// reaches; a zero source, all of whose edges are 0, asks for -infinity if its bound lets them through.
__device__ __forceinline__ float dot_bound(float bound, float inv, bool there)
{
    const float lowered = bound - 2.f * (4e-6f + 1e-5f * fabsf(bound));
    return !there ? INFINITY : (inv > 0.f ? lowered / inv : (lowered <= 0.f ? -INFINITY : INFINITY));
}

// |k_j| as the test takes it.  A zero key's edges are 0: with the smallest norm in place of 0 its dots, which are 0,
// reach what is not positive, and an infinite bound times the norm is a number.
__device__ __forceinline__ float norm_for_test(float norm) { return fmaxf(norm, FLT_MIN); }

// Four sources' bits, the fourth's highest, below those in `misses`: 1 = the dot does not reach.  NaN (a key with an
// infinity, whatever it is multiplied by) does not, whichever sign it has: a row past the last source has no list to write to.
__device__ __forceinline__ uint32_t push_misses(uint32_t misses, const float (&dot)[4], const float (&det)[4], float norm)
{
#pragma unroll
    for (int u = 3; u >= 0; --u) {
        const float over = fmaxf(fmaf(-det[u], norm, dot[u]), -1.f);   // (a maximum passes NaN by)
        misses = (misses << 1) | (__builtin_bit_cast(uint32_t, over) >> 31);
    }
    return misses;
}

}  // namespace gkv
