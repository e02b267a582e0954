// unit_walk.hpp -- how the batched sweep's wavefronts walk over the site
// words of a colour.  Host and device: which words a walk may touch follows
// from the sizes alone, so it can be checked without a GPU.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pa {

// x / d for 0 <= x < 2^21 and a divisor known only at run time, from
// inv = 1 / d: the error of the product (below 2^-23 of it) is less than the
// distance 1 / (2d) of (x + 1/2) / d from the next integer.
__host__ __device__ __forceinline__ int div_small(int x, float inv) { return (int)(((float)x + 0.5f) * inv); }

// Lattice of side L as the sweep keeps it: two colours of nh words each, a
// colour's words in rows of half.
struct LatticeShape {
    int L, N, half, nh;
};

// A lane's walk over its wavefront's units in steps of 64: replica group gs
// within the workgroup, site k = y L/2 + m of the colour, first lattice word
// a = gs N + k (colour 0).  No division per step: the step's rows, columns
// and groups are known beforehand and each carries at most once.
struct UnitWalk {
    int gs, k, y, m, a;
    __host__ __device__ __forceinline__ void start(const LatticeShape &J, int u)
    {
        gs = div_small(u, 1.0f / (float)J.nh);
        k = u - gs * J.nh;
        y = div_small(k, 1.0f / (float)J.half);
        m = k - y * J.half;
        a = gs * J.N + k;
    }
    __host__ __device__ __forceinline__ void step(const LatticeShape &J, int gq, int kr, int yr, int mr)
    {
        gs += gq;
        k += kr;
        y += yr;
        m += mr;
        a += gq * J.N + kr;
        if (m >= J.half) {
            m -= J.half;
            ++y;
        }
        if (k >= J.nh) {
            k -= J.nh;
            y -= J.L;
            a += J.N - J.nh;
            ++gs;
        }
    }
    // the unit's word of a colour
    __host__ __device__ __forceinline__ int word(const LatticeShape &J, int colour) const { return a + colour * J.nh; }
    // offset of the other horizontal neighbour, p = x & 1
    __host__ __device__ __forceinline__ int dh(const LatticeShape &J, int p) const
    {
        return p ? (m + 1 == J.half ? 1 - J.half : 1) : (m == 0 ? J.half - 1 : -1);
    }
    __host__ __device__ __forceinline__ int du(const LatticeShape &J) const { return y == 0 ? J.nh - J.half : -J.half; }
    __host__ __device__ __forceinline__ int dd(const LatticeShape &J) const
    {
        return y + 1 == J.L ? J.half - J.nh : J.half;
    }
};

// Does f with a unit's word, where there is a unit: lanes past the wavefront's
// last one have walked into a group that the workgroup does not hold, and
// touch no word.  (With a word of their own to leave as it is, chosen by a
// select instead of a branch: 1024 runs of four sizes 1548 against 1531 us per
// step, L = 80 441 against 438.)
template <class F>
__host__ __device__ __forceinline__ void at_unit(bool in, int word, F f)
{
    if (in) f(word);
}

}  // namespace pa
