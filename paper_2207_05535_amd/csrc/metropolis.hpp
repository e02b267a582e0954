// metropolis.hpp -- bit-sliced checkerboard Metropolis update of one site for
// 64 replicas at once.
//
// A 64-bit word holds one site of 64 consecutive replicas (bit b = replica
// 64g + b; a set bit is spin -1).  For the site's four bonds the word
// s ^ s_k ^ j_k has bit b set where the bond is unsatisfied (J s s_k = -1).
// With u = number of unsatisfied bonds the energy change of a flip is
// dE = 2 s h = 8 - 4u: u >= 2 means dE <= 0 (always flip), u = 1 means
// dE = +4 and u = 0 means dE = +8 (flip iff the replica's 32-bit draw is
// below the threshold T(beta_i, dE)).
//
// The sweeps are bound by the vector ALU's issue rate, so the form of this
// logic is chosen for its instruction count: one mask of the undecided
// replicas and one of their class (rather than one mask per class) takes 12
// instead of 20 instructions per Philox call for its two planes, the
// classification 10 instead of 26 per ferromagnetic site.  Measured against
// that earlier form: 3.08e8 instead of 3.53e8 vector instructions per sweep
// launch at L = 64, R = 1e5, 617 -> 576 us; a mix of ten spin-glass runs
// 1884 -> 1767 us; two populations of 2e5 at L = 32 stay at 657 us (9 %
// fewer instructions, but their launch ends unevenly).
//
// The draw of replica b is the 32-bit number whose bit 31-p is bit b of bit
// plane p; Philox call c (counter (n | c << 20, g, i, tag)) yields planes 2c
// (o0 | o1 << 32) and 2c + 1 (o2 | o3 << 32).  Comparing u < T most
// significant bit first, a lane is decided at the first plane where its bit
// differs from T's bit (accept if T's bit is 1).  Planes are generated only
// while some lane of the word is undecided; the result is identical to the
// full 32-bit comparison.
#pragma once

#include "philox.hpp"

namespace pa {

struct Thresholds {
    uint32_t t4, t8;        // low 32 bits of T(beta, 4), T(beta, 8)
    bool all4, all8;        // T == 2^32: every such move is accepted
};

constexpr int LUT_SEL = lut3((LUT_A & LUT_B) | (~LUT_A & LUT_C));   // a ? b : c, bitwise
constexpr int LUT_MAJ = lut3((LUT_A & LUT_B) | (LUT_A & LUT_C) | (LUT_B & LUT_C));
constexpr int LUT_BOTH_DIFFER = lut3((LUT_A ^ LUT_B) & (LUT_A ^ LUT_C));
constexpr int LUT_ANY_DIFFERS = lut3((LUT_A ^ LUT_B) | (LUT_A ^ LUT_C));
constexpr int LUT_NEITHER = lut3(~((LUT_A ^ LUT_B) | LUT_C));       // a = b and not c
constexpr int LUT_KEEP = lut3(LUT_A & ~(LUT_B ^ LUT_C));            // a where b = c
constexpr int LUT_LESS = lut3((LUT_A & ~LUT_B) | (~(LUT_A ^ LUT_B) & LUT_C));   // a where a != b, else c
constexpr int LUT_ANDN2 = lut3(LUT_A & LUT_B & ~LUT_C);             // a and b, not c

// Site classes of 64 replicas: und = the replicas whose flip costs energy
// (dE > 0: they draw), one = those of them with dE = +4 (the others have
// dE = +8; bits outside und mean nothing).  From the word w, its four
// neighbours (for the spin glass already multiplied by their bonds: XOR with
// all ones where J = -1).  Of the neighbours a, b, c, d that differ from w,
// two or more mean dE <= 0: with s = a ^ b ^ c and m = maj(a, b, c) that is
// "m differs from w, or both s and d do", and where neither holds exactly
// one differs iff s or d does.  Five three-input operations per 32 bits.
struct SiteClass {
    uint64_t und, one;
};

__device__ __forceinline__ SiteClass classify(uint64_t w, uint64_t a, uint64_t b, uint64_t c, uint64_t d)
{
    const uint64_t s = bop3<LUT_XOR3>(a, b, c), m = bop3<LUT_MAJ>(a, b, c);
    SiteClass k;
    k.und = bop3<LUT_NEITHER>(w, m, bop3<LUT_BOTH_DIFFER>(w, s, d));
    k.one = bop3<LUT_ANY_DIFFERS>(w, s, d);
    return k;
}

// Temperatures where a threshold is 2^32 (beta_i = 0): moves of that class
// are accepted without a draw.
__device__ __forceinline__ void accept_saturated(SiteClass &k, const Thresholds &T)
{
    if (T.all4) k.und &= ~k.one;
    if (T.all8) k.und &= k.one;
}

// The two bit planes of one Philox call in the most-significant-first
// comparison u < T for the undecided replicas und.  m4 / m8: all ones where
// T(beta, 4) / T(beta, 8) has a 1 at that plane (.x the first plane, .y the
// second); a replica's T bit is its class's.  A replica whose draw bit
// differs from its T bit is decided, and accepted iff the T bit is 1; on
// return und holds those equal at both planes, and `less` the verdict of the
// ones decided here (bits of other replicas mean nothing).  Six three-input
// operations per 32 bits for both planes.
struct alignas(16) PlaneMasks {
    uint32_t a4, b4, a8, b8;   // first and second plane, dE = +4 and +8
};

__device__ __forceinline__ uint64_t plane_pair(uint64_t pa, uint64_t pb, const PlaneMasks &m, uint64_t one,
                                               uint64_t &und)
{
    uint32_t less[2], left[2];
    const uint32_t a[2] = {(uint32_t)pa, (uint32_t)(pa >> 32)}, b[2] = {(uint32_t)pb, (uint32_t)(pb >> 32)};
    const uint32_t u[2] = {(uint32_t)und, (uint32_t)(und >> 32)}, k[2] = {(uint32_t)one, (uint32_t)(one >> 32)};
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const uint32_t ta = bop3<LUT_SEL>(k[h], m.a4, m.a8), tb = bop3<LUT_SEL>(k[h], m.b4, m.b8);
        left[h] = bop3<LUT_KEEP>(bop3<LUT_KEEP>(u[h], a[h], ta), b[h], tb);
        less[h] = bop3<LUT_LESS>(ta, a[h], tb);
    }
    und = (uint64_t)left[0] | ((uint64_t)left[1] << 32);
    return (uint64_t)less[0] | ((uint64_t)less[1] << 32);
}

// T's bits at the planes of call c as all-ones or zero masks: first plane 2c
// (bit 31 - 2c), second plane 2c + 1 (bit 30 - 2c).
__device__ __forceinline__ PlaneMasks call_masks(uint32_t t4, uint32_t t8, uint32_t c)
{
    const uint32_t sh = 31u - 2u * c;
    return {0u - ((t4 >> sh) & 1u), 0u - ((t4 >> (sh - 1u)) & 1u), 0u - ((t8 >> sh) & 1u),
            0u - ((t8 >> (sh - 1u)) & 1u)};
}

// Philox call c of a site, planes 2c and 2c + 1, against the masks m of
// that call: returns the verdicts of plane_pair.
__device__ __forceinline__ uint64_t draw_call(uint32_t c, const PlaneMasks &m, uint64_t one, uint64_t &und,
                                              uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                              uint32_t k1)
{
    const u32x4 o = philox10_sweep<false>(c0 | (c << 20), c1, c2, c3, k0, k1);
    const uint64_t pa = (uint64_t)o.x | ((uint64_t)o.y << 32);
    const uint64_t pb = (uint64_t)o.z | ((uint64_t)o.w << 32);
    return plane_pair(pa, pb, m, one, und);
}

// Thresholds of temperature i, read once per workgroup and kept in scalar
// registers.
__device__ __forceinline__ Thresholds thresholds_of(const uint64_t *tabT, int i)
{
    Thresholds T;
    const uint64_t a = tabT[2 * i], b = tabT[2 * i + 1];
    T.t4 = __builtin_amdgcn_readfirstlane((uint32_t)a);
    T.t8 = __builtin_amdgcn_readfirstlane((uint32_t)b);
    T.all4 = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32)) != 0;
    T.all8 = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32)) != 0;
    return T;
}

// Sign bits of 16 int8 spins (+1 = 0x01, -1 = 0xFF; four bytes per 32-bit
// lane of v, byte k of v.x first): bit k = 1 iff byte k is negative.  Each
// byte's bit 7 is isolated (0x80 or 0) and weighted by a power of two in an
// unsigned 4-byte dot product, so two dwords give 128 x (their 8 bits).
__device__ __forceinline__ uint32_t signs16(const uint4 &v)
{
    uint32_t lo = __builtin_amdgcn_udot4(v.x & 0x80808080u, 0x08040201u, 0u, false);
    lo = __builtin_amdgcn_udot4(v.y & 0x80808080u, 0x80402010u, lo, false);
    uint32_t hi = __builtin_amdgcn_udot4(v.z & 0x80808080u, 0x08040201u, 0u, false);
    hi = __builtin_amdgcn_udot4(v.w & 0x80808080u, 0x80402010u, hi, false);
    return (lo >> 7) | ((hi >> 7) << 8);
}

__device__ __forceinline__ uint64_t pack64(const uint4 v[4])
{
    return (uint64_t)(signs16(v[0]) | (signs16(v[1]) << 16)) |
           ((uint64_t)(signs16(v[2]) | (signs16(v[3]) << 16)) << 32);
}

// Four canonical spin bytes from 4 sign bits f4 (bit k set: byte k = 0xFF,
// else 0x01).  The multiply by 2^0 + 2^7 + 2^14 + 2^21 moves bit k to bit 8k
// among terms at pairwise distinct positions (no carries); each selected bit
// then becomes 0xFE + 0x01 in its byte.
__device__ __forceinline__ uint32_t spins4(uint32_t f4)
{
    const uint32_t e = (f4 * 0x00204081u) & 0x01010101u;
    return e * 0xFEu + 0x01010101u;
}

// 16 canonical spin bytes from 16 sign bits (the inverse of signs16).
__device__ __forceinline__ uint4 spins16(uint32_t b)
{
    uint4 v;
    v.x = spins4(b & 15u);
    v.y = spins4((b >> 4) & 15u);
    v.z = spins4((b >> 8) & 15u);
    v.w = spins4((b >> 12) & 15u);
    return v;
}

}  // namespace pa
