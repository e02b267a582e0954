// kernels.hip -- HIP kernels of the population-annealing temperature step
// for gfx950 (CDNA4, 64-wide wavefronts).
//
// Step (i)   k_init_couplings, k_init_spins, k_init_fam (Sec. II B, III A)
// Step (ii)  k_rw_chunk                                (Eqs. (QBoltz), (F))
// Step (iii) k_resample_run (one workgroup per population), or k_cnt_chunk,
//            k_mn_draws, k_cnt_scan_chunk, k_parent; k_copy
//                                                      (Sec. II B, IV D, V A 1)
// Step (iv)  k_sweep_msc (all runs, lattice in LDS for all theta sweeps;
//            also compiled per lattice size and model), k_sweep_wide (one
//            colour of one run per launch, from memory), k_bytes_words (the
//            int8 layout to words and back), k_dos_sample (the theta =
//            infinity limit, Sec. V C)
// Step (v)   k_wang_lds, k_wang_pairs, k_wang_rows, k_wang_gather (permutation pairing,
//            Sec. III D), k_measure, k_meas_chunk
//                                                      (Eqs. (e)-(chi), Sec. III D)
// Sec. IV    k_logw, k_qweights, k_wavg, k_wavg_cumsum, k_wqhist, k_famstats
// Diagnostic k_philox_rate (integer-VALU calibration)
//
// Population-wide reductions and scans are split into fixed-size chunks of
// CH replicas (one workgroup each) plus a pass over the chunk totals by the
// workgroup that comes last, so every result is independent of the launch
// shape and the floating-point sums have one fixed order.
#include <float.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <map>
#include <mutex>
#include <type_traits>
#include <utility>
#include <vector>
#include <math.h>
#include <stdint.h>

#include "launch.hpp"
#include "metropolis.hpp"
#include "pa_internal.hpp"
#include "philox.hpp"
#include "unit_walk.hpp"

namespace pa {

// Index of this thread's wavefront in the workgroup, as a value the compiler
// knows to be uniform in the wavefront (loop bounds and counts derived from it
// then stay in scalar registers).
__device__ __forceinline__ int wave_id()
{
    return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
}

// ------------------------------------------------------------- utilities

__device__ __forceinline__ uint64_t umul64hi(uint64_t a, uint64_t b) { return __umul64hi(a, b); }

// Quotient and remainder of a / d, and floor(rem 2^32 / d), for d < 2^63 and
// quotients below 2^32: the FP64 estimates (relative error below 2^-50) are
// at most one off, which the exact remainder shows.  inv = 1 / (double)d.
__device__ __forceinline__ uint64_t div_exact(uint64_t a, uint64_t d, double inv, uint64_t &rem)
{
    uint64_t q = (uint64_t)((double)a * inv);
    int64_t r = (int64_t)(a - q * d);   // in (-d, 2d): a < 2^63, so no ambiguity
    if (r < 0) {
        --q;
        r += (int64_t)d;
    } else if ((uint64_t)r >= d) {
        ++q;
        r -= (int64_t)d;
    }
    rem = (uint64_t)r;
    return q;
}

__device__ __forceinline__ uint32_t frac32(uint64_t rem, uint64_t d, double inv)
{
    uint64_t q = (uint64_t)((double)rem * inv * 4294967296.0);
    // rem 2^32 - q d in 128 bits
    const uint64_t alo = rem << 32, plo = q * d, lo = alo - plo;
    const int64_t hi = (int64_t)((rem >> 32) - umul64hi(q, d) - (alo < plo ? 1u : 0u));
    if (hi < 0) --q;
    else if (hi > 0 || lo >= d) ++q;
    return (uint32_t)q;
}

template <typename T>
__device__ __forceinline__ T wave_sum(T v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

__device__ __forceinline__ int wave_min(int v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o, 64));
    return v;
}

// Values passed between workgroups of one launch: device-coherent stores and
// loads, ordered by waiting for the stores before the counter that announces
// them (no write-back of an L2).
template <typename T>
__device__ __forceinline__ void put(T *p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ T take(const T *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A thread's CH_PER consecutive elements, from index jb (a multiple of CH_PER)
// of a 256-byte aligned array: 16-byte accesses where all of them are below
// `end`, one by one in the last, partial block.  (A thread's elements one at
// a time touch as many lines per instruction as the wavefront has lanes.)
template <typename T>
__device__ __forceinline__ void load_block(const T *a, int jb, int end, T fill, T (&v)[CH_PER])
{
    constexpr int PER = 16 / sizeof(T);
    if (jb + CH_PER <= end) {
#pragma unroll
        for (int q = 0; q < CH_PER / PER; ++q) {
            const uint4 w = ((const uint4 *)(a + jb))[q];
            __builtin_memcpy(&v[q * PER], &w, 16);
        }
    } else {
#pragma unroll
        for (int q = 0; q < CH_PER; ++q) v[q] = jb + q < end ? a[jb + q] : fill;
    }
}

template <typename T>
__device__ __forceinline__ void store_block(T *a, int jb, int end, const T (&v)[CH_PER])
{
    constexpr int PER = 16 / sizeof(T);
    if (jb + CH_PER <= end) {
#pragma unroll
        for (int q = 0; q < CH_PER / PER; ++q) {
            uint4 w;
            __builtin_memcpy(&w, &v[q * PER], 16);
            ((uint4 *)(a + jb))[q] = w;
        }
    } else {
#pragma unroll
        for (int q = 0; q < CH_PER; ++q)
            if (jb + q < end) a[jb + q] = v[q];
    }
}

// Counts this workgroup in once its first thread's stores and atomics have
// completed; true in the workgroup that comes last of n.  The counter is zero
// again when it has come (one kernel of a step uses it after the other).  To
// be called by the whole workgroup; a barrier only for n > 1.
__device__ __forceinline__ bool last_of(int32_t *done, int n)
{
    __shared__ int last;
    if (n == 1) return true;   // nobody else: what it put is still its own
    if (threadIdx.x == 0) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        const int k = __hip_atomic_fetch_add(done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        last = k == n - 1;
        if (last) put(done, 0);
    }
    __syncthreads();
    return last;
}

__device__ __forceinline__ bool pop_active(const PopState &S) { return S.moved && S.status == PA_OK; }

// Value of lane (lane ^ J) for a 32-bit register, with the cheapest gfx950
// cross-lane form for each distance: permlane swaps for 32 and 16, an LDS
// swizzle for 8 and 4, DPP quad permutes for 2 and 1.
template <int J>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v)
{
    if constexpr (J == 32) {
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        return (threadIdx.x & 32) ? r[0] : r[1];
    } else if constexpr (J == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        return (threadIdx.x & 16) ? r[0] : r[1];
    } else if constexpr (J == 8 || J == 4) {
        return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, (J << 10) | 0x1f);
    } else if constexpr (J == 2) {
        return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, false);   // quad_perm [2,3,0,1]
    } else {
        return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, false);   // quad_perm [1,0,3,2]
    }
}

// One block-swap stage of the transpose for J < 32, on each 32-bit half:
// m holds the bit positions without bit J.  A lane without bit J keeps
// those and sends the others, moved down by J; its partner (lane ^ J) keeps
// the others and sends those, moved up by J.  Both moves are one rotation
// (right by J, or by 32 - J) followed by the kept-bits mask, since the bits
// that wrap around land outside it; no branch on the lane's side.
template <int J>
__device__ __forceinline__ void transpose_stage(uint32_t &lo, uint32_t &hi, uint32_t m)
{
    const uint32_t up = 0u - ((threadIdx.x / J) & 1u);   // all ones on lanes with bit J
    const uint32_t keep = m ^ up;
    const uint32_t sh = J + (up & (32u - 2u * J));
    const uint32_t slo = __builtin_amdgcn_alignbit(lo, lo, sh) & keep;
    const uint32_t shi = __builtin_amdgcn_alignbit(hi, hi, sh) & keep;
    lo = (lo & keep) | lane_xor<J>(slo);
    hi = (hi & keep) | lane_xor<J>(shi);
}

// 64 x 64 bit transpose across a wavefront: lane r holds row r (bit c =
// element (r, c)); on return lane r holds column r.  Six block-swap stages
// (distances 32, 16, 8, 4, 2, 1): the first exchanges one 32-bit half, the
// others exchange within each half.
__device__ __forceinline__ uint64_t transpose64(uint64_t x)
{
    uint32_t lo = (uint32_t)x, hi = (uint32_t)(x >> 32);
    {
        const bool up = threadIdx.x & 32;
        const uint32_t r = lane_xor<32>(up ? lo : hi);
        lo = up ? r : lo;
        hi = up ? hi : r;
    }
    transpose_stage<16>(lo, hi, 0x0000FFFFu);
    transpose_stage<8>(lo, hi, 0x00FF00FFu);
    transpose_stage<4>(lo, hi, 0x0F0F0F0Fu);
    transpose_stage<2>(lo, hi, 0x33333333u);
    transpose_stage<1>(lo, hi, 0x55555555u);
    return (uint64_t)lo | ((uint64_t)hi << 32);
}

// Bit-sliced (vertical) counters: plane k holds bit k of 64 per-lane counts.
constexpr int VB = 6;   // counts up to 63 per lane

// Carry-save counting of a block of 16 sites per lane, Harley and Seal's
// scheme in bit-sliced form: a three-input adder (sum = XOR, carry =
// majority, one bitop3 each per 32 bits) folds each site's inputs into the
// ones plane and passes its carry up; carries of equal weight wait for a
// partner from a later site, so after the 16th site the planes ones, twos,
// fours, eights and the sixteens are the binary digits of every lane's count.
// The site index t (the same on every lane) decides which carries pair up;
// every block takes exactly the 16 sites t = 0 .. 15 in order (zero inputs
// for missing ones).
__device__ __forceinline__ void csa(uint64_t &carry, uint64_t &sum, uint64_t a, uint64_t b, uint64_t c)
{
    const uint64_t s = bop3<LUT_XOR3>(a, b, c);
    carry = bop3<LUT_MAJ>(a, b, c);
    sum = s;
}

// One input per site: counts up to 16 in five planes.
struct Csa1 {
    uint64_t p1 = 0, p2 = 0, p4 = 0, p8 = 0, p16 = 0, w1 = 0, w2 = 0, w4 = 0, w8 = 0;
    __device__ __forceinline__ void add(int t, uint64_t a)
    {
        if (!(t & 1)) { w1 = a; return; }
        uint64_t c2, c4, c8;
        csa(c2, p1, p1, w1, a);
        if (!(t & 2)) { w2 = c2; return; }
        csa(c4, p2, p2, w2, c2);
        if (!(t & 4)) { w4 = c4; return; }
        csa(c8, p4, p4, w4, c4);
        if (!(t & 8)) { w8 = c8; return; }
        csa(p16, p8, p8, w8, c8);
    }
    __device__ __forceinline__ void planes(uint64_t (&p)[VB]) const
    {
        p[0] = p1; p[1] = p2; p[2] = p4; p[3] = p8; p[4] = p16; p[5] = 0;
    }
};

// Two inputs per site: counts up to 32 in six planes.
struct Csa2 {
    uint64_t p1 = 0, p2 = 0, p4 = 0, p8 = 0, s16a = 0, s16b = 0, w2 = 0, w4 = 0, w8 = 0;
    __device__ __forceinline__ void add(int t, uint64_t a, uint64_t b)
    {
        uint64_t c2, c4, c8;
        csa(c2, p1, p1, a, b);
        if (!(t & 1)) { w2 = c2; return; }
        csa(c4, p2, p2, w2, c2);
        if (!(t & 2)) { w4 = c4; return; }
        csa(c8, p4, p4, w4, c4);
        if (!(t & 4)) { w8 = c8; return; }
        csa((t & 8) ? s16b : s16a, p8, p8, w8, c8);
    }
    __device__ __forceinline__ void planes(uint64_t (&p)[VB]) const
    {
        p[0] = p1; p[1] = p2; p[2] = p4; p[3] = p8; p[4] = s16a ^ s16b; p[5] = s16a & s16b;
    }
};

// Incremental form (a half-adder chain per input), used where fewer
// registers matter more than fewer operations.
__device__ __forceinline__ void vinc(uint64_t (&p)[VB], uint64_t x)
{
#pragma unroll
    for (int k = 0; k < VB; ++k) {
        const uint64_t t = p[k] & x;
        p[k] ^= x;
        x = t;
    }
}

// add the 2-bit per-lane values a + b
__device__ __forceinline__ void vinc2(uint64_t (&p)[VB], uint64_t a, uint64_t b)
{
    const uint64_t s = a ^ b, c = a & b;
    const uint64_t t0 = p[0] & s;
    p[0] ^= s;
    uint64_t x = t0 | c;
#pragma unroll
    for (int k = 1; k < VB; ++k) {
        const uint64_t t = p[k] & x;
        p[k] ^= x;
        x = t;
    }
}

// Per-lane counts summed over the wavefront: on return lane b holds the
// total over all lanes of bit b's count, and the planes are cleared.  Only
// the lowest `used` planes (wavefront-uniform) can be non-zero.
__device__ __forceinline__ uint32_t vflush(uint64_t (&p)[VB], int used = VB)
{
    uint32_t total = 0;
#pragma unroll
    for (int k = 0; k < VB; ++k) {
        if (k < used) total += (uint32_t)__popcll(transpose64(p[k])) << k;
        p[k] = 0;
    }
    return total;
}

// Bit planes that hold counts up to c.
__device__ __forceinline__ int planes_for(int c) { return 32 - __clz(c); }

// Exclusive scan of one value per thread across a workgroup of BS threads
// (BS a multiple of 64); returns the exclusive prefix, *total the sum.
template <typename T, int BS>
__device__ __forceinline__ T block_exscan(T v, T *lds, T *total)
{
    const int lane = threadIdx.x & 63, wv = wave_id();
    T incl = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        T t = __shfl_up(incl, o, 64);
        if (lane >= o) incl += t;
    }
    if (lane == 63) lds[wv] = incl;
    __syncthreads();
    if (threadIdx.x == 0) {
        T run = 0;
        for (int k = 0; k < BS / 64; ++k) {
            T t = lds[k];
            lds[k] = run;
            run += t;
        }
        lds[BS / 64] = run;
    }
    __syncthreads();
    T res = lds[wv] + incl - v;
    *total = lds[BS / 64];
    __syncthreads();
    return res;
}

// ------------------------------------------------------------------ fill

__global__ void k_fill_u32(uint32_t *p, uint32_t v, uint64_t n)
{
    for (uint64_t k = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; k < n;
         k += (uint64_t)gridDim.x * blockDim.x)
        p[k] = v;
}

// -------------------------------------------------------------- step (i)

// Couplings of the +-J model: J_R(n) = -1 iff bit 0 of o0, J_D(n) = -1 iff
// bit 0 of o1, of Philox(disorder seed; n, 0, 0, TAG_J << 28).
__global__ void k_init_couplings(const RunInfo *runs, const uint64_t *dseed)
{
    const RunInfo &R = runs[blockIdx.x];
    const uint64_t ds = dseed[blockIdx.x];
    for (int n = threadIdx.x; n < R.N; n += blockDim.x) {
        uint8_t b = 0;
        if (R.model == PA_EA_PMJ) {
            const u32x4 o = philox10((uint32_t)n, 0, 0, TAG_J << 28, (uint32_t)ds, (uint32_t)(ds >> 32));
            b = (uint8_t)((o.x & 1u) | ((o.y & 1u) << 1));
        }
        R.jbits[n] = b;
    }
}

// Spins at beta_0 = 0: bit b of o0 | o1 << 32 of Philox(seed; n, g, 0,
// TAG_INIT << 28 | pop << 24) is replica 64 g + b at site n (set = -1).
template <int REPR>
__global__ void k_init_spins(const Item *items, const RunInfo *runs)
{
    const Item it = items[blockIdx.x];
    const RunInfo &R = runs[it.run];
    const uint32_t c3 = (TAG_INIT << 28) | ((uint32_t)it.pop << 24);
    for (int n = threadIdx.x; n < R.N; n += blockDim.x) {
        const u32x4 o = philox10((uint32_t)n, (uint32_t)it.group, 0, c3, R.key0, R.key1);
        const uint64_t plane = (uint64_t)o.x | ((uint64_t)o.y << 32);
        const size_t site = (size_t)it.group * R.N + n;
        if (REPR == PA_MSC64) {
            ((uint64_t *)R.spins[it.pop][0])[site] = plane;
        } else {
            uint4 *dst = (uint4 *)(R.spins[it.pop][0] + site * 64);
            for (int q = 0; q < 4; ++q) dst[q] = spins16((uint32_t)(plane >> (16 * q)) & 0xFFFFu);
        }
    }
}

__global__ void k_init_fam(const RunInfo *runs)
{
    const RunInfo &R = runs[blockIdx.x];
    for (int p = 0; p < R.npop; ++p)
        for (int j = threadIdx.x; j < R.R_cap; j += blockDim.x) {
            R.fam[p][0][j] = j < R.R ? j : 0;
            R.E[p][0][j] = 0;
        }
}

// ------------------------------------------------------------- step (ii)

// Reweighting, Eq. (tauBoltz)/(QBoltz): per chunk of CH replicas the partial
// sums of x_j = exp(-dbeta (E_j - E_min)) (FP64) and of X_j = floor(x_j 2^40)
// (exact); for multinomial resampling also the chunk-local exclusive prefix
// of X_j.  The temperature index is i = (index of the population) + 1.  The
// population's last chunk finishes the step: chunk bases of the prefix, ln Q_i
// and A_i.  (In a launch of its own that took 2-12 us, counting in takes 1-4;
// with 16-byte accesses 256 populations of 2e4 take 30 us, 65 in three
// launches.)
__global__ void __launch_bounds__(CH_THREADS) k_rw_chunk(const ChunkItem *items, const RunInfo *runs, PopState *st)
{
    __shared__ uint64_t lds64[CH_THREADS / 64 + 1];
    __shared__ double ldsd[CH_THREADS];
    const ChunkItem it = items[blockIdx.x];
    const RunInfo &R = runs[it.run];
    PopState &S = st[it.run * MAX_POP + it.pop];
    const int i = S.i + 1;
    if (S.status != PA_OK || i >= R.K) {
        if (it.chunk == 0 && threadIdx.x == 0) S.moved = 0;
        return;
    }
    const int Rp = S.Rcur;
    const int j0 = it.chunk * CH;
    if (j0 >= Rp) return;
    const int32_t *E = R.E[it.pop][S.cur];
    const int Np1 = R.N + 1;
    const uint64_t *X = R.tabX + (size_t)i * Np1;
    const double *x = R.tabx + (size_t)i * Np1;
    const int Emin = S.Emin;
    // each thread: CH_PER consecutive replicas, summed in order
    const int jb = j0 + threadIdx.x * CH_PER;
    double s = 0.0;
    uint64_t sx = 0;
    int32_t Ej[CH_PER];
    load_block(E, jb, Rp, Emin, Ej);
    uint64_t loc[CH_PER];
#pragma unroll
    for (int q = 0; q < CH_PER; ++q) {
        uint64_t Xj = 0;
        if (jb + q < Rp) {
            const int k = min(max((Ej[q] - Emin) >> 2, 0), R.N);
            Xj = X[k];
            s += x[k];
        }
        loc[q] = sx;
        sx += Xj;
    }
    uint64_t tot;
    const uint64_t pre = block_exscan<uint64_t, CH_THREADS>(sx, lds64, &tot);
    if (R.resampling == PA_MULTINOMIAL) {
#pragma unroll
        for (int q = 0; q < CH_PER; ++q) loc[q] += pre;
        store_block(R.P[it.pop], jb, Rp, loc);
    }
    // fixed-order FP64 tree: wave shuffles then waves in order
    double ws = s;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) ws += __shfl_xor(ws, o, 64);
    if ((threadIdx.x & 63) == 0) ldsd[threadIdx.x >> 6] = ws;
    __syncthreads();
    const int nch = (Rp + CH - 1) / CH;
    double part = 0.0;
    if (threadIdx.x == 0) {
        for (int k = 0; k < CH_THREADS / 64; ++k) part += ldsd[k];
        if (nch > 1) {
            put(&R.partS[it.pop][it.chunk], part);
            put(&R.tot64[it.pop][it.chunk], tot);
        }
    }
    if (!last_of(&S.done, nch)) return;

    // ln Q_i = ln S - ln R_{i-1} - dbeta E_min and A_i = A_{i-1} + ln Q_i,
    // Eqs. (QBoltz), (F); the chunks' sums added in order
    uint64_t carry = nch > 1 ? 0 : tot;
    double Ssum = nch > 1 ? 0.0 : part;
    if (nch == 1 && threadIdx.x == 0) R.base64[it.pop][0] = 0;
    for (int base = 0; nch > 1 && base < nch; base += CH_THREADS) {
        const int c = base + threadIdx.x;
        const uint64_t v = c < nch ? take(&R.tot64[it.pop][c]) : 0;
        ldsd[threadIdx.x] = c < nch ? take(&R.partS[it.pop][c]) : 0.0;
        uint64_t all;
        const uint64_t before = block_exscan<uint64_t, CH_THREADS>(v, lds64, &all);
        if (c < nch) R.base64[it.pop][c] = carry + before;
        carry += all;
        if (threadIdx.x == 0) {
            const int n = min(CH_THREADS, nch - base);
            for (int k = 0; k < n; ++k) Ssum += ldsd[k];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double db = R.beta[i] - R.beta[i - 1];
        const double lnQ = log(Ssum) - log((double)Rp) - db * (double)Emin;
        S.lnQ = lnQ;
        S.A = S.A + lnQ;
        S.S = Ssum;
        S.SX = carry;
        S.Rprev = Rp;
        S.i = i;
        S.moved = 1;
    }
}

// Clears what k_mn_draws adds to, for restored populations (k_parent leaves it
// clear, a checkpoint of an earlier build may not).
__global__ void __launch_bounds__(CH_THREADS) k_clear_draws(const ChunkItem *items, const RunInfo *runs)
{
    const ChunkItem it = items[blockIdx.x];
    const RunInfo &R = runs[it.run];
    if (R.resampling != PA_MULTINOMIAL || R.fused) return;
    for (int q = 0; q < CH_PER; ++q) {
        const int j = it.chunk * CH + q * CH_THREADS + (int)threadIdx.x;
        if (j < R.R_cap) R.C[it.pop][j] = 0;
    }
}

// ------------------------------------------------------------ step (iii)

__device__ __forceinline__ pa_obs &obs_at(const RunInfo &R, int i, int pop)
{
    return R.obs[(size_t)i * R.obs_stride + R.obs_off + pop];
}

__device__ void freeze_run(const RunInfo &R, PopState &S, int i, int pop, int32_t status)
{
    for (int k = i + threadIdx.x; k < R.K; k += blockDim.x) {
        pa_obs o = {};
        o.status = status;
        obs_at(R, k, pop) = o;
    }
    if (threadIdx.x == 0) {
        S.status = status;
        S.moved = 0;
    }
}

// R_i = sum r_j: capacity and empty-population checks (the run is frozen
// with that status); otherwise the new population becomes current: the copy
// reads buffer src, writes cur.  False if frozen.  By the whole workgroup.
__device__ __forceinline__ bool accept_counts(const RunInfo &R, PopState &S, int pop, int64_t total)
{
    if (total > R.R_cap || total == 0) {
        freeze_run(R, S, S.i, pop, total ? PA_ERR_CAPACITY : PA_ERR_NUMERIC);
        return false;
    }
    if (threadIdx.x == 0) {
        S.src = S.cur;
        S.cur = S.cur ^ 1;
        S.Rcur = (int32_t)total;
    }
    return true;
}

// Nearest-integer count of replica j with energy E: r_j = n_j + [u_j < t_j],
// n_j = floor(R X_j / S_X), t_j = floor((R X_j mod S_X) 2^32 / S_X), u_j = o0
// of Philox(seed; j, 0, i, TAG_NI << 28 | pop << 24).
__device__ __forceinline__ int nearest_count(const RunInfo &R, const PopState &S, int pop, int j, int E,
                                             const uint64_t *X, double invSX)
{
    const uint64_t RX = (uint64_t)R.R * X[min(max((E - S.Emin) >> 2, 0), R.N)];
    uint64_t rem;
    const uint64_t n = div_exact(RX, S.SX, invSX, rem);
    const uint32_t t = frac32(rem, S.SX, invSX);
    const u32x4 o = philox10((uint32_t)j, 0, (uint32_t)S.i, (TAG_NI << 28) | ((uint32_t)pop << 24), R.key0, R.key1);
    return (int)n + (o.x < t ? 1 : 0);
}

// Chunk bases of the count prefix and the checks, by the population's last
// chunk (the chunks' totals are in tot32).
__device__ __forceinline__ void finish_counts(const RunInfo &R, PopState &S, int pop, int tot0, int64_t *lds64)
{
    const int nch = (S.Rprev + CH - 1) / CH;
    int64_t carry = nch > 1 ? 0 : tot0;
    if (nch == 1 && threadIdx.x == 0) R.base32[pop][0] = 0;
    for (int base = 0; nch > 1 && base < nch; base += CH_THREADS) {
        const int c = base + threadIdx.x;
        const int64_t v = c < nch ? take(&R.tot32[pop][c]) : 0;
        int64_t tot;
        const int64_t pre = block_exscan<int64_t, CH_THREADS>(v, lds64, &tot);
        if (c < nch) R.base32[pop][c] = (int32_t)(carry + pre);
        carry += tot;
    }
    accept_counts(R, S, pop, carry);
}

// Nearest-integer counts and their chunk-local exclusive prefix.  The counts
// are taken a replica per thread and round (a thread's own eight in turn
// would be a chain of eight draws and divisions), then scanned from LDS in
// order.
__global__ void __launch_bounds__(CH_THREADS) k_cnt_chunk(const ChunkItem *items, const RunInfo *runs, PopState *st)
{
    __shared__ int32_t lds[CH_THREADS / 64 + 1];
    __shared__ int64_t lds64[CH_THREADS / 64 + 1];
    __shared__ int32_t cnt[CH];
    const ChunkItem it = items[blockIdx.x];
    const RunInfo &R = runs[it.run];
    PopState &S = st[it.run * MAX_POP + it.pop];
    if (!pop_active(S) || R.resampling != PA_NEAREST_INT || R.fused) return;
    const int Rp = S.Rprev;
    const int j0 = it.chunk * CH;
    if (j0 >= Rp) return;
    const int32_t *E = R.E[it.pop][S.cur];
    const uint64_t *X = R.tabX + (size_t)S.i * (R.N + 1);
    const double invSX = 1.0 / (double)S.SX;
    int32_t *r = R.r[it.pop];
    for (int q = 0; q < CH_PER; ++q) {
        const int k = q * CH_THREADS + threadIdx.x, j = j0 + k;
        int rj = 0;
        if (j < Rp) {
            rj = nearest_count(R, S, it.pop, j, E[j], X, invSX);
            r[j] = rj;
        }
        cnt[k] = rj;
    }
    __syncthreads();
    int32_t loc[CH_PER];
    int32_t sum = 0;
#pragma unroll
    for (int q = 0; q < CH_PER; ++q) {
        loc[q] = sum;
        sum += cnt[threadIdx.x * CH_PER + q];
    }
    int32_t tot;
    const int32_t pre = block_exscan<int32_t, CH_THREADS>(sum, lds, &tot);
#pragma unroll
    for (int q = 0; q < CH_PER; ++q) loc[q] += pre;
    store_block(R.C[it.pop], j0 + threadIdx.x * CH_PER, Rp, loc);
    if (threadIdx.x == 0) put(&R.tot32[it.pop][it.chunk], tot);
    if (last_of(&S.done, (Rp + CH - 1) / CH)) finish_counts(R, S, it.pop, tot, lds64);
}

// The largest j < n with P_j <= t, for ascending P, P_0 = 0, t < tot, P
// 16-byte aligned.  The weights of a population differ little, so P is close
// to a line: from the entry that the line gives, its distance to t gives one
// within a few places, and eight entries around that are read at once: two
// loads one after the other where halving takes eleven.  What lies further
// off is followed the same way, then by halving.
__device__ __forceinline__ int last_not_above(const uint64_t *P, int n, uint64_t tot, uint64_t t)
{
    const double per = (double)n / (double)tot;
    int lo = 0, hi = n;   // P_lo <= t, P_hi > t
    int g = min(n - 1, (int)((double)t * per));
    g += (int)((double)(int64_t)(t - P[g]) * per);
    for (int tries = 0; tries < 4 && hi - lo > 1; ++tries) {
        const int w = max(0, min(g - 4, n - 8)) & ~1;
        uint64_t e[8];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (w + 8 <= n) {
                const ulonglong2 v = ((const ulonglong2 *)(P + w))[q];
                e[2 * q] = v.x;
                e[2 * q + 1] = v.y;
            } else {
                e[2 * q] = w + 2 * q < n ? P[w + 2 * q] : ~(uint64_t)0;
                e[2 * q + 1] = w + 2 * q + 1 < n ? P[w + 2 * q + 1] : ~(uint64_t)0;
            }
        }
        int c = 0;
#pragma unroll
        for (int q = 0; q < 8; ++q) c += e[q] <= t ? 1 : 0;
        if (c == 0) {
            hi = w;
            g = w - 1 - (int)((double)(e[0] - t) * per);
        } else if (c == 8 && w + 8 < n) {
            lo = w + 7;
            g = w + 8 + (int)((double)(t - e[7]) * per);
        } else {
            lo = w + c - 1;
            hi = lo + 1;
        }
    }
    while (hi - lo > 1) {
        const int m = (lo + hi) >> 1;
        if (P[m] <= t) lo = m;
        else hi = m;
    }
    return lo;
}

// Multinomial draws: draw d picks the parent j with P_j <= t < P_j + X_j,
// t = floor(v S_X / 2^64), v = o0 | o1 << 32 of Philox(seed; d, 0, i,
// TAG_MN << 28 | pop << 24); P_j = base64[chunk] + chunk-local prefix.
// CH_PER workgroups per chunk item, each one round of CH_THREADS draws: the
// searches are chains of dependent loads at scattered addresses, so they are
// spread over as many compute units as possible.  Two populations of 2e5:
// 24 us, 32 by halving; 2e4: 5.4 and 6.7.  They are counted in C, which is
// clear here: the counts of the last resampling stay in r until the next one
// has its own.
__global__ void __launch_bounds__(CH_THREADS) k_mn_draws(const ChunkItem *items, const RunInfo *runs,
                                                          const PopState *st)
{
    const int part = blockIdx.x % CH_PER;
    const ChunkItem it = items[blockIdx.x / CH_PER];
    const RunInfo &R = runs[it.run];
    const PopState &S = st[it.run * MAX_POP + it.pop];
    if (!pop_active(S) || R.resampling != PA_MULTINOMIAL || R.fused) return;
    const int d0 = it.chunk * CH;
    if (d0 >= R.R) return;
    const int Rp = S.Rprev;
    const uint64_t SX = S.SX;
    const uint64_t *P = R.P[it.pop];
    const uint64_t *B = R.base64[it.pop];
    const uint32_t c3 = (TAG_MN << 28) | ((uint32_t)it.pop << 24);
    int32_t *C = R.C[it.pop];
    __shared__ uint64_t sB[CH];   // the chunk bases
    // largest j with P_j <= t in two levels: the last chunk whose base is
    // <= t (chunk bases staged in LDS), then inside it (last_not_above)
    const int nch = (Rp + CH - 1) / CH;
    const bool staged = nch <= CH;
    if (staged)
        for (int k = threadIdx.x; k < nch; k += CH_THREADS) sB[k] = B[k];
    __syncthreads();
    const int d = d0 + part * CH_THREADS + (int)threadIdx.x;
    if (d < R.R) {
        const u32x4 o = philox10((uint32_t)d, 0, (uint32_t)S.i, c3, R.key0, R.key1);
        const uint64_t v = (uint64_t)o.x | ((uint64_t)o.y << 32);
        const uint64_t t = umul64hi(v, SX);
        // the chunk, by halving in power-of-two steps from the first, whose
        // base is 0
        int k = 0;
        for (int step = nch > 1 ? 1 << (31 - __builtin_clz(nch - 1)) : 0; step > 0; step >>= 1) {
            const int m = k + step;
            if (m < nch && (staged ? sB[m] : B[m]) <= t) k = m;
        }
        const uint64_t base = staged ? sB[k] : B[k];
        const uint64_t tot = (k + 1 < nch ? (staged ? sB[k + 1] : B[k + 1]) : SX) - base;
        atomicAdd(&C[k * CH + last_not_above(P + (size_t)k * CH, min(CH, Rp - k * CH), tot, t - base)], 1);
    }
}

// Multinomial: the counts r and their chunk-local exclusive prefix C, from the
// draws counted in C.
__global__ void __launch_bounds__(CH_THREADS) k_cnt_scan_chunk(const ChunkItem *items, const RunInfo *runs,
                                                                PopState *st)
{
    __shared__ int32_t lds[CH_THREADS / 64 + 1];
    __shared__ int64_t lds64[CH_THREADS / 64 + 1];
    const ChunkItem it = items[blockIdx.x];
    const RunInfo &R = runs[it.run];
    PopState &S = st[it.run * MAX_POP + it.pop];
    if (!pop_active(S) || R.resampling != PA_MULTINOMIAL || R.fused) return;
    const int Rp = S.Rprev;
    const int j0 = it.chunk * CH;
    if (j0 >= Rp) return;
    const int jb = j0 + threadIdx.x * CH_PER;
    int32_t rj[CH_PER], loc[CH_PER];
    load_block(R.C[it.pop], jb, Rp, 0, rj);
    store_block(R.r[it.pop], jb, Rp, rj);
    int32_t sum = 0;
#pragma unroll
    for (int q = 0; q < CH_PER; ++q) {
        loc[q] = sum;
        sum += rj[q];
    }
    int32_t tot;
    const int32_t pre = block_exscan<int32_t, CH_THREADS>(sum, lds, &tot);
#pragma unroll
    for (int q = 0; q < CH_PER; ++q) loc[q] += pre;
    store_block(R.C[it.pop], jb, Rp, loc);
    if (threadIdx.x == 0) put(&R.tot32[it.pop][it.chunk], tot);
    if (last_of(&S.done, (Rp + CH - 1) / CH)) finish_counts(R, S, it.pop, tot, lds64);
}

// Parent of every child slot: parent j's r_j children occupy the slots
// C_j .. C_j + r_j - 1, so each parent writes its own.  A lane writes the
// first few; the slots of larger families are written by the whole
// wavefront, one family at a time.  By the whole wavefront, rj = 0 on lanes
// without a parent.
constexpr int PARENT_LANE_MAX = 4;

__device__ __forceinline__ void write_children(int32_t *par, int j, int cj, int rj)
{
    const int lane = threadIdx.x & 63;
    const int mine = min(rj, PARENT_LANE_MAX);
    for (int m = 0; m < mine; ++m) par[cj + m] = j;
    uint64_t big = __ballot(rj > PARENT_LANE_MAX);
    while (big) {
        const int src = __ffsll((unsigned long long)big) - 1;
        big &= big - 1;
        const int bj = __builtin_amdgcn_readlane(j, src), bc = __builtin_amdgcn_readlane(cj, src),
                  br = __builtin_amdgcn_readlane(rj, src);
        for (int m = PARENT_LANE_MAX + lane; m < br; m += 64) par[bc + m] = bj;
    }
}

// C_j = base32[chunk] + chunk-local prefix; multinomial draws find C clear again.
__global__ void __launch_bounds__(CH_THREADS) k_parent(const ChunkItem *items, const RunInfo *runs,
                                                        const PopState *st)
{
    const ChunkItem it = items[blockIdx.x];
    const RunInfo &R = runs[it.run];
    const PopState &S = st[it.run * MAX_POP + it.pop];
    if (!pop_active(S) || R.fused) return;
    const int Rp = S.Rprev;
    const int j0 = it.chunk * CH;
    if (j0 >= Rp) return;
    int32_t *C = R.C[it.pop];
    const int32_t *r = R.r[it.pop];
    const int32_t base = R.base32[it.pop][it.chunk];
    const bool mn = R.resampling == PA_MULTINOMIAL;
#pragma unroll
    for (int q = 0; q < CH_PER; ++q) {
        const int j = j0 + q * CH_THREADS + (int)threadIdx.x;
        const bool in = j < Rp;
        const int cj = in ? base + C[j] : 0;
        if (in && mn) C[j] = 0;
        write_children(R.parent[it.pop], j, cj, in ? r[j] : 0);
    }
}

// Step (iii) up to the copy for a run that fits one workgroup per population
// (R.fused): counts in LDS, their prefix, the checks and the parent map, in
// place of four launches.  The counts are 16 bits wide (a run of at most
// FUSED_MAX replicas draws no more), two to a word.  Multinomial draws search
// in LDS alone: a guide (where in the coarse prefix a draw with these high
// bits must lie), the coarse prefix (every CH_PER-th replica), then the fine
// one inside the block, kept as the 32 high bits of its offset from the
// block's first (offsets are below CH_PER 2^40); a draw whose high bits equal
// the one found reads the exact prefix.  Bound by the latency of a single
// workgroup's passes where there are few populations, by LDS reads and the
// generator where every CU has one.  Draws, scan, checks and parent map for
// 256 populations of 2e4: 58 us, 303 in launches with eleven dependent reads
// of memory per draw; one of 1000: 10, 16 before.  Where it pays against the
// present launches: resampled_alone.
constexpr int FINE_SHIFT = 11;
static_assert(CH_PER == 8, "40 + 3 bits of offset");
constexpr int GUIDE_BITS = 11;

__global__ void __launch_bounds__(1024) k_resample_run(const RunInfo *runs, PopState *st)
{
    // counts, coarse prefix, fine prefix (fused_lds)
    extern __shared__ __align__(16) uint64_t lds[];
    __shared__ uint16_t guide[(1 << GUIDE_BITS) + 2];
    __shared__ int32_t wsum[17];
    const int run = blockIdx.x, pop = blockIdx.y;
    const RunInfo &R = runs[run];
    if (pop >= R.npop || !R.fused) return;
    PopState &S = st[run * MAX_POP + pop];
    if (!pop_active(S)) return;
    const int tid = threadIdx.x, T = blockDim.x, lane = tid & 63, wv = wave_id(), nw = T >> 6;
    const int Rp = S.Rprev, n8 = (Rp + CH_PER - 1) / CH_PER;
    const bool mn = R.resampling == PA_MULTINOMIAL;
    uint32_t *cnt = (uint32_t *)lds;
    uint64_t *T8 = lds + 2 * (size_t)n8;
    uint32_t *F = (uint32_t *)((uint8_t *)lds + fused_fine_at(n8));
    const uint64_t SX = S.SX;
    if (mn) {
        for (int k = tid; k < n8 * (CH_PER / 2); k += T) cnt[k] = 0;
        // a thread takes blocks of CH_PER prefixes with 16-byte loads, all of a
        // block in flight together
        const uint64_t *B = R.base64[pop], *P = R.P[pop];
        for (int k = tid; k < n8; k += T) {
            uint64_t p[CH_PER];
            load_block(P, k * CH_PER, Rp, ~(uint64_t)0, p);
            T8[k] = B[k / (CH / CH_PER)] + p[0];
            uint32_t f[CH_PER];
#pragma unroll
            for (int q = 0; q < CH_PER; ++q) f[q] = k * CH_PER + q < Rp ? (uint32_t)((p[q] - p[0]) >> FINE_SHIFT) : ~0u;
#pragma unroll
            for (int q = 0; q < CH_PER; q += 4)
                ((uint4 *)F)[k * (CH_PER / 4) + q / 4] = make_uint4(f[q], f[q + 1], f[q + 2], f[q + 3]);
        }
        __syncthreads();
        // largest b with T8[b] <= t, starting from block b0 (T8[b0] <= t) in
        // power-of-two steps below span
        auto search = [&](uint64_t t, int b0, int span) {
            int b = b0;
            for (int step = span; step > 0; step >>= 1) {
                const int m = b + step;
                if (m < n8 && T8[m] <= t) b = m;
            }
            return b;
        };
        const int top = n8 > 1 ? 1 << (31 - __builtin_clz(n8 - 1)) : 0;
        const bool guided = n8 > 128;
        if (guided) {
            for (int g = tid; g <= (1 << GUIDE_BITS); g += T)
                guide[g] = (uint16_t)(g >> GUIDE_BITS ? n8 - 1
                                                      : search(umul64hi((uint64_t)g << (64 - GUIDE_BITS), SX), 0, top));
            __syncthreads();
        }
        // draw d picks the largest j with P_j <= t (see k_mn_draws)
        const uint32_t c3 = (TAG_MN << 28) | ((uint32_t)pop << 24);
        for (int d = tid; d < R.R; d += T) {
            const u32x4 o = philox10((uint32_t)d, 0, (uint32_t)S.i, c3, R.key0, R.key1);
            const uint64_t t = umul64hi((uint64_t)o.x | ((uint64_t)o.y << 32), SX);
            int b = 0, span = top;
            if (guided) {
                const int g = (int)(o.y >> (32 - GUIDE_BITS));
                b = guide[g];
                const int w = guide[g + 1] - b;   // t is below the next entry's block end
                span = w > 0 ? 1 << (31 - __builtin_clz(w)) : 0;
            }
            b = search(t, b, span);
            const uint64_t rel = t - T8[b];
            const uint32_t f = (uint32_t)(rel >> FINE_SHIFT);
            const uint32_t *Fb = F + b * CH_PER;
            int j = 0;
#pragma unroll
            for (int step = CH_PER / 2; step > 0; step >>= 1)
                if (Fb[j + step] <= f) j += step;
            if (j > 0 && Fb[j] == f) {   // the exact prefix decides
                const uint64_t *P = R.P[pop] + (size_t)b * CH_PER;
                while (j > 0 && P[j] - P[0] > rel) --j;
            }
            j += b * CH_PER;
            atomicAdd(&cnt[j >> 1], 1u << (16 * (j & 1)));
        }
    } else {
        const int32_t *E = R.E[pop][S.cur];
        const uint64_t *X = R.tabX + (size_t)S.i * (R.N + 1);
        const double invSX = 1.0 / (double)SX;
        // every count is stored here, those past the population as zeros: a
        // clearing pass before this one would be other wavefronts' stores to
        // the same words
        for (int j = tid; j < n8 * CH_PER; j += T)
            ((uint16_t *)cnt)[j] = j < Rp ? (uint16_t)nearest_count(R, S, pop, j, E[j], X, invSX) : (uint16_t)0;
    }
    __syncthreads();
    // population size first: nothing is written for one that is refused
    auto block_sum = [&](int v) {
        const int w = wave_sum<int>(v);
        if (lane == 0) wsum[wv] = w;
        __syncthreads();
        int t = 0;
        for (int k = 0; k < nw; ++k) t += wsum[k];
        __syncthreads();
        return t;
    };
    int total = R.R;
    if (!mn) {
        int s = 0;
        for (int k = tid; k < n8 * (CH_PER / 2); k += T) s += (int)(cnt[k] & 0xFFFFu) + (int)(cnt[k] >> 16);
        total = block_sum(s);
    }
    int32_t *r = R.r[pop], *par = R.parent[pop];
    if (!accept_counts(R, S, pop, total)) {
        for (int j = tid; j < Rp; j += T) r[j] = ((const uint16_t *)cnt)[j];
        return;
    }
    // exclusive prefix over blocks of CH_PER consecutive replicas per thread,
    // and each parent's children (slots C_j .. C_j + r_j - 1)
    int carry = 0;
    for (int base = 0; base < n8; base += T) {
        const int b = base + tid;
        int c[CH_PER], s = 0;
#pragma unroll
        for (int q = 0; q < CH_PER / 2; ++q) {
            const uint32_t w = b < n8 ? cnt[b * (CH_PER / 2) + q] : 0u;
            c[2 * q] = (int)(w & 0xFFFFu);
            c[2 * q + 1] = (int)(w >> 16);
            s += c[2 * q] + c[2 * q + 1];
        }
        int incl = s;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int t = __shfl_up(incl, o, 64);
            if (lane >= o) incl += t;
        }
        if (lane == 63) wsum[wv] = incl;
        __syncthreads();
        int before = carry, all = 0;
        for (int k = 0; k < nw; ++k) {
            before += k < wv ? wsum[k] : 0;
            all += wsum[k];
        }
        __syncthreads();
        carry += all;
        int slot = before + incl - s;
        store_block(r, b * CH_PER, Rp, c);
#pragma unroll
        for (int q = 0; q < CH_PER; ++q) {
            write_children(par, b * CH_PER + q, slot, c[q]);
            slot += c[q];
        }
    }
}

// Copy of spins, energies and family labels into the child slots.  One
// wavefront per 64 children (one replica group) and 64 sites at a time.
// MSC: the children's parents lie in a few consecutive source groups; each
// source block (64 sites x 64 replicas) is transposed so that a lane holds
// one replica's 64 sites, every child pulls its parent's row from the lane
// that holds it, and the child block is transposed back and stored
// (falls back to a per-site bit gather when the parents span many groups).
// int8: lane = child, one byte per site.
constexpr int COPY_MAX_SRC = 4;

template <int REPR>
__device__ __forceinline__ void copy_group(const RunInfo &R, const PopState &S, int pop, int G, int sub, int wpg)
{
    const int Rc = S.Rcur;
    const int lane = threadIdx.x & 63;
    const int c = G * 64 + lane;
    const bool valid = c < Rc;
    const int clast = min(Rc, G * 64 + 64) - 1;
    const int p = R.parent[pop][valid ? c : clast];
    const int N = R.N;
    if (REPR == PA_MSC64) {
        const uint64_t *src = (const uint64_t *)R.spins[pop][S.src];
        uint64_t *dst = (uint64_t *)R.spins[pop][S.cur] + (size_t)G * N;
        // parents ascend with the children: the first and last lanes bound them
        const int g_lo = __builtin_amdgcn_readlane(p, 0) >> 6;
        const int g_hi = __builtin_amdgcn_readlane(p, 63) >> 6;
        if (g_hi - g_lo < COPY_MAX_SRC) {
            const int nsrc = g_hi - g_lo + 1;   // uniform over the wavefront
            // two 64-site blocks per step: their source loads are issued together
            for (int n0 = sub * 64; n0 < N; n0 += 2 * wpg * 64) {
                const int na = n0 + lane, nb = n0 + wpg * 64 + lane;
                uint64_t xa[COPY_MAX_SRC], xb[COPY_MAX_SRC];
#pragma unroll
                for (int q = 0; q < COPY_MAX_SRC; ++q) {
                    const size_t gofs = (size_t)(g_lo + q) * N;
                    xa[q] = (q < nsrc && na < N) ? src[gofs + na] : 0ull;
                    xb[q] = (q < nsrc && nb < N) ? src[gofs + nb] : 0ull;
                }
                uint64_t rowa = 0, rowb = 0;
#pragma unroll
                for (int q = 0; q < COPY_MAX_SRC; ++q) {
                    if (q < nsrc) {
                        const uint64_t va = __shfl(transpose64(xa[q]), p & 63, 64);
                        const uint64_t vb = __shfl(transpose64(xb[q]), p & 63, 64);
                        if ((p >> 6) == g_lo + q) {
                            rowa = va;
                            rowb = vb;
                        }
                    }
                }
                if (!valid) rowa = rowb = 0;
                const uint64_t outa = transpose64(rowa), outb = transpose64(rowb);
                if (na < N) dst[na] = outa;
                if (nb < N) dst[nb] = outb;
            }
        } else {
            const uint64_t *ps = src + (size_t)(p >> 6) * N;
            const int pb = p & 63;
            for (int nb = sub * 64; nb < N; nb += wpg * 64) {
                uint64_t mine = 0;
                const int cnt = min(64, N - nb);
                for (int k = 0; k < cnt; ++k) {
                    const int bit = valid ? (int)((ps[nb + k] >> pb) & 1u) : 0;
                    const uint64_t m = __ballot(bit);
                    if (lane == k) mine = m;
                }
                if (lane < cnt) dst[nb + lane] = mine;
            }
        }
    } else if ((__builtin_amdgcn_readlane(p, 63) >> 6) - (__builtin_amdgcn_readlane(p, 0) >> 6) < 2) {
        // the parents lie in at most two source groups: each lane packs the
        // 64 spin bytes of one site of each source group into a word (16-byte
        // loads), the words go through the bit-packed copy above, and the
        // child word is unpacked into 64 canonical bytes (16-byte stores)
        const uint8_t *srcb = R.spins[pop][S.src];
        uint8_t *dstb = R.spins[pop][S.cur] + (size_t)G * N * 64;
        const int g_lo = __builtin_amdgcn_readlane(p, 0) >> 6;
        const int nsrc = (__builtin_amdgcn_readlane(p, 63) >> 6) - g_lo + 1;   // 1 or 2, uniform
        for (int n0 = sub * 64; n0 < N; n0 += 2 * wpg * 64) {
            uint4 v[2][2][4];
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const int n = min(n0 + b * wpg * 64 + lane, N - 1);
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const uint4 *s4 = (const uint4 *)(srcb + ((size_t)(g_lo + min(q, nsrc - 1)) * N + n) * 64);
#pragma unroll
                    for (int k = 0; k < 4; ++k) v[b][q][k] = s4[k];
                }
            }
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                uint64_t row = 0;
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    if (q < nsrc) {
                        const uint64_t t = __shfl(transpose64(pack64(v[b][q])), p & 63, 64);
                        if ((p >> 6) == g_lo + q) row = t;
                    }
                }
                if (!valid) row = 0;   // slots past the population hold +1 spins
                const uint64_t out = transpose64(row);
                const int n = n0 + b * wpg * 64 + lane;
                if (n0 + b * wpg * 64 < N && n < N) {
                    uint4 *d4 = (uint4 *)(dstb + (size_t)n * 64);
#pragma unroll
                    for (int k = 0; k < 4; ++k) d4[k] = spins16((uint32_t)(out >> (16 * k)) & 0xFFFFu);
                }
            }
        }
    } else {
        const uint8_t *src = R.spins[pop][S.src] + (size_t)(p >> 6) * N * 64 + (p & 63);
        uint8_t *dst = R.spins[pop][S.cur] + (size_t)G * N * 64 + lane;
        // eight sites per step, all loads issued before the stores (the
        // buffers differ, but the compiler cannot know it)
        constexpr int U = 8;
        for (int n0 = sub; n0 < N; n0 += U * wpg) {
            uint8_t v[U];
#pragma unroll
            for (int q = 0; q < U; ++q) {
                const int n = n0 + q * wpg;
                v[q] = (valid && n < N) ? src[(size_t)n * 64] : (uint8_t)1;
            }
#pragma unroll
            for (int q = 0; q < U; ++q) {
                const int n = n0 + q * wpg;
                if (n < N) dst[(size_t)n * 64] = v[q];
            }
        }
    }
    if (sub == 0 && valid) {
        R.E[pop][S.cur][c] = R.E[pop][S.src][p];
        R.fam[pop][S.cur][c] = R.fam[pop][S.src][p];
    }
}

// Workgroup b of a launch runs on XCD b mod 8 (round-robin dispatch, one L2
// per XCD).  The item taken by b gives every XCD a contiguous range of
// items, so neighbouring items share their XCD's L2.  A bijection of
// [0, n) for any n.
__device__ __forceinline__ int xcd_item(int b, int n)
{
    const int q = n >> 3, r = n & 7, x = b & 7;
    return x * q + min(x, r) + (b >> 3);
}

// Workgroups of MEAS_WAVES wavefronts over the measure items: each group
// gets meas_waves_per_group(N) wavefronts, which split its sites.  The
// children of neighbouring groups have parents in shared source groups, so
// neighbouring items run on one XCD.
// split workgroups share an item: workgroup h of it takes the h-th share of
// each group's 64-site blocks (more wavefronts in flight for large lattices,
// each with a shorter chain of loads and transposes).
template <int REPR>
__global__ void __launch_bounds__(MEAS_THREADS) k_copy(const SweepItem *items, const RunInfo *runs,
                                                       const PopState *st, int split)
{
    const int b = xcd_item(blockIdx.x, gridDim.x);
    const SweepItem it = items[b / split];
    const int h = b - (b / split) * split;
    const RunInfo &R = runs[it.run];
    const PopState &S = st[it.run * MAX_POP + it.pop];
    if (!pop_active(S)) return;
    const int wpg = meas_waves_per_group(R.N);
    const int wv = wave_id();
    const int k = wv / wpg, sub = wv - k * wpg;
    const int G = it.group0 + k;
    if (k >= it.ngroups || G * 64 >= S.Rcur) return;
    copy_group<REPR>(R, S, it.pop, G, h * wpg + sub, split * wpg);
}

// ------------------------------------------------------------- step (iv)

// The sweep kernels' exact work counters: one set of atomics per
// wavefront, into a slot chosen by workgroup and wavefront.
__device__ __forceinline__ void flush_stats(unsigned long long *stats, uint64_t words, uint32_t calls,
                                            uint64_t flips)
{
    const unsigned long long w = wave_sum<unsigned long long>(words);
    const unsigned long long c = wave_sum<unsigned long long>(calls);
    const unsigned long long f = wave_sum<unsigned long long>(flips);
    if ((threadIdx.x & 63) == 0) {
        const unsigned slot = (blockIdx.x * 16u + (threadIdx.x >> 6)) % STAT_SLOTS;
        unsigned long long *p = stats + (size_t)slot * NSTAT;
        atomicAdd(&p[ST_WORDS], w);
        atomicAdd(&p[ST_CALLS], c);
        atomicAdd(&p[ST_FLIPS], f);
    }
}

__device__ __forceinline__ uint64_t jmask(uint8_t b, int bit) { return ((b >> bit) & 1u) ? ~0ull : 0ull; }

// Configurations of a population as bit-packed words ([group][site], 64
// replicas each): the population itself in the bit-packed layout; in the int8
// layout ([group][site][64 replicas] bytes) a copy in the idle spin buffer
// that the sweeps work on and the measurement reads (the second eighth of it:
// the first holds the permutation pairing's partner words).
__device__ __forceinline__ uint64_t *words_of(const RunInfo &R, const PopState &S, int pop)
{
    return R.bytes ? (uint64_t *)R.spins[pop][S.cur ^ 1] + (size_t)R.groups_cap * R.N
                   : (uint64_t *)R.spins[pop][S.cur];
}

// The words of the int8 layout are current from a step's sweeps until its
// population is resampled.
__device__ __forceinline__ bool words_current(const RunInfo &R, const PopState &S)
{
    return !R.bytes || (R.theta > 0 && S.i > 0);
}

// int8 layout: a population's bytes to its words and back, around the sweeps.
// A thread takes 16-byte chunks (16 replicas of one site) at consecutive
// addresses; a workgroup WORDS_SEG sites of one replica group.  Bound by
// memory: 72 bytes per site and group of 64 replicas either way.  (The byte
// layout was swept in place before, one colour per launch: 608 us for ten
// sweeps at L = 64, R = 2e4, where conversions and sweeps take 219.)
constexpr int WORDS_SEG = 1024;

template <bool TO_WORDS>
__global__ void __launch_bounds__(256) k_bytes_words(const Item *items, const RunInfo *runs, const PopState *st)
{
    const Item it = items[blockIdx.x];
    const RunInfo &R = runs[it.run];
    const PopState &S = st[it.run * MAX_POP + it.pop];
    const int n0 = blockIdx.y * WORDS_SEG;
    if (!pop_active(S) || R.theta == 0 || it.group * 64 >= S.Rcur || n0 >= R.N) return;
    const int chunks = 4 * min(WORDS_SEG, R.N - n0);
    uint4 *bytes = (uint4 *)(R.spins[it.pop][S.cur] + ((size_t)it.group * R.N + n0) * 64);
    uint16_t *words = (uint16_t *)(words_of(R, S, it.pop) + (size_t)it.group * R.N + n0);
    // the chunks of a round in flight together, with no branch around a load
    constexpr int U = 4;
    for (int c0 = threadIdx.x; c0 < chunks; c0 += 256 * U) {
        if constexpr (TO_WORDS) {
            uint4 v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = bytes[min(c0 + 256 * u, chunks - 1)];
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (c0 + 256 * u < chunks) words[c0 + 256 * u] = (uint16_t)signs16(v[u]);
        } else {
            uint32_t v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = words[min(c0 + 256 * u, chunks - 1)];
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (c0 + 256 * u < chunks) bytes[c0 + 256 * u] = spins16(v[u]);
        }
    }
}

// Batched path: every (run, pop, block of G replica groups) item of the
// context in one launch.  The G lattices (colour-split, so a colour's sites
// are contiguous) and the couplings stay in LDS for all theta sweeps.
//
// Draw scheduling.  A site needs as many Philox calls as its slowest
// undecided replica (about 3-4 on average, up to 16).  Each wavefront owns a
// contiguous range of a colour's sites, whole chunks of 64, and works in
// rounds:
//  - dense rounds: chunks of 64 sites are classified and make calls
//    0 .. dense-1 in lockstep; nearly every site needs that many, so few
//    lanes idle;
//  - sparse rounds: the sites still undecided are kept in a wave-private LDS
//    list.  It is a queue (stream_item) whose entries are the site's next
//    Philox counter word itself, and every round takes the next 64 entries
//    whatever call each is at; or (general_item: several groups of a lattice
//    above 4096 sites, 16 lockstep calls, or lists pooled over the workgroup)
//    the list is compacted in place after every call index.  Either way the
//    calls run on full wavefronts until the last entries.
// Every site's result is still the plain most-significant-first comparison
// of its own bit planes; only the order of the work changes.

// Lanes of the wavefront where p holds.  Unlike __ballot(int), the
// predicate stays a lane mask: a condition combined from several compares
// is not turned into an integer and compared again.
__device__ __forceinline__ uint64_t wave_ballot(bool p)
{
    return __builtin_amdgcn_ballot_w64(p);
}

// Flips the accepted replicas of a lattice word in LDS with one atomic XOR
// that returns nothing: no read into registers, no wait, and no test for an
// empty mask (XOR with zero changes nothing).  The words of one round are
// distinct sites, and a wavefront's LDS operations complete in order.
__device__ __forceinline__ void flip_word(uint64_t *w, uint64_t acc)
{
    __hip_atomic_fetch_xor(w, acc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// b plus the number of lanes below this one whose bit is set in the
// wavefront mask m (two mbcnt instructions).
__device__ __forceinline__ int rank_below(uint64_t m, int b)
{
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, (uint32_t)b));
}

// A list entry's undecided replicas and their class (set: dE = +4), kept
// side by side so that one LDS address serves both.  Reads are one 16-byte
// access (ds_read_b128).  Writes go out as two 8-byte halves of one
// instruction (ds_write2_b64): with 16-byte writes the wavefronts waited
// longer for LDS issue and the sweep was slower.
struct alignas(16) UndPair {
    uint64_t und, one;
};

__device__ __forceinline__ void und_load(const UndPair *p, uint64_t &und, uint64_t &one)
{
    const UndPair v = *p;
    und = v.und;
    one = v.one;
}

__device__ __forceinline__ void und_store(UndPair *p, uint64_t und, uint64_t one)
{
    uint64_t *w = (uint64_t *)(void *)p;   // 8-byte alignment: two 8-byte halves
    w[0] = und;
    w[1] = one;
}

// Sparse rounds of one wavefront over its own compacted list of `cnt`
// undecided sites (entries: lanes of each class, LDS word << 16 | site):
// call c for every entry, survivors compacted in place; once one pass holds
// every remaining entry it runs all their remaining calls without writing
// the list back.
__device__ __forceinline__ void sweep_sparse_wave(uint64_t *lat, UndPair *eu, uint32_t *en, int cnt,
                                                  int c_first, float invN, int group0, const Thresholds &Th, uint32_t i,
                                                  uint32_t c3, uint32_t key0, uint32_t key1, uint32_t &wcalls)
{
    const int lane = threadIdx.x & 63;
    for (int c = c_first; c < 16 && cnt > 0; ++c) {
        if (cnt <= 64) {
            uint64_t und = 0, one = 0, acc = 0;
            int addr = 0;
            uint32_t n = 0, g = 0;
            if (lane < cnt) {
                und_load(&eu[lane], und, one);
                const uint32_t pk = en[lane];
                addr = (int)(pk >> 16);
                n = pk & 0xFFFFu;
                g = (uint32_t)(group0 + div_small(addr, invN));
            }
            const uint64_t drew = und;
            for (; c < 16; ++c) {
                const uint64_t live = wave_ballot(und != 0);
                if (live == 0) break;
                wcalls += (uint32_t)__popcll(live);
                if (und != 0) {
                    const uint64_t was = und;
                    const uint64_t less = draw_call((uint32_t)c, call_masks(Th.t4, Th.t8, (uint32_t)c), one, und, n, g,
                                                    i, c3, key0, key1);
                    acc = bop3<LUT_SEL>(was, less, acc);
                }
            }
            flip_word(&lat[addr], bop3<LUT_ANDN2>(acc, drew, und));
            return;
        }
        int wcnt = 0;
        for (int e0 = 0; e0 < cnt; e0 += 64) {
            const int e = e0 + lane;
            uint64_t und = 0, one = 0;
            uint32_t pk = 0;
            wcalls += (uint32_t)min(64, cnt - e0);
            if (e < cnt) {
                und_load(&eu[e], und, one);
                pk = en[e];
                const int addr = (int)(pk >> 16);
                const uint32_t g = (uint32_t)(group0 + div_small(addr, invN));
                const uint64_t was = und;
                const uint64_t less = draw_call((uint32_t)c, call_masks(Th.t4, Th.t8, (uint32_t)c), one, und,
                                                pk & 0xFFFFu, g, i, c3, key0, key1);
                flip_word(&lat[addr], bop3<LUT_ANDN2>(less, was, und));
            }
            const uint64_t need = wave_ballot(und != 0);
            if (und != 0) {
                const int slot = rank_below(need, wcnt);
                und_store(&eu[slot], und, one);
                en[slot] = pk;
            }
            wcnt += __popcll(need);
        }
        cnt = wcnt;
    }
}

// Sparse rounds over one list shared by the workgroup (ctl[h & 1] entries,
// appended by every wavefront in the dense rounds): each round takes the
// list in passes of one wavefront-load per wavefront; after a pass the
// wavefronts' survivor counts (ctl[2 + 16 par + w], alternating buffers)
// give every survivor its place in the compacted list, which always lies
// before the entries of later passes, so the list is compacted in place.
// When at most two wavefront-loads remain, two wavefronts (one if the
// workgroup has only one) run all their remaining calls without writing the
// list back.
__device__ __forceinline__ void sweep_sparse_pooled(uint64_t *lat, UndPair *eu, uint32_t *en,
                                                    int *ctl, int h, int c_first, float invN, int group0,
                                                    const Thresholds &Th, uint32_t i, uint32_t c3, uint32_t key0,
                                                    uint32_t key1, uint32_t &wcalls)
{
    const int lane = threadIdx.x & 63, wv = wave_id(), nw = blockDim.x >> 6;
    const int tailw = min(2, nw);   // wavefronts that finish the last entries
    __syncthreads();   // every wavefront's appends are in the list
    int cnt = ctl[h & 1];
    int par = 0;
    for (int c = c_first; c < 16 && cnt > 0; ++c) {
        if (cnt <= 64 * tailw) {
            if (wv < tailw) {
                const int e = wv * 64 + lane;
                uint64_t und = 0, one = 0, acc = 0;
                int addr = 0;
                uint32_t n = 0, g = 0;
                if (e < cnt) {
                    und_load(&eu[e], und, one);
                    const uint32_t pk = en[e];
                    addr = (int)(pk >> 16);
                    n = pk & 0xFFFFu;
                    g = (uint32_t)(group0 + div_small(addr, invN));
                }
                const uint64_t drew = und;
                for (; c < 16; ++c) {
                    const uint64_t live = wave_ballot(und != 0);
                    if (live == 0) break;
                    wcalls += (uint32_t)__popcll(live);
                    if (und != 0) {
                        const uint64_t was = und;
                        const uint64_t less = draw_call((uint32_t)c, call_masks(Th.t4, Th.t8, (uint32_t)c), one, und,
                                                        n, g, i, c3, key0, key1);
                        acc = bop3<LUT_SEL>(was, less, acc);
                    }
                }
                flip_word(&lat[addr], bop3<LUT_ANDN2>(acc, drew, und));
            }
            return;
        }
        int out = 0;
        for (int s0 = 0; s0 < cnt; s0 += 64 * nw) {
            const int e = s0 + wv * 64 + lane;
            uint64_t und = 0, one = 0;
            uint32_t pk = 0;
            wcalls += (uint32_t)max(0, min(64, cnt - (s0 + wv * 64)));
            if (e < cnt) {
                und_load(&eu[e], und, one);
                pk = en[e];
                const int addr = (int)(pk >> 16);
                const uint32_t g = (uint32_t)(group0 + div_small(addr, invN));
                const uint64_t was = und;
                const uint64_t less = draw_call((uint32_t)c, call_masks(Th.t4, Th.t8, (uint32_t)c), one, und,
                                                pk & 0xFFFFu, g, i, c3, key0, key1);
                flip_word(&lat[addr], bop3<LUT_ANDN2>(less, was, und));
            }
            const uint64_t need = wave_ballot(und != 0);
            int *cw = ctl + 2 + 16 * par;
            if (lane == 0) cw[wv] = __popcll(need);
            __syncthreads();
            int off = out, tot = 0;
            for (int w = 0; w < nw; ++w) {
                const int v = cw[w];
                off += w < wv ? v : 0;
                tot += v;
            }
            if (und != 0) {
                const int slot = rank_below(need, off);
                und_store(&eu[slot], und, one);
                en[slot] = pk;
            }
            out += tot;
            par ^= 1;
        }
        __syncthreads();   // the compacted list is complete
        cnt = out;
    }
}

// One item of the batched sweep, read into scalar registers before the first
// barrier: a barrier orders memory, so values left in global memory would be
// loaded again after every one of them.
struct SweepJob : LatticeShape {
    int G, group0, lastg, units;
    int s_begin, s_end;      // this item's sweeps
    int ub, ue;              // this wavefront's units (site words of one colour)
    uint32_t key0, key1, i, c3p;
    uint64_t vlast;          // valid replicas of the last group
    Thresholds Th;
    uint64_t *base;          // the groups' lattices in memory
};

template <int LT>
__device__ __forceinline__ bool sweep_job(const SweepItem &item, const RunInfo &R, const PopState &S, SweepJob &J)
{
    J.L = LT > 0 ? LT : __builtin_amdgcn_readfirstlane(R.L);
    J.N = J.L * J.L;
    J.half = J.L >> 1;
    J.nh = J.N >> 1;
    const int Rc = __builtin_amdgcn_readfirstlane(S.Rcur);
    const int pop = __builtin_amdgcn_readfirstlane(item.pop);
    J.group0 = __builtin_amdgcn_readfirstlane(item.group0);
    J.G = min(__builtin_amdgcn_readfirstlane(item.ngroups), (Rc + 63) / 64 - J.group0);
    if (J.G <= 0) return false;
    // a chunk of the sweeps (boundaries chosen by the plan,
    // expand_sweep_chunks), or all theta
    const int theta = __builtin_amdgcn_readfirstlane(R.theta);
    const int nchunk = max(1, __builtin_amdgcn_readfirstlane(item.nchunk));
    const int chunk = __builtin_amdgcn_readfirstlane(item.chunk);
    J.s_begin = 0;
    J.s_end = theta;
    if (nchunk == 2) {
        const int cut = min(max(__builtin_amdgcn_readfirstlane(item.cut), 0), theta);
        J.s_begin = chunk ? cut : 0;
        J.s_end = chunk ? theta : cut;
    } else if (nchunk > 2) {
        const int sq = theta / nchunk, sr = theta - sq * nchunk;
        J.s_begin = chunk * sq + min(chunk, sr);
        J.s_end = J.s_begin + sq + (chunk < sr ? 1 : 0);
    }
    J.key0 = __builtin_amdgcn_readfirstlane(R.key0);
    J.key1 = __builtin_amdgcn_readfirstlane(R.key1);
    const int i = __builtin_amdgcn_readfirstlane(S.i);
    J.i = (uint32_t)i;
    J.c3p = (TAG_SWEEP << 28) | ((uint32_t)pop << 24);
    J.Th = thresholds_of(R.tabT, i);
    J.lastg = J.group0 + J.G - 1;
    J.vlast = (Rc - J.lastg * 64 >= 64) ? ~0ull : ((1ull << (Rc - J.lastg * 64)) - 1);
    J.units = J.G * J.nh;
    const int upw = msc_units_per_wave(J.units, blockDim.x >> 6);
    J.ub = min(J.units, wave_id() * upw);
    J.ue = min(J.units, J.ub + upw);
    J.base = words_of(R, S, pop) + (size_t)J.group0 * J.N;
    return true;
}

// Lattice word of site n of group gs: colour (x + y) & 1, then the site's
// place n >> 1 among its colour (rows of L/2).
__device__ __forceinline__ int lattice_word(const SweepJob &J, int gs, int n, int y)
{
    return gs * J.N + ((n + y) & 1) * J.nh + (n >> 1);
}

// handed: the other end is another workgroup of this launch (put, take).
template <int LT, bool STORE>
__device__ __forceinline__ void move_lattices(const SweepJob &J, uint64_t *lat, bool handed)
{
    const float invN = 1.0f / (float)J.N, invL = 1.0f / (float)J.L;
    for (int u = threadIdx.x; u < J.G * J.N; u += blockDim.x) {
        const int gs = LT > 0 ? u / J.N : div_small(u, invN);
        const int n = u - gs * J.N;
        const int y = LT > 0 ? n / J.L : div_small(n, invL);
        uint64_t &l = lat[lattice_word(J, gs, n, y)];
        if (STORE && handed) put(&J.base[u], l);
        else if (STORE) J.base[u] = l;
        else l = handed ? take(&J.base[u]) : J.base[u];
    }
}

// Signs of the four bonds of site k of a colour, in the order of its
// neighbours in the other colour's array: k itself and k - 1 or k + 1 within
// the row (the horizontal pair), k - L/2 (up), k + L/2 (down).  Bit set: J = -1.
__device__ __forceinline__ void bond_signs(const SweepJob &J, const uint8_t *jbits, uint8_t *jb)
{
    const float invH = 1.0f / (float)J.half;
    for (int v = threadIdx.x; v < J.N; v += blockDim.x) {
        const int colour = v >= J.nh ? 1 : 0, k = v - colour * J.nh;
        const int y = div_small(k, invH), m = k - y * J.half;
        const int p = (y + colour) & 1, x = 2 * m + p;
        const int xl = x == 0 ? J.L - 1 : x - 1, yu = y == 0 ? J.L - 1 : y - 1;
        const uint8_t jn = jbits[y * J.L + x];
        const uint32_t jr = jn & 1u, jd = (jn >> 1) & 1u;
        const uint32_t jl = jbits[y * J.L + xl] & 1u, ju = (jbits[yu * J.L + x] >> 1) & 1u;
        // k is the right neighbour when p = 0 and the left one when p = 1
        const uint32_t jk = p ? jl : jr, jh = p ? jr : jl;
        jb[v] = (uint8_t)(jk | (jh << 1) | (ju << 2) | (jd << 3));
    }
}

// Classes of one unit: w its word, oth + k (+ offsets) the other colour's.
template <bool EA>
__device__ __forceinline__ SiteClass classify_unit(uint64_t w, const uint64_t *o, int dh, int du, int dd, uint32_t jm)
{
    uint64_t n0 = o[0], n1 = o[dh], n2 = o[du], n3 = o[dd];
    if (EA) {
        n0 ^= jmask((uint8_t)jm, 0);
        n1 ^= jmask((uint8_t)jm, 1);
        n2 ^= jmask((uint8_t)jm, 2);
        n3 ^= jmask((uint8_t)jm, 3);
    }
    return classify(w, n0, n1, n2, n3);
}

// Work counters of an item: word-site updates and attempted flips in closed
// form (the item's sweeps x 2 colours x its units, 64 replicas each except
// the valid ones of the last group), the calls as counted.
__device__ __forceinline__ void item_stats(const SweepJob &J, uint32_t wcalls, unsigned long long *stats)
{
    const int mine = max(J.ue - J.ub, 0);
    const int nlast = max(J.ue - max(J.ub, (J.G - 1) * J.nh), 0);   // its units in the last group
    const uint64_t nsw = (uint64_t)(J.s_end - J.s_begin);
    const uint64_t nwords = nsw * 2u * (uint64_t)mine;
    const uint64_t nflips =
        nsw * 2u * ((uint64_t)(mine - nlast) * 64u + (uint64_t)nlast * (uint64_t)__popcll(J.vlast));
    const bool first = (threadIdx.x & 63) == 0;
    flush_stats(stats, first ? nwords : 0ull, first ? wcalls : 0u, first ? nflips : 0ull);
}

// A wavefront's queue of undecided sites: a ring of `slots` entries (a power
// of two).  An entry's word is the counter word of its next call, site |
// call << 20, with the replica group's index within the workgroup between
// them (bits 12 .. 19, sites below 4096) unless the wavefront's sites are all
// of one group (ONE).  Every round takes the next 64 entries whatever call
// each is at, makes that call and appends the sites still undecided, so the
// rounds run on full wavefronts until at most 64 entries are left.
struct Stream {
    UndPair *eu;
    uint32_t *en;
    const PlaneMasks *tmask;   // T's bits at the planes of each call
    int slots;
    uint32_t i, c3, key0, key1;
    int hs = 0, ts = 0, left = 0;   // slot of the head, slot of the tail, entries
};

constexpr uint32_t ENTRY_CALL = 1u << 20;        // the call index's unit
constexpr uint32_t ENTRY_LAST = 15u << 20;       // last call
constexpr uint32_t ENTRY_SITE = 0xFFFu;          // site where entries carry a group

template <bool UNIFORM>
__device__ __forceinline__ uint64_t stream_call(const Stream &q, uint32_t c0, uint32_t g, const PlaneMasks &m,
                                                uint64_t one, uint64_t &und)
{
    const u32x4 o = philox10_sweep<UNIFORM>(c0, g, q.i, q.c3, q.key0, q.key1);
    return plane_pair((uint64_t)o.x | ((uint64_t)o.y << 32), (uint64_t)o.z | ((uint64_t)o.w << 32), m, one, und);
}

__device__ __forceinline__ void stream_push(Stream &q, uint64_t und, uint64_t one, uint32_t pk)
{
    const uint64_t need = wave_ballot(und != 0);
    if (und != 0) {
        const int out = (rank_below(need, 0) + q.ts) & (q.slots - 1);
        und_store(&q.eu[out], und, one);
        q.en[out] = pk;
    }
    const int nn = __popcll(need);
    q.ts = (q.ts + nn) & (q.slots - 1);
    q.left += nn;
}

// Full rounds while more than 64 entries wait.  word(pk): where an entry's
// flips go (LDS); group(pk): its replica group.
template <bool ONE, class Word, class Group>
__device__ __forceinline__ void stream_rounds(Stream &q, Word word, Group group, uint32_t &wcalls)
{
    const int lane = threadIdx.x & 63;
    while (q.left > 64) {
        const int slot = (q.hs + lane) & (q.slots - 1);
        uint64_t und, one;
        und_load(&q.eu[slot], und, one);
        const uint32_t pk = q.en[slot];
        const uint64_t was = und;
        const uint64_t less = stream_call<ONE>(q, ONE ? pk : pk & (ENTRY_LAST | ENTRY_SITE), group(pk),
                                               q.tmask[pk >> 20], one, und);
        flip_word(word(pk), bop3<LUT_ANDN2>(less, was, und));
        wcalls += 64;
        const bool more = und != 0 && pk < ENTRY_LAST;
        // the two compares' masks, combined on the scalar unit
        const uint64_t need = wave_ballot(und != 0) & wave_ballot(pk < ENTRY_LAST);
        if (more) {
            const int out = (rank_below(need, 0) + q.ts) & (q.slots - 1);
            und_store(&q.eu[out], und, one);
            q.en[out] = pk + ENTRY_CALL;
        }
        const int nn = __popcll(need);
        q.ts = (q.ts + nn) & (q.slots - 1);
        q.hs = (q.hs + 64) & (q.slots - 1);
        q.left += nn - 64;
    }
}

// The last (at most 64) entries: each lane runs all the remaining calls of
// its own entry.
template <bool ONE, class Word, class Group>
__device__ __forceinline__ void stream_tail(const Stream &q, uint64_t *any, Word word, Group group, uint32_t &wcalls)
{
    const int lane = threadIdx.x & 63;
    uint64_t und = 0, one = 0, acc = 0;
    uint32_t pk = ~0u;
    uint64_t *w = any;   // lanes without an entry flip nothing there
    if (lane < q.left) {
        const int slot = (q.hs + lane) & (q.slots - 1);
        und_load(&q.eu[slot], und, one);
        pk = q.en[slot];
        w = word(pk);
    }
    const uint64_t drew = und;
    const uint32_t g = group(pk);
    for (;;) {
        const bool live = und != 0 && pk < ENTRY_LAST + ENTRY_CALL;
        const uint64_t lv = wave_ballot(und != 0) & wave_ballot(pk < ENTRY_LAST + ENTRY_CALL);
        if (lv == 0) break;
        wcalls += (uint32_t)__popcll(lv);
        if (live) {
            const uint64_t was = und;
            const uint64_t less =
                stream_call<ONE>(q, ONE ? pk : pk & (ENTRY_LAST | ENTRY_SITE), g, q.tmask[pk >> 20], one, und);
            acc = bop3<LUT_SEL>(was, less, acc);
            pk += ENTRY_CALL;
        }
    }
    flip_word(w, bop3<LUT_ANDN2>(acc, drew, und));
}

// Masks of the first calls; one of each pair in a vector register (an
// instruction reads one scalar operand), where the compiler would otherwise
// copy it again for every call.
struct LockstepMasks {
    PlaneMasks m[4];
    __device__ __forceinline__ LockstepMasks(const Thresholds &Th)
    {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            m[c] = call_masks(Th.t4, Th.t8, (uint32_t)c);
            asm volatile("" : "+v"(m[c].a8), "+v"(m[c].b8));
        }
    }
};

// Calls 0 .. dense-1 of one site per lane, without branches or lane masks (a
// decided lane's call changes nothing): und keeps the undecided, the
// verdicts of the others go to acc.
template <bool UNIFORM>
__device__ __forceinline__ void lockstep_calls(const Stream &q, int dense, const LockstepMasks &dm,
                                               const Thresholds &Th, uint32_t n, uint32_t g, uint64_t one,
                                               uint64_t &und, uint64_t &acc, uint32_t &wcalls)
{
    auto call = [&](uint32_t c, const PlaneMasks &m) {
        wcalls += (uint32_t)__popcll(wave_ballot(und != 0));
        const uint64_t was = und;
        const uint64_t less = stream_call<UNIFORM>(q, n | (c << 20), g, m, one, und);
        acc = bop3<LUT_SEL>(was, less, acc);
    };
    if (dense > 0) call(0, dm.m[0]);
    if (dense > 1) call(1, dm.m[1]);
    if (dense > 2) call(2, dm.m[2]);
    if (dense > 3) call(3, dm.m[3]);
    for (int c = 4; c < dense; ++c) call((uint32_t)c, call_masks(Th.t4, Th.t8, (uint32_t)c));
}

// The sweeps of a streamed item.  A site's place among its colour is
// site >> 1, so an entry's lattice word follows from its counter word.
//
// Bound by the vector ALU's issue rate (at L = 64 it issues in 97 % of the
// slots while the CU has work), so everything here is counted in
// instructions: the lockstep calls run without branches or lane masks on
// masks held in registers, a chunk of whole rows finds its neighbours at
// constant offsets, the entry word needs no unpacking.  Against a form with a
// branch and an exec mask per call, divisions per chunk for the sizes without
// a kernel of their own, and one kernel body per size in the dispatching
// kernel (100 registers instead of 61, so two workgroups per CU instead of
// three), per launch: L = 64, R = 1e5 576 -> 531 us (2.76e8 instead of 3.08e8
// vector instructions); two populations of 2e5 at L = 32 657 -> 570; 1024
// runs of four sizes 1520 -> 1297; ten spin-glass runs of five sizes 1765 ->
// 1604; R = 1e5 at L = 20 184 -> 144; 3840 runs at L = 10 322 -> 166.
template <int LT, bool EA, bool ONE>
__device__ __forceinline__ uint32_t stream_sweeps(const SweepJob &J, uint64_t *lat, UndPair *eu, uint32_t *en,
                                                  const uint8_t *jb, const PlaneMasks *tmask, int slots, int dense)
{
    const int L = LT > 0 ? LT : J.L, N = L * L, half = L >> 1, nh = N >> 1;
    const int lane = threadIdx.x & 63;
    const bool saturated = J.Th.all4 || J.Th.all8;
    const bool partial = J.vlast != ~0ull;
    const LockstepMasks dm(J.Th);
    // steps of a walk over 64 units
    const int gq = 64 / nh, kr = 64 - gq * nh, yr = kr / half, mr = kr - yr * half;
    UnitWalk first;
    first.start(J, min(J.ub, J.units - 1) + lane);
    uint32_t wcalls = 0;   // Philox calls of this wavefront (uniform)
    for (int s = J.s_begin; s < J.s_end; ++s) {
        for (int colour = 0; colour < 2; ++colour) {
            __syncthreads();
            const int cb = colour * nh;            // this colour's words
            const int od = colour ? -nh : nh;      // from a word to the same place of the other colour
            Stream q = {eu, en, tmask, slots, J.i, J.c3p | (uint32_t)s, J.key0, J.key1};
            auto word = [&](uint32_t pk) {
                if constexpr (ONE) return lat + cb + (int)((pk & 0xFFFFFu) >> 1);
                else return lat + cb + (int)((pk >> 1) & 0x7FFu) + (int)((pk >> 12) & 0xFFu) * N;
            };
            auto group = [&](uint32_t pk) {
                return (uint32_t)(ONE ? J.group0 : J.group0 + (int)((pk >> 12) & 0xFFu));
            };
            using UG = std::integral_constant<bool, ONE>;
            // one chunk: a unit (site word) per lane.  own: its lattice word;
            // dh, du, dd: offsets of the neighbours beside the word at the
            // same place of the other colour; ug: gs is the same on every lane
            auto chunk = [&](bool in, int own, int dh, int du, int dd, uint32_t n, int gs, auto ug) {
                uint64_t und = 0, one = 0, acc = 0;
                const uint32_t g = (uint32_t)(J.group0 + gs);
                if (in) {
                    uint32_t jm = 0;
                    if (EA) jm = jb[cb + (int)(n >> 1)];
                    SiteClass sc = classify_unit<EA>(lat[own], lat + own + od, dh, du, dd, jm);
                    if (saturated) accept_saturated(sc, J.Th);   // uniform, only where a threshold is 2^32
                    und = sc.und;
                    one = sc.one;
                    acc = ~0ull;   // flips unless a draw says otherwise
                    if (partial && (int)g == J.lastg) {   // only valid replicas draw and flip
                        und &= J.vlast;
                        acc = J.vlast;
                    }
                }
                lockstep_calls<decltype(ug)::value>(q, dense, dm, J.Th, n, g, one, und, acc, wcalls);
                at_unit(in, own, [&](int w) { flip_word(&lat[w], acc & ~und); });
                stream_push(q, und, one, n | ((uint32_t)dense << 20) | (ONE ? 0u : (uint32_t)gs << 12));
                stream_rounds<ONE>(q, word, group, wcalls);   // room for the next chunk's entries
            };
            // A chunk of whole rows (64 a multiple of two row halves, the
            // colour's half-lattice a multiple of 64): every lane keeps its
            // column, parity and horizontal neighbour for the whole walk,
            // all lanes are in one replica group, and only the chunks at the
            // lattice's top and bottom have wrapped neighbours.
            constexpr bool ROWS = LT > 0 && 64 % LT == 0 && (LT * LT / 2) % 64 == 0;
            if constexpr (ROWS) {
                int gs = __builtin_amdgcn_readfirstlane(first.gs);
                int kb = J.ub - gs * nh;   // lane 0's place among the colour: uniform
                const int p = (first.y + colour) & 1;
                const int dh = first.dh(J, p);
                uint32_t n = 2u * (uint32_t)first.k + (uint32_t)p;
                int own = first.a + cb;
                for (int u0 = J.ub; u0 < J.ue; u0 += 64) {
                    int du = -half, dd = half;
                    if (kb == 0) du += lane < half ? nh : 0;
                    if (kb == nh - 64) dd -= lane >= 64 - half ? nh : 0;
                    chunk(true, own, dh, du, dd, n, ONE ? 0 : gs, std::true_type{});
                    kb += 64;
                    own += 64;
                    n += 128;
                    if (kb == nh) {   // every lane at once: the next replica group
                        kb = 0;
                        own += N - nh;
                        n -= (uint32_t)N;
                        ++gs;
                    }
                }
            } else {
                UnitWalk w = first;
                for (int u0 = J.ub; u0 < J.ue; u0 += 64) {
                    const int p = (w.y + colour) & 1;
                    const bool in = u0 + lane < J.ue;
                    chunk(in, w.word(J, colour), w.dh(J, p), w.du(J), w.dd(J),
                          2u * (uint32_t)w.k + (uint32_t)p, ONE ? 0 : w.gs, UG{});
                    w.step(J, gq, kr, yr, mr);
                }
            }
            stream_tail<ONE>(q, lat, word, group, wcalls);
        }
    }
    return wcalls;
}

// LDS layout: msc_stream_lds.
template <int LT, bool EA>
__device__ __forceinline__ void stream_item(const SweepItem &item, const RunInfo &R, const PopState &S, uint64_t *lds,
                                            int mode, unsigned long long *stats)
{
    SweepJob J;
    if (!sweep_job<LT>(item, R, S, J)) return;
    const int nw = blockDim.x >> 6, slots = msc_ring_slots(J.units, nw);
    PlaneMasks *tmask = (PlaneMasks *)lds;
    uint64_t *lat = lds + 32;
    UndPair *eu = (UndPair *)(lat + (size_t)J.G * J.N);
    uint32_t *en = (uint32_t *)(eu + nw * slots);
    uint8_t *jb = (uint8_t *)(en + nw * slots);
    move_lattices<LT, false>(J, lat, item.chunk > 0);
    if (EA) bond_signs(J, R.jbits, jb);
    if (threadIdx.x < 16) tmask[threadIdx.x] = call_masks(J.Th.t4, J.Th.t8, threadIdx.x);   // read after a barrier
    const int ring = wave_id() * slots;
    const uint32_t wcalls =
        J.G == 1 ? stream_sweeps<LT, EA, true>(J, lat, eu + ring, en + ring, jb, tmask, slots, mode & 0xFF)
                 : stream_sweeps<LT, EA, false>(J, lat, eu + ring, en + ring, jb, tmask, slots, mode & 0xFF);
    __syncthreads();
    move_lattices<LT, true>(J, lat, item.chunk + 1 < item.nchunk);
    item_stats(J, wcalls, stats);
}

// Items whose lists are not streamed.  LDS layout: msc_list_lds.
template <bool EA>
__device__ __forceinline__ void general_item(const SweepItem &item, const RunInfo &R, const PopState &S, uint64_t *lds,
                                             int mode, unsigned long long *stats)
{
    SweepJob J;
    if (!sweep_job<0>(item, R, S, J)) return;
    const int N = J.N, nh = J.nh;
    const int lane = threadIdx.x & 63;
    const bool pool = (mode >> 8) & 1;
    const int dense = mode & 0xFF;
    uint64_t *lat = lds;                                  // [G][2][nh]
    UndPair *eu = (UndPair *)(lds + (size_t)J.G * N);     // [units] undecided replicas and classes
    uint32_t *en = (uint32_t *)(eu + J.units);            // [units] (LDS word << 16) | site
    uint8_t *jb = (uint8_t *)(en + J.units);              // [2][nh] bond signs of each site (spin glass)
    int *ctl = (int *)(jb + (EA ? N : 0));                // pooled list counts [2], pass counts [2][16]
    move_lattices<0, false>(J, lat, item.chunk > 0);
    if (EA) bond_signs(J, R.jbits, jb);
    if (threadIdx.x == 0) ctl[0] = ctl[1] = 0;
    const float invN = 1.0f / (float)N;
    const int gq = 64 / nh, kr = 64 - gq * nh, yr = kr / J.half, mr = kr - yr * J.half;
    UnitWalk first;
    first.start(J, min(J.ub, J.units - 1) + lane);
    uint32_t wcalls = 0;   // Philox calls of this wavefront (uniform)
    for (int s = J.s_begin; s < J.s_end; ++s) {
        const uint32_t c3 = J.c3p | (uint32_t)s;
        for (int colour = 0; colour < 2; ++colour) {
            const int h = 2 * s + colour;   // half-sweep index: its list count is ctl[h & 1]
            __syncthreads();
            if (threadIdx.x == 0) ctl[(h + 1) & 1] = 0;   // the next half-sweep's count; last read before this barrier
            const int cb = colour * nh, od = colour ? -nh : nh;
            int cnt = 0;
            UnitWalk w = first;
            for (int u0 = J.ub; u0 < J.ue; u0 += 64) {
                const bool in = u0 + lane < J.ue;
                const int p = (w.y + colour) & 1, own = w.word(J, colour);
                const uint32_t n = 2u * (uint32_t)w.k + (uint32_t)p, g = (uint32_t)(J.group0 + w.gs);
                uint64_t und = 0, one = 0, acc = 0;
                if (in) {
                    uint32_t jm = 0;
                    if (EA) jm = jb[cb + w.k];
                    SiteClass sc = classify_unit<EA>(lat[own], lat + own + od, w.dh(J, p), w.du(J), w.dd(J), jm);
                    accept_saturated(sc, J.Th);
                    und = sc.und;
                    one = sc.one;
                    acc = ~0ull;   // flips unless a draw says otherwise
                    if ((int)g == J.lastg) {   // only valid replicas draw and flip
                        und &= J.vlast;
                        acc = J.vlast;
                    }
                }
                for (int c = 0; c < dense; ++c) {
                    const uint64_t live = wave_ballot(und != 0);
                    if (live == 0) break;
                    wcalls += (uint32_t)__popcll(live);
                    if (und != 0) {
                        const uint64_t was = und;
                        const uint64_t less = draw_call((uint32_t)c, call_masks(J.Th.t4, J.Th.t8, (uint32_t)c), one,
                                                        und, n, g, J.i, c3, J.key0, J.key1);
                        acc = bop3<LUT_SEL>(was, less, acc);
                    }
                }
                at_unit(in, own, [&](int w) { flip_word(&lat[w], acc & ~und); });
                const uint64_t need = wave_ballot(und != 0);
                int base_slot = J.ub + cnt;
                if (pool && need) {
                    int b0 = 0;
                    if (lane == 0) b0 = atomicAdd(&ctl[h & 1], __popcll(need));
                    base_slot = __builtin_amdgcn_readlane(b0, 0);
                }
                if (und != 0) {
                    const int slot = rank_below(need, base_slot);
                    und_store(&eu[slot], und, one);
                    en[slot] = ((uint32_t)own << 16) | n;
                }
                cnt += __popcll(need);
                w.step(J, gq, kr, yr, mr);
            }
            if (pool)
                sweep_sparse_pooled(lat, eu, en, ctl, h, dense, invN, J.group0, J.Th, J.i, c3, J.key0, J.key1,
                                    wcalls);
            else
                sweep_sparse_wave(lat, eu + J.ub, en + J.ub, cnt, dense, invN, J.group0, J.Th, J.i, c3, J.key0,
                                  J.key1, wcalls);
        }
    }
    __syncthreads();
    move_lattices<0, true>(J, lat, item.chunk + 1 < item.nchunk);
    item_stats(J, wcalls, stats);
}

// LS >= 0: every item of the launch has the model EA and, for LS > 0, L = LS,
// and its lists are streamed (a kernel of its own allocates only the
// registers that one form needs).  LS < 0: any size, model and list scheme,
// chosen per item.
template <int LS, bool EA>
__device__ __forceinline__ void sweep_one(const SweepItem &it, const RunInfo *runs, const PopState *st,
                                          uint64_t *lds, uint32_t lds_bytes, int mode, unsigned long long *stats)
{
    const RunInfo &R = runs[it.run];
    const PopState &S = st[it.run * MAX_POP + it.pop];
    if (!pop_active(S) || R.theta == 0) return;
    // an item that does not fit the LDS of this launch (a list that does not
    // belong to the launch's plan) is skipped and counted, never run
    const bool ea = R.model == PA_EA_PMJ;
    if (msc_lds_need(R.N, it.ngroups, ea, (int)(blockDim.x >> 6), mode) > lds_bytes) {
        if (threadIdx.x == 0) atomicAdd(&stats[ST_STALL], 1ull);
        return;
    }
    if constexpr (LS >= 0) {
        stream_item<LS, EA>(it, R, S, lds, mode, stats);
    } else if (msc_streamed(R.N, it.ngroups, mode)) {
        if (ea) stream_item<0, true>(it, R, S, lds, mode, stats);
        else stream_item<0, false>(it, R, S, lds, mode, stats);
    } else {
        if (ea) general_item<true>(it, R, S, lds, mode, stats);
        else general_item<false>(it, R, S, lds, mode, stats);
    }
}

// One workgroup per item, or (queue != nullptr) a persistent grid whose
// workgroups take items from the front of a list until none is left: of the
// whole list (n_lists = 0), or of the list of their CU (SweepList), and of
// the others' when it is empty.  queue[0] is the next item of the whole list,
// queue[1] counts workgroups that found nothing left; the last of them resets
// the lists, so the next launch (or graph replay) starts without a separate
// clear.
//
// Lists per CU: the workgroups on a CU do not advance alike (the oldest goes
// first: 109 / 220 / 395 us for equal items of three of them), so the last
// items of one list for all leave some CUs with two items to go when others
// are done, and every workgroup's first item is an atomic on one address,
// about 10 ns each.  Workgroups whose numbers differ by a multiple of the CU
// count share a CU (when nothing else runs; if not, only time is lost).
// Step at L = 64, R = 1e5 (1563 items, three workgroups per CU; the launch
// ends 11 % after the mean CU with whole items from one list, 2 % with these):
// one list 635 us, in two chunks each 622, lists 591; two populations at
// L = 32 716, 735, 699.  (Sizes mixed, where the cost of an item is known less
// well: no better than one list, 1769 against 1684 for five sizes.)
//
// Sweep chunks (persistent grid only): an item may cover a part of its
// groups' theta sweeps.  When a chunk has stored its lattices (put), its
// workgroup publishes (launch generation << 4 | chunk + 1) in the groups'
// flag slot; the next chunk waits for that value before it loads them.
// queue[2] is the launch generation: every workgroup reads it before taking
// an item, and the last one to leave increments it, so values left by earlier
// launches or graph replays never match.  The wait ends because a workgroup
// that runs holds the previous chunk: it stands earlier in the whole list,
// or it is the first item of the CU list after this one, and a workgroup that
// finds it still there takes it first.  The wait is bounded all the same, and
// one that runs out is counted in the stall counter (the results of that step
// are then not trustworthy, and reading the work counters reports it).
constexpr unsigned int SWEEP_WAIT_SPINS = 1u << 22;
constexpr unsigned int NO_ITEM = ~0u;

// The next item, of list l if it has one, else of another list (l becomes
// it); NO_ITEM if all are empty.  Called by the whole workgroup.
__device__ unsigned int next_item(SweepList *lists, int n_lists, int &l, unsigned int *sh)
{
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) {
            const unsigned int t = atomicAdd(&lists[l].next, 1u);
            *sh = t < lists[l].end ? t : NO_ITEM;
        }
        __syncthreads();
        const unsigned int t = *sh;
        if (t != NO_ITEM) return t;
        __syncthreads();
        if (threadIdx.x < 64) {
            unsigned int found = NO_ITEM;
            for (int base = 1; base < n_lists && found == NO_ITEM; base += 64) {
                const int q = base + (int)threadIdx.x, j = l + q < n_lists ? l + q : l + q - n_lists;
                const bool has = q < n_lists && take(&lists[j].next) < lists[j].end;
                const uint64_t bal = __ballot(has);
                if (bal) found = (unsigned int)(l + base + __ffsll((unsigned long long)bal) - 1) % (unsigned int)n_lists;
            }
            if (threadIdx.x == 0) *sh = found;
        }
        __syncthreads();
        if (*sh == NO_ITEM) return NO_ITEM;
        l = (int)*sh;
    }
}

template <int LS, bool EA>
__global__ void __launch_bounds__(1024) k_sweep_msc(const SweepItem *items, int n_items, const RunInfo *runs,
                                                    const PopState *st, int mode, unsigned long long *stats,
                                                    unsigned int *queue, unsigned int *flags, SweepList *lists,
                                                    int n_lists, uint32_t lds_bytes)
{
    extern __shared__ __align__(16) uint64_t lds[];
    __shared__ unsigned int sh, gen;
    const bool persistent = queue != nullptr;
    unsigned int t = blockIdx.x, later = NO_ITEM;
    int l = n_lists ? (int)(blockIdx.x % (unsigned int)n_lists) : 0;
    if (persistent && threadIdx.x == 0) gen = take(&queue[2]);
    for (;;) {
        if (later != NO_ITEM) {
            t = later;
            later = NO_ITEM;
        } else if (persistent && n_lists) {
            t = next_item(lists, n_lists, l, &sh);
        } else if (persistent) {
            __syncthreads();
            if (threadIdx.x == 0) sh = atomicAdd(&queue[0], 1u);
            __syncthreads();
            t = sh;
        }
        if (t >= (unsigned int)n_items) break;
        SweepItem it = items[t];
        if (persistent && it.chunk > 0) {
            __syncthreads();
            if (threadIdx.x == 0) {
                // the item's beginning, if nobody has it
                sh = NO_ITEM;
                if (n_lists) {
                    const unsigned int first = lists[l + 1].first;
                    if (atomicCAS(&lists[l + 1].next, first, first + 1) == first) sh = first;
                }
                const unsigned int want = (gen << 4) | (unsigned int)it.chunk;
                unsigned int spins = 0;
                while (sh == NO_ITEM && take(&flags[it.base]) != want) {
                    if (++spins == SWEEP_WAIT_SPINS) {
                        atomicAdd(&stats[ST_STALL], 1ull);
                        break;
                    }
                    __builtin_amdgcn_s_sleep(2);
                }
            }
            __syncthreads();
            if (sh != NO_ITEM) {
                later = t;
                it = items[sh];
            }
        }
        sweep_one<LS, EA>(it, runs, st, lds, lds_bytes, mode, stats);
        if (!persistent) return;
        if (it.chunk + 1 < it.nchunk) {
            // every wavefront waits for its own device-coherent lattice
            // stores (a barrier alone does not)
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            if (threadIdx.x == 0) put(&flags[it.base], (gen << 4) | (unsigned int)(it.chunk + 1));
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) sh = atomicAdd(&queue[1], 1u);
    __syncthreads();
    if (sh != gridDim.x - 1) return;
    for (int j = threadIdx.x; j < n_lists; j += blockDim.x) put(&lists[j].next, lists[j].first);
    if (threadIdx.x == 0) {
        put(&queue[0], 0u);
        put(&queue[1], 0u);
        put(&queue[2], gen + 1);
    }
}

// Lattices swept from memory, one colour per launch: sizes beyond a
// workgroup's LDS, and few groups of large ones, which a workgroup per group
// would sweep on few compute units.  A wavefront takes cpw chunks of 64 site
// words of one replica group through the same lockstep calls and queue as the
// batched sweep, collecting the flips in LDS, and applies them at the end;
// the neighbours are the other colour's words, which this launch only reads.
// In place of one byte per spin read and written per colour (and the halo
// rows of the tiles that took): 8 bytes per 64 spins, so the working set is
// an eighth and mostly in L2; bound by launches where the run is small, by
// the calls' instructions where it is not.  Step (iv) of ten sweeps with the
// conversions: L = 128, R = 2000 (spin glass) 388 -> 209 us; L = 256, R = 5000
// 3400 -> 874; L = 512, R = 200 732 -> 335.
constexpr int WIDE_WAVES = 4;
constexpr int WIDE_CHUNKS = 4;   // most chunks per wavefront

template <bool EA>
__global__ void __launch_bounds__(64 * WIDE_WAVES) k_sweep_wide(const RunInfo *runs, const PopState *st, int run,
                                                                int s, int colour, int cpw, int tiles,
                                                                unsigned long long *stats)
{
    __shared__ PlaneMasks tmask[16];
    __shared__ UndPair eu[WIDE_WAVES][128];
    __shared__ uint32_t en[WIDE_WAVES][128];
    __shared__ uint64_t fm[WIDE_WAVES][64 * WIDE_CHUNKS];
    const RunInfo &R = runs[run];
    const int pop = blockIdx.y;
    const PopState &S = st[run * MAX_POP + pop];
    const int g = blockIdx.x / tiles, tile = blockIdx.x - g * tiles;
    const int Rc = S.Rcur;
    if (!pop_active(S) || g * 64 >= Rc) return;
    const int L = R.L, N = R.N, half = L >> 1, nh = N >> 1;
    const int lane = threadIdx.x & 63, wv = wave_id();
    const Thresholds Th = thresholds_of(R.tabT, S.i);
    if (threadIdx.x < 16) tmask[threadIdx.x] = call_masks(Th.t4, Th.t8, threadIdx.x);
    __syncthreads();
    const int k0 = (tile * WIDE_WAVES + wv) * 64 * cpw, k1 = min(nh, k0 + 64 * cpw);
    if (k0 >= nh) return;
    uint64_t *words = words_of(R, S, pop) + (size_t)g * N;
    const uint8_t *jbits = R.jbits;
    const uint64_t valid = (Rc - g * 64 >= 64) ? ~0ull : ((1ull << (Rc - g * 64)) - 1);
    const float invH = 1.0f / (float)half;
    const LockstepMasks dm(Th);
    uint32_t wcalls = 0;
    Stream q = {eu[wv], en[wv], tmask, 128, (uint32_t)S.i, (TAG_SWEEP << 28) | ((uint32_t)pop << 24) | (uint32_t)s,
                R.key0, R.key1};
    auto word = [&](uint32_t pk) { return &fm[wv][(int)((pk & 0xFFFFFu) >> 1) - k0]; };
    auto group = [&](uint32_t) { return (uint32_t)g; };
    auto site = [&](int k, int &y, int &x) {
        y = div_small(k, invH);
        x = 2 * (k - y * half) + ((y + colour) & 1);
        return y * L + x;
    };
    for (int kb = k0; kb < k1; kb += 64) {
        const int k = kb + lane;
        uint64_t und = 0, one = 0, acc = 0;
        int n = 0;
        if (k < k1) {
            int y, x;
            n = site(k, y, x);
            const int nr = x + 1 == L ? n + 1 - L : n + 1, nl = x == 0 ? n + L - 1 : n - 1;
            const int nd = y + 1 == L ? n + L - N : n + L, nu = y == 0 ? n + N - L : n - L;
            uint64_t wr = words[nr], wl = words[nl], wd = words[nd], wu = words[nu];
            if (EA) {
                const uint8_t jn = jbits[n];
                wr ^= jmask(jn, 0);
                wl ^= jmask(jbits[nl], 0);
                wd ^= jmask(jn, 1);
                wu ^= jmask(jbits[nu], 1);
            }
            SiteClass sc = classify(words[n], wr, wl, wd, wu);
            accept_saturated(sc, Th);
            und = sc.und & valid;
            one = sc.one;
            acc = valid;   // flips unless a draw says otherwise
        }
        lockstep_calls<true>(q, 3, dm, Th, (uint32_t)n, (uint32_t)g, one, und, acc, wcalls);
        fm[wv][kb - k0 + lane] = acc & ~und;
        stream_push(q, und, one, (uint32_t)n | 3u * ENTRY_CALL);
        stream_rounds<true>(q, word, group, wcalls);
    }
    stream_tail<true>(q, &fm[wv][0], word, group, wcalls);
    for (int kb = k0; kb < k1; kb += 64)
        if (kb + lane < k1) {
            int y, x;
            const int n = site(kb + lane, y, x);
            words[n] ^= fm[wv][kb - k0 + lane];
        }
    const bool first = lane == 0;
    flush_stats(stats, first ? (uint64_t)(k1 - k0) : 0ull, first ? wcalls : 0u,
                first ? (uint64_t)(k1 - k0) * (uint64_t)__popcll(valid) : 0ull);
}

// -------------------------------------------------------------- step (v)

// Partner words of the permutation pairing ([group][site] u64): the spare
// spin buffer of population 0 (its previous population is no longer needed
// once the step's copies are done; it holds at least 8 bytes per site and
// group in either layout).
__device__ __forceinline__ uint8_t *wang_partner_words(const RunInfo &R, const PopState &S)
{
    return R.spins[0][S.cur ^ 1];
}

// Word of 64 replicas of group g at site n, from either layout.
template <int REPR>
__device__ __forceinline__ uint64_t load_word(const uint8_t *buf, int g, int n, int N)
{
    if (REPR == PA_MSC64) return ((const uint64_t *)buf)[(size_t)g * N + n];
    const uint4 *q = (const uint4 *)(buf + ((size_t)g * N + n) * 64);
    uint4 v[4] = {q[0], q[1], q[2], q[3]};
    return pack64(v);
}

// Spins that a measurement of layout REPR reads: bytes, or words (in the
// int8 layout the words that the sweeps left).
template <int REPR>
__device__ __forceinline__ const uint8_t *spin_buf(const RunInfo &R, const PopState &S, int pop)
{
    return REPR == PA_INT8 ? R.spins[pop][S.cur] : (const uint8_t *)words_of(R, S, pop);
}

// Measurement of replica groups (64 replicas each).  A workgroup of
// W (MEAS_WAVES or four times as many) wavefronts takes a measure item of
// consecutive groups of one (run, pop); each group gets
// meas_waves_per_group(N) wavefronts (or four times that), which split its
// sites 64 at a time.  A lane accumulates, in bit-sliced
// counters over its sites, the per-replica numbers of unsatisfied bonds
// (E = 2 #unsat - 2N), down spins (M = N - 2 #down), and for overlap pairs
// the Hamming distance (Q = N - 2 d) and the number of bonds whose product
// differs (Q_l = 2N - 2 d_l); neighbour words are read straight from
// memory (the lattice block of a group is contiguous, so they hit the
// caches).  The counters are turned into per-replica integers by
// transposes, the wavefronts of a group are summed in LDS, the energies are
// stored, and the group's integer sums go to its slot of the partial-sum
// array; k_meas_chunk reduces those per chunk.
template <int REPR, int LT, bool WITH_Q, int W>
__device__ __forceinline__ void measure_group(const SweepItem &it, int g, int sub, int wpg, bool live,
                                              const RunInfo &R, const PopState &S, const PopState *st,
                                              uint32_t (*red)[W][64], const uint64_t *lw)
{
    const uint8_t *buf = spin_buf<REPR>(R, S, it.pop);
    // the group's own words come from LDS when the workgroup staged them
    // (lw != nullptr), else from memory
    auto own = [&](int gg, int n, int NN) -> uint64_t { return lw ? lw[n] : load_word<REPR>(buf, gg, n, NN); };
    const int L = LT ? LT : R.L;
    const int N = L * L;
    const int Rc = S.Rcur;
    const int lane = threadIdx.x & 63, wv = wave_id();
    // overlap partners of this group's replicas
    int mode = 0;                      // 0 none, 1 index shift, 2 two populations, 3 permutation pairs
    uint64_t pairmask = 0;
    const uint8_t *pbuf = buf;
    int pg = 0, sh = 0;
    const int pgroups = R.groups_cap;
    if (!WITH_Q) {
        // no run of the launch measures overlaps
    } else if (live && R.overlap == PA_Q_INDEX_SHIFT) {
        const int h = Rc >> 1;
        const int lo = g * 64;
        if (lo < h) {
            mode = 1;
            const int cntp = min(64, h - lo);
            pairmask = cntp >= 64 ? ~0ull : ((1ull << cntp) - 1);
            pg = (lo + h) >> 6;
            sh = (lo + h) & 63;
        }
    } else if (live && R.overlap == PA_Q_TWO_POP && it.pop == 0) {
        const PopState &S1 = st[it.run * MAX_POP + 1];
        if (pop_active(S1)) {
            const int m = min(Rc, S1.Rcur);
            const int lo = g * 64;
            if (lo < m) {
                mode = 2;
                const int cntp = min(64, m - lo);
                pairmask = cntp >= 64 ? ~0ull : ((1ull << cntp) - 1);
                pbuf = spin_buf<REPR>(R, S1, 1);
                pg = g;
            }
        }
    } else if (live && is_wang(R.overlap) && wang_bufs(R.wang, R.R_cap, R.wang_lb).hdr[0] == 0) {
        // permutation pairs (j, pi_j) for every replica: the partners'
        // configurations were gathered into bit-packed words (k_wang_gather)
        mode = 3;
        const int cntp = min(64, Rc - g * 64);
        pairmask = cntp >= 64 ? ~0ull : ((1ull << cntp) - 1);
        pbuf = wang_partner_words(R, S);
        pg = g;
    }
    if (R.exact_dos && S.i > 0) {
        // theta = infinity: the energies were drawn (k_dos_sample); only
        // their sums and minimum are recorded.  One barrier, as below.
        __syncthreads();
        if (!live || sub != 0) return;
        const int j = g * 64 + lane;
        const bool valid = j < Rc;
        const int64_t E = valid ? R.E[it.pop][S.cur][j] : 0;
        int64_t part[MEAS_PART];
        part[0] = wave_sum<int64_t>(E);
        part[1] = wave_sum<int64_t>(E * E);
        for (int k = 2; k < MEAS_PART - 1; ++k) part[k] = 0;
        part[MEAS_PART - 1] = wave_min(valid ? (int)E : INT32_MAX);
        if (lane < MEAS_PART) {
            int64_t mine = 0;
#pragma unroll
            for (int k = 0; k < MEAS_PART; ++k)
                if (lane == k) mine = part[k];
            R.part[it.pop][(size_t)g * MEAS_PART + lane] = mine;
        }
        return;
    }
    uint32_t totU = 0, totD = 0, totH = 0, totK = 0;
    // every lane of the wavefront runs the same iterations (flushes are
    // wave-wide).  Counts are flushed after every block of 16 sites per lane
    // (at most 2 per site: 32 < 2^VB); mode is uniform over the wavefront, so
    // are the overlap counts.
    if constexpr (WITH_Q) {
        // four counters: the incremental form keeps the loop within the
        // registers of four wavefronts per SIMD
        uint64_t cU[VB] = {}, cD[VB] = {}, cH[VB] = {}, cK[VB] = {};
        for (int b0 = 64 * sub; b0 < N; b0 += 16 * 64 * wpg) {
            // sites per lane in this block of 16 (uniform): bounds the counts
            const int tsites = min(16, (N - b0 + 64 * wpg - 1) / (64 * wpg));
#pragma unroll 4
            for (int t = 0; t < 16; ++t) {
                const int n = b0 + t * 64 * wpg + lane;
                if (live && n < N) {
                    const int y = n / L, x = n - y * L;
                    const int nr = y * L + (x + 1 == L ? 0 : x + 1);
                    const int nd = (y + 1 == L ? 0 : y + 1) * L + x;
                    const uint8_t jn = R.jbits[n];
                    const uint64_t w = own(g, n, N);
                    const uint64_t wr = own(g, nr, N);
                    const uint64_t wd = own(g, nd, N);
                    const uint64_t br = w ^ wr, bd = w ^ wd;
                    vinc2(cU, br ^ ((jn & 1) ? ~0ull : 0ull), bd ^ ((jn & 2) ? ~0ull : 0ull));
                    vinc(cD, w);
                    if (mode) {
                        uint64_t q, qr, qd;
                        if (mode == 3) {
                            const uint64_t *pw = (const uint64_t *)pbuf + (size_t)pg * N;
                            q = pw[n];
                            qr = pw[nr];
                            qd = pw[nd];
                        } else if (mode == 1 && sh) {
                            const bool two = pg + 1 < pgroups;
                            q = (load_word<REPR>(buf, pg, n, N) >> sh) |
                                (two ? load_word<REPR>(buf, pg + 1, n, N) << (64 - sh) : 0ull);
                            qr = (load_word<REPR>(buf, pg, nr, N) >> sh) |
                                 (two ? load_word<REPR>(buf, pg + 1, nr, N) << (64 - sh) : 0ull);
                            qd = (load_word<REPR>(buf, pg, nd, N) >> sh) |
                                 (two ? load_word<REPR>(buf, pg + 1, nd, N) << (64 - sh) : 0ull);
                        } else {
                            q = load_word<REPR>(pbuf, pg, n, N);
                            qr = load_word<REPR>(pbuf, pg, nr, N);
                            qd = load_word<REPR>(pbuf, pg, nd, N);
                        }
                        vinc(cH, w ^ q);
                        vinc2(cK, br ^ q ^ qr, bd ^ q ^ qd);
                    }
                }
            }
            const int p1 = planes_for(tsites), p2 = planes_for(2 * tsites);
            totU += vflush(cU, p2);
            totD += vflush(cD, p1);
            if (mode) {
                totH += vflush(cH, p1);
                totK += vflush(cK, p2);
            }
        }
    } else {
        // energies and magnetisations only: carry-save counting
        const bool ea = R.model == PA_EA_PMJ;      // the ferromagnet's bond signs are all +1
        const int gl = live ? g : it.group0;       // a group that exists, for lanes that drop their loads
        for (int b0 = 64 * sub; b0 < N; b0 += 16 * 64 * wpg) {
            const int tsites = min(16, (N - b0 + 64 * wpg - 1) / (64 * wpg));
            Csa2 cU;
            Csa1 cD;
            // U sites at a time, all their loads issued before the first use
            // and none behind a branch (a wavefront or lane with no site
            // there loads one that exists and drops it); the carries of
            // weight 4 and up pair up on uniform branches
            constexpr int U = REPR == PA_MSC64 ? 4 : 2;
#pragma unroll 1
            for (int t0 = 0; t0 < 16; t0 += U) {
                uint64_t w[U], wr[U], wd[U];
                uint32_t jn[U];
                bool ok[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int n = b0 + (t0 + u) * 64 * wpg + lane;
                    ok[u] = live && n < N;
                    const int nn = ok[u] ? n : 0;
                    const int y = nn / L, x = nn - y * L;
                    const int nr = y * L + (x + 1 == L ? 0 : x + 1);
                    const int nd = (y + 1 == L ? 0 : y + 1) * L + x;
                    jn[u] = ea ? R.jbits[nn] : 0u;
                    w[u] = own(gl, nn, N);
                    wr[u] = own(gl, nr, N);
                    wd[u] = own(gl, nd, N);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const uint64_t z = ok[u] ? ~0ull : 0ull;   // zero inputs past the last site
                    const uint64_t ur = (w[u] ^ wr[u] ^ ((jn[u] & 1) ? ~0ull : 0ull)) & z;
                    const uint64_t ud = (w[u] ^ wd[u] ^ ((jn[u] & 2) ? ~0ull : 0ull)) & z;
                    cU.add(t0 + u, ur, ud);
                    cD.add(t0 + u, w[u] & z);
                }
            }
            uint64_t pl[VB];
            cU.planes(pl);
            totU += vflush(pl, planes_for(2 * tsites));
            cD.planes(pl);
            totD += vflush(pl, planes_for(tsites));
        }
    }
    if (wpg > 1) {
        red[0][wv][lane] = totU;
        red[1][wv][lane] = totD;
        red[2][wv][lane] = totH;
        red[3][wv][lane] = totK;
    }
    __syncthreads();
    if (!live || sub != 0) return;
    uint32_t U = totU, D = totD, H = totH, Kc = totK;
    for (int k = 1; k < wpg; ++k) {
        U += red[0][wv + k][lane];
        D += red[1][wv + k][lane];
        H += red[2][wv + k][lane];
        Kc += red[3][wv + k][lane];
    }
    const int j = g * 64 + lane;
    const bool valid = j < Rc;
    const int64_t E = 2 * (int64_t)U - 2 * (int64_t)N;
    const int64_t M = R.exact_dos ? 0 : (int64_t)N - 2 * (int64_t)D;   // energies only at theta = infinity
    if (valid) R.E[it.pop][S.cur][j] = (int32_t)E;
    const int64_t v = valid ? 1 : 0;
    const bool pair = mode && ((pairmask >> lane) & 1u);
    const int64_t pv = pair ? 1 : 0;
    const int64_t Q = (int64_t)N - 2 * (int64_t)H, Ql = 2 * (int64_t)N - 2 * (int64_t)Kc;
    int64_t part[MEAS_PART];
    part[0] = wave_sum<int64_t>(v * E);
    part[1] = wave_sum<int64_t>(v * E * E);
    part[2] = wave_sum<int64_t>(v * (M < 0 ? -M : M));
    part[3] = wave_sum<int64_t>(v * M * M);
    part[4] = wave_sum<int64_t>(pv);
    part[5] = wave_sum<int64_t>(pv * Q);
    part[6] = wave_sum<int64_t>(pv * (Q < 0 ? -Q : Q));
    part[7] = wave_sum<int64_t>(pv * Q * Q);
    part[8] = wave_sum<int64_t>(pv * Ql);
    part[9] = wave_sum<int64_t>(pv * Ql * Ql);
    part[10] = wave_min(valid ? (int)E : INT32_MAX);
    if (R.qhist) {
        const size_t Np1 = (size_t)N + 1;
        int32_t *h0 = &R.qh[((size_t)it.pop * R.K + S.i) * Np1];
        auto add = [&](uint32_t bin, int n) {
            atomicAdd(&h0[bin], n);
            if (R.overlap == PA_Q_TWO_POP) atomicAdd(&R.qh[((size_t)1 * R.K + S.i) * Np1 + bin], n);
        };
        // Few bins: all pairs of a wavefront with one distance at once (atomics
        // on one address follow one another: L = 4, R = 58348 128 -> 42 us per
        // launch; step at L = 6, R = 2e4 93 -> 89, but L = 8 86 -> 91)
        if (N <= 36) {
            for (uint64_t left = wave_ballot(pair); left != 0;) {
                const int lead = __ffsll((unsigned long long)left) - 1;
                const uint32_t bin = (uint32_t)__builtin_amdgcn_readlane((int)H, lead);
                const uint64_t same = wave_ballot(pair && H == bin);
                if (lane == lead) add(bin, __popcll(same));
                left &= ~same;
            }
        } else if (pair) {
            add(H, 1);
        }
    }
    if (lane < MEAS_PART) {
        int64_t mine = 0;
#pragma unroll
        for (int k = 0; k < MEAS_PART; ++k)
            if (lane == k) mine = part[k];
        R.part[it.pop][(size_t)g * MEAS_PART + lane] = mine;
    }
}

template <int REPR, bool WITH_Q, int W>
__global__ void __launch_bounds__(64 * W) k_measure(const SweepItem *items, const RunInfo *runs, const PopState *st)
{
    __shared__ uint32_t red[4][W][64];
    extern __shared__ uint64_t words[];   // [groups of the item][N] when staged
    const SweepItem it = items[blockIdx.x];
    const RunInfo &R = runs[it.run];
    const PopState &S = st[it.run * MAX_POP + it.pop];
    if (!pop_active(S) || words_current(R, S) != (REPR == PA_MSC64)) return;
    const int wpg = meas_waves_per_group(R.N) * (W / MEAS_WAVES);
    const int wv = wave_id();
    const int k = wv / wpg, sub = wv - k * wpg;
    const int g = it.group0 + k;
    const bool live = k < it.ngroups && g * 64 < S.Rcur;
    // int8 layout: each group's words are read once from memory into LDS
    // (four 16-byte loads per site, packed on the way), then every site reads
    // itself and its neighbours from there instead of loading and packing
    // three 64-byte rows.  Not for lattices above MEAS_STAGE_N sites, nor at
    // theta = infinity (no lattice to read).  The bit-packed layout reads its
    // 8-byte words straight from memory: staging them measured slower (34
    // against 22 us at L = 64, R = 1e5), the barrier after the staging pass
    // keeping loads and counting from overlapping.
    const bool staged = REPR == PA_INT8 && R.N <= MEAS_STAGE_N && !(R.exact_dos && S.i > 0);
    const uint64_t *lw = nullptr;
    if (staged) {
        uint64_t *mine = words + (size_t)k * R.N;
        if (live) {
            const uint8_t *buf = R.spins[it.pop][S.cur];
            for (int n = sub * 64 + (threadIdx.x & 63); n < R.N; n += 64 * wpg)
                mine[n] = load_word<REPR>(buf, g, n, R.N);
        }
        __syncthreads();
        lw = mine;
    }
    switch (R.L) {
    case 8: measure_group<REPR, 8, WITH_Q, W>(it, g, sub, wpg, live, R, S, st, red, lw); break;
    case 16: measure_group<REPR, 16, WITH_Q, W>(it, g, sub, wpg, live, R, S, st, red, lw); break;
    case 24: measure_group<REPR, 24, WITH_Q, W>(it, g, sub, wpg, live, R, S, st, red, lw); break;
    case 32: measure_group<REPR, 32, WITH_Q, W>(it, g, sub, wpg, live, R, S, st, red, lw); break;
    case 48: measure_group<REPR, 48, WITH_Q, W>(it, g, sub, wpg, live, R, S, st, red, lw); break;
    case 64: measure_group<REPR, 64, WITH_Q, W>(it, g, sub, wpg, live, R, S, st, red, lw); break;
    default: measure_group<REPR, 0, WITH_Q, W>(it, g, sub, wpg, live, R, S, st, red, lw); break;
    }
}

// ----------------------------------------------- theta = infinity draws
//
// Step (iv) in the theta = infinity limit (Sec. V C): every replica's energy
// is an independent draw from the exact distribution at beta_i.  One thread
// per replica (a wavefront per replica group): a 64-bit Philox draw and a
// binary search over the level thresholds C[i][0..N] (non-decreasing) for
// the first level with v < C_m, the top level if there is none.
__global__ void __launch_bounds__(256) k_dos_sample(const Item *items, int n_items, const RunInfo *runs,
                                                    const PopState *st)
{
    const int idx = blockIdx.x * 4 + wave_id(), lane = threadIdx.x & 63;
    if (idx >= n_items) return;
    const Item it = items[idx];
    const RunInfo &R = runs[it.run];
    if (!R.exact_dos) return;
    const PopState &S = st[it.run * MAX_POP + it.pop];
    if (!pop_active(S)) return;
    const int j = it.group * 64 + lane;
    if (j >= S.Rcur) return;
    const int N = R.N, i = S.i;
    const u32x4 o = philox10((uint32_t)j, 0u, (uint32_t)i, (TAG_DOS << 28) | ((uint32_t)it.pop << 24), R.key0,
                             R.key1);
    const uint64_t v = (uint64_t)o.x | ((uint64_t)o.y << 32);
    const uint64_t *C = R.tabD + (size_t)i * (N + 1);
    int lo = 0, hi = N + 1;
    while (lo < hi) {
        const int m = (lo + hi) >> 1;
        if (v < C[m]) hi = m;
        else lo = m + 1;
    }
    R.E[it.pop][S.cur][j] = -2 * N + 4 * min(lo, N);
}

// ---------------------------------------------- permutation pairing (q)
//
// Sec. III D, pairings from permutations (Wang et al.), for runs with
// PA_Q_WANG / PA_Q_WANG_RDM, before the measurement of every temperature:
//   k_wang_lds     one workgroup per run: the permutations and the repair
//   k_wang_pairs   (the same for runs too large for LDS);
//   k_wang_rows    the population as bit rows, one per replica;
//   k_wang_gather  the partners' configurations as bit-packed words;
// then k_measure takes the pairs (j, pi_j) like any other overlap pairs.
//
// The random permutations are index orders of 64-bit Philox keys: a key's
// top bits pick one of B >= R_i buckets (a power of two, so about one key
// per bucket), the bucket counts are scanned into starts, the indices are
// scattered into their buckets, and an index's rank is its bucket's start
// plus the members of the bucket with a smaller (key, index).  The repair is
// serial by nature: the mismatched positions are listed in search order,
// then one wavefront takes them in turn and finds each exchange partner
// with a 64-wide search (a ballot over consecutive candidates).  With the
// identity search pattern the candidates inside the mismatched replica's
// own family, which is one run of equal labels, are skipped without being
// tested: none of them can qualify.  Data that other wavefronts wrote in
// the same launch is read with device-coherent loads after the writers have
// waited for their stores.

constexpr int WANG_THREADS = 1024;

__device__ __forceinline__ int32_t ldc(const int32_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void stc(int32_t *p, int32_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Barrier after which every wavefront's earlier stores have completed.
__device__ __forceinline__ void wg_sync_stores()
{
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
}

// Key of index k for the pairing at temperature i: words 0-1 (pi) or 2-3
// (the search pattern) of Philox(seed; k, 0, i, TAG_PERM << 28).
__device__ __forceinline__ uint64_t perm_key(int k, int i, int which, uint32_t key0, uint32_t key1)
{
    const u32x4 o = philox10((uint32_t)k, 0u, (uint32_t)i, TAG_PERM << 28, key0, key1);
    return which == 0 ? ((uint64_t)o.x | ((uint64_t)o.y << 32)) : ((uint64_t)o.z | ((uint64_t)o.w << 32));
}

// Exclusive prefix over the workgroup of one value per thread; *total gets
// the sum.  sh: 17 ints of LDS.
__device__ int block_scan_excl(int v, int *sh, int *total)
{
    const int lane = threadIdx.x & 63, wv = wave_id(), nw = blockDim.x >> 6;
    int x = v;
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) sh[wv] = x;
    __syncthreads();
    if (threadIdx.x == 0) {
        int a = 0;
        for (int w = 0; w < nw; ++w) {
            const int t = sh[w];
            sh[w] = a;
            a += t;
        }
        sh[16] = a;
    }
    __syncthreads();
    const int r = sh[wv] + x - v;
    *total = sh[16];
    __syncthreads();
    return r;
}

// For runs too large for k_wang_lds: the same in global memory.
__global__ void __launch_bounds__(WANG_THREADS) k_wang_pairs(const RunInfo *runs, const PopState *st, int run0,
                                                              uint32_t lds_bytes)
{
    __shared__ int sh[17];
    __shared__ int big;
    const int run = run0 + blockIdx.x;
    const RunInfo &R = runs[run];
    if (!is_wang(R.overlap) || wang_lds_bytes(R.R_cap) <= lds_bytes) return;
    const PopState &S = st[run * MAX_POP];
    if (!pop_active(S)) return;
    const int Rc = S.Rcur, i = S.i;
    const int T = blockDim.x, tid = threadIdx.x;
    const int32_t *fam = R.fam[0][S.cur];
    const WangBufs W = wang_bufs(R.wang, R.R_cap, R.wang_lb);
    const bool rdm = R.overlap == PA_Q_WANG_RDM;
    const uint32_t key0 = R.key0, key1 = R.key1;
    // A family of more than Rc / 2 replicas (then no valid pairing exists)
    // covers the middle index: it is one run of equal labels.
    if (tid == 0) {
        const int h = Rc >> 1, f = fam[h];
        int lo = 0, hi = h;
        while (lo < hi) {
            const int m = (lo + hi) >> 1;
            if (fam[m] < f) lo = m + 1;
            else hi = m;
        }
        const int first = lo;
        lo = h + 1;
        hi = Rc;
        while (lo < hi) {
            const int m = (lo + hi) >> 1;
            if (fam[m] <= f) lo = m + 1;
            else hi = m;
        }
        big = 2 * (int64_t)(lo - first) > (int64_t)Rc ? 1 : 0;
        if (big) stc(&W.hdr[0], 1);
    }
    __syncthreads();
    if (big) return;

    int lbc = 1;
    while ((1 << lbc) < Rc) ++lbc;
    const int B = 1 << lbc, shift = 64 - lbc;
    for (int which = 0; which < (rdm ? 2 : 1); ++which) {
        int32_t *out = which == 0 ? W.pi : W.sigma;
        for (int b = tid; b < B; b += T) stc(&W.cnt[b], 0);
        wg_sync_stores();
        for (int k = tid; k < Rc; k += T) atomicAdd(&W.cnt[perm_key(k, i, which, key0, key1) >> shift], 1);
        wg_sync_stores();
        const int seg = (B + T - 1) / T;
        const int b0 = min(B, tid * seg), b1 = min(B, b0 + seg);
        int sum = 0;
        for (int b = b0; b < b1; ++b) sum += ldc(&W.cnt[b]);
        int total;
        int acc = block_scan_excl(sum, sh, &total);
        for (int b = b0; b < b1; ++b) {
            const int c = ldc(&W.cnt[b]);
            stc(&W.start[b], acc);
            stc(&W.cnt[b], acc);   // fill cursor of the bucket
            acc += c;
        }
        if (tid == 0) stc(&W.start[B], Rc);
        wg_sync_stores();
        for (int k = tid; k < Rc; k += T) {
            const int b = (int)(perm_key(k, i, which, key0, key1) >> shift);
            stc(&W.members[atomicAdd(&W.cnt[b], 1)], k);
        }
        wg_sync_stores();
        for (int k = tid; k < Rc; k += T) {
            const uint64_t kk = perm_key(k, i, which, key0, key1);
            const int b = (int)(kk >> shift);
            const int lo = ldc(&W.start[b]), hi = ldc(&W.start[b + 1]);
            int r = lo;
            for (int q = lo; q < hi; ++q) {
                const int m = ldc(&W.members[q]);
                if (m == k) continue;
                const uint64_t km = perm_key(m, i, which, key0, key1);
                r += (km < kk || (km == kk && m < k)) ? 1 : 0;
            }
            stc(&out[r], k);
        }
        wg_sync_stores();
    }

    // families of the initial partners, and the mismatched positions in
    // search order (ascending)
    for (int k = tid; k < Rc; k += T) stc(&W.fampi[k], fam[ldc(&W.pi[k])]);
    wg_sync_stores();
    const int seg = (Rc + T - 1) / T;
    const int t0 = min(Rc, tid * seg), t1 = min(Rc, t0 + seg);
    int mine = 0;
    for (int t = t0; t < t1; ++t) {
        const int k = rdm ? ldc(&W.sigma[t]) : t;
        mine += ldc(&W.fampi[k]) == fam[k] ? 1 : 0;
    }
    int nlist;
    int pos = block_scan_excl(mine, sh, &nlist);
    for (int t = t0; t < t1; ++t) {
        const int k = rdm ? ldc(&W.sigma[t]) : t;
        if (ldc(&W.fampi[k]) == fam[k]) stc(&W.list[pos++], t);
    }
    wg_sync_stores();
    // The repair, one wavefront, over the list in batches of 64 entries.
    // What does not change during the repair (position, its place in the
    // search order, its family, the end of its family's run of labels, its
    // initial partner) is loaded for a whole batch at once; an entry is
    // still open unless an earlier exchange in this repair took its
    // position as the partner (an exchange leaves both of its positions
    // matched for good), which the lanes track by comparing positions.
    // With the identity pattern the mismatches of one family come one after
    // the other, and a candidate that failed for one of them fails for the
    // next as well (exchanges only hand this family's replicas to
    // candidates), so the search resumes after the previous partner
    // (unwrapped candidate index prev_u).
    int status = 0;
    if (tid < 64) {
        const int lane = tid;
        int prev_f = -1;
        int64_t prev_u = 0;
        for (int e0 = 0; e0 < nlist && status == 0; e0 += 64) {
            const int e = e0 + lane;
            int t_l = 0, k_l = -1, f_l = 0, hi_l = 0, p_l = 0;
            bool open_l = false;
            if (e < nlist) {
                t_l = ldc(&W.list[e]);
                k_l = rdm ? ldc(&W.sigma[t_l]) : t_l;
                f_l = fam[k_l];
                open_l = ldc(&W.fampi[k_l]) == f_l;
                p_l = ldc(&W.pi[k_l]);
                if (!rdm) {   // the first later index with another label
                    int lo = t_l + 1, hi = Rc;
                    while (lo < hi) {
                        const int m = (lo + hi) >> 1;
                        if (fam[m] == f_l) lo = m + 1;
                        else hi = m;
                    }
                    hi_l = lo;
                }
            }
            const int nb = min(64, nlist - e0);
            for (int j = 0; j < nb; ++j) {
                if (!__builtin_amdgcn_readlane((int)open_l, j)) continue;
                const int t = __builtin_amdgcn_readlane(t_l, j), k = __builtin_amdgcn_readlane(k_l, j);
                const int fk = __builtin_amdgcn_readlane(f_l, j), pk = __builtin_amdgcn_readlane(p_l, j);
                int64_t u = t + 1;
                if (!rdm) {
                    u = __builtin_amdgcn_readlane(hi_l, j);
                    if (fk == prev_f && prev_u + 1 > u) u = prev_u + 1;
                }
                const int64_t uend = (int64_t)t + Rc;   // candidates t + 1 .. t + Rc - 1, indices mod Rc
                int found = -1, fm = 0;
                for (; u < uend; u += 64) {
                    const int64_t uu = u + lane;
                    bool ok = false;
                    int m = 0, fpm = 0;
                    if (uu < uend) {
                        const int q = (int)(uu >= Rc ? uu - Rc : uu);
                        m = rdm ? ldc(&W.sigma[q]) : q;
                        fpm = ldc(&W.fampi[m]);
                        ok = fam[m] != fk && fpm != fk;
                    }
                    const uint64_t bal = __ballot(ok);
                    if (bal) {
                        const int first = __ffsll((unsigned long long)bal) - 1;
                        found = __builtin_amdgcn_readlane(m, first);
                        fm = __builtin_amdgcn_readlane(fpm, first);
                        prev_u = u + first;
                        break;
                    }
                }
                if (found < 0) {   // impossible with no family above Rc / 2
                    status = 2;
                    break;
                }
                if (lane == 0) {
                    const int pm = ldc(&W.pi[found]);
                    stc(&W.pi[k], pm);
                    stc(&W.pi[found], pk);
                    stc(&W.fampi[k], fm);
                    stc(&W.fampi[found], fk);
                }
                __builtin_amdgcn_s_waitcnt(0);
                if (k_l == found) open_l = false;
                prev_f = fk;
            }
        }
    }
    if (tid == 0) {
        stc(&W.hdr[0], status);
        stc(&W.hdr[1], nlist);
    }
}

// Permutation pairing of a run whose arrays fit a workgroup's LDS
// (wang_lds_bytes): everything k_wang_pairs does, in LDS with 16-bit indices
// and family numbers (the labels are runs, so their ranks do), and the repair
// along the identity pattern a family at a time.  A mismatched position of
// family f takes the first later position of another family whose partner is
// not of f either; the mismatches of one family follow one another, a
// position that fails for one of them fails for the next, and an exchange
// changes none of the positions still ahead.  So the n-th open mismatch of the
// family takes the n-th position that qualifies, and a wavefront makes up to
// 64 exchanges at once instead of one after the other.  The random pattern
// mixes the families: one exchange at a time, in registers, which hold 128
// positions of the pattern.  16 runs of 2e4 replicas at L = 32, beta 0 to 2.4,
// average per launch: 2219 us in global memory, 189 here; random pattern 2734
// and 781 (1220 with the positions read from LDS for each exchange).
__global__ void __launch_bounds__(WANG_THREADS) k_wang_lds(const RunInfo *runs, const PopState *st, int run0,
                                                           uint32_t lds_bytes)
{
    extern __shared__ __align__(16) uint16_t w16[];
    __shared__ int sh[17];
    __shared__ uint16_t kq[64];
    const int run = run0 + blockIdx.x;
    const RunInfo &R = runs[run];
    if (!is_wang(R.overlap) || wang_lds_bytes(R.R_cap) > lds_bytes) return;
    const PopState &S = st[run * MAX_POP];
    if (!pop_active(S)) return;
    const int Rc = S.Rcur, i = S.i;
    constexpr int T = WANG_THREADS;
    const int tid = threadIdx.x, lane = tid & 63;
    const int32_t *fam = R.fam[0][S.cur];
    const WangBufs W = wang_bufs(R.wang, R.R_cap, R.wang_lb);
    const bool rdm = R.overlap == PA_Q_WANG_RDM;
    const uint32_t key0 = R.key0, key1 = R.key1;
    const int Re = (Rc + 7) & ~7;   // 16-byte steps between the arrays
    uint16_t *Lpi = w16;

    // The permutations: index orders of the keys.  A key's top bits pick one
    // of B buckets; counts, their prefix (the fill cursors, which end as the
    // buckets' ends), members, and an index's rank from its bucket's members.
    int lbc = 1;
    while ((1 << lbc) < Rc) ++lbc;
    const int B = 1 << lbc, shift = 64 - lbc;
    uint32_t *cnt = (uint32_t *)(w16 + Re);      // B u16, two to a word
    uint16_t *members = w16 + Re + B;
    auto bump = [&](int b) { return (int)(atomicAdd(&cnt[b >> 1], 1u << (16 * (b & 1))) >> (16 * (b & 1))) & 0xFFFF; };
    auto cursor = [&](int b) { return (int)((const uint16_t *)cnt)[b]; };
    for (int which = rdm ? 1 : 0; which >= 0; --which) {
        for (int k = tid; k < (B + 1) / 2; k += T) cnt[k] = 0;
        __syncthreads();
        for (int k = tid; k < Rc; k += T) bump((int)(perm_key(k, i, which, key0, key1) >> shift));
        __syncthreads();
        const int seg = (B + T - 1) / T, b0 = min(B, tid * seg), b1 = min(B, b0 + seg);
        int sum = 0;
        for (int b = b0; b < b1; ++b) sum += cursor(b);
        int total;
        int acc = block_scan_excl(sum, sh, &total);
        for (int b = b0; b < b1; ++b) {
            const int c = cursor(b);
            ((uint16_t *)cnt)[b] = (uint16_t)acc;
            acc += c;
        }
        __syncthreads();
        for (int k = tid; k < Rc; k += T)
            members[bump((int)(perm_key(k, i, which, key0, key1) >> shift))] = (uint16_t)k;
        __syncthreads();
        for (int k = tid; k < Rc; k += T) {
            const uint64_t kk = perm_key(k, i, which, key0, key1);
            const int b = (int)(kk >> shift);
            const int lo = b ? cursor(b - 1) : 0, hi = cursor(b);
            int r = lo;
            for (int q = lo; q < hi; ++q) {
                const int m = members[q];
                if (m == k) continue;
                const uint64_t km = perm_key(m, i, which, key0, key1);
                r += (km < kk || (km == kk && m < k)) ? 1 : 0;
            }
            if (which) W.sigma[r] = k;
            else Lpi[r] = (uint16_t)k;
        }
        __syncthreads();   // (of the workgroup's global stores, too: sigma is read back below)
    }

    // Family numbers: the rank of a label among the runs of equal labels.
    // (Then the labels' space becomes the partners' numbers and the list.)
    uint16_t *Lfam = w16 + Re, *Lfpi = w16 + 2 * Re, *aux = w16 + 3 * Re;
    int32_t *lab = (int32_t *)(w16 + 2 * Re);
    for (int k = tid; k < Rc; k += T) lab[k] = fam[k];
    __syncthreads();
    const int seg = (Rc + T - 1) / T, t0 = min(Rc, tid * seg), t1 = min(Rc, t0 + seg);
    int starts = 0;
    for (int t = t0; t < t1; ++t) starts += t > 0 && lab[t] != lab[t - 1] ? 1 : 0;
    int all;
    int number = block_scan_excl(starts, sh, &all);
    for (int t = t0; t < t1; ++t) {
        number += t > 0 && lab[t] != lab[t - 1] ? 1 : 0;
        Lfam[t] = (uint16_t)number;
    }
    __syncthreads();
    // A family of more than Rc / 2 replicas covers the middle index; then no
    // valid pairing exists.
    int mine = 0;
    for (int t = t0; t < t1; ++t) mine += Lfam[t] == Lfam[Rc >> 1] ? 1 : 0;
    int most;
    block_scan_excl(mine, sh, &most);
    if (2 * most > Rc) {
        if (tid == 0) W.hdr[0] = 1;
        return;
    }
    for (int k = tid; k < Rc; k += T) Lfpi[k] = Lfam[Lpi[k]];
    if (rdm)
        for (int k = tid; k < Rc; k += T) aux[k] = (uint16_t)W.sigma[k];
    __syncthreads();
    // the mismatched positions, ascending (what the random pattern needs is
    // their number)
    mine = 0;
    for (int t = t0; t < t1; ++t) mine += Lfpi[t] == Lfam[t] ? 1 : 0;
    int nlist;
    int pos = block_scan_excl(mine, sh, &nlist);
    if (!rdm)
        for (int t = t0; t < t1; ++t)
            if (Lfpi[t] == Lfam[t]) aux[pos++] = (uint16_t)t;
    __syncthreads();
    int status = 0;
    if (tid < 64 && !rdm) {
        int prev_f = -1, u = 0;   // the family of the last exchange, the next candidate (unwrapped)
        for (int e0 = 0; e0 < nlist && status == 0; e0 += 64) {
            const bool in = e0 + lane < nlist;
            const int k_l = in ? (int)aux[e0 + lane] : 0, f_l = in ? (int)Lfam[k_l] : -1;
            int hi_l = k_l + 1;   // the first later index of another family
            for (int top = in ? Rc : 0; hi_l < top;) {
                const int m = (hi_l + top) >> 1;
                if (Lfam[m] == f_l) hi_l = m + 1;
                else top = m;
            }
            bool todo = in;
            while (status == 0) {
                // open: not taken as a partner by an earlier exchange
                const bool open = todo && Lfpi[k_l] == f_l;
                const uint64_t bal = __ballot(open);
                if (bal == 0) break;
                const int first = __ffsll((unsigned long long)bal) - 1;
                const int f = __builtin_amdgcn_readlane(f_l, first), hi = __builtin_amdgcn_readlane(hi_l, first);
                const uint64_t same = __ballot(open && f_l == f);
                if (open && f_l == f) {
                    kq[rank_below(same, 0)] = (uint16_t)k_l;
                    todo = false;
                }
                __builtin_amdgcn_wave_barrier();
                if (f != prev_f) u = hi;
                prev_f = f;
                const int end = hi + Rc;   // past every position once
                int left = __popcll(same), base = 0;
                while (left > 0 && u < end) {
                    const int uu = u + lane, m = wang_candidate(uu, Rc);
                    const int fm = Lfpi[m];
                    const bool ok = uu < end && Lfam[m] != f && fm != f;
                    const uint64_t v = __ballot(ok);
                    const int r = rank_below(v, 0), take = min(__popcll(v), left);
                    if (ok && r < take) {
                        const int k = kq[base + r];
                        const uint16_t a = Lpi[k], b = Lpi[m];
                        Lpi[k] = b;
                        Lpi[m] = a;
                        Lfpi[k] = (uint16_t)fm;
                        Lfpi[m] = (uint16_t)f;
                    }
                    __builtin_amdgcn_wave_barrier();
                    const uint64_t lastb = __ballot(ok && r == left - 1);   // the candidate that ends the family
                    u += lastb ? __ffsll((unsigned long long)lastb) : 64;
                    left -= take;
                    base += take;
                }
                if (left > 0) status = 2;   // impossible with no family above Rc / 2
            }
        }
    } else if (tid < 64) {
        // two windows of 64 search positions in registers: (m, pi, family,
        // partner's family), a position past the end in no family
        int m0, p0, f0, q0, m1, p1, f1, q1;
        auto take_in = [&](int base, int &m, int &p, int &f, int &q) {
            const int t = base + lane;
            m = t < Rc ? (int)aux[t] : -1;
            p = m < 0 ? 0 : (int)Lpi[m];
            f = m < 0 ? -1 : (int)Lfam[m];
            q = m < 0 ? -2 : (int)Lfpi[m];
        };
        auto put_back = [&](int m, int p, int q) {
            if (m < 0) return;
            Lpi[m] = (uint16_t)p;
            Lfpi[m] = (uint16_t)q;
        };
        take_in(0, m0, p0, f0, q0);
        for (int base = 0; base < Rc && status == 0; base += 64) {
            take_in(base + 64, m1, p1, f1, q1);
            for (;;) {
                const uint64_t bal = __ballot(f0 == q0);
                if (bal == 0) break;
                const int j = __ffsll((unsigned long long)bal) - 1;
                const int fk = __builtin_amdgcn_readlane(f0, j), pk = __builtin_amdgcn_readlane(p0, j);
                const uint64_t v0 = __ballot(m0 >= 0 && f0 != fk && q0 != fk) & (~(uint64_t)0 << j);
                const uint64_t v1 = __ballot(m1 >= 0 && f1 != fk && q1 != fk);
                if (v0 | v1) {
                    const int first = __ffsll((unsigned long long)(v0 ? v0 : v1)) - 1;
                    const int pm = __builtin_amdgcn_readlane(v0 ? p0 : p1, first);
                    const int fm = __builtin_amdgcn_readlane(v0 ? q0 : q1, first);
                    if (v0 && lane == first) {
                        p0 = pk;
                        q0 = fk;
                    }
                    if (!v0 && lane == first) {
                        p1 = pk;
                        q1 = fk;
                    }
                    if (lane == j) {
                        p0 = pm;
                        q0 = fm;
                    }
                    continue;
                }
                // further on, round the end up to position base + j again
                put_back(m0, p0, q0);
                put_back(m1, p1, q1);
                __builtin_amdgcn_wave_barrier();
                const int t = base + j, k = __builtin_amdgcn_readlane(m0, j);
                bool found = false;
                for (int u = min(base + 128, Rc); u < t + Rc && !found; u += 64) {
                    const int uu = u + lane;
                    const int m = (int)aux[uu < t + Rc ? (uu >= Rc ? uu - Rc : uu) : t];
                    const int fm = Lfpi[m];
                    const uint64_t v = __ballot(uu < t + Rc && Lfam[m] != fk && fm != fk);
                    if (v == 0) continue;
                    found = true;
                    if (lane == __ffsll((unsigned long long)v) - 1) {
                        Lpi[k] = Lpi[m];
                        Lpi[m] = (uint16_t)pk;
                        Lfpi[k] = (uint16_t)fm;
                        Lfpi[m] = (uint16_t)fk;
                    }
                    __builtin_amdgcn_wave_barrier();
                }
                if (!found) {
                    status = 2;
                    break;
                }
                take_in(base, m0, p0, f0, q0);
                take_in(base + 64, m1, p1, f1, q1);
            }
            put_back(m0, p0, q0);
            m0 = m1;
            p0 = p1;
            f0 = f1;
            q0 = q1;
        }
    }
    if (tid == 0) {
        W.hdr[0] = status;
        W.hdr[1] = nlist;
    }
    __syncthreads();
    for (int k = tid; k < Rc; k += T) W.pi[k] = Lpi[k];
}

// Calibration: two independent chains of Philox calls per lane, all in
// registers (the outputs feed the next call's counter); an empty statement
// keeps the final values alive without a memory write.
__global__ void __launch_bounds__(256) k_philox_rate(int calls, uint32_t k0, uint32_t k1)
{
    uint32_t a0 = threadIdx.x, a1 = blockIdx.x, a2 = 0, a3 = 1;
    uint32_t b0 = threadIdx.x ^ 0x9E3779B9u, b1 = blockIdx.x, b2 = 2, b3 = 3;
    for (int k = 0; k < calls; ++k) {
        const u32x4 x = philox10(a0, a1, a2, a3, k0, k1);
        const u32x4 y = philox10(b0, b1, b2, b3, k0, k1);
        a0 = x.x; a1 = x.y; a2 = x.z; a3 = x.w;
        b0 = y.x; b1 = y.y; b2 = y.z; b3 = y.w;
    }
    asm volatile("" ::"v"(a0), "v"(a1), "v"(a2), "v"(a3), "v"(b0), "v"(b1), "v"(b2), "v"(b3));
}

hipError_t launch_philox_rate(int calls, hipStream_t s, int *blocks, int *threads)
{
    *blocks = 2048;
    *threads = 256;
    k_philox_rate<<<*blocks, *threads, 0, s>>>(calls, 0x01234567u, 0x89ABCDEFu);
    return hipGetLastError();
}


__device__ __forceinline__ bool wang_group_live(const Item &it, const RunInfo &R, const PopState &S)
{
    return is_wang(R.overlap) && it.pop == 0 && pop_active(S) && it.group * 64 < S.Rcur &&
           wang_bufs(R.wang, R.R_cap, R.wang_lb).hdr[0] == 0;
}

// Bit rows of population 0: word blk * 64 groups_cap + j holds, in bit s,
// the spin of replica j at site 64 blk + s.  One wavefront per replica
// group: lane s takes the word of site 64 blk + s (64 replicas), and a
// 64 x 64 transpose turns the 64 site words into the group's 64 rows.
template <int REPR>
__global__ void __launch_bounds__(256) k_wang_rows(const Item *items, int n_items, const RunInfo *runs,
                                                   const PopState *st)
{
    const int idx = blockIdx.x * 4 + wave_id(), lane = threadIdx.x & 63;
    if (idx >= n_items) return;
    const Item it = items[idx];
    const RunInfo &R = runs[it.run];
    const PopState &S = st[it.run * MAX_POP];
    if (!wang_group_live(it, R, S)) return;
    const int N = R.N, g = it.group, nb = (N + 63) / 64;
    const size_t R64 = (size_t)R.groups_cap * 64;
    uint64_t *rows = wang_rows(R.wang, R.R_cap) + (size_t)g * 64 + lane;
    const uint8_t *buf = R.spins[0][S.cur];
#pragma unroll 4
    for (int blk = 0; blk < nb; ++blk) {
        const int n = blk * 64 + lane;
        const uint64_t w = n < N ? load_word<REPR>(buf, g, n, N) : 0ull;
        rows[(size_t)blk * R64] = transpose64(w);
    }
}

// Partner words: bit b of word (g, n) is the spin at site n of the partner
// pi_j of replica j = 64 g + b.  One wavefront per group: lane b reads its
// partner's bit row one 64-site block at a time, and a transpose turns the
// 64 rows into the block's 64 site words.  Lanes past R_i read replica 0
// (their bits are never used).
__global__ void __launch_bounds__(256) k_wang_gather(const Item *items, int n_items, const RunInfo *runs,
                                                     const PopState *st)
{
    const int idx = blockIdx.x * 4 + wave_id(), lane = threadIdx.x & 63;
    if (idx >= n_items) return;
    const Item it = items[idx];
    const RunInfo &R = runs[it.run];
    const PopState &S = st[it.run * MAX_POP];
    if (!wang_group_live(it, R, S)) return;
    const int N = R.N, g = it.group, nb = (N + 63) / 64;
    const size_t R64 = (size_t)R.groups_cap * 64;
    const WangBufs W = wang_bufs(R.wang, R.R_cap, R.wang_lb);
    const int j = g * 64 + lane;
    const int p = j < S.Rcur ? W.pi[j] : 0;
    const uint64_t *rows = wang_rows(R.wang, R.R_cap) + p;
    uint64_t *dst = (uint64_t *)wang_partner_words(R, S) + (size_t)g * N;
#pragma unroll 4
    for (int blk = 0; blk < nb; ++blk) {
        const uint64_t col = transpose64(rows[(size_t)blk * R64]);
        const int n = blk * 64 + lane;
        if (n < N) dst[n] = col;
    }
}

// The record of a population's temperature from its sums (in the order of
// the accumulators) and the pair sums of population 0 (with two populations
// both records carry them).
__device__ __forceinline__ void write_record(const RunInfo &R, PopState &S, int pop, const int64_t *acc,
                                             const int64_t *acc0, int32_t emin)
{
    pa_obs o;
    o.R_i = S.Rcur;
    o.lnQ = S.i == 0 ? 0.0 : S.lnQ;
    o.A = S.A;
    o.sumE = acc[A_SUME];
    o.sumE2 = acc[A_SUME2];
    o.sumAbsM = acc[A_SUMABSM];
    o.sumM2 = acc[A_SUMM2];
    o.nPairs = acc0[A_NPAIRS];
    o.sumQ = acc0[A_SUMQ];
    o.sumAbsQ = acc0[A_SUMABSQ];
    o.sumQ2 = acc0[A_SUMQ2];
    o.sumQl = acc0[A_SUMQL];
    o.sumQl2 = acc0[A_SUMQL2];
    o.famSumSq = acc[A_FAMSQ];
    o.famMax = acc[A_FAMMAX];
    o.nFam = acc[A_NFAM];
    o.Emin = emin;
    o.status = PA_OK;
    obs_at(R, S.i, pop) = o;
    S.Emin = emin;
}

// The records of a run's populations from the accumulators that other
// workgroups of the launch added to, and the accumulators reset (one thread).
__device__ __forceinline__ void write_records(const RunInfo &R, PopState *st)
{
    int64_t acc0[NACC] = {};
    for (int p = 0; p < R.npop; ++p) {
        PopState &S = st[p];
        if (!pop_active(S)) continue;
        int64_t acc[NACC];
#pragma unroll
        for (int k = 0; k < NACC; ++k) {
            acc[k] = take(&S.acc[k]);
            if (p == 0) acc0[k] = acc[k];
        }
        write_record(R, S, p, acc, acc0, take(&S.EminAcc));
        for (int k = 0; k < NACC; ++k) put(&S.acc[k], (int64_t)0);
        put(&S.EminAcc, (int32_t)INT32_MAX);
    }
}

// Per chunk of CH replicas (CH / 64 groups): the groups' partial sums, and
// the family statistics.  Family labels are non-decreasing in the replica
// index (they start as f_j = j and every resampling copies parents in
// order), so each family is one run of equal labels.  A replica at rank r
// inside its family contributes 2r + 1 to sum_f c_f^2 (the ranks of a
// family of size c give c^2), r + 1 to max_f c_f, and 1 to the number of
// families if r = 0.  The rank needs the family's first index: the last
// start at or before the replica inside the chunk, else (a family that
// began in an earlier chunk) found by binary search for the first label
// equal to the chunk's first.
__global__ void __launch_bounds__(CH_THREADS) k_meas_chunk(const ChunkItem *items, const RunInfo *runs,
                                                           PopState *st)
{
    __shared__ int64_t red[3][CH_THREADS / 64];
    __shared__ int lds_scan[CH_THREADS / 64 + 1];
    __shared__ int first_start;
    const ChunkItem it = items[blockIdx.x];
    const RunInfo &R = runs[it.run];
    PopState &S = st[it.run * MAX_POP + it.pop];
    if (!pop_active(S)) return;
    const int Rc = S.Rcur;
    const int j0 = it.chunk * CH;
    if (j0 >= Rc) return;
    const int lane = threadIdx.x & 63, wv = wave_id();
    int chunks = 0;   // of the run's populations
    for (int p = 0; p < R.npop; ++p)
        if (pop_active(st[it.run * MAX_POP + p])) chunks += (st[it.run * MAX_POP + p].Rcur + CH - 1) / CH;
    // group partials: groups [j0/64, j0/64 + CH/64), one per lane of wave 0
    int64_t part[NACC];   // as the accumulators: the first ten, then the families
#pragma unroll
    for (int k = 0; k < NACC; ++k) part[k] = 0;
    int emin = INT32_MAX;
    const int g = j0 / 64 + lane;
    if (wv == 0 && lane < CH / 64 && g * 64 < Rc) {
#pragma unroll
        for (int k = 0; k < MEAS_PART - 1; ++k) part[k] = R.part[it.pop][(size_t)g * MEAS_PART + k];
        emin = (int)R.part[it.pop][(size_t)g * MEAS_PART + MEAS_PART - 1];
    }
    // families
    const int32_t *fam = R.fam[it.pop][S.cur];
    if (wv == 0) {
        // first index with the label of replica j0 (labels ascend): a
        // 64-way search by the whole wavefront, the first such index lying
        // in [lo, hi] with fam[hi] equal to the label
        int fs = j0;
        if (j0 > 0 && fam[j0 - 1] == fam[j0]) {
            const int32_t f = fam[j0];
            int lo = 0, hi = j0 - 1;
            while (lo < hi) {
                const int step = (hi - lo + 63) / 64;
                const int p = lo + lane * step;
                const int c = __popcll(__ballot(p < hi && fam[p] < f));   // probes below the first index
                if (c == 0) break;   // fam[lo] is the label
                lo += (c - 1) * step + 1;
                hi = min(hi, lo - 1 + step);
            }
            fs = lo;
        }
        if (lane == 0) first_start = fs;
    }
    const int jb = j0 + threadIdx.x * CH_PER;
    int32_t lab[CH_PER];
    load_block(fam, jb, Rc, 0, lab);
    // the label before each of them: the previous lane's last, or memory
    int32_t prev = __shfl_up(lab[CH_PER - 1], 1, 64);
    if (lane == 0) prev = jb > 0 && jb < Rc ? fam[jb - 1] : -1;   // labels are not negative
    bool start[CH_PER];
    int last = -1;
#pragma unroll
    for (int q = 0; q < CH_PER; ++q) {
        start[q] = jb + q < Rc && (q ? lab[q - 1] : prev) != lab[q];
        if (start[q]) last = jb + q;
    }
    // exclusive max-scan of the threads' last starts
    int incl = last;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(incl, o, 64);
        if (lane >= o) incl = max(incl, t);
    }
    if (lane == 63) lds_scan[wv] = incl;
    __syncthreads();
    int before = first_start;   // start of the family of replica j0
    for (int k = 0; k < wv; ++k) before = max(before, lds_scan[k]);
    {
        const int t = __shfl_up(incl, 1, 64);
        if (lane >= 1) before = max(before, t);
    }
    int64_t sq = 0, mx = 0, nf = 0;
    int s = before;
#pragma unroll
    for (int q = 0; q < CH_PER; ++q) {
        const int j = jb + q;
        if (j < Rc) {
            if (start[q]) s = j;
            const int64_t r = j - s;
            sq += 2 * r + 1;
            mx = r + 1 > mx ? r + 1 : mx;
            nf += start[q] ? 1 : 0;
        }
    }
    sq = wave_sum<int64_t>(sq);
    nf = wave_sum<int64_t>(nf);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const int64_t t = __shfl_xor(mx, o, 64);
        mx = t > mx ? t : mx;
    }
    if (wv == 0) {
#pragma unroll
        for (int k = 0; k < MEAS_PART - 1; ++k) part[k] = wave_sum<int64_t>(part[k]);
        emin = wave_min(emin);
    }
    if (lane == 0) {
        red[0][wv] = sq;
        red[1][wv] = mx;
        red[2][wv] = nf;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t a = 0, b = 0, c = 0;
        for (int k = 0; k < CH_THREADS / 64; ++k) {
            a += red[0][k];
            b = red[1][k] > b ? red[1][k] : b;
            c += red[2][k];
        }
        part[A_FAMSQ] = a;
        part[A_FAMMAX] = b;
        part[A_NFAM] = c;
        if (chunks == 1) {   // the run's only chunk: its sums are the record's
            const int64_t none[A_FAMSQ] = {};
            write_record(R, S, it.pop, part, it.pop == 0 ? part : none, emin);
        } else {
            unsigned long long *acc = (unsigned long long *)S.acc;
#pragma unroll
            for (int k = 0; k < NACC; ++k) {
                if (k == A_FAMMAX) atomicMax(&acc[k], (unsigned long long)part[k]);
                else if (k < A_NPAIRS || k >= A_FAMSQ || part[A_NPAIRS]) atomicAdd(&acc[k], (unsigned long long)part[k]);
            }
            atomicMin(&S.EminAcc, emin);
        }
    }
    // the last chunk of the run's populations writes the records
    if (chunks > 1 && last_of(&st[it.run * MAX_POP].done, chunks) && threadIdx.x == 0)
        write_records(R, st + it.run * MAX_POP);
}

// ---------------------------------------------------------------- Sec. IV

// Log free-energy weights per run and temperature: simplified
// ln R_i + A_i (Eq. (simpleWeight)) and full ln R_i + sum_{k<=i}
// ln(R_{k-1}/R) + A_i (Eq. (appropriateWeight)); NaN where the record is not
// OK or the temperature is not reached yet.  One workgroup per run, over the
// temperatures a tile at a time: every thread reads its temperature's
// records and takes the logarithms, then one thread adds the ln(R_{k-1}/R)
// terms from LDS in order of k (the same sums as a sequential pass), instead
// of one thread per run walking all K records with a load and a logarithm in
// each step of a dependent chain.
constexpr int SCAN_THREADS = 256;

__global__ void __launch_bounds__(SCAN_THREADS) k_logw(const RunInfo *runs, const pa_obs *obs, int n_runs,
                                                       int npop_ctx, int pop, int kind, int i_done, double *logw)
{
    __shared__ double term[SCAN_THREADS];   // ln(R_{i-1}/R) of the tile's temperatures, then the running sums
    __shared__ double carry;
    const int run = blockIdx.x, t = threadIdx.x;
    const RunInfo &R = runs[run];
    const bool full = (kind & 1) == PA_W_FULL;
    if (t == 0) carry = 0.0;
    for (int base = 0; base < R.K; base += SCAN_THREADS) {
        const int i = base + t;
        double a = NAN;   // ln R_i + A_i
        if (i < R.K) {
            const pa_obs &o = obs[((size_t)i * n_runs + run) * npop_ctx + pop];
            term[t] = i > 0 ? log((double)obs[((size_t)(i - 1) * n_runs + run) * npop_ctx + pop].R_i /
                                  (double)R.R)
                            : 0.0;
            if (i <= i_done && o.status == PA_OK && pop < R.npop) a = log((double)o.R_i) + o.A;
        }
        __syncthreads();
        if (t == 0) {
            double cum = carry;
            const int n = min(SCAN_THREADS, R.K - base);
            for (int k = 0; k < n; ++k) {
                if (base + k > 0) cum += term[k];
                term[k] = cum;
            }
            carry = cum;
        }
        __syncthreads();
        if (i < R.K) logw[(size_t)run * R.K + i] = a + (full ? term[t] : 0.0);
        __syncthreads();   // the next tile rewrites term
    }
}

// Per (group of M runs, temperature i): weights w = softmax of
// the log weights over the included runs; configurational averages; the
// weighted variance estimators through the Eq. (Wvar_bound) identity; the
// sample variance of w and its log-normal prediction; and ln W[Q_i] with
// the weights of temperature i-1 renormalised over the runs included at i
// (stored in minus_beta_WF, summed over i by k_wavg_cumsum).
// T = 1: a thread per (group, temperature) goes through the group's M runs;
// T = 64: a wavefront does, a run to a lane, and adds the runs' terms in the
// same order, one sum to a lane, from LDS (in one thread a long group is a
// chain of loads and divisions: a weighted average of 256 runs at 89
// temperatures 867 -> 82 us with the copy of its result).
template <int T>
struct GroupSums {
    static constexpr int MOST = 10;
    double *lds;   // T = 64: MOST rows of 65 of this wavefront

    // out[s] = the sum of t[s] over the runs m for which f(m, t) is true
    template <int NS, typename F>
    __device__ __forceinline__ void add(int M, double (&out)[NS], F f) const
    {
        static_assert(NS <= MOST, "");
        const int lane = threadIdx.x & (T - 1);
        double acc = 0.0;
#pragma unroll
        for (int s = 0; s < NS; ++s) out[s] = 0.0;
        for (int m0 = 0; m0 < M; m0 += T) {
            double t[NS] = {};
            const bool in = m0 + lane < M && f(m0 + lane, t);
            if (T == 1) {
#pragma unroll
                for (int s = 0; s < NS; ++s) out[s] = in ? out[s] + t[s] : out[s];
                continue;
            }
            // a run left out adds zero, which changes no sum (none is -0)
#pragma unroll
            for (int s = 0; s < NS; ++s) lds[s * 65 + lane] = in ? t[s] : 0.0;
            sync();
            if (lane < NS)
                for (int q = 0; q < min(T, M - m0); ++q) acc += lds[lane * 65 + q];
            sync();
        }
        if (T > 1) {
#pragma unroll
            for (int s = 0; s < NS; ++s) out[s] = __shfl(acc, s, 64);
        }
    }
    // the largest f(m), NaN left out, and how many there are
    template <typename F>
    __device__ __forceinline__ double largest(int M, int *count, F f) const
    {
        const int lane = threadIdx.x & (T - 1);
        double mx = -INFINITY;
        int n = 0;
        for (int m = lane; m < M; m += T) {
            const double a = f(m);
            if (isnan(a)) continue;
            mx = fmax(mx, a);
            ++n;
        }
        if (T > 1) {
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                mx = fmax(mx, __shfl_xor(mx, o, 64));
                n += __shfl_xor(n, o, 64);
            }
        }
        *count = n;
        return mx;
    }

private:
    static __device__ __forceinline__ void sync()
    {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
};
constexpr int GROUP_THREADS = 128;

template <int T>
__global__ void __launch_bounds__(GROUP_THREADS) k_wavg(const RunInfo *runs, const pa_obs *obs, const double *logw,
                                                        const double *qw, int n_runs, int npop_ctx, int pop, int M,
                                                        int K, pa_wavg *out)
{
    __shared__ double lds[T > 1 ? GROUP_THREADS / 64 : 1][T > 1 ? GroupSums<T>::MOST * 65 : 1];
    const int gi = (blockIdx.x * blockDim.x + threadIdx.x) / T;
    const int ngroups = n_runs / M;
    if (gi >= ngroups * K) return;
    const GroupSums<T> sums = {lds[T > 1 ? threadIdx.x >> 6 : 0]};
    const bool writes = (threadIdx.x & (T - 1)) == 0;
    const int grp = gi / K, i = gi - grp * K, run0 = grp * M;
    const int N = runs[run0].N;
    const double b = runs[run0].beta[i];
    auto lw = [&](int m) { return logw[(size_t)(run0 + m) * K + i]; };
    auto rec = [&](int m) -> const pa_obs & { return obs[((size_t)i * n_runs + run0 + m) * npop_ctx + pop]; };
    pa_wavg w = {};
    int n = 0;
    const double amax = sums.largest(M, &n, lw);
    w.n_included = n;
    if (n == 0) {
        const double nan = NAN;
        w.W_e = w.W_e2 = w.Wvar_c = w.Wconf_c = w.W_m = w.W_m2 = nan;
        w.Wvar_chi = w.Wconf_chi = w.W_absq = w.W_q2 = w.W_ql = nan;
        w.minus_beta_WF = w.var_w = w.var_w_pred = nan;
        if (writes) out[(size_t)grp * K + i] = w;
        return;
    }
    double z[1];
    sums.add(M, z, [&](int m, double *t) {
        const double a = lw(m);
        t[0] = exp(a - amax);
        return !isnan(a);
    });
    const double Z = z[0];
    const double dN = (double)N;
    double f[10];
    sums.add(M, f, [&](int m, double *t) {
        const double a = lw(m);
        if (isnan(a)) return false;
        const pa_obs &o = rec(m);
        const double wm = exp(a - amax) / Z;
        const double Ri = (double)o.R_i;
        const __int128 vE = (__int128)o.R_i * o.sumE2 - (__int128)o.sumE * o.sumE;
        const __int128 vM = (__int128)o.R_i * o.sumM2 - (__int128)o.sumAbsM * o.sumAbsM;
        t[0] = wm * ((double)o.sumE / (dN * Ri));
        t[1] = wm * ((double)o.sumE2 / (dN * dN * Ri));
        t[2] = wm * (b * b * (double)vE / (dN * Ri * Ri));
        t[3] = wm * ((double)o.sumAbsM / (dN * Ri));
        t[4] = wm * ((double)o.sumM2 / (dN * dN * Ri));
        t[5] = wm * (b * (double)vM / (dN * Ri * Ri));
        const double wq = qw[(size_t)(run0 + m) * K + i];   // overlap weights (exclusion applied)
        if (o.nPairs > 0 && !isnan(wq)) {
            const double np = (double)o.nPairs;
            t[6] = wq * ((double)o.sumAbsQ / (dN * np));
            t[7] = wq * ((double)o.sumQ2 / (dN * dN * np));
            t[8] = wq * ((double)o.sumQl / (2.0 * dN * np));
        }
        t[9] = o.A;
        return true;
    });
    w.W_e = f[0];
    w.W_e2 = f[1];
    w.Wconf_c = f[2];
    w.W_m = f[3];
    w.W_m2 = f[4];
    w.Wconf_chi = f[5];
    w.W_absq = f[6];
    w.W_q2 = f[7];
    w.W_ql = f[8];
    if (isnan(qw[(size_t)run0 * K + i])) w.W_absq = w.W_q2 = w.W_ql = NAN;
    const double meanA = f[9] / n;
    double v[4];
    sums.add(M, v, [&](int m, double *t) {
        const double a = lw(m);
        if (isnan(a)) return false;
        const pa_obs &o = rec(m);
        const double wm = exp(a - amax) / Z;
        const double Ri = (double)o.R_i;
        const double e = (double)o.sumE / (dN * Ri), mm = (double)o.sumAbsM / (dN * Ri);
        t[0] = wm * (e - w.W_e) * (e - w.W_e);
        t[1] = wm * (mm - w.W_m) * (mm - w.W_m);
        t[2] = (wm - 1.0 / n) * (wm - 1.0 / n);
        t[3] = (o.A - meanA) * (o.A - meanA);
        return true;
    });
    w.Wvar_c = w.Wconf_c + b * b * dN * v[0];
    w.Wvar_chi = w.Wconf_chi + b * dN * v[1];
    w.var_w = v[2] / n;
    w.var_w_pred = (exp(v[3] / n) - 1.0) / ((double)n * n);
    if (i == 0) {
        w.minus_beta_WF = NAN;
        for (int m = 0; m < M; ++m)
            if (!isnan(lw(m))) {
                w.minus_beta_WF = rec(m).A;
                break;
            }
    } else {
        auto before = [&](int m) { return logw[(size_t)(run0 + m) * K + i - 1]; };
        int any;
        const double mx = sums.largest(M, &any, [&](int m) { return isnan(lw(m)) ? NAN : before(m) + rec(m).lnQ; });
        const double mx0 = sums.largest(M, &any, [&](int m) { return isnan(lw(m)) ? NAN : before(m); });
        double s[2];
        sums.add(M, s, [&](int m, double *t) {
            if (isnan(lw(m))) return false;
            t[0] = exp(before(m) + rec(m).lnQ - mx);
            t[1] = exp(before(m) - mx0);
            return true;
        });
        w.minus_beta_WF = (mx + log(s[0])) - (mx0 + log(s[1]));
    }
    if (writes) out[(size_t)grp * K + i] = w;
}

// A family holds more than R_i / 2 replicas in run `run` at temperature i
// (population pop, or either population of a two-population run).
__device__ __forceinline__ bool large_family(const RunInfo &R, const pa_obs *obs, int i, int run, int n_runs,
                                             int npop_ctx, int pop)
{
    for (int p = 0; p < R.npop; ++p) {
        if (p != pop && R.overlap != PA_Q_TWO_POP) continue;
        const pa_obs &o = obs[((size_t)i * n_runs + run) * npop_ctx + p];
        if (2 * o.famMax > o.R_i) return true;
    }
    return false;
}

// Weights of the overlap averages: the free-energy weights of k_logw,
// normalised over the included runs of the group (with
// PA_W_EXCLUDE_LARGE_FAMILY also leaving out runs with a family above
// R_i / 2); 0 for a run left out, NaN for every run if none is left.
template <int T>
__global__ void __launch_bounds__(GROUP_THREADS) k_qweights(const RunInfo *runs, const pa_obs *obs,
                                                            const double *logw, int n_runs, int npop_ctx, int pop,
                                                            int M, int K, int flags, double *qw)
{
    __shared__ double lds[T > 1 ? GROUP_THREADS / 64 : 1][T > 1 ? GroupSums<T>::MOST * 65 : 1];
    const int gi = (blockIdx.x * blockDim.x + threadIdx.x) / T;
    const int ngroups = n_runs / M;
    if (gi >= ngroups * K) return;
    const GroupSums<T> sums = {lds[T > 1 ? threadIdx.x >> 6 : 0]};
    const int grp = gi / K, i = gi - grp * K, run0 = grp * M;
    const bool excl = flags & PA_W_EXCLUDE_LARGE_FAMILY;
    auto lw = [&](int m) {
        return excl && large_family(runs[run0 + m], obs, i, run0 + m, n_runs, npop_ctx, pop)
                   ? NAN
                   : logw[(size_t)(run0 + m) * K + i];
    };
    int n = 0;
    const double amax = sums.largest(M, &n, lw);
    double Z[1];
    sums.add(M, Z, [&](int m, double *t) {
        const double a = lw(m);
        t[0] = exp(a - amax);
        return !isnan(a);
    });
    for (int m = threadIdx.x & (T - 1); m < M; m += T) {
        const double a = lw(m);
        qw[(size_t)(run0 + m) * K + i] = n == 0 ? NAN : (isnan(a) ? 0.0 : exp(a - amax) / Z[0]);
    }
}

// Eq. (W_conf_q): one workgroup per (group, temperature), threads over the
// N + 1 bins: W[P(q)](d) = sum_m w_m h_m(d) / nPairs_m, runs in group order.
__global__ void k_wqhist(const RunInfo *runs, const pa_obs *obs, const double *qw, int n_runs, int npop_ctx,
                         int pop, int M, int K, double *out)
{
    const int grp = blockIdx.x / K, i = blockIdx.x - grp * K;
    const int N = runs[grp * M].N;
    const size_t Np1 = (size_t)N + 1;
    double *o = out + ((size_t)grp * K + i) * Np1;
    for (size_t d = threadIdx.x; d < Np1; d += blockDim.x) {
        double acc = 0.0;
        bool none = false;
        for (int m = 0; m < M; ++m) {
            const int run = grp * M + m;
            const double w = qw[(size_t)run * K + i];
            if (isnan(w)) {
                none = true;
                break;
            }
            if (w == 0.0) continue;
            const pa_obs &ob = obs[((size_t)i * n_runs + run) * npop_ctx + pop];
            if (ob.nPairs <= 0) continue;
            const int32_t h = runs[run].qh[((size_t)pop * K + i) * Np1 + d];
            acc += w * ((double)h / (double)ob.nPairs);
        }
        o[d] = none ? NAN : acc;
    }
}

// Family statistics of every (run, temperature) of population pop.
__global__ void k_famstats(const RunInfo *runs, const pa_obs *obs, int n_runs, int npop_ctx, int pop, int K,
                           int i_done, pa_famstat *out)
{
    const int gi = blockIdx.x * blockDim.x + threadIdx.x;
    if (gi >= n_runs * K) return;
    const int run = gi / K, i = gi - run * K;
    const RunInfo &R = runs[run];
    pa_famstat f;
    f.rho_t = NAN;
    f.R_i = 0;
    f.famMax = 0;
    f.large = 0;
    f.excluded = 1;
    if (pop < R.npop && i < R.K && i <= i_done) {
        const pa_obs &o = obs[((size_t)i * n_runs + run) * npop_ctx + pop];
        f.R_i = (int32_t)o.R_i;
        f.famMax = (int32_t)o.famMax;
        if (o.status == PA_OK && o.R_i > 0) {
            f.rho_t = (double)o.famSumSq / (double)o.R_i;
            f.large = 2 * o.famMax > o.R_i ? 1 : 0;
            f.excluded = large_family(R, obs, i, run, n_runs, npop_ctx, pop) ? 1 : 0;
        }
    }
    out[gi] = f;
}

// -beta_i W[F_i] = ln Z(beta_0) + sum_{k=1..i} ln W[Q_k], Eq. (W_F); NaN
// from the first temperature with no run included on.  One workgroup per
// group of runs: the tile's terms are staged in LDS by all threads and
// summed in order of i by one thread.
__global__ void __launch_bounds__(SCAN_THREADS) k_wavg_cumsum(pa_wavg *out, int ngroups, int K)
{
    __shared__ double v[SCAN_THREADS];
    __shared__ uint8_t none[SCAN_THREADS];   // no run included at that temperature
    __shared__ double carry;
    const int grp = blockIdx.x, t = threadIdx.x;
    if (grp >= ngroups) return;
    if (t == 0) carry = 0.0;
    for (int base = 0; base < K; base += SCAN_THREADS) {
        const int i = base + t;
        if (i < K) {
            const pa_wavg &w = out[(size_t)grp * K + i];
            v[t] = w.minus_beta_WF;
            none[t] = w.n_included == 0;
        }
        __syncthreads();
        if (t == 0) {
            double c = carry;
            const int n = min(SCAN_THREADS, K - base);
            for (int k = 0; k < n; ++k) {
                if (none[k]) c = NAN;
                else c = base + k == 0 ? v[k] : c + v[k];
                v[k] = c;
            }
            carry = c;
        }
        __syncthreads();
        if (i < K) out[(size_t)grp * K + i].minus_beta_WF = v[t];
        __syncthreads();   // the next tile rewrites v and none
    }
}

// ------------------------------------------------------------- launchers

#define PA_CHECK_LAUNCH()                          \
    do {                                           \
        hipError_t e_ = hipGetLastError();         \
        if (e_ != hipSuccess) return e_;           \
    } while (0)

hipError_t launch_fill_u32(void *p, uint32_t v, size_t n, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    const unsigned blocks = (unsigned)std::min<size_t>((n + 255) / 256, 4096);
    k_fill_u32<<<blocks, 256, 0, s>>>((uint32_t *)p, v, n);
    return hipGetLastError();
}

hipError_t launch_init(const LaunchCtx &c, const uint64_t *dseed)
{
    k_init_couplings<<<c.n_runs, 256, 0, c.stream>>>(c.runs + c.run0, dseed);
    PA_CHECK_LAUNCH();
    k_init_fam<<<c.n_runs, 256, 0, c.stream>>>(c.runs + c.run0);
    PA_CHECK_LAUNCH();
    if (c.repr == PA_MSC64) k_init_spins<PA_MSC64><<<c.n_items, 256, 0, c.stream>>>(c.items, c.runs);
    else k_init_spins<PA_INT8><<<c.n_items, 256, 0, c.stream>>>(c.items, c.runs);
    return hipGetLastError();
}

hipError_t launch_anneal(const LaunchCtx &c)
{
    k_rw_chunk<<<c.n_chunk_items, CH_THREADS, 0, c.stream>>>(c.chunk_items, c.runs, c.st);
    return hipGetLastError();
}

hipError_t launch_resample(const LaunchCtx &c)
{
    if (c.fused_max > 0) {
        const int threads = c.fused_max <= 512 ? 64 : (c.fused_max <= CH ? 256 : 1024);
        k_resample_run<<<dim3(c.n_runs, c.npop_ctx), threads, fused_lds(c.fused_max, c.any_multinomial), c.stream>>>(
            c.runs + c.run0, c.st + (size_t)c.run0 * MAX_POP);
        PA_CHECK_LAUNCH();
    }
    if (c.any_chained) {
        if (c.any_nearest) {
            k_cnt_chunk<<<c.n_chunk_items, CH_THREADS, 0, c.stream>>>(c.chunk_items, c.runs, c.st);
            PA_CHECK_LAUNCH();
        }
        if (c.any_multinomial) {
            k_mn_draws<<<c.n_chunk_items * CH_PER, CH_THREADS, 0, c.stream>>>(c.chunk_items, c.runs, c.st);
            PA_CHECK_LAUNCH();
            k_cnt_scan_chunk<<<c.n_chunk_items, CH_THREADS, 0, c.stream>>>(c.chunk_items, c.runs, c.st);
            PA_CHECK_LAUNCH();
        }
        k_parent<<<c.n_chunk_items, CH_THREADS, 0, c.stream>>>(c.chunk_items, c.runs, c.st);
        PA_CHECK_LAUNCH();
    }
    if (c.n_meas_items > 0) {
        const int split = c.copy_split > 1 ? c.copy_split : 1;
        if (c.repr == PA_MSC64)
            k_copy<PA_MSC64><<<c.n_meas_items * split, MEAS_THREADS, 0, c.stream>>>(c.meas_items, c.runs, c.st,
                                                                                  split);
        else
            k_copy<PA_INT8><<<c.n_meas_items * split, MEAS_THREADS, 0, c.stream>>>(c.meas_items, c.runs, c.st,
                                                                                 split);
    }
    return hipGetLastError();
}

hipError_t launch_clear_draws(const LaunchCtx &c)
{
    k_clear_draws<<<c.n_chunk_items, CH_THREADS, 0, c.stream>>>(c.chunk_items, c.runs);
    return hipGetLastError();
}

// Allows launches of a kernel on this device with `bytes` of dynamic LDS.  The
// permission is the kernel's, not a context's, so it is only ever raised:
// contexts and servers that live beside each other launch with what each of
// them needs.  Up to 64 KB, the kernel's own arrays included, needs none.
static hipError_t allow_lds(const void *kernel, size_t bytes)
{
    constexpr size_t OWN = 8192;   // no kernel has more of its own
    if (bytes + OWN <= 65536) return hipSuccess;
    static std::mutex mu;
    static std::map<std::pair<int, const void *>, size_t> allowed;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lock(mu);
    size_t &have = allowed[{dev, kernel}];
    if (bytes <= have) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e == hipSuccess) have = bytes;
    return e;
}

hipError_t prepare_fused_lds(size_t bytes) { return allow_lds((const void *)k_resample_run, bytes); }
hipError_t prepare_wang_lds(size_t bytes) { return allow_lds((const void *)k_wang_lds, bytes); }

hipError_t launch_words(const LaunchCtx &c, int max_N)
{
    k_bytes_words<true><<<dim3(c.n_items, (max_N + WORDS_SEG - 1) / WORDS_SEG), 256, 0, c.stream>>>(c.items, c.runs,
                                                                                                  c.st);
    return hipGetLastError();
}

hipError_t launch_sweep_bytes(const LaunchCtx &c, const WideRun *wide, int n_wide, int max_N)
{
    if (!c.any_swept || c.n_items == 0) return hipSuccess;
    hipError_t e = launch_words(c, max_N);
    if (e != hipSuccess) return e;
    if ((e = launch_sweep_msc(c)) != hipSuccess) return e;
    for (int k = 0; k < n_wide; ++k) {
        const WideRun &w = wide[k];
        const int nh = w.L * w.L / 2;
        // chunks per wavefront by the chunks there are per SIMD (1024), as in
        // the batched sweep's default shape
        const double chunks = (double)w.groups_cap * w.npop * nh / 64.0;
        const int cpw = chunks < 2 * 1024.0 ? 1 : (chunks < 12 * 1024.0 ? 2 : WIDE_CHUNKS);
        const int tiles = (nh + 64 * WIDE_WAVES * cpw - 1) / (64 * WIDE_WAVES * cpw);
        const dim3 grid((unsigned)w.groups_cap * tiles, w.npop);
        for (int s = 0; s < w.theta; ++s)
            for (int colour = 0; colour < 2; ++colour) {
                if (w.ea)
                    k_sweep_wide<true><<<grid, 64 * WIDE_WAVES, 0, c.stream>>>(c.runs, c.st, w.run, s, colour, cpw,
                                                                              tiles, c.stats);
                else
                    k_sweep_wide<false><<<grid, 64 * WIDE_WAVES, 0, c.stream>>>(c.runs, c.st, w.run, s, colour, cpw,
                                                                               tiles, c.stats);
                PA_CHECK_LAUNCH();
            }
    }
    k_bytes_words<false><<<dim3(c.n_items, (max_N + WORDS_SEG - 1) / WORDS_SEG), 256, 0, c.stream>>>(c.items, c.runs,
                                                                                                   c.st);
    return hipGetLastError();
}

size_t msc_lds_bytes(int N, int groups, bool ea, int threads, int mode)
{
    return msc_lds_need(N, groups, ea, threads / 64, mode);
}

// The sweep kernel for a launch: one compiled for a single (L, model), the one
// for any size of a model (L = 0), or the one that dispatches per item.
using SweepKernel = void (*)(const SweepItem *, int, const RunInfo *, const PopState *, int, unsigned long long *,
                             unsigned int *, unsigned int *, SweepList *, int, uint32_t);

SweepKernel msc_kernel(int L, int ea)
{
    if (L < 0) return k_sweep_msc<-1, false>;
    switch (2 * L + (ea ? 1 : 0)) {
    case 0: return k_sweep_msc<0, false>;
    case 1: return k_sweep_msc<0, true>;
    case 16: return k_sweep_msc<8, false>;
    case 17: return k_sweep_msc<8, true>;
    case 32: return k_sweep_msc<16, false>;
    case 33: return k_sweep_msc<16, true>;
    case 48: return k_sweep_msc<24, false>;
    case 49: return k_sweep_msc<24, true>;
    case 64: return k_sweep_msc<32, false>;
    case 65: return k_sweep_msc<32, true>;
    case 96: return k_sweep_msc<48, false>;
    case 97: return k_sweep_msc<48, true>;
    case 128: return k_sweep_msc<64, false>;
    case 129: return k_sweep_msc<64, true>;
    default: return k_sweep_msc<-1, false>;
    }
}

bool msc_specialised(int L) { return L == 8 || L == 16 || L == 24 || L == 32 || L == 48 || L == 64; }

hipError_t prepare_msc_lds(size_t bytes)
{
    static const int Ls[] = {8, 16, 24, 32, 48, 64, 0, -1};
    for (int L : Ls)
        for (int ea = 0; ea < 2; ++ea) {
            const hipError_t e = allow_lds((const void *)msc_kernel(L, ea), bytes);
            if (e != hipSuccess) return e;
        }
    return hipSuccess;
}

// One launch per class (sweep_classes below): the kernel compiled for the
// lattice size and model when every sweeping run shares them; one such
// kernel per (size, model) when every class is large enough to fill the
// chip; else the kernel for any size of the model they share, or the one that
// dispatches per item.  (On the serving mix,
// whose per-size launches are too small to fill the chip, launching each
// size on its own measured 3.03 against 3.54 thousand flips/ns while busy.)
hipError_t launch_sweep_msc(const LaunchCtx &c)
{
    for (int k = 0; k < c.n_sweep_classes; ++k) {
        const SweepClass &q = c.sweep_cls[k];
        if (q.count == 0) continue;
        const bool persistent = q.grid > 0 && q.grid < q.count;
        // chunked items wait on one another, which only the list order of
        // the persistent grid makes safe
        if (q.nchunk > 1 && !persistent) return hipErrorInvalidConfiguration;
        const int grid = persistent ? q.grid : q.count;
        const int mode = c.sweep_dense | (c.sweep_pooled << 8);
        msc_kernel(q.L, q.ea)<<<grid, c.sweep_threads, q.lds, c.stream>>>(
            c.sweep_items + q.first, q.count, c.runs, c.st, mode, c.stats,
            persistent ? c.sweep_queue : nullptr, c.sweep_flags, q.lists, q.n_lists, (uint32_t)q.lds);
        PA_CHECK_LAUNCH();
    }
    return hipSuccess;
}

int sweep_classes(std::vector<SweepItem> &items, const std::vector<int> &run_L, const std::vector<int> &run_ea,
                  SweepClass *cls, int threads, int mode, bool split_ok)
{
    // items of runs without Metropolis sweeps are not launched at all (the
    // kernel of another size must never see them)
    std::vector<SweepItem> out;
    out.reserve(items.size());
    // per kept item: 2 L + ea of the kernel that sweeps it, 0 + ea for a size
    // without a kernel of its own, -1 where the lists are not streamed
    std::vector<int> keys;
    for (const SweepItem &it : items) {
        const int L = run_L[it.run];
        if (L == 0) continue;
        const int ea = run_ea[it.run] ? 1 : 0;
        keys.push_back(!msc_streamed(L * L, it.ngroups, mode) ? -1 : (msc_specialised(L) ? 2 * L : 0) + ea);
        out.push_back(it);
    }
    items.swap(out);
    if (items.empty()) return 0;
    auto lds_of = [&](const SweepItem &it) {
        const int L = run_L[it.run];
        return msc_lds_bytes(L * L, it.ngroups, run_ea[it.run] != 0, threads, mode);
    };
    // One launch per (size, model) when every item has a kernel compiled
    // for its size and each class fills at least half of the workgroups
    // that kernel keeps resident: those kernels use fewer registers and the
    // queue rings, so they run more workgroups per CU than the dispatching
    // kernel (the 4096-run batch of four sizes: 6.00 against 6.63 ms per
    // sweep).  Small classes (a serving mix) keep one dispatching launch,
    // since launches that cannot fill the chip one after another are slower.
    std::vector<int> ks(keys);
    std::sort(ks.begin(), ks.end());
    ks.erase(std::unique(ks.begin(), ks.end()), ks.end());
    bool split = split_ok && ks.size() > 1 && (int)ks.size() <= MAX_SWEEP_CLASSES && ks[0] > 1;
    std::vector<SweepClass> cand(ks.size());
    for (size_t q = 0; split && q < ks.size(); ++q) {
        SweepClass &C = cand[q];
        C.L = ks[q] / 2;
        C.ea = ks[q] & 1;
        C.count = 0;
        C.lds = 0;
        C.grid = 0;
        for (size_t t = 0; t < items.size(); ++t)
            if (keys[t] == ks[q]) {
                ++C.count;
                C.lds = std::max(C.lds, lds_of(items[t]));
            }
        const int resident = sweep_msc_resident(threads, C.lds, C.L, C.ea);
        if (resident <= 0 || 2 * C.count < resident) split = false;
    }
    if (split) {
        // the items of each class together, in their largest-first order
        std::vector<SweepItem> sorted;
        sorted.reserve(items.size());
        for (size_t q = 0; q < ks.size(); ++q) {
            cand[q].first = (int)sorted.size();
            for (size_t t = 0; t < items.size(); ++t)
                if (keys[t] == ks[q]) sorted.push_back(items[t]);
            cls[q] = cand[q];
        }
        items.swap(sorted);
        return (int)ks.size();
    }
    // several sizes of one model share the kernel for any size of that model;
    // anything else takes the one that chooses per item
    int key = ks[0];
    for (int k : ks) key = key < 0 || k < 0 || ((key ^ k) & 1) ? -1 : (key == k ? k : key & 1);
    SweepClass &C = cls[0];
    C.first = 0;
    C.count = (int)items.size();
    C.L = key < 0 ? -1 : key / 2;
    C.ea = key < 0 ? 0 : key & 1;
    C.grid = 0;
    C.lds = 0;
    for (const SweepItem &it : items) C.lds = std::max(C.lds, lds_of(it));
    return 1;
}

// Two chunks: a list of items per CU, and only what has to be cut is.  The
// items (dealt out so that every list gets its share of each size) are laid
// end to end over the lists, each of capacity T; one that crosses from a
// list's end into the next one's beginning is cut there, its first sweeps the
// beginning of the next.  Taken in the order beginning, whole items (largest
// first), end, every CU is busy until about T, and an item's beginning is done
// long before its end is taken (McNaughton's wrap-around rule).  A cut falls
// between sweeps, so the least T that fits is searched upwards from the mean.
// A chunk costs its sweeps and about a third of one for moving its lattices.
struct SweepPlan {
    std::vector<SweepItem> items;
    std::vector<SweepList> lists;
};

static bool wrap_around(const std::vector<SweepItem> &items, int n_lists, double T, const std::vector<double> &cost,
                        const std::vector<int> &run_theta, SweepPlan &P)
{
    constexpr double MOVE = 0.3;
    const int n = (int)items.size();
    P.items.clear();
    P.lists.clear();
    double room = T;
    unsigned int first = 0;
    for (int k = 0; k < n; ++k) {
        const int rows = (n + n_lists - 1) / n_lists, full = n - (rows - 1) * n_lists;   // columns with `rows` items
        const int b = k < full * rows ? (k % rows) * n_lists + k / rows
                                      : ((k - full * rows) % (rows - 1)) * n_lists + full + (k - full * rows) / (rows - 1);
        SweepItem it = items[b];
        const int theta = run_theta[it.run];
        it.base = b;
        it.chunk = 0;
        it.nchunk = 1;
        it.cut = 0;
        if (cost[b] * (theta + MOVE) > room) {
            const int end = (int)std::floor(room / cost[b] - MOVE);   // sweeps that still fit here
            if (end >= 1 && end < theta) {
                it.nchunk = 2;
                it.cut = theta - end;
                it.chunk = 1;
                P.items.push_back(it);
                it.chunk = 0;
            }
            P.lists.push_back({first, first, (unsigned int)P.items.size(), {}});
            if ((int)P.lists.size() == n_lists) return false;
            first = (unsigned int)P.items.size();
            room = T;
        }
        P.items.push_back(it);
        room -= cost[b] * ((it.nchunk == 2 ? it.cut : theta) + MOVE);
    }
    while ((int)P.lists.size() < n_lists) {
        P.lists.push_back({first, first, (unsigned int)P.items.size(), {}});
        first = (unsigned int)P.items.size();
    }
    return room >= 0;
}

bool sweep_lists(std::vector<SweepItem> &items, SweepClass &cls, int n_lists, const std::vector<int> &run_theta,
                 const std::vector<int> &run_L, std::vector<SweepList> &lists)
{
    const int n = (int)items.size();
    if (cls.first != 0 || cls.count != n || n_lists < 1 || n <= n_lists) return false;
    std::vector<double> cost(n);
    double T = 0;
    for (int b = 0; b < n; ++b) {
        cost[b] = (double)run_L[items[b].run] * run_L[items[b].run] * items[b].ngroups;
        T += cost[b] * run_theta[items[b].run] / n_lists;
    }
    SweepPlan P;
    for (int k = 0; k < 100; ++k, T *= 1.003) {
        if (!wrap_around(items, n_lists, T, cost, run_theta, P)) continue;
        items.swap(P.items);
        lists.swap(P.lists);
        cls.count = (int)items.size();
        cls.nchunk = 2;
        cls.n_lists = n_lists;
        return true;
    }
    return false;
}

int expand_sweep_chunks(std::vector<SweepItem> &items, SweepClass &cls, int K, const std::vector<int> &run_theta)
{
    cls.nchunk = 1;
    if (K <= 1 || cls.count == 0) return 0;
    if (K > MAX_SWEEP_CHUNKS || cls.first != 0 || cls.count != (int)items.size()) return -1;
    const int n = cls.count;
    std::vector<SweepItem> out((size_t)n * K);
    for (int c = 0; c < K; ++c)
        for (int b = 0; b < n; ++b) {
            SweepItem it = items[b];
            it.chunk = c;
            it.nchunk = K;
            it.base = b;
            it.cut = (run_theta[it.run] + 1) / 2;
            out[(size_t)c * n + b] = it;
        }
    items.swap(out);
    cls.count = n * K;
    cls.nchunk = K;
    return 0;
}

bool sweep_class_grids(SweepClass *cls, int n, int threads, bool persistent)
{
    for (int k = 0; k < n; ++k) {
        cls[k].grid = 0;
        if (!persistent) continue;
        const int resident = sweep_msc_resident(threads, cls[k].lds, cls[k].L, cls[k].ea);
        if (resident <= 0) return false;
        cls[k].grid = resident;
    }
    return true;
}

int sweep_msc_resident(int threads, size_t lds, int L, int ea)
{
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, msc_kernel(L, ea), threads, lds) != hipSuccess)
        return 0;
    return per_cu * device_cus();
}

int device_cus()
{
    int dev = 0, cus = 0;
    return hipGetDevice(&dev) == hipSuccess &&
                   hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess
               ? cus
               : 0;
}

hipError_t launch_dos_sample(const LaunchCtx &c)
{
    if (!c.any_exact_dos || c.n_items == 0) return hipSuccess;
    k_dos_sample<<<(c.n_items + 3) / 4, 256, 0, c.stream>>>(c.items, c.n_items, c.runs, c.st);
    return hipGetLastError();
}

hipError_t launch_measure(const LaunchCtx &c, bool first)
{
    if (c.any_wang && c.n_runs > 0) {
        if (c.wang_lds) {
            k_wang_lds<<<c.n_runs, WANG_THREADS, c.wang_lds, c.stream>>>(c.runs, c.st, c.run0, (uint32_t)c.wang_lds);
            PA_CHECK_LAUNCH();
        }
        if (c.wang_large) {
            k_wang_pairs<<<c.n_runs, WANG_THREADS, 0, c.stream>>>(c.runs, c.st, c.run0, (uint32_t)c.wang_lds);
            PA_CHECK_LAUNCH();
        }
        const int blocks = (c.n_items + 3) / 4;
        if (c.repr == PA_INT8)
            k_wang_rows<PA_INT8><<<blocks, 256, 0, c.stream>>>(c.items, c.n_items, c.runs, c.st);
        else
            k_wang_rows<PA_MSC64><<<blocks, 256, 0, c.stream>>>(c.items, c.n_items, c.runs, c.st);
        PA_CHECK_LAUNCH();
        k_wang_gather<<<blocks, 256, 0, c.stream>>>(c.items, c.n_items, c.runs, c.st);
        PA_CHECK_LAUNCH();
    }
    if (c.n_meas_items > 0) {
        // the variant without overlap counters when no run measures overlaps
        // (fewer registers live in the site loop); in the int8 layout the
        // swept runs are measured from their words, the others from bytes
        const bool words = c.repr == PA_MSC64 || (!first && c.any_swept);
        const bool bytes = c.repr == PA_INT8 && (first || c.any_unswept);
        // With overlaps four times the wavefronts per group where a wavefront
        // per SIMD would be left over (us, L = 128, R = 2000 97 / 41; L = 20,
        // R = 5003 18.7 / 14.9; L = 16, R = 2000 13.1 / 10.5).  Without, the
        // larger workgroups' start costs more (L = 8, R = 1000 7.3 / 10.8;
        // L = 16, R = 2e4 8.7 / 12.4), and on bytes they spill registers.
        constexpr int W = MEAS_WAVES;
        const bool few = c.n_meas_items * W <= 1024;
        if (words && c.any_overlap && few)
            k_measure<PA_MSC64, true, 4 * W><<<c.n_meas_items, 256 * W, 0, c.stream>>>(c.meas_items, c.runs, c.st);
        else if (words && c.any_overlap)
            k_measure<PA_MSC64, true, W><<<c.n_meas_items, 64 * W, 0, c.stream>>>(c.meas_items, c.runs, c.st);
        else if (words)
            k_measure<PA_MSC64, false, W><<<c.n_meas_items, 64 * W, 0, c.stream>>>(c.meas_items, c.runs, c.st);
        PA_CHECK_LAUNCH();
        if (bytes && c.any_overlap)
            k_measure<PA_INT8, true, W><<<c.n_meas_items, 64 * W, MEAS_STAGE_BYTES, c.stream>>>(c.meas_items, c.runs, c.st);
        else if (bytes)
            k_measure<PA_INT8, false, W><<<c.n_meas_items, 64 * W, MEAS_STAGE_BYTES, c.stream>>>(c.meas_items, c.runs, c.st);
        PA_CHECK_LAUNCH();
    }
    k_meas_chunk<<<c.n_chunk_items, CH_THREADS, 0, c.stream>>>(c.chunk_items, c.runs, c.st);
    return hipGetLastError();
}

// A wavefront per (group, temperature) from this many runs a group (whole
// calls, thread / wavefront: 16 groups of 16, 89 temperatures 172 / 121 us; 240
// of 16, 61 temperatures 269 / 241; one of 16 92 / 48).
constexpr int WIDE_GROUP = 16;
static int group_blocks(int n, int M)
{
    const int per = M >= WIDE_GROUP ? GROUP_THREADS / 64 : GROUP_THREADS;
    return (n + per - 1) / per;
}

hipError_t launch_qweights(const LaunchCtx &c, const pa_obs *obs, int M, int kind, int pop, int K, int i_done,
                           double *logw, double *qw)
{
    k_logw<<<c.n_runs, SCAN_THREADS, 0, c.stream>>>(c.runs, obs, c.n_runs, c.npop_ctx, pop, kind, i_done, logw);
    PA_CHECK_LAUNCH();
    const int ng = c.n_runs / M;
    auto kernel = M >= WIDE_GROUP ? k_qweights<64> : k_qweights<1>;
    kernel<<<group_blocks(ng * K, M), GROUP_THREADS, 0, c.stream>>>(c.runs, obs, logw, c.n_runs, c.npop_ctx, pop, M,
                                                                    K, kind & ~1, qw);
    return hipGetLastError();
}

hipError_t launch_wqhist(const LaunchCtx &c, const pa_obs *obs, int M, int kind, int pop, int K, int i_done,
                         double *logw, double *qw, double *out)
{
    if (launch_qweights(c, obs, M, kind, pop, K, i_done, logw, qw) != hipSuccess) return hipGetLastError();
    const int ng = c.n_runs / M;
    k_wqhist<<<ng * K, 256, 0, c.stream>>>(c.runs, obs, qw, c.n_runs, c.npop_ctx, pop, M, K, out);
    return hipGetLastError();
}

hipError_t launch_famstats(const LaunchCtx &c, const pa_obs *obs, int pop, int K, int i_done, pa_famstat *out)
{
    k_famstats<<<(c.n_runs * K + 255) / 256, 256, 0, c.stream>>>(c.runs, obs, c.n_runs, c.npop_ctx, pop, K,
                                                                 i_done, out);
    return hipGetLastError();
}

hipError_t launch_wavg(const LaunchCtx &c, const pa_obs *obs, int M, int kind, int pop, int K,
                       int i_done, double *logw, double *qw, pa_wavg *out)
{
    if (launch_qweights(c, obs, M, kind, pop, K, i_done, logw, qw) != hipSuccess) return hipGetLastError();
    const int ng = c.n_runs / M;
    auto kernel = M >= WIDE_GROUP ? k_wavg<64> : k_wavg<1>;
    kernel<<<group_blocks(ng * K, M), GROUP_THREADS, 0, c.stream>>>(c.runs, obs, logw, qw, c.n_runs, c.npop_ctx, pop,
                                                                    M, K, out);
    PA_CHECK_LAUNCH();
    k_wavg_cumsum<<<ng, SCAN_THREADS, 0, c.stream>>>(out, ng, K);
    return hipGetLastError();
}

}  // namespace pa
