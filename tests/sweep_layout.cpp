// LDS addresses of the kernels, from the headers they are built from, for
// test_sweep_layout.py.
#include <algorithm>
#include <vector>

#include "pa_internal.hpp"
#include "unit_walk.hpp"

using namespace pa;

// Walks every wavefront of `threads` over `groups` lattices of side L as the
// sweep does.  out[0], out[1]: the smallest and the largest lattice word that
// a lane flips; out[2], out[3]: the same for the
// neighbours it reads; out[4]: how often the units are visited twice or not
// at all; out[5]: lanes without a unit.
extern "C" void sweep_walk(int L, int threads, int groups, int64_t *out)
{
    const LatticeShape J = {L, L * L, L / 2, L * L / 2};
    const int units = groups * J.nh, upw = msc_units_per_wave(units, threads / 64);
    const int gq = 64 / J.nh, kr = 64 - gq * J.nh, yr = kr / J.half, mr = kr - yr * J.half;
    out[0] = out[2] = INT32_MAX;
    out[1] = out[3] = INT32_MIN;
    out[4] = out[5] = 0;
    for (int colour = 0; colour < 2; ++colour) {
        std::vector<int> seen((size_t)groups * J.N, 0);
        for (int wave = 0; wave < threads / 64; ++wave)
            for (int lane = 0; lane < 64; ++lane) {
                const int ub = std::min(units, wave * upw), ue = std::min(units, ub + upw);
                UnitWalk w;
                w.start(J, std::min(ub, units - 1) + lane);
                for (int u0 = ub; u0 < ue; u0 += 64) {
                    const bool in = u0 + lane < ue;
                    const int own = w.word(J, colour), o = own + (colour ? -J.nh : J.nh);
                    at_unit(in, own, [&](int word) {
                        out[0] = std::min<int64_t>(out[0], word);
                        out[1] = std::max<int64_t>(out[1], word);
                        if (word >= 0 && word < groups * J.N) ++seen[word];
                    });
                    out[5] += in ? 0 : 1;
                    if (in) {
                        for (int d : {0, w.dh(J, (w.y + colour) & 1), w.du(J), w.dd(J)}) {
                            out[2] = std::min<int64_t>(out[2], o + d);
                            out[3] = std::max<int64_t>(out[3], o + d);
                        }
                    }
                    w.step(J, gq, kr, yr, mr);
                }
            }
        for (int g = 0; g < groups; ++g)
            for (int k = 0; k < J.nh; ++k) out[4] += seen[(size_t)g * J.N + colour * J.nh + k] != 1;
    }
}

extern "C" int64_t sweep_lds(int L, int threads, int groups, int ea)
{
    return (int64_t)msc_stream_lds(L * L, groups, ea != 0, threads / 64);
}

// The pairing repair's candidates for a population of Rc: how many are not the
// position they stand for, or (past the search's end) no position at all.
extern "C" int64_t wrong_candidates(int Rc)
{
    int64_t wrong = 0;
    for (int hi = 1; hi <= Rc; ++hi)
        for (int u = hi; u < hi + Rc; ++u)
            for (int lane = 0; lane < 64; ++lane) {
                const int m = wang_candidate(u + lane, Rc);
                wrong += m < 0 || m >= Rc || (u + lane < hi + Rc && m != (u + lane) % Rc);
            }
    return wrong;
}

// Layout of the one-workgroup resampling: the end of the coarse prefix, the
// start of the fine one, its end, and the LDS asked for.
extern "C" void fused_layout(int R_cap, int64_t *out)
{
    const int n8 = (R_cap + CH_PER - 1) / CH_PER;
    out[0] = (int64_t)n8 * (2 * CH_PER + 8);
    out[1] = (int64_t)fused_fine_at(n8);
    out[2] = out[1] + (int64_t)n8 * 4 * CH_PER;
    out[3] = (int64_t)fused_lds(R_cap, true);
}

extern "C" int fused_max() { return FUSED_MAX; }

extern "C" int64_t pairing_lds(int R_cap) { return (int64_t)wang_lds_bytes(R_cap); }
