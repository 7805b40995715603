// Likelihood-ratio scores of the gradient walks, device side.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "photonmc.h"
#include "walk.hpp"

namespace pmc {

// Likelihood-ratio (perturbation Monte Carlo) scores of the track-length
// estimator.  The sampled path density is mu_s^k exp(-mu_t l_solid) prod p_HG;
// its log-derivatives give the scores S_mus = k/mu_s - l_solid,
// S_mua = -l_solid and S_g = sum_i d ln p_HG(cos_i)/dg.  A segment of length d
// starting with those scores adds w (S d - [solid] d^2/2) to the mu_s and mu_a
// bins (the d^2/2 is the survival inside the segment) and w S_g d to the g bin,
// per (parameter, phase, depth), in fixed point 2^-MC_GRAD_FIXED_BITS of a Q31
// weight x voxel, each segment's value rounded to nearest.  Roulette decisions
// carry no score: survival 1/m with weight x m is unbiased.
constexpr double kGradScale = 1.0 / (double)(1ll << MC_GRAD_FIXED_BITS);

// The block keeps its score bins in LDS as int32 words (half the space of int64
// bins: four 256-thread walk workgroups still fit per CU at nz = 256) and moves a
// word to the global (hi, lo) int64 pairs before it can overflow.  A value of
// magnitude >= kGradDirect goes to the global pair directly; any other is added
// to its word, and a lane whose add leaves the word at magnitude >= kGradSpill
// swaps the word for 0 and adds what it took to the global pair.  A lane that
// sees the threshold swaps before its next add, so at most one add per thread of
// the block lands on a word between its crossing and the swap: |word| < kGradSpill
// + 512 * kGradDirect = 2^28 + 2^30.  Every transfer is exact, so the totals are
// the integer sums of the segments' fixed-point values whatever the order.  The
// global pairs are few (6 nz, a hot address each), so the direct path must stay
// rare: at 2^-20 a value reaches 2^21 only where (w / 2^31) |S| d reaches 1024
// voxels, while under implicit capture (w / 2^31) l_solid peaks at 1 / (e mu_a),
// 37 voxels at mu_a = 0.01.
constexpr long long kGradDirect = 1ll << 21;
constexpr int kGradSpill = 1 << 28;

__device__ __forceinline__ void grad_global_add(unsigned long long *grad, int32_t i, long long v)
{
    atomicAdd(&grad[2 * i], (unsigned long long)(v >> 32));
    atomicAdd(&grad[2 * i + 1], (unsigned long long)v & 0xFFFFFFFFull);
}

__device__ __forceinline__ void grad_bin_add(int *bins, unsigned long long *grad, int32_t i, long long v)
{
    if (v == 0) return;
    if (v >= kGradDirect || v <= -kGradDirect) {
        grad_global_add(grad, i, v);
        return;
    }
    const long long nv = (long long)atomicAdd(&bins[i], (int)v) + v;
    if (nv >= kGradSpill || nv <= -kGradSpill) grad_global_add(grad, i, (long long)atomicExch(&bins[i], 0));
}

__device__ __forceinline__ double hg_score(double ct, double g)
{
    return -2.0 * g / (1.0 - g * g) + 3.0 * (ct - g) / (1.0 + g * g - 2.0 * g * ct);
}

// The three score values of a segment of length dd that starts with photon p's scores.
template <class P>
__device__ __forceinline__ void grad_values(const P &p, double inv_mu_s, double dd, bool solid, long long &vs,
                                            long long &va, long long &vg)
{
    const double ls = p.l_tot - p.l_void;                  // solid path before this segment
    const double sq = solid ? 0.5 * dd * dd : 0.0;
    const double sw = (double)p.w * kGradScale;
    vs = __double2ll_rn(sw * (((double)p.k * inv_mu_s - ls) * dd - sq));
    va = __double2ll_rn(sw * (-ls * dd - sq));
    vg = __double2ll_rn(sw * (p.score_g * dd));
}

}  // namespace pmc
