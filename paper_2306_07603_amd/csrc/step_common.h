// step_common.h -- difference stencils and residual sums shared by the kernels
// of the fused schedule (step_fused.hip, step_tile.hip, step_block.hip), so that all store
// the same bits.
#pragma once

#include <type_traits>

#include "ifdlbm_internal.h"

namespace ifd {
namespace {

// Weights of Eq. (2.5) times sign(c) * 2h on the upwind-sorted points a2
// (two behind), a1 (one behind), c0 and f1 (one ahead):
// sign(c) * central = f1 - a1 (Eq. 2.6), sign(c) * upwind = 3 c0 - 4 a1 + a2
// (Eq. 2.7), so eps * central + (1 - eps) * upwind is
// eps f1 - (4 - 3 eps) a1 + 3 (1 - eps) c0 + (1 - eps) a2.
template <typename T>
struct MixedWeights {
    T wf, wa1, wc, wa2;
    __device__ __forceinline__ MixedWeights(T eps, T scale)
        : wf(scale * eps), wa1(-scale * (T(4) - T(3) * eps)), wc(scale * T(3) * (T(1) - eps)),
          wa2(scale * (T(1) - eps))
    {
    }
    __device__ __forceinline__ T apply(T a2, T a1, T c0, T f1) const { return ((wc * c0 + wa1 * a1) + wa2 * a2) + wf * f1; }
    // The same on differences, which FP32 arithmetic needs: neighbouring
    // values agree to many digits, so the weighted sum of the values above
    // loses to cancellation what differences keep (an error of order one ulp
    // of f per step that does not average out over a steady run).  With the
    // backward differences B(m) = x(m) - x(m - 1) along the upwind direction,
    // n = B at the point (c0 - a1), f = B one further upwind (a1 - a2) and
    // o = B one downwind (f1 - a1 = n + o), it is
    // (eps + 3 (1 - eps)) n - (1 - eps) f + eps o.
    __device__ __forceinline__ T apply_back(T n, T f, T o) const { return ((wc + wf) * n - wa2 * f) + wf * o; }
    // r minus the same, as three multiply-adds into r
    __device__ __forceinline__ T sub_back(T r, T n, T f, T o) const
    {
        return __builtin_fmaf(-(wc + wf), n, __builtin_fmaf(wa2, f, __builtin_fmaf(-wf, o, r)));
    }
};

// Mixed differences from differences first where the distributions are FP32.
template <typename T> constexpr bool kDiffForm = sizeof(T) == 4;

// r minus w times the mixed xi difference of a node from its upwind-sorted
// points; at a wall-adjacent column (edge) the second upwind point is replaced
// by the first-order form of Eq. (2.7).
template <typename T>
__device__ __forceinline__ T xi_term(T r, T w, const MixedWeights<T>& m, T a2, T a1, T c0, T f1, bool edge)
{
    if constexpr (kDiffForm<T>) {
        const T n = c0 - a1;
        const T t = m.apply_back(n, edge ? n : a1 - a2, f1 - c0);
        return r - w * t;
    } else {
        a2 = edge ? T(2) * a1 - c0 : a2;
        return r - w * m.apply(a2, a1, c0, f1);
    }
}

// The eta counterpart (unit weight).
template <typename T>
__device__ __forceinline__ T eta_term(T r, const MixedWeights<T>& m, T b2, T b1, T c0, T h1, bool edge)
{
    if constexpr (kDiffForm<T>) {
        const T n = c0 - b1;
        return m.sub_back(r, n, edge ? n : b1 - b2, h1 - c0);
    } else {
        b2 = edge ? T(2) * b1 - c0 : b2;
        return r - m.apply(b2, b1, c0, h1);
    }
}

// Element of a plane at a 32-bit byte offset from a uniform base.
template <typename X> __device__ __forceinline__ X& plane_at(X* base, uint32_t id)
{
    using C = std::conditional_t<std::is_const<X>::value, const char, char>;
    return *reinterpret_cast<X*>(reinterpret_cast<C*>(base) + id * (uint32_t)sizeof(X));
}

// Eq. (2.19) sums of one node (the layout of kPartials); ref holds the
// cavity's shifts r_d, r_p.
template <typename T>
__device__ __forceinline__ void residual_add(const T (&gn)[9], const T (&old)[3], const double (&ref)[2],
                                             double (&acc)[kPartials])
{
    T P, ux, uy;
    moments(gn, P, ux, uy);
    const double du = (double)ux - (double)old[1], dv = (double)uy - (double)old[2], dp = (double)P - (double)old[0];
    const double sd = dp - ref[0], sp = (double)P - ref[1];
    acc[0] = fused(du, du, fused(dv, dv, acc[0]));
    acc[1] = fused((double)ux, (double)ux, fused((double)uy, (double)uy, acc[1]));
    acc[2] = fused(dp, dp, acc[2]);
    acc[3] = fused((double)P, (double)P, acc[3]);
    acc[4] += sd;
    acc[5] += sp;
    acc[6] += (isfinite((double)ux) && isfinite((double)uy) && isfinite((double)P)) ? 0.0 : 1.0;
    acc[7] = fused(sd, sd, acc[7]);
    acc[8] = fused(sp, sp, acc[8]);
}

// Sums of the residual terms over the wavefront, in a fixed order: lane q < kPartials returns sum q.  Eight of the nine
// are halved between the lanes at each of the first three exchanges: 16 exchanges in all instead of 54.
__device__ __forceinline__ double wave_sums(const double (&acc)[kPartials])
{
    const int lane = (int)__lane_id();
    double v[8] = {acc[0], acc[1], acc[2], acc[3], acc[4], acc[5], acc[7], acc[8]}, n = acc[6];
    // after the exchange with lane ^ m, lanes with that bit set hold the upper half of the values
    auto halve = [&](int m, int h) {
        const bool up = lane & m;
#pragma unroll
        for (int q = 0; q < h; ++q) {
            const double keep = up ? v[q + h] : v[q], give = up ? v[q] : v[q + h];
            v[q] = keep + __shfl_xor(give, m, kWaveLanes);
        }
    };
    halve(32, 4);
    halve(16, 2);
    halve(8, 1);
#pragma unroll
    for (int m = 4; m > 0; m >>= 1) v[0] += __shfl_xor(v[0], m, kWaveLanes);
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) n += __shfl_xor(n, m, kWaveLanes);
    // value q is in the lanes whose bits 5, 4, 3 spell it (bit 5 the highest); bring it to its lane
    const int q = lane > 6 ? lane - 1 : lane;
    const double r = __shfl(v[0], (q & 7) << 3, kWaveLanes);
    return lane == 6 ? n : r;
}

}  // namespace
}  // namespace ifd
