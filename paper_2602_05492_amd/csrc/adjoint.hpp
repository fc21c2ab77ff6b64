// adjoint.hpp - per-pair pieces shared by the float64 adjoint (vjp.hip) and the mixed one (vjp_mixed.hip).
#pragma once

#include "common.hpp"
#include "cells.hpp"

namespace bem {

constexpr int kV = kSegVjpVals;   // 16 sums per segment
constexpr int kNearCopies = 16;   // partial rows the near pairs of the mixed adjoint add into

template <class T>
__device__ inline void add_pair(T* acc, const Grad4<T>& gr, const Moments<T>& m, T g0, T g1, T g2)
{
    acc[0] += gr.ax; acc[1] += gr.ay; acc[2] += gr.bx; acc[3] += gr.by;
    acc[4] += m.da * g0; acc[5] += m.da * g1; acc[6] += m.da * g2;
    acc[7] += m.db * g0; acc[8] += m.db * g1; acc[9] += m.db * g2;
    acc[10] += m.sa * g0; acc[11] += m.sa * g1; acc[12] += m.sa * g2;
    acc[13] += m.sb * g0; acc[14] += m.sb * g1; acc[15] += m.sb * g2;
}

// Float64 adjoint of one near (sample, segment) pair: the 16 per-segment sums of the pair in a[].
__device__ inline void near_segment_values(const double* __restrict__ s, double X, double Y, double g0, double g1,
                                           double g2, double eps2, double* __restrict__ a)
{
    for (int v = 0; v < kV; ++v) a[v] = 0.0;
    const SegGeom<double> g = load_geom(s);
    if (g.L2 == 0.0) return;
    const double wa = g0 * s[kWdA] + g1 * s[kWdA + 1] + g2 * s[kWdA + 2];
    const double wb = g0 * s[kWdB] + g1 * s[kWdB + 1] + g2 * s[kWdB + 2];
    const double sa = g0 * s[kWcA] + g1 * s[kWcA + 1] + g2 * s[kWcA + 2];
    const double sb = g0 * s[kWcB] + g1 * s[kWcB + 1] + g2 * s[kWcB + 2];
    const PairState<double> st = pair_forward<double, DevF64, true>(g, X, Y, eps2);
    add_pair(a, pair_backward(g, st, eps2, wa, wb, sa, sb), pair_moments(g, st), g0, g1, g2);
}

// vjp_mixed.hip
Grouping adj_mixed_rows(bem_ctx* ctx, int K, int64_t N, int* seg_rows, int* el_rows);
int adj_mixed(bem_ctx* ctx, const double* x, int64_t N, const float* gbar, int K, Grouping g, int seg_rows, int el_rows,
              double* part, double* epart, hipStream_t s);

}  // namespace bem
