// jtj.hip - Monte Carlo normal equations (Eq. losshessian, Eq. lossjacobian)
// with the Jacobian of the differential BIE (Eq. diffbie, Sec. 3.2):
//
//   J_c(x) = df_c/dtheta(x) + sum_i beta_i(x) Z_c[i, :],   Z = A+ dF/dtheta.
//
// Per sample x and channel c the augmented row a_c(x) = [g_c(x) | e(x) | beta(x)]
// holds the G*H geometry derivatives of f_c, the C*H channel-independent colour
// coefficients and the M outer-element weights, so that J_c(x) = a_c(x) S_c with
// S_c = [E_c ; Z_c'] (E_c a column selection).  Cubic handles: G = 8 (control
// points), C = 4 (wd and wc at both ends); straight handles: G = 4 (end points),
// C = 2 (the constant wd and wc).
// Sample tiles of feature rows Xt = [g_1 | g_2 | g_3 | e | beta] (feature-major,
// W = (3G + C)H + M rows) are formed by the feature kernels and contracted into the
// Gram G = sum_x Xt Xt^T (only the blocks the three channels need).  Afterwards, per channel,
//   J^T J += E_c^T A_c E_c + sym(E_c^T B_c Z_c') + Z_c'^T D Z_c'
// with A_c, B_c, D the channel's blocks of G.  J^T r is the adjoint's (vjp.hip).
#include <algorithm>
#include <cstring>
#include <tuple>
#include <type_traits>
#include <vector>

#include "normal.hpp"

namespace bem {

namespace {

constexpr double kGaussNode = 0.77459666924148337703585307995647992;
constexpr double kGaussW0 = 5.0 / 9.0, kGaussW1 = 8.0 / 9.0;

// ---- output element types of the feature kernels ------------------------------
// Feature element (f, t) of a tile.  float64 / float32 tiles are row-major with
// row stride ld; the split-bfloat16 tile is stored in blocks of 32 samples,
// [t / 32][f][t % 32] with ld = the number of rows, so that one 32-sample stage
// of consecutive rows is one contiguous run of memory for the Gram kernel.
template <class OutT> struct Store;
template <> struct Store<double> {
    __device__ static void put(double* hi, uint16_t*, int64_t f, int64_t t, int64_t ld, double v) { hi[f * ld + t] = v; }
};
template <> struct Store<float> {
    __device__ static void put(float* hi, uint16_t*, int64_t f, int64_t t, int64_t ld, double v)
    {
        hi[f * ld + t] = (float)v;
    }
};
// hi + lo bfloat16 split of the float value
template <> struct Store<uint16_t> {
    __device__ static void put(uint16_t* hi, uint16_t* lo, int64_t f, int64_t t, int64_t ld, double v)
    {
        const size_t i = (size_t)(t >> 5) * (size_t)(ld << 5) + (size_t)(f << 5) + (size_t)(t & 31);
        const float x = (float)v;
        const uint16_t h = bf16_bits(x);
        hi[i] = h;
        lo[i] = bf16_bits(x - bf16_value(h));
    }
};

// Feature rows of one (point, handle): the chained gradients geo[c][q] on the four weights of
// vertex_weights and the coefficients col[m] of wd0, wd1, wc0, wc1 (jumps at t = 0 and t = 1).
// Channel c's geometry rows start at c * gp, gp = G H rounded up to a multiple of 256 (the
// Gram's tile), so that no Gram tile mixes two channels; the colour rows start at 3 gp.
// Cubic handles (model 0, G = 8): rows c gp + 8h + q and 3 gp + 4h + m.  Straight handles
// (model 1, G = 4): the end-point gradients are geo[c][0..3], rows c gp + 4h + q, and the
// constant jumps take the sum of their two end coefficients, rows 3 gp + 2h + {0: wd, 1: wc}.
template <class OutT, class A>
__device__ inline void store_handle_rows(int model, OutT* Xt, uint16_t* Xlo, int H, int h, int64_t t, int64_t ld,
                                         int64_t gp, const A (&geo)[3][8], const A (&col)[4])
{
    if (model == 1) {
        for (int c = 0; c < 3; ++c)
            for (int q = 0; q < 4; ++q)
                Store<OutT>::put(Xt, Xlo, (int64_t)c * gp + 4 * h + q, t, ld, (double)geo[c][q]);
        Store<OutT>::put(Xt, Xlo, 3 * gp + 2 * h, t, ld, (double)col[0] + (double)col[1]);
        Store<OutT>::put(Xt, Xlo, 3 * gp + 2 * h + 1, t, ld, (double)col[2] + (double)col[3]);
        return;
    }
    for (int c = 0; c < 3; ++c)
        for (int q = 0; q < 8; ++q)
            Store<OutT>::put(Xt, Xlo, (int64_t)c * gp + 8 * h + q, t, ld, (double)geo[c][q]);
    for (int q = 0; q < 4; ++q) Store<OutT>::put(Xt, Xlo, 3 * gp + 4 * h + q, t, ld, (double)col[q]);
}

// Padding rows [c gp + G H, (c + 1) gp) of the three geometry blocks are zero in every tile.
template <class OutT>
__global__ void k_zero_pad(OutT* __restrict__ Xt, uint16_t* __restrict__ Xlo, int64_t ld, int64_t gp, int64_t gh,
                           int64_t npts)
{
    const int64_t pad = gp - gh;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= 3 * pad * npts) return;
    const int64_t r = i / npts, t = i % npts;
    Store<OutT>::put(Xt, Xlo, (r / pad) * gp + gh + r % pad, t, ld, 0.0);
}

// Handle features of one point and one handle (thread per (point, handle)):
//   rows c*8H + 8h + 2j + d : d f_c / d P_{h,j,d}      (c = 0..2, j = 0..3, d = x, y)
//   rows 24H + 4h + m       : coefficient of wd0, wd1, wc0, wc1 of handle h (any channel)
// The vertex gradient of the polyline is chained to control points with the
// Bernstein weights of the vertex parameter t_k = k/S (straight handles: to the end
// points with 1 - t_k, t_k; rows as store_handle_rows).
//
// Float64 (Mixed = false), or mixed with near pairs inline in float64: the latter
// runs only for the samples flagged in `only` (their near-pair list overflowed).
//
// Split = 4 (float64): a block takes 64 points, wavefront w the w-th quarter of the handle's segments, summed
// in LDS; for few points and handles, whose blocks of 256 points leave most of the chip idle (4 handles x 32 segments
// and 16,384 points: 256 blocks, 52 us; 1,024, 32 us).
template <bool Mixed, class OutT, int Split = 1>
__global__ void __launch_bounds__(256) k_features(const double* __restrict__ x, int64_t npts,
                                                  const double* __restrict__ seg64, const float* __restrict__ seg32,
                                                  int H, int S, int model, int64_t gp, double eps2, float eps2f,
                                                  float near2, const uint8_t* __restrict__ only,
                                                  OutT* __restrict__ Xt, uint16_t* __restrict__ Xlo, int64_t ld)
{
    using A = typename std::conditional<Mixed, float, double>::type;
    const int h = blockIdx.y;
    // all points: one per thread; only the flagged ones (only != null): a few blocks stride
    // over the tile, so that a tile with few or no flagged samples costs a small launch
    const int64_t stride = only ? (int64_t)gridDim.x * blockDim.x : npts;
    const int part = Split > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0;
    const int j0 = S * part / Split, j1 = S * (part + 1) / Split;
    const int64_t first = Split > 1 ? (int64_t)blockIdx.x * 64 + (threadIdx.x & 63)
                                    : (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int64_t t = first; t < npts || Split > 1; t += stride) {
        if (only && !only[t]) continue;
        const int64_t tl = t < npts ? t : npts - 1;
        const double X = x[2 * tl], Y = x[2 * tl + 1];
        const float Xf = (float)X, Yf = (float)Y;
        A geo[3][8];
        A col[4];
        A pv[3][2];   // gradient carried to the next vertex (from the previous segment's b end)
        for (int c = 0; c < 3; ++c) {
            for (int q = 0; q < 8; ++q) geo[c][q] = A(0);
            pv[c][0] = pv[c][1] = A(0);
        }
        for (int q = 0; q < 4; ++q) col[q] = A(0);
        double tb = (double)j0 / (double)S;
        for (int j = j0; j <= j1; ++j) {
            // contributions to vertex j: a end of segment j (if j < j1) + b end of segment j-1 (carried)
            const double ta = tb;
            tb = (double)(j + 1) / (double)S;
            A va[3][2] = {{A(0), A(0)}, {A(0), A(0)}, {A(0), A(0)}};
            A vb[3][2] = {{A(0), A(0)}, {A(0), A(0)}, {A(0), A(0)}};
            if (j < j1) {
                const int k = h * S + j;
                const double* s64 = seg64 + (size_t)k * kSegStride;
                Moments<A> m{A(0), A(0), A(0), A(0)};
                bool done = false;
                if (s64[6] == 0.0) done = true;                  // degenerate segment: nothing
                if (!done && Mixed) {
                    const float* s32 = seg32 + (size_t)k * kSegStride;
                    const SegGeom<float> gf = load_geom(s32);
                    if (!near_segment(gf.ax, gf.ay, gf.bx, gf.by, gf.L2, Xf, Yf, near2)) {
                        const PairState<float> st = pair_forward<float, DevF32, false>(gf, Xf, Yf, eps2f);
                        const Moments<float> mf = pair_moments(gf, st);
                        m = Moments<A>{(A)mf.da, (A)mf.db, (A)mf.sa, (A)mf.sb};
                        for (int c = 0; c < 3; ++c) {
                            const Grad4<float> gr = pair_backward(gf, st, eps2f, s32[kWdA + c], s32[kWdB + c],
                                                                  s32[kWcA + c], s32[kWcB + c]);
                            va[c][0] = gr.ax; va[c][1] = gr.ay; vb[c][0] = gr.bx; vb[c][1] = gr.by;
                        }
                        done = true;
                    }
                }
                if (!done) {
                    const SegGeom<double> g = load_geom(s64);
                    const PairState<double> st = pair_forward<double, DevF64, true>(g, X, Y, eps2);
                    const Moments<double> md = pair_moments(g, st);
                    m = Moments<A>{(A)md.da, (A)md.db, (A)md.sa, (A)md.sb};
                    // the end-point gradient is linear in the channel's end densities: one matrix per pair serves
                    // the three channels
                    const GradMatrix<double> G = pair_grad_matrix(g, st, eps2);
                    for (int c = 0; c < 3; ++c) {
                        const Grad4<double> gr = grad_apply(G, s64[kWdA + c], s64[kWdB + c], s64[kWcA + c], s64[kWcB + c]);
                        va[c][0] = (A)gr.ax; va[c][1] = (A)gr.ay; vb[c][0] = (A)gr.bx; vb[c][1] = (A)gr.by;
                    }
                }
                col[0] += m.da * (A)(1.0 - ta) + m.db * (A)(1.0 - tb);
                col[1] += m.da * (A)ta + m.db * (A)tb;
                col[2] += m.sa * (A)(1.0 - ta) + m.sb * (A)(1.0 - tb);
                col[3] += m.sa * (A)ta + m.sb * (A)tb;
            }
            double B[4];
            vertex_weights(model, ta, B);
            for (int c = 0; c < 3; ++c) {
                const A gx = va[c][0] + pv[c][0], gy = va[c][1] + pv[c][1];
                for (int q = 0; q < 4; ++q) {
                    geo[c][2 * q] += (A)B[q] * gx;
                    geo[c][2 * q + 1] += (A)B[q] * gy;
                }
                pv[c][0] = vb[c][0];
                pv[c][1] = vb[c][1];
            }
        }
        if constexpr (Split > 1) {
            __shared__ A red[Split - 1][28][64];
            const int lane = threadIdx.x & 63;
            if (part > 0) {
                for (int c = 0; c < 3; ++c)
                    for (int q = 0; q < 8; ++q) red[part - 1][8 * c + q][lane] = geo[c][q];
                for (int q = 0; q < 4; ++q) red[part - 1][24 + q][lane] = col[q];
            }
            __syncthreads();
            if (part > 0 || t >= npts) return;
            for (int p = 0; p < Split - 1; ++p) {
                for (int c = 0; c < 3; ++c)
                    for (int q = 0; q < 8; ++q) geo[c][q] += red[p][8 * c + q][lane];
                for (int q = 0; q < 4; ++q) col[q] += red[p][24 + q][lane];
            }
        }
        store_handle_rows(model, Xt, Xlo, H, h, t, ld, gp, geo, col);
        if (Split > 1) return;
    }
}

// One (sample, segment) pair of the mixed feature kernel by the closed forms: its moments and end-point
// gradients, chained into col and geo (V: the vertex table at the segment's a end); nothing where !on.
__device__ __forceinline__ void closed_pair_features(const float* __restrict__ s32, const float* __restrict__ V, float X,
                                                     float Y, float eps2f, bool on, float (&geo)[3][8], float (&col)[4])
{
    const SegGeom<float> g = load_geom(s32);
    const PairState<float> st = pair_forward<float, DevF32, false>(g, X, Y, eps2f);
    const Moments<float> m = pair_moments(g, st);
    // the end-point gradient is linear in the channel's end densities: one matrix per pair serves
    // the three channels
    const GradMatrix<float> G = pair_grad_matrix(g, st, eps2f);
    col[0] += on ? m.da * V[5] + m.db * V[13] : 0.f;
    col[1] += on ? m.da * V[4] + m.db * V[12] : 0.f;
    col[2] += on ? m.sa * V[5] + m.sb * V[13] : 0.f;
    col[3] += on ? m.sa * V[4] + m.sb * V[12] : 0.f;
    for (int c = 0; c < 3; ++c) {
        const Grad4<float> gr = grad_apply(G, s32[kWdA + c], s32[kWdB + c], s32[kWcA + c], s32[kWcB + c]);
        for (int q = 0; q < 4; ++q) {
            geo[c][2 * q] += on ? V[q] * gr.ax + V[8 + q] * gr.bx : 0.f;
            geo[c][2 * q + 1] += on ? V[q] * gr.ay + V[8 + q] * gr.by : 0.f;
        }
    }
}

constexpr int kFeatVals = 28;   // chained contributions of one pair: geo[3][8] and col[4]

// Mixed handle features: float32 pairs, near pairs skipped (same predicate as the
// classification), then the float64 contributions of this sample's listed near pairs
// with this handle's segments are added.  runs (k_near_runs) gives the range of the
// handle's entries in the wavefront's slice; the wavefront walks it with uniform
// (scalar) loads and each lane takes the entries of its own sample.  x points at the
// tile's first sample, whose global index is t0 (a multiple of 64); flagged samples
// are rewritten afterwards by k_features<true>.  The float32 pairs go by quadrature: cheaper than the closed
// forms and their gradients, and without their cancellation at a distance, which beside a gradient from the
// adjoint cost the full-size LM step (FP32 Gram) 8.6e-3 against 7.7e-4.  Band (near radius below two lengths): pairs
// with both end points within two lengths keep the closed forms.
template <bool Band, class OutT>
__global__ void __launch_bounds__(256, Band ? 4 : 6) k_features_far(const double* __restrict__ x, int64_t npts, int64_t t0,
                                                      const float* __restrict__ seg32, int H, int S, int model,
                                                      int64_t gp, float eps2f,
                                                      float near2, const NearPair* __restrict__ list, int slots,
                                                      const int2* __restrict__ runs,
                                                      const uint8_t* __restrict__ flag, const float* __restrict__ corr,
                                                      const float* __restrict__ vtab, const float4* __restrict__ box,
                                                      OutT* __restrict__ Xt, uint16_t* __restrict__ Xlo, int64_t ld)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int h = blockIdx.y;
    const bool valid = t < npts;
    float geo[3][8];
    float col[4] = {0.f, 0.f, 0.f, 0.f};
    for (int c = 0; c < 3; ++c)
        for (int q = 0; q < 8; ++q) geo[c][q] = 0.f;
    // the wavefront's sample box (every lane takes part in the reductions, so before the branch on
    // valid): groups of segments farther than their near radius take the loop without near tests
    // (handles of few segments keep every near test: there a box lookup per pair and the box itself
    // would cost more than they save; paper-native handles, S = 1: +0.25 ms per LM step)
    const bool cull = S >= 8;
    const float Xv = valid ? (float)x[2 * t] : 0.f, Yv = valid ? (float)x[2 * t + 1] : 0.f;
    float wx0 = 0.f, wx1 = 0.f, wy0 = 0.f, wy1 = 0.f;
    if (cull) {
        wx0 = uniform_f32(wave_min(valid ? Xv : INFINITY));
        wx1 = uniform_f32(wave_max(valid ? Xv : -INFINITY));
        wy0 = uniform_f32(wave_min(valid ? Yv : INFINITY));
        wy1 = uniform_f32(wave_max(valid ? Yv : -INFINITY));
    }
    if (valid) {
        const float Xf = Xv, Yf = Yv;
        // test: whether the pairs need the near test (false once the segment's group of kBoxGroup
        // segments is out of the wavefront's reach; wave-uniform, looked up at each group's start)
        bool test = true;
#pragma unroll 1
        for (int j = 0; j < S; ++j) {
            const int k = h * S + j;
            if (cull && (j == 0 || k % kBoxGroup == 0)) test = !box_culled(box, k / kBoxGroup, wx0, wy0, wx1, wy1);
            const float* s = seg32 + (size_t)k * kSegStride;
            const float* V = vtab + 8 * j;
            const bool on = !(test & near_segment(s[0], s[1], s[2], s[3], s[6], Xf, Yf, near2));
            if (Band) {
                const bool band = on & near_segment(s[0], s[1], s[2], s[3], s[6], Xf, Yf, 4.0f);
                add_pair_features<6>(s, V, V + 8, Xf, Yf, eps2f, on & !band, geo, col);
                if (__any(band)) closed_pair_features(s, V, Xf, Yf, eps2f, band, geo, col);
            } else {
                add_pair_features<6>(s, V, V + 8, Xf, Yf, eps2f, on, geo, col);
            }
        }
        const int64_t i = t0 + t;
        const bool take = !flag[i];
        // the wavefront's index within the tile (the same for all its lanes, as t0 is a multiple of 64)
        const int wl = __builtin_amdgcn_readfirstlane((int)(t >> 6));
        const int2 run = runs[(size_t)wl * H + h];
        const NearPair* sl = list + ((t0 >> 6) + wl) * (int64_t)slots;
        const float* cw = corr + (size_t)wl * slots * kFeatVals;
        for (int e = run.x; e < run.y; ++e) {
            const NearPair p = sl[e];
            if (!take || p.sample != (int32_t)i) continue;
            const float* cr = cw + (size_t)e * kFeatVals;
            for (int c = 0; c < 3; ++c)
                for (int q = 0; q < 8; ++q) geo[c][q] += cr[8 * c + q];
            for (int q = 0; q < 4; ++q) col[q] += cr[24 + q];
        }
        store_handle_rows(model, Xt, Xlo, H, h, t, ld, gp, geo, col);
    }
}

// Ranges of each handle's entries in the near-pair slices of a tile's wavefronts
// w0 .. w0 + nw - 1 (entries sorted by segment; element entries come last):
// runs[(w - w0) H + h] = [first entry with seg >= h S, first entry with seg >= (h + 1) S).
__global__ void __launch_bounds__(256) k_near_runs(const NearPair* __restrict__ list, int slots,
                                                   const int* __restrict__ wave_count, int64_t w0, int64_t nw, int H,
                                                   int S, int2* __restrict__ runs)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nw * H) return;
    const int64_t w = w0 + t / H;
    const int h = (int)(t % H);
    const NearPair* sl = list + w * slots;
    const int cnt = wave_count[w];
    int b[2];
    for (int k = 0; k < 2; ++k) {
        const int key = (h + k) * S;
        int lo = 0, hi = cnt;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (sl[mid].seg < key) lo = mid + 1;
            else hi = mid;
        }
        b[k] = lo;
    }
    runs[t] = make_int2(b[0], b[1]);
}

// Zero the samples [n, n rounded up to 32) of every row of a blocked split-bfloat16
// tile: the Gram kernel reads whole 32-sample blocks.
__global__ void k_zero_tail(uint16_t* __restrict__ Xh, uint16_t* __restrict__ Xl, int64_t W, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t tail = ((n + 31) & ~(int64_t)31) - n;
    if (i >= W * tail) return;
    const int64_t f = i / tail, t = n + i % tail;
    const size_t e = (size_t)(t >> 5) * (size_t)(W << 5) + (size_t)(f << 5) + (size_t)(t & 31);
    Xh[e] = 0;
    Xl[e] = 0;
}

// Vertex table of the float32 feature kernel: vtab[8 j + q] = the vertex weights at t_j
// (vertex_weights), vtab[8 j + 4] = t_j, vtab[8 j + 5] = 1 - t_j, t_j = j / S.
__global__ void k_vertex_table(int S, int model, float* __restrict__ vtab)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j > S) return;
    const double t = (double)j / (double)S;
    double B[4];
    vertex_weights(model, t, B);
    for (int q = 0; q < 4; ++q) vtab[8 * j + q] = (float)B[q];
    vtab[8 * j + 4] = (float)t;
    vtab[8 * j + 5] = (float)(1.0 - t);
    vtab[8 * j + 6] = vtab[8 * j + 7] = 0.0f;
}

// Float64 contributions of one listed near (sample, segment) pair to its handle's
// features: o[28] = geo[3][8] and col[4] as in store_handle_rows (geometry already
// chained with the vertex weights); k_features_near stores them at the pair's slot
// of the tile (wavefronts w0 .. w0 + nw - 1), corr[slot][28].
__device__ inline void features_near_pair(const NearPair p, const double* __restrict__ x,
                                          const double* __restrict__ seg64, int S, int model, double eps2,
                                          float* __restrict__ o)
{
    const double X = x[2 * (int64_t)p.sample], Y = x[2 * (int64_t)p.sample + 1];
    const double* s64 = seg64 + (size_t)p.seg * kSegStride;
    const SegGeom<double> g = load_geom(s64);
    const int j = p.seg % S;
    const double ta = (double)j / (double)S, tb = (double)(j + 1) / (double)S;
    double Ba[4], Bb[4];
    vertex_weights(model, ta, Ba);
    vertex_weights(model, tb, Bb);
    const PairState<double> st = pair_forward<double, DevF64, true>(g, X, Y, eps2);
    const Moments<double> m = pair_moments(g, st);
    for (int c = 0; c < 3; ++c) {
        const Grad4<double> gr = pair_backward(g, st, eps2, s64[kWdA + c], s64[kWdB + c], s64[kWcA + c], s64[kWcB + c]);
        for (int q = 0; q < 4; ++q) {
            o[8 * c + 2 * q] = (float)(Ba[q] * gr.ax + Bb[q] * gr.bx);
            o[8 * c + 2 * q + 1] = (float)(Ba[q] * gr.ay + Bb[q] * gr.by);
        }
    }
    o[24] = (float)(m.da * (1.0 - ta) + m.db * (1.0 - tb));
    o[25] = (float)(m.da * ta + m.db * tb);
    o[26] = (float)(m.sa * (1.0 - ta) + m.sb * (1.0 - tb));
    o[27] = (float)(m.sa * ta + m.sb * tb);
}

// block per wavefront slice w0 + blockIdx.x, its threads looping over the slice's entries
__global__ void __launch_bounds__(256) k_features_near(const NearPair* __restrict__ list, int slots,
                                                       const int* __restrict__ wave_count,
                                                       const uint8_t* __restrict__ flag, int64_t w0,
                                                       const double* __restrict__ x, const double* __restrict__ seg64,
                                                       int K, int S, int model, double eps2,
                                                       float* __restrict__ corr)
{
    const int64_t w = w0 + blockIdx.x;
    const int cnt = wave_count[w];
    for (int e = threadIdx.x; e < cnt; e += blockDim.x) {
        const NearPair p = list[w * slots + e];
        if (p.seg >= K || flag[p.sample]) continue;
        features_near_pair(p, x, seg64, S, model, eps2, corr + ((size_t)blockIdx.x * slots + e) * kFeatVals);
    }
}

// beta rows: Xt[row0 + j][t] = beta_j(x_t); thread per point, each block row of the grid a
// run of kBetaRun elements (element data by uniform loads), so that a launch has few, long
// blocks rather than one short block per element.
constexpr int kBetaRun = 32;
template <bool Mixed, class OutT>
__global__ void __launch_bounds__(256) k_beta_rows(const double* __restrict__ x, int64_t npts,
                                                   const double* __restrict__ el64, const float* __restrict__ el32,
                                                   int M, float near2, OutT* __restrict__ Xt, uint16_t* __restrict__ Xlo,
                                                   int64_t ld, int64_t row0)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= npts) return;
    const double X = x[2 * t], Y = x[2 * t + 1];
    const float Xf = (float)X, Yf = (float)Y;
    const int j0 = blockIdx.y * kBetaRun, j1 = j0 + kBetaRun < M ? j0 + kBetaRun : M;
    for (int j = j0; j < j1; ++j) {
        const double* e = el64 + (size_t)j * kElemStride;
        double b;
        if (Mixed) {
            const float* f = el32 + (size_t)j * kElemStride;
            if (near_element(f[0], f[1], f[2], f[3], Xf, Yf, near2))
                b = element_beta<double, DevF64>(e[0], e[1], e[2], e[3], X, Y);
            else
                b = (double)element_beta<float, DevF32>(f[0], f[1], f[2], f[3], Xf, Yf);
        } else {
            b = element_beta<double, DevF64>(e[0], e[1], e[2], e[3], X, Y);
        }
        Store<OutT>::put(Xt, Xlo, row0 + j, t, ld, b);
    }
}

// beta rows into a split-bfloat16 tile in the blocked layout [t / 32][row][t % 32]: the block
// computes its 256 samples x kBetaRunBlocked elements into LDS, then writes whole runs: the
// kBetaRunBlocked rows of one 32-sample block are one contiguous 1 KiB run (hi, and another for
// lo), written with 16-byte stores.  (Written lane by lane, each store instruction of a
// wavefront covered two 64-byte halves of cache lines; beside the Gram that took 1.5-2.4 ms
// per 32,768-sample tile against 0.05 ms alone.)  LDS rows hold their 8-sample chunks in
// XOR-swizzled order (chunk q of row r at q ^ (r & 7)), so that the 16-byte reads of 16 rows
// at one chunk fall in different banks; 16 KiB, so that a block fits beside a Gram block.
// Samples past npts in a written block are zeros.
constexpr int kBetaRunBlocked = 16;
template <bool Mixed>
__global__ void __launch_bounds__(256) k_beta_rows_blocked(const double* __restrict__ x, int64_t npts,
                                                           const double* __restrict__ el64,
                                                           const float* __restrict__ el32, int M, float near2,
                                                           uint16_t* __restrict__ Xh, uint16_t* __restrict__ Xl,
                                                           int64_t ld, int64_t row0)
{
    constexpr int R = kBetaRunBlocked;
    __shared__ __attribute__((aligned(16))) uint16_t sh[2][R][256];
    const int64_t t0 = (int64_t)blockIdx.x * 256;
    const int64_t t = t0 + threadIdx.x;
    const int j0 = blockIdx.y * R, nj = M - j0 < R ? M - j0 : R;
    const bool live = t < npts;
    const double X = live ? x[2 * t] : 0.0, Y = live ? x[2 * t + 1] : 0.0;
    const float Xf = (float)X, Yf = (float)Y;
#pragma unroll
    for (int jj = 0; jj < R; ++jj) {
        if (jj >= nj) continue;
        const int j = j0 + jj;
        const double* e = el64 + (size_t)j * kElemStride;
        double b = 0.0;
        if (live) {
            if (Mixed) {
                const float* f = el32 + (size_t)j * kElemStride;
                if (near_element(f[0], f[1], f[2], f[3], Xf, Yf, near2))
                    b = element_beta<double, DevF64>(e[0], e[1], e[2], e[3], X, Y);
                else
                    b = (double)element_beta<float, DevF32>(f[0], f[1], f[2], f[3], Xf, Yf);
            } else {
                b = element_beta<double, DevF64>(e[0], e[1], e[2], e[3], X, Y);
            }
        }
        const float v = (float)b;
        const uint16_t h = bf16_bits(v);
        const int col = threadIdx.x ^ ((jj & 7) << 3);
        sh[0][jj][col] = h;
        sh[1][jj][col] = bf16_bits(v - bf16_value(h));
    }
    __syncthreads();
    // hi and lo x 8 sample blocks x R rows x 4 chunks of 8 samples; a wavefront writes the R rows of
    // one sample block (R x 64 bytes, contiguous)
    constexpr int per = 8 * R * 4;
    for (int e = threadIdx.x; e < 2 * per; e += 256) {
        const int which = e / per, r = e % per;
        const int sb = r / (R * 4), jj = (r >> 2) % R, c = r & 3;
        // sample blocks wholly past npts are not written: the tile holds npts rounded up to 32
        // (64) samples, which need not reach the block's 256
        if (jj >= nj || t0 + sb * 32 >= npts) continue;
        const int q = (sb * 4 + c) ^ (jj & 7);          // swizzled 8-sample chunk of this row
        const uint4 v = *reinterpret_cast<const uint4*>(&sh[which][jj][q * 8]);
        uint16_t* dst = (which ? Xl : Xh) + (size_t)((t0 >> 5) + sb) * (size_t)(ld << 5) +
                        (size_t)((row0 + j0 + jj) << 5) + c * 8;
        *reinterpret_cast<uint4*>(dst) = v;
    }
}

__global__ void k_gauss_points(int M, const double* __restrict__ eg, double* __restrict__ gx)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= 3 * M) return;
    const int i = t / 3, q = t % 3;
    double ax, ay, bx, by;
    load_element(eg, i, ax, ay, bx, by);
    const double node = q == 0 ? -kGaussNode : (q == 1 ? 0.0 : kGaussNode);
    gx[2 * t] = 0.5 * (ax + bx) + node * 0.5 * (bx - ax);
    gx[2 * t + 1] = 0.5 * (ay + by) + node * 0.5 * (by - ay);
}

// dF[f][i] = sum_q w_q |G_i|/2 Xg[f][3i + q], zeros for i in [M, Mp)
__global__ void k_boundary_features(const double* __restrict__ Xg, int nf, int M, int Mp, const double* __restrict__ eg,
                                    double* __restrict__ dF)
{
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < (int64_t)nf * Mp; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t f = e / Mp;
        const int i = (int)(e % Mp);
        double v = 0.0;
        if (i < M) {
            double ax, ay, bx, by;
            load_element(eg, i, ax, ay, bx, by);
            const double half = 0.5 * sqrt((bx - ax) * (bx - ax) + (by - ay) * (by - ay));
            const double* r = Xg + f * 3 * M + 3 * i;
            v = half * (kGaussW0 * r[0] + kGaussW1 * r[1] + kGaussW0 * r[2]);
        }
        dF[e] = v;
    }
}

// X [rows][ldx] (transposed: [cols][ldx]) into Y [rp][cp], zeros outside
__global__ void k_pad(const double* __restrict__ X, int64_t ldx, bool transposed, int64_t rows, int cols, int64_t rp, int cp,
                      double* __restrict__ Y)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t r = e / cp, c = e % cp;
    if (r < rp) Y[e] = r < rows && c < cols ? X[transposed ? c * ldx + r : r * ldx + c] : 0.0;
}

// Zeros in columns [n, n rounded up to kGemmPad) of a float64 tile's W rows
__global__ void k_zero_tail_f64(double* __restrict__ Xt, int64_t W, int64_t ld, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t t = n + i % kGemmPad;
    if (i < W * kGemmPad && t < (n + kGemmPad - 1) / kGemmPad * kGemmPad) Xt[i / kGemmPad * ld + t] = 0.0;
}

__global__ void k_fill(double* __restrict__ p, int64_t n, double v)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = v;
}

// Augmented Gram of channel c = blockIdx.z in compact order [g_c (GH) | e (CH) | beta (M)], rows of Wp with zeros
// past Wc, symmetric fill from the upper triangle of G.  The compact-to-row map is increasing, so
// entry (a, b) comes from G[row(a)][row(b)] for a <= b and from G[row(b)][row(a)] below the
// diagonal.  A block owns a 32 x 32 tile of (a, b); a tile below the diagonal reads its
// mirror tile along a (coalesced) and transposes it through LDS.
__global__ void __launch_bounds__(256) k_gather_gram(const double* __restrict__ G, int64_t W, Layout L, int Wc, int Wp,
                                                     double* __restrict__ Gc)
{
    __shared__ double T[32][33];
    const int c = blockIdx.z;
    Gc += (size_t)c * Wc * Wp;
    const int a0 = blockIdx.y * 32, b0 = blockIdx.x * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    if (b0 + 31 < a0) {                  // wholly below the diagonal: T[b][a] = G[row(b)][row(a)]
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int bb = b0 + ty + 8 * k, aa = a0 + tx;
            if (aa < Wc) T[ty + 8 * k][tx] = G[(size_t)L.row(bb, c) * W + L.row(aa, c)];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int a = a0 + ty + 8 * k, b = b0 + tx;
            if (a < Wc) Gc[(size_t)a * Wp + b] = T[tx][ty + 8 * k];
        }
        return;
    }
    const int b = b0 + tx;
    if (b >= Wp) return;
    const int64_t ib = b < Wc ? L.row(b, c) : 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int a = a0 + ty + 8 * k;
        if (a >= Wc) break;
        const int64_t ia = L.row(a, c);
        // the upper triangle holds every needed entry (diagonal tiles are computed whole)
        Gc[(size_t)a * Wp + b] = b >= Wc ? 0.0 : ia <= ib ? G[(size_t)ia * W + ib] : G[(size_t)ib * W + ia];
    }
}

// Zc[c][a][i] = Z[row(a, c)][i] for the handle part of the compact order (a < (G + C)H), rows of Mp
__global__ void k_gather_z(const double* __restrict__ Z, Layout L, int Mp, double* __restrict__ Zc)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int c = blockIdx.y;
    const int64_t a = e / Mp;
    if (a < L.compact()) Zc[(int64_t)c * L.compact() * Mp + e] = Z[(size_t)L.row((int)a, c) * Mp + e % Mp];
}

// Every entry of J^T J from the three channels' blocks v_c(a, b) = Gc_c[a][b] + (S_c[a][b] +
// S_c[b][a]) (compact indices a, b < n12), written once (no fill, no read-modify-write):
// geometry x geometry entries are shared by the channels and take v_0 + v_1 + v_2; an entry
// with a colour parameter of channel c takes v_c; colour entries of two different channels
// are zero.  A block owns a 32 x 32 tile of (a, b) and reads S_c[b][a] through LDS, so both
// reads of S are coalesced; v_c(a, b) = v_c(b, a) bit for bit, so J^T J is exactly symmetric.
__global__ void __launch_bounds__(256) k_scatter_jtj(const double* __restrict__ Gc, int64_t gcs, int Wp,
                                                     const double* __restrict__ S, int64_t ss, Layout L, double s,
                                                     double* __restrict__ JtJ, int64_t P)
{
    __shared__ double T[3][32][33];
    const int n = L.compact();
    const int a0 = blockIdx.y * 32, b0 = blockIdx.x * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int bb = b0 + ty + 8 * k, aa = a0 + tx;   // S_c[bb][aa], aa contiguous
            T[c][ty + 8 * k][tx] = (bb < n && aa < n) ? S[c * ss + (size_t)bb * n + aa] : 0.0;
        }
    __syncthreads();
    const int b = b0 + tx;
    if (b >= n) return;
    const int64_t geo = L.geo();
    const int Q = L.params();
    const bool gb = b < geo;
    const int64_t cb = gb ? (int64_t)Q * (b / L.G) + b % L.G
                          : (int64_t)Q * ((b - geo) / L.C) + L.G + 3 * ((b - geo) % L.C);   // + channel
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int a = a0 + ty + 8 * k;
        if (a >= n) break;
        double v[3];
        for (int c = 0; c < 3; ++c)
            v[c] = Gc[c * gcs + (size_t)a * Wp + b] + (S[c * ss + (size_t)a * n + b] + T[c][tx][ty + 8 * k]);
        const bool ga = a < geo;
        const int64_t ca = ga ? (int64_t)Q * (a / L.G) + a % L.G
                              : (int64_t)Q * ((a - geo) / L.C) + L.G + 3 * ((a - geo) % L.C);
        if (ga && gb) {
            JtJ[ca * P + cb] = s * ((v[0] + v[1]) + v[2]);
        } else if (ga) {
            for (int c = 0; c < 3; ++c) JtJ[ca * P + cb + c] = s * v[c];
        } else if (gb) {
            for (int c = 0; c < 3; ++c) JtJ[(ca + c) * P + cb] = s * v[c];
        } else {
            for (int c = 0; c < 3; ++c)
                for (int d = 0; d < 3; ++d) JtJ[(ca + c) * P + cb + d] = c == d ? s * v[c] : 0.0;
        }
    }
}

// J[n][c][p] assembly for the explicit Jacobian: features + beta . Z
__global__ void k_assemble_jacobian(const double* __restrict__ Xt, int64_t ld, const double* __restrict__ BZ, Layout L,
                                    int64_t npts, double* __restrict__ J)
{
    const int64_t t = blockIdx.y;
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    const int Q = L.params();
    const int P = Q * L.H;
    const int64_t nf = L.handle_rows();
    if (p >= P || t >= npts) return;
    const int h = p / Q, q = p % Q;
    for (int c = 0; c < 3; ++c) {
        double v;
        if (q < L.G) {
            const int64_t f = (int64_t)c * L.Gp + (int64_t)L.G * h + q;
            v = Xt[(size_t)f * ld + t] + BZ[(size_t)t * nf + f];
        } else {
            const int m = (q - L.G) / 3, cc = (q - L.G) % 3;
            const int64_t f = 3 * L.Gp + (int64_t)L.C * h + m;
            v = cc == c ? Xt[(size_t)f * ld + t] + BZ[(size_t)t * nf + f] : 0.0;
        }
        J[((size_t)t * 3 + c) * P + p] = v;
    }
}

}  // namespace

int fill_f64(bem_ctx* ctx, double* p, int64_t n, double v, hipStream_t s)
{
    if (n <= 0) return BEM_OK;
    int blocks = (int)((n + 255) / 256);
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(k_fill, dim3(blocks), dim3(256), 0, s, p, n, v);
    return check_launch(ctx, "fill");
}

constexpr int64_t kGeoAlign = 256;   // the split-BF16 Gram's tile
Layout layout_of(const bem_ctx* ctx, int H)
{
    const int64_t gh = (int64_t)ctx->ngeo * H;
    // few handles: without the padding a tile mixes channels, but the padded rows would be most of the
    // Gram (4 cubic handles: 1,808 rows of which 672 are padding)
    if (gh < kGeoAlign) return Layout{ctx->ngeo, ctx->ncol, H, gh};
    return Layout{ctx->ngeo, ctx->ncol, H, (gh + kGeoAlign - 1) / kGeoAlign * kGeoAlign};
}

// Feature rows of npts points into Xt (ld: row stride of float64 / float32 tiles,
// row count of the blocked bfloat16 tile); rows 0..(3G + C)H - 1 handle
// features, the next M rows beta when with_beta.  OutT: double, float or uint16_t (bf16 hi, lo in Xlo).
// Mixed precision needs the near-pair list of the whole sample set (nl), the tile's
// first global sample index t0 (a multiple of 64), the global samples xg and a
// correction buffer of ceil(npts / 64) * nl->slots * 28 floats and a run table of
// ceil(npts / 64) * H entries.
template <class OutT>
static int launch_features(bem_ctx* ctx, const double* x, int64_t npts, int H, bool mixed, bool with_beta, OutT* Xt,
                           uint16_t* Xlo, int64_t ld, hipStream_t s, const NearList* nl = nullptr, int64_t t0 = 0,
                           const double* xg = nullptr, float* corr = nullptr, const float* vtab = nullptr,
                           int2* runs = nullptr, const float4* box = nullptr)
{
    if (npts == 0) return BEM_OK;
    const int S = ctx->opts.segs_per_handle;
    const int model = ctx->model;
    const double eps2 = ctx->opts.eps * ctx->opts.eps;
    const double nf = near_radius(ctx->opts.near_factor);
    const float near2 = (float)(nf * nf);
    const Layout L = layout_of(ctx, H);
    const int64_t beta_row0 = L.handle_rows();
    const int64_t gp = L.Gp;
    const dim3 grid(blocks_for(npts, 256), H);
    if (mixed && (!nl || !xg || !corr || !vtab || !runs || !box || (t0 & 63)))
        return set_error(ctx, BEM_EINVAL, "mixed features need the near-pair list (internal)");
    if (H > 0) {
        if (mixed) {
            const int64_t nw = (npts + 63) / 64;
            {
                ProfScope ps_(ctx, PT_NEAR, s);
                hipLaunchKernelGGL(k_features_near, dim3(nw), dim3(256), 0, s, nl->list, nl->slots, nl->count, nl->flag,
                                   t0 >> 6, xg, (const double*)ctx->seg64.ptr, H * S, S, model, eps2, corr);
                hipLaunchKernelGGL(k_near_runs, dim3(blocks_for(nw * H, 256)), dim3(256), 0, s, nl->list, nl->slots,
                                   nl->count, t0 >> 6, nw, H, S, runs);
            }
            ProfScope ps_(ctx, PT_FEATURES, s);
            const auto far = nf < 2.0 ? k_features_far<true, OutT> : k_features_far<false, OutT>;
            hipLaunchKernelGGL(far, grid, dim3(256), 0, s, x, npts, t0, (const float*)ctx->seg32.ptr,
                               H, S, model, gp, (float)eps2, near2, nl->list, nl->slots, (const int2*)runs, nl->flag, corr,
                               vtab, box, Xt, Xlo, ld);
            const int fb = blocks_for(npts, 256) < 16 ? blocks_for(npts, 256) : 16;
            if (nl->overflowed)
                hipLaunchKernelGGL((k_features<true, OutT>), dim3(fb, H), dim3(256), 0, s, x, npts, (const double*)ctx->seg64.ptr,
                               (const float*)ctx->seg32.ptr, H, S, model, gp, eps2, (float)eps2, near2, nl->flag + t0,
                               Xt, Xlo, ld);
        } else {
            ProfScope ps_(ctx, PT_FEATURES, s);
            const bool split = S >= 8 && (int64_t)grid.x * grid.y < 1024;
            hipLaunchKernelGGL((split ? k_features<false, OutT, 4> : k_features<false, OutT>),
                               split ? dim3(blocks_for(npts, 64), H) : grid, dim3(256), 0, s, x, npts,
                               (const double*)ctx->seg64.ptr, (const float*)ctx->seg32.ptr, H, S, model, gp, eps2, (float)eps2,
                               near2, (const uint8_t*)nullptr, Xt, Xlo, ld);
        }
    }
    if (H > 0 && gp > L.geo()) {
        const int64_t nz = 3 * (gp - L.geo()) * npts;
        hipLaunchKernelGGL((k_zero_pad<OutT>), dim3(blocks_for(nz, 256)), dim3(256), 0, s, Xt, Xlo, ld, gp, L.geo(), npts);
    }
    if (with_beta && std::is_same<OutT, uint16_t>::value) {
        const dim3 gb(blocks_for(npts, 256), blocks_for(ctx->M, kBetaRunBlocked));
        ProfScope ps_(ctx, PT_BETA_ROWS, s);
        if (mixed)
            hipLaunchKernelGGL((k_beta_rows_blocked<true>), gb, dim3(256), 0, s, x, npts, (const double*)ctx->elem64.ptr,
                               (const float*)ctx->elem32.ptr, ctx->M, near2, (uint16_t*)Xt, Xlo, ld, beta_row0);
        else
            hipLaunchKernelGGL((k_beta_rows_blocked<false>), gb, dim3(256), 0, s, x, npts, (const double*)ctx->elem64.ptr,
                               (const float*)ctx->elem32.ptr, ctx->M, near2, (uint16_t*)Xt, Xlo, ld, beta_row0);
    } else if (with_beta) {
        const dim3 gb(blocks_for(npts, 256), blocks_for(ctx->M, kBetaRun));
        if (mixed)
            {
                ProfScope ps_(ctx, PT_BETA_ROWS, s);
                hipLaunchKernelGGL((k_beta_rows<true, OutT>), gb, dim3(256), 0, s, x, npts, (const double*)ctx->elem64.ptr,
                                   (const float*)ctx->elem32.ptr, ctx->M, near2, Xt, Xlo, ld, beta_row0);
            }
        else
            {
                ProfScope ps_(ctx, PT_BETA_ROWS, s);
                hipLaunchKernelGGL((k_beta_rows<false, OutT>), gb, dim3(256), 0, s, x, npts, (const double*)ctx->elem64.ptr,
                                   (const float*)ctx->elem32.ptr, ctx->M, near2, Xt, Xlo, ld, beta_row0);
            }
    }
    return check_launch(ctx, "features");
}

// also leaves Gauss features in tmp3
int boundary_derivatives(bem_ctx* ctx, int H, hipStream_t s, double** Zout)
{
    int rc;
    const int M = ctx->M, Mp = gemm_pad(M);
    const int nf = (int)layout_of(ctx, H).handle_rows();
    const size_t gxs = (size_t)3 * M * 2, xgs = (size_t)nf * 3 * M;
    const size_t aps = Mp == M ? 0 : (size_t)Mp * Mp;
    if ((rc = ensure(ctx, ctx->tmp3, (gxs + xgs + aps) * sizeof(double) + 16, s))) return rc;
    if ((rc = ensure(ctx, ctx->tmp4, (size_t)2 * Mp * nf * sizeof(double), s))) return rc;
    double* gx = (double*)ctx->tmp3.ptr;
    double* Xg = gx + gxs;
    const double* Ap = (const double*)ctx->Apinv.ptr;
    double* dF = (double*)ctx->tmp4.ptr;
    double* Z = dF + (size_t)Mp * nf;
    if (aps) {
        double* t = Xg + xgs + (xgs & 1);        // gxs is even: 16-byte aligned
        hipLaunchKernelGGL(k_pad, dim3(blocks_for((int64_t)Mp * Mp, 256)), dim3(256), 0, s, Ap, (int64_t)M, false, (int64_t)M, M,
                           (int64_t)Mp, Mp, t);
        Ap = t;
    }
    hipLaunchKernelGGL(k_gauss_points, dim3(blocks_for(3 * M, 256)), dim3(256), 0, s, M, (const double*)ctx->egeo.ptr, gx);
    if ((rc = launch_features<double>(ctx, gx, 3 * (int64_t)M, H, false, false, Xg, nullptr, 3 * (int64_t)M, s))) return rc;
    // (a launch holds fewer than 2^32 threads)
    hipLaunchKernelGGL(k_boundary_features, dim3(std::min(blocks_for((int64_t)nf * Mp, 256), 1 << 22)), dim3(256), 0, s, Xg, nf, M, Mp,
                       (const double*)ctx->egeo.ptr, dF);
    if ((rc = check_launch(ctx, "boundary features"))) return rc;
    if ((rc = gemm_f64(ctx, Gemm64{nf, Mp, Mp, 1.0, dF, Mp, Ap, Mp, 0.0, Z, Mp}, 1, s))) return rc;
    *Zout = Z;
    return BEM_OK;
}

static std::vector<int> gram_tiles(const Layout& L, int W, int ts)
{
    // upper-triangle ts x ts tiles, skipping pairs of tiles that lie inside two
    // different channels' geometry blocks (those products never enter J^T J)
    const int nt = (W + ts - 1) / ts;
    const int64_t g = L.Gp;
    auto region = [&](int t) {
        const int64_t lo = (int64_t)t * ts, hi = lo + ts - 1;
        if (lo >= 3 * g) return -1;                              // colour coefficients / beta: shared
        if (hi >= 3 * g) return -2;                              // straddles geometry and shared rows
        const int64_t c0 = lo / g, c1 = hi / g;
        return c0 == c1 ? (int)c0 : -2;
    };
    std::vector<int> t;
    for (int i = 0; i < nt; ++i)
        for (int j = i; j < nt; ++j) {
            const int ri = region(i), rj = region(j);
            if (ri >= 0 && rj >= 0 && ri != rj) continue;
            t.push_back(i);
            t.push_back(j);
        }
    return t;
}

// Work list of the MFMA Grams: (row tile, column tile, sample part) for every
// needed tile and part, part-major, then by super-tiles of 4 x 8 output tiles,
// then row and column.  Consecutive entries share operand panels (the Gram
// kernels give each XCD a contiguous run of entries).
static std::vector<int> gram_work(const std::vector<int>& tiles, int parts)
{
    const int nt = (int)tiles.size() / 2;
    std::vector<int> order(nt);
    for (int t = 0; t < nt; ++t) order[t] = t;
    auto key = [&](int t) {
        const int i = tiles[2 * t], j = tiles[2 * t + 1];
        return std::make_tuple(i / 4, j / 8, i, j);
    };
    std::sort(order.begin(), order.end(), [&](int a, int b) { return key(a) < key(b); });
    std::vector<int> w;
    w.reserve((size_t)3 * nt * parts);
    for (int p = 0; p < parts; ++p)
        for (int t : order) {
            w.push_back(tiles[2 * t]);
            w.push_back(tiles[2 * t + 1]);
            w.push_back(p);
        }
    return w;
}

// Sample parts of the float64 Gram: 512 blocks (two 128 x 128 tiles a CU) run at a time, so the parts are
// chosen to fill one, two or three such rounds, the fewest that leave at most 2% more of them empty than the best
// (at most 16 parts and 2 GiB of partial Grams).  45 tiles (4 cubic handles, 16,384 samples): 16 parts, 1.4 rounds,
// 427 us and 44 us to sum them; 11 parts, one round, 412 and 12 us.
static int f64_parts(int ntiles, int64_t W)
{
    const int64_t most = std::max<int64_t>(1, std::min<int64_t>(16, ((int64_t)2 << 30) / (W * W * 8)));
    const auto fill = [&](int64_t p) { return (double)(ntiles * p) / (double)((ntiles * p + 511) / 512 * 512); };
    int64_t best = 1;
    for (int rounds = 1; rounds <= 3 && ntiles > 0; ++rounds) {
        const int64_t p = std::min<int64_t>(most, 512 * rounds / ntiles);
        if (p >= 1 && fill(p) > fill(best) + 0.02) best = p;
    }
    return (int)best;
}

// Sample parts of the split-BF16 Gram, one 256 x 256 tile a CU: at least 3 (float32 runs no longer than a third of a
// sample tile), and for few tiles those that fill up to three rounds of 256 best (60 straight handles, 15,000 samples,
// 36 tiles: 3 parts 305 us, 7 parts 95 us and 40 us more to sum them).
static int bf16_parts(int ntiles, int64_t W)
{
    const int64_t most = std::max<int64_t>(3, std::min<int64_t>(16, ((int64_t)2 << 30) / (W * W * 8)));
    const auto fill = [&](int64_t p) { return (double)(ntiles * p) / (double)((ntiles * p + 255) / 256 * 256); };
    int64_t best = 3;
    for (int rounds = 1; rounds <= 3 && ntiles > 0; ++rounds) {
        const int64_t p = std::min<int64_t>(most, 256 * rounds / ntiles);
        if (p > 3 && fill(p) > fill(best) + 0.02) best = p;
    }
    return (int)best;
}

namespace {
// G[0] += G[1] + ... + G[parts - 1] (fixed order) over the ts x ts output tile of work entry
// blockIdx.x, rows split over gridDim.y blocks (blockDim.x = ts, a thread per column)
__global__ void __launch_bounds__(256) k_sum_parts(double* __restrict__ G, int parts, int64_t W,
                                                   const int* __restrict__ work, int ts)
{
    const int64_t c0 = (int64_t)work[3 * blockIdx.x + 1] * ts;
    const int64_t rt = (int64_t)work[3 * blockIdx.x] * ts;   // the tile's first row
    const int rows = (ts + gridDim.y - 1) / gridDim.y;
    const int64_t r0 = rt + (int64_t)blockIdx.y * rows;
    const int64_t r1 = rt + ts < r0 + rows ? rt + ts : r0 + rows;
    const int64_t c = c0 + threadIdx.x % ts;
    for (int64_t r = r0 + threadIdx.x / ts; r < r1; r += blockDim.x / ts) {
        if (r >= W || c >= W) continue;
        const size_t e = (size_t)r * W + c;
        double v = G[e];
        for (int p = 1; p < parts; ++p) v += G[(size_t)p * W * W + e];
        G[e] = v;
    }
}
}  // namespace

// A work list lives on the device; it is uploaded when its configuration changes, the only host
// synchronisation of bem_jtj apart from workspace growth.
static int upload_tiles(bem_ctx* ctx, WorkList& list, const std::vector<int>& tiles, int64_t W, int H, int gram, int parts,
                        hipStream_t s)
{
    int rc;
    const int64_t key[4] = {W, H, ctx->model, gram + 8 * (int64_t)parts};
    if (std::memcmp(key, list.key, sizeof(key)) == 0) return BEM_OK;
    list.key[0] = -1;
    if ((rc = ensure(ctx, list.buf, tiles.size() * sizeof(int), s))) return rc;
    if (hipMemcpyAsync(list.buf.ptr, tiles.data(), tiles.size() * sizeof(int), hipMemcpyHostToDevice, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)           // the host copy goes out of scope at the caller
        return set_error(ctx, BEM_EHIP, "tile list upload");
    std::memcpy(list.key, key, sizeof(key));
    return BEM_OK;
}

int contract_gram(bem_ctx* ctx, int H, const Layout& L, int64_t W, double* G, int parts, int ts, const int* work, int nwork,
                  const double* Z, double sc, double* JtJ, hipStream_t s)
{
    int rc;
    const int M = ctx->M;
    const int64_t P = (int64_t)L.params() * H;
    const int n12 = L.compact();          // handle part of one channel's compact order
    const int Wc = n12 + M;
    if (parts > 1) {
        // the first nwork / parts work entries are part 0's, one per tile of the list
        hipLaunchKernelGGL(k_sum_parts, dim3(nwork / parts, nwork / parts < 64 ? 32 : 8), dim3(256), 0, s, G, parts, W, work, ts);
        if ((rc = check_launch(ctx, "gram parts"))) return rc;
    }
    // contraction: the channels' compact Grams and S, then every entry of J^T J in one pass.
    // A channel's block of J^T J is G + B Zc + (B Zc)^T + Zc^T D Zc (Zc [M][n12] = Z's columns) with B = Gc[0:n12, n12:Wc]
    // and D = Gc[n12:, n12:] (symmetric), which equals G + S + S^T with S = Y Zc and
    // Y = B + (1/2) Zc^T D: two products instead of three.  Y overwrites B in Gc.
    const int Mp = gemm_pad(M), Wp = n12 + Mp;
    const int64_t wc2 = (int64_t)Wc * Wp, szc = (int64_t)Mp * n12, sn = (int64_t)n12 * n12;
    if ((rc = ensure(ctx, ctx->tmp2, 3 * (wc2 + szc + sn) * sizeof(double), s))) return rc;
    double* Gc3 = (double*)ctx->tmp2.ptr;
    double* Zc = Gc3 + 3 * wc2;
    double* S3 = Zc + 3 * szc;
    if (n12 > 0) {
        hipLaunchKernelGGL(k_gather_gram, dim3(blocks_for(Wp, 32), blocks_for(Wc, 32), 3), dim3(256), 0, s, G, W, L, Wc, Wp, Gc3);
        hipLaunchKernelGGL(k_gather_z, dim3(blocks_for((int64_t)n12 * Mp, 256), 3), dim3(256), 0, s, Z, L, Mp, Zc);
        if ((rc = check_launch(ctx, "gather"))) return rc;
        if ((rc = gemm_f64(ctx, Gemm64{n12, M, Mp, 0.5, Zc, Mp, Gc3 + (size_t)n12 * Wp + n12, Wp, 1.0, Gc3 + n12, Wp, szc, wc2, wc2},
                           3, s)))
            return rc;
        if ((rc = gemm_f64(ctx, Gemm64{n12, n12, Mp, 1.0, Gc3 + n12, Wp, Zc, Mp, 0.0, S3, n12, wc2, szc, sn}, 3, s))) return rc;
        hipLaunchKernelGGL(k_scatter_jtj, dim3(blocks_for(n12, 32), blocks_for(n12, 32)), dim3(256), 0, s, Gc3, wc2, Wp, S3, sn, L,
                           sc, JtJ, P);
        if ((rc = check_launch(ctx, "scatter"))) return rc;
    }
    return BEM_OK;
}

int run_jtj(bem_ctx* ctx, const double* theta, int H, const double* x, int64_t N, bool mixed, int gram, double* JtJ,
            hipStream_t s, const NearList* pre, double norm)
{
    int rc;
    const int M = ctx->M;
    const Layout L = layout_of(ctx, H);
    const int64_t W = L.handle_rows() + M;
    if (H == 0) return BEM_OK;
    if ((rc = launch_expand(ctx, theta, H, s))) return rc;
    double* Z = nullptr;
    if ((rc = boundary_derivatives(ctx, H, s, &Z))) return rc;
    // sample tiles
    // sample tile: large for the float64 Gram; for the MFMA Grams small enough that the tile of
    // feature rows (W x T, 4 bytes per entry) stays resident in the last-level cache while every
    // output tile re-reads it
    // sample tile: 32,768 for the split-BF16 Gram (1 GB of blocked bf16 pairs at the LM workload; 3
    // parts of 10,944 samples per launch)
    // float64 Gram on MFMA (BEM_GRAM_FP64) or on the VALU (BEM_GRAM_FP64_VALU): float64 tiles
    const bool f64 = gram == BEM_GRAM_FP64 || gram == BEM_GRAM_FP64_VALU;
    int64_t T = ctx->opts.tile_rows > 0 ? ctx->opts.tile_rows
                                        : (gram == BEM_GRAM_FP32_MFMA ? 8192 : 32768);
    const size_t elem = f64 ? 8 : 4;
    while (T > 1024 && (size_t)W * T * elem > ((size_t)3 << 30)) T /= 2;
    if (T > N) T = N > 0 ? N : 1;
    T = (T + 63) / 64 * 64;
    if (gram == BEM_GRAM_BF16X3_MFMA)
        while (T > 64 && W * T >= ((int64_t)1 << 31)) T = (T / 2 + 63) / 64 * 64;   // 32-bit offsets in the Gram
    // default tile size: a short last tile (at most a quarter of a tile) is spread over the others,
    // since it would cost a Gram launch of its own (the launch's partial-Gram traffic does not
    // shrink with the samples)
    if (ctx->opts.tile_rows <= 0 && N > T) {
        const int64_t nt = N / T, tail = N - nt * T;
        const int64_t T2 = ((N + nt - 1) / nt + 63) / 64 * 64;
        if (tail > 0 && tail <= T / 4 && (size_t)W * T2 * elem <= ((size_t)3 << 30) &&
            (gram != BEM_GRAM_BF16X3_MFMA || W * T2 < ((int64_t)1 << 31)))
            T = T2;
    }
    // MFMA Grams with several sample tiles: the Gram of tile t runs on a second stream while tile t+1's
    // feature rows are formed on the caller's stream (two tile buffers), so the VALU-bound feature
    // kernels and the MFMA-bound Gram share the chip.  Sharing slows a Gram launch by about a third
    // and short launches beside it several-fold (measured), so it pays only when the feature work
    // (handle segment pairs per sample, H S) is a sizeable share of the Gram's (its distinct output
    // area): from about a third of the Gram's time, H S >= area / 8000.
    const int64_t gram_area = (int64_t)(gram_tiles(L, (int)W, 256).size() / 2) * 256 * 256;
    const bool shares = !f64 && (int64_t)H * ctx->opts.segs_per_handle * 8000 >= gram_area;
    // default split-BF16 tile when the Gram runs alone: the fewest tiles the tile buffer holds,
    // balanced (fewer Gram launches and partial-Gram read-modify-writes: paper-native step -0.2 ms
    // with 2 tiles of 50,048 samples against 3 of 33,344)
    if (ctx->opts.tile_rows <= 0 && gram == BEM_GRAM_BF16X3_MFMA && !shares && N > T) {
        int64_t Tmax = (int64_t)(((size_t)3 << 30) / ((size_t)W * elem)) / 64 * 64;
        const int64_t Toff = (((int64_t)1 << 31) - 1) / W / 64 * 64;          // 32-bit offsets in the Gram
        if (Toff < Tmax) Tmax = Toff;
        if (Tmax > T) {
            const int64_t nt = (N + Tmax - 1) / Tmax;
            const int64_t T2 = ((N + nt - 1) / nt + 63) / 64 * 64;
            if (T2 > T) T = T2;
        }
    }
    // the sample tile is split into parts with partial Grams of their own, so that a launch fills the CUs and stays
    // deterministic (no atomics)
    const int ts = gram == BEM_GRAM_FP64_VALU ? 64 : (gram == BEM_GRAM_BF16X3_MFMA ? 256 : 128);
    const std::vector<int> out_tiles = gram_tiles(L, (int)W, ts);
    const int least = gram == BEM_GRAM_BF16X3_MFMA ? 3 : 1;
    int parts = gram == BEM_GRAM_BF16X3_MFMA ? bf16_parts((int)out_tiles.size() / 2, W)
                : gram == BEM_GRAM_FP64 ? f64_parts((int)out_tiles.size() / 2, W) : 1;
    // tmp0: feature tile(s); tmp1: G [parts][W][W].  With no memory for them the fewest parts, then (float64) smaller tiles
    bool overlap;
    size_t tile_bytes;
    for (;;) {
        overlap = shares && N > T;
        tile_bytes = ((size_t)W * T * elem + 255) / 256 * 256;
        rc = ensure(ctx, ctx->tmp0, tile_bytes * (overlap ? 2 : 1), s);
        if (!rc) rc = ensure(ctx, ctx->tmp1, (size_t)parts * W * W * sizeof(double), s);
        if (!rc) break;
        const bool smaller = f64 && ctx->opts.tile_rows <= 0 && T > 16384;
        if (rc != BEM_ENOMEM || !(parts > least || smaller)) return rc;
        if (parts > least) parts = least;
        else T = (T / 2 + 63) / 64 * 64;
        if (hipStreamSynchronize(s) != hipSuccess) return set_error(ctx, BEM_EHIP, "stream sync");
        release(ctx->tmp0);
        ctx->err.clear();
    }
    const int64_t kchunk = ((T + parts - 1) / parts + 31) / 32 * 32;
    hipStream_t sg = s;
    if (overlap && (rc = aux_stream(ctx, &sg))) return rc;
    double* G = (double*)ctx->tmp1.ptr;
    // the first sample tile's Gram writes G (every entry of its tile list, in every part)
    if (N == 0 && (rc = fill_f64(ctx, G, (int64_t)parts * W * W, 0.0, s))) return rc;
    const bool valu = gram == BEM_GRAM_FP64_VALU;
    const std::vector<int> tiles = valu ? out_tiles : gram_work(out_tiles, parts);
    const int ntiles = (int)tiles.size() / (valu ? 2 : 3);
    if ((rc = upload_tiles(ctx, ctx->tilew, tiles, W, H, gram, parts, s))) return rc;
    const int* dtiles = (const int*)ctx->tilew.buf.ptr;
    // tmp5: the vertex table, then the near-pair corrections and run table of one sample tile
    const int S = ctx->opts.segs_per_handle;
    const size_t vtab_bytes = ((size_t)(S + 1) * 8 * sizeof(float) + 255) / 256 * 256;
    NearList nl{};
    if (mixed && N > 0) {
        if (pre) nl = *pre;
        else if ((rc = near_classify(ctx, ctx->nearf, x, N, H * ctx->opts.segs_per_handle, 0, &nl, s))) return rc;
    }
    const size_t corr_bytes = mixed ? ((size_t)((T + 63) / 64) * nl.slots * kFeatVals * sizeof(float) + 255) / 256 * 256 : 0;
    const size_t runs_bytes = mixed ? ((size_t)((T + 63) / 64) * H * sizeof(int2) + 255) / 256 * 256 : 0;
    if ((rc = ensure(ctx, ctx->tmp5, vtab_bytes + corr_bytes + runs_bytes + 256, s))) return rc;
    float* vtab = (float*)ctx->tmp5.ptr;
    float* corr = mixed ? (float*)((char*)ctx->tmp5.ptr + vtab_bytes) : nullptr;
    int2* runs = mixed ? (int2*)((char*)ctx->tmp5.ptr + vtab_bytes + corr_bytes) : nullptr;
    hipLaunchKernelGGL(k_vertex_table, dim3(blocks_for(S + 1, 64)), dim3(64), 0, s, S, ctx->model, vtab);
    const float4* box = nullptr;        // culling boxes of the segment groups (mixed feature kernel)
    if (mixed && (rc = near_boxes(ctx, H * S, 0, &box, s))) return rc;
    hipEvent_t* evF = ctx->ev;          // features of the tile in buffer b done
    hipEvent_t* evG = ctx->ev + 2;      // Gram of the tile in buffer b done
    if (overlap) {                      // the Gram stream starts after everything queued so far
        if (hipEventRecord(ctx->ev[4], s) != hipSuccess || hipStreamWaitEvent(sg, ctx->ev[4], 0) != hipSuccess)
            return set_error(ctx, BEM_EHIP, "stream fork");
    }
    int it = 0;
    for (int64_t t0 = 0; t0 < N; t0 += T, ++it) {
        const int64_t n = N - t0 < T ? N - t0 : T;
        const double* xt = x + 2 * t0;
        const int buf = overlap ? (it & 1) : 0;
        void* tile = (char*)ctx->tmp0.ptr + (size_t)buf * tile_bytes;
        if (overlap && it >= 2 && hipStreamWaitEvent(s, evG[buf], 0) != hipSuccess)
            return set_error(ctx, BEM_EHIP, "stream wait");
        if (f64) {
            double* Xt = (double*)tile;
            if ((rc = launch_features<double>(ctx, xt, n, H, mixed, true, Xt, nullptr, T, s, &nl, t0, x, corr, vtab, runs,
                                              box)))
                return rc;
            if (n % kGemmPad)
                hipLaunchKernelGGL(k_zero_tail_f64, dim3(blocks_for(W * kGemmPad, 256)), dim3(256), 0, s, Xt, W, T, n);
            {
                ProfScope ps_(ctx, PT_GRAM_F64, s);
                const Gemm64 g{(int)W, (int)W, gemm_pad(n), 1.0, Xt, T, Xt, T, it > 0 ? 1.0 : 0.0, G, W};
                rc = valu ? gemm_f64_valu(ctx, g, s, dtiles, ntiles) : gemm_f64_list(ctx, g, s, dtiles, ntiles, (int)kchunk, W * W);
            }
            if (rc) return rc;
        } else if (gram == BEM_GRAM_FP32_MFMA) {
            float* Xt = (float*)tile;
            if ((rc = launch_features<float>(ctx, xt, n, H, mixed, true, Xt, nullptr, T, s, &nl, t0, x, corr, vtab, runs,
                                             box)))
                return rc;
            if (overlap && (hipEventRecord(evF[buf], s) != hipSuccess || hipStreamWaitEvent(sg, evF[buf], 0) != hipSuccess))
                return set_error(ctx, BEM_EHIP, "stream wait");
            if ((rc = launch_gram_mfma(ctx, gram, Xt, nullptr, T, (int)W, n, dtiles, ntiles, kchunk, G, W * W, it > 0, sg)))
                return rc;
        } else {
            uint16_t* Xh = (uint16_t*)tile;
            uint16_t* Xl = Xh + (size_t)W * T;
            // blocked layout: ld is the row count
            if ((rc = launch_features<uint16_t>(ctx, xt, n, H, mixed, true, Xh, Xl, W, s, &nl, t0, x, corr, vtab, runs,
                                                box)))
                return rc;
            if (n & 31)
                hipLaunchKernelGGL(k_zero_tail, dim3(blocks_for(W * (32 - (n & 31)), 256)), dim3(256), 0, s, Xh, Xl, W, n);
            if (overlap && (hipEventRecord(evF[buf], s) != hipSuccess || hipStreamWaitEvent(sg, evF[buf], 0) != hipSuccess))
                return set_error(ctx, BEM_EHIP, "stream wait");
            if ((rc = launch_gram_mfma(ctx, gram, Xh, Xl, T, (int)W, n, dtiles, ntiles, kchunk, G, W * W, it > 0, sg)))
                return rc;
        }
        if (overlap && hipEventRecord(evG[buf], sg) != hipSuccess) return set_error(ctx, BEM_EHIP, "stream event");
    }
    if (overlap) {                      // join: the caller's stream continues after the last Gram
        if (hipEventRecord(ctx->ev[5], sg) != hipSuccess || hipStreamWaitEvent(s, ctx->ev[5], 0) != hipSuccess)
            return set_error(ctx, BEM_EHIP, "stream join");
    }
    // (1/N) sum over the samples, or (1/norm): the samples drawn over the whole image
    const double sc = N > 0 ? 1.0 / (norm > 0.0 ? norm : (double)N) : 0.0;
    return contract_gram(ctx, H, L, W, G, N > 0 ? parts : 1, ts, dtiles, ntiles, Z, sc, JtJ, s);
}

int launch_vertex_table(bem_ctx* ctx, float* vtab, hipStream_t s)
{
    const int S = ctx->opts.segs_per_handle;
    hipLaunchKernelGGL(k_vertex_table, dim3(blocks_for(S + 1, 64)), dim3(64), 0, s, S, ctx->model, vtab);
    return check_launch(ctx, "vertex table");
}

int gram_tiles_half(const Layout& L, int64_t W) { return (int)gram_tiles(L, (int)W, 256).size() / 2; }

int gram_work_half(bem_ctx* ctx, const Layout& L, int64_t W, int parts, const int** work, int* ntiles, hipStream_t s)
{
    const std::vector<int> w = gram_work(gram_tiles(L, (int)W, 256), parts);
    *ntiles = (int)w.size() / (3 * parts);
    const int rc = upload_tiles(ctx, ctx->halfw, w, W, L.H, BEM_GRAM_BF16X3_MFMA, parts, s);
    *work = (const int*)ctx->halfw.buf.ptr;
    return rc;
}

int run_jacobian(bem_ctx* ctx, const double* theta, int H, const double* x, int64_t N, double* J, hipStream_t s)
{
    int rc;
    const int M = ctx->M;
    const Layout L = layout_of(ctx, H);
    const int nf = (int)L.handle_rows();
    const int64_t W = nf + M;
    if (H == 0 || N == 0) return BEM_OK;
    if ((rc = launch_expand(ctx, theta, H, s))) return rc;
    double* Z = nullptr;
    if ((rc = boundary_derivatives(ctx, H, s, &Z))) return rc;
    // beta rows are transposed and multiplied 16,384 samples at a time: their copy of all samples was as large as the
    // features
    const int64_t ld = N, P = (int64_t)L.params() * H, step = N < 16384 ? N : 16384;
    const int Mp = gemm_pad(M);
    const size_t xs = ((size_t)W * N + 1) / 2 * 2;
    if ((rc = ensure(ctx, ctx->tmp0, (xs + (size_t)step * Mp + (size_t)step * nf) * sizeof(double), s))) return rc;
    double* Xt = (double*)ctx->tmp0.ptr;
    double* Bt = Xt + xs;
    double* BZ = Bt + (size_t)step * Mp;
    if ((rc = launch_features<double>(ctx, x, N, H, false, true, Xt, nullptr, ld, s))) return rc;
    for (int64_t t0 = 0; t0 < N; t0 += step) {
        const int64_t n = N - t0 < step ? N - t0 : step;
        // BZ[t][f] = sum_i beta_i(t) Z[f][i]  (beta rows of Xt transposed)
        hipLaunchKernelGGL(k_pad, dim3(blocks_for(n * Mp, 256)), dim3(256), 0, s, (const double*)(Xt + (size_t)nf * ld + t0), ld,
                           true, n, M, n, Mp, Bt);
        if ((rc = gemm_f64(ctx, Gemm64{(int)n, nf, Mp, 1.0, Bt, Mp, Z, Mp, 0.0, BZ, nf}, 1, s))) return rc;
        hipLaunchKernelGGL(k_assemble_jacobian, dim3(blocks_for(P, 256), n), dim3(256), 0, s, Xt + t0, ld, BZ, L, n,
                           J + (size_t)t0 * 3 * P);
    }
    return check_launch(ctx, "jacobian");
}

}  // namespace bem
