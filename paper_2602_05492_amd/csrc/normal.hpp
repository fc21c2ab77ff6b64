// normal.hpp - layout of the normal equations' feature rows and the pieces shared by the two ways of
// forming their Gram: over all samples (jtj.hip) and over cells (jtj_cells.hip).
#pragma once

#include <vector>

#include "common.hpp"
#include "sweep_common.hpp"

namespace bem {

__device__ inline uint16_t bf16_bits(float v)
{
    // round to nearest even (inputs are finite)
    const uint32_t u = __float_as_uint(v);
    return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}
__device__ inline float bf16_value(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// Feature layout of the normal equations: G geometry rows per handle and channel, C
// channel-shared colour rows per handle, H handles (the rows of Xt are
// [g_0 (GH) | g_1 | g_2 | e (CH) | beta (M)]).
struct Layout {
    int G, C, H;
    int64_t Gp;     // rows of one channel's geometry block in Xt (G H rounded up to the Gram tile)
    __host__ __device__ int64_t geo() const { return (int64_t)G * H; }
    __host__ __device__ int64_t handle_rows() const { return 3 * Gp + (int64_t)C * H; }
    __host__ __device__ int compact() const { return (G + C) * H; }
    __host__ __device__ int params() const { return G + 3 * C; }
    // row of Xt of compact index a of channel c ([g_c | e | beta])
    __host__ __device__ int64_t row(int a, int c) const
    {
        return a < geo() ? (int64_t)c * Gp + a : 3 * Gp + (a - geo());
    }
};

// Adds one float32 pair to a handle's features, by quadrature: moments into col, the channels' end-point
// gradients chained with the vertex weights Va (a end) and Vb (b end) into geo.  A masked pair (on = false)
// is taken at a point eight lengths beside the segment and counts zero times.
template <int NQ>
__device__ __forceinline__ void add_pair_features(const float* __restrict__ s, const float* __restrict__ Va,
                                                  const float* __restrict__ Vb, float X, float Y, float eps2f, bool on,
                                                  float (&geo)[3][8], float (&col)[4])
{
    const SegGeom<float> g = load_geom(s);
    const QuadSums<float> q = quad_sums<float, DevF32, NQ, true>(g, on ? X : g.ax - 8.0f * g.vy,
                                                                 on ? Y : g.ay + 8.0f * g.vx, eps2f);
    const float one = on ? 1.0f : 0.0f;
    const Moments<float> m = quad_moments(q, s[kLen] * one);
    const float da = m.da * one, db = m.db * one;
    const float ta = Va[4], ua = Va[5], tb = Vb[4], ub = Vb[5];
    col[0] += da * ua + db * ub;
    col[1] += da * ta + db * tb;
    col[2] += m.sa * ua + m.sb * ub;
    col[3] += m.sa * ta + m.sb * tb;
    float wa[4], wb[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        wa[k] = Va[k] * one;
        wb[k] = Vb[k] * one;
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const Grad4<float> gr = quad_gradient(g, q, s[kLen], s[kILen], s[kWdA + c], s[kWdB + c], s[kWcA + c], s[kWcB + c]);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            geo[c][2 * k] += wa[k] * gr.ax + wb[k] * gr.bx;
            geo[c][2 * k + 1] += wa[k] * gr.ay + wb[k] * gr.by;
        }
    }
}


// jtj.hip
Layout layout_of(const bem_ctx* ctx, int H);
// Z = A+ dF/dtheta, transposed: [handle rows][M padded by zeros to kGemmPad] -> ctx->tmp4
int boundary_derivatives(bem_ctx* ctx, int H, hipStream_t s, double** Zout);
int launch_vertex_table(bem_ctx* ctx, float* vtab, hipStream_t s);
// work list of 256 x 256 tiles in parts (or runs of columns), part-major, on the device
int gram_work_half(bem_ctx* ctx, const Layout& L, int64_t W, int parts, const int** work, int* ntiles, hipStream_t s);
int gram_tiles_half(const Layout& L, int64_t W);            // tiles of that list
// J^T J of the partial Grams G [parts][W][W]
int contract_gram(bem_ctx* ctx, int H, const Layout& L, int64_t W, double* G, int parts, int ts, const int* work, int nwork,
                  const double* Z, double sc, double* JtJ, hipStream_t s);
// jtj_cells.hip: J^T J of the mixed LM step over cells; *done = false where the samples are better taken
// one by one (nothing is written then).  Synchronises the stream.
int run_jtj_cells(bem_ctx* ctx, const double* theta, int H, const double* x, int64_t N, double* JtJ, double norm,
                  bool* done, hipStream_t s);
// gram_mfma.hip
int launch_gram_half(bem_ctx* ctx, const uint16_t* Yh, const uint16_t* Yl, int W, int64_t n, const float* rscale,
                     const int* work, int runs, int ntiles, int64_t kchunk, float* part, double* G, bool accumulate,
                     hipStream_t s);
int launch_gram_cells(bem_ctx* ctx, const uint16_t* Eh, const uint16_t* El, const uint16_t* Z, int64_t zstep,
                      const CellInfo* ci, int nc, const int* hl, const int* el, int H, int M, const Layout& L, int64_t W,
                      const int* work, int nwork, double* G, hipStream_t s);

}  // namespace bem
