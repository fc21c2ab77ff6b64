// sweep_f64.hip - float64 forward sweep u(x) = cbar + sum_j beta_j(x) U_j + f(x): every pair in float64.
//
// Few samples: blocks of 256 samples times chunks of the tables (k_sweep_f64), whose sums are added in a
// fixed order (k_sweep_f64_sum), so that 16,384 samples still fill the chip.  Many samples (cells.hpp):
// the segments and elements far from a cell are summed at its 256 nodes or those of a cell above it (k_far_nodes_f64), turned into
// Chebyshev coefficients (k_far_coef_f64) and expanded at its samples, which take only the near ones pair
// by pair (k_sweep_cells_f64).  Results are reproducible: every sum has a fixed order.
// Bound by the float64 vector ALUs (about 155 instructions a segment pair, 55 an element's).  Measured
// against one thread a sample over all pairs, one MI355X: 512 segments and 262,144 samples 1.75 -> 0.43 ms
// a call; 128 segments and 16,384 samples (the sweep) 564 -> 83 us; errors against float64 sums of the same
// formulas 7e-16 before and after.
#include "cells.hpp"

namespace bem {

namespace {

struct Tables64 {
    const double* seg;
    const double* el;
    int K, M;
    double eps2;
};

__device__ inline void add_segment(const Tables64& t, int k, double X, double Y, double (&f)[3])
{
    const double* s = t.seg + (size_t)k * kSegStride;
    const Moments<double> m = seg_moments<double, DevF64>(load_geom(s), X, Y, t.eps2);
#pragma unroll
    for (int c = 0; c < 3; ++c)
        f[c] += m.da * s[kWdA + c] + m.db * s[kWdB + c] + m.sa * s[kWcA + c] + m.sb * s[kWcB + c];
}
__device__ inline void add_element(const Tables64& t, int j, double X, double Y, double (&f)[3])
{
    const double* e = t.el + (size_t)j * kElemStride;
    const double beta = element_beta<double, DevF64>(e[0], e[1], e[2], e[3], X, Y);
    f[0] += beta * e[4]; f[1] += beta * e[5]; f[2] += beta * e[6];
}

// Chunk y takes groups [y gpc, (y + 1) gpc) of gs segments, then of gs elements.  part == null (one chunk):
// u is written here.
__global__ void __launch_bounds__(256) k_sweep_f64(const double* __restrict__ x, int64_t N, Tables64 t, int gs, int gpc,
                                                   double c0, double c1, double c2, double* __restrict__ part,
                                                   double* __restrict__ u)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= N) return;
    const double X = x[2 * i], Y = x[2 * i + 1];
    const int nsg = (t.K + gs - 1) / gs;
    const int g0 = blockIdx.y * gpc, g1 = g0 + gpc;
    const int k1 = g1 < nsg ? g1 * gs : t.K;
    double f[3] = {0.0, 0.0, 0.0}, b[3] = {0.0, 0.0, 0.0};
    for (int k = g0 * gs; k < k1; ++k) add_segment(t, k, X, Y, f);
    const int j1 = (g1 - nsg) * gs < t.M ? (g1 - nsg) * gs : t.M;
#pragma unroll 2
    for (int j = (g0 > nsg ? g0 - nsg : 0) * gs; j < j1; ++j) add_element(t, j, X, Y, b);
    const double c[3] = {c0, c1, c2};
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        if (part) part[(size_t)blockIdx.y * 3 * N + 3 * i + q] = b[q] + f[q];
        else u[3 * i + q] = c[q] + b[q] + f[q];
    }
}

__global__ void __launch_bounds__(256) k_sweep_f64_sum(const double* __restrict__ part, int nparts, int64_t N, double c0,
                                                       double c1, double c2, double* __restrict__ u)
{
    __shared__ double red[3][64];
    const int64_t i = (int64_t)blockIdx.x * 64 + (threadIdx.x & 63);
    const double v = sum_chunks(part, nparts, 3 * N, i, red);
    if (threadIdx.x < 64 && i < 3 * N) u[i] = (i % 3 == 0 ? c0 : (i % 3 == 1 ? c1 : c2)) + v;
}

// The tables' coordinates from the grid's origin: a node's place in the domain rounds with the domain's distance from 0 (at
// 1e4 the colours were off by 9e-13, now 7e-16), its place in the grid and the records' differences to the origin do not.
__global__ void __launch_bounds__(256) k_relative(Tables64 t, double x0, double y0, double* __restrict__ seg,
                                                  double* __restrict__ el)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= t.K + t.M) return;
    const bool s = i < t.K;
    const int n = s ? kSegStride : kElemStride;
    const double* from = s ? t.seg + (size_t)i * kSegStride : t.el + (size_t)(i - t.K) * kElemStride;
    double* to = s ? seg + (size_t)i * kSegStride : el + (size_t)(i - t.K) * kElemStride;
    for (int k = 0; k < n; ++k) to[k] = from[k] - (k < (s ? 4 : 2) ? (k & 1 ? y0 : x0) : 0.0);
}

constexpr int kLowParts = 4;

// Far sums at the nodes, thread = node, tables and grid from the grid's origin.  First the top level, chunk y of it words [y gpc, (y + 1) gpc), sums to
// part [y][cell]; then kLowParts blocks a row of the levels below,
// which take its words by turns, sums to low [part][row].  Cells without samples have no
// far bits.
__global__ void __launch_bounds__(256) k_far_nodes_f64(CellPlan p, Tables64 t, int gpc, int nparts,
                                                       double* __restrict__ part, double* __restrict__ low)
{
    const CellLevels& lv = p.lv;
    const int ntop = lv.top_cells(), n = threadIdx.x;
    const bool top = (int)blockIdx.x < ntop * nparts;
    const int nlow = lv.low_rows(), lb = (int)blockIdx.x - ntop * nparts;
    const int y = top ? (int)blockIdx.x / ntop : lb / nlow, i = top ? (int)blockIdx.x % ntop : lb % nlow;
    if (!top && i == p.grid.nc) return;
    const int row = top ? lv.base[lv.n - 1] + i : i;
    int l, cx, cy;
    level_cell(lv, row, l, cx, cy);
    double X, Y;
    level_node<kFarQ64>(p.grid, l, cx, cy, n, X, Y);
    const uint32_t* far_bits = p.far + (size_t)row * p.words;
    const int w0 = top ? y * gpc : 0, w1 = !top || w0 + gpc > p.words ? p.words : w0 + gpc;
    double f[3] = {0.0, 0.0, 0.0};
    int turn = 0;
    for (int w = w0; w < w1; ++w) {
        const bool seg = w < p.seg_words;
        const int i0 = 32 * (seg ? w : w - p.seg_words);
        uint32_t far = far_bits[w];
        if (!top && far != 0 && (turn++ & (kLowParts - 1)) != y) continue;
        for (; far; far &= far - 1u) {
            const int k = i0 + __builtin_ctz(far);
            if (seg) add_segment(t, k, X, Y, f);
            else add_element(t, k, X, Y, f);
        }
    }
    double* o = top ? part + ((size_t)y * ntop + i) * 3 * kFarNodes64 : low + ((size_t)y * nlow + row) * 3 * kFarNodes64;
    for (int q = 0; q < 3; ++q) o[q * kFarNodes64 + n] = f[q];
}

// Node sums to Chebyshev coefficients, block (cell, channel): as k_far_coef, 16 nodes a side.
__global__ void __launch_bounds__(256) k_far_coef_f64(const double* __restrict__ part, int nparts,
                                                      const double* __restrict__ low, CellPlan pl,
                                                      double* __restrict__ coef)
{
    constexpr int Q = kFarQ64;
    __shared__ double v[kFarNodes64], h[kFarNodes64], cs[4 * Q], I[2][Q][Q];
    const CellLevels& lv = pl.lv;
    const int c = blockIdx.x, ch = blockIdx.y, n = threadIdx.x, a = n & (Q - 1), b = n / Q;
    if (pl.off[c + 1] == pl.off[c]) return;
    if (n < 4 * Q) cs[n] = cospi((double)n / (2.0 * Q));
    const int cx = c % lv.nx[0], cy = c / lv.nx[0], top = lv.n - 1, ntop = lv.top_cells();
    const int ct = (cy >> top) * lv.nx[top] + (cx >> top);
    double s = 0.0;
#pragma unroll 4
    for (int p = 0; p < nparts; ++p) s += part[(((size_t)p * ntop + ct) * 3 + ch) * kFarNodes64 + n];
    __syncthreads();
    if (top > 0) child_matrix<Q>(n, 256, cs, I);
    for (int l = top - 1; l >= 0; --l) {
        const int sx = (cx >> l) & 1, sy = (cy >> l) & 1;
        v[n] = s;
        __syncthreads();
        double r = 0.0;
        for (int i = 0; i < Q; ++i) r += I[sx][a][i] * v[Q * b + i];
        h[n] = r;
        __syncthreads();
        r = 0.0;
        for (int j = 0; j < Q; ++j) r += I[sy][b][j] * h[Q * j + a];
        for (int p = 0; p < kLowParts; ++p)
            r += low[(((size_t)p * lv.low_rows() + level_row(lv, l, cx >> l, cy >> l)) * 3 + ch) * kFarNodes64 + n];
        s = r;
    }
    v[n] = s;
    __syncthreads();
    double r = 0.0;
    for (int i = 0; i < Q; ++i) r += v[Q * b + i] * cs[(a * (2 * i + 1)) & (4 * Q - 1)];
    h[n] = r * (a == 0 ? 1.0 / Q : 2.0 / Q);
    __syncthreads();
    r = 0.0;
    for (int j = 0; j < Q; ++j) r += h[Q * j + a] * cs[(b * (2 * j + 1)) & (4 * Q - 1)];
    coef[((size_t)c * 3 + ch) * kFarNodes64 + n] = r * (b == 0 ? 1.0 / Q : 2.0 / Q);
}

// A wavefront of up to 64 samples of one cell: its near segments and elements, then the expansion.
__global__ void __launch_bounds__(256) k_sweep_cells_f64(CellPlan p, Tables64 t, const double* __restrict__ coef,
                                                         double c0, double c1, double c2, double* __restrict__ u)
{
    const int w = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const int nl = p.grid.nc + 1;
    if (w >= p.wave0[nl]) return;
    const int c = unit_label(p.wave0, nl, w);
    const int i = p.off[c] + (w - p.wave0[c]) * 64 + lane;
    if (i >= p.off[c + 1]) return;
    const double X = p.xs[2 * (size_t)i], Y = p.xs[2 * (size_t)i + 1];
    const uint32_t* row = p.bits + (size_t)c * p.words;
    double f[3] = {0.0, 0.0, 0.0}, b[3] = {0.0, 0.0, 0.0};
    for (int q = 0; q < p.seg_words; ++q)
        for (uint32_t word = row[q]; word; word &= word - 1u) add_segment(t, 32 * q + __builtin_ctz(word), X, Y, f);
    for (int q = p.seg_words; q < p.words; ++q)
        for (uint32_t word = row[q]; word; word &= word - 1u)
            add_element(t, 32 * (q - p.seg_words) + __builtin_ctz(word), X, Y, b);
    double far[3] = {0.0, 0.0, 0.0};
    if (c < p.grid.nc) {
        // (from the grid's origin, as the nodes)
        const double cx = (double)(c % p.grid.nx) * p.grid.h, cy = (double)(c / p.grid.nx) * p.grid.h;
        double Ta[kFarQ64];
        cheb_values<double, kFarQ64>(((X - p.grid.x0) - cx) * (2.0 * p.grid.inv_h) - 1.0, Ta);
        const double y = ((Y - p.grid.y0) - cy) * (2.0 * p.grid.inv_h) - 1.0;
        const double* cf = coef + (size_t)c * 3 * kFarNodes64;
        double T0 = 1.0, T1 = y;                     // T_j(y), T_{j+1}(y)
        for (int j = 0; j < kFarQ64; ++j) {
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const double* r = cf + q * kFarNodes64 + kFarQ64 * j;
                double v = r[0];
#pragma unroll
                for (int k = 1; k < kFarQ64; ++k) v += r[k] * Ta[k];
                far[q] += T0 * v;
            }
            const double T2 = 2.0 * y * T1 - T0;
            T0 = T1;
            T1 = T2;
        }
    }
    const size_t o = 3 * (size_t)p.perm[i];
    const double cb[3] = {c0, c1, c2};
#pragma unroll
    for (int q = 0; q < 3; ++q) u[o + q] = cb[q] + ((b[q] + f[q]) + far[q]);
}

}  // namespace

int launch_sweep_f64(bem_ctx* ctx, const double* x, int64_t N, int K, const double* cbar, double* u, hipStream_t s)
{
    if (N == 0) return BEM_OK;
    int rc;
    const int M = ctx->M;
    const Tables64 t{(const double*)ctx->seg64.ptr, (const double*)ctx->elem64.ptr, K, M, ctx->opts.eps * ctx->opts.eps};
    const int64_t groups = (K + 31) / 32 + (M + 31) / 32;
    Grouping g = cells_for(ctx, N, K, kFarQ64, 1.0, 1e7, 1.0, 3000.0);
    ProfScope ps_(ctx, PT_SWEEP_F64, s);
    CellPlan p;
    int nc = 0, ntop = 0, nlow = 0, gpc = 0, nparts = 0;
    size_t pb = 0, lb = 0, cb = 0;
    if (g.g) {
        rc = cell_plan(ctx, x, N, g, &p, s);
        if (!rc) rc = cell_bits(ctx, &p, K, M, false, s);
        if (!rc) {
            nc = p.grid.nc;
            ntop = p.lv.top_cells();
            nlow = p.lv.low_rows();
            gpc = groups_per_chunk(groups, ntop);
            nparts = (int)((groups + gpc - 1) / gpc);
            const size_t cell = 3 * kFarNodes64 * sizeof(double);
            pb = (size_t)nparts * ntop * cell;
            lb = (size_t)kLowParts * nlow * cell;
            cb = nc * cell;
            const bool away = p.grid.x0 != 0.0 || p.grid.y0 != 0.0;
            const size_t rb = away ? ((size_t)K * kSegStride + (size_t)M * kElemStride) * sizeof(double) : 0;
            rc = ensure(ctx, ctx->farw, pb + lb + cb + rb, s);
        }
        if (rc && rc != BEM_ENOMEM) return rc;
        if (rc) {                            // no memory for them: the direct sums
            ctx->err.clear();
            g.g = 0;
        }
    }
    if (g.g == 0) {
        const int64_t nb = blocks_for(N, 256);
        const int gs = direct_group(nb, K, M);
        const int64_t groups = blocks_for(K, gs) + blocks_for(M, gs);
        gpc = groups_per_chunk(groups, nb);
        nparts = (int)((groups + gpc - 1) / gpc);
        double* part = nullptr;
        if (nparts > 1) {
            rc = ensure(ctx, ctx->farw, (size_t)nparts * 3 * N * sizeof(double), s);
            if (rc && rc != BEM_ENOMEM) return rc;
            if (rc) {                        // no memory for the chunks' sums: one chunk
                ctx->err.clear();
                gpc = (int)groups;
                nparts = 1;
            } else {
                part = (double*)ctx->farw.ptr;
            }
        }
        hipLaunchKernelGGL(k_sweep_f64, dim3(nb, nparts), dim3(256), 0, s, x, N, t, gs, gpc, cbar[0], cbar[1], cbar[2], part,
                           u);
        if (part)
            hipLaunchKernelGGL(k_sweep_f64_sum, dim3(blocks_for(3 * N, 64)), dim3(256), 0, s, (const double*)part, nparts,
                               N, cbar[0], cbar[1], cbar[2], u);
        return check_launch(ctx, "sweep_f64");
    }
    double* part = (double*)ctx->farw.ptr;
    double* low = (double*)((char*)ctx->farw.ptr + pb);
    double* coef = (double*)((char*)ctx->farw.ptr + pb + lb);
    Tables64 tf = t;
    CellPlan pf = p;
    pf.grid.x0 = pf.grid.y0 = 0.0;
    if (p.grid.x0 != 0.0 || p.grid.y0 != 0.0) {
        double* seg = (double*)((char*)ctx->farw.ptr + pb + lb + cb);
        double* el = seg + (size_t)K * kSegStride;
        hipLaunchKernelGGL(k_relative, dim3(blocks_for(K + M, 256)), dim3(256), 0, s, t, p.grid.x0, p.grid.y0, seg, el);
        tf.seg = seg;
        tf.el = el;
    }
    hipLaunchKernelGGL(k_far_nodes_f64, dim3(kLowParts * nlow + ntop * nparts), dim3(256), 0, s, pf, tf, gpc, nparts, part, low);
    hipLaunchKernelGGL(k_far_coef_f64, dim3(nc, 3), dim3(256), 0, s, (const double*)part, nparts, (const double*)low, p, coef);
    hipLaunchKernelGGL(k_sweep_cells_f64, dim3((p.max_waves + 3) / 4), dim3(256), 0, s, p, t, (const double*)coef, cbar[0],
                       cbar[1], cbar[2], u);
    return check_launch(ctx, "sweep_cells_f64");
}

}  // namespace bem
