// cells.hpp - samples grouped by the cells of a square grid, and the far field of a cell by
// interpolation (cells.hip).
//
// Seen from one cell of the grid, the handle term of every segment that stays kFarCells cell widths
// away is a smooth function of the sample: it is evaluated at the kFarQ x kFarQ Chebyshev nodes of
// the cell instead of at the cell's samples, and expanded there in products T_a(xi) T_b(eta) of
// Chebyshev polynomials.  The nearest singularity in either coordinate lies at least kFarCells cell
// widths = 4 half widths off the cell, on an ellipse of parameter 4 + sqrt(17) = 8.1, so that eight
// nodes a side leave a relative error of a few 1e-9 in the field and a few 1e-8 in its derivatives
// with respect to the end points (measured against float64 sums over cells of 1/16 and 1/32 and
// segments of 1/100): below the float32 rounding of a pair.
// The other pairs of the cell, and those the mixed precision evaluates in float64, are evaluated
// sample by sample.
//
// Levels.  2 x 2 cells form a cell of the next level, up to kMaxLevels of them.  A segment far from a cell is
// summed at the nodes of the largest cell above it that it is far from (the top level sums every far segment, the
// levels below only those near the parent, of some 75 cell areas), and node sums are carried down exactly: a
// polynomial's values at the children's nodes.  Far from the parent implies far from the child (the bits say so by
// construction), so that every pair is counted once.
#pragma once

#include "common.hpp"
#include "sweep_common.hpp"

namespace bem {

constexpr int kFarQ = 8;                       // nodes a side: 64 nodes, one wavefront
constexpr int kFarNodes = kFarQ * kFarQ;
// The float64 sweep takes the same far set with 16 nodes a side: 8.1^-16 = 3e-15 of a segment's part,
// 1e-14 and less against direct sums (their own rounding).
constexpr int kFarQ64 = 16;
constexpr int kFarNodes64 = kFarQ64 * kFarQ64;
constexpr double kFarCells = 2.0;              // a segment nearer than this many cell widths is not far
constexpr int kMaxGrid = 64;                   // cells a side
constexpr int kMaxCellLabels = kMaxGrid * kMaxGrid + 1;

// Square cells of width h from (x0, y0); label nc = nx ny holds the samples outside the grid (and
// those that are not finite): no segment is far for them.
struct CellGrid {
    double x0, y0, h, inv_h;
    int nx, ny, nc;
};

// Levels of the grid: rows of the bit tables and node sums, level 0 (the cells, then the stray label nc) first; level
// l's cells from base[l] on.
constexpr int kMaxLevels = 3;
struct CellLevels {
    int n = 1, rows = 0;
    int nx[kMaxLevels] = {}, ny[kMaxLevels] = {}, base[kMaxLevels] = {};
    __host__ __device__ int top_cells() const { return nx[n - 1] * ny[n - 1]; }
    __host__ __device__ int low_rows() const { return n > 1 ? base[n - 1] : 0; }         // rows below the top level
};
__device__ inline void level_cell(const CellLevels& lv, int row, int& l, int& cx, int& cy)
{
    l = 0;
    while (l + 1 < lv.n && row >= lv.base[l + 1]) ++l;
    cx = (row - lv.base[l]) % lv.nx[l];
    cy = (row - lv.base[l]) / lv.nx[l];
}
__device__ inline int level_row(const CellLevels& lv, int l, int cx, int cy) { return lv.base[l] + cy * lv.nx[l] + cx; }
// whether a cell of level l holds samples (off: first sample of every level-0 cell)
__device__ inline bool level_used(const CellLevels& lv, const int* __restrict__ off, int l, int cx, int cy)
{
    const int x0 = cx << l, x1 = (cx + 1) << l < lv.nx[0] ? (cx + 1) << l : lv.nx[0];
    const int y1 = (cy + 1) << l < lv.ny[0] ? (cy + 1) << l : lv.ny[0];
    for (int y = cy << l; y < y1; ++y)
        if (off[y * lv.nx[0] + x1] > off[y * lv.nx[0] + x0]) return true;
    return false;
}

__device__ inline int cell_of(const CellGrid& g, double X, double Y)
{
    const double fx = (X - g.x0) * g.inv_h, fy = (Y - g.y0) * g.inv_h;
    if (!(fx >= 0.0 && fy >= 0.0 && fx <= (double)g.nx && fy <= (double)g.ny)) return g.nc;
    const int cx = (int)fx < g.nx ? (int)fx : g.nx - 1;
    const int cy = (int)fy < g.ny ? (int)fy : g.ny - 1;
    return cy * g.nx + cx;
}
__device__ inline void cell_corner(const CellGrid& g, int c, double& X, double& Y)
{
    X = g.x0 + (double)(c % g.nx) * g.h;
    Y = g.y0 + (double)(c / g.nx) * g.h;
}
// Chebyshev node i of Q: cos((2 i + 1) pi / (2 Q))
template <int Q> __device__ inline double cheb_node(int i);
template <> __device__ inline double cheb_node<8>(int i)
{
    constexpr double t[4] = {0.98078528040323044913, 0.83146961230254523708, 0.55557023301960222474,
                             0.19509032201612826785};
    return i < 4 ? t[i] : -t[7 - i];
}
template <> __device__ inline double cheb_node<16>(int i)
{
    constexpr double t[8] = {0.99518472667219688624, 0.95694033573220886494, 0.88192126434835502971,
                             0.77301045336273696081, 0.63439328416364549822, 0.47139673682599764856,
                             0.29028467725446236764, 0.098017140329560601994};
    return i < 8 ? t[i] : -t[15 - i];
}
template <int Q>
__device__ inline void cell_node(const CellGrid& g, int c, int node, double& X, double& Y)
{
    cell_corner(g, c, X, Y);
    X += 0.5 * g.h * (1.0 + cheb_node<Q>(node & (Q - 1)));
    Y += 0.5 * g.h * (1.0 + cheb_node<Q>(node / Q));
}
template <int Q>
__device__ inline void level_node(const CellGrid& g, int l, int cx, int cy, int node, double& X, double& Y)
{
    const double h = g.h * (double)(1 << l);
    X = g.x0 + (double)cx * h + 0.5 * h * (1.0 + cheb_node<Q>(node & (Q - 1)));
    Y = g.y0 + (double)cy * h + 0.5 * h * (1.0 + cheb_node<Q>(node / Q));
}
// T_0 .. T_{Q-1} at t
template <class T, int Q>
__device__ inline void cheb_values(T t, T (&v)[Q])
{
    v[0] = T(1);
    v[1] = t;
#pragma unroll
    for (int k = 2; k < Q; ++k) v[k] = T(2) * t * v[k - 1] - v[k - 2];
}

// Values of a polynomial of degree Q - 1 a side, given at a cell's Q x Q nodes, at those of its child on side s (0 lower,
// 1 upper) of one axis: I[s][i][n] = l_n((t_i + 2 s - 1) / 2).  Threads t of n; cs[k] = cos(k pi / (2 Q)), k < 4 Q.
template <int Q>
__device__ inline void child_matrix(int t, int n, const double* cs, double (*I)[Q][Q])
{
    for (int e = t; e < 2 * Q * Q; e += n) {
        const int s = e / (Q * Q), i = e / Q % Q, k = e % Q;
        double T[Q];
        cheb_values<double, Q>(0.5 * (cheb_node<Q>(i) + 2.0 * s - 1.0), T);
        double v = 1.0 / Q;
        for (int a = 1; a < Q; ++a) v += 2.0 / Q * T[a] * cs[(a * (2 * k + 1)) & (4 * Q - 1)];
        I[s][i][k] = v;
    }
}

// Cells a side of the finest level, levels; g = 0: direct sums.
struct Grouping {
    int g = 0, levels = 1;
};

// The samples of a call in cell order, on the device (workspace of the context, valid until the
// next plan): sorted sample i is sample perm[i]; cell c holds the sorted samples off[c] ..
// off[c + 1] - 1 and the wavefronts wave0[c] .. wave0[c + 1] - 1 of 64 of them (the last one
// short), and likewise the runs run0[c] .. of `run` samples.
struct CellPlan {
    CellGrid grid;
    CellLevels lv;
    const int* perm = nullptr;
    const double* xs = nullptr;
    const int* off = nullptr;
    const int* wave0 = nullptr;
    const int* run0 = nullptr;
    int run = 64;
    int64_t max_waves = 0, max_runs = 0;       // bounds known on the host
    // near bits of the current tables: word w of cell c at bits[c * words + w]; the segments' words
    // first (bit k % 32 of word k / 32), then the outer elements'
    const uint32_t* bits = nullptr;
    const uint32_t* far = nullptr;             // the pairs a row's nodes take; likewise, row r of every level at far[r * words]
    int seg_words = 0, words = 0;
};

// The grid for N samples with q nodes a side, g = 0 where the direct sums are the better choice; ratio: time of a near
// pair over that of a far one; worth: pairs that take as long as the plan, the bits and the node sums' launches; low:
// time of a far pair below the top level over one at it; row: pairs that take as long as a row's own work; places:
// where lanes are segments, how many places 64 of them lie in.
Grouping cells_for(const bem_ctx* ctx, int64_t N, int K, int q, double ratio, double worth, double low, double row,
                   double places = 1.0);
// Cells a side where every cell costs q^2 pairs of its own (one level)
int cells_one_level(const bem_ctx* ctx, int64_t N, int q, double ratio);
int cell_plan(bem_ctx* ctx, const double* x, int64_t N, Grouping g, CellPlan* p, hipStream_t s);
// near and far bits of the segment and element tables (expanded before) for every cell of the plan; mixed: the
// pairs of the near radius as well
int cell_bits(bem_ctx* ctx, CellPlan* p, int K, int M, bool mixed, hipStream_t s);

// groups of 32 segments or elements a chunk so that `blocks` blocks a chunk make about 2048 blocks in all
inline int groups_per_chunk(int64_t groups, int64_t blocks)
{
    const int64_t n = (groups * blocks + 2047) / 2048;
    return (int)(n < 1 ? 1 : (n > groups ? groups : n));
}

// Segments or elements a group of the direct sums over nb blocks of samples: 32, or 8 where those leave most of the
// chip idle (1,000 samples, 128 segments, 1,024 elements: 144 blocks, sweep 16 us; 576 blocks, 8 us).
inline int direct_group(int64_t nb, int K, int M) { return nb * (((int64_t)K + M + 63) / 32) < 512 ? 8 : 32; }

// Sum of the chunks' partial results i (chunks n apart): a block of 256 threads 64 results, each wavefront every fourth
// chunk, in a fixed order; the result is in the first wavefront.
__device__ inline double sum_chunks(const double* __restrict__ part, int nparts, int64_t n, int64_t i, double (*red)[64])
{
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    double v = 0.0;
    if (i < n) {
#pragma unroll 8
        for (int p = w; p < nparts; p += 4) v += part[(size_t)p * n + i];
    }
    if (w > 0) red[w - 1][lane] = v;
    __syncthreads();
    return w == 0 ? ((v + red[0][lane]) + red[1][lane]) + red[2][lane] : 0.0;
}

// label of unit u in a first-unit table t[0 .. nl] (t[nl] = number of units > u)
__device__ inline int unit_label(const int* __restrict__ t, int nl, int u)
{
    int lo = 0, hi = nl;                        // t[lo] <= u < t[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (t[mid] <= u) lo = mid;
        else hi = mid;
    }
    return lo;
}

}  // namespace bem
