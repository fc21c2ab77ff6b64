// cells.hip - the cell plan of the mixed sweeps: samples grouped by grid cell (a stable counting
// sort without readback) and, per cell, which segments and outer elements are too near for its
// interpolated far field.
#include <algorithm>
#include <cmath>

#include "cells.hpp"

#include <cmath>

namespace bem {

namespace {

// Histogram of the cell labels of one chunk of samples.
__global__ void __launch_bounds__(256) k_cell_hist(const double* __restrict__ x, int64_t N, int chunk, CellGrid g,
                                                   int nb, int* __restrict__ cnt)
{
    __shared__ int h[kMaxCellLabels];
    for (int d = threadIdx.x; d <= g.nc; d += 256) h[d] = 0;
    __syncthreads();
    const int64_t lo = (int64_t)blockIdx.x * chunk, hi = lo + chunk < N ? lo + chunk : N;
    for (int64_t i = lo + threadIdx.x; i < hi; i += 256) {
        atomicAdd(&h[cell_of(g, x[2 * i], x[2 * i + 1])], 1);
    }
    __syncthreads();
    for (int d = threadIdx.x; d <= g.nc; d += 256) cnt[(size_t)d * nb + blockIdx.x] = h[d];
}

__device__ inline int wave_scan(int v)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int w = __shfl_up(v, o);
        if (lane >= o) v += w;
    }
    return v;
}

// Per label the exclusive scan of its chunk counts, in place, and the label's total: a wavefront a
// label.
__global__ void __launch_bounds__(256) k_cell_scan(int* __restrict__ cnt, int nlab, int nb, int* __restrict__ total)
{
    const int d = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (d >= nlab) return;
    int run = 0;
    for (int b0 = 0; b0 < nb; b0 += 64) {
        const int b = b0 + lane;
        const int c = b < nb ? cnt[(size_t)d * nb + b] : 0;
        const int s = wave_scan(c);
        if (b < nb) cnt[(size_t)d * nb + b] = run + s - c;
        run += __shfl(s, 63);
    }
    if (lane == 0) total[d] = run;
}

// First sample, first wavefront and first run of every label (one block, five labels a thread).
__global__ void __launch_bounds__(1024) k_cell_offsets(const int* __restrict__ total, int nlab, int run,
                                                       int* __restrict__ off, int* __restrict__ wave0,
                                                       int* __restrict__ run0)
{
    constexpr int kEach = (kMaxCellLabels + 1 + 1023) / 1024;
    __shared__ int part[3][16];
    const int t = threadIdx.x, w = t >> 6;
    int v[3][kEach], s[3] = {0, 0, 0};
#pragma unroll
    for (int k = 0; k < kEach; ++k) {
        const int d = kEach * t + k;
        const int n = d < nlab ? total[d] : 0;
        v[0][k] = n;
        v[1][k] = (n + 63) / 64;
        v[2][k] = (n + run - 1) / run;
        for (int q = 0; q < 3; ++q) s[q] += v[q][k];
    }
    int e[3];
    for (int q = 0; q < 3; ++q) {
        const int inc = wave_scan(s[q]);
        if ((t & 63) == 63) part[q][w] = inc;
        e[q] = inc - s[q];
    }
    __syncthreads();
    int* out[3] = {off, wave0, run0};
    for (int q = 0; q < 3; ++q) {
        for (int k = 0; k < w; ++k) e[q] += part[q][k];
#pragma unroll
        for (int k = 0; k < kEach; ++k) {
            if (kEach * t + k <= nlab) out[q][kEach * t + k] = e[q];
            e[q] += v[q][k];
        }
    }
}

// Stable scatter of one chunk: 64 samples at a time take consecutive places of their labels in lane
// order (equal labels found by one ballot per label bit), the block's wavefronts in turn.
__global__ void __launch_bounds__(256) k_cell_scatter(const double* __restrict__ x, int64_t N, int chunk, CellGrid g,
                                                      int nb, const int* __restrict__ base, const int* __restrict__ off,
                                                      int* __restrict__ perm, double* __restrict__ xs)
{
    __shared__ int cur[kMaxCellLabels];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    for (int d = t; d <= g.nc; d += 256) cur[d] = off[d] + base[(size_t)d * nb + blockIdx.x];
    const int64_t lo = (int64_t)blockIdx.x * chunk, hi = lo + chunk < N ? lo + chunk : N;
    __syncthreads();
    for (int64_t r0 = lo; r0 < hi; r0 += 256) {
        const int64_t i = r0 + t;
        const bool live = i < hi;
        const double X = live ? x[2 * i] : 0.0, Y = live ? x[2 * i + 1] : 0.0;
        const int l = live ? cell_of(g, X, Y) : -1;
        uint64_t peers = __ballot(live);
#pragma unroll
        for (int b = 0; b < 13; ++b) {          // labels are below 8192
            const bool bit = (l >> b) & 1;
            const uint64_t m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        const int rank = __popcll(peers & ((1ull << lane) - 1ull));
        int dest = -1;
        for (int k = 0; k < 4; ++k) {
            if (w == k && live) dest = cur[l] + rank;
            __syncthreads();
            if (w == k && live && rank == 0) cur[l] += __popcll(peers);
            __syncthreads();
        }
        if (live) {
            perm[dest] = (int)i;
            reinterpret_cast<double2*>(xs)[dest] = make_double2(X, Y);
        }
    }
}

// Near and far bits: a lane a segment (or outer element), two words a wavefront at a time, kBitWords a wavefront;
// blockIdx.y a row.  A segment is far from a cell when its extent stays kFarCells cell widths away from the cell's square
// in x or in y and no sample of the square can have both of its end points within the near radius (the pairs the mixed
// sweeps evaluate in float64; margins far above the float32 rounding of that test), or when it is far from a cell above
// it.  Coordinates are taken from the grid's origin in the sweep's own precision T before the test's float32: a float64
// sweep's domain may lie anywhere (from float32 coordinates, segments of a unit domain at 1e7 were far from cells that
// they cross); the mixed sweeps' pairs are those of the float32 tables themselves (4,096 segments, 1,048,576 samples: a
// call takes 678 us, with the float64 tables 703).
// Far bit: far here, near the parent (top level: far), and the cell holds samples.
constexpr int kBitWords = 16;
template <class T>
__global__ void __launch_bounds__(256) k_cell_bits(CellGrid g, CellLevels lv, const int* __restrict__ off,
                                                   const T* __restrict__ segs, int K,
                                                   const T* __restrict__ els, int M, float near2, int seg_words,
                                                   int words, uint32_t* __restrict__ bits, uint32_t* __restrict__ fbits)
{
    const int row = blockIdx.y, lane = threadIdx.x & 63;
    int l = 0, cx = 0, cy = 0;
    const bool stray = row == g.nc;
    if (!stray) level_cell(lv, row, l, cx, cy);
    const bool used = !stray && level_used(lv, off, l, cx, cy);
    const T ox = (T)g.x0, oy = (T)g.y0;
    // squares of the cell (0) and the cells above it
    float x0[kMaxLevels], y0[kMaxLevels], x1[kMaxLevels], y1[kMaxLevels], d[kMaxLevels];
#pragma unroll
    for (int m = 0; m < kMaxLevels; ++m) {
        const double h = g.h * (double)(1 << (l + m));
        const double X0 = (double)(cx >> m) * h, Y0 = (double)(cy >> m) * h;
        x0[m] = (float)X0; y0[m] = (float)Y0; x1[m] = (float)(X0 + h); y1[m] = (float)(Y0 + h);
        d[m] = (float)(kFarCells * h);
    }
    const int first = (blockIdx.x * 4 + (threadIdx.x >> 6)) * kBitWords;
    for (int w0 = first; w0 < first + kBitWords && w0 < words; w0 += 2) {
        const int w = w0 + (lane >> 5);
        const bool seg = w < seg_words;
        const int i = (seg ? w : w - seg_words) * 32 + (lane & 31);
        bool near = false, far = false;
        if (w < words && i < (seg ? K : M)) {
            float ax, ay, bx, by, L2;
            if (seg) {
                const T* s = segs + (size_t)i * kSegStride;
                ax = (float)(s[0] - ox); ay = (float)(s[1] - oy);
                bx = (float)(s[2] - ox); by = (float)(s[3] - oy);
                L2 = (float)s[6];
            } else {
                const T* e = els + (size_t)i * kElemStride;
                const T x = e[0] - ox, y = e[1] - oy;
                ax = (float)x; ay = (float)y;
                bx = (float)(x + e[2]); by = (float)(y + e[3]);
                L2 = (float)(e[2] * e[2] + e[3] * e[3]);
            }
            const float r2 = 1.01f * near2 * L2 + 1e-9f;
            const float lox = fminf(ax, bx), hix = fmaxf(ax, bx), loy = fminf(ay, by), hiy = fmaxf(ay, by);
            near = true;
#pragma unroll
            for (int m = kMaxLevels - 1; m >= 0; --m) {
                if (stray || l + m >= lv.n) continue;
                auto dist2 = [&](float px, float py) {
                    const float dx = fmaxf(0.0f, fmaxf(x0[m] - px, px - x1[m]));
                    const float dy = fmaxf(0.0f, fmaxf(y0[m] - py, py - y1[m]));
                    return dx * dx + dy * dy;
                };
                const bool clear = (lox >= x1[m] + d[m]) | (hix <= x0[m] - d[m]) | (loy >= y1[m] + d[m]) | (hiy <= y0[m] - d[m]);
                const bool near_m = !(clear && !(dist2(ax, ay) < r2 && dist2(bx, by) < r2));
                if (m == 0) far = near && !near_m;           // near every cell above
                near = near && near_m;
            }
        }
        const uint64_t nm = __ballot(near), fm = __ballot(far && used);
        if ((lane & 31) == 0 && w < words) {
            bits[(size_t)row * words + w] = (uint32_t)(lane ? nm >> 32 : nm);
            fbits[(size_t)row * words + w] = (uint32_t)(lane ? fm >> 32 : fm);
        }
    }
}

// cells of the longer side's g a side, the shorter one in proportion
double aspect_of(const bem_ctx* ctx, bool* ok)
{
    const double bw = ctx->bbox[2] - ctx->bbox[0], bh = ctx->bbox[3] - ctx->bbox[1];
    *ok = bw > 0.0 && bh > 0.0;
    return bw > bh ? bh / bw : bw / bh;
}

}  // namespace

// Direct sums evaluate N (K + M) pairs.  With n_l cells at level l, each near some (2 kFarCells + 1)^2 of its own area,
// the nodes take q^2 n_l pairs of every segment near the parent but not near the cell (top level: not near the
// cell), and the samples the near ones of the finest level: the least of that over the cells a side and the levels.
// Where a wavefront's lanes are 64 segments in `places` places, it takes a row for all of them if any needs it.  A row's
// own work (bits, node sums, coefficients) takes as long as `row` pairs.  Measured, one level at its best against the
// choice here: 4,096 segments and 1,048,576 samples 1.08 -> 0.69 ms; 500 and 262,144 215 -> 180 us; 512 in float64 (16
// nodes a side) and 262,144 645 -> 500 us; adjoint of 8,192 and 4,194,304 13.1 -> 10.4 ms.
Grouping cells_for(const bem_ctx* ctx, int64_t N, int K, int q, double ratio, double worth, double low,
                   double row, double places)
{
    Grouping best;
    bool ok;
    const double aspect = aspect_of(ctx, &ok);
    if (!ok || N < 8192 || N > ((int64_t)1 << 30)) return best;
    const double reach = (2.0 * kFarCells + 1.0) * (2.0 * kFarCells + 1.0);
    double least = 0.0, share = 1.0;
    for (int levels = 1; levels <= kMaxLevels; ++levels)
        for (int g = levels > 1 ? 1 << (levels - 1) : 2; g <= kMaxGrid; g += 1 << (levels - 1)) {     // (no ragged parents)
            int nx = g, ny = (int)std::ceil(g * aspect);
            double nodes = 0.0, rows = 0.0, near0 = 1.0, n = (double)nx * ny, near = std::min(1.0, reach / n);
            near0 = near;
            for (int l = 0; l < levels; ++l) {
                const double above = (double)((nx + 1) / 2) * ((ny + 1) / 2);
                const double up = l + 1 < levels ? std::min(1.0, reach / above) : 1.0;
                nodes += (l + 1 < levels ? low : 1.0) * q * q * n * std::min(1.0, places * (up - near));
                rows += n;
                nx = (nx + 1) / 2;
                ny = (ny + 1) / 2;
                n = above;
                near = up;
            }
            const double cost = nodes + ratio * (double)N * near0 + rows * row / ((double)K + 0.4 * ctx->M);
            if (best.g == 0 || cost < least) {
                best.g = g;
                best.levels = levels;
                least = cost;
                share = nodes / (double)N + near0;
            }
        }
    if (!((1.0 - share) * (double)N * ((double)K + 0.4 * ctx->M) > worth)) best.g = 0;
    return best;
}

// q^2 n + (2 kFarCells + 1)^2 ratio N / n is least at n = ((2 kFarCells + 1) / q) sqrt(ratio N).
int cells_one_level(const bem_ctx* ctx, int64_t N, int q, double ratio)
{
    bool ok;
    const double aspect = aspect_of(ctx, &ok);
    if (!ok || N < 8192 || N > ((int64_t)1 << 30)) return 0;
    const double g = std::sqrt((2.0 * kFarCells + 1.0) / q * std::sqrt(ratio * (double)N) / aspect);
    const int n = (int)(g > kMaxGrid ? kMaxGrid : g);
    const double cells = (double)n * std::ceil(n * aspect);
    const double share = q * q * cells / (double)N + (2.0 * kFarCells + 1.0) * (2.0 * kFarCells + 1.0) / cells;
    return n >= 2 && share < 1.0 ? n : 0;
}

int cell_plan(bem_ctx* ctx, const double* x, int64_t N, Grouping choice, CellPlan* p, hipStream_t s)
{
    int rc;
    const int g = choice.g;
    const double bw = ctx->bbox[2] - ctx->bbox[0], bh = ctx->bbox[3] - ctx->bbox[1];
    CellGrid& G = p->grid;
    G.x0 = ctx->bbox[0];
    G.y0 = ctx->bbox[1];
    G.h = (bw > bh ? bw : bh) / g;
    G.inv_h = 1.0 / G.h;
    auto cells = [&](double w) {
        const int n = (int)std::ceil(w * G.inv_h - 1e-9);
        return n < 1 ? 1 : (n > g ? g : n);
    };
    G.nx = cells(bw);
    G.ny = cells(bh);
    G.nc = G.nx * G.ny;
    const int nlab = G.nc + 1;
    CellLevels& lv = p->lv;
    lv.n = choice.levels;
    for (int l = 0, next = 0; l < lv.n; ++l) {
        lv.nx[l] = l ? (lv.nx[l - 1] + 1) / 2 : G.nx;
        lv.ny[l] = l ? (lv.ny[l - 1] + 1) / 2 : G.ny;
        lv.base[l] = next;
        next += lv.nx[l] * lv.ny[l] + (l == 0);
        lv.rows = next;
    }
    int chunk = 256;
    while (chunk < 4096 && N / chunk > 512) chunk *= 2;
    const int nb = blocks_for(N, chunk);
    // perm [N] | xs [N][2] | counts [nlab][nb] | totals, off, wave0, run0 [nlab + 1] each
    auto up = [](size_t b) { return (b + 255) / 256 * 256; };
    const size_t pb = up((size_t)N * sizeof(int)), xb = up((size_t)N * 2 * sizeof(double)),
                 cb = up((size_t)nlab * nb * sizeof(int)), lb = up((size_t)(nlab + 1) * sizeof(int));
    if ((rc = ensure(ctx, ctx->cellw, pb + xb + cb + 4 * lb, s))) return rc;
    char* base = (char*)ctx->cellw.ptr;
    int* perm = (int*)base;
    double* xs = (double*)(base + pb);
    int* cnt = (int*)(base + pb + xb);
    int* total = (int*)(base + pb + xb + cb);
    int* off = (int*)((char*)total + lb);
    int* wave0 = (int*)((char*)off + lb);
    int* run0 = (int*)((char*)wave0 + lb);
    // runs of samples for the adjoint: enough of them to fill the chip, long enough to pay for their sums
    int run = 64;
    while (run < 1024 && N / run > 4096) run *= 2;
    p->run = run;
    hipLaunchKernelGGL(k_cell_hist, dim3(nb), dim3(256), 0, s, x, N, chunk, G, nb, cnt);
    hipLaunchKernelGGL(k_cell_scan, dim3(blocks_for(nlab, 4)), dim3(256), 0, s, cnt, nlab, nb, total);
    hipLaunchKernelGGL(k_cell_offsets, dim3(1), dim3(1024), 0, s, (const int*)total, nlab, run, off, wave0, run0);
    hipLaunchKernelGGL(k_cell_scatter, dim3(nb), dim3(256), 0, s, x, N, chunk, G, nb, (const int*)cnt, (const int*)off,
                       perm, xs);
    p->perm = perm;
    p->xs = xs;
    p->off = off;
    p->wave0 = wave0;
    p->run0 = run0;
    p->max_waves = N / 64 + nlab;
    p->max_runs = N / run + nlab;
    return check_launch(ctx, "cell plan");
}

int cell_bits(bem_ctx* ctx, CellPlan* p, int K, int M, bool mixed, hipStream_t s)
{
    int rc;
    const double nf = mixed ? near_radius(ctx->opts.near_factor) : 0.0;
    p->seg_words = (K + 31) / 32;
    p->words = p->seg_words + (M + 31) / 32;
    const int64_t n = (int64_t)p->lv.rows * p->words;
    if ((rc = ensure(ctx, ctx->cellb, (size_t)n * 2 * sizeof(uint32_t), s))) return rc;
    uint32_t* bits = (uint32_t*)ctx->cellb.ptr;
    const dim3 grid(blocks_for(p->words, 4 * kBitWords), p->lv.rows);
    if (mixed)
        hipLaunchKernelGGL(k_cell_bits<float>, grid, dim3(256), 0, s, p->grid, p->lv, p->off, (const float*)ctx->seg32.ptr, K,
                           (const float*)ctx->elem32.ptr, M, (float)(nf * nf), p->seg_words, p->words, bits, bits + n);
    else
        hipLaunchKernelGGL(k_cell_bits<double>, grid, dim3(256), 0, s, p->grid, p->lv, p->off, (const double*)ctx->seg64.ptr, K,
                           (const double*)ctx->elem64.ptr, M, 0.0f, p->seg_words, p->words, bits, bits + n);
    p->bits = bits;
    p->far = bits + n;
    return check_launch(ctx, "cell bits");
}

}  // namespace bem
