// sweep_eval.hip - mixed-precision forward sweep u(x) = cbar + sum_j beta_j(x) U_j + f(x) of bem_eval.
//
// Pairs run in float32 from the float32 tables, except those of a segment (or outer element) whose two
// end points lie within the near radius of the sample (near_segment): a wavefront collects these in
// LDS, and whenever its list is full evaluates them in float64, one pair a lane, into float64 sums per
// sample.  Nothing is listed in memory and no list can overflow.
//
// Few samples (k_sweep_direct): blocks of 256 samples times chunks of the tables, so that a thousand
// samples still fill the chip; the chunks' float64 sums are added in a fixed order (k_sweep_sum).
// Many samples (cells.hpp): samples grouped by cell; the segments and elements far from a cell are
// summed at its 64 nodes or those of a cell above it (k_far_nodes), turned into Chebyshev coefficients (k_far_coef) and expanded at
// its samples, which evaluate only the near ones pair by pair (k_sweep_cells).
// Both are bound by the float32 vector ALUs (about 110 flops a pair).  The line between them is
// cells_for's count of pairs.  Measured against one thread a sample over all pairs, one MI355X: 128
// segments and 1,000 samples 315 -> 26 us a call; 500 segments and 262,144 samples 722 -> 180 us; 4,096
// segments and 1,048,576 samples 9.85 -> 0.69 ms; the error against float64 went down with it (6.9e-7 ->
// 1.4e-7 for the last).
#include "cells.hpp"

namespace bem {

namespace {

// time of a near pair over that of a far one
constexpr double kEvalRatio = 2.0;
constexpr int kListCap = 320;                        // near pairs a wavefront holds
constexpr int kListFull = kListCap - 64;
constexpr int kIndexBits = 26;                       // K + M < 2^26 (check_common, build_context)

struct Tables {
    const float* seg32;
    const double* seg64;
    const float* el32;
    const double* el64;
    int K, M;
    float eps2f, near2;
    double eps2;
};

struct NearBuf {
    uint32_t list[kListCap];                         // lane << kIndexBits | segment, or K + element
    double acc[64 * 3];
};

__device__ inline void push_near(bool near, uint32_t id, NearBuf& b, int& cnt)
{
    const uint64_t mask = __ballot(near);
    if (mask == 0) return;
    const int lane = threadIdx.x & 63;
    if (near) b.list[cnt + __popcll(mask & ((1ull << lane) - 1ull))] = ((uint32_t)lane << kIndexBits) | id;
    cnt += __popcll(mask);
}

// The wavefront's listed pairs in float64, samples at x[2 * lane]; the list is empty afterwards.
__device__ inline void flush_near(const Tables& t, const double* __restrict__ x, NearBuf& b, int& cnt)
{
    __threadfence_block();
    for (int e = threadIdx.x & 63; e < cnt; e += 64) {
        const uint32_t v = b.list[e];
        const int ls = v >> kIndexBits, k = v & ((1u << kIndexBits) - 1u);
        const double X = x[2 * ls], Y = x[2 * ls + 1];
        double v0, v1, v2;
        if (k < t.K) {
            const double* s = t.seg64 + (size_t)k * kSegStride;
            const Moments<double> m = seg_moments<double, DevF64>(load_geom(s), X, Y, t.eps2);
            v0 = m.da * s[kWdA + 0] + m.db * s[kWdB + 0] + m.sa * s[kWcA + 0] + m.sb * s[kWcB + 0];
            v1 = m.da * s[kWdA + 1] + m.db * s[kWdB + 1] + m.sa * s[kWcA + 1] + m.sb * s[kWcB + 1];
            v2 = m.da * s[kWdA + 2] + m.db * s[kWdB + 2] + m.sa * s[kWcA + 2] + m.sb * s[kWcB + 2];
        } else {
            const double* el = t.el64 + (size_t)(k - t.K) * kElemStride;
            const double beta = element_beta<double, DevF64>(el[0], el[1], el[2], el[3], X, Y);
            v0 = beta * el[4]; v1 = beta * el[5]; v2 = beta * el[6];
        }
        atomicAdd(&b.acc[3 * ls + 0], v0);
        atomicAdd(&b.acc[3 * ls + 1], v1);
        atomicAdd(&b.acc[3 * ls + 2], v2);
    }
    __threadfence_block();
    cnt = 0;
}

__device__ inline void add_segment(const float* __restrict__ s, const SegGeom<float>& g, float X, float Y, float eps2f,
                                   bool near, float (&f)[3])
{
    // (a near pair counts zero times; regularised as if eps = 1, so that it is finite on an end point as well)
    const Moments<float> m = seg_moments<float, DevF32, false>(g, X, Y, near ? 1.0f : eps2f);
    const float on = near ? 0.0f : 1.0f;
#pragma unroll
    for (int c = 0; c < 3; ++c)
        f[c] += on * (m.da * s[kWdA + c] + m.db * s[kWdB + c] + m.sa * s[kWcA + c] + m.sb * s[kWcB + c]);
}

// The same for a segment at least four of its lengths away (NQ = 4), or outside the near radius of a near
// factor of at least 1 (NQ = 6), by quadrature.
template <int NQ>
__device__ inline void add_segment_quad(const float* __restrict__ s, float X, float Y, float eps2f, float (&f)[3])
{
    const Moments<float> m = quad_moments(quad_sums<float, DevF32, NQ, false>(load_geom(s), X, Y, eps2f), s[kLen]);
#pragma unroll
    for (int c = 0; c < 3; ++c)
        f[c] += m.da * s[kWdA + c] + m.db * s[kWdB + c] + m.sa * s[kWcA + c] + m.sb * s[kWcB + c];
}

constexpr int kStage = 128;                          // segment records staged at a time (12 KiB)

// Groups of gs segments, then of gs elements; chunk y of a launch takes groups [y gpc, (y + 1) gpc).
// part == null (one chunk): u is written here.
__global__ void __launch_bounds__(256, 4) k_sweep_direct(const double* __restrict__ x, int64_t N, Tables t, int gs, int gpc,
                                                      double c0, double c1, double c2, double* __restrict__ part,
                                                      float* __restrict__ u)
{
    __shared__ float4 stage[kStage * (kSegStride / 4)];
    __shared__ NearBuf nb[4];
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const bool live = i < N;
    const double* xw = x + 2 * ((int64_t)blockIdx.x * 256 + w * 64);
    NearBuf& b = nb[w];
    for (int c = 0; c < 3; ++c) b.acc[64 * c + lane] = 0.0;
    const float X = live ? (float)x[2 * i] : 0.0f, Y = live ? (float)x[2 * i + 1] : 0.0f;
    const int nsg = (t.K + gs - 1) / gs;
    const int g0 = blockIdx.y * gpc, g1 = g0 + gpc;
    const int k0 = g0 * gs, k1 = g1 < nsg ? g1 * gs : t.K;
    float f[3] = {0.f, 0.f, 0.f}, e3[3] = {0.f, 0.f, 0.f};
    int cnt = 0;
    for (int s0 = k0; s0 < k1; s0 += kStage) {
        const int n = k1 - s0 < kStage ? k1 - s0 : kStage;
        __syncthreads();
        const float4* src = reinterpret_cast<const float4*>(t.seg32 + (size_t)s0 * kSegStride);
        for (int e = threadIdx.x; e < n * (kSegStride / 4); e += 256) stage[e] = src[e];
        __syncthreads();
        for (int k = 0; k < n;) {
            for (; k < n && cnt <= kListFull; ++k) {
                const float* s = reinterpret_cast<const float*>(stage + k * (kSegStride / 4));
                const SegGeom<float> g = load_geom(s);
                const bool near = live & near_segment(g.ax, g.ay, g.bx, g.by, g.L2, X, Y, t.near2);
                push_near(near, (uint32_t)(s0 + k), b, cnt);
                add_segment(s, g, X, Y, t.eps2f, near, f);
            }
            if (cnt > kListFull) flush_near(t, xw, b, cnt);
        }
    }
    const int j0 = (g0 > nsg ? g0 - nsg : 0) * gs, j1 = (g1 - nsg) * gs < t.M ? (g1 - nsg) * gs : t.M;
    for (int j = j0; j < j1;) {
        for (; j < j1 && cnt <= kListFull; ++j) {
            const float* e = t.el32 + (size_t)j * kElemStride;
            const bool near = live & near_element(e[0], e[1], e[2], e[3], X, Y, t.near2);
            push_near(near, (uint32_t)(t.K + j), b, cnt);
            const float beta = near ? 0.0f : element_beta<float, DevF32>(e[0], e[1], e[2], e[3], X, Y);
            e3[0] += beta * e[4]; e3[1] += beta * e[5]; e3[2] += beta * e[6];
        }
        if (cnt > kListFull) flush_near(t, xw, b, cnt);
    }
    flush_near(t, xw, b, cnt);
    if (!live) return;
    const double c[3] = {c0, c1, c2};
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const double v = ((double)e3[q] + (double)f[q]) + b.acc[3 * lane + q];
        if (part) part[(size_t)blockIdx.y * 3 * N + 3 * i + q] = v;
        else u[3 * i + q] = (float)(c[q] + v);
    }
}

// a block 64 results, each wavefront every fourth chunk
__global__ void __launch_bounds__(256) k_sweep_sum(const double* __restrict__ part, int nparts, int64_t N, double c0,
                                                   double c1, double c2, float* __restrict__ u)
{
    __shared__ double red[3][64];
    const int64_t i = (int64_t)blockIdx.x * 64 + (threadIdx.x & 63);
    const double v = sum_chunks(part, nparts, 3 * N, i, red);
    if (threadIdx.x < 64 && i < 3 * N) u[i] = (float)((i % 3 == 0 ? c0 : (i % 3 == 1 ? c1 : c2)) + v);
}

// Far sums at the nodes, lane = node.  First the top level: a wavefront a cell, four cells a block share the staged
// records; chunk y takes groups [y gpc, (y + 1) gpc) as in k_sweep_direct, sums to part [y][cell].  Then a block a row of the
// levels below, whose wavefronts share the words of its few far segments (wave-uniform loads), sums to low [row].  The float32 sums of a group of 32 are added in float64.  Cells without samples have no far bits.
__global__ void __launch_bounds__(256) k_far_nodes(CellPlan p, Tables t, int gpc, int nparts, double* __restrict__ part,
                                                   double* __restrict__ low)
{
    __shared__ float4 stage[kStage * (kSegStride / 4)];
    const CellLevels& lv = p.lv;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ntop = lv.top_cells(), bt = (ntop + 3) >> 2;
    const bool top = (int)blockIdx.x < bt * nparts;
    const int y = top ? (int)blockIdx.x / bt : 0;
    const int i = top ? (int)blockIdx.x % bt * 4 + wave : (int)blockIdx.x - bt * nparts;       // cell of the top level, or row
    const bool used = top ? i < ntop : i != p.grid.nc;
    const int row = !used ? 0 : top ? lv.base[lv.n - 1] + i : i;
    int l = 0, cx = 0, cy = 0;
    level_cell(lv, row, l, cx, cy);
    double Xd, Yd;
    level_node<kFarQ>(p.grid, l, cx, cy, lane, Xd, Yd);
    const float X = (float)Xd, Y = (float)Yd;
    const uint32_t* far_bits = p.far + (size_t)row * p.words;
    const float short_len = (float)(kFarCells * p.grid.h * (1 << l) / kQuadFar);
    const bool outside = t.near2 >= 4.0f;
    auto add_far = [&](const float* s, float (&f)[3]) {
        if (s[kLen] <= short_len) add_segment_quad<4>(s, X, Y, t.eps2f, f);
        else if (outside) add_segment_quad<6>(s, X, Y, t.eps2f, f);
        else add_segment(s, load_geom(s), X, Y, t.eps2f, false, f);
    };
    auto add_far_element = [&](int j, float (&f)[3]) {
        const float* e = t.el32 + (size_t)j * kElemStride;
        const float beta = element_beta<float, DevF32>(e[0], e[1], e[2], e[3], X, Y);
        f[0] += beta * e[4]; f[1] += beta * e[5]; f[2] += beta * e[6];
    };
    double d[3] = {0.0, 0.0, 0.0};
    if (!top) {
        if (!used) return;
        double(*red)[3][kFarNodes] = (double(*)[3][kFarNodes])stage;
        int turn = 0;
        for (int w0 = 0; w0 < p.words; w0 += 64) {
            const uint32_t mine = w0 + lane < p.words ? far_bits[w0 + lane] : 0u;
            for (uint64_t some = __ballot(mine != 0); some; some &= some - 1) {
                if ((turn++ & 3) != wave) continue;
                const int w = w0 + __builtin_ctzll(some);
                float f[3] = {0.f, 0.f, 0.f};
                for (uint32_t far = __builtin_amdgcn_readlane(mine, w - w0); far; far &= far - 1u) {
                    const int k = __builtin_ctz(far);
                    if (w < p.seg_words) add_far(t.seg32 + (size_t)(w * 32 + k) * kSegStride, f);
                    else add_far_element((w - p.seg_words) * 32 + k, f);
                }
                for (int q = 0; q < 3; ++q) d[q] += (double)f[q];
            }
        }
        for (int q = 0; q < 3; ++q) red[wave][q][lane] = d[q];
        __syncthreads();
        if (threadIdx.x < 3 * kFarNodes)
            low[(size_t)row * 3 * kFarNodes + threadIdx.x] =
                (red[0][wave][lane] + red[1][wave][lane]) + (red[2][wave][lane] + red[3][wave][lane]);
        return;
    }
    const int g0 = y * gpc, g1 = g0 + gpc;
    const int k0 = g0 * 32, k1 = g1 < p.seg_words ? g1 * 32 : t.K;
    for (int s0 = k0; s0 < k1; s0 += kStage) {
        const int n = k1 - s0 < kStage ? k1 - s0 : kStage;
        __syncthreads();
        const float4* src = reinterpret_cast<const float4*>(t.seg32 + (size_t)s0 * kSegStride);
        for (int e = threadIdx.x; e < n * (kSegStride / 4); e += 256) stage[e] = src[e];
        __syncthreads();
        if (!used) continue;
        for (int q = 0; q < n; q += 32) {
            uint32_t far = far_bits[(s0 + q) >> 5];
            float f[3] = {0.f, 0.f, 0.f};
            if (far == 0xFFFFFFFFu) {
                for (int k = q; k < q + 32; ++k) add_far(reinterpret_cast<const float*>(stage + k * (kSegStride / 4)), f);
            } else {
                for (; far; far &= far - 1u)
                    add_far(reinterpret_cast<const float*>(stage + (q + __builtin_ctz(far)) * (kSegStride / 4)), f);
            }
            for (int q3 = 0; q3 < 3; ++q3) d[q3] += (double)f[q3];
        }
    }
    if (!used) return;
    for (int w = g0 > p.seg_words ? g0 : p.seg_words; w < g1 && w < p.words; ++w) {
        float f[3] = {0.f, 0.f, 0.f};
        for (uint32_t far = far_bits[w]; far; far &= far - 1u) add_far_element((w - p.seg_words) * 32 + __builtin_ctz(far), f);
        for (int q3 = 0; q3 < 3; ++q3) d[q3] += (double)f[q3];
    }
    for (int q = 0; q < 3; ++q) part[(((size_t)y * ntop + i) * 3 + q) * kFarNodes + lane] = d[q];
}

// Node sums to Chebyshev coefficients, a block a cell (thread (channel, node)): the sums of its cells above carried
// down level by level, then values v at the nodes (t_i, t_j) have
// c_ab = s_a s_b sum_ij v_ij T_a(t_i) T_b(t_j), s_0 = 1 / kFarQ, s_a = 2 / kFarQ.
__global__ void __launch_bounds__(192) k_far_coef(const double* __restrict__ part, int nparts,
                                                  const double* __restrict__ low, CellPlan pl, float* __restrict__ coef)
{
    __shared__ double v[3][kFarNodes], h[3][kFarNodes], cs[32], I[2][kFarQ][kFarQ];
    const CellLevels& lv = pl.lv;
    const int c = blockIdx.x;
    if (pl.off[c + 1] == pl.off[c]) return;
    const int ch = threadIdx.x >> 6, n = threadIdx.x & 63, a = n & 7, b = n >> 3;
    if (threadIdx.x < 32) cs[threadIdx.x] = cospi((double)threadIdx.x / 16.0);
    const int cx = c % lv.nx[0], cy = c / lv.nx[0], top = lv.n - 1, ntop = lv.top_cells();
    const int ct = (cy >> top) * lv.nx[top] + (cx >> top);
    double s = 0.0;
#pragma unroll 8
    for (int p = 0; p < nparts; ++p) s += part[(((size_t)p * ntop + ct) * 3 + ch) * kFarNodes + n];
    __syncthreads();
    if (top > 0) child_matrix<kFarQ>(threadIdx.x, 192, cs, I);
    for (int l = top - 1; l >= 0; --l) {
        const int sx = (cx >> l) & 1, sy = (cy >> l) & 1;
        v[ch][n] = s;
        __syncthreads();
        double r = 0.0;
        for (int i = 0; i < kFarQ; ++i) r += I[sx][a][i] * v[ch][8 * b + i];
        h[ch][n] = r;
        __syncthreads();
        r = low[((size_t)level_row(lv, l, cx >> l, cy >> l) * 3 + ch) * kFarNodes + n];
        for (int j = 0; j < kFarQ; ++j) r += I[sy][b][j] * h[ch][8 * j + a];
        s = r;
    }
    v[ch][n] = s;
    __syncthreads();
    // T_a(t_i) = cos(a (2 i + 1) pi / 16): entry m = a (2 i + 1) mod 32 of a cosine table
    auto tab = [&](int k, int i) { return cs[(k * (2 * i + 1)) & 31]; };
    double r = 0.0;
    for (int i = 0; i < kFarQ; ++i) r += v[ch][8 * b + i] * tab(a, i);
    h[ch][n] = r * (a == 0 ? 0.125 : 0.25);
    __syncthreads();
    r = 0.0;
    for (int j = 0; j < kFarQ; ++j) r += h[ch][8 * j + a] * tab(b, j);
    coef[((size_t)c * 3 + ch) * kFarNodes + n] = (float)(r * (b == 0 ? 0.125 : 0.25));
}

// A wavefront of up to 64 samples of one cell: the cell's near segments and elements pair by pair, the
// far ones from its coefficients.  The records are read by wave-uniform (scalar) loads.  Split 4: a block's four
// wavefronts share the samples and take every fourth bit each.  Bound by the vector ALUs (0.20 of 0.25 issue).
template <int Split>
__global__ void __launch_bounds__(256, 4) k_sweep_cells(CellPlan p, Tables t, const float* __restrict__ coef, double c0,
                                                     double c1, double c2, float* __restrict__ u)
{
    __shared__ NearBuf nb[4];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, part = wave % Split;
    const int w = __builtin_amdgcn_readfirstlane(blockIdx.x * (4 / Split) + wave / Split);
    const int nl = p.grid.nc + 1;
    if (w >= p.wave0[nl]) return;                    // (Split 4: the whole block)
    const int c = unit_label(p.wave0, nl, w);
    const int i0 = p.off[c] + (w - p.wave0[c]) * 64;
    const int i = i0 + lane;
    const bool live = i < p.off[c + 1];
    const double* xw = p.xs + 2 * (size_t)i0;
    constexpr uint32_t kMine = Split == 4 ? 0x11111111u : 0xFFFFFFFFu;
    NearBuf& b = nb[wave];
    for (int q = 0; q < 3; ++q) b.acc[64 * q + lane] = 0.0;
    const double Xd = live ? xw[2 * lane] : 0.0, Yd = live ? xw[2 * lane + 1] : 0.0;
    const float X = (float)Xd, Y = (float)Yd;
    const uint32_t* row = p.bits + (size_t)c * p.words;
    float f[3] = {0.f, 0.f, 0.f}, e3[3] = {0.f, 0.f, 0.f};
    int cnt = 0;
    int w0 = -64, wi = 0;                            // word batch, current word
    uint32_t mine = 0, word = 0;
    uint64_t some = 0;
    for (bool done = false; !done;) {
        while (cnt <= kListFull) {
            if (word == 0) {
                while (some == 0 && !done) {
                    w0 += 64;
                    if (w0 >= p.words) done = true;
                    else {
                        mine = w0 + lane < p.words ? row[w0 + lane] & (kMine << part) : 0u;
                        some = __ballot(mine != 0);
                    }
                }
                if (done) break;
                const int q = __builtin_ctzll(some);
                some &= some - 1ull;
                word = __builtin_amdgcn_readlane(mine, q);
                wi = w0 + q;
            }
            const int bit = __builtin_ctz(word);
            word &= word - 1u;
            if (wi < p.seg_words) {
                const int k = wi * 32 + bit;
                const float* s = t.seg32 + (size_t)k * kSegStride;
                const SegGeom<float> g = load_geom(s);
                const bool near = live & near_segment(g.ax, g.ay, g.bx, g.by, g.L2, X, Y, t.near2);
                push_near(near, (uint32_t)k, b, cnt);
                add_segment(s, g, X, Y, t.eps2f, near, f);
            } else {
                const int j = (wi - p.seg_words) * 32 + bit;
                const float* e = t.el32 + (size_t)j * kElemStride;
                const bool near = live & near_element(e[0], e[1], e[2], e[3], X, Y, t.near2);
                push_near(near, (uint32_t)(t.K + j), b, cnt);
                const float beta = near ? 0.0f : element_beta<float, DevF32>(e[0], e[1], e[2], e[3], X, Y);
                e3[0] += beta * e[4]; e3[1] += beta * e[5]; e3[2] += beta * e[6];
            }
        }
        flush_near(t, xw, b, cnt);
    }
    double sum[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) sum[q] = ((double)e3[q] + (double)f[q]) + b.acc[3 * lane + q];
    if constexpr (Split > 1) {
#pragma unroll
        for (int q = 0; q < 3; ++q) b.acc[3 * lane + q] = sum[q];
        __syncthreads();
        if (part > 0) return;
#pragma unroll
        for (int q = 0; q < 3; ++q)
            sum[q] = (sum[q] + nb[1].acc[3 * lane + q]) + (nb[2].acc[3 * lane + q] + nb[3].acc[3 * lane + q]);
    }
    float far[3] = {0.f, 0.f, 0.f};
    if (c < p.grid.nc) {
        double cx, cy;
        cell_corner(p.grid, c, cx, cy);
        float Ta[kFarQ], Tb[kFarQ];
        cheb_values((float)((Xd - cx) * (2.0 * p.grid.inv_h) - 1.0), Ta);
        cheb_values((float)((Yd - cy) * (2.0 * p.grid.inv_h) - 1.0), Tb);
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const float* cf = coef + ((size_t)c * 3 + q) * kFarNodes;
#pragma unroll
            for (int j = 0; j < kFarQ; ++j) {
                float r = cf[8 * j];
#pragma unroll
                for (int k = 1; k < kFarQ; ++k) r += cf[8 * j + k] * Ta[k];
                far[q] += Tb[j] * r;
            }
        }
    }
    if (!live) return;
    const size_t o = 3 * (size_t)p.perm[i];
    const double cb[3] = {c0, c1, c2};
#pragma unroll
    for (int q = 0; q < 3; ++q)
        u[o + q] = (float)(cb[q] + (sum[q] + (double)far[q]));
}

}  // namespace

// Below this many wavefronts of samples, each cell's near pairs go to four wavefronts a unit: with one, 100,000 samples are
// 1.5 wavefronts a SIMD.  500 straight handles, 100,003 samples (1,900 units) 82 and 59 us with one and four, 262,144
// (5,000) 102 and 93; from 6,144 on the chip is full.
constexpr int64_t kSplitWaves = 6144;

int launch_sweep_eval(bem_ctx* ctx, const double* x, int64_t N, int K, const double* cbar, float* u, hipStream_t s)
{
    if (N == 0) return BEM_OK;
    int rc;
    const double nf = near_radius(ctx->opts.near_factor);
    const double eps2 = ctx->opts.eps * ctx->opts.eps;
    const int M = ctx->M;
    const Tables t{(const float*)ctx->seg32.ptr, (const double*)ctx->seg64.ptr, (const float*)ctx->elem32.ptr,
                   (const double*)ctx->elem64.ptr, K, M, (float)eps2, (float)(nf * nf), eps2};
    const int64_t groups = (K + 31) / 32 + (M + 31) / 32;
    Grouping g = cells_for(ctx, N, K, kFarQ, kEvalRatio, 2e7, 2.0, 12000.0);
    ProfScope ps_(ctx, PT_SWEEP_MIXED, s);
    CellPlan p;
    int nc = 0, ntop = 0, nlow = 0, gpc = 0, nparts = 0;
    size_t pb = 0, lb = 0;
    if (g.g) {
        rc = cell_plan(ctx, x, N, g, &p, s);
        if (!rc) rc = cell_bits(ctx, &p, K, M, true, s);
        if (!rc) {
            nc = p.grid.nc;
            ntop = p.lv.top_cells();
            nlow = p.lv.low_rows();
            gpc = groups_per_chunk(groups, (ntop + 3) / 4);
            nparts = (int)((groups + gpc - 1) / gpc);
            const size_t cell = 3 * kFarNodes * sizeof(double);
            pb = (size_t)nparts * ntop * cell;
            lb = (size_t)nlow * cell;
            rc = ensure(ctx, ctx->farw, pb + lb + (size_t)nc * 3 * kFarNodes * sizeof(float), s);
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
        hipLaunchKernelGGL(k_sweep_direct, dim3(nb, nparts), dim3(256), 0, s, x, N, t, gs, gpc, cbar[0], cbar[1], cbar[2],
                           part, u);
        if (part)
            hipLaunchKernelGGL(k_sweep_sum, dim3(blocks_for(3 * N, 64)), dim3(256), 0, s, (const double*)part, nparts, N,
                               cbar[0], cbar[1], cbar[2], u);
        return check_launch(ctx, "sweep_direct");
    }
    double* part = (double*)ctx->farw.ptr;
    double* low = (double*)((char*)ctx->farw.ptr + pb);
    float* coef = (float*)((char*)ctx->farw.ptr + pb + lb);
    hipLaunchKernelGGL(k_far_nodes, dim3(nlow + (ntop + 3) / 4 * nparts), dim3(256), 0, s, p, t, gpc, nparts, part, low);
    hipLaunchKernelGGL(k_far_coef, dim3(nc), dim3(192), 0, s, (const double*)part, nparts, (const double*)low, p, coef);
    if (p.max_waves < kSplitWaves)
        hipLaunchKernelGGL(k_sweep_cells<4>, dim3(p.max_waves), dim3(256), 0, s, p, t, (const float*)coef, cbar[0], cbar[1],
                           cbar[2], u);
    else
        hipLaunchKernelGGL(k_sweep_cells<1>, dim3((p.max_waves + 3) / 4), dim3(256), 0, s, p, t, (const float*)coef, cbar[0],
                           cbar[1], cbar[2], u);
    return check_launch(ctx, "sweep_cells");
}

}  // namespace bem
