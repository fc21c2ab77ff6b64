// vjp_mixed.hip - the sample sums of the mixed adjoint: per segment the 16 sums of adjoint.hpp, per
// outer element psi_j = sum_x gbar(x) beta_j(x), over the samples of a call.
//
// Many samples (cells.hpp) take the transpose of the forward sweep's split.  The far part of a
// cell is linear in its node values, u = sum_n phi_n(x) v_n, so its cotangents are moved to the nodes,
// gbar_n = sum_x gbar(x) phi_n(x) (k_cell_moments, k_node_cotangent), and every segment sums the 64 nodes
// of its far cells, of every level, instead of their samples (k_adj_far_segments, k_adj_far_elements).  The near
// segments and elements of a cell sum its samples pair by pair (k_adj_near), pairs within the near
// radius in float64.  Few samples: k_adj_near takes every segment and element for runs of samples in
// their own order.
//
// Mapping: lanes own segments (or elements) and walk samples whose records are wave-uniform (scalar
// loads).  Float32 sums run over at most 64 samples and are added in float64.  The far sums are
// reduced in a fixed order; the near sums are added with atomics into kNearCopies partial rows.
// Bound by the float32 vector ALUs (about 200 flops a pair).  Measured against one pass of all pairs (closed
// forms), with the forward sweep of the same step, one MI355X: 8,192 segments and 4,194,304 samples 215 ->
// 10.9 ms; 500 segments and 100,003 samples 2.77 -> 0.50 ms.  Gradient error against float64 for white
// cotangents 1.7e-5 -> 6.6e-7 (8,192 segments, 1,048,576 samples), 6.1e-5 -> 1.2e-7 (128 segments, one
// sample): the quadrature does not cancel where the closed forms do.
#include "adjoint.hpp"
#include "cells.hpp"

namespace bem {

namespace {

constexpr int kRec = 8;            // sample record: X, Y, g0, g1, g2 in float32, padded to 32 bytes
// time of a near pair over that of a far one (1.3e11 against 2.2e11 pairs/s at 8,192 segments)
constexpr double kAdjRatio = 3.0;
constexpr int kMomParts = 4;       // blocks a cell that sum its moments

// Sample records in plan order (perm == null: the samples' own order).
__global__ void __launch_bounds__(256) k_sample_records(const double* __restrict__ xs, const float* __restrict__ g,
                                                        const int* __restrict__ perm, int64_t N, float* __restrict__ rec)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= N) return;
    const int64_t o = perm ? perm[i] : i;
    float4* r = reinterpret_cast<float4*>(rec + i * kRec);
    r[0] = make_float4((float)xs[2 * i], (float)xs[2 * i + 1], g[3 * o], g[3 * o + 1]);
    r[1] = make_float4(g[3 * o + 2], 0.f, 0.f, 0.f);
}

// Chebyshev moments of the cotangents of a cell, sum_x gbar(x) T_a(xi) T_b(eta): lane = (a, b), the
// wavefront's 64 samples through LDS.  Block (cell, part); float32 over 64 samples, then float64.
__global__ void __launch_bounds__(256) k_cell_moments(CellPlan p, const float* __restrict__ g,
                                                      double* __restrict__ part)
{
    constexpr int kRow = 2 * kFarQ + 3;          // odd: the lanes' stores spread over the banks
    __shared__ float sm[4][64][kRow];
    __shared__ double red[4][3][kFarNodes];
    const int c = blockIdx.x, w = threadIdx.x >> 6, lane = threadIdx.x & 63, a = lane & 7, b = lane >> 3;
    const int i0 = p.off[c], i1 = p.off[c + 1];
    if (i0 == i1) return;
    double cx, cy;
    cell_corner(p.grid, c, cx, cy);
    double m[3] = {0.0, 0.0, 0.0};
    for (int s0 = i0 + (blockIdx.y * 4 + w) * 64; s0 < i1; s0 += kMomParts * 4 * 64) {
        const int i = s0 + lane;
        float Ta[kFarQ], Tb[kFarQ], gv[3] = {0.f, 0.f, 0.f};
        double X = cx, Y = cy;
        if (i < i1) {
            X = p.xs[2 * (size_t)i];
            Y = p.xs[2 * (size_t)i + 1];
            const size_t o = 3 * (size_t)p.perm[i];
            for (int q = 0; q < 3; ++q) gv[q] = g[o + q];
        }
        cheb_values((float)((X - cx) * (2.0 * p.grid.inv_h) - 1.0), Ta);
        cheb_values((float)((Y - cy) * (2.0 * p.grid.inv_h) - 1.0), Tb);
        float* row = sm[w][lane];
#pragma unroll
        for (int q = 0; q < kFarQ; ++q) {
            row[q] = Ta[q];
            row[kFarQ + q] = Tb[q];
        }
        for (int q = 0; q < 3; ++q) row[2 * kFarQ + q] = gv[q];
        __threadfence_block();
        float f[3] = {0.f, 0.f, 0.f};
        const int n = i1 - s0 < 64 ? i1 - s0 : 64;
#pragma unroll 8
        for (int s = 0; s < n; ++s) {
            const float t = sm[w][s][a] * sm[w][s][kFarQ + b];
            for (int q = 0; q < 3; ++q) f[q] += t * sm[w][s][2 * kFarQ + q];
        }
        for (int q = 0; q < 3; ++q) m[q] += (double)f[q];
        __threadfence_block();
    }
    for (int q = 0; q < 3; ++q) red[w][q][lane] = m[q];
    __syncthreads();
    if (threadIdx.x < 3 * kFarNodes) {
        const int q = threadIdx.x >> 6;
        part[(((size_t)blockIdx.y * p.grid.nc + c) * 3 + q) * kFarNodes + lane] =
            (red[0][q][lane] + red[1][q][lane]) + (red[2][q][lane] + red[3][q][lane]);
    }
}

// Node records of a row (block a row, thread (channel, node)): gbar_ij = sum_ab s_a s_b T_a(t_i) T_b(t_j) m_ab,
// the transpose of k_far_coef.  A cell of a higher level takes its moments from those of its level-0 cells: with r of them
// a side, T_a((t + o) / r) = sum_k S_o[a][k] T_k(t), o = 1 - r, 3 - r, .., r - 1.
__global__ void __launch_bounds__(192) k_node_cotangent(const double* __restrict__ part, CellPlan pl,
                                                        float* __restrict__ rec)
{
    constexpr int kMost = 1 << (kMaxLevels - 1);
    __shared__ double v[3][kFarNodes], h[3][kFarNodes], cs[32], S[kMost][kFarQ][kFarQ];
    const CellLevels& lv = pl.lv;
    const int row = blockIdx.x;
    if (row == pl.grid.nc) return;
    int l, cx, cy;
    level_cell(lv, row, l, cx, cy);
    if (!level_used(lv, pl.off, l, cx, cy)) return;
    const int ch = threadIdx.x >> 6, n = threadIdx.x & 63, i = n & 7, j = n >> 3, r = 1 << l;
    if (threadIdx.x < 32) cs[threadIdx.x] = cospi((double)threadIdx.x / 16.0);
    __syncthreads();
    if (l > 0) {
        for (int e = threadIdx.x; e < r * kFarNodes; e += 192) {
            const int o = e >> 6, a = (e >> 3) & 7, k = e & 7;
            double s = 0.0;
            for (int m = 0; m < kFarQ; ++m) {
                double T[kFarQ];
                cheb_values<double, kFarQ>((cheb_node<kFarQ>(m) + (double)(2 * o + 1 - r)) / (double)r, T);
                double t = T[0];
                for (int q = 1; q < kFarQ; ++q) t = q == a ? T[q] : t;
                s += t * cs[(k * (2 * m + 1)) & 31];
            }
            S[o][a][k] = s * (k == 0 ? 0.125 : 0.25);
        }
    }
    double m = 0.0;
    const int x1 = (cx + 1) << l < lv.nx[0] ? (cx + 1) << l : lv.nx[0], y1 = (cy + 1) << l < lv.ny[0] ? (cy + 1) << l : lv.ny[0];
    for (int fy = cy << l; fy < y1; ++fy)
        for (int fx = cx << l; fx < x1; ++fx) {
            const int c = fy * lv.nx[0] + fx;
            if (pl.off[c + 1] == pl.off[c]) continue;                  // its moments were not written
            double s = 0.0;
            for (int p = 0; p < kMomParts; ++p) s += part[(((size_t)p * pl.grid.nc + c) * 3 + ch) * kFarNodes + n];
            if (l == 0) {
                m = s;
                continue;
            }
            v[ch][n] = s;
            __syncthreads();
            s = 0.0;
            for (int k = 0; k < kFarQ; ++k) s += S[fx - (cx << l)][i][k] * v[ch][8 * j + k];
            h[ch][n] = s;
            __syncthreads();
            for (int k = 0; k < kFarQ; ++k) m += S[fy - (cy << l)][j][k] * h[ch][8 * k + i];
        }
    __syncthreads();
    v[ch][n] = m * (i == 0 ? 0.125 : 0.25) * (j == 0 ? 0.125 : 0.25);
    __syncthreads();
    double s = 0.0;                               // over a: T_a(t_i) = cos(a (2 i + 1) pi / 16)
    for (int a = 0; a < kFarQ; ++a) s += v[ch][8 * j + a] * cs[(a * (2 * i + 1)) & 31];
    h[ch][n] = s;
    __syncthreads();
    s = 0.0;
    for (int b = 0; b < kFarQ; ++b) s += h[ch][8 * b + i] * cs[(b * (2 * j + 1)) & 31];
    float* o = rec + ((size_t)row * kFarNodes + n) * kRec;
    o[2 + ch] = (float)s;
    if (ch == 0) {
        double X, Y;
        level_node<kFarQ>(pl.grid, l, cx, cy, n, X, Y);
        o[0] = (float)X;
        o[1] = (float)Y;
    }
}

// One float32 pair of the adjoint; a masked pair (on = false) is taken at a point eight lengths beside the
// segment, with zero cotangents.  NQ: by quadrature (seg_math.hpp); 0: the closed forms, for near factors below 1.
template <int NQ>
__device__ inline void adj_pair(const SegGeom<float>& g, float len, float ilen, const float (&w)[12],
                                const float* __restrict__ r, bool on, float eps2f, float* __restrict__ af)
{
    const float X = on ? r[0] : g.ax - 8.0f * g.vy, Y = on ? r[1] : g.ay + 8.0f * g.vx;
    const float f0 = on ? r[2] : 0.f, f1 = on ? r[3] : 0.f, f2 = on ? r[4] : 0.f;
    const float wa = f0 * w[0] + f1 * w[1] + f2 * w[2];
    const float wb = f0 * w[3] + f1 * w[4] + f2 * w[5];
    const float sa = f0 * w[6] + f1 * w[7] + f2 * w[8];
    const float sb = f0 * w[9] + f1 * w[10] + f2 * w[11];
    if constexpr (NQ > 0) {
        const QuadSums<float> q = quad_sums<float, DevF32, NQ, true>(g, X, Y, eps2f);
        add_pair(af, quad_gradient(g, q, len, ilen, wa, wb, sa, sb), quad_moments(q, len), f0, f1, f2);
    } else {
        const PairState<float> st = pair_forward<float, DevF32, false>(g, X, Y, eps2f);
        add_pair(af, pair_backward(g, st, eps2f, wa, wb, sa, sb), pair_moments(g, st), f0, f1, f2);
    }
}

// Far rows of 64 segments: the wavefronts of the grid's y share the rows by turns (a segment's far rows below the top
// level lie together).
__global__ void __launch_bounds__(256) k_adj_far_segments(const float* __restrict__ rec, CellPlan p,
                                                          const float* __restrict__ seg32, int K, float eps2f, bool outside,
                                                          double* __restrict__ partial)
{
    __shared__ double red[3][64][kV + 1];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int k = blockIdx.x * 64 + lane, w0 = blockIdx.x * 2;
    double acc[kV];
    for (int v = 0; v < kV; ++v) acc[v] = 0.0;
    const float* s32 = seg32 + (size_t)(k < K ? k : 0) * kSegStride;
    if (k < K && s32[6] > 0.0f) {
        const SegGeom<float> g = load_geom(s32);
        float w[12];
        for (int c = 0; c < 12; ++c) w[c] = s32[kWdA + c];
        const float len = s32[kLen], ilen = s32[kILen];
        // levels whose far distance is four lengths for every lane
        const float reach = (float)(kFarCells * p.grid.h / kQuadFar);
        int first_short = 0;
        while (first_short < kMaxLevels && __any(len > reach * (float)(1 << first_short))) ++first_short;
        int l = 0;
        for (int row = blockIdx.y * 4 + wave; row < p.lv.rows; row += 4 * gridDim.y) {
            const uint32_t* fb = p.far + (size_t)row * p.words + w0;
            const uint64_t far = fb[0] | (w0 + 1 < p.seg_words ? (uint64_t)fb[1] << 32 : 0ull);
            if (far == 0) continue;
            while (l + 1 < p.lv.n && row >= p.lv.base[l + 1]) ++l;
            const bool on = (far >> lane) & 1ull;
            const float* r = rec + (size_t)row * kFarNodes * kRec;
            float af[kV];
            for (int v = 0; v < kV; ++v) af[v] = 0.0f;
            if (l >= first_short)
                for (int n = 0; n < kFarNodes; ++n) adj_pair<4>(g, len, ilen, w, r + n * kRec, on, eps2f, af);
            else if (outside)
                for (int n = 0; n < kFarNodes; ++n) adj_pair<6>(g, len, ilen, w, r + n * kRec, on, eps2f, af);
            else
                for (int n = 0; n < kFarNodes; ++n) adj_pair<0>(g, len, ilen, w, r + n * kRec, on, eps2f, af);
            for (int v = 0; v < kV; ++v) acc[v] += (double)af[v];
        }
    }
    if (wave > 0)
        for (int v = 0; v < kV; ++v) red[wave - 1][lane][v] = acc[v];
    __syncthreads();
    if (wave == 0 && k < K) {
        double* o = partial + ((size_t)blockIdx.y * K + k) * kV;
        for (int v = 0; v < kV; ++v) o[v] = ((acc[v] + red[0][lane][v]) + red[1][lane][v]) + red[2][lane][v];
    }
}

// Far rows of 64 outer elements, as k_adj_far_segments.
__global__ void __launch_bounds__(256) k_adj_far_elements(const float* __restrict__ rec, CellPlan p,
                                                          const float* __restrict__ el32, int M,
                                                          double* __restrict__ partial)
{
    __shared__ double red[3][64][3];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int j = blockIdx.x * 64 + lane, w0 = p.seg_words + blockIdx.x * 2;
    double acc[3] = {0.0, 0.0, 0.0};
    const float* e = el32 + (size_t)(j < M ? j : 0) * kElemStride;
    const float ax = e[0], ay = e[1], vx = e[2], vy = e[3];
    for (int row = blockIdx.y * 4 + wave; row < p.lv.rows; row += 4 * gridDim.y) {
        const uint32_t* fb = p.far + (size_t)row * p.words + w0;
        const uint64_t far = fb[0] | (w0 + 1 < p.words ? (uint64_t)fb[1] << 32 : 0ull);
        if (far == 0) continue;
        const bool on = (far >> lane) & 1ull;
        const float* r = rec + (size_t)row * kFarNodes * kRec;
        float f[3] = {0.f, 0.f, 0.f};
        for (int n = 0; n < kFarNodes; ++n) {
            const float* q = r + n * kRec;
            const float b = on ? element_beta<float, DevF32>(ax, ay, vx, vy, q[0], q[1]) : 0.0f;
            f[0] += b * q[2]; f[1] += b * q[3]; f[2] += b * q[4];
        }
        for (int v = 0; v < 3; ++v) acc[v] += (double)f[v];
    }
    if (wave > 0)
        for (int v = 0; v < 3; ++v) red[wave - 1][lane][v] = acc[v];
    __syncthreads();
    if (wave == 0 && j < M) {
        double* o = partial + ((size_t)blockIdx.y * M + j) * 3;
        for (int v = 0; v < 3; ++v) o[v] = ((acc[v] + red[0][lane][v]) + red[1][lane][v]) + red[2][lane][v];
    }
}

constexpr int kAdjTake = 4, kAdjCap = 512, kAdjFull = kAdjCap - 64 * kAdjTake;
constexpr int kSumLd = kV + 1;

// Appends (sample << 6 | lane) of the near pairs of samples s, s + 1, ... to the list until it is full or the samples
// end; returns the next sample.  Four at a time: one by one, each sample's record is waited for.
template <class Near>
__device__ inline int list_near(const float* __restrict__ rec, int s, int ns, uint32_t* list, int& cnt, Near near)
{
    const int lane = threadIdx.x;
    for (; s < ns && cnt <= kAdjFull; s += kAdjTake) {
        bool n[kAdjTake];
        bool any = false;
#pragma unroll
        for (int q = 0; q < kAdjTake; ++q) {
            const float* r = rec + (s + q < ns ? s + q : s) * kRec;
            n[q] = (s + q < ns) & near(r[0], r[1]);
            any |= n[q];
        }
        if (__ballot(any) == 0) continue;
#pragma unroll
        for (int q = 0; q < kAdjTake; ++q) {
            const uint64_t mask = __ballot(n[q]);
            if (n[q]) list[cnt + __popcll(mask & ((1ull << lane) - 1ull))] = ((uint32_t)(s + q) << 6) | lane;
            cnt += __popcll(mask);
        }
    }
    return s < ns ? s : ns;
}

// A run of samples against the segments and elements whose near bits are set (bits == null: all of
// them).  One wavefront a block: it counts the set bits of 64 words at a time and takes every
// gridDim.y-th group of 64 of them (groups hold one kind: segments, or elements), a lane each.
// Singular = false: the pairs outside the near radius, in float32.  Singular = true: only those inside
// it, listed in LDS and evaluated in float64 a pair a lane (bound by its waits, 1.37 ms at 4,194,304 samples x 8,192
// segments, 1.54 with the samples tested one by one); a kernel of its own, so that the float32
// loop keeps twice the wavefronts (the test it repeats is 10 of 330 instructions a pair).
template <bool Singular, bool Quad>
__global__ void __launch_bounds__(64, Singular ? 2 : 4)
    k_adj_near(CellPlan p, int64_t N, const double* __restrict__ x, const float* __restrict__ rec,
               const float* __restrict__ seg32, const double* __restrict__ seg64, int K, const float* __restrict__ el32,
               const double* __restrict__ el64, int M, float eps2f, double eps2, float near2,
               double* __restrict__ segsum, double* __restrict__ psisum)
{
    __shared__ int ids[64];
    __shared__ uint32_t list[Singular ? kAdjCap : 1];              // sample of the run << 6 | lane
    __shared__ double sum[64 * kSumLd];
    const int lane = threadIdx.x;
    const int u = blockIdx.x;
    int64_t i0, i1;
    const uint32_t* row = nullptr;
    if (p.bits) {
        const int nl = p.grid.nc + 1;
        if (u >= p.run0[nl]) return;
        const int c = unit_label(p.run0, nl, u);
        i0 = p.off[c] + (int64_t)(u - p.run0[c]) * p.run;
        i1 = i0 + p.run < p.off[c + 1] ? i0 + p.run : p.off[c + 1];
        row = p.bits + (size_t)c * p.words;
    } else {
        i0 = (int64_t)u * p.run;
        i1 = i0 + p.run < N ? i0 + p.run : N;
    }
    const int ns = (int)(i1 - i0);
    rec += (size_t)i0 * kRec;
    x += 2 * (size_t)i0;
    int turn = blockIdx.y;                        // groups until this block's next one
    for (int b0 = 0; b0 < p.words;) {
        const bool seg = b0 < p.seg_words;
        const int top = seg ? p.seg_words : p.words;
        const int b1 = b0 + 64 < top ? b0 + 64 : top;
        const int w = b0 + lane;
        uint32_t word = 0;
        if (w < b1) {
            if (row) word = row[w];
            else {
                const int n = seg ? K - w * 32 : M - (w - p.seg_words) * 32;
                word = n >= 32 ? 0xFFFFFFFFu : (1u << n) - 1u;
            }
        }
        int pre = __popc(word);
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int v = __shfl_up(pre, o);
            if (lane >= o) pre += v;
        }
        const int total = __builtin_amdgcn_readlane(pre, 63);
        pre -= __popc(word);
        const int groups = (total + 63) / 64;
        for (; turn < groups; turn += gridDim.y) {
            const int q = turn * 64;
            {
                int r = pre - q;
                for (uint32_t m = word; m && r < 64; m &= m - 1u, ++r)
                    if (r >= 0) ids[r] = (seg ? w : w - p.seg_words) * 32 + __builtin_ctz(m);
            }
            __threadfence_block();
            const bool own = q + lane < total;
            const int id = own ? ids[lane] : 0;
            for (int v = 0; v < kV; ++v) sum[lane * kSumLd + v] = 0.0;
            if (seg) {
                const float* s32 = seg32 + (size_t)id * kSegStride;
                const SegGeom<float> g = load_geom(s32);
                const bool some = own && g.L2 > 0.0f;
                if constexpr (Singular) {
                    int cnt = 0;
                    for (int s = 0; s < ns;) {
                        s = list_near(rec, s, ns, list, cnt, [&](float X, float Y) {
                            return some & near_segment(g.ax, g.ay, g.bx, g.by, g.L2, X, Y, near2);
                        });
                        __threadfence_block();
                        for (int e = lane; e < cnt; e += 64) {
                            const int sl = list[e] >> 6, ln = list[e] & 63;
                            const float* r = rec + sl * kRec;
                            double a[kV];
                            near_segment_values(seg64 + (size_t)ids[ln] * kSegStride, x[2 * sl], x[2 * sl + 1],
                                                (double)r[2], (double)r[3], (double)r[4], eps2, a);
                            for (int v = 0; v < kV; ++v) atomicAdd(&sum[ln * kSumLd + v], a[v]);
                        }
                        __threadfence_block();
                        cnt = 0;
                    }
                } else {
                    float wt[12];
                    for (int c = 0; c < 12; ++c) wt[c] = s32[kWdA + c];
                    for (int s = 0; s < ns;) {
                        // float32 sums over at most 64 samples
                        float af[kV];
                        for (int v = 0; v < kV; ++v) af[v] = 0.0f;
                        const int s1 = s + 64 < ns ? s + 64 : ns;
                        for (; s < s1; ++s) {
                            const float* r = rec + s * kRec;
                            const bool near = near_segment(g.ax, g.ay, g.bx, g.by, g.L2, r[0], r[1], near2);
                            adj_pair<Quad ? 6 : 0>(g, s32[kLen], s32[kILen], wt, r, some & !near, eps2f, af);
                        }
                        for (int v = 0; v < kV; ++v) sum[lane * kSumLd + v] += (double)af[v];
                    }
                }
                // value v goes to copy (run + v) mod kNearCopies: a segment's values, and the runs near
                // it, to different lines
                if (some)
                    for (int v = 0; v < kV; ++v) {
                        const double t = sum[lane * kSumLd + v];
                        if (t != 0.0) atomicAdd(segsum + ((size_t)((u + v) % kNearCopies) * K + id) * kV + v, t);
                    }
            } else {
                const float* e = el32 + (size_t)id * kElemStride;
                const float ax = e[0], ay = e[1], vx = e[2], vy = e[3];
                if constexpr (Singular) {
                    int cnt = 0;
                    for (int s = 0; s < ns;) {
                        s = list_near(rec, s, ns, list, cnt, [&](float X, float Y) {
                            return own & near_element(ax, ay, vx, vy, X, Y, near2);
                        });
                        __threadfence_block();
                        for (int n = lane; n < cnt; n += 64) {
                            const int sl = list[n] >> 6, ln = list[n] & 63;
                            const float* r = rec + sl * kRec;
                            const double* e64 = el64 + (size_t)ids[ln] * kElemStride;
                            const double b = element_beta<double, DevF64>(e64[0], e64[1], e64[2], e64[3], x[2 * sl],
                                                                          x[2 * sl + 1]);
                            for (int v = 0; v < 3; ++v) atomicAdd(&sum[ln * kSumLd + v], b * (double)r[2 + v]);
                        }
                        __threadfence_block();
                        cnt = 0;
                    }
                } else {
                    for (int s = 0; s < ns;) {
                        float f[3] = {0.f, 0.f, 0.f};
                        const int s1 = s + 64 < ns ? s + 64 : ns;
                        for (; s < s1; ++s) {
                            const float* r = rec + s * kRec;
                            const bool near = near_element(ax, ay, vx, vy, r[0], r[1], near2);
                            const float b = near ? 0.0f : element_beta<float, DevF32>(ax, ay, vx, vy, r[0], r[1]);
                            f[0] += b * r[2]; f[1] += b * r[3]; f[2] += b * r[4];
                        }
                        for (int v = 0; v < 3; ++v) sum[lane * kSumLd + v] += (double)f[v];
                    }
                }
                if (own)
                    for (int v = 0; v < 3; ++v) {
                        const double t = sum[lane * kSumLd + v];
                        if (t != 0.0) atomicAdd(psisum + ((size_t)((u + v) % kNearCopies) * M + id) * 3 + v, t);
                    }
            }
            __threadfence_block();
        }
        turn -= groups;
        b0 = b1;
    }
}

}  // namespace

// Rows of segment partials (times K x 16) and of element partials (times M x 3) that adj_mixed writes.
Grouping adj_mixed_rows(bem_ctx* ctx, int K, int64_t N, int* seg_rows, int* el_rows)
{
    // 64 segments are 64 / S handles, each some places long
    const int S = ctx->opts.segs_per_handle;
    const Grouping g = cells_for(ctx, N, K, kFarQ, kAdjRatio, 2e7, 1.0, 12000.0, S < 64 ? 128.0 / S : 2.0);
    auto rows = [&](int n) {
        const int groups = (n + 63) / 64;
        const int r = (2048 + groups - 1) / (groups > 0 ? groups : 1);
        return r < 1 ? 1 : (r > g.g * g.g / 4 ? (g.g * g.g + 3) / 4 : r);
    };
    *seg_rows = kNearCopies + (g.g ? rows(K) : 0);
    *el_rows = kNearCopies + (g.g ? rows(ctx->M) : 0);
    return g;
}

// The sample sums of the mixed adjoint into partial rows part [seg_rows][K][16] and epart
// [el_rows][M][3] (every entry written), the tables of theta expanded before.
int adj_mixed(bem_ctx* ctx, const double* x, int64_t N, const float* gbar, int K, Grouping g, int seg_rows, int el_rows,
              double* part, double* epart, hipStream_t s)
{
    int rc;
    const int M = ctx->M;
    const double eps2 = ctx->opts.eps * ctx->opts.eps, nf = near_radius(ctx->opts.near_factor);
    const float near2 = (float)(nf * nf);
    const float* seg32 = (const float*)ctx->seg32.ptr;
    const float* el32 = (const float*)ctx->elem32.ptr;
    // the near copies are the first rows
    if ((rc = fill_f64(ctx, part, (int64_t)kNearCopies * K * kV, 0.0, s))) return rc;
    if ((rc = fill_f64(ctx, epart, (int64_t)kNearCopies * M * 3, 0.0, s))) return rc;
    CellPlan p;
    int64_t runs;
    if (g.g) {
        if ((rc = cell_plan(ctx, x, N, g, &p, s))) return rc;
        if ((rc = cell_bits(ctx, &p, K, M, true, s))) return rc;
        runs = p.max_runs;
    } else {
        // few samples: runs of 64 in their own order
        p.seg_words = (K + 31) / 32;
        p.words = p.seg_words + (M + 31) / 32;
        p.xs = x;
        runs = (N + 63) / 64;
        while (p.run < 1024 && runs > 4096) {
            p.run *= 2;
            runs = (N + p.run - 1) / p.run;
        }
    }
    // blocks a run: about 8,192 in all, at most one a group
    const int64_t most = (p.words + 1) / 2, want = (8191 + runs) / runs;
    const int split = (int)(want < 4 ? (most < 4 ? most : 4) : (want < most ? want : most));
    const int nc = p.grid.nc;
    const size_t rb = ((size_t)N * kRec * sizeof(float) + 255) / 256 * 256;
    const size_t nb = g.g ? (size_t)p.lv.rows * kFarNodes * kRec * sizeof(float) : 0;
    const size_t mb = g.g ? (size_t)kMomParts * nc * 3 * kFarNodes * sizeof(double) : 0;
    if ((rc = ensure(ctx, ctx->farw, rb + nb + mb, s))) return rc;
    float* rec = (float*)ctx->farw.ptr;
    float* nrec = (float*)((char*)ctx->farw.ptr + rb);
    double* mpart = (double*)((char*)ctx->farw.ptr + rb + nb);
    hipLaunchKernelGGL(k_sample_records, dim3(blocks_for(N, 256)), dim3(256), 0, s, p.xs, gbar, p.perm, N, rec);
    if (g.g) {
        hipLaunchKernelGGL(k_cell_moments, dim3(nc, kMomParts), dim3(256), 0, s, p, gbar, mpart);
        hipLaunchKernelGGL(k_node_cotangent, dim3(p.lv.rows), dim3(192), 0, s, (const double*)mpart, p, nrec);
        const int rs = seg_rows - kNearCopies, re = el_rows - kNearCopies;
        {
            ProfScope ps_(ctx, PT_VJP_SEGMENTS, s);
            hipLaunchKernelGGL(k_adj_far_segments, dim3((K + 63) / 64, rs), dim3(256), 0, s, (const float*)nrec, p, seg32, K,
                               (float)eps2, near2 >= 4.0f, part + (size_t)kNearCopies * K * kV);
        }
        ProfScope ps_(ctx, PT_VJP_ELEMENTS, s);
        hipLaunchKernelGGL(k_adj_far_elements, dim3((M + 63) / 64, re), dim3(256), 0, s, (const float*)nrec, p, el32, M,
                           epart + (size_t)kNearCopies * M * 3);
    }
    const double* seg64 = (const double*)ctx->seg64.ptr;
    const double* el64 = (const double*)ctx->elem64.ptr;
    {
        ProfScope ps_(ctx, PT_VJP_SEGMENTS, s);
        hipLaunchKernelGGL((near2 >= 4.0f ? k_adj_near<false, true> : k_adj_near<false, false>), dim3(runs, split),
                           dim3(64), 0, s, p, N, p.xs, (const float*)rec, seg32, seg64, K, el32, el64, M, (float)eps2,
                           eps2, near2, part, epart);
    }
    ProfScope ps_(ctx, PT_NEAR, s);
    hipLaunchKernelGGL((k_adj_near<true, true>), dim3(runs, split), dim3(64), 0, s, p, N, p.xs, (const float*)rec, seg32, seg64, K,
                       el32, el64, M, (float)eps2, eps2, near2, part, epart);
    return check_launch(ctx, "mixed adjoint");
}

}  // namespace bem
