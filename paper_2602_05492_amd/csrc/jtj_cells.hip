// jtj_cells.hip - J^T J of the mixed LM step over grid cells (cells.hpp).
//
// Over the n samples of a cell every feature row is X = V Phi + E: Phi [64][n] the cell's interpolation
// weights, V [W][64] the row's far part at the cell's nodes, and E the part of the near segments and elements,
// zero but for the rows of the handles and elements near the cell.  With R R^T = Phi Phi^T (64 x 64, pivoted:
// cell_factor.hpp) and R Q = Phi,
//     sum over the cell of X X^T = Y Y^T + E E^T - Z Z^T,     Z = E Q^T,   Y = V R + Z.
// So 64 columns Y stand for the cell's samples in the Gram of all W rows, and the samples themselves
// enter only the Gram of the cell's near rows.  A cell whose samples do not determine all 64 node functions (fewer
// samples, or samples in a corner or strip of it) has fewer columns, the others zero.
//
//   k_cell_rows       near handles and elements of every cell
//   k_cell_gramian    Phi Phi^T from the 15 x 15 Chebyshev moments of the samples (float64)
//   k_cell_factor     R, and C = R^-1 D^T with which q(x) = C T(x)
//   k_cell_basis      Q in split bfloat16, 32-sample blocks
//   k_near_features   E in split bfloat16, 32-sample blocks; pairs within the near radius in float64
//   k_near_project    Z on bf16 MFMA
//   k_far_parents     V's part of the segments far from 2 x 2 cells, at the nodes of those
//   k_far_features    V at the nodes, times R, plus Z: Y in float32
//   k_split_half      Y as scaled float16 pairs
//   launch_gram_half  Y Y^T, launch_gram_cells: E E^T - Z Z^T, added into the same float64 Gram
// Rounding.  The split-bfloat16 products of E average over the samples as those of the Gram over all
// samples do; the fewer columns Y and Z carry 22 and 24 bits instead of 16.  Accumulation in float32 within a
// run and in float64 beyond is the same.  Pairs by quadrature (seg_math.hpp), so near factors of at least 1.
// Measured, 2,097,152 samples, 256 cubic handles x 32 segments (W = 8,192 rows): Y Y^T 8.6 ms, far features
// 3.3 ms, near Gram 3.1 ms, near features 5.4 ms, where the tiles over all samples took 360 ms.  Error of the
// step against float64: 8.1e-4 at lambda = 1e-3 and 1.7e-5 at 0.1, against 1.1e-3 and 5.4e-5.
#include <algorithm>
#include <cmath>
#include <numeric>

#include "cell_factor.hpp"
#include "cells.hpp"
#include "normal.hpp"

namespace bem {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));

constexpr int kFeatVals = 28;                  // geo[3][8], col[4] of a handle at a point
constexpr double kNeRatio = 2.0;               // near pair over far pair, in time
constexpr int kGramianParts = 4;

// Near handles (any near segment) and near elements of every cell, in order; hpos / epos the place of a
// handle / element in its cell's list, or -1.  Counts: n, nh, ne per cell.
__global__ void __launch_bounds__(256) k_cell_rows(const int* __restrict__ off, const uint32_t* __restrict__ bits,
                                                   int words, int seg_words, int H, int S, int M, int nc,
                                                   int* __restrict__ hl, int* __restrict__ el, int* __restrict__ hpos,
                                                   int* __restrict__ epos, int* __restrict__ cnt)
{
    __shared__ int part[4];
    const int c = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int n = off[c + 1] - off[c];
    const uint32_t* row = bits + (size_t)c * words;
    for (int pass = 0; pass < 2; ++pass) {
        const int total = pass ? M : H;
        int* list = (pass ? el : hl) + (size_t)c * total;
        int* pos = (pass ? epos : hpos) + (size_t)c * total;
        int base = 0;
        for (int i0 = 0; i0 < total; i0 += 256) {
            const int i = i0 + tid;
            bool near = false;
            if (n > 0 && i < total) {
                const int b0 = pass ? i : i * S, b1 = pass ? i + 1 : (i + 1) * S;      // bits [b0, b1)
                const int w0 = pass ? seg_words : 0;
                for (int w = b0 >> 5; w <= (b1 - 1) >> 5; ++w) {
                    uint32_t m = 0xFFFFFFFFu;
                    if (w == b0 >> 5) m &= 0xFFFFFFFFu << (b0 & 31);
                    if (w == (b1 - 1) >> 5) m &= 0xFFFFFFFFu >> (31 - ((b1 - 1) & 31));
                    near |= (row[w0 + w] & m) != 0u;
                }
            }
            const uint64_t mask = __ballot(near);
            if (lane == 0) part[wv] = __popcll(mask);
            __syncthreads();
            int at = base + __popcll(mask & ((1ull << lane) - 1ull));
            for (int k = 0; k < wv; ++k) at += part[k];
            if (i < total) {
                pos[i] = near ? at : -1;
                if (near) list[at] = i;
            }
            base += part[0] + part[1] + part[2] + part[3];
            __syncthreads();
        }
        if (tid == 0) cnt[3 * c + 1 + pass] = base;
    }
    if (tid == 0) cnt[3 * c] = n;
}

// Chebyshev moments mu_pq = sum over the cell of T_p(xi) T_q(eta), p, q < 15, in float64: block (cell,
// part), a wavefront stages 32 samples and its lane (p, q / 4) sums four q.
__global__ void __launch_bounds__(256) k_cell_gramian(CellPlan p, double* __restrict__ part)
{
    __shared__ double sx[4][32][kMom + 1], sy[4][32][kMom + 1];
    const int c = blockIdx.x, wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int i0 = p.off[c], i1 = p.off[c + 1];
    if (i0 == i1) return;
    double cx, cy;
    cell_corner(p.grid, c, cx, cy);
    double m[4] = {0.0, 0.0, 0.0, 0.0};
    const int pp = lane & 15, q4 = (lane >> 4) * 4;
    for (int s0 = i0 + (blockIdx.y * 4 + wv) * 32; s0 < i1; s0 += kGramianParts * 4 * 32) {
        const int n = i1 - s0 < 32 ? i1 - s0 : 32;
        if ((lane & 31) < n) {                       // lanes 0..31: T(xi), 32..63: T(eta)
            const size_t i = s0 + (lane & 31);
            const double t = lane < 32 ? (p.xs[2 * i] - cx) * (2.0 * p.grid.inv_h) - 1.0
                                       : (p.xs[2 * i + 1] - cy) * (2.0 * p.grid.inv_h) - 1.0;
            double* o = lane < 32 ? sx[wv][lane] : sy[wv][lane - 32];
            double a = 1.0, b = t;
            for (int k = 0; k < kMom; ++k) {
                o[k] = a;
                const double d = 2.0 * t * b - a;
                a = b;
                b = d;
            }
        }
        __threadfence_block();
        for (int s = 0; s < n; ++s) {
            const double t = sx[wv][s][pp];
#pragma unroll
            for (int k = 0; k < 4; ++k) m[k] += t * sy[wv][s][q4 + k];
        }
        __threadfence_block();
    }
    __syncthreads();
    double* red = &sx[0][0][0];                      // [4][16 * 16]
    for (int k = 0; k < 4; ++k) red[wv * 256 + (q4 + k) * kMom + pp] = m[k];
    __syncthreads();
    const int t = threadIdx.x;
    part[((size_t)blockIdx.y * p.grid.nc + c) * 256 + t] = (red[t] + red[256 + t]) + (red[512 + t] + red[768 + t]);
}

// One workgroup's threads in cell_factor: every wavefront looks for the pivot by itself, the low six bits of a value
// replaced by its node (the first of equal ones).
struct BlockTeam {
    int t;
    static constexpr int n = 256;
    __device__ void sync() const { __syncthreads(); }
    __device__ int largest(const double (*A)[kFarNodes + 1], const int* step) const
    {
        const int lane = t & 63;
        const double v = A[lane][lane];
        unsigned long long key = step[lane] < 0 && v > 0.0 ? ((unsigned long long)__double_as_longlong(v) & ~63ull) | (63 - lane) : 0ull;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const unsigned long long u = __shfl_xor(key, o);
            key = u > key ? u : key;
        }
        return key ? 63 - (int)(key & 63ull) : -1;
    }
};

// Block a cell: the factor R of its Gramian (Rf [n][k], float32) and C with which q(x) = C T(x) ([k][ab], float64).
// Bound by the factor's chain of 64 steps: 0.16 ms for 289 cells, 0.50 ms for 1,296 (in node order 0.12 and 0.37).
__global__ void __launch_bounds__(256) k_cell_factor(const double* __restrict__ part, int nc, const int* __restrict__ off,
                                                     float* __restrict__ Rf, double* __restrict__ Cq)
{
    constexpr int Q = kFarQ, NN = kFarNodes;
    static_assert(Q == kFactorSide, "");
    __shared__ CellFactor w;
    const int c = blockIdx.x, t = threadIdx.x;
    if (off[c + 1] == off[c]) {
        for (int e = t; e < NN * NN; e += 256) Rf[(size_t)c * NN * NN + e] = 0.0f;
        return;
    }
    double s = 0.0;
    for (int p = 0; p < kGramianParts; ++p) s += part[((size_t)p * nc + c) * 256 + t];
    w.mu[t] = s;
    if (t < Q * Q) {
        const int a = t / Q, i = t % Q;
        w.d[a][i] = cospi((double)(a * (2 * i + 1)) / (2.0 * Q)) * (a == 0 ? 1.0 / Q : 2.0 / Q);
    }
    __syncthreads();
    cell_factor(BlockTeam{t}, w);
    for (int e = t; e < NN * NN; e += 256) {
        Rf[(size_t)c * NN * NN + e] = (float)w.R[e >> 6][e & 63];
        Cq[(size_t)c * NN * NN + e] = w.A[e >> 6][e & 63];
    }
}

__device__ inline void put_split(uint16_t* __restrict__ hi, uint16_t* __restrict__ lo, size_t i, float v)
{
    const uint16_t h = bf16_bits(v);
    hi[i] = h;
    lo[i] = bf16_bits(v - bf16_value(h));
}

// q(x) = C T(x) of every sample, in float64, stored split: a wavefront of a cell's samples.
__global__ void __launch_bounds__(256) k_cell_basis(CellPlan p, const CellInfo* __restrict__ ci,
                                                    const double* __restrict__ Cq, uint16_t* __restrict__ Qh,
                                                    uint16_t* __restrict__ Ql)
{
    const int w = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const int nl = p.grid.nc + 1;
    if (w >= p.wave0[nl]) return;
    const int c = unit_label(p.wave0, nl, w);
    if (c == p.grid.nc) return;
    const int n = ci[c].n, t = (w - p.wave0[c]) * 64 + lane;
    if (t >= ((n + 31) & ~31)) return;
    const bool live = t < n;
    const size_t i = (size_t)p.off[c] + (live ? t : 0);
    double cx, cy, Ta[kFarQ], Tb[kFarQ];
    cell_corner(p.grid, c, cx, cy);
    cheb_values<double, kFarQ>((p.xs[2 * i] - cx) * (2.0 * p.grid.inv_h) - 1.0, Ta);
    cheb_values<double, kFarQ>((p.xs[2 * i + 1] - cy) * (2.0 * p.grid.inv_h) - 1.0, Tb);
    const double* C = Cq + (size_t)c * kFarNodes * kFarNodes;
    const size_t o = ((size_t)ci[c].tb + (t >> 5)) * (kFarNodes * 32) + (t & 31);
#pragma unroll 1
    for (int k = 0; k < kFarNodes; ++k) {
        const double* r = C + k * kFarNodes;
        double v = 0.0;
#pragma unroll
        for (int b = 0; b < kFarQ; ++b) {
            double u = r[8 * b];
#pragma unroll
            for (int a = 1; a < kFarQ; ++a) u += r[8 * b + a] * Ta[a];
            v += Tb[b] * u;
        }
        put_split(Qh, Ql, o + (size_t)k * 32, live ? (float)v : 0.0f);
    }
}

constexpr int kListCap = 256, kListFull = kListCap - 64;
struct NearFeat {
    uint32_t list[kListCap];                       // lane << 26 | segment
    float corr[64][kFeatVals + 1];
};

// Float64 features of one listed pair, added to its sample's row of corr.
__device__ inline void near_pair_features(const double* __restrict__ s64, int j, int S, int model, double X, double Y,
                                          double eps2, float* __restrict__ corr)
{
    const SegGeom<double> g = load_geom(s64);
    const double ta = (double)j / (double)S, tb = (double)(j + 1) / (double)S;
    double Ba[4], Bb[4];
    vertex_weights(model, ta, Ba);
    vertex_weights(model, tb, Bb);
    const PairState<double> st = pair_forward<double, DevF64, true>(g, X, Y, eps2);
    const Moments<double> m = pair_moments(g, st);
    for (int c = 0; c < 3; ++c) {
        const Grad4<double> gr = pair_backward(g, st, eps2, s64[kWdA + c], s64[kWdB + c], s64[kWcA + c], s64[kWcB + c]);
        for (int q = 0; q < 4; ++q) {
            atomicAdd(corr + 8 * c + 2 * q, (float)(Ba[q] * gr.ax + Bb[q] * gr.bx));
            atomicAdd(corr + 8 * c + 2 * q + 1, (float)(Ba[q] * gr.ay + Bb[q] * gr.by));
        }
    }
    atomicAdd(corr + 24, (float)(m.da * (1.0 - ta) + m.db * (1.0 - tb)));
    atomicAdd(corr + 25, (float)(m.da * ta + m.db * tb));
    atomicAdd(corr + 26, (float)(m.sa * (1.0 - ta) + m.sb * (1.0 - tb)));
    atomicAdd(corr + 27, (float)(m.sa * ta + m.sb * tb));
}

// E of a cell: a wavefront of its samples, every gridDim.y-th near handle and element.  Rows in the order of
// the whole Gram: [g_0 (G nh) | g_1 | g_2 | e (C nh) | beta (ne)].
__global__ void __launch_bounds__(256, 2)
    k_near_features(CellPlan p, const CellInfo* __restrict__ ci, const int* __restrict__ hl, const int* __restrict__ el,
                    Layout L, int S, int M, int model, const float* __restrict__ seg32, const double* __restrict__ seg64,
                    const float* __restrict__ el32, const double* __restrict__ el64, const float* __restrict__ vtab,
                    float eps2f, double eps2, float near2, uint16_t* __restrict__ Eh, uint16_t* __restrict__ El)
{
    __shared__ NearFeat nf[4];
    const int w = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const int nl = p.grid.nc + 1;
    if (w >= p.wave0[nl]) return;
    const int c = unit_label(p.wave0, nl, w);
    const int n = ci[c].n, nh = ci[c].nh, ne = ci[c].ne, rows = ci[c].rows;
    const int t0 = (w - p.wave0[c]) * 64, t = t0 + lane;
    const bool live = t < n, store = t < ((n + 31) & ~31);
    const double* xw = p.xs + 2 * ((size_t)p.off[c] + t0);
    const float X = live ? (float)xw[2 * lane] : 0.0f, Y = live ? (float)xw[2 * lane + 1] : 0.0f;
    const uint32_t* bits = p.bits + (size_t)c * p.words;
    NearFeat& nb = nf[threadIdx.x >> 6];
    const size_t base = (size_t)ci[c].eoff + (size_t)(t >> 5) * ((size_t)rows << 5) + (t & 31);
    auto put = [&](int row, float v) {
        if (store) put_split(Eh, El, base + ((size_t)row << 5), live ? v : 0.0f);
    };
    for (int hi = blockIdx.y; hi < nh; hi += gridDim.y) {
        const int h = hl[(size_t)c * L.H + hi];
        float geo[3][8], col[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
            for (int k = 0; k < 8; ++k) geo[q][k] = 0.f;
        int cnt = 0;
        bool any = false;
        const int k1 = (h + 1) * S;
        for (int k = h * S; k < k1;) {
            for (; k < k1 && cnt <= kListFull; ++k) {
                if (!((bits[k >> 5] >> (k & 31)) & 1u)) continue;
                const float* s = seg32 + (size_t)k * kSegStride;
                const bool near = live & near_segment(s[0], s[1], s[2], s[3], s[6], X, Y, near2);
                const uint64_t mask = __ballot(near);
                if (mask != 0) {
                    if (near) nb.list[cnt + __popcll(mask & ((1ull << lane) - 1ull))] = ((uint32_t)lane << 26) | (uint32_t)k;
                    cnt += __popcll(mask);
                }
                const float* V = vtab + 8 * (k - h * S);
                add_pair_features<6>(s, V, V + 8, X, Y, eps2f, !near, geo, col);
            }
            if (cnt > kListFull || (k == k1 && cnt > 0)) {
                if (!any)
                    for (int q = 0; q < kFeatVals; ++q) nb.corr[lane][q] = 0.0f;
                any = true;
                __threadfence_block();
                for (int e = lane; e < cnt; e += 64) {
                    const uint32_t v = nb.list[e];
                    const int ls = v >> 26, kk = v & 0x3FFFFFFu;
                    near_pair_features(seg64 + (size_t)kk * kSegStride, kk - h * S, S, model, xw[2 * ls], xw[2 * ls + 1], eps2,
                                       nb.corr[ls]);
                }
                __threadfence_block();
                cnt = 0;
            }
        }
        if (any) {
#pragma unroll
            for (int q = 0; q < 3; ++q)
#pragma unroll
                for (int k = 0; k < 8; ++k) geo[q][k] += nb.corr[lane][8 * q + k];
#pragma unroll
            for (int k = 0; k < 4; ++k) col[k] += nb.corr[lane][24 + k];
            __threadfence_block();
        }
        if (model == 1) {
            for (int q = 0; q < 3; ++q)
#pragma unroll
                for (int k = 0; k < 4; ++k) put((q * nh + hi) * 4 + k, geo[q][k]);
            put(12 * nh + 2 * hi, col[0] + col[1]);
            put(12 * nh + 2 * hi + 1, col[2] + col[3]);
        } else {
#pragma unroll
            for (int q = 0; q < 3; ++q)
#pragma unroll
                for (int k = 0; k < 8; ++k) put((q * nh + hi) * 8 + k, geo[q][k]);
#pragma unroll
            for (int k = 0; k < 4; ++k) put(24 * nh + 4 * hi + k, col[k]);
        }
    }
    const int b0 = (3 * L.G + L.C) * nh;
    for (int i = blockIdx.y; i < ne; i += gridDim.y) {
        const int j = el[(size_t)c * M + i];
        const float* e = el32 + (size_t)j * kElemStride;
        const bool near = live & near_element(e[0], e[1], e[2], e[3], X, Y, near2);
        float b = element_beta<float, DevF32>(e[0], e[1], e[2], e[3], X, Y);
        if (near) {
            const double* e64 = el64 + (size_t)j * kElemStride;
            b = (float)element_beta<double, DevF64>(e64[0], e64[1], e64[2], e64[3], xw[2 * lane], xw[2 * lane + 1]);
        }
        put(b0 + i, b);
    }
}

// Z = E Q^T of 128 rows of a cell (work entry: cell, row block), a wavefront 32 rows x 64 columns on bf16
// MFMA: float32 to Zf [row][64], and as three bfloat16 terms in the 32-column blocks of the near tile's layout:
// Zt = terms of Z, zeros, terms of -Z, zstep apart.
__global__ void __launch_bounds__(256) k_near_project(const CellInfo* __restrict__ ci, const int* __restrict__ work,
                                                      const uint16_t* __restrict__ Eh, const uint16_t* __restrict__ El,
                                                      const uint16_t* __restrict__ Qh, const uint16_t* __restrict__ Ql,
                                                      float* __restrict__ Zf, uint16_t* __restrict__ Zt, int64_t zstep)
{
    const int c = work[2 * blockIdx.x], wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int li = lane & 31, lk = lane >> 5;
    const int rows = ci[c].rows, r0 = work[2 * blockIdx.x + 1] * 128 + wv * 32;
    if (r0 >= rows) return;
    const int ra = r0 + li < rows ? r0 + li : rows - 1;
    const int nb = (ci[c].n + 31) >> 5;
    const uint16_t* eh = Eh + ci[c].eoff + ((size_t)ra << 5) + 8 * lk;
    const uint16_t* elo = El + ci[c].eoff + ((size_t)ra << 5) + 8 * lk;
    const size_t qo = (size_t)ci[c].tb * (kFarNodes * 32) + ((size_t)li << 5) + 8 * lk;
    floatx16 acc[2];
    for (int j = 0; j < 2; ++j)
        for (int r = 0; r < 16; ++r) acc[j][r] = 0.0f;
    auto ld = [](const uint16_t* q) { return __builtin_bit_cast(bf16x8, *(const u16x8*)q); };
#pragma unroll 2
    for (int b = 0; b < nb; ++b) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const size_t ao = (size_t)b * ((size_t)rows << 5) + 16 * h;
            const bf16x8 ah = ld(eh + ao), al = ld(elo + ao);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const size_t bo = qo + (size_t)b * (kFarNodes * 32) + 1024 * j + 16 * h;
                const bf16x8 bh = ld(Qh + bo), bl = ld(Ql + bo);
                acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bh, acc[j], 0, 0, 0);
                acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bl, acc[j], 0, 0, 0);
                acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, bh, acc[j], 0, 0, 0);
            }
        }
    }
    const size_t zb = (size_t)ci[c].rb * kFarNodes;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int row = r0 + 8 * (r >> 2) + 4 * lk + (r & 3);
            if (row >= rows) continue;
            const float v = acc[j][r];
            Zf[((size_t)ci[c].rb + row) * kFarNodes + 32 * j + li] = v;
            const size_t o = zb + (size_t)j * ((size_t)rows << 5) + ((size_t)row << 5) + li;
            const uint16_t h = bf16_bits(v);
            const float v1 = v - bf16_value(h);
            const uint16_t m = bf16_bits(v1);
            const uint16_t l = bf16_bits(v1 - bf16_value(m));
            const uint16_t term[3] = {h, m, l};
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                Zt[o + k * zstep] = term[k];
                Zt[o + (4 + k) * zstep] = term[k] ^ 0x8000u;
            }
            Zt[o + 3 * zstep] = 0;
        }
}

// largest of 32 lanes (each half of the wavefront by itself), values >= 0 or NaN
__device__ inline float half_max(float v)
{
    auto step = [&](float u) { v = fmaxf(v, u); };
    step(__int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x128, 0xf, 0xf, false)));       // row_ror:8
    step(__int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x124, 0xf, 0xf, false)));
    step(__int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x122, 0xf, 0xf, false)));
    step(__int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x121, 0xf, 0xf, false)));
    step(__shfl_xor(v, 16));
    return v;
}

// Rows of an item: a cubic handle, two straight ones, or 32 elements.
constexpr int kFarLd = 66;
struct FarItems {
    int H, S, M, model, seg_words, per, handles, all;    // handles an item, items of handles, items
    __host__ __device__ FarItems(int H_, int S_, int M_, int model_, int seg_words_)
        : H(H_), S(S_), M(M_), model(model_), seg_words(seg_words_), per(model_ == 1 ? 2 : 1), handles((H_ + per - 1) / per),
          all(handles + (M_ + 31) / 32)
    {
    }
    // whether any of the item's segments or elements is far in a row of far bits
    __device__ bool any(int it, const uint32_t* __restrict__ far) const
    {
        if (it >= handles) return far[seg_words + it - handles] != 0;
        const int a = it * per * S, h1 = (it + 1) * per < H ? (it + 1) * per : H, e = h1 * S;
        uint32_t some = 0;
        for (int k0 = a; k0 < e; k0 = (k0 | 31) + 1) some |= word(far, k0, e);
        return some != 0;
    }
    // far segments k0 .. e - 1 in the word that holds k0
    __device__ static uint32_t word(const uint32_t* __restrict__ far, int k0, int e)
    {
        uint32_t w = far[k0 >> 5] & (~0u << (k0 & 31));
        if (e <= (k0 | 31)) w &= (1u << (e & 31)) - 1u;
        return w;
    }
};

// The item's rows over the far pairs of a row of far bits at the node (X, Y) of this lane, to v[row][lane].
__device__ __forceinline__ void far_rows(const FarItems& I, int it, const uint32_t* __restrict__ far, float X, float Y,
                                         float short_len, float eps2f, const float* __restrict__ seg32,
                                         const float* __restrict__ el32, const float* __restrict__ vtab, float (*v)[kFarLd])
{
    const int lane = threadIdx.x & 63;
    if (it >= I.handles) {
        const int j0 = (it - I.handles) * 32;
        const uint32_t w = far[I.seg_words + it - I.handles];
#pragma unroll 4
        for (int i = 0; i < 32; ++i) {
            float b = 0.0f;
            if ((w >> i) & 1u) {
                const float* e = el32 + (size_t)(j0 + i) * kElemStride;
                b = element_beta<float, DevF32>(e[0], e[1], e[2], e[3], X, Y);
            }
            v[i][lane] = b;
        }
        return;
    }
    for (int sub = 0; sub < I.per; ++sub) {
        const int h = it * I.per + sub;
        float geo[3][8], col[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
            for (int k = 0; k < 8; ++k) geo[q][k] = 0.f;
        const int k1 = h < I.H ? (h + 1) * I.S : 0;
        for (int k0 = h * I.S; k0 < k1; k0 = (k0 | 31) + 1)
            for (uint32_t w = FarItems::word(far, k0, k1); w; w &= w - 1u) {
                const int k = (k0 & ~31) + __builtin_ctz(w);
                const float* s = seg32 + (size_t)k * kSegStride;
                const float* B = vtab + 8 * (k - h * I.S);
                if (s[kLen] <= short_len) add_pair_features<4>(s, B, B + 8, X, Y, eps2f, true, geo, col);
                else add_pair_features<6>(s, B, B + 8, X, Y, eps2f, true, geo, col);
            }
        if (I.model == 1) {
            float(*u)[kFarLd] = v + 14 * sub;
#pragma unroll
            for (int q = 0; q < 3; ++q)
#pragma unroll
                for (int k = 0; k < 4; ++k) u[4 * q + k][lane] = geo[q][k];
            u[12][lane] = col[0] + col[1];
            u[13][lane] = col[2] + col[3];
        } else {
#pragma unroll
            for (int q = 0; q < 3; ++q)
#pragma unroll
                for (int k = 0; k < 8; ++k) v[8 * q + k][lane] = geo[q][k];
#pragma unroll
            for (int k = 0; k < 4; ++k) v[24 + k][lane] = col[k];
        }
    }
}

// Two levels save an item the pairs that are far from the 2 x 2 cells above and cost it a second product, which takes as
// long as some six pairs, and a launch: where an item has 16 segments or more and a quarter of the grid at most lies within
// reach of a cell above.  Steps at one level and at two: 256 cubic handles x 32 segments and 2,097,152 samples (36 cells
// a side) 41.5 and 39.6 ms, 128 x 32 and 262,144 (20) 10.25 and 10.15, 32 x 16 (20) 3.88 and 3.87, 128 x 32 and 65,536 (14)
// 7.65 and 7.70; 500 straight handles (two segments an item, 16) 10.45 and 10.53.
bool two_levels(int g, int S, int model) { return S * (model == 1 ? 2 : 1) >= 16 && g >= 20; }

// Far rows of the cells of 2 x 2 at their own nodes: block (cell, part), a wavefront an item at a time.  To Vp, 16 steps
// of 64 lanes' pairs an item, in the operand order of the product in k_far_features.
__global__ void __launch_bounds__(256, 2)
    k_far_parents(CellGrid g, CellLevels lv, const int* __restrict__ off, const uint32_t* __restrict__ far, int words,
                  FarItems I, const float* __restrict__ seg32, const float* __restrict__ el32, const float* __restrict__ vtab,
                  float eps2f, float2* __restrict__ Vp)
{
    __shared__ float V[4][32][kFarLd];
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, li = lane & 31, lk = lane >> 5;
    const int cx = blockIdx.x % lv.nx[1], cy = blockIdx.x / lv.nx[1];
    if (!level_used(lv, off, 1, cx, cy)) return;
    float(*v)[kFarLd] = V[wv];
    for (int i = 28; i < 32; ++i) v[i][lane] = 0.0f;
    double Xd, Yd;
    level_node<kFarQ>(g, 1, cx, cy, lane, Xd, Yd);
    const uint32_t* row = far + (size_t)level_row(lv, 1, cx, cy) * words;
    for (int it = wv + 4 * blockIdx.y; it < I.all; it += 4 * gridDim.y) {
        if (!I.any(it, row)) continue;
        far_rows(I, it, row, (float)Xd, (float)Yd, (float)(2.0 * kFarCells * g.h / kQuadFar), eps2f, seg32, el32, vtab, v);
        __threadfence_block();
        float2* o = Vp + ((size_t)blockIdx.x * I.all + it) * (16 * 64) + lane;
#pragma unroll
        for (int s = 0; s < 16; ++s) o[64 * s] = *reinterpret_cast<const float2*>(&v[li][4 * s + 2 * lk]);
        __threadfence_block();
    }
}

// Y of one cell: block (cell, part), four wavefronts that share the cell's R.  A wavefront takes an item (up to 32 rows)
// at a time: the far part at the 64 nodes (lane = node) into LDS, times R on float32 MFMA, plus Z on near rows; float32
// to Yf.  With two levels (lv.n = 2) the pairs far from the 2 x 2 cells above are in Vp at that cell's nodes, times A^T R
// with A the child's values of its nodes' polynomials.  rmax: largest magnitude of every row, as float bits; an atomic
// only where the value read beforehand is smaller.  LDS rows of kFarLd floats: 32 rows at one pair of nodes fall in
// distinct banks.  One level was bound by the vector ALUs (the pairs): 5.4 ms (8,192 segments, 1,296 cells) and 0.45 ms
// (500 straight handles, 289 cells); two levels 2.4 ms and 0.9 ms for the cells above, bound by the products and Y's stores.
template <bool Two>
__global__ void __launch_bounds__(256, 2)
    k_far_features(CellGrid g, CellLevels lv, const int* __restrict__ off, const CellInfo* __restrict__ ci,
                   const int* __restrict__ hpos, const int* __restrict__ epos, const uint32_t* __restrict__ far, int words,
                   FarItems I, Layout L, const float* __restrict__ seg32, const float* __restrict__ el32,
                   const float* __restrict__ vtab, float eps2f, const float* __restrict__ Rf, const float* __restrict__ Zf,
                   const float2* __restrict__ Vp, int64_t W, int stride, float* __restrict__ Yf, uint32_t* __restrict__ rmax)
{
    constexpr int NN = kFarNodes;
    __shared__ float Rt[1 + Two][NN][kFarLd];            // R transposed: [column][node]; then A^T R
    __shared__ float V[4][32][kFarLd];
    const int c = blockIdx.x, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int li = lane & 31, lk = lane >> 5;
    const int cx = c % g.nx, cy = c / g.nx, M = I.M;
    const bool used = off[c + 1] > off[c];
    for (int e = threadIdx.x; e < NN * NN; e += 256) Rt[0][e & 63][e >> 6] = Rf[(size_t)c * NN * NN + e];
    if constexpr (Two) {
        __shared__ double cs[4 * kFarQ], A[2][kFarQ][kFarQ];
        float(*t)[kFarLd] = V[0];                        // [column][node], over two wavefronts' rows
        if (threadIdx.x < 4 * kFarQ) cs[threadIdx.x] = cospi((double)threadIdx.x / (2 * kFarQ));
        __syncthreads();
        child_matrix<kFarQ>(threadIdx.x, 256, cs, A);
        __syncthreads();
        for (int e = threadIdx.x; e < NN * NN; e += 256) {
            const int k = e >> 6, n = e & 63;
            double s = 0.0;
#pragma unroll
            for (int i = 0; i < kFarQ; ++i) s += A[cx & 1][i][n & 7] * (double)Rt[0][k][(n & ~7) + i];
            t[k][n] = (float)s;
        }
        __syncthreads();
        for (int e = threadIdx.x; e < NN * NN; e += 256) {
            const int k = e >> 6, n = e & 63;
            double s = 0.0;
#pragma unroll
            for (int j = 0; j < kFarQ; ++j) s += A[cy & 1][j][n >> 3] * (double)t[k][8 * j + (n & 7)];
            Rt[1][k][n] = (float)s;
        }
    }
    __syncthreads();
    float(*v)[kFarLd] = V[wv];
    for (int i = 28; i < 32; ++i) v[i][lane] = 0.0f;
    const int nh = ci[c].nh;
    double Xd, Yd;
    cell_node<kFarQ>(g, c, lane, Xd, Yd);
    const uint32_t* row = far + (size_t)c * words;
    const int above = (cy >> 1) * lv.nx[1] + (cx >> 1);
    const uint32_t* up = Two ? far + (size_t)(lv.base[1] + above) * words : row;
    const float short_len = (float)(kFarCells * g.h / kQuadFar);
    // the cells' columns are dealt out in a stride permutation: in cell order the float32 sums over
    // consecutive columns see long coherent runs, and their partial sums wander
    const size_t yb = (size_t)(2 * ((int64_t)c * stride % g.nc)) * ((size_t)W << 5) + li;
    const float* z0 = Zf + (size_t)ci[c].rb * NN + li;
    for (int it = wv + 4 * blockIdx.y; it < I.all; it += 4 * gridDim.y) {
        const bool handle = it < I.handles;
        const int h0 = it * I.per, j0 = (it - I.handles) * 32;
        // row i = li of the item: its row of Y (-1: none), its near row (-1: not near), and the largest magnitude so far
        int my_f = -1, my_z = -1;
        if (!handle) {
            if (j0 + li < M) {
                my_f = (int)L.handle_rows() + j0 + li;
                const int p = used ? epos[(size_t)c * M + j0 + li] : -1;
                if (p >= 0) my_z = (3 * L.G + L.C) * nh + p;
            }
        } else {
            const int all = 3 * L.G + L.C, sub = li >= all, e = li - all * sub, h = h0 + sub;
            if (sub < I.per && e < all && h < L.H) {
                const int p = used ? hpos[(size_t)c * L.H + h] : -1, q = e / L.G, k = e % L.G;
                my_f = q < 3 ? q * (int)L.Gp + L.G * h + k : 3 * (int)L.Gp + L.C * h + (e - 3 * L.G);
                if (p >= 0) my_z = q < 3 ? (q * nh + p) * L.G + k : 3 * L.G * nh + L.C * p + (e - 3 * L.G);
            }
        }
        const uint32_t seen = my_f >= 0 ? rmax[my_f] : 0;
        floatx16 acc[2];
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[0][r] = acc[1][r] = 0.0f;
        auto product = [&](const float (*R)[kFarLd], int n, float2 a) {
            const float2 b0 = *reinterpret_cast<const float2*>(&R[li][n]);
            const float2 b1 = *reinterpret_cast<const float2*>(&R[32 + li][n]);
            acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, b0.x, acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, b1.x, acc[1], 0, 0, 0);
            acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, b0.y, acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, b1.y, acc[1], 0, 0, 0);
        };
        if constexpr (Two) {
            if (used && I.any(it, up)) {
                const float2* q = Vp + ((size_t)above * I.all + it) * (16 * 64) + lane;
                float2 a[16];
#pragma unroll
                for (int n = 0; n < 16; ++n) a[n] = q[64 * n];
#pragma unroll
                for (int n = 0; n < 16; ++n) product(Rt[1], 4 * n + 2 * lk, a[n]);
            }
        }
        if (used && I.any(it, row)) {
            far_rows(I, it, row, (float)Xd, (float)Yd, short_len, eps2f, seg32, el32, vtab, v);
            __threadfence_block();
#pragma unroll 4
            for (int n = 2 * lk; n < NN; n += 4) product(Rt[0], n, *reinterpret_cast<const float2*>(&v[li][n]));
            __threadfence_block();
        }
        // outputs: lane i (and i + 32) keeps row i's maximum
        float most = 0.0f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int i = 8 * (r >> 2) + 4 * lk + (r & 3);
            const int f = __shfl(my_f, i), z = __shfl(my_z, i);
            if (z >= 0) {
                acc[0][r] += z0[(size_t)z * NN];
                acc[1][r] += z0[(size_t)z * NN + 32];
            }
            if (f >= 0) {
                float* o = Yf + yb + ((size_t)f << 5);
                o[0] = acc[0][r];
                o[(size_t)W << 5] = acc[1][r];
            }
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float m = half_max(fmaxf(fabsf(acc[0][r]), fabsf(acc[1][r])));
            if (li == 8 * (r >> 2) + 4 * lk + (r & 3)) most = m;
        }
        if (my_f >= 0 && __float_as_uint(most) > seen) atomicMax(rmax + my_f, __float_as_uint(most));
    }
}

// Rows scaled by powers of two to magnitudes below 2^14 and split into float16 pairs; the padding rows of
// the geometry blocks are zero.  rscale undoes the scale.
__global__ void __launch_bounds__(256) k_split_half(const float* __restrict__ Yf, const uint32_t* __restrict__ rmax,
                                                    Layout L, int64_t W, int64_t nblk, uint16_t* __restrict__ Yh,
                                                    uint16_t* __restrict__ Yl, float* __restrict__ rscale)
{
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;      // four columns of one row
    if (i >= nblk * W * 32) return;
    const int64_t f = (i >> 5) % W;
    const float m = __uint_as_float(rmax[f]);
    const int e = m > 0.0f ? 14 - __builtin_amdgcn_frexp_expf(m) : 0;
    const float4 v = *reinterpret_cast<const float4*>(Yf + i);
    const bool pad = f < 3 * L.Gp && f % L.Gp >= L.geo();
    const float x[4] = {v.x, v.y, v.z, v.w};
    uint16_t h[4], l[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float t = pad ? 0.0f : __builtin_amdgcn_ldexpf(x[k], e);
        const _Float16 a = (_Float16)t, b = (_Float16)(t - (float)a);
        h[k] = __builtin_bit_cast(uint16_t, a);
        l[k] = __builtin_bit_cast(uint16_t, b);
    }
    *reinterpret_cast<uint2*>(Yh + i) = make_uint2(h[0] | (uint32_t)h[1] << 16, h[2] | (uint32_t)h[3] << 16);
    *reinterpret_cast<uint2*>(Yl + i) = make_uint2(l[0] | (uint32_t)l[1] << 16, l[2] | (uint32_t)l[3] << 16);
    if (i < W * 32 && (i & 31) == 0) rscale[f] = __builtin_amdgcn_ldexpf(1.0f, -e);
}

// As run_jtj_cells, BEM_ENOMEM without memory for its workspaces (J^T J is written last).
int over_cells(bem_ctx* ctx, const double* theta, int H, const double* x, int64_t N, double* JtJ, double norm, bool* done,
               hipStream_t s)
{
    int rc;
    const int S = ctx->opts.segs_per_handle, K = H * S, M = ctx->M;
    const double nf = near_radius(ctx->opts.near_factor), eps2 = ctx->opts.eps * ctx->opts.eps;
    const float near2 = (float)(nf * nf);
    const Layout L = layout_of(ctx, H);
    const int64_t W = L.handle_rows() + M;
    // a tile of the caller's own size is kept to
    const int g = near2 >= 4.0f && ctx->opts.tile_rows <= 0 ? cells_one_level(ctx, N, kFarQ, kNeRatio) : 0;
    if (g == 0) return BEM_OK;
    CellPlan p;
    if ((rc = launch_expand(ctx, theta, H, s))) return rc;
    if ((rc = cell_plan(ctx, x, N, two_levels(g, S, ctx->model) ? Grouping{g & ~1, 2} : Grouping{g, 1}, &p, s)))
        return rc;
    if ((rc = cell_bits(ctx, &p, K, M, true, s))) return rc;
    const int nc = p.grid.nc, nl = nc + 1;
    if (W * 64 * (int64_t)nc >= ((int64_t)1 << 31)) return BEM_OK;            // 32-bit offsets in the Gram
    // necw: counts | lists | vertex table | cell table | R | C | Gramian parts
    auto up = [](size_t b) { return (b + 255) / 256 * 256; };
    const size_t cb = up((size_t)3 * nl * sizeof(int)), hb = up((size_t)nl * H * sizeof(int)), eb = up((size_t)nl * M * sizeof(int)),
                 vb = up((size_t)(S + 1) * 8 * sizeof(float)), ib = up((size_t)nl * sizeof(CellInfo)),
                 rb = up((size_t)nc * kFarNodes * kFarNodes * sizeof(float)),
                 qb = up((size_t)nc * kFarNodes * kFarNodes * sizeof(double)),
                 gb = up((size_t)kGramianParts * nc * 256 * sizeof(double));
    if ((rc = ensure(ctx, ctx->necw, cb + 2 * hb + 2 * eb + vb + ib + rb + qb + gb, s))) return rc;
    char* b = (char*)ctx->necw.ptr;
    auto take = [&](size_t n) { char* q = b; b += n; return q; };
    int* cnt = (int*)take(cb);
    int *hl = (int*)take(hb), *hpos = (int*)take(hb), *el = (int*)take(eb), *epos = (int*)take(eb);
    float* vtab = (float*)take(vb);
    CellInfo* ci = (CellInfo*)take(ib);
    float* Rf = (float*)take(rb);
    double* Cq = (double*)take(qb);
    double* gpart = (double*)take(gb);
    hipLaunchKernelGGL(k_cell_rows, dim3(nl), dim3(256), 0, s, p.off, p.bits, p.words, p.seg_words, H, S, M, nc, hl, el,
                       hpos, epos, cnt);
    if ((rc = check_launch(ctx, "cell rows"))) return rc;
    // the counts decide the sizes of what follows, and whether it is worth it
    std::vector<int> hc(3 * (size_t)nl);
    if (hipMemcpyAsync(hc.data(), cnt, hc.size() * sizeof(int), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return set_error(ctx, BEM_EHIP, "cell rows readback");
    std::vector<CellInfo>& info = ctx->ne_info;
    std::vector<int>& work = ctx->ne_work;           // Gram entries (cell, row tile, column tile), then (cell, row block)
    info.assign(nl, CellInfo{});
    work.clear();
    int64_t blocks = 0, rows = 0, elems = 0;
    double near = 0.0;                               // near Gram, in 256 x 256 tiles x samples
    for (int c = 0; c < nl; ++c) {
        CellInfo& q = info[c];
        q.n = hc[3 * c];
        q.nh = q.n ? hc[3 * c + 1] : 0;
        q.ne = q.n ? hc[3 * c + 2] : 0;
        q.rows = (3 * L.G + L.C) * q.nh + q.ne;
        q.tb = (int)blocks;
        q.rb = (int)rows;
        q.eoff = elems;
        const int64_t nb = (q.n + 31) / 32, t = (q.rows + 255) / 256;
        if (nb * 32 * q.rows >= ((int64_t)1 << 31)) return BEM_OK;            // 32-bit offsets in a near tile
        if (c < nc) blocks += nb;
        rows += q.rows;
        elems += nb * 32 * q.rows;
        near += 0.5 * t * (t + 1) * (q.n + 64.0 + 200.0);     // an entry's start and sums cost about 200 samples
    }
    const double tiles = gram_tiles_half(L, W);
    // near and node Gram, and the pairs' share, against the Gram over all samples; the rest (basis, projection,
    // factors) costs up to two fifths of that Gram at the smallest grouped sizes, so cells serve below 0.6
    if (near + tiles * 64.0 * nc > 0.6 * tiles * (double)N || elems > ((int64_t)1 << 30) || rows >= (1 << 24)) return BEM_OK;
    for (int c = 0; c < nl; ++c) {
        const int t = (info[c].rows + 255) / 256;
        for (int i = 0; i < t; ++i)
            for (int j = i; j < t; ++j) work.insert(work.end(), {c, i, j});
    }
    const int nnear = (int)work.size() / 3;
    for (int c = 0; c < nc; ++c)
        for (int i = 0; i * 128 < info[c].rows; ++i) work.insert(work.end(), {c, i});
    const int nproj = ((int)work.size() - 3 * nnear) / 2;
    // nezw: work | Q hi, lo | Z float32 | Z hi, lo, -Z hi, lo
    const size_t wb = up(work.size() * sizeof(int)), qt = up((size_t)blocks * kFarNodes * 32 * sizeof(uint16_t)),
                 zf = up((size_t)rows * kFarNodes * sizeof(float)), zs = up((size_t)rows * kFarNodes * sizeof(uint16_t)),
                 mb = up((size_t)W * sizeof(float));
    // the sizes follow the parameters, so that a buffer that grows takes a quarter more
    auto grow = [&](DevBuf& q, size_t n) { return ensure(ctx, q, n <= q.bytes ? n : n + n / 4, s); };
    if ((rc = grow(ctx->nezw, wb + 2 * qt + zf + 7 * zs + 2 * mb + 256))) return rc;
    b = (char*)ctx->nezw.ptr;
    int* dwork = (int*)take(wb);
    uint16_t *Qh = (uint16_t*)take(qt), *Ql = (uint16_t*)take(qt);
    float* Zf = (float*)take(zf);
    uint16_t* Zt = (uint16_t*)take(7 * zs);
    const int64_t zstep = (int64_t)(zs / sizeof(uint16_t));
    uint32_t* rmax = (uint32_t*)take(mb);
    float* rscale = (float*)take(mb);
    const size_t et = up((size_t)elems * sizeof(uint16_t));
    if ((rc = grow(ctx->neew, 2 * et + 256))) return rc;
    uint16_t *Eh = (uint16_t*)ctx->neew.ptr, *El = (uint16_t*)((char*)ctx->neew.ptr + et);
    // Y in float32, then its float16 pairs
    const size_t yt = up((size_t)W * 64 * nc * sizeof(uint16_t));
    if ((rc = ensure(ctx, ctx->tmp0, 4 * yt, s))) return rc;
    if (p.lv.n > 1 && (size_t)p.lv.nx[1] * p.lv.ny[1] * FarItems(H, S, M, ctx->model, p.seg_words).all * 8192 > 2 * yt)
        return BEM_ENOMEM;                               // (not at any shape of cells: a fourth to a half as many)
    float* Yf = (float*)ctx->tmp0.ptr;
    uint16_t *Yh = (uint16_t*)((char*)ctx->tmp0.ptr + 2 * yt), *Yl = (uint16_t*)((char*)ctx->tmp0.ptr + 3 * yt);
    if ((rc = ensure(ctx, ctx->tmp1, (size_t)W * W * sizeof(double), s))) return rc;
    double* G = (double*)ctx->tmp1.ptr;
    // Columns summed in float32 before they are added in float64: rounding errors of k-column sums add up to
    // sqrt(k n) / n of the whole, so that n columns in the place of N samples summed in runs of 10,923
    // (a third of their tile) take 10,923 sqrt(n / N).  Up to 4 GiB of runs at a time.
    const int64_t n = (int64_t)64 * nc;
    const int64_t kchunk = (int64_t)(10923.0 * std::sqrt((double)n / (double)N) / 64.0 + 1.0) * 64;
    const int64_t run_bytes = (int64_t)tiles * (256 * 256 * sizeof(float));
    const int64_t all_runs = (n + kchunk - 1) / kchunk, most_runs = std::max<int64_t>(1, ((int64_t)4 << 30) / run_bytes);
    const int runs = (int)std::min(all_runs, most_runs);
    if ((rc = ensure(ctx, ctx->tmp2, (size_t)(runs * run_bytes), s))) return rc;
    float* part = (float*)ctx->tmp2.ptr;
    const int* gwork;
    int ntiles;
    if ((rc = gram_work_half(ctx, L, W, runs, &gwork, &ntiles, s))) return rc;
    // info and work stay in the context until the next step, past the copies' end
    if (hipMemcpyAsync(ci, info.data(), info.size() * sizeof(CellInfo), hipMemcpyHostToDevice, s) != hipSuccess ||
        (!work.empty() &&
         hipMemcpyAsync(dwork, work.data(), work.size() * sizeof(int), hipMemcpyHostToDevice, s) != hipSuccess))
        return set_error(ctx, BEM_EHIP, "cell table upload");
    double* Z = nullptr;
    if ((rc = boundary_derivatives(ctx, H, s, &Z))) return rc;
    if ((rc = launch_vertex_table(ctx, vtab, s))) return rc;
    const float* seg32 = (const float*)ctx->seg32.ptr;
    const double* seg64 = (const double*)ctx->seg64.ptr;
    const float* el32 = (const float*)ctx->elem32.ptr;
    const double* el64 = (const double*)ctx->elem64.ptr;
    const int wblocks = (int)((p.max_waves + 3) / 4);
    hipLaunchKernelGGL(k_cell_gramian, dim3(nc, kGramianParts), dim3(256), 0, s, p, gpart);
    hipLaunchKernelGGL(k_cell_factor, dim3(nc), dim3(256), 0, s, (const double*)gpart, nc, p.off, Rf, Cq);
    hipLaunchKernelGGL(k_cell_basis, dim3(wblocks), dim3(256), 0, s, p, (const CellInfo*)ci, (const double*)Cq, Qh, Ql);
    {
        ProfScope ps_(ctx, PT_NEAR, s);
        const int split = p.max_waves >= 8192 ? 1 : (int)(8192 / p.max_waves);
        hipLaunchKernelGGL(k_near_features, dim3(wblocks, split), dim3(256), 0, s, p, (const CellInfo*)ci, (const int*)hl,
                           (const int*)el, L, S, M, ctx->model, seg32, seg64, el32, el64, (const float*)vtab, (float)eps2, eps2,
                           near2, Eh, El);
    }
    if (nproj > 0)
        hipLaunchKernelGGL(k_near_project, dim3(nproj), dim3(256), 0, s, (const CellInfo*)ci, (const int*)(dwork + 3 * nnear),
                           (const uint16_t*)Eh, (const uint16_t*)El, (const uint16_t*)Qh, (const uint16_t*)Ql, Zf, Zt, zstep);
    if ((rc = fill_i32(ctx, (int*)rmax, W, 0, s))) return rc;
    {
        ProfScope ps_(ctx, PT_FEATURES, s);
        const FarItems items(H, S, M, ctx->model, p.seg_words);
        auto parts = [&](int cells) { return std::min((items.all + 3) / 4, 1 + 4096 / cells); };
        // the rows of the cells above lie where Y's halves go afterwards
        float2* Vp = (float2*)Yh;
        if (p.lv.n > 1) {
            const int np = p.lv.nx[1] * p.lv.ny[1];
            hipLaunchKernelGGL(k_far_parents, dim3(np, parts(np)), dim3(256), 0, s, p.grid, p.lv, p.off, p.far, p.words, items,
                               seg32, el32, (const float*)vtab, (float)eps2, Vp);
        }
        int stride = (int)(0.382 * nc) | 1;
        while (std::gcd(stride, nc) != 1) stride += 2;
        hipLaunchKernelGGL(p.lv.n > 1 ? k_far_features<true> : k_far_features<false>, dim3(nc, parts(nc)), dim3(256), 0, s, p.grid, p.lv, p.off, (const CellInfo*)ci,
                           (const int*)hpos, (const int*)epos, p.far, p.words, items, L, seg32, el32, (const float*)vtab,
                           (float)eps2, (const float*)Rf, (const float*)Zf, (const float2*)Vp, W, stride, Yf, rmax);
        hipLaunchKernelGGL(k_split_half, dim3(blocks_for((int64_t)nc * 16 * W, 256)), dim3(256), 0, s, (const float*)Yf,
                           (const uint32_t*)rmax, L, W, (int64_t)2 * nc, Yh, Yl, rscale);
    }
    if ((rc = check_launch(ctx, "cell features"))) return rc;
    for (int64_t r0 = 0; r0 < all_runs; r0 += runs) {
        const int rs = (int)std::min<int64_t>(runs, all_runs - r0);
        const int64_t k0 = r0 * kchunk, m = std::min(n - k0, rs * kchunk);
        if ((rc = launch_gram_half(ctx, Yh + k0 * W, Yl + k0 * W, (int)W, m, rscale, gwork, rs, ntiles, kchunk, part, G, r0 > 0,
                                   s)))
            return rc;
    }
    if ((rc = launch_gram_cells(ctx, Eh, El, Zt, zstep, ci, nc, hl, el, H, M, L, W, dwork, nnear, G, s))) return rc;
    const double sc = 1.0 / (norm > 0.0 ? norm : (double)N);
    if ((rc = contract_gram(ctx, H, L, W, G, 1, 256, gwork, ntiles, Z, sc, JtJ, s))) return rc;
    *done = true;
    return BEM_OK;
}

}  // namespace

int run_jtj_cells(bem_ctx* ctx, const double* theta, int H, const double* x, int64_t N, double* JtJ, double norm,
                  bool* done, hipStream_t s)
{
    *done = false;
    const int rc = over_cells(ctx, theta, H, x, N, JtJ, norm, done, s);
    if (rc != BEM_ENOMEM) return rc;
    // the samples are taken one by one, and what the workspaces held is given back
    if (hipStreamSynchronize(s) != hipSuccess) return set_error(ctx, BEM_EHIP, "stream sync");
    for (DevBuf* q : {&ctx->cellw, &ctx->cellb, &ctx->necw, &ctx->nezw, &ctx->neew, &ctx->tmp0, &ctx->tmp1, &ctx->tmp2}) release(*q);
    ctx->err.clear();
    return BEM_OK;
}

}  // namespace bem
