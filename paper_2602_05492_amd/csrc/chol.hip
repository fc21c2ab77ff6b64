// chol.hip - float64 Cholesky of the damped approximate Hessian
// lambda D + J^T J (Eq. optimstep: positive definite, solved by Cholesky,
// Sec. 4.3) and the two triangular solves for the LM step.
// Blocked right-looking factorisation with 128-column panels: the diagonal block
// in one workgroup's LDS, inverted in the same kernel; the panel as a GEMM
// with that inverse; the trailing update as a rank-128 symmetric update.  The solves
// use the inverted 64 x 64 diagonal blocks: one launch per block and direction.  A
// non-positive or non-finite pivot raises a device flag.
#include <utility>

#include "common.hpp"
#include "math64.hpp"
#include "sweep_common.hpp"

namespace bem {

namespace {

constexpr int NB = 64;       // blocks of the solves
constexpr int KB = 2 * NB;   // columns of a factorisation step
typedef double d2_t __attribute__((ext_vector_type(2)));

// dmax[0] = max_i H_ii (one block)
__global__ void k_diag_max(const double* __restrict__ H, int64_t P, double* __restrict__ dmax)
{
    __shared__ double red[256];
    double m = 0.0;
    for (int64_t i = threadIdx.x; i < P; i += blockDim.x) m = fmax(m, H[i * P + i]);
    red[threadIdx.x] = m;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + s]);
        __syncthreads();
    }
    if (threadIdx.x == 0) dmax[0] = red[0];
}

// A = H + lam * diag(max(H_ii, 1e-12 * max_j H_jj))
__global__ void k_damp(const double* __restrict__ H, int64_t P, double lam, const double* __restrict__ dmax,
                       double* __restrict__ A)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t i = blockIdx.y;
    if (j >= P) return;
    double v = H[i * P + j];
    if (i == j) v += lam * fmax(v, 1e-12 * dmax[0]);
    A[i * P + j] = v;
}

// lane K's value of each row of 16 lanes
template <int K>
__device__ inline double bcast16(double v)
{
    return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), 0x150 + K, 0xf, 0xf, false),
                            __builtin_amdgcn_mov_dpp(__double2loint(v), 0x150 + K, 0xf, 0xf, false));
}

// ---- diagonal block ------------------------------------------------------------------------
// A 128-column step is bound by its serial chain: the diagonal block's 128 pivots, which nothing else of the
// step can start without.  One workgroup factors it as two 64 x 64 blocks in LDS, those by 16-column panels.
// A panel is one wavefront's: each of its four rows of 16 lanes holds the panel's 16 x 16 diagonal block, three of
// them 16 rows below it as well and the fourth an identity, so that a pivot's broadcasts (within 16 lanes, no
// scalar registers) serve the factor, the rows below and the inverse of the 16 x 16 block at once.  Everything else
// (trailing updates, the inverse's off-diagonal blocks) is float64 MFMA out of LDS, spread over 8 wavefronts.  LDS rows of kLd doubles: the 16 rows x 4 k of an operand read fall in distinct
// banks.  Operand and accumulator layout of v_mfma_f64_16x16x4f64 (lane l, rr = l mod 16, lk = l / 16): A[rr][lk],
// B[lk][rr], element q of the accumulator is row 4 q + lk, column rr; so element q of a product is the B operand of
// k step q of the next product.
// Measured: 45 us a block of 128, 57 us with its update (blocks of 64 by broadcast sums: 2 x 47 us).
typedef double d4_t __attribute__((ext_vector_type(4)));
constexpr int DB = 16, kLd = 68;
typedef double Tile[NB][kLd];

__device__ inline d4_t mfma(double a, double b, d4_t c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }

// Columns J + 1 .. 15 of a panel after pivot J: a (diagonal block) and b (rows below or identity).
template <int J, int... D>
__device__ __forceinline__ void panel_update(double (&a)[DB], double (&b)[DB], std::integer_sequence<int, D...>)
{
    (
        [&] {
            constexpr int K = J + 1 + D;
            const double l = bcast16<K>(a[J]);
            a[K] = fma(-a[J], l, a[K]);
            b[K] = fma(-b[J], l, b[K]);
            asm volatile("" : "+v"(b[K]));          // now: not kept back, with its operands, to where b is stored
        }(),
        ...);
}
template <int... J>
__device__ __forceinline__ void panel_factor(double (&a)[DB], double (&b)[DB], bool& bad, std::integer_sequence<int, J...>)
{
    (
        [&] {
            const double d = bcast16<J>(a[J]);
            const bool ok = (d > 0.0) & (d < INFINITY);
            bad |= !ok;
            double r = rsqrt_f64(d);
            r = ok ? r : 1.0;
            a[J] *= r;                      // the pivot itself: d / sqrt(d)
            b[J] *= r;
            panel_update<J>(a, b, std::make_integer_sequence<int, DB - 1 - J>{});
        }(),
        ...);
}

// S [64][64] (lower triangle) -> its factor in place, X (zeros) -> the inverse (lower triangle).  All 8 wavefronts.
__device__ __forceinline__ void factor_block(Tile& S, Tile& X, bool& bad)
{
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rr = lane & 15, lk = lane >> 4;
    for (int p = 0; p < NB / DB; ++p) {
        const int d0 = p * DB;
        if (w == 0) {
            const int r = d0 + DB * (lk + 1) + rr;       // this lane's row below the diagonal block
            const bool below = lk < 3 && r < NB;
            double a[DB], b[DB];
#pragma unroll
            for (int k = 0; k < DB; ++k) {
                const double v = S[d0 + rr][d0 + k], u = S[below ? r : 0][d0 + k];
                a[k] = k <= rr ? v : 0.0;
                b[k] = below ? u : (lk == 3 && k == rr ? 1.0 : 0.0);
            }
            panel_factor(a, b, bad, std::make_integer_sequence<int, DB>{});
#pragma unroll
            for (int k = 0; k < DB; ++k) {
                if (lk == 0 && k <= rr) S[d0 + rr][d0 + k] = a[k];
                if (below) S[r][d0 + k] = b[k];
                if (lk == 3 && k >= rr) X[d0 + k][d0 + rr] = b[k];       // (L^-T)[rr][k]
            }
        }
        __syncthreads();
        // trailing 16 x 16 tiles (I, J), I >= J: S -= L L^T
        const int t = NB / DB - 1 - p;
        for (int i = w; i < t * (t + 1) / 2; i += 8) {
            const int I = i < 1 ? 0 : i < 3 ? 1 : 2, J = i - I * (I + 1) / 2;
            const int r0 = d0 + DB * (I + 1), c0 = d0 + DB * (J + 1);
            d4_t acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int k = 0; k < DB; k += 4) acc = mfma(S[r0 + rr][d0 + k + lk], S[c0 + rr][d0 + k + lk], acc);
#pragma unroll
            for (int q = 0; q < 4; ++q) S[r0 + 4 * q + lk][c0 + rr] -= acc[q];
        }
        __syncthreads();
    }
    // off-diagonal blocks of the inverse, X_10 = -X_11 (L_10 X_00): of the two 32 x 32 blocks, then of the whole
    if (w < 2) {
        const int o = 32 * w;
        d4_t t = {0.0, 0.0, 0.0, 0.0}, v = t;
#pragma unroll
        for (int k = 0; k < DB; k += 4) t = mfma(S[o + DB + rr][o + k + lk], X[o + k + lk][o + rr], t);
#pragma unroll
        for (int q = 0; q < 4; ++q) v = mfma(X[o + DB + rr][o + DB + 4 * q + lk], t[q], v);
#pragma unroll
        for (int q = 0; q < 4; ++q) X[o + DB + 4 * q + lk][o + rr] = -v[q];
    }
    __syncthreads();
    if (w < 4) {
        const int I = 2 + (w >> 1), J = w & 1;
        d4_t v = {0.0, 0.0, 0.0, 0.0};
        for (int K = 2; K <= I; ++K) {
            d4_t t = {0.0, 0.0, 0.0, 0.0};
            for (int k = DB * J; k < 2 * DB; k += 4) t = mfma(S[DB * K + rr][k + lk], X[k + lk][DB * J + rr], t);
#pragma unroll
            for (int q = 0; q < 4; ++q) v = mfma(X[DB * I + rr][DB * K + 4 * q + lk], t[q], v);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) X[DB * I + 4 * q + lk][DB * J + rr] = -v[q];
    }
    __syncthreads();
}

// LDS of a step's workgroup: the diagonal block's four tiles, or the slabs [2 groups][2 stages][A, B][64][16] of the
// trailing update.
constexpr int kStepLds = 4 * sizeof(Tile);
constexpr int kSlab = 16;
// 16-byte chunk position of k pair kp (k = 2 kp) in a slab row (as k_gemm_f64_nt)
__device__ inline int slab_pos(int row, int kp) { return 2 * (kp ^ ((row >> 1) & 7)); }
__device__ inline void load_lds(const double* g, double* lds)
{
    __builtin_amdgcn_global_load_lds((const void*)g, (void*)lds, 16, 0, 0);
}
// every load of this wavefront has landed, then every wavefront's
__device__ inline void loads_landed()
{
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
}

// Update diagonal block kb (128 columns) with the panel of block kb - 1 (kb > 0) and factor it in place (lower
// triangle); inverses of its two 64 x 64 blocks to linv64 [64-block][64][64] (for the solves) and of the whole to
// inv [128][128] (for the panel).  Rows and columns past the matrix are an identity block.
__device__ __forceinline__ void diag_block(double* lds, double* __restrict__ A, int64_t P, int kb, int* __restrict__ flag,
                                           double* __restrict__ linv64, double* __restrict__ inv)
{
    Tile& B0 = *(Tile*)lds;
    Tile& B1 = *((Tile*)lds + 1);
    Tile& S10 = *((Tile*)lds + 2);
    Tile& S11 = *((Tile*)lds + 3);
    const int64_t o = (int64_t)kb * KB;
    const int nb = (int)(P - o < KB ? P - o : KB);
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rr = lane & 15, lk = lane >> 4;
    // wavefront w takes rows w, w + 8, ... of each block, a lane a column; all loads in flight at once (entries
    // outside load the block's first element and are then replaced)
    double g[3][NB / 8];
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
        for (int q = 0; q < NB / 8; ++q) {
            const int r = (b > 0 ? NB : 0) + w + 8 * q, c = (b > 1 ? NB : 0) + lane;
            const bool in = r < nb && c <= r;
            g[b][q] = A[(o + (in ? r : 0)) * P + o + (in ? c : 0)];
        }
    // L L^T of the panel's rows at this block: 36 tiles (R, C), C <= R < 8, wavefront w takes w, w + 8, ...
    d4_t acc[5];
    int tr[5], tc[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        const int t = w + 8 * i;
        int R = 0;
        while ((R + 1) * (R + 2) / 2 <= t) ++R;
        tr[i] = R;
        tc[i] = t - R * (R + 1) / 2;
        acc[i] = d4_t{0.0, 0.0, 0.0, 0.0};
    }
    if (kb > 0) {
        double(*sl)[KB][kSlab] = (double(*)[KB][kSlab])&B1;        // two stages
        const double* gp[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int r = 16 * w + 8 * i + (lane >> 3);
            gp[i] = A + (o + (r < nb ? r : 0)) * P + (o - KB) + slab_pos(r, lane & 7);
        }
        auto load = [&](int buf, int s) {
#pragma unroll
            for (int i = 0; i < 2; ++i) load_lds(gp[i] + kSlab * s, &sl[buf][16 * w + 8 * i][0]);
        };
        load(0, 0);
        loads_landed();
        for (int s = 0; s < KB / kSlab; ++s) {
            const int cur = s & 1;
            if (s + 1 < KB / kSlab) load(cur ^ 1, s + 1);
#pragma unroll
            for (int i = 0; i < 5; ++i) {
                if (w + 8 * i >= 36) continue;
                const int ra = DB * tr[i] + rr, rb = DB * tc[i] + rr;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const d2_t a = *(const d2_t*)&sl[cur][ra][slab_pos(ra, 4 * h + lk)];
                    const d2_t b = *(const d2_t*)&sl[cur][rb][slab_pos(rb, 4 * h + lk)];
                    acc[i] = mfma(a[0], b[0], acc[i]);
                    acc[i] = mfma(a[1], b[1], acc[i]);
                }
            }
            loads_landed();
        }
    }
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
        for (int q = 0; q < NB / 8; ++q) {
            const int r = (b > 0 ? NB : 0) + w + 8 * q, c = (b > 1 ? NB : 0) + lane;
            const double v = r < nb && c <= r ? g[b][q] : (r == c && r >= nb ? 1.0 : 0.0);
            Tile& T = b == 0 ? B0 : b == 1 ? S10 : S11;
            T[w + 8 * q][lane] = v;
            if (b == 0) B1[w + 8 * q][lane] = 0.0;
        }
    __syncthreads();
    if (kb > 0) {
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            if (w + 8 * i >= 36) continue;
            Tile& T = tr[i] < 4 ? B0 : tc[i] < 4 ? S10 : S11;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (DB * tr[i] + 4 * q + lk < nb) T[(DB * tr[i] & 63) + 4 * q + lk][(DB * tc[i] & 63) + rr] -= acc[i][q];
        }
        __syncthreads();
    }
    bool bad = false;
    factor_block(B0, B1, bad);                     // B0 = L_00, B1 = X_00
    // L_10 = S_10 X_00^T: two 16 x 16 tiles a wavefront
    const int I = w & 3, Ja = w >> 2, Jb = 3 - Ja;
    d4_t t0 = {0.0, 0.0, 0.0, 0.0}, t1 = t0;
    for (int k = 0; k < DB * (Ja + 1); k += 4) t0 = mfma(S10[DB * I + rr][k + lk], B1[DB * Ja + rr][k + lk], t0);
    for (int k = 0; k < DB * (Jb + 1); k += 4) t1 = mfma(S10[DB * I + rr][k + lk], B1[DB * Jb + rr][k + lk], t1);
    auto put = [&](const Tile& T, int r0, int c0) {
#pragma unroll
        for (int q = 0; q < NB / 8; ++q) {
            const int r = r0 + w + 8 * q, c = c0 + lane;
            if (r < nb && c <= r) A[(o + r) * P + o + c] = T[w + 8 * q][lane];
        }
    };
    put(B0, 0, 0);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        S10[DB * I + 4 * q + lk][DB * Ja + rr] = t0[q];
        S10[DB * I + 4 * q + lk][DB * Jb + rr] = t1[q];
    }
#pragma unroll
    for (int q = 0; q < NB / 8; ++q) B0[w + 8 * q][lane] = 0.0;
    __syncthreads();
    // S_11 -= L_10 L_10^T
    for (int i = w; i < 10; i += 8) {
        const int R = i < 1 ? 0 : i < 3 ? 1 : i < 6 ? 2 : 3, C = i - R * (R + 1) / 2;
        d4_t acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < NB; k += 4) acc = mfma(S10[DB * R + rr][k + lk], S10[DB * C + rr][k + lk], acc);
#pragma unroll
        for (int q = 0; q < 4; ++q) S11[DB * R + 4 * q + lk][DB * C + rr] -= acc[q];
    }
    put(S10, NB, 0);
    __syncthreads();
    factor_block(S11, B0, bad);                    // S11 = L_11, B0 = X_11
    put(S11, NB, NB);
    if (tid == 0 && bad) flag[0] = 1;
    // X_10 = -X_11 (L_10 X_00): wavefront w column tile w mod 4, row tiles 0, 1 or 2, 3
    {
        const int J = w & 3, I0 = 2 * (1 - (w >> 2));
        d4_t v[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
        for (int K = 0; K <= I0 + 1; ++K) {
            d4_t t = {0.0, 0.0, 0.0, 0.0};
            for (int k = DB * J; k < NB; k += 4) t = mfma(S10[DB * K + rr][k + lk], B1[k + lk][DB * J + rr], t);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                v[1] = mfma(B0[DB * (I0 + 1) + rr][DB * K + 4 * q + lk], t[q], v[1]);
                if (K <= I0) v[0] = mfma(B0[DB * I0 + rr][DB * K + 4 * q + lk], t[q], v[0]);
            }
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) inv[(NB + DB * (I0 + i) + 4 * q + lk) * KB + DB * J + rr] = -v[i][q];
    }
    double* l0 = linv64 + (size_t)2 * kb * NB * NB;
#pragma unroll
    for (int q = 0; q < NB / 8; ++q) {
        const int r = w + 8 * q;
        const double x0 = B1[r][lane], x1 = B0[r][lane];
        inv[r * KB + lane] = x0;
        inv[r * KB + NB + lane] = 0.0;
        inv[(NB + r) * KB + NB + lane] = x1;
        l0[r * NB + lane] = x0;
        if (nb > NB) l0[NB * NB + r * NB + lane] = x1;
    }
}

// Step kb > 0: block 0 the diagonal block above; the other blocks the rest of the trailing update with the panel of
// block kb - 1, C -= L L^T on the 64 x 64 tiles of the lower triangle of C = A[o:, o:], o = 128 kb, but the first
// three (row by row; they are the diagonal block).  Step 0: the diagonal block alone.  One launch for the two, because
// on two streams the diagonal block's workgroup had to wait for a whole CU's LDS until the update drained.
//
// Update: a workgroup's two groups of 4 wavefronts take a tile each, 32 x 32 a wavefront, k in slabs of 16 straight
// into LDS, the next slab (or the next tile's first) in flight behind the products; C is read when its tile starts.
// Bound by the matrix cores at P = 5,000 (3,000 tiles of 1 MFLOP on the first step, 40 us).  Each XCD takes a contiguous
// run of the tiles, so that its L2 holds their panel rows.
constexpr int kStepBlocks = 256;
__global__ void __launch_bounds__(512) k_chol_step(double* __restrict__ A, int64_t P, int kb, int ntile,
                                                   int* __restrict__ flag, double* __restrict__ linv64,
                                                   double* __restrict__ inv)
{
    __shared__ __attribute__((aligned(1024))) double lds[kStepLds / sizeof(double)];
    if (blockIdx.x == 0) {
        diag_block(lds, A, P, kb, flag, linv64, inv);
        return;
    }
    const int l = threadIdx.x & 63, w8 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), w = w8 & 3, grp = w8 >> 2;
    const int rr = l & 15, lk = l >> 4, wr = w >> 1, wc = w & 1;
    // this group's tiles: t0, t0 + step, ... below t1; the workgroup runs as many rounds as its first group needs
    const int x = blockIdx.x & 7, per = (ntile + 7) >> 3;
    const int slot = (int)(blockIdx.x >> 3) - (x == 0), step = 2 * (kStepBlocks / 8 - (x == 0));
    const int t1 = (x + 1) * per < ntile ? (x + 1) * per : ntile;
    const int first = x * per + 2 * slot, rounds = first < t1 ? (t1 - first + step - 1) / step : 0;
    const int64_t o = (int64_t)kb * KB, rem = P - o;
    double(*sl)[2][NB][kSlab] = (double(*)[2][NB][kSlab])(lds + grp * (4 * NB * kSlab));
    const double *ga[2], *gb[2];
    auto tile = [&](int round, int64_t& r0, int64_t& c0) {
        const int t = first + grp + round * step;
        const int b = (t < t1 ? t : first) + 3;              // (past the end: any tile, not stored)
        int I = (int)((sqrtf(8.0f * b + 1.0f) - 1.0f) * 0.5f);
        while ((I + 1) * (I + 2) / 2 <= b) ++I;
        while (I * (I + 1) / 2 > b) --I;
        r0 = (int64_t)I * NB;
        c0 = (int64_t)(b - I * (I + 1) / 2) * NB;
        return t < t1;
    };
    auto point = [&](int64_t r0, int64_t c0) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int r = 16 * w + 8 * i + (l >> 3);
            const int c = slab_pos(r, l & 7);
            ga[i] = A + (o + (r0 + r < rem ? r0 + r : rem - 1)) * P + (o - KB) + c;
            gb[i] = A + (o + (c0 + r < rem ? c0 + r : rem - 1)) * P + (o - KB) + c;
        }
    };
    auto load = [&](int buf, int s) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            load_lds(ga[i] + kSlab * s, &sl[buf][0][16 * w + 8 * i][0]);
            load_lds(gb[i] + kSlab * s, &sl[buf][1][16 * w + 8 * i][0]);
        }
    };
    if (rounds == 0) return;
    int64_t r0, c0, rn = 0, cn = 0;
    bool live = tile(0, r0, c0), next = false;
    point(r0, c0);
    load(0, 0);
    loads_landed();
    for (int round = 0; round < rounds; ++round) {
        double c[2][2][4];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int64_t r = r0 + 32 * wr + 16 * i + 4 * q + lk, k = c0 + 32 * wc + 16 * j + rr;
                    const bool in = r < rem && k <= r;
                    c[i][j][q] = A[(o + (in ? r : 0)) * P + o + (in ? k : 0)];
                }
        d4_t acc[2][2];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = d4_t{0.0, 0.0, 0.0, 0.0};
        for (int s = 0; s < KB / kSlab; ++s) {
            const int cur = s & 1;
            if (s + 1 < KB / kSlab) {
                load(cur ^ 1, s + 1);
            } else if (round + 1 < rounds) {
                next = tile(round + 1, rn, cn);
                point(rn, cn);
                load(0, 0);
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                d2_t a[2], b[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int ra = 32 * wr + 16 * i + rr, rb = 32 * wc + 16 * i + rr;
                    a[i] = *(const d2_t*)&sl[cur][0][ra][slab_pos(ra, 4 * h + lk)];
                    b[i] = *(const d2_t*)&sl[cur][1][rb][slab_pos(rb, 4 * h + lk)];
                }
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int j = 0; j < 2; ++j) acc[i][j] = mfma(a[i][t], b[j][t], acc[i][j]);
            }
            loads_landed();
        }
        if (live) {
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int64_t r = r0 + 32 * wr + 16 * i + 4 * q + lk, k = c0 + 32 * wc + 16 * j + rr;
                        if (r < rem && k <= r) A[(o + r) * P + o + k] = c[i][j][q] - acc[i][j][q];
                    }
        }
        live = next;
        r0 = rn;
        c0 = cn;
    }
}

// Panel rows (32 a block) below block kb, in place: row <- row L_kk^{-T}, with inv the block's inverse
// [128][128].  Operands go straight into LDS and from there to the MFMAs as in k_gemm_f64_nt (gemm.hip); a block
// owns whole rows, so that its stores, after its last load, meet no other block's loads.  P is even (16-byte loads).
// Bound by latency (8 slabs of 16 k); 32 rows a block for 150 blocks at P = 5,000.
constexpr int kPanelRows = 32;
__global__ void __launch_bounds__(256) k_panel(double* __restrict__ A, int64_t P, int kb, const double* __restrict__ inv)
{
    __shared__ __attribute__((aligned(1024))) double Sa[2][kPanelRows][kSlab], Sb[2][KB][kSlab];
    const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rr = l & 15, lk = l >> 4;
    const int64_t o = (int64_t)kb * KB, row0 = o + KB + (int64_t)blockIdx.x * kPanelRows;
    const int ra = 8 * w + (l >> 3);
    const double* ga = A + (row0 + ra < P ? row0 + ra : P - 1) * P + o + slab_pos(ra, l & 7);
    const double* gb[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = 32 * w + 8 * i + (l >> 3);
        gb[i] = inv + (size_t)r * KB + slab_pos(r, l & 7);
    }
    auto load = [&](int buf, int s) {
        load_lds(ga + kSlab * s, &Sa[buf][8 * w][0]);
#pragma unroll
        for (int i = 0; i < 4; ++i) load_lds(gb[i] + kSlab * s, &Sb[buf][32 * w + 8 * i][0]);
    };
    d4_t acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = d4_t{0.0, 0.0, 0.0, 0.0};
    load(0, 0);
    loads_landed();
    for (int s = 0; s < KB / kSlab; ++s) {
        const int cur = s & 1;
        if (s + 1 < KB / kSlab) load(cur ^ 1, s + 1);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            d2_t a[2], b[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int r = 16 * i + rr, c = 32 * w + r;
                a[i] = *(const d2_t*)&Sa[cur][r][slab_pos(r, 4 * h + lk)];
                b[i] = *(const d2_t*)&Sb[cur][c][slab_pos(c, 4 * h + lk)];
            }
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) acc[i][j] = mfma(a[i][t], b[j][t], acc[i][j]);
        }
        loads_landed();
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t r = row0 + 16 * i + 4 * q + lk;
            if (r >= P) continue;
#pragma unroll
            for (int j = 0; j < 2; ++j) A[r * P + o + 32 * w + 16 * j + rr] = acc[i][j][q];
        }
}

// Forward step kb of L y = b with the inverted diagonal blocks, B [P][nrhs]: every block
// forms y_kb = Linv_kb b_kb; block 0 writes it to Y, block t >= 1 subtracts L y_kb from the
// 64 rows starting at o + 64 t (B rows of block kb itself are not modified in this step).
// 256 threads: operand tiles are staged in LDS, each wave loading 16 rows, and the products
// are split over the 4 waves by k and summed in LDS.
constexpr int kMaxRhs = 4;
// the four waves' partial sums of row t
__device__ inline void solve_sum(const double (*part)[NB][kMaxRhs], int t, int nrhs, double* out)
{
    for (int c = 0; c < nrhs; ++c) out[c] = part[0][t][c] + part[1][t][c] + part[2][t][c] + part[3][t][c];
}

template <int nrhs>
__global__ void __launch_bounds__(256) k_fwd_step(const double* __restrict__ A, int64_t P, int kb,
                                                  const double* __restrict__ Linv, double* __restrict__ B,
                                                  double* __restrict__ Y)
{
    __shared__ double T[NB][NB + 1];
    __shared__ double At[NB][NB + 1];   // the block's rows of L (loaded with T: it does not depend on y)
    __shared__ double bk[NB][kMaxRhs];
    __shared__ double y[NB][kMaxRhs];
    __shared__ double part[4][NB][kMaxRhs];
    const int64_t o = (int64_t)kb * NB;
    const int nb = (int)(P - o < NB ? P - o : NB);
    const int t = threadIdx.x & 63, w = threadIdx.x >> 6;
    const double* L0 = Linv + (size_t)kb * NB * NB;
    const int64_t r0 = o + (int64_t)blockIdx.x * NB;
    const int nr = blockIdx.x == 0 ? 0 : (int)(P - r0 < NB ? P - r0 : NB);
    // loads first (all in flight; entries past the matrix read an in-bounds one and are then zeroed)
    double gl[NB / 4], ga[NB / 4];
#pragma unroll
    for (int q = 0; q < NB / 4; ++q) {
        const int r = w + 4 * q;
        gl[q] = L0[(size_t)r * NB + t];
        ga[q] = blockIdx.x != 0 ? A[(r0 + (r < nr ? r : 0)) * P + o + (t < nb ? t : 0)] : 0.0;
    }
#pragma unroll
    for (int q = 0; q < NB / 4; ++q) {
        const int r = w + 4 * q;
        T[r][t] = gl[q];
        At[r][t] = (r < nr && t < nb) ? ga[q] : 0.0;
    }
    if (w == 0)
        for (int c = 0; c < nrhs; ++c) bk[t][c] = t < nb ? B[(o + t) * nrhs + c] : 0.0;
    __syncthreads();
    {
        double acc[nrhs] = {};
        for (int k = 16 * w; k < 16 * w + 16; ++k) {
            const double l = T[t][k];
            for (int c = 0; c < nrhs; ++c) acc[c] += l * bk[k][c];
        }
        for (int c = 0; c < nrhs; ++c) part[w][t][c] = acc[c];
    }
    __syncthreads();
    if (w == 0) {
        double v[nrhs];
        solve_sum(part, t, nrhs, v);
        for (int c = 0; c < nrhs; ++c) y[t][c] = v[c];
        if (blockIdx.x == 0 && t < nb)
            for (int c = 0; c < nrhs; ++c) Y[(o + t) * nrhs + c] = v[c];
    }
    if (blockIdx.x == 0) return;
    __syncthreads();
    {
        double acc[nrhs] = {};
        for (int k = 16 * w; k < 16 * w + 16; ++k) {
            const double l = At[t][k];
            for (int c = 0; c < nrhs; ++c) acc[c] += l * y[k][c];
        }
        for (int c = 0; c < nrhs; ++c) part[w][t][c] = acc[c];
    }
    __syncthreads();
    if (w == 0 && t < nr) {
        double v[nrhs];
        solve_sum(part, t, nrhs, v);
        for (int c = 0; c < nrhs; ++c) B[(r0 + t) * nrhs + c] -= v[c];
    }
}

// Backward step kb of L^T x = y: every block forms x_kb = Linv_kb^T y_kb; block 0 writes it
// to X, block t >= 1 subtracts L[block kb rows, c]^T x_kb from the 64 entries of Y starting
// at column c = 64 (t - 1) (only columns before block kb; Y rows of block kb are only read).
template <int nrhs>
__global__ void __launch_bounds__(256) k_bwd_step(const double* __restrict__ A, int64_t P, int kb,
                                                  const double* __restrict__ Linv, double* __restrict__ Y,
                                                  double* __restrict__ X)
{
    __shared__ double T[NB][NB + 1];
    __shared__ double At[NB][NB + 1];   // block kb's rows of L at this block's columns (loaded with T)
    __shared__ double yk[NB][kMaxRhs];
    __shared__ double x[NB][kMaxRhs];
    __shared__ double part[4][NB][kMaxRhs];
    const int64_t o = (int64_t)kb * NB;
    const int nb = (int)(P - o < NB ? P - o : NB);
    const int t = threadIdx.x & 63, w = threadIdx.x >> 6;
    const double* L0 = Linv + (size_t)kb * NB * NB;
    const int64_t col = (int64_t)(blockIdx.x - 1) * NB + t;
    // loads first (all in flight; entries past the matrix read an in-bounds one and are then zeroed)
    double gl[NB / 4], ga[NB / 4];
#pragma unroll
    for (int q = 0; q < NB / 4; ++q) {
        const int r = w + 4 * q;
        gl[q] = L0[(size_t)r * NB + t];
        ga[q] = blockIdx.x != 0 ? A[(o + (r < nb ? r : 0)) * P + (col < o ? col : 0)] : 0.0;
    }
#pragma unroll
    for (int q = 0; q < NB / 4; ++q) {
        const int r = w + 4 * q;
        T[r][t] = gl[q];
        At[r][t] = (r < nb && col < o) ? ga[q] : 0.0;
    }
    if (w == 0)
        for (int c = 0; c < nrhs; ++c) yk[t][c] = t < nb ? Y[(o + t) * nrhs + c] : 0.0;
    __syncthreads();
    {
        double acc[nrhs] = {};
        for (int k = 16 * w; k < 16 * w + 16; ++k) {
            const double l = T[k][t];                  // (Linv^T)[t][k]
            for (int c = 0; c < nrhs; ++c) acc[c] += l * yk[k][c];
        }
        for (int c = 0; c < nrhs; ++c) part[w][t][c] = acc[c];
    }
    __syncthreads();
    if (w == 0) {
        double v[nrhs];
        solve_sum(part, t, nrhs, v);
        for (int c = 0; c < nrhs; ++c) x[t][c] = v[c];
        if (blockIdx.x == 0 && t < nb)
            for (int c = 0; c < nrhs; ++c) X[(o + t) * nrhs + c] = v[c];
    }
    if (blockIdx.x == 0) return;
    __syncthreads();
    {
        double acc[nrhs] = {};
        for (int r = 16 * w; r < 16 * w + 16; ++r) {
            const double l = At[r][t];
            for (int c = 0; c < nrhs; ++c) acc[c] += l * x[r][c];
        }
        for (int c = 0; c < nrhs; ++c) part[w][t][c] = acc[c];
    }
    __syncthreads();
    if (w == 0 && col < o) {
        double v[nrhs];
        solve_sum(part, t, nrhs, v);
        for (int c = 0; c < nrhs; ++c) Y[col * nrhs + c] -= v[c];
    }
}

}  // namespace

// Damp, factor and check: returns BEM_ENOTPD when a pivot fails (host sync).  Blocked right-looking with
// 128-column steps of two launches: the panel as A21 L^{-T} (in place), then the next diagonal block (updated, factored,
// inverted) beside the rest of the trailing lower triangle's rank-128 update.  The inverted 64 x 64 diagonal blocks stay in
// the context for chol_solve.  P is even (handles have 14 or 20 parameters).  64-column steps, the diagonal chain and
// the update on two streams, took 5.8 ms at P = 5,000: a 65 us chain a step, and 5 GB of reading and writing the
// trailing matrix.  Now 2.9 ms.
int chol_factor(bem_ctx* ctx, const double* H, int64_t P, double lam, double* A, int* dflag, double* dscal,
                hipStream_t s)
{
    int rc;
    const int nblk = (int)((P + KB - 1) / KB), n64 = (int)((P + NB - 1) / NB);
    // cholw: inverted diagonal blocks [n64][64][64] | solve vector [P][4] | the step's inverse [128][128]
    const size_t vo = (size_t)n64 * NB * NB, io = vo + (size_t)P * kMaxRhs;
    if ((rc = ensure(ctx, ctx->cholw, (io + KB * KB) * sizeof(double), s))) return rc;
    double* linv = (double*)ctx->cholw.ptr;
    double* inv = linv + io;
    hipLaunchKernelGGL(k_diag_max, dim3(1), dim3(256), 0, s, H, P, dscal);
    hipLaunchKernelGGL(k_damp, dim3(blocks_for(P, 256), P), dim3(256), 0, s, H, P, lam, dscal, A);
    if ((rc = fill_i32(ctx, dflag, 1, 0, s))) return rc;
    ProfScope ps_(ctx, PT_CHOLESKY, s);
    for (int kb = 0; kb < nblk; ++kb) {
        const int64_t rem = P - (int64_t)kb * KB;                   // the trailing matrix of the step before
        const int nt = blocks_for(rem, NB), ntile = kb > 0 && rem > KB ? nt * (nt + 1) / 2 - 3 : 0;
        if (kb > 0)
            hipLaunchKernelGGL(k_panel, dim3(blocks_for(rem, kPanelRows)), dim3(256), 0, s, A, P, kb - 1, (const double*)inv);
        hipLaunchKernelGGL(k_chol_step, dim3(ntile > 0 ? kStepBlocks : 1), dim3(512), 0, s, A, P, kb, ntile, dflag, linv, inv);
    }
    if ((rc = check_launch(ctx, "cholesky"))) return rc;
    ctx->chol_P = P;
    int hflag = 0;
    if (hipMemcpyAsync(&hflag, dflag, sizeof(int), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return set_error(ctx, BEM_EHIP, "cholesky flag readback");
    return hflag ? BEM_ENOTPD : BEM_OK;
}

// B <- (L L^T)^{-1} B with the factor in A and the inverted diagonal blocks of the last
// chol_factor; B [P][nrhs] row-major, nrhs <= 4.  One launch per block and direction.
// Forward then backward block steps for nrhs right-hand sides (B [P][nrhs] in, solution out; Y [P][nrhs] scratch).
template <int nrhs>
static void solve_steps(const double* A, int64_t P, int nblk, const double* linv, double* B, double* Y, hipStream_t s)
{
    for (int kb = 0; kb < nblk; ++kb) {
        const int64_t rem = P - (int64_t)(kb + 1) * NB;
        const int nbk = 1 + (rem > 0 ? blocks_for(rem, NB) : 0);
        hipLaunchKernelGGL(k_fwd_step<nrhs>, dim3(nbk), dim3(256), 0, s, A, P, kb, linv, B, Y);
    }
    for (int kb = nblk - 1; kb >= 0; --kb) {
        const int64_t o = (int64_t)kb * NB;
        const int nbk = 1 + (o > 0 ? blocks_for(o, NB) : 0);
        hipLaunchKernelGGL(k_bwd_step<nrhs>, dim3(nbk), dim3(256), 0, s, A, P, kb, linv, Y, B);
    }
}

int chol_solve(bem_ctx* ctx, const double* A, int64_t P, double* B, int nrhs, hipStream_t s)
{
    if (nrhs < 1 || nrhs > kMaxRhs) return set_error(ctx, BEM_EINVAL, "chol_solve: 1..4 right-hand sides");
    if (ctx->chol_P != P) return set_error(ctx, BEM_ESTATE, "chol_solve without a matching chol_factor");
    ProfScope ps_(ctx, PT_CHOLESKY, s);
    const int nblk = (int)((P + NB - 1) / NB);
    const double* linv = (const double*)ctx->cholw.ptr;
    double* Y = (double*)ctx->cholw.ptr + (size_t)nblk * NB * NB;
    switch (nrhs) {
    case 1: solve_steps<1>(A, P, nblk, linv, B, Y, s); break;
    case 2: solve_steps<2>(A, P, nblk, linv, B, Y, s); break;
    case 3: solve_steps<3>(A, P, nblk, linv, B, Y, s); break;
    default: solve_steps<4>(A, P, nblk, linv, B, Y, s); break;
    }
    return check_launch(ctx, "cholesky solve");
}

}  // namespace bem
