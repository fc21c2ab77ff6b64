// chol.hip - float64 Cholesky of the damped approximate Hessian
// lambda D + J^T J (Eq. optimstep: positive definite, solved by Cholesky,
// Sec. 4.3) and the two triangular solves for the LM step.
// Blocked right-looking factorisation with 128-column panels: the diagonal block
// in one workgroup's LDS, inverted in the same kernel; the panel as a GEMM
// with that inverse; the trailing update as a rank-128 symmetric update.  The solves
// use the inverted diagonal blocks: the forward one as further rows of the matrix, the
// backward one a launch per block.  A
// non-positive or non-finite pivot raises a device flag.
#include <utility>

#include "common.hpp"
#include "math64.hpp"
#include "sweep_common.hpp"

namespace bem {

namespace {

constexpr int NB = 64;       // half a diagonal block, and the trailing update's tile
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

// A = H + lam * diag(max(H_ii, 1e-12 * max_j H_jj)), lower triangle
__global__ void k_damp(const double* __restrict__ H, int64_t P, double lam, const double* __restrict__ dmax,
                       double* __restrict__ A)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t i = blockIdx.y;
    if (j > i) return;
    double v = H[i * P + j];
    if (i == j) v += lam * fmax(v, 1e-12 * dmax[0]);
    A[i * P + j] = v;
}

// The right-hand sides B [P][nrhs] as rows of A from Ar on, then KB zeros: the last block's panel loads whole slabs
// past the rows' ends.
__global__ void k_rhs_rows(const double* __restrict__ B, int64_t P, int nrhs, double* __restrict__ Ar)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int c = blockIdx.y;
    if (c == nrhs) {
        if (j < KB) Ar[nrhs * P + j] = 0.0;
    } else if (j < P) {
        Ar[c * P + j] = B[j * nrhs + c];
    }
}

// rows of the matrix being factored: the first P and the right-hand sides'
struct Rows {
    int64_t P, Pr;
    int nrhs;
    __device__ bool has(int64_t r) const { return r < P || (r >= Pr && r < Pr + nrhs); }
};

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
// (trailing updates, the inverse's off-diagonal blocks) is float64 MFMA out of LDS, spread over 8 wavefronts, and where
// nothing waits for it beside the panels.  LDS rows of kLd doubles: the 16 rows x 4 k of an operand read fall in distinct
// banks.  Operand and accumulator layout of v_mfma_f64_16x16x4f64 (lane l, rr = l mod 16, lk = l / 16): A[rr][lk],
// B[lk][rr], element q of the accumulator is row 4 q + lk, column rr; so element q of a product is the B operand of
// k step q of the next product.
// Measured: 45 us a block of 128 with its update (55 us with the whole update first and the inverse after; blocks of
// 64 by broadcast sums: 2 x 47 us); the 8 panels are 15 us of it.
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

// Every LDS access before is done, in every wavefront; global stores stay in flight (__syncthreads waits for them).
__device__ inline void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// S [64][64] (lower triangle) -> its factor in place, X -> the inverse (lower triangle).  All 8 wavefronts; while one
// factors panel p the others do side(p).
template <class Side>
__device__ __forceinline__ void factor_block(Tile& S, Tile& X, bool& bad, Side side)
{
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rr = lane & 15, lk = lane >> 4;
#pragma unroll 1                                     // (unrolled, the code outgrows the instruction cache)
    for (int p = 0; p < NB / DB; ++p) {
        const int d0 = p * DB;
        if (w == 0) {
            __builtin_amdgcn_s_setprio(3);
            const int r = d0 + DB * (lk + 1) + rr;       // this lane's row below the diagonal block
            const bool below = lk < 3 && r < NB;
            double a[DB], b[DB];
#pragma unroll
            for (int k = 0; k < DB; k += 2) {
                const d2_t v = *(const d2_t*)&S[d0 + rr][d0 + k], u = *(const d2_t*)&S[below ? r : 0][d0 + k];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    a[k + h] = k + h <= rr ? v[h] : 0.0;
                    b[k + h] = below ? u[h] : (lk == 3 && k + h == rr ? 1.0 : 0.0);
                }
            }
            panel_factor(a, b, bad, std::make_integer_sequence<int, DB>{});
            // (above the diagonal S gets values that nothing reads, X its zeros)
            if (lk == 0) {
#pragma unroll
                for (int k = 0; k < DB; k += 2) *(d2_t*)&S[d0 + rr][d0 + k] = d2_t{a[k], a[k + 1]};
            }
            if (below) {
#pragma unroll
                for (int k = 0; k < DB; k += 2) *(d2_t*)&S[r][d0 + k] = d2_t{b[k], b[k + 1]};
            }
            if (lk == 3) {
#pragma unroll
                for (int k = 0; k < DB; ++k) X[d0 + k][d0 + rr] = b[k];       // (L^-T)[rr][k]
            }
            __builtin_amdgcn_s_setprio(0);
        } else {
            side(p);
        }
        lds_barrier();
        // trailing 16 x 16 tiles (I, J), I >= J: S -= L L^T
        const int t = NB / DB - 1 - p;
        if (w < t * (t + 1) / 2) {
            const int I = w < 1 ? 0 : w < 3 ? 1 : 2, J = w - I * (I + 1) / 2;
            const int r0 = d0 + DB * (I + 1), c0 = d0 + DB * (J + 1);
            d4_t acc = {0.0, 0.0, 0.0, 0.0};
            double c[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) c[q] = S[r0 + 4 * q + lk][c0 + rr];
#pragma unroll
            for (int k = 0; k < DB; k += 4) acc = mfma(S[r0 + rr][d0 + k + lk], S[c0 + rr][d0 + k + lk], acc);
#pragma unroll
            for (int q = 0; q < 4; ++q) S[r0 + 4 * q + lk][c0 + rr] = c[q] - acc[q];
        }
        if (t > 0) lds_barrier();
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
    lds_barrier();
    if (w < 4) {
        const int I = 2 + (w >> 1), J = w & 1;
        // (L_10 X_00)(K, J), K = 2, 3; X_00's upper block is zero, and skipped
        d4_t t[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}}, v = t[0];
        auto add = [&](int k0) {
#pragma unroll
            for (int k = k0; k < k0 + DB; k += 4)
#pragma unroll
                for (int K = 0; K < 2; ++K)
                    t[K] = mfma(S[DB * (K + 2) + rr][k + lk], X[k + lk][DB * J + rr], t[K]);
        };
        if (J == 0) add(0);
        add(DB);
#pragma unroll
        for (int K = 0; K < 2; ++K) {
            if (K + 2 > I) continue;
#pragma unroll
            for (int q = 0; q < 4; ++q) v = mfma(X[DB * I + rr][DB * (K + 2) + 4 * q + lk], t[K][q], v);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) X[DB * I + 4 * q + lk][DB * J + rr] = -v[q];
    }
    lds_barrier();
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
// triangle); its inverse to inv [128][128].  Rows and columns past the matrix are an identity block.
// Only the first 64 x 64 block's update is waited for.  Beside its panels, which are one wavefront's, the
// others update the rest, a quarter of the previous panel's columns each time, and beside the second block's they finish
// that block's update, take the inverse's first product and store what is done.
__device__ __forceinline__ void diag_block(double* lds, double* __restrict__ A, int64_t P, int kb, int* __restrict__ flag,
                                           double* __restrict__ inv)
{
    Tile& B0 = *(Tile*)lds;
    Tile& B1 = *((Tile*)lds + 1);
    Tile& S10 = *((Tile*)lds + 2);
    Tile& S11 = *((Tile*)lds + 3);
    const int64_t o = (int64_t)kb * KB;
    const int nb = (int)(P - o < KB ? P - o : KB);
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rr = lane & 15, lk = lane >> 4;
    // rows 8 i .. 8 i + 7 of slab s of the previous panel's rows at this block, to row 8 i of sl
    auto load = [&](int s, int i, double (*sl)[kSlab]) {
        const int r = 8 * i + (lane >> 3);
        load_lds(A + (o + (r < nb ? r : 0)) * P + (o - KB) + kSlab * s + slab_pos(r, lane & 7), &sl[8 * i][0]);
    };
    // acc += L L^T, 16 x 16 tile (R, C) of a slab
    auto product = [&](int R, int C, double (*sl)[kSlab], d4_t& acc) {
        const int ra = DB * R + rr, rb = DB * C + rr;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const d2_t a = *(const d2_t*)&sl[ra][slab_pos(ra, 4 * h + lk)];
            const d2_t b = *(const d2_t*)&sl[rb][slab_pos(rb, 4 * h + lk)];
            acc = mfma(a[0], b[0], acc);
            acc = mfma(a[1], b[1], acc);
        }
    };
    // tile (R, C) of the matrix (outside it the first element is read and then replaced), and less acc into LDS
    auto read = [&](int R, int C, double (&v)[4]) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int r = DB * R + 4 * q + lk, c = DB * C + rr;
            const bool in = r < nb && c <= r;
            v[q] = A[(o + (in ? r : 0)) * P + o + (in ? c : 0)];
        }
    };
    auto place = [&](int R, int C, const double (&v)[4], const d4_t& acc) {
        Tile& T = R < 4 ? B0 : C < 4 ? S10 : S11;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int r = DB * R + 4 * q + lk, c = DB * C + rr;
            T[r & (NB - 1)][c & (NB - 1)] = r >= nb ? (r == c ? 1.0 : 0.0) : c <= r ? v[q] - acc[q] : 0.0;
        }
    };
    constexpr int kFirst = 10, kTiles = 36;          // tiles (R, C), C <= R < 8, row by row; those of the first block
    auto tile_of = [](int t, int& R, int& C) {
        R = t < 1 ? 0 : t < 3 ? 1 : t < 6 ? 2 : t < 10 ? 3 : t < 15 ? 4 : t < 21 ? 5 : t < 28 ? 6 : 7;
        C = t - R * (R + 1) / 2;
    };
    // the first block's rows whole in B1 and S10, the first quarter of all rows in S11; quarters 1 and 3 go to S10
    constexpr int kSlabs = KB / kSlab, kQuarter = kSlabs / (NB / DB), kRows8 = KB / 8;
    double(*whole)[NB][kSlab] = (double(*)[NB][kSlab])&B1;
    double(*quarter[2])[KB][kSlab] = {(double(*)[KB][kSlab])&S11, (double(*)[KB][kSlab])&S10};
    static_assert(kSlabs * sizeof(*whole) <= 2 * sizeof(Tile) && kQuarter * sizeof(*quarter[0]) <= sizeof(Tile), "");
    if (kb > 0) {
#pragma unroll
        for (int s = 0; s < kSlabs; ++s) load(s, w, whole[s]);
#pragma unroll
        for (int j = 0; j < kQuarter * kRows8 / 8; ++j) load(j >> 1, w + 8 * (j & 1), quarter[0][j >> 1]);
    }
    {
        double v[2][4];
        d4_t acc[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
        int R[2], C[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            tile_of(w + 8 * i < kFirst ? w + 8 * i : 0, R[i], C[i]);
            read(R[i], C[i], v[i]);
        }
        if (kb > 0) {
            loads_landed();
#pragma unroll
            for (int s = 0; s < kSlabs; ++s) {
                product(R[0], C[0], whole[s], acc[0]);
                if (w + 8 < kFirst) product(R[1], C[1], whole[s], acc[1]);
            }
        }
        place(R[0], C[0], v[0], acc[0]);
        if (w + 8 < kFirst) place(R[1], C[1], v[1], acc[1]);
        lds_barrier();
    }
    bool bad = false;
    // the other 26: four for wavefronts 1 to 3 and 5 to 7, two for 4, which shares the panel's SIMD
    constexpr int kSide = 4;
    const int side = w == 0 ? kTiles : w == 4 ? kTiles - 2 : kFirst + w - (w < 4 ? 1 : 2), side_step = w == 4 ? 1 : 6;
    d4_t acc[kSide];
    double v[kSide][4];
    int tr[kSide], tc[kSide];
#pragma unroll
    for (int i = 0; i < kSide; ++i) {
        acc[i] = d4_t{0.0, 0.0, 0.0, 0.0};
        const int t = side + side_step * i;
        tile_of(t < kTiles ? t : kTiles - 1, tr[i], tc[i]);
    }
    factor_block(B0, B1, bad, [&](int p) {           // B0 = L_00, B1 = X_00
        if (kb > 0) {
            if (p + 1 < NB / DB)
                for (int j = w - 1; j < kQuarter * kRows8; j += 7)
                    load(kQuarter * (p + 1) + j / kRows8, j % kRows8, quarter[(p + 1) & 1][j / kRows8]);
#pragma unroll
            for (int s = 0; s < kQuarter; ++s)
#pragma unroll
                for (int i = 0; i < kSide; ++i)
                    if (side + side_step * i < kTiles) product(tr[i], tc[i], quarter[p & 1][s], acc[i]);
        }
        if (p + 1 == NB / DB) {
#pragma unroll
            for (int i = 0; i < kSide; ++i) read(tr[i], tc[i], v[i]);
        }
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0);               // the next quarter has landed
    });
    // rows first, first + step, ... of a factor's tile to the matrix
    auto put = [&](const Tile& T, int r0, int c0, int first, auto step) {
#pragma unroll
        for (int i = 0; i < NB; i += decltype(step)::value) {
            const int r = r0 + i + first, c = c0 + lane;
            const double x = T[i + first][lane];
            if (r < nb && c <= r) A[(o + r) * P + o + c] = x;
        }
    };
    put(B0, 0, 0, w, std::integral_constant<int, 8>{});
#pragma unroll
    for (int i = 0; i < kSide; ++i)
        if (side + side_step * i < kTiles) place(tr[i], tc[i], v[i], acc[i]);
    lds_barrier();
    // L_10 = S_10 X_00^T: two 16 x 16 tiles a wavefront, columns J and 3 - J
    const int I = w & 3;
    d4_t t0 = {0.0, 0.0, 0.0, 0.0}, t1 = t0;
    auto solve = [&](auto first) {
        constexpr int Ja = decltype(first)::value, Jb = 3 - Ja;
#pragma unroll
        for (int k = 0; k < DB * (Jb + 1); k += 4) {
            const double a = S10[DB * I + rr][k + lk];
            if (k < DB * (Ja + 1)) t0 = mfma(a, B1[DB * Ja + rr][k + lk], t0);
            t1 = mfma(a, B1[DB * Jb + rr][k + lk], t1);
        }
    };
    if (w < 4) solve(std::integral_constant<int, 0>{});
    else solve(std::integral_constant<int, 1>{});
    lds_barrier();
    {
        const int Ja = w >> 2, Jb = 3 - Ja;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int r = DB * I + 4 * q + lk;
            S10[r][DB * Ja + rr] = t0[q];
            S10[r][DB * Jb + rr] = t1[q];
            if (NB + r < nb) {
                A[(o + NB + r) * P + o + DB * Ja + rr] = t0[q];
                A[(o + NB + r) * P + o + DB * Jb + rr] = t1[q];
            }
        }
    }
    lds_barrier();
    // S_11 -= L_10 L_10^T: the first tile column now, the other six tiles beside the first panel
    auto reduce = [&](int R, int C) {
        d4_t s[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
#pragma unroll
        for (int k = 0; k < NB; k += 4)
            s[(k >> 2) & 1] = mfma(S10[DB * R + rr][k + lk], S10[DB * C + rr][k + lk], s[(k >> 2) & 1]);
#pragma unroll
        for (int q = 0; q < 4; ++q) S11[DB * R + 4 * q + lk][DB * C + rr] -= s[0][q] + s[1][q];
    };
    if (w < 4) reduce(w, 0);
    lds_barrier();
    // wavefronts 4 to 7: tile column J of T = L_10 X_00, in registers; 1 to 3: X_00 to inv
    const int J = 7 - w;
    d4_t T[NB / DB];
#pragma unroll
    for (int K = 0; K < NB / DB; ++K) T[K] = d4_t{0.0, 0.0, 0.0, 0.0};
    factor_block(S11, B0, bad, [&](int p) {          // S11 = L_11, B0 = X_11
        if (p == 0 && w < 7) {
            const int R = w < 2 ? 1 : w < 4 ? 2 : 3;
            reduce(R, w - R * (R - 1) / 2);
        }
        if (w >= 4) {
            d4_t t = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int k0 = 0; k0 < NB; k0 += DB) {
                if (k0 < DB * J) continue;           // X_00 is zero there
#pragma unroll
                for (int k = k0; k < k0 + DB; k += 4)
                    t = mfma(S10[DB * p + rr][k + lk], B1[k + lk][DB * J + rr], t);
            }
#pragma unroll
            for (int K = 0; K < NB / DB; ++K)
                if (K == p) T[K] = t;
        } else {
            for (int i = DB * p + w - 1; i < DB * (p + 1); i += 3) {
                inv[i * KB + lane] = lane <= i ? B1[i][lane] : 0.0;
                inv[i * KB + NB + lane] = 0.0;
            }
        }
    });
    if (tid == 0 && bad) flag[0] = 1;
    if (w >= 4) {                                    // X_10 = -X_11 T
#pragma unroll
        for (int i = 0; i < NB / DB; ++i) {
            d4_t x = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int K = 0; K <= i; ++K)
#pragma unroll
                for (int q = 0; q < 4; ++q) x = mfma(B0[DB * i + rr][DB * K + 4 * q + lk], T[K][q], x);
#pragma unroll
            for (int q = 0; q < 4; ++q) inv[(NB + DB * i + 4 * q + lk) * KB + DB * J + rr] = -x[q];
        }
    } else {
        put(S11, NB, NB, w, std::integral_constant<int, 4>{});
#pragma unroll
        for (int i = 0; i < NB; i += 4) {
            const double x = B0[i + w][lane];
            inv[(NB + i + w) * KB + NB + lane] = lane <= i + w ? x : 0.0;
        }
    }
}

// Step kb > 0: block 0 the diagonal block above; the other blocks the rest of the trailing update with the panel of
// block kb - 1, C -= L L^T on the 64 x 64 tiles of the lower triangle of C = A[o:, o:], o = 128 kb, but the first
// three (row by row; they are the diagonal block), and on the right-hand sides' rows.  Step 0: the diagonal block alone.  One launch for the two, because
// on two streams the diagonal block's workgroup had to wait for a whole CU's LDS until the update drained.
//
// Update: a workgroup's two groups of 4 wavefronts take a tile each, 32 x 32 a wavefront, k in slabs of 16 straight
// into LDS, the next slab (or the next tile's first) in flight behind the products; C is read when its tile starts.
// Bound by the matrix cores at P = 5,000 (3,000 tiles of 1 MFLOP on the first step, 40 us).  Each XCD takes a contiguous
// run of the tiles, so that its L2 holds their panel rows.
constexpr int kStepBlocks = 256;
__global__ void __launch_bounds__(512) k_chol_step(double* __restrict__ A, Rows R, int kb, int ntile,
                                                   int* __restrict__ flag, double* __restrict__ inv)
{
    __shared__ __attribute__((aligned(1024))) double lds[kStepLds / sizeof(double)];
    const int64_t P = R.P;
    if (blockIdx.x == 0) {
        diag_block(lds, A, P, kb, flag, inv);
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
            ga[i] = A + (R.has(o + r0 + r) ? o + r0 + r : o) * P + (o - KB) + c;
            gb[i] = A + (c0 + r < rem ? o + c0 + r : o) * P + (o - KB) + c;
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
                    const bool in = R.has(o + r) && k <= r && k < rem;
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
                        if (R.has(o + r) && k <= r && k < rem) A[(o + r) * P + o + k] = c[i][j][q] - acc[i][j][q];
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
__global__ void __launch_bounds__(256) k_panel(double* __restrict__ A, Rows R, int kb, const double* __restrict__ inv)
{
    __shared__ __attribute__((aligned(1024))) double Sa[2][kPanelRows][kSlab], Sb[2][KB][kSlab];
    const int64_t P = R.P;
    const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rr = l & 15, lk = l >> 4;
    const int64_t o = (int64_t)kb * KB, row0 = o + KB + (int64_t)blockIdx.x * kPanelRows;
    const int ra = 8 * w + (l >> 3);
    const double* ga = A + (R.has(row0 + ra) ? row0 + ra : 0) * P + o + slab_pos(ra, l & 7);
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
            if (!R.has(r)) continue;
#pragma unroll
            for (int j = 0; j < 2; ++j)
                if (o + 32 * w + 16 * j + rr < P) A[r * P + o + 32 * w + 16 * j + rr] = acc[i][j][q];
        }
}

constexpr int kMaxRhs = 4;

// Backward step kb of L^T x = y (128 columns), Y [nrhs][P]: every block forms x_kb = L_kk^{-T} y_kb; block 0 writes it
// to X [P][nrhs], block t >= 1 subtracts L[block kb rows, c]^T x_kb from the 64 entries of Y starting at column
// c = 64 (t - 1) (only columns before block kb; Y's entries of block kb are only read).  Bound by latency: every element
// of the two matrices is used once, so all of a thread's are loaded first, straight into registers.
template <int nrhs>
__global__ void __launch_bounds__(512) k_bwd_step(const double* __restrict__ A, int64_t P, int kb,
                                                  const double* __restrict__ inv, double* __restrict__ Y,
                                                  double* __restrict__ X)
{
    __shared__ double y[KB][nrhs], x[KB][nrhs], part[8][KB][nrhs];
    const int64_t o = (int64_t)kb * KB;
    const int nb = (int)(P - o < KB ? P - o : KB);
    const int tid = threadIdx.x;
    const int c = tid & (KB - 1), kq = tid >> 7;           // column of the inverse, rows kq, kq + 4, ...
    const int lc = tid & 63, lq = tid >> 6;                // column of L, rows lq, lq + 8, ...
    const int64_t col = (int64_t)(blockIdx.x - 1) * 64 + lc;
    const bool in = blockIdx.x > 0 && col < o;
    double gi[KB / 4], gl[KB / 8];
#pragma unroll
    for (int i = 0; i < KB / 4; ++i) gi[i] = inv[(kq + 4 * i) * KB + c];
#pragma unroll
    for (int i = 0; i < KB / 8; ++i) {
        const int r = lq + 8 * i;
        gl[i] = A[(o + (r < nb ? r : 0)) * P + (in ? col : 0)];
    }
    for (int e = tid; e < KB * nrhs; e += 512) {
        const int r = e & (KB - 1), n = e >> 7;
        y[r][n] = r < nb ? Y[n * P + o + r] : 0.0;
    }
    __syncthreads();
    double acc[nrhs] = {};
#pragma unroll
    for (int i = 0; i < KB / 4; ++i)
        for (int n = 0; n < nrhs; ++n) acc[n] += gi[i] * y[kq + 4 * i][n];
    for (int n = 0; n < nrhs; ++n) part[kq][c][n] = acc[n];
    __syncthreads();
    for (int e = tid; e < KB * nrhs; e += 512) {
        const int r = e & (KB - 1), n = e >> 7;
        const double v = (part[0][r][n] + part[1][r][n]) + (part[2][r][n] + part[3][r][n]);
        x[r][n] = r < nb ? v : 0.0;
        if (blockIdx.x == 0 && r < nb) X[(o + r) * nrhs + n] = v;
    }
    if (blockIdx.x == 0) return;
    __syncthreads();
    for (int n = 0; n < nrhs; ++n) acc[n] = 0.0;
#pragma unroll
    for (int i = 0; i < KB / 8; ++i)
        for (int n = 0; n < nrhs; ++n) acc[n] += gl[i] * x[lq + 8 * i][n];
    for (int n = 0; n < nrhs; ++n) part[lq][lc][n] = acc[n];
    __syncthreads();
    if (tid < 64 && in)
        for (int n = 0; n < nrhs; ++n) {
            double v = 0.0;
            for (int q = 0; q < 8; ++q) v += part[q][lc][n];
            Y[n * P + col] -= v;
        }
}

}  // namespace

// Doubles of chol_factor's buffer: the matrix's rows in whole steps, the right-hand sides' rows, zeros.
int64_t chol_size(int64_t P) { return ((P + KB - 1) / KB * KB + kMaxRhs) * P + KB; }

// Damp, factor and check: returns BEM_ENOTPD when a pivot fails (host sync).  Blocked right-looking with
// 128-column steps of two launches: the panel as A21 L^{-T} (in place), then the next diagonal block (updated, factored,
// inverted) beside the rest of the trailing lower triangle's rank-128 update.  The right-hand sides B [P][nrhs], nrhs <= 4,
// are further rows of the matrix, so that the forward solve comes with its panels (a launch a block of 64 before:
// 0.4 ms at P = 5,000).  Inverted diagonal blocks and solved rows stay for chol_solve.  P is even (handles have 10 or 20
// parameters).  64-column steps, the diagonal chain and the update on two streams, took 5.8 ms at P = 5,000: a 65 us
// chain a step, and 5 GB of reading and writing the trailing matrix.  Now 2.8 ms: steps 2.2, panels 0.4,
// backward steps 0.2.
int chol_factor(bem_ctx* ctx, const double* H, int64_t P, double lam, const double* B, int nrhs, double* A, int* dflag,
                double* dscal, hipStream_t s)
{
    int rc;
    if (nrhs < 1 || nrhs > kMaxRhs) return set_error(ctx, BEM_EINVAL, "chol_factor: 1..4 right-hand sides");
    const int nblk = (int)((P + KB - 1) / KB);
    const Rows R{P, (int64_t)nblk * KB, nrhs};
    // cholw: inverted diagonal blocks [nblk][128][128]
    if ((rc = ensure(ctx, ctx->cholw, (size_t)nblk * KB * KB * sizeof(double), s))) return rc;
    double* inv = (double*)ctx->cholw.ptr;
    hipLaunchKernelGGL(k_diag_max, dim3(1), dim3(256), 0, s, H, P, dscal);
    hipLaunchKernelGGL(k_damp, dim3(blocks_for(P, 256), P), dim3(256), 0, s, H, P, lam, dscal, A);
    hipLaunchKernelGGL(k_rhs_rows, dim3(blocks_for(P, 256), nrhs + 1), dim3(256), 0, s, B, P, nrhs, A + R.Pr * P);
    if ((rc = fill_i32(ctx, dflag, 1, 0, s))) return rc;
    ProfScope ps_(ctx, PT_CHOLESKY, s);
    for (int kb = 0; kb <= nblk; ++kb) {
        double* Li = inv + (size_t)kb * KB * KB;
        const int64_t rows = R.Pr + nrhs - (int64_t)kb * KB;          // rows left, the gap before the last ones counted
        if (kb > 0)
            hipLaunchKernelGGL(k_panel, dim3(blocks_for(rows, kPanelRows)), dim3(256), 0, s, A, R, kb - 1,
                               (const double*)(Li - KB * KB));
        if (kb == nblk) break;
        const int nt = blocks_for(rows, NB), ntile = kb > 0 ? nt * (nt + 1) / 2 - 3 : 0;
        hipLaunchKernelGGL(k_chol_step, dim3(ntile > 0 ? kStepBlocks : 1), dim3(512), 0, s, A, R, kb, ntile, dflag, Li);
    }
    if ((rc = check_launch(ctx, "cholesky"))) return rc;
    ctx->chol_P = P;
    int hflag = 0;
    if (hipMemcpyAsync(&hflag, dflag, sizeof(int), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return set_error(ctx, BEM_EHIP, "cholesky flag readback");
    return hflag ? BEM_ENOTPD : BEM_OK;
}

template <int nrhs>
static void solve_steps(double* A, int64_t P, int nblk, const double* inv, double* X, hipStream_t s)
{
    for (int kb = nblk - 1; kb >= 0; --kb)
        hipLaunchKernelGGL(k_bwd_step<nrhs>, dim3(1 + 2 * kb), dim3(512), 0, s, A, P, kb, inv + (size_t)kb * KB * KB,
                           A + (size_t)nblk * KB * P, X);
}

// X [P][nrhs] = (L L^T)^{-1} B of the last chol_factor (in A): the backward solve of its solved rows, one launch per
// block, which overwrites them.
int chol_solve(bem_ctx* ctx, double* A, int64_t P, double* X, int nrhs, hipStream_t s)
{
    if (ctx->chol_P != P) return set_error(ctx, BEM_ESTATE, "chol_solve without a matching chol_factor");
    ProfScope ps_(ctx, PT_CHOLESKY, s);
    const int nblk = (int)((P + KB - 1) / KB);
    const double* inv = (const double*)ctx->cholw.ptr;
    switch (nrhs) {
    case 1: solve_steps<1>(A, P, nblk, inv, X, s); break;
    case 2: solve_steps<2>(A, P, nblk, inv, X, s); break;
    case 3: solve_steps<3>(A, P, nblk, inv, X, s); break;
    default: solve_steps<4>(A, P, nblk, inv, X, s); break;
    }
    return check_launch(ctx, "cholesky solve");
}

}  // namespace bem
