// gemm.hip - float64 dense products used around the normal equations:
//   C = alpha op(A) op(B) + beta C   (row-major, op = identity or transpose)
// k_gemm_f64_mfma: 128 x 128 (or 64 x 64) output tiles on float64 MFMA (v_mfma_f64_16x16x4f64), 16-deep
//   k slabs staged through LDS (double buffered, the next slab prefetched into registers while
//   the current one is multiplied); also the float64 Gram restricted to a list of output tiles.
// k_gemm_f64: the plain VALU product (64 x 64 tiles, 4 x 4 outputs per thread), kept for the
//   float64 VALU Gram mode.
#include "common.hpp"
#include "sweep_common.hpp"

namespace bem {

namespace {

constexpr int TM = 64, TN = 64, TK = 16;

__global__ void __launch_bounds__(256) k_gemm_f64(int m, int n, int k, double alpha, const double* __restrict__ A,
                                                  int64_t lda, int ta, const double* __restrict__ B, int64_t ldb, int tb,
                                                  double beta, double* __restrict__ C, int64_t ldc,
                                                  const int* __restrict__ tiles)
{
    __shared__ double As[TK][TM + 1];
    __shared__ double Bs[TK][TN + 1];
    const int bm = tiles[2 * blockIdx.x], bn = tiles[2 * blockIdx.x + 1];
    const int row0 = bm * TM, col0 = bn * TN;
    const int tx = threadIdx.x % 16, ty = threadIdx.x / 16;
    double acc[4][4];
    for (int i = 0; i < 4; ++i)
        for (int j = 0; j < 4; ++j) acc[i][j] = 0.0;
    for (int k0 = 0; k0 < k; k0 += TK) {
        // load a TM x TK slab of op(A) and a TK x TN slab of op(B)
        for (int e = threadIdx.x; e < TM * TK; e += 256) {
            int r, kk;
            if (ta) { r = e % TM; kk = e / TM; }
            else { kk = e % TK; r = e / TK; }
            const int gr = row0 + r, gk = k0 + kk;
            double v = 0.0;
            if (gr < m && gk < k) v = ta ? A[(size_t)gk * lda + gr] : A[(size_t)gr * lda + gk];
            As[kk][r] = v;
        }
        for (int e = threadIdx.x; e < TK * TN; e += 256) {
            int c, kk;
            if (tb) { kk = e % TK; c = e / TK; }
            else { c = e % TN; kk = e / TN; }
            const int gc = col0 + c, gk = k0 + kk;
            double v = 0.0;
            if (gc < n && gk < k) v = tb ? B[(size_t)gc * ldb + gk] : B[(size_t)gk * ldb + gc];
            Bs[kk][c] = v;
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < TK; ++kk) {
            double a[4], b[4];
            for (int i = 0; i < 4; ++i) a[i] = As[kk][ty + 16 * i];
            for (int j = 0; j < 4; ++j) b[j] = Bs[kk][tx + 16 * j];
            for (int i = 0; i < 4; ++i)
                for (int j = 0; j < 4; ++j) acc[i][j] += a[i] * b[j];
        }
        __syncthreads();
    }
    for (int i = 0; i < 4; ++i) {
        const int r = row0 + ty + 16 * i;
        if (r >= m) continue;
        for (int j = 0; j < 4; ++j) {
            const int c = col0 + tx + 16 * j;
            if (c >= n) continue;
            double* o = C + (size_t)r * ldc + c;
            *o = alpha * acc[i][j] + (beta == 0.0 ? 0.0 : beta * *o);
        }
    }
}


// ---- float64 MFMA product ------------------------------------------------------------------
// Block tile kMB x kMB, 4 wavefronts as 2 x 2, each wavefront 64 x 64 as 4 x 4 tiles of
// v_mfma_f64_16x16x4f64.  Operand lane layout of that instruction: lane l holds A[l mod 16][l / 16]
// of its 16 x 4 slice and B[l / 16][l mod 16] of its 4 x 16 slice; accumulator element q of lane l
// is row 4 q + l / 16, column l mod 16 of the 16 x 16 tile.  Both operand slabs are stored in LDS
// k-major ([k][row] and [k][col]) so that each operand is one ds_read_b64 per lane.
typedef double d4_t __attribute__((ext_vector_type(4)));
constexpr int kMB = 128, kMK = 16;

// element e of a BM x kMK slab of op(X) starting at (r0, k0): its slab coordinates, and whether it lies
// in the rows x kd operand.  Non-transposed X is row-major [row][k] (16 consecutive threads read one
// row's 16 k values); transposed X is stored [k][row].
template <int BM>
__device__ inline bool slab_at(int tx, int r0, int k0, int rows, int kd, int e, int& sr, int& sk)
{
    if (tx) { sk = e / BM; sr = e % BM; }
    else { sr = e / kMK; sk = e % kMK; }
    return r0 + sr < rows && k0 + sk < kd;
}
// The element there, or element (0, 0) of X outside the operand (replaced by 0 where the slab is stored:
// a select beside the load would wait for it, and the loads are to stay in flight behind the products).
template <int BM>
__device__ inline double slab_load(const double* __restrict__ X, int64_t ldx, int tx, int r0, int k0, int rows, int kd,
                                   int e)
{
    int sr, sk;
    const bool in = slab_at<BM>(tx, r0, k0, rows, kd, e, sr, sk);
    const int gr = in ? r0 + sr : 0, gk = in ? k0 + sk : 0;
    return X[tx ? (int64_t)gk * ldx + gr : (int64_t)gr * ldx + gk];
}

// BM x BM output tile per block (BM = 128: each wavefront 64 x 64 as 4 x 4 MFMA tiles; BM = 64:
// 32 x 32 as 2 x 2, for products whose 128-tile grid would leave most CUs idle).
//
// Blocks go to the 8 XCDs round-robin, each XCD with an L2 of its own, so XCD x is given a contiguous run
// of the tiles: of the work list (row tile, column tile, part: k range [part kchunk, (part + 1) kchunk),
// result at C + part cstride), or of the whole grid in bands of 8 tile columns.
template <int BM>
__global__ void __launch_bounds__(256, BM == 128 ? 2 : 4) k_gemm_f64_mfma(int m, int n, int k_all, double alpha,
                                                                        const double* __restrict__ A, int64_t lda, int ta,
                                                                        const double* __restrict__ B, int64_t ldb, int tb,
                                                                        double beta, double* __restrict__ C, int64_t ldc,
                                                                        const int* __restrict__ work, int nwork,
                                                                        int kchunk, int64_t cstride)
{
    constexpr int LD = BM + 4;                  // LDS row stride (doubles)
    constexpr int NL = BM * kMK / 256;          // slab elements per thread and operand
    constexpr int TI = BM / 32;                 // 16 x 16 MFMA tiles per wavefront and dimension
    __shared__ double As[2][kMK][LD];
    __shared__ double Bs[2][kMK][LD];
    const int wi = (int)(blockIdx.x & 7) * ((nwork + 7) >> 3) + (int)(blockIdx.x >> 3);
    if (wi >= nwork) return;
    int bm, bn, k0 = 0;
    if (work) {
        bm = work[3 * wi];
        bn = work[3 * wi + 1];
        k0 = work[3 * wi + 2] * kchunk;
        C += (int64_t)work[3 * wi + 2] * cstride;
    } else {
        const int nbm = (m + BM - 1) / BM, band = wi / (8 * nbm), r = wi % (8 * nbm);
        bm = r >> 3;
        bn = band * 8 + (r & 7);
        if (bn * BM >= n) return;
    }
    const int k = k0 + kchunk < k_all ? k0 + kchunk : k_all;      // this block's k range [k0, k)
    const int row0 = bm * BM, col0 = bn * BM;
    const int tid = threadIdx.x, l = tid & 63, w = tid >> 6;
    const int wr = w >> 1, wc = w & 1;
    // B as a (k x n) operand: op(B) row-major [k][col] unless transposed ([col][k]); slab_load takes
    // the "row" index as the column of op(B), so its transposition flag is the opposite one
    const int tbB = tb ? 0 : 1;
    double pa[NL], pb[NL];
    auto load = [&](int ks) {
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            pa[i] = slab_load<BM>(A, lda, ta, row0, ks, m, k, tid + 256 * i);
            pb[i] = slab_load<BM>(B, ldb, tbB, col0, ks, n, k, tid + 256 * i);
        }
    };
    auto store = [&](int buf, int ks) {
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            int r, kk;
            const bool ia = slab_at<BM>(ta, row0, ks, m, k, tid + 256 * i, r, kk);
            As[buf][kk][r] = ia ? pa[i] : 0.0;
            const bool ib = slab_at<BM>(tbB, col0, ks, n, k, tid + 256 * i, r, kk);
            Bs[buf][kk][r] = ib ? pb[i] : 0.0;
        }
    };
    load(k0);
    store(0, k0);
    __syncthreads();
    d4_t acc[TI][TI];
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TI; ++j) acc[i][j] = d4_t{0.0, 0.0, 0.0, 0.0};
    const int nk = k > k0 ? (k - k0 + kMK - 1) / kMK : 0;
    for (int s = 0; s < nk; ++s) {
        const int cur = s & 1;
        const bool more = s + 1 < nk;
        if (more) load(k0 + (s + 1) * kMK);
        __builtin_amdgcn_sched_barrier(0);        // the loads go out before the products, and are waited for after
#pragma unroll
        for (int ks = 0; ks < kMK; ks += 4) {
            const int kk = ks + (l >> 4), rr = l & 15;
            double a[TI], b[TI];
#pragma unroll
            for (int i = 0; i < TI; ++i) a[i] = As[cur][kk][(BM / 2) * wr + 16 * i + rr];
#pragma unroll
            for (int j = 0; j < TI; ++j) b[j] = Bs[cur][kk][(BM / 2) * wc + 16 * j + rr];
#pragma unroll
            for (int i = 0; i < TI; ++i)
#pragma unroll
                for (int j = 0; j < TI; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (more) store(cur ^ 1, k0 + (s + 1) * kMK);
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TI; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int r = row0 + (BM / 2) * wr + 16 * i + 4 * q + (l >> 4);
                const int c = col0 + (BM / 2) * wc + 16 * j + (l & 15);
                if (r < m && c < n) {
                    double* o = C + (size_t)r * ldc + c;
                    *o = alpha * acc[i][j][q] + (beta == 0.0 ? 0.0 : beta * *o);
                }
            }
}

}  // namespace

// C + part cstride = alpha op(A) op(B) + beta C over the k range of each part, on the 128 x 128 output
// tiles of a work list (row tile, column tile, part).
int gemm_f64_list(bem_ctx* ctx, int m, int n, int k, double alpha, const double* A, int64_t lda, bool ta, const double* B,
                  int64_t ldb, bool tb, double beta, double* C, int64_t ldc, hipStream_t s, const int* work, int nwork,
                  int kchunk, int64_t cstride)
{
    if (nwork <= 0) return BEM_OK;
    hipLaunchKernelGGL(k_gemm_f64_mfma<kMB>, dim3(8 * ((nwork + 7) / 8)), dim3(256), 0, s, m, n, k, alpha, A, lda,
                       ta ? 1 : 0, B, ldb, tb ? 1 : 0, beta, C, ldc, work, nwork, kchunk, cstride);
    return check_launch(ctx, "gemm_f64");
}

int gemm_f64(bem_ctx* ctx, int m, int n, int k, double alpha, const double* A, int64_t lda, bool ta, const double* B,
             int64_t ldb, bool tb, double beta, double* C, int64_t ldc, hipStream_t s, const int* tiles, int ntiles)
{
    if (m <= 0 || n <= 0) return BEM_OK;
    if (tiles) {                      // a list of 64 x 64 output tiles, on the vector ALUs
        if (ntiles <= 0) return BEM_OK;
        hipLaunchKernelGGL(k_gemm_f64, dim3(ntiles), dim3(256), 0, s, m, n, k, alpha, A, lda, ta ? 1 : 0, B, ldb,
                           tb ? 1 : 0, beta, C, ldc, tiles);
        return check_launch(ctx, "gemm_f64");
    }
    const auto count = [&](int bm) { return 8 * blocks_for(blocks_for(n, bm), 8) * blocks_for(m, bm); };
    if ((int64_t)blocks_for(n, kMB) * blocks_for(m, kMB) >= 1024) {
        const int nw = count(kMB);
        hipLaunchKernelGGL(k_gemm_f64_mfma<kMB>, dim3(8 * ((nw + 7) / 8)), dim3(256), 0, s, m, n, k, alpha, A, lda,
                           ta ? 1 : 0, B, ldb, tb ? 1 : 0, beta, C, ldc, (const int*)nullptr, nw, k, (int64_t)0);
    } else {
        // fewer than two rounds of 128-tiles over the CUs: 64-tiles, 4x the blocks
        const int nw = count(64);
        hipLaunchKernelGGL(k_gemm_f64_mfma<64>, dim3(8 * ((nw + 7) / 8)), dim3(256), 0, s, m, n, k, alpha, A, lda,
                           ta ? 1 : 0, B, ldb, tb ? 1 : 0, beta, C, ldc, (const int*)nullptr, nw, k, (int64_t)0);
    }
    return check_launch(ctx, "gemm_f64");
}

}  // namespace bem
