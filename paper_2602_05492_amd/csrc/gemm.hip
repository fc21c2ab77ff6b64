// gemm.hip - float64 dense products used around the normal equations, row-major:
// k_gemm_f64_nt: C = alpha A B^T + beta C on float64 MFMA (v_mfma_f64_16x16x4f64), k contiguous in both operands
//   and padded with zeros to kMK, one product or a batch; also the float64 Gram restricted to a list of
//   output tiles.
// k_gemm_f64: the plain VALU product (64 x 64 tiles, 4 x 4 outputs per thread), kept for the
//   float64 VALU Gram mode.
#include "common.hpp"
#include "sweep_common.hpp"

namespace bem {

namespace {

constexpr int TM = 64, TN = 64, TK = 16;

__global__ void __launch_bounds__(256) k_gemm_f64(int m, int n, int k, double alpha, const double* __restrict__ A,
                                                  int64_t lda, const double* __restrict__ B, int64_t ldb, double beta,
                                                  double* __restrict__ C, int64_t ldc, const int* __restrict__ tiles)
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
        for (int e = threadIdx.x; e < TM * TK; e += 256) {
            const int kk = e % TK, r = e / TK, gk = k0 + kk;
            As[kk][r] = row0 + r < m && gk < k ? A[(size_t)(row0 + r) * lda + gk] : 0.0;
            Bs[kk][r] = col0 + r < n && gk < k ? B[(size_t)(col0 + r) * ldb + gk] : 0.0;
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
// Block tile BM x BM, 4 wavefronts as 2 x 2, each BM/2 x BM/2 in 16 x 16 tiles of v_mfma_f64_16x16x4f64.  Operand
// lane layout of that instruction: lane l holds A[l mod 16][l / 16] of its 16 x 4 slice and B[l / 16][l mod 16] of
// its 4 x 16 slice; accumulator element q of lane l is row 4 q + l / 16, column l mod 16 of the 16 x 16 tile.
//
// Bound by the matrix cores (64 cycles an instruction): all else is to stay out of their way.  Both operands
// are [row][k], so that a 16-deep k slab of a row is a 128-byte line, and go straight from global memory into
// LDS (16 bytes a lane, no registers, no address arithmetic per element, no masks); the next slab is in flight
// behind the products of the current one.  Rows past the operands' last repeat it (their products are not
// stored); k is padded with zeros by whoever writes the operands.  LDS rows are 8 chunks of two k, chunk c of row
// r at position c ^ ((r / 2) mod 8), so that the 16 lanes of a 16-byte read at one chunk fall in distinct
// banks; a lane's load fetches the chunk whose position is its own.  A lane's two consecutive k go to two
// instructions: which k an instruction sums is free as long as A and B agree.
//
// Gram of 1,920 rows over 32,768 samples: 2.82 ms (41 TFLOP/s, operands through registers with masks) -> 1.79 ms (65 TFLOP/s).
typedef double d2_t __attribute__((ext_vector_type(2)));
typedef double d4_t __attribute__((ext_vector_type(4)));
constexpr int kMB = 128, kMK = kGemmPad;

// Blocks go to the 8 XCDs round-robin, each XCD with an L2 of its own, so XCD x is given a contiguous run
// of the tiles: of the work list (row tile, column tile, part: k range [part kchunk, (part + 1) kchunk),
// result at C + part cstride), or of the grid of tiles (part-major, bands of 8 tile columns).
template <int BM>
__global__ void __launch_bounds__(256, BM == 128 ? 2 : 4) k_gemm_f64_nt(Gemm64 g, const int* __restrict__ work, int nwork,
                                                                      int kchunk, int64_t cstride)
{
    constexpr int TI = BM / 32;                 // 16 x 16 MFMA tiles per wavefront and dimension
    constexpr int NL = BM / 32;                 // load instructions (8 rows) per wavefront, slab and operand
    __shared__ __attribute__((aligned(1024))) double Sm[2][2][BM][kMK];
    const int wi = (int)(blockIdx.x & 7) * ((nwork + 7) >> 3) + (int)(blockIdx.x >> 3);
    if (wi >= nwork) return;
    int bm, bn, part;
    if (work) {
        bm = work[3 * wi];
        bn = work[3 * wi + 1];
        part = work[3 * wi + 2];
    } else {
        const int nbm = (g.m + BM - 1) / BM, per = 8 * nbm * ((g.n + 8 * BM - 1) / (8 * BM));
        part = wi / per;
        const int t = wi % per, r = t % (8 * nbm);
        bm = r >> 3;
        bn = t / (8 * nbm) * 8 + (r & 7);
        if (bn * BM >= g.n) return;
    }
    const int k0 = part * kchunk, k1 = k0 + kchunk < g.k ? k0 + kchunk : g.k;
    const int ns = k1 > k0 ? (k1 - k0) / kMK : 0;
    const int row0 = bm * BM, col0 = bn * BM;
    const double* A = g.A + blockIdx.y * g.sa + k0;
    const double* B = g.B + blockIdx.y * g.sb + k0;
    double* C = g.C + blockIdx.y * g.sc + part * cstride;
    const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wr = w >> 1, wc = w & 1;
    // wavefront w loads rows BM/4 w .. BM/4 (w + 1) - 1 of both slabs
    const double *ga[NL], *gb[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        const int r = BM / 4 * w + 8 * i + (l >> 3), c = 2 * ((l & 7) ^ ((r >> 1) & 7));
        ga[i] = A + (int64_t)(row0 + r < g.m ? row0 + r : g.m - 1) * g.lda + c;
        gb[i] = B + (int64_t)(col0 + r < g.n ? col0 + r : g.n - 1) * g.ldb + c;
    }
    auto load = [&](int buf, int s) {
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            __builtin_amdgcn_global_load_lds((const void*)(ga[i] + s * kMK), (void*)&Sm[buf][0][BM / 4 * w + 8 * i][0], 16, 0, 0);
            __builtin_amdgcn_global_load_lds((const void*)(gb[i] + s * kMK), (void*)&Sm[buf][1][BM / 4 * w + 8 * i][0], 16, 0, 0);
        }
    };
    d4_t acc[TI][TI];
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TI; ++j) acc[i][j] = d4_t{0.0, 0.0, 0.0, 0.0};
    if (ns > 0) load(0, 0);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    const int rr = l & 15, lk = l >> 4;
    for (int s = 0; s < ns; ++s) {
        const int cur = s & 1;
        if (s + 1 < ns) load(cur ^ 1, s + 1);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            d2_t a[TI], b[TI];
#pragma unroll
            for (int i = 0; i < TI; ++i) {
                const int r = BM / 2 * wr + 16 * i + rr;
                a[i] = *(const d2_t*)&Sm[cur][0][r][2 * ((4 * h + lk) ^ ((r >> 1) & 7))];
            }
#pragma unroll
            for (int j = 0; j < TI; ++j) {
                const int r = BM / 2 * wc + 16 * j + rr;
                b[j] = *(const d2_t*)&Sm[cur][1][r][2 * ((4 * h + lk) ^ ((r >> 1) & 7))];
            }
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int i = 0; i < TI; ++i)
#pragma unroll
                    for (int j = 0; j < TI; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i][t], b[j][t], acc[i][j], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0);          // this wavefront's share of the next slab is in LDS
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TI; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int r = row0 + BM / 2 * wr + 16 * i + 4 * q + lk;
                const int c = col0 + BM / 2 * wc + 16 * j + rr;
                if (r < g.m && c < g.n) {
                    double* o = C + (int64_t)r * g.ldc + c;
                    *o = g.alpha * acc[i][j][q] + (g.beta == 0.0 ? 0.0 : g.beta * *o);
                }
            }
}

// C = alpha sum of the parts (P + part cstride, batch entries m n apart) + beta C, in the parts' order
__global__ void __launch_bounds__(256) k_gemm_sum(const double* __restrict__ P, int parts, int64_t cstride, Gemm64 g)
{
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= (int64_t)g.m * g.n) return;
    const double* p = P + blockIdx.y * (int64_t)g.m * g.n + e;
    double v = 0.0;
    for (int i = 0; i < parts; ++i) v += p[i * cstride];
    double* o = g.C + blockIdx.y * g.sc + (e / g.n) * g.ldc + e % g.n;
    *o = g.alpha * v + (g.beta == 0.0 ? 0.0 : g.beta * *o);
}

// what k_gemm_f64_nt assumes of its operands
bool loads_aligned(const Gemm64& g)
{
    return g.k % kMK == 0 && !((g.lda | g.ldb | g.sa | g.sb) & 1) && !(((uintptr_t)g.A | (uintptr_t)g.B) & 15);
}

}  // namespace

int gemm_f64_list(bem_ctx* ctx, const Gemm64& g, hipStream_t s, const int* work, int nwork, int kchunk, int64_t cstride)
{
    if (nwork <= 0) return BEM_OK;
    if (!loads_aligned(g) || kchunk % kMK) return set_error(ctx, BEM_EINVAL, "float64 Gram operands (internal)");
    hipLaunchKernelGGL(k_gemm_f64_nt<kMB>, dim3(8 * ((nwork + 7) / 8)), dim3(256), 0, s, g, work, nwork, kchunk, cstride);
    return check_launch(ctx, "gemm_f64");
}

int gemm_f64_valu(bem_ctx* ctx, const Gemm64& g, hipStream_t s, const int* tiles, int ntiles)
{
    if (ntiles <= 0) return BEM_OK;
    hipLaunchKernelGGL(k_gemm_f64, dim3(ntiles), dim3(256), 0, s, g.m, g.n, g.k, g.alpha, g.A, g.lda, g.B, g.ldb, g.beta, g.C,
                       g.ldc, tiles);
    return check_launch(ctx, "gemm_f64");
}

int gemm_f64(bem_ctx* ctx, const Gemm64& g, int batch, hipStream_t s)
{
    if (g.m <= 0 || g.n <= 0 || batch <= 0) return BEM_OK;
    if (!loads_aligned(g)) return set_error(ctx, BEM_EINVAL, "float64 product operands (internal)");
    const auto count = [&](int bm) { return 8 * blocks_for(g.n, 8 * bm) * blocks_for(g.m, bm); };
    const auto tiles = [&](int bm) { return (int64_t)blocks_for(g.n, bm) * blocks_for(g.m, bm) * batch; };
    if (tiles(kMB) >= 2048) {
        const int nw = count(kMB);
        hipLaunchKernelGGL(k_gemm_f64_nt<kMB>, dim3(8 * ((nw + 7) / 8), batch), dim3(256), 0, s, g, (const int*)nullptr, nw, g.k,
                           (int64_t)0);
        return check_launch(ctx, "gemm_f64");
    }
    // fewer than four rounds of 128-tiles over the CUs: 64-tiles (500 straight handles, 89 GFLOP in three
    // products: 2.5 -> 1.6 ms); fewer than two a CU of those: k in parts of at least 128, summed afterwards (4 cubic
    // handles, the three products 580 -> 47 us)
    int parts = (int)(512 / tiles(64));
    if (parts > g.k / 128) parts = g.k / 128;
    if (parts < 2) parts = 1;
    const int kchunk = parts > 1 ? blocks_for(blocks_for(g.k, parts), kMK) * kMK : g.k;
    if (parts > 1) parts = blocks_for(g.k, kchunk);
    const int nw = count(64) * parts;
    Gemm64 p = g;
    const int64_t cstride = (int64_t)batch * g.m * g.n;
    if (parts > 1) {
        int rc;
        if ((rc = ensure(ctx, ctx->gemmw, (size_t)parts * cstride * sizeof(double), s))) return rc;
        p.C = (double*)ctx->gemmw.ptr;
        p.ldc = g.n;
        p.sc = (int64_t)g.m * g.n;
        p.alpha = 1.0;
        p.beta = 0.0;
    }
    hipLaunchKernelGGL(k_gemm_f64_nt<64>, dim3(8 * ((nw + 7) / 8), batch), dim3(256), 0, s, p, (const int*)nullptr, nw, kchunk,
                       cstride);
    if (parts > 1)
        hipLaunchKernelGGL(k_gemm_sum, dim3(blocks_for((int64_t)g.m * g.n, 256), batch), dim3(256), 0, s, (const double*)p.C,
                           parts, cstride, g);
    return check_launch(ctx, "gemm_f64");
}

}  // namespace bem
