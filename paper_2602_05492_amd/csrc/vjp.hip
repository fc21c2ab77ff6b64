// vjp.hip - reverse mode of the forward path (Eq. diffbie, Sec. 3.2), as a
// vector-Jacobian product with cotangents gbar(x) of u(x):
//
//   segments  per handle segment, sums over samples of the pair adjoint:
//             d/da, d/db of sum_c gbar_c f_c   and  sum gbar_c M_m  (16 sums)
//   psi       psi_j = sum_x gbar(x) beta_j(x) for every outer element
//   mu        mu = A+^T psi  (the transposed boundary solve)
//   boundary  the same segment adjoint at the 3M boundary Gauss points with
//             cotangent mu_i w_q |G_i|/2 (F_i = sum_q w_q |G_i|/2 f(x_iq))
//   chain     segment end points -> Bezier control points (Bernstein weights),
//             end densities -> handle-end jumps (1 - t, t)
//
// Sweep mapping: the 64 lanes of a wavefront own 64 consecutive segments (or
// outer elements) and keep their sums in registers; the wavefront walks a
// chunk of samples whose positions and cotangents are wave-uniform (scalar
// loads).  Four wavefronts of a block split the chunk and are summed through
// LDS; chunks are summed by a separate fixed-order pass, so results do not
// depend on scheduling.
#include <mutex>

#include "adjoint.hpp"

namespace bem {

namespace {

__device__ inline void load_cot(const double* __restrict__ gbar, int64_t s, double& g0, double& g1, double& g2)
{
    g0 = gbar[3 * s]; g1 = gbar[3 * s + 1]; g2 = gbar[3 * s + 2];
}

__global__ void __launch_bounds__(256) k_vjp_segments(const double* __restrict__ x, const double* __restrict__ gbar,
                                                      int64_t N, int64_t chunk, const double* __restrict__ seg64,
                                                      int K, double eps2, double* __restrict__ partial)
{
    __shared__ double red[3][64][kV + 1];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int k = blockIdx.x * 64 + lane;
    const int64_t n0 = (int64_t)blockIdx.y * chunk;
    const int64_t n1 = n0 + chunk < N ? n0 + chunk : N;
    double acc[kV];
    for (int v = 0; v < kV; ++v) acc[v] = 0.0;
    if (k < K) {
        const double* s64 = seg64 + (size_t)k * kSegStride;
        const SegGeom<double> g = load_geom(s64);
        if (g.L2 > 0.0) {
            double w[12];
            for (int c = 0; c < 12; ++c) w[c] = s64[kWdA + c];
            for (int64_t s = n0 + wave; s < n1; s += 4) {
                const double X = x[2 * s], Y = x[2 * s + 1];
                double g0, g1, g2;
                load_cot(gbar, s, g0, g1, g2);
                const double wa = g0 * w[0] + g1 * w[1] + g2 * w[2];
                const double wb = g0 * w[3] + g1 * w[4] + g2 * w[5];
                const double sa = g0 * w[6] + g1 * w[7] + g2 * w[8];
                const double sb = g0 * w[9] + g1 * w[10] + g2 * w[11];
                const PairState<double> st = pair_forward<double, DevF64, true>(g, X, Y, eps2);
                add_pair(acc, pair_backward(g, st, eps2, wa, wb, sa, sb), pair_moments(g, st), g0, g1, g2);
            }
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

// psi_j = sum_x gbar(x) beta_j(x): lanes own outer elements.
__global__ void __launch_bounds__(256) k_vjp_elements(const double* __restrict__ x, const double* __restrict__ gbar,
                                                      int64_t N, int64_t chunk, const double* __restrict__ el64,
                                                      int M,
                                                      double* __restrict__ partial)
{
    __shared__ double red[3][64][3];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int j = blockIdx.x * 64 + lane;
    const int64_t n0 = (int64_t)blockIdx.y * chunk;
    const int64_t n1 = n0 + chunk < N ? n0 + chunk : N;
    double a0 = 0.0, a1 = 0.0, a2 = 0.0;
    if (j < M) {
        const double* e = el64 + (size_t)j * kElemStride;
        const double ax = e[0], ay = e[1], vx = e[2], vy = e[3];
        for (int64_t s = n0 + wave; s < n1; s += 4) {
            double g0, g1, g2;
            load_cot(gbar, s, g0, g1, g2);
            const double b = element_beta<double, DevF64>(ax, ay, vx, vy, x[2 * s], x[2 * s + 1]);
            a0 += b * g0; a1 += b * g1; a2 += b * g2;
        }
    }
    if (wave > 0) { red[wave - 1][lane][0] = a0; red[wave - 1][lane][1] = a1; red[wave - 1][lane][2] = a2; }
    __syncthreads();
    if (wave == 0 && j < M) {
        double* o = partial + ((size_t)blockIdx.y * M + j) * 3;
        o[0] = ((a0 + red[0][lane][0]) + red[1][lane][0]) + red[2][lane][0];
        o[1] = ((a1 + red[0][lane][1]) + red[1][lane][1]) + red[2][lane][1];
        o[2] = ((a2 + red[0][lane][2]) + red[1][lane][2]) + red[2][lane][2];
    }
}

// out[i] = sum_p partial[p * len + i], fixed order: 64 values a block, its 16 wavefronts taking every
// sixteenth row each, then added through LDS (one thread a value over all rows was a chain of up to 512
// dependent loads).
__global__ void __launch_bounds__(1024) k_reduce_parts(const double* __restrict__ partial, int nparts, int64_t len,
                                                       double* __restrict__ out)
{
    __shared__ double red[16][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t i = (int64_t)blockIdx.x * 64 + lane;
    double s = 0.0;
    if (i < len) {
#pragma unroll 4
        for (int p = w; p < nparts; p += 16) s += partial[(size_t)p * len + i];
    }
    red[w][lane] = s;
    __syncthreads();
    if (w == 0 && i < len) {
        for (int k = 1; k < 16; ++k) s += red[k][lane];
        out[i] = s;
    }
}

// Segment sums -> theta gradient: a thread per parameter.  Cubic handles chain the vertex gradients to
// the control points with Bernstein weights and the end jumps with (1 - t, t); straight handles (model 1)
// chain them to the end points with (1 - t, t) and sum the jumps.  (A thread per handle read its S x 16 sums
// one after the other: 28 us for 4 handles of 32 segments.)
__global__ void __launch_bounds__(64) k_chain_theta(const double* __restrict__ sg, int H, int S, int model,
                                                    double* __restrict__ grad)
{
    const bool straight = model == 1;
    const int Q = straight ? 10 : 20, ngeo = straight ? 4 : 8;
    const int t = blockIdx.x * 64 + threadIdx.x;
    if (t >= H * Q) return;
    const int h = t / Q, p = t % Q;
    const double* v = sg + (size_t)h * S * kV;
    double out = 0.0;
    if (p < ngeo) {
        const int q = p >> 1, d = p & 1;
#pragma unroll 8
        for (int j = 0; j < S; ++j) {
            double Ba[4], Bb[4];
            vertex_weights(model, (double)j / (double)S, Ba);
            vertex_weights(model, (double)(j + 1) / (double)S, Bb);
            const double a = q == 0 ? Ba[0] : (q == 1 ? Ba[1] : (q == 2 ? Ba[2] : Ba[3]));
            const double b = q == 0 ? Bb[0] : (q == 1 ? Bb[1] : (q == 2 ? Bb[2] : Bb[3]));
            out += a * v[(size_t)j * kV + d] + b * v[(size_t)j * kV + 2 + d];
        }
    } else if (straight) {
        const int c = (p - 4) % 3, m = 4 + 6 * ((p - 4) / 3) + c;         // wd, wc
        for (int j = 0; j < S; ++j) out += v[(size_t)j * kV + m] + v[(size_t)j * kV + m + 3];
    } else {
        const int c = (p - 8) % 3, k = (p - 8) / 3, m = 4 + 6 * (k >> 1) + c;   // wd0, wd1, wc0, wc1
        const bool end = k & 1;
#pragma unroll 8
        for (int j = 0; j < S; ++j) {
            const double ta = (double)j / (double)S, tb = (double)(j + 1) / (double)S;
            out += (end ? ta : 1.0 - ta) * v[(size_t)j * kV + m] + (end ? tb : 1.0 - tb) * v[(size_t)j * kV + m + 3];
        }
    }
    grad[t] = out;
}

// Chunks of N samples over `groups` groups of 64 segments or elements: about 4,096 blocks, each with at least
// 256 samples, or (fine) 32 while there are fewer than 1,024 blocks.
int chunks_for(int64_t N, int groups, bool fine, int64_t& chunk)
{
    int64_t nch = (4096 + groups - 1) / groups;
    const int64_t few = !fine ? 0 : (N + 31) / 32 < 1024 / groups ? (N + 31) / 32 : 1024 / groups;
    const int64_t cap = (N + 255) / 256 > few ? (N + 255) / 256 : few;
    if (nch > cap) nch = cap;
    if (nch < 1) nch = 1;
    chunk = (N + nch - 1) / nch;
    if (chunk < 1) chunk = 1;
    nch = (N + chunk - 1) / chunk;
    if (nch < 1) nch = 1;
    return (int)nch;
}

}  // namespace

// Bytes of device workspace the float64 adjoint carves for K segments, M elements and N samples
// (tables, partial sums, psi, mu, boundary Gauss points, segment sums), each piece 256-aligned.
static size_t carve_round(size_t b) { return (b + 255) / 256 * 256; }

size_t vjp_f64_workspace_bytes(int K, int M, int64_t N, bool fine)
{
    const int kgroups = (K + 63) / 64, mgroups = (M + 63) / 64;
    int64_t c = 1;
    const int ns = N > 0 ? chunks_for(N, kgroups, fine, c) : 0;
    const int ng = chunks_for(3 * (int64_t)M, kgroups, fine, c);
    const int ne = N > 0 ? chunks_for(N, mgroups, fine, c) : 0;
    const size_t k1 = (size_t)(K > 0 ? K : 1);
    return carve_round(k1 * kSegStride * sizeof(double)) + carve_round(k1 * kSegStride * sizeof(float)) +
           carve_round((size_t)M * kElemStride * sizeof(double)) + carve_round((size_t)M * kElemStride * sizeof(float)) +
           carve_round((size_t)M * 3 * sizeof(double)) + carve_round((size_t)(ns + ng) * k1 * kV * sizeof(double)) +
           carve_round(((size_t)(ne > 0 ? ne : 1) * M * 3 + 2 * (size_t)M * 3) * sizeof(double)) +
           carve_round((size_t)3 * M * 5 * sizeof(double)) + carve_round(k1 * kV * sizeof(double));
}

int run_vjp(bem_ctx* ctx, const double* theta, int H, const double* x, int64_t N, const void* gbar, bool mixed,
            double* grad, hipStream_t s, const Carve* carve)
{
    int rc;
    const int S = ctx->opts.segs_per_handle;
    const int K = H * S;
    const int M = ctx->M;
    const double eps2 = ctx->opts.eps * ctx->opts.eps;
    if (H == 0) return BEM_OK;
    if (carve && mixed) return set_error(ctx, BEM_EINVAL, "the carved adjoint is float64 only (internal)");
    const int kgroups = (K + 63) / 64, mgroups = (M + 63) / 64;
    int64_t chunk_s = 1, chunk_g = 1, chunk_e = 1;
    // partial rows of the segment and element sums: the samples', then the boundary Gauss points'
    const bool fine = !carve || vjp_f64_workspace_bytes(K, M, N, true) <= carve->bytes;
    int ns = N > 0 ? chunks_for(N, kgroups, fine, chunk_s) : 0;
    const int ng = chunks_for(3 * (int64_t)M, kgroups, fine, chunk_g);
    int ne = N > 0 ? chunks_for(N, mgroups, fine, chunk_e) : 0;
    const Grouping grid = mixed && N > 0 ? adj_mixed_rows(ctx, K, N, &ns, &ne) : Grouping{};
    const size_t seg_part = (size_t)(ns + ng) * K * kV;
    const size_t el_rows = (size_t)(ne > 0 ? ne : 1);
    const size_t seg_n = (size_t)(K > 0 ? K : 1) * kSegStride;
    double *seg64w, *el64w, *part, *epart, *gx, *redw;
    float *seg32w, *el32w;
    if (carve) {
        // every workspace from the caller's device memory, in the order vjp_f64_workspace_bytes counts
        const size_t need = vjp_f64_workspace_bytes(K, M, N, fine);
        if (need > carve->bytes)
            return set_error(ctx, BEM_EINVAL, "%zu bytes of workspace for K = %d, M = %d, N = %lld exceed the %zu "
                             "available", need, K, M, (long long)N, carve->bytes);
        char* p = carve->base;
        auto take = [&](size_t b) { char* q = p; p += carve_round(b); return q; };
        seg64w = (double*)take(seg_n * sizeof(double));
        seg32w = (float*)take(seg_n * sizeof(float));
        el64w = (double*)take((size_t)M * kElemStride * sizeof(double));
        el32w = (float*)take((size_t)M * kElemStride * sizeof(float));
        take((size_t)M * 3 * sizeof(double));
        part = (double*)take(seg_part * sizeof(double));
        epart = (double*)take((el_rows * M * 3 + 2 * (size_t)M * 3) * sizeof(double));
        gx = (double*)take((size_t)3 * M * 5 * sizeof(double));
        redw = (double*)take((size_t)K * kV * sizeof(double));
    } else {
        // workspaces: tmp1 segment partials, tmp2 element partials + psi + mu, tmp3 Gauss points, red segment sums
        if ((rc = ensure(ctx, ctx->seg64, seg_n * sizeof(double), s))) return rc;
        if ((rc = ensure(ctx, ctx->seg32, seg_n * sizeof(float), s))) return rc;
        if ((rc = ensure(ctx, ctx->tmp1, seg_part * sizeof(double), s))) return rc;
        if ((rc = ensure(ctx, ctx->tmp2, (el_rows * M * 3 + 2 * (size_t)M * 3) * sizeof(double), s))) return rc;
        if ((rc = ensure(ctx, ctx->tmp3, (size_t)3 * M * 5 * sizeof(double), s))) return rc;
        if ((rc = ensure(ctx, ctx->red, (size_t)K * kV * sizeof(double), s))) return rc;
        seg64w = (double*)ctx->seg64.ptr;
        seg32w = (float*)ctx->seg32.ptr;
        el64w = (double*)ctx->elem64.ptr;
        el32w = (float*)ctx->elem32.ptr;
        part = (double*)ctx->tmp1.ptr;
        epart = (double*)ctx->tmp2.ptr;
        gx = (double*)ctx->tmp3.ptr;
        redw = (double*)ctx->red.ptr;
    }
    if ((rc = launch_expand_into(ctx, theta, H, seg64w, seg32w, s))) return rc;
    if (carve && (rc = launch_pack_elements_into(ctx, el64w, el32w, s))) return rc;
    double* psi = epart + el_rows * M * 3;
    double* mu = psi + (size_t)M * 3;
    double* gc = gx + (size_t)3 * M * 2;
    const double* seg64 = seg64w;
    const double* el64 = el64w;
    if (N > 0) {
        if (!mixed) {
            {
                ProfScope ps_(ctx, PT_VJP_SEGMENTS, s);
                hipLaunchKernelGGL(k_vjp_segments, dim3(kgroups, ns), dim3(256), 0, s, x, (const double*)gbar, N, chunk_s,
                                   seg64, K, eps2, part);
            }
            ProfScope ps_(ctx, PT_VJP_ELEMENTS, s);
            hipLaunchKernelGGL(k_vjp_elements, dim3(mgroups, ne), dim3(256), 0, s, x, (const double*)gbar, N, chunk_e,
                               el64, M, epart);
        } else if ((rc = adj_mixed(ctx, x, N, (const float*)gbar, K, grid, ns, ne, part, epart, s))) {
            return rc;
        }
        hipLaunchKernelGGL(k_reduce_parts, dim3(blocks_for((int64_t)M * 3, 64)), dim3(1024), 0, s, epart, ne,
                           (int64_t)M * 3, psi);
        if ((rc = check_launch(ctx, "vjp sweeps"))) return rc;
        if ((rc = launch_boundary_adjoint(ctx, psi, mu, gx, gc, s))) return rc;
        {
            ProfScope ps_(ctx, PT_VJP_SEGMENTS, s);
            hipLaunchKernelGGL(k_vjp_segments, dim3(kgroups, ng), dim3(256), 0, s, gx, gc, (int64_t)3 * M, chunk_g, seg64,
                               K, eps2, part + (size_t)ns * K * kV);
        }
        hipLaunchKernelGGL(k_reduce_parts, dim3(blocks_for((int64_t)K * kV, 64)), dim3(1024), 0, s, part,
                           ns + ng, (int64_t)K * kV, redw);
    } else {
        hipLaunchKernelGGL(k_reduce_parts, dim3(blocks_for((int64_t)K * kV, 64)), dim3(1024), 0, s, part, 0,
                           (int64_t)K * kV, redw);
    }
    hipLaunchKernelGGL(k_chain_theta, dim3(blocks_for((int64_t)H * ctx->npar, 64)), dim3(64), 0, s, (const double*)redw, H,
                       S, ctx->model, grad);
    return check_launch(ctx, "vjp");
}

}  // namespace bem

// ---- allocation-free float64 adjoint ----------------------------------------------------------
// Every workspace of bem_vjp_noalloc (segment and element tables, partial sums, psi, mu, boundary
// Gauss points, segment sums) is carved from this array; each device that runs the library holds
// its own copy for the life of the process.  Host code never passes the array's name to a kernel:
// its device address, found once per device with hipGetSymbolAddress, is kept in g_scratch.
namespace {
constexpr size_t kScratchBytes = (size_t)64 << 20;
constexpr int kScratchDevices = 64;
__device__ __align__(256) unsigned char scratch[kScratchBytes];
std::mutex g_scratch_mu;
void* g_scratch[kScratchDevices] = {};

// device address of this device's scratch array (the context's device is current)
int scratch_address(bem_ctx* ctx, char** out)
{
    const int dev = ctx->device;
    if (dev < 0 || dev >= kScratchDevices)
        return bem::set_error(ctx, BEM_EINVAL, "device %d beyond the %d the scratch table covers", dev, kScratchDevices);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch[dev]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return bem::set_error(ctx, BEM_EHIP, "hipGetSymbolAddress(scratch) on device %d: %s", dev,
                                  hipGetErrorString(e));
        g_scratch[dev] = p;
    }
    *out = (char*)g_scratch[dev];
    return BEM_OK;
}
}  // namespace

extern "C" int bem_vjp_noalloc(bem_ctx* ctx, const double* theta, int32_t H, const double* x, int64_t N,
                               const double* gbar, double* grad, hipStream_t stream)
{
    using namespace bem;
    int rc = check_common(ctx, theta, H, x, N);
    if (rc) return rc;
    if (N > 0 && !gbar) return set_error(ctx, BEM_EINVAL, "gbar is null");
    if (H > 0 && !grad) return set_error(ctx, BEM_EINVAL, "grad is null");
    const int K = H * ctx->opts.segs_per_handle;
    const size_t need = vjp_f64_workspace_bytes(K, ctx->M, N, false);       // the least run_vjp can do with
    if (need > kScratchBytes)
        return set_error(ctx, BEM_EINVAL, "bem_vjp_noalloc: %zu bytes of workspace for K = %d segments, M = %d "
                         "elements, N = %lld samples exceed its %zu-byte scratch", need, K, ctx->M, (long long)N,
                         kScratchBytes);
    char* base = nullptr;
    if ((rc = scratch_address(ctx, &base))) return rc;
    // no profiling events for this call (recording them may allocate)
    const bool prof = ctx->prof.on;
    ctx->prof.on = false;
    const Carve carve{base, kScratchBytes};
    rc = run_vjp(ctx, theta, H, x, N, gbar, false, grad, stream, &carve);
    ctx->prof.on = prof;
    return rc;
}

