// common.hpp - context, workspaces and launch helpers shared by the library's
// translation units.  Not part of the public ABI (see include/bem.h).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdio>
#include <string>
#include <vector>

#include "../../include/bem.h"
#include "math64.hpp"
#include "seg_math.hpp"

namespace bem {

// ---- device math policies ---------------------------------------------------
struct DevF64 {
    __device__ static double log(double x) { return log_f64(x); }
    __device__ static double rcp(double x) { return rcp_f64(x); }
    __device__ static double rsqrt(double x) { return rsqrt_f64(x); }
    __device__ static double atan2(double y, double x) { return atan2_f64(y, x); }
    __device__ static double log_ratio(double R0, double R1, double dR) { return log_ratio_f64(R0, R1, dR); }
};

// Segments no longer than this (domain-width units) are degenerate: their
// integral is below ~1e-11 for the regularised kernels and the derivative
// with respect to their end points has no limit as the length goes to 0, so
// they contribute nothing (an expansion of a zero-length handle carries
// rounding-level lengths of ~1e-16).
constexpr double kDegenerateLength = 1e-12;

// ---- layouts ----------------------------------------------------------------
// Segment record: SegGeom (9 values) + wd_a, wd_b, wc_a, wc_b RGB (12) + 1/L2 + L + 1/L.
constexpr int kSegStride = 24;
// Element record: ax, ay, vx, vy, U0, U1, U2, pad.
constexpr int kElemStride = 8;

// density offsets inside a segment record, and the slots of 1/L2, L and 1/L (0 for a degenerate segment)
constexpr int kWdA = 9, kWdB = 12, kWcA = 15, kWcB = 18, kIL2 = 21, kLen = 22, kILen = 23;

template <class T>
__device__ inline SegGeom<T> load_geom(const T* __restrict__ s)
{
    SegGeom<T> g;
    g.ax = s[0]; g.ay = s[1]; g.bx = s[2]; g.by = s[3];
    g.vx = s[4]; g.vy = s[5]; g.L2 = s[6]; g.kd = s[7]; g.ks = s[8]; g.iL2 = s[kIL2];
    return g;
}

// ---- device buffers -----------------------------------------------------------
// A grid cell in the normal equations over cells (jtj_cells.hip)
struct CellInfo {
    int n;             // samples
    int nh, ne;        // near handles and outer elements
    int rows;          // near rows: (3 G + C) nh + ne
    int tb;            // first 32-sample block of the basis tile
    int rb;            // first row of the cell in the projections
    int64_t eoff;      // first element of its near tile
};

struct DevBuf {
    void* ptr = nullptr;
    size_t bytes = 0;
};

// A work list on the device and the configuration it was made for
struct WorkList {
    DevBuf buf;
    int64_t key[4] = {-1, -1, -1, -1};
};

}  // namespace bem

namespace bem {
// Kernel families timed with HIP events when profiling is on (bem_profile).
enum ProfTag {
    PT_SWEEP_F64 = 0, PT_SWEEP_MIXED, PT_VJP_SEGMENTS, PT_VJP_ELEMENTS, PT_FEATURES, PT_BETA_ROWS, PT_GRAM_F64,
    PT_GRAM_MFMA, PT_XR, PT_CHOLESKY, PT_BOUNDARY, PT_NEAR, PT_COUNT
};
struct ProfState {
    bool on = false;
    std::vector<hipEvent_t> pool;
    std::vector<int> tags;
    std::vector<hipEvent_t> starts, stops;
    double total_ms[PT_COUNT] = {};
    int64_t launches[PT_COUNT] = {};
};
}  // namespace bem

struct bem_ctx {
    bem_opts opts{};
    int M = 0;               // outer elements
    int per_side = 0;
    int state = 0;           // 0 empty, 1 built, 2 factored
    int device = 0;
    // handle parametrisation: parameters per handle, and per handle in a feature row of the
    // normal equations the geometry columns of one channel and the channel-shared colour columns
    int model = 0, npar = 20, ngeo = 8, ncol = 4;
    bem_reg reg{};           // regularisation terms of lm_step (all off by default)
    int64_t chol_P = -1;     // order of the last Cholesky factor (its inverted diagonal blocks are in cholw)
    // second stream (the Gram of a sample tile runs on it while the next tile's feature rows are
    // formed on the caller's stream; the Cholesky's panel and trailing update run on it beside the
    // diagonal blocks) and its events, created on first use
    hipStream_t s2 = nullptr;
    hipEvent_t ev[6] = {};
    // near-pair slots per wavefront of the mixed J tiles' lists (a multiple of 256, raised by
    // lm_step when a wavefront's near pairs overflow it)
    int near_slots = 1024;
    double bbox[4] = {0.0, 0.0, 1.0, 1.0};   // outer boundary's bounding box (x0, y0, x1, y1)
    double sigma_n = 0.0, shift = 0.0;
    std::string err;
    bem::ProfState prof;
    // one-time boundary system
    bem::DevBuf A, Apinv, LU, piv, un, vn, flag, scal, egeo;   // LU: A+^T once factored; egeo: outer elements [M][4] (a, b)
    // per-call workspaces
    bem::DevBuf seg64, seg32, F, U, elem64, elem32, red, tmp0, tmp1, tmp2, tmp3, tmp4, tmp5, lmw, nearf, regw, cholw, sortw,
        boxw, cellw, cellb, farw, necw, nezw, neew, gemmw;
    // cell table and work list of the normal equations over cells, kept until their upload has ended
    std::vector<bem::CellInfo> ne_info;
    std::vector<int> ne_work;
    // Gram work list of the normal equations on the device, uploaded once per (W, H, handle
    // model, Gram arithmetic) and kept, so that later calls enqueue without a host synchronisation
    // (that over cells has its own, so that steps between calls of bem_jtj leave theirs in place)
    bem::WorkList tilew, halfw;
};

namespace bem {

int set_error(bem_ctx* ctx, int code, const char* fmt, ...);
void prof_begin(bem_ctx* ctx, int tag, hipStream_t s, hipEvent_t* start);
void prof_end(bem_ctx* ctx, int tag, hipStream_t s, hipEvent_t start);

// Records HIP events around the launches of its scope when profiling is on.
struct ProfScope {
    bem_ctx* ctx;
    int tag;
    hipStream_t s;
    hipEvent_t start = nullptr;
    ProfScope(bem_ctx* c, int t, hipStream_t st) : ctx(c), tag(t), s(st) { prof_begin(ctx, tag, s, &start); }
    ~ProfScope() { prof_end(ctx, tag, s, start); }
};
int ensure(bem_ctx* ctx, DevBuf& b, size_t bytes, hipStream_t stream);
void release(DevBuf& b);         // (no kernel queued may use it)
// argument checks shared by the per-call entry points; makes the context's device current
int check_common(bem_ctx* ctx, const double* theta, int32_t H, const double* x, int64_t N);
int aux_stream(bem_ctx* ctx, hipStream_t* out);
int check_launch(bem_ctx* ctx, const char* what);

inline int blocks_for(int64_t n, int threads) { return (int)((n + threads - 1) / threads); }

// ---- kernels' host launchers (defined in the .hip files) ----------------------
// factor.hip
int launch_square_elements(bem_ctx* ctx, hipStream_t s);
int launch_assemble(bem_ctx* ctx, hipStream_t s);
int launch_factor(bem_ctx* ctx, hipStream_t s);
// forward.hip
int launch_expand(bem_ctx* ctx, const double* theta, int H, hipStream_t s);
int launch_expand_into(bem_ctx* ctx, const double* theta, int H, double* seg64, float* seg32, hipStream_t s);
int launch_boundary_rhs(bem_ctx* ctx, int K, double* F, bool mixed, hipStream_t s);
int launch_boundary_solve(bem_ctx* ctx, const double* F, double* U, hipStream_t s);
int launch_boundary_adjoint(bem_ctx* ctx, const double* psi, double* mu, double* gx, double* gc, hipStream_t s);
int launch_pack_elements(bem_ctx* ctx, hipStream_t s);
int launch_pack_elements_into(bem_ctx* ctx, double* el64, float* el32, hipStream_t s);
int launch_sweep_f64(bem_ctx* ctx, const double* x, int64_t N, int K, const double* cbar_host, double* u, hipStream_t s);
// mixed forward sweep (sweep_eval.hip)
int launch_sweep_eval(bem_ctx* ctx, const double* x, int64_t N, int K, const double* cbar_host, float* u, hipStream_t s);
// Near-pair list of the mixed J tiles (sweep_common.hpp): the samples' near pairs with segments (and with
// outer elements when M > 0)
struct NearList;
int near_classify(bem_ctx* ctx, DevBuf& buf, const double* x, int64_t N, int K, int M, NearList* out, hipStream_t s);
// culling boxes of the current segment table (groups of kBoxGroup segments, then of M outer
// elements) into the context's box buffer
int near_boxes(bem_ctx* ctx, int K, int M, const float4** box, hipStream_t s);
// partition.hip (off_host may be null: no readback and no host synchronisation)
int run_partition(bem_ctx* ctx, const int32_t* labels, int64_t N, int D, const double* x, const double* T, double* xo,
                  double* To, int64_t* off_host, hipStream_t s);
// reg.hip
bool reg_active(const bem_ctx* ctx);
int check_reg(const bem_reg& r, char* why, size_t n);
int reg_terms(bem_ctx* ctx, const double* theta, int H, bool choose, double* g, double* Hm, double* value, int* pairs,
              hipStream_t s);
int run_prune(bem_ctx* ctx, double* theta, int H, double thr, int* H_out, hipStream_t s);
// vjp.hip
// Device memory the float64 adjoint may carve every workspace from instead of allocating (the
// allocation-free entry point's static array); null: the context's workspaces.
struct Carve {
    char* base;
    size_t bytes;
};
int run_vjp(bem_ctx* ctx, const double* theta, int H, const double* x, int64_t N, const void* gbar, bool mixed,
            double* grad, hipStream_t s, const Carve* carve = nullptr);
// api.hip: the forward set-up: expand, boundary right-hand side (float32 far pairs when mixed), boundary
// solve into the element tables
int prepare_forward(bem_ctx* ctx, const double* theta, int H, bool mixed, hipStream_t s);
// gemm.hip
// C = alpha A B^T + beta C, row-major, A [m][k], B [n][k]; a batch's operands sa, sb, sc apart
constexpr int kGemmPad = 16;
struct Gemm64 {
    int m, n, k;                 // k a multiple of kGemmPad (zeros), rows of A and B 16-byte aligned
    double alpha;
    const double* A;
    int64_t lda;
    const double* B;
    int64_t ldb;
    double beta;
    double* C;
    int64_t ldc;
    int64_t sa = 0, sb = 0, sc = 0;
};
inline int gemm_pad(int64_t k) { return (int)((k + kGemmPad - 1) / kGemmPad * kGemmPad); }
// on float64 MFMA
int gemm_f64(bem_ctx* ctx, const Gemm64& g, int batch, hipStream_t s);
// the float64 Gram on float64 MFMA: work entries (row tile, column tile, part) of 128 x 128 output tiles, part p of
// k range [p kchunk, (p + 1) kchunk) into C + p cstride
int gemm_f64_list(bem_ctx* ctx, const Gemm64& g, hipStream_t s, const int* work, int nwork, int kchunk, int64_t cstride);
// on the VALU (Gram mode FP64_VALU): a list of 64 x 64 output tiles
int gemm_f64_valu(bem_ctx* ctx, const Gemm64& g, hipStream_t s, const int* tiles, int ntiles);
// jtj.hip
int fill_f64(bem_ctx* ctx, double* p, int64_t n, double v, hipStream_t s);
int run_jtj(bem_ctx* ctx, const double* theta, int H, const double* x, int64_t N, bool mixed, int gram, double* JtJ,
            hipStream_t s, const NearList* pre = nullptr, double norm = 0.0);
int run_jacobian(bem_ctx* ctx, const double* theta, int H, const double* x, int64_t N, double* J, hipStream_t s);
// gram_mfma.hip
int launch_gram_mfma(bem_ctx* ctx, int gram, const void* Xhi, const uint16_t* Xlo, int64_t ld, int W, int64_t n,
                     const int* work, int nwork, int64_t kchunk, double* G, int64_t gstride, bool accumulate,
                     hipStream_t s);
// chol.hip
int64_t chol_size(int64_t P);
int chol_factor(bem_ctx* ctx, const double* H, int64_t P, double lam, const double* B, int nrhs, double* A, int* dflag,
                double* dscal, hipStream_t s);
int chol_solve(bem_ctx* ctx, double* A, int64_t P, double* X, int nrhs, hipStream_t s);
// lm.hip
int fill_i32(bem_ctx* ctx, int* p, int64_t n, int v, hipStream_t s);
int scale_f64(bem_ctx* ctx, double* p, int64_t n, double v, hipStream_t s);
int run_lm_step(bem_ctx* ctx, double* theta, int H, const double* x, int64_t N, const double* T, bem_lm_state* st,
                int gram, bool mixed, hipStream_t s);

}  // namespace bem

namespace bem {
// float32 policy of the mixed sweeps: hardware log2, reciprocal, reciprocal
// square root and square root (about 1 ulp); log1p(z) = log(w) z / (w - 1) with
// w = 1 + z rounded (Goldberg 1991: the rounding error of w cancels between the
// two factors), z itself when w == 1; atan2 by reduction to [0, 1] and a
// degree-7 odd minimax polynomial in z (relative error 1e-7; coefficients from
// csrc/fit_atan.py), reflected about pi/4 and pi/2.
struct DevF32 {
    // v_log_f32 (log2, ~1 ulp) times ln 2; arguments here are normal numbers (>= eps^2 or near 1)
    __device__ static float log(float x) { return __builtin_amdgcn_logf(x) * 0.693147180559945309f; }
    __device__ static float log2(float x) { return __builtin_amdgcn_logf(x); }
    __device__ static float rcp(float x) { return __builtin_amdgcn_rcpf(x); }
    __device__ static float rsqrt(float x) { return __builtin_amdgcn_rsqf(x); }
    __device__ static float sqrt(float x) { return __builtin_amdgcn_sqrtf(x); }
    __device__ static float log1p(float z)
    {
        const float w = 1.0f + z;
        const float d = w - 1.0f;
        return d == 0.0f ? z : (__builtin_amdgcn_logf(w) * 0.693147180559945309f) * (z * __builtin_amdgcn_rcpf(d));
    }
    __device__ static float atan2(float y, float x)
    {
        const float ax = fabsf(x), ay = fabsf(y);
        if (__all(ay < 0.2f * x)) {          // most wavefronts (see atan2_f64): atan's series, next term 9e-9 of z
            const float z = y * __builtin_amdgcn_rcpf(x), s = z * z;
            return z + z * s * (-3.333333433e-01f + s * (2.000000030e-01f + s * (-1.428571492e-01f + s * 1.111111119e-01f)));
        }
        const float mx = fmaxf(ax, ay), mn = fminf(ax, ay);
        const float z = mx > 0.0f ? mn * __builtin_amdgcn_rcpf(mx) : 0.0f;
        const float s = z * z;
        float p = -4.693678257e-03f;
        p = p * s + 2.425393176e-02f;
        p = p * s - 5.948871678e-02f;
        p = p * s + 9.914472679e-02f;
        p = p * s - 1.401955544e-01f;
        p = p * s + 1.996973974e-01f;
        p = p * s - 3.333199223e-01f;
        p = p * s + 9.999999014e-01f;
        float r = z * p;
        r = ay > ax ? 1.57079632679489662f - r : r;
        r = x < 0.0f ? 3.14159265358979324f - r : r;
        return __builtin_copysignf(r, y);
    }
};
}  // namespace bem
