// near_list.hip - near-pair lists of the mixed J tiles (jtj.hip) and the boxes that cull their tests.
//
// A pair whose two end points both lie within max(2 nf, nf + 1)*L of the sample, nf = near_factor (a set
// containing every sample closer than nf*L to the segment), is left out of the float32 features: the
// wavefront of its sample appends (sample, segment) to its own slice of a list, from which the pairs are
// evaluated in float64.  Should a wavefront's slice overflow, the samples whose pairs did not fit are
// flagged and recomputed by kernels that evaluate near pairs inline.
#include "common.hpp"
#include "sweep_common.hpp"

namespace bem {

namespace {


// Appending needs no atomics: each wavefront owns a slice and counts its entries
// in a wave-uniform register.

__device__ inline void append_near(bool near, int32_t sample, int32_t seg, NearPair* __restrict__ slice, int slots,
                                   int& used, bool& overflow)
{
    const uint64_t mask = __ballot(near);
    if (mask == 0) return;
    const int lane = threadIdx.x & 63;
    if (near) {
        const int slot = used + __popcll(mask & ((1ull << lane) - 1ull));
        if (slot < slots) slice[slot] = NearPair{sample, seg};
        else overflow = true;
    }
    used += __popcll(mask);
}

// Bounding boxes for culling near-pair tests per wavefront: box g (g < ceil(K / kBoxGroup): segments
// [kBoxGroup g, kBoxGroup (g + 1)); after those, group g - nsg of kBoxGroup outer elements) = the end
// points' extent (xmin, ymin, xmax, ymax) and the largest near radius sqrt(near2 L2) of its members.
// Degenerate segments (L2 = 0) are never near and are left out; a box with no member is empty
// (min > max) and culls everything.
__global__ void k_near_boxes(const float* __restrict__ seg32, int K, const float* __restrict__ el32, int M,
                             float near2, float4* __restrict__ box)
{
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    const int nsg = (K + kBoxGroup - 1) / kBoxGroup;
    if (g >= nsg + (M + kBoxGroup - 1) / kBoxGroup) return;
    float x0 = INFINITY, y0 = INFINITY, x1 = -INFINITY, y1 = -INFINITY, r = 0.0f;
    if (g < nsg) {
        const int k1 = (g + 1) * kBoxGroup < K ? (g + 1) * kBoxGroup : K;
        for (int k = g * kBoxGroup; k < k1; ++k) {
            const float* sg = seg32 + (size_t)k * kSegStride;
            if (sg[6] == 0.0f) continue;
            x0 = fminf(x0, fminf(sg[0], sg[2])); x1 = fmaxf(x1, fmaxf(sg[0], sg[2]));
            y0 = fminf(y0, fminf(sg[1], sg[3])); y1 = fmaxf(y1, fmaxf(sg[1], sg[3]));
            r = fmaxf(r, sqrtf(near2 * sg[6]));
        }
    } else {
        const int j0 = (g - nsg) * kBoxGroup, j1 = j0 + kBoxGroup < M ? j0 + kBoxGroup : M;
        for (int j = j0; j < j1; ++j) {
            const float* e = el32 + (size_t)j * kElemStride;
            const float bx = e[0] + e[2], by = e[1] + e[3];
            x0 = fminf(x0, fminf(e[0], bx)); x1 = fmaxf(x1, fmaxf(e[0], bx));
            y0 = fminf(y0, fminf(e[1], by)); y1 = fmaxf(y1, fmaxf(e[1], by));
            r = fmaxf(r, sqrtf(near2 * (e[2] * e[2] + e[3] * e[3])));
        }
    }
    box[2 * g] = make_float4(x0, y0, x1, y1);
    box[2 * g + 1] = make_float4(r, 0.0f, 0.0f, 0.0f);
}

// Near-pair classification.  Each wavefront first bounds its samples and skips every
// group of kBoxGroup segments (and of outer elements) whose box is farther than its near radius;
// the exact test runs for the others, in segment order.  With samples visited cell by cell a
// wavefront's box is small and most groups are skipped.
__global__ void __launch_bounds__(256) k_classify(const double* __restrict__ x, int64_t N,
                                                  const float* __restrict__ seg32, int K,
                                                  const float* __restrict__ el32, int M, float near2,
                                                  const float4* __restrict__ box,
                                                  NearPair* __restrict__ list, int slots, int* __restrict__ wave_count,
                                                  uint8_t* __restrict__ flag, int* __restrict__ need)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t wave = i >> 6;
    NearPair* slice = list + wave * slots;
    const bool live = i < N;
    const float Xf = live ? (float)x[2 * i] : 0.0f, Yf = live ? (float)x[2 * i + 1] : 0.0f;
    const float wx0 = uniform_f32(wave_min(live ? Xf : INFINITY)), wx1 = uniform_f32(wave_max(live ? Xf : -INFINITY));
    const float wy0 = uniform_f32(wave_min(live ? Yf : INFINITY)), wy1 = uniform_f32(wave_max(live ? Yf : -INFINITY));
    bool overflow = false;
    int used = 0;
    const int nsg = (K + kBoxGroup - 1) / kBoxGroup;
    for (int g = 0; g < nsg; ++g) {
        if (box_culled(box, g, wx0, wy0, wx1, wy1)) continue;
        const int k1 = (g + 1) * kBoxGroup < K ? (g + 1) * kBoxGroup : K;
        for (int k = g * kBoxGroup; k < k1; ++k) {
            const float* s = seg32 + (size_t)k * kSegStride;
            const bool near = live & near_segment(s[0], s[1], s[2], s[3], s[6], Xf, Yf, near2);
            append_near(near, (int32_t)i, k, slice, slots, used, overflow);
        }
    }
    for (int g = 0; g * kBoxGroup < M; ++g) {
        if (box_culled(box, nsg + g, wx0, wy0, wx1, wy1)) continue;
        const int j1 = (g + 1) * kBoxGroup < M ? (g + 1) * kBoxGroup : M;
        for (int j = g * kBoxGroup; j < j1; ++j) {
            const float* e = el32 + (size_t)j * kElemStride;
            const bool near = live & near_element(e[0], e[1], e[2], e[3], Xf, Yf, near2);
            append_near(near, (int32_t)i, K + j, slice, slots, used, overflow);
        }
    }
    if ((threadIdx.x & 63) == 0) {
        wave_count[wave] = used < slots ? used : slots;
        if (used > slots) atomicMax(need, used);
    }
    if (live) flag[i] = overflow ? 1 : 0;
}

}  // namespace

int near_boxes(bem_ctx* ctx, int K, int M, const float4** box, hipStream_t s)
{
    int rc;
    const int nbox = (K + kBoxGroup - 1) / kBoxGroup + (M + kBoxGroup - 1) / kBoxGroup;
    if ((rc = ensure(ctx, ctx->boxw, (size_t)(nbox > 0 ? nbox : 1) * 2 * sizeof(float4), s))) return rc;
    const double nf = near_radius(ctx->opts.near_factor);
    if (nbox > 0)
        hipLaunchKernelGGL(k_near_boxes, dim3(blocks_for(nbox, 256)), dim3(256), 0, s, (const float*)ctx->seg32.ptr, K,
                           (const float*)ctx->elem32.ptr, M, (float)(nf * nf), (float4*)ctx->boxw.ptr);
    *box = (const float4*)ctx->boxw.ptr;
    return check_launch(ctx, "near boxes");
}

// Classify the near pairs of samples x[0..N) (segments, and outer elements when M > 0) into buf.
int near_classify(bem_ctx* ctx, DevBuf& buf, const double* x, int64_t N, int K, int M, NearList* out, hipStream_t s)
{
    int rc;
    const double nf = near_radius(ctx->opts.near_factor);
    const int64_t nwaves = N > 0 ? (int64_t)blocks_for(N, 256) * 4 : 0;
    const int slots = near_slots_for(ctx->near_slots, nwaves);
    // list [nwaves][slots] | counts [nwaves] | overflow count (256 bytes) | flags [N]
    const size_t list_bytes = ((size_t)nwaves * slots * sizeof(NearPair) + 255) / 256 * 256;
    const size_t cnt_bytes = ((size_t)nwaves * sizeof(int) + 255) / 256 * 256;
    if ((rc = ensure(ctx, buf, list_bytes + cnt_bytes + 256 + (size_t)N + 256, s))) return rc;
    char* base = (char*)buf.ptr;
    out->list = (NearPair*)base;
    out->count = (int*)(base + list_bytes);
    out->need = (int*)(base + list_bytes + cnt_bytes);
    out->flag = (uint8_t*)(base + list_bytes + cnt_bytes + 256);
    out->nwaves = nwaves;
    out->slots = slots;
    if ((rc = fill_i32(ctx, out->need, 1, 0, s))) return rc;
    if (N == 0) return BEM_OK;
    ProfScope ps_(ctx, PT_NEAR, s);
    const float4* box;
    if ((rc = near_boxes(ctx, K, M, &box, s))) return rc;
    hipLaunchKernelGGL(k_classify, dim3(blocks_for(N, 256)), dim3(256), 0, s, x, N, (const float*)ctx->seg32.ptr, K,
                       (const float*)ctx->elem32.ptr, M, (float)(nf * nf), box, out->list, slots,
                       out->count, out->flag, out->need);
    return check_launch(ctx, "classify");
}

}  // namespace bem
