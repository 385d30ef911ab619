// One weight update of Alg. 2: Adam on the mixed loss (reweighted training: the regulariser's
// gradient of Eq. 3, with the factors held fixed, is added to the incoming gradient on the fly)
// or on the prediction loss followed by W = W * Mask (retraining), in one pass over the state.
//
// Per parameter 16 bytes are read (w, g, m, v) and 12 written (w, m, v); the factor and the mask
// byte of a group once per four.  The path is HBM-bound; a lane takes about four rows of a group (a column segment
// of a row-block), and nothing crosses lanes.
// Adam itself is Kingma & Ba's Algorithm 1, evaluated in fp32 with one rounding per operation.
#include "bsp_common.h"

#include <cmath>

namespace bsp {
namespace {

constexpr int kThreads = 256;

struct AdamScalars {
    float lr, beta1, beta2, omb1, omb2, c1, c2, eps;
};

// grid.x covers the columns, one per lane (4-byte lanes stream faster here than 16-byte ones: measured 5.4 against
// 5.1 TB/s on 0.8 G parameters), grid.y the row-blocks, each in `parts` pieces of `rows` rows.  REG: the regulariser's gradient is added (alpha != nullptr);
// MASK: pruned groups are written as +0 (keep != nullptr).
template <int GDT, bool REG, bool MASK>
__global__ __launch_bounds__(kThreads) void adam_step_kernel(float *__restrict__ W, const void *__restrict__ G,
                                                             float *__restrict__ m, float *__restrict__ v, int64_t N,
                                                             int32_t R, int32_t rows, int32_t parts,
                                                             const float *__restrict__ alpha, float lambda,
                                                             int mode, const uint8_t *__restrict__ keep, AdamScalars h) {
    const int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (j >= N) return;
    const int32_t b = blockIdx.y / parts, r0 = (blockIdx.y - b * parts) * rows, r1 = r0 + rows < R ? r0 + rows : R;
    const int64_t base = (int64_t)b * R * N + j;
    float coef = 0.0f;
    bool kept = true;
    if constexpr (REG) {
        coef = lambda * alpha[(int64_t)b * N + j];
        if (mode == BSP_ALPHA_NORM) {  // the factor multiplies the norm itself: d||w||/dw = w / ||w||
            float s = 0.0f;
#pragma unroll 4
            for (int32_t r = 0; r < R; ++r) {
                const float w = W[base + (int64_t)r * N];
                s = __builtin_fmaf(w, w, s);
            }
            coef = (s > 0.0f) ? coef / __builtin_sqrtf(s) : 0.0f;
        }
    }
    if constexpr (MASK) kept = keep[(int64_t)b * N + j] != 0;
#pragma unroll 4
    for (int32_t r = r0; r < r1; ++r) {
        const int64_t off = base + (int64_t)r * N;
        const float w = W[off];
        float g = elem<GDT>::load(G, off);
        if constexpr (REG) g = __builtin_fmaf(coef, w, g);
        const float t1 = h.beta1 * m[off];
        const float t2 = h.omb1 * g;
        const float mn = t1 + t2;
        const float t3 = h.beta2 * v[off];
        float t4 = h.omb2 * g;
        t4 = t4 * g;
        const float vn = t3 + t4;
        const float mh = mn / h.c1;
        const float vh = vn / h.c2;
        const float num = h.lr * mh;
        const float den = __builtin_sqrtf(vh) + h.eps;
        const float q = num / den;
        float wn = w - q;
        if constexpr (MASK) wn = kept ? wn : 0.0f;
        W[off] = wn;
        m[off] = mn;
        v[off] = vn;
    }
}

template <int GDT>
void launch_adam(dim3 grid, hipStream_t s, float *W, const void *G, float *m, float *v, int64_t N, int32_t R,
                 int32_t rows, int32_t parts, const float *alpha, float lambda, int mode, const uint8_t *keep, const AdamScalars &h) {
    if (alpha && keep)
        adam_step_kernel<GDT, true, true><<<grid, kThreads, 0, s>>>(W, G, m, v, N, R, rows, parts, alpha, lambda, mode, keep, h);
    else if (alpha)
        adam_step_kernel<GDT, true, false><<<grid, kThreads, 0, s>>>(W, G, m, v, N, R, rows, parts, alpha, lambda, mode, keep, h);
    else if (keep)
        adam_step_kernel<GDT, false, true><<<grid, kThreads, 0, s>>>(W, G, m, v, N, R, rows, parts, alpha, lambda, mode, keep, h);
    else
        adam_step_kernel<GDT, false, false><<<grid, kThreads, 0, s>>>(W, G, m, v, N, R, rows, parts, alpha, lambda, mode, keep, h);
}

}  // namespace
}  // namespace bsp

using namespace bsp;

extern "C" int bsp_adam_step(float *W, const void *G, int gdt, float *m, float *v, int64_t M, int64_t N, int32_t R,
                             const float *alpha, float lambda, int mode, const uint8_t *keep, float lr, float beta1,
                             float beta2, float eps, int64_t t, void *stream) {
    if (!W || !G || !m || !v) return BSP_ERR_NULL;
    if (!valid_dtype(gdt)) return BSP_ERR_DTYPE;
    if (M <= 0 || N <= 0 || R <= 0 || M % R != 0 || t < 1) return BSP_ERR_SHAPE;
    if (alpha && mode != BSP_ALPHA_SQNORM && mode != BSP_ALPHA_NORM) return BSP_ERR_DTYPE;
    const int64_t B = M / R;
    if (B > 65535) return BSP_ERR_SHAPE;
    AdamScalars h;
    h.lr = lr;
    h.beta1 = beta1;
    h.beta2 = beta2;
    h.omb1 = 1.0f - beta1;
    h.omb2 = 1.0f - beta2;
    h.c1 = (float)(1.0 - std::pow((double)beta1, (double)t));
    h.c2 = (float)(1.0 - std::pow((double)beta2, (double)t));
    h.eps = eps;
    hipStream_t s = (hipStream_t)stream;
    const int64_t cols = (N + kThreads - 1) / kThreads;
    // About four rows of a row-block per thread: a thread with all of them walks them four loads at a time, and small
    // matrices then have one wavefront per SIMD.  Measured (fp32 state): 24576 x 1024, R = 16, bf16 gradient 121 -> 110 us, fp32
    // gradient 137 -> 127; 1024 x 1024 10.6 -> 7.1.  In pieces of one size: a piece of one row is a workgroup for a quarter of
    // the work (R = 5 in pieces of 4 and 1, 27190 x 258: 65.6 us, 44 in one piece; 319 matrices of R = 5 took 1.06 of the time of
    // whole row-blocks, up to 1.43).  From R = 8 on pieces of at most 5 rows take 0.92 (R = 8) to 0.79 (R = 15) of it; R = 7 0.94
    // on average, but one matrix in forty 1.1.  The printed form's factor needs the norm of the whole group: all rows.
    int32_t parts = alpha && mode == BSP_ALPHA_NORM ? 1 : (R + 1) / 4;
    if (R < 8 || B * parts > 65535) parts = 1;
    const int32_t rows = (R + parts - 1) / parts;
    const dim3 grid((unsigned)cols, (unsigned)(B * parts));
    BSP_DISPATCH_DTYPE(gdt, GDT, { launch_adam<GDT>(grid, s, W, G, m, v, N, R, rows, parts, alpha, lambda, mode, keep, h); });
    return check_launch();
}
