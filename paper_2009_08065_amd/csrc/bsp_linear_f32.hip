// The layer on its compact storage in single precision (Sec. 3.1, Sec. 4.4), from a tile of X in LDS; gfx950.
//
// The direct-gather kernel of bsp_linear.hip reads X from memory element by element: the 64 lanes of a load name 64
// different lines, so the 768 x 768 layer at 2x and 128 tokens took 15.4 us for 75 MFLOP.  Here a workgroup copies its
// 16 token rows into LDS once, whole lines at a time, transposed to [column][16 tokens], and gathers there: 7.4 us.
// A unit of work is 16 rows of a row-block (a slab); a workgroup takes `nu` units and NW / nu wavefronts share the kept
// columns of one, 16 at a time: lane group g = lane / 16 holds columns 4 g .. 4 g + 3 of the 16 as one 16-byte load each of
// weights and column numbers, and v_mfma_f32_16x16x4_f32 j takes the j-th of them, so a load serves four products.
// What a small call waits for is the chain blk_ptr -> operands -> product; the operands of the wavefront's first
// kMacros pieces are asked for before the copy-in, whose latency they share.  Partial sums meet in LDS in the order
// of the columns.
#include "bsp_common.h"
#include "bsp_linear_internal.h"
#include "bsp_mfma_device.h"
#include "bsp_tile_device.h"

namespace bsp {
namespace {

constexpr int kF32Waves = 8;
constexpr int kF32Threads = kF32Waves * 64;
constexpr int kMacros = 4;  // pieces of 16 kept columns whose operands are on their way
constexpr size_t kF32MaxLds = 160 * 1024;

__global__ __launch_bounds__(kF32Threads) void linear_f32_tile_kernel(
    const float *__restrict__ X, int64_t T, int64_t M, int64_t N, int32_t R, int32_t slabs, int64_t units, int32_t nu,
    int32_t ntiles, const int32_t *__restrict__ blk_ptr, const int32_t *__restrict__ col_idx,
    const float *__restrict__ vals, const float *__restrict__ bias, float *__restrict__ Y, int32_t vec_out) {
    const int tile = blockIdx.x % ntiles;
    const int64_t u0 = (int64_t)(blockIdx.x / ntiles) * nu;
    const int64_t t0 = (int64_t)tile * 16;
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    float *xt = reinterpret_cast<float *>(smem_x);
    const int kw = nu < kF32Waves ? kF32Waves / nu : 1;  // wavefronts per unit
    const int part = wave % kw;

    int64_t base = 0, m0 = 0;
    int kp = 0, lo = 0, hi = 0;  // this wavefront's pieces
    const float *wrow = vals;
    bool row_ok = false;
    auto locate = [&](int64_t u) {
        const int64_t b = u / slabs;
        const int r0 = (int)(u % slabs) * 16;
        base = blk_ptr[b];
        kp = blk_ptr[b + 1] - (int)base;
        const int pieces = (kp + 15) >> 4;
        lo = pieces * part / kw;
        hi = pieces * (part + 1) / kw;
        row_ok = r0 + l16 < R;
        wrow = vals + (int64_t)R * base + (int64_t)(row_ok ? r0 + l16 : 0) * kp;
        m0 = b * R + r0;
    };
    f32x4 w[kMacros];
    int4 c[kMacros];
    const int zero_col = (int)N;  // (places past the storage multiply zeros, never an infinite input)
    auto ask = [&](auto slot, int piece) {  // (rows, columns and pieces start at multiples of 4 elements)
        constexpr int j = decltype(slot)::value;
        const int k = 16 * piece + 4 * g;
        const bool ok = piece < hi && k < kp;
        c[j] = make_int4(zero_col, zero_col, zero_col, zero_col);
        w[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (ok) c[j] = *reinterpret_cast<const int4 *>(col_idx + base + k);
        if (ok && row_ok) w[j] = *reinterpret_cast<const f32x4 *>(wrow + k);
    };
    int64_t u = u0 + wave / kw;
    if (u < units) {
        locate(u);
        static_for<0, kMacros>([&](auto j) { ask(j, lo + j); });
    }

    // ---- 16 token rows into LDS; past T zeros ----
    {
        const int quads = (int)(N >> 2);
        const bool t_ok = t0 + l16 < T;
        const float *xrow = X + (t_ok ? t0 + l16 : 0) * N;
        constexpr int kBatch = 6, kPer = kF32Threads / 16;
        for (int q0 = tid >> 4; q0 < quads; q0 += kBatch * kPer) {
            f32x4 a[kBatch];
#pragma unroll
            for (int i = 0; i < kBatch; ++i) {
                const int q = q0 + i * kPer;
                a[i] = (t_ok && q < quads) ? *reinterpret_cast<const f32x4 *>(xrow + 4 * q) : f32x4{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int i = 0; i < kBatch; ++i) {
                const int q = q0 + i * kPer;
                if (q >= quads) break;
                // lane group g starts with the quad's column g, so that the four quads a wavefront writes at a time fall
                // into different banks
                float *dst = xt + 64 * q + l16;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int e = (k + g) & 3;
                    const float lo2 = e & 1 ? a[i][1] : a[i][0], hi2 = e & 1 ? a[i][3] : a[i][2];
                    dst[16 * e] = e & 2 ? hi2 : lo2;
                }
            }
        }
        if (tid < 16) xt[N * 16 + tid] = 0.0f;
    }
    __syncthreads();

    auto gather = [&](int col) { return xt[col * 16 + l16]; };
    // Four sums per output, for the latency of the products and so that a sum's error does not grow when fewer wavefronts
    // share a unit (2-norm 1.2e-7 to 1.8e-7 of the result over the shapes named at the launch, where the direct-gather kernel has 1.1e-7
    // to 2.9e-7).
    auto walk = [&]() {
        f32x4 acc[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int s = lo; s < hi; s += kMacros) {
            static_for<0, kMacros>([&](auto slot) {
                constexpr int j = decltype(slot)::value;
                const float x[4] = {gather(c[j].x), gather(c[j].y), gather(c[j].z), gather(c[j].w)};
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[j][i], x[i], acc[i], 0, 0, 0);
                ask(slot, s + kMacros + j);
            });
        }
        return (acc[0] + acc[1]) + (acc[2] + acc[3]);
    };
    // rows m .. m + 3 (of them `rows` inside the row-block) of one token
    auto finish = [&](f32x4 s, int64_t t, int64_t m, int rows) {
        if (t >= T || rows <= 0) return;
        if (vec_out) {
            if (bias) {
#pragma unroll
                for (int v = 0; v < 4; ++v) s[v] += bias[m + v];
            }
            *reinterpret_cast<f32x4 *>(Y + t * M + m) = s;
        } else {
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (v < rows) Y[t * M + m + v] = s[v] + (bias ? bias[m + v] : 0.0f);
        }
    };
    if (kw == 1) {  // whole units one after the other, straight from the registers
        for (; u < units && u < u0 + nu; u += kF32Waves) {  // (uniform in a wavefront; no barrier behind this point)
            if (u >= u0 + kF32Waves) {
                locate(u);
                static_for<0, kMacros>([&](auto j) { ask(j, lo + j); });
            }
            const f32x4 acc = walk();
            finish(acc, t0 + l16, m0 + 4 * g, R - (int)(u % slabs) * 16 - 4 * g);
        }
        return;
    }
    const f32x4 acc = walk();
    __syncthreads();  // the tile has been read
    f32x4 *red = reinterpret_cast<f32x4 *>(smem_x);
    red[tid] = acc;
    __syncthreads();
    if (part != 0 || u >= units) return;
    f32x4 sum = acc;
    for (int p = 1; p < kw; ++p) sum += red[tid + 64 * p];
    finish(sum, t0 + l16, m0 + 4 * g, R - (int)(u % slabs) * 16 - 4 * g);
}

size_t f32_lds(int64_t N) {
    const size_t tile = (size_t)(N + 1) * 64, red = (size_t)kF32Threads * 16;
    return tile > red ? tile : red;
}

}  // namespace

// Whole 16-byte pieces everywhere (k_align a multiple of 4, rows of X too), and 16 tokens of X inside the LDS.  Wider
// layers stay with the direct-gather kernel.
bool linear_f32_tile_supported(int64_t N, int32_t k_align, const int32_t *col_idx, const float *vals) {
    return N % 4 == 0 && k_align % 4 == 0 && col_idx && vals && aligned(col_idx, 16) && f32_lds(N) <= kF32MaxLds;
}

// The direct-gather kernel stays the faster one where row-blocks keep so little that copying whole rows of X costs more than
// naming its elements, and all of it fits the chip at once.  Measured, us, direct gather / tile: 512 x 2048 at 100x, 17 tokens
// 4.3 / 8.3, at 5x 10.2 / 8.9; 2304 x 768, R = 8, one token at 20x 4.3 / 6.9, at 1.43x 10.5 / 7.5; 64 x 64 at every rate 3.9 / 4.7;
// 512 x 2048 at 100x, 1024 tokens 10 / 12.  Of 936 calls of 64 to 8192 rows, 64 to 2556 columns, 1 to 1024 tokens, 1.43x to
// 100x, 177 were slower by more than 8 % in the tile, with this rule 31 (most of them up to 20 %).
bool linear_f32_tile_pays(int64_t T, int64_t M, int64_t N, int32_t R, int64_t capacity_cols) {
    const double slabs = (double)((R + 15) / 16), blocks = (double)(M / R);
    const double cols = (double)capacity_cols < blocks * (double)N ? (double)capacity_cols : blocks * (double)N;
    return cols / blocks * slabs > 64.0 + 0.03 * (double)N ||
           cols * slabs * (double)((T + 15) / 16) / 256.0 > 128.0 + 0.2 * (double)N;
}

int launch_linear_f32_tile(const float *X, int64_t T, int64_t M, int64_t N, int32_t R, const int32_t *blk_ptr,
                           const int32_t *col_idx, const float *vals, const float *bias, float *Y, hipStream_t s) {
    const int32_t slabs = (R + 15) / 16;
    const int64_t units = M / R * slabs, ntiles = (T + 15) / 16;
    // More units per workgroup share one copy-in, fewer leave compute units idle.  Measured, us for 1 / 2 / 4 / 8 / 16 / 32
    // units: 768 x 768 at 2x, 16 tokens 6.3 / 7.2 / 9.5 / 12.4 / .., 128 tokens 8.7 / 7.4 / 9.5 / .., 1024 tokens
    // 42 / 27 / 21.0 / 20.5 / 21.2 / 37; 2304 x 768 at 1.43x, 400 tokens 58 / 41 / 33 / 26.6 / 28.5 / 51; 3072 x 768 at 2x,
    // 1024 tokens 165 / 99 / 73 / 57 / 53 / 65; 512 x 2048 at 2x, 128 tokens 10.9 / 12.8 / ..
    auto workgroups = [&](int32_t n) { return ntiles * ((units + n - 1) / n); };
    int32_t nu = 8;
    if (workgroups(16) >= 512) nu = 16;
    while (nu > 1 && workgroups(nu) < 192) nu >>= 1;
    const int64_t wgs = workgroups(nu);
    if (wgs >= ((int64_t)1 << 31)) return BSP_ERR_SHAPE;
    static thread_local size_t configured = 65536;
    const size_t lds = f32_lds(N);
    const int st = raise_lds_limit(linear_f32_tile_kernel, lds, configured);
    if (st != BSP_OK) return st;
    const int32_t vec_out = R % 4 == 0 && aligned(Y, 16) ? 1 : 0;  // (so M % 4 == 0)
    linear_f32_tile_kernel<<<dim3((unsigned)wgs), kF32Threads, lds, s>>>(X, T, M, N, R, slabs, units, nu, (int32_t)ntiles,
                                                                        blk_ptr, col_idx, vals, bias, Y, vec_out);
    return check_launch();
}

}  // namespace bsp
