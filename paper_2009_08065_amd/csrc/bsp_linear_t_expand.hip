// The transposed product Z = U Wp (+ bias) (see bsp_linear_t.hip) as a dense product on the expanded matrix, both
// written here; bf16 / fp16, R % 8 == 0, with a workspace for the expanded matrix.
//
// Measured (MI355X, 8192 tokens, R = 16, 5x, both kernels): 4096 x 1024 64 us, 3072 x 1024 51, 1024 x 1024 27,
// 1024 x 4096 76, against 217 / 171 / 67 / 227 of the scattering kernel; 2304 x 768, R = 8, 2x, 509 tokens: 15.7 against 337.
//
// Why dense: the result of a row-block's small product has to be scattered to the kept columns' positions, and an
// addition to a scattered position costs an LDS read and write of 4 bytes for R multiply-adds.  That bounds the
// scattering kernel of bsp_linear_t.hip near 160 TFLOP/s of useful work for R = 16, and it reached 60.  Multiplying
// the pruned zeros as well costs 1 / density times the products, but the sums stay in registers.
// It is taken at every rate: the scattering kernel's time falls with what is kept, but only to its walk over the row-blocks and the
// sums in LDS.  Of 8714 calls of 128 to 16384 rows, 64 to 4096 columns, 1 to 8192 tokens, R = 8 to 64, 1.1x to 100x, one was
// slower by more than 1 % (1472 x 1304, R = 64, 61x, 2303 tokens 29.1 us, 27.0 there); beyond 50x and 1024 tokens the mean is 0.43 of its time.
//
// Two kernels: expand_kernel writes Wp as matrix-core operands, tile_kernel multiplies.
//
// A pruned weight must not meet U: 0 times an infinite input would be NaN.  Every column of a token with a
// non-finite input gets a non-finite sum here, so sums that are all finite are the right ones.  The tokens with a
// non-finite sum are multiplied again, each row-block's products by themselves, and only what the kept positions give is
// taken (kept_sums); the expansion writes one bit per row-block and column for that.
#include "bsp_common.h"
#include "bsp_linear_internal.h"
#include "bsp_mfma_device.h"

// The layer itself on its compact storage (bsp_linear_ws) is the same product with the roles of rows and columns changed:
// Y = X Wp^T, expanded by expand_rows_kernel, for layers that keep so much that the gather of their columns costs more than
// multiplying the zeros (linear_expand_pays).
namespace bsp {
namespace {

constexpr int kThreadsX = 256;  // of the expansions
constexpr int kRing = 4;       // stages of U in LDS
constexpr int kStageK = 64;    // rows of the matrix per stage
constexpr int kRowBytes = 2 * kStageK;
constexpr int kColPad = 256;   // columns of the expanded matrix are padded to whole workgroup tiles
constexpr uint32_t kRangeGroup = 4;
constexpr int kFrag = 1024;    // bytes of an operand of v_mfma_f32_32x32x16: 32 columns x 16 rows

// Bit n of row b of `kept`: row-block b keeps column n; rows are whole groups of kColPad columns.  (The workgroup of 256
// columns whose thread t holds column t's place, of the row-block's first slab.)
__device__ __forceinline__ void write_kept(uint64_t *__restrict__ kept, int b, int place) {
    const uint64_t bits = __ballot(place >= 0);
    if (blockIdx.z == 0 && (threadIdx.x & 63) == 0)
        kept[((int64_t)b * gridDim.y + blockIdx.y) * (kColPad / 64) + (threadIdx.x >> 6)] = bits;
}

// ---------------------------------------------------------------------------------------
// Expansion.  The expanded matrix is stored as operands: fragment (n / 32, m / 16) at (n / 32) frags_m + m / 16, lane l
// of it holding column n % 32 = l % 32, rows 8 (l / 32) .. + 7 of the 16.  One workgroup per row-block, 256 columns and
// 16 of its rows: an inverse map (column -> kept position) in LDS, then one 16-byte piece per thread and 8 rows, its
// values gathered down the panel (neighbouring kept columns are neighbouring positions).  It is a chain of four loads
// that wait for each other, so what counts is that all of them are in flight at once: 1024 columns per workgroup
// took 9 us for the BERT-large matrices.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(kThreadsX) void expand_kernel(int32_t R, int32_t B, int32_t frags_m,
                                                           const int32_t *__restrict__ blk_cnt,
                                                           const int32_t *__restrict__ blk_ptr,
                                                           const int32_t *__restrict__ col_idx,
                                                           const uint16_t *__restrict__ vals, uint8_t *__restrict__ out,
                                                           uint64_t *__restrict__ kept) {
    __shared__ int32_t place[kColPad];
    const int tid = threadIdx.x, b = blockIdx.x, c0 = blockIdx.y * kColPad, r0 = blockIdx.z * 16;
    place[tid] = -1;
    const int64_t base = blk_ptr[b];
    const int kp = (int)(blk_ptr[b + 1] - base), k = blk_cnt[b];
    __syncthreads();
    for (int p = tid; p < k; p += kThreadsX) {
        const int c = col_idx[base + p] - c0;
        if ((unsigned)c < (unsigned)kColPad) place[c] = p;
    }
    __syncthreads();
    const int p = place[tid], n = c0 + tid;
    write_kept(kept, b, p);
    const uint16_t *v = vals + ((int64_t)R * base + (int64_t)r0 * kp + (p < 0 ? 0 : p));
    uint8_t *column = out + (int64_t)(n >> 5) * frags_m * kFrag + (n & 31) * 16;
    const int o0 = (b * R + r0) >> 3;
#pragma unroll
    for (int o = 0; o < 2; ++o) {
        if (r0 + 8 * o >= R) break;  // uniform (R is a multiple of 8)
        uint32_t d[4] = {0u, 0u, 0u, 0u};
        if (p >= 0) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                d[j] = v[(int64_t)(8 * o + 2 * j) * kp] | ((uint32_t)v[(int64_t)(8 * o + 2 * j + 1) * kp] << 16);
        }
        *reinterpret_cast<uint4 *>(column + (int64_t)((o0 + o) >> 1) * kFrag + (((o0 + o) & 1) << 9)) = make_uint4(d[0], d[1], d[2], d[3]);
    }
    if (b == B - 1 && blockIdx.z == 0)  // the zero rows that fill the last stage
        for (int o = (B * R) >> 3; o < 2 * frags_m; ++o)
            *reinterpret_cast<uint4 *>(column + (int64_t)(o >> 1) * kFrag + ((o & 1) << 9)) = make_uint4(0u, 0u, 0u, 0u);
}

// The same for Wp itself: operand (m / 32, n / 16), lane l of it row m % 32 = l % 32, columns 8 (l / 32) .. + 7 of the 16.
// One workgroup per row-block, 256 columns and 16 of its rows; row-blocks past the last write the zero rows that fill
// the last tile.
__global__ __launch_bounds__(kThreadsX) void expand_rows_kernel(int32_t R, int32_t B, int32_t rows_pad, int32_t frags_n,
                                                                const int32_t *__restrict__ blk_cnt,
                                                                const int32_t *__restrict__ blk_ptr,
                                                                const int32_t *__restrict__ col_idx,
                                                                const uint16_t *__restrict__ vals, uint8_t *__restrict__ out,
                                                                uint64_t *__restrict__ kept) {
    __shared__ int32_t place[kColPad];
    const int tid = threadIdx.x, b = blockIdx.x, c0 = blockIdx.y * kColPad, r0 = blockIdx.z * 16;
    place[tid] = -1;
    const int64_t base = b < B ? blk_ptr[b] : 0;
    const int kp = b < B ? (int)(blk_ptr[b + 1] - base) : 0, k = b < B ? blk_cnt[b] : 0;
    __syncthreads();
    for (int p = tid; p < k; p += kThreadsX) {
        const int c = col_idx[base + p] - c0;
        if ((unsigned)c < (unsigned)kColPad) place[c] = p;
    }
    __syncthreads();
    if (b < B) write_kept(kept, b, place[tid]);
    const int r = r0 + (tid & 15), m = b * R + r;
    if (r >= R || m >= rows_pad) return;
    const uint16_t *v = vals + ((int64_t)R * base + (int64_t)r * kp);
    uint8_t *row = out + (int64_t)(m >> 5) * frags_n * kFrag + (m & 31) * 16;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int o = (tid >> 4) + 16 * j, n8 = (c0 >> 3) + o;  // 8 columns
        if (n8 >= 2 * frags_n) break;
        uint32_t d[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int p = place[8 * o + i];
            if (p >= 0) d[i >> 1] |= (uint32_t)v[p] << (16 * (i & 1));
        }
        *reinterpret_cast<uint4 *>(row + (int64_t)(n8 >> 1) * kFrag + ((n8 & 1) << 9)) = make_uint4(d[0], d[1], d[2], d[3]);
    }
}

// The wavefront's sums of 32 tokens over the kept positions alone, into acc (its FN pieces of 32 columns).  It costs a few times
// the dense product, for every input alike: with every token of the batch not finite (an overflow in fp16 training), us, the kernel
// on the storage / this: Z, 4096 x 1024, 8192 tokens, R = 16 at 5x 229 / 533 (61 where all sums are finite), 768 x 3072, 4096 tokens,
// R = 8 at 2x 271 / 228; Y, 1024 x 4096, 8192 tokens, R = 16 at 5x 122 / 436, at 1.43x 349 / 456.  One such token: 170 and 163.
// (Each token by itself from the storage, as it was, took 25 and 44 ms for whole batches of 4096 tokens.)
//   Z = U Wp: the rows of a step of 16 belong to one row-block, or 8 and 8 to two (R % 8 == 0): each one's products start
//   from zero and are added where the row-block keeps the column.
//   Y = X Wp^T: two row-blocks at a time, X zeroed where each prunes the column; of the sums of 32 rows its own are taken.
//   A row-block's pads are zero weights of its last kept column, and part of the layer's sum.
// u: the lane's token's row.
template <int DT, int FN, bool ROWS>
__device__ __forceinline__ void kept_sums(const uint8_t *u, int32_t M, int32_t N, int32_t R, int32_t frags_m,
                                          const uint8_t *wcol, int wcol0, const uint32_t *__restrict__ kept,
                                          const int32_t *__restrict__ blk_cnt, const int32_t *__restrict__ blk_ptr,
                                          const int32_t *__restrict__ col_idx, f32x16 (&acc)[FN]) {
    constexpr int kDepth = ROWS ? 2 : 4;                 // steps whose operands are on their way (what the registers allow)
    constexpr int kW = ROWS ? 1 : FN, kB = ROWS ? 2 : FN;  // of a step: weight operands, words of `kept`
    const int lane = threadIdx.x & 63, kh = lane >> 5;
    const int words = ((ROWS ? M : N) + kColPad - 1) / kColPad * (kColPad / 32);  // of a row of `kept`
    const int steps = (M + 15) / 16;
    // the row-block of rows 8 o .. 8 o + 7 (Z = U Wp: R % 8 == 0); exact below 2^28, and o is below 2^20
    const uint32_t per_block = ROWS ? 1u : (0x80000000u + (uint32_t)(R >> 3) - 1u) / (uint32_t)(R >> 3);
    auto block_of = [&](int o) { return (int)__umulhi(2u * (uint32_t)o, per_block); };
    uint4 w[kDepth][kW], x[kDepth];
    uint32_t bits[kDepth][kB];
    // n0: first piece.  ROWS: row-blocks b and b2; else lanes 0 and 1 hold the words of the row-blocks of the step's halves
    auto ask = [&](auto slot, int step, int n0, int b, int b2) {
        constexpr int s = decltype(slot)::value;
        const int f = step < steps ? step : steps - 1;
#pragma unroll
        for (int n = 0; n < kW; ++n) w[s][n] = *reinterpret_cast<const uint4 *>(wcol + ((int64_t)(n0 + n) * frags_m + f) * kFrag + lane * 16);
        const int k = 16 * f + 8 * kh;  // past the last row: any value, zeroed below (M is a multiple of 8)
        x[s] = *reinterpret_cast<const uint4 *>(u + 2 * (int64_t)(k < M ? k : M - 8));
        if constexpr (ROWS) {
            bits[s][0] = kept[(int64_t)b * words + (f >> 1)];
            bits[s][1] = kept[(int64_t)b2 * words + (f >> 1)];
        } else {
            const int o = 2 * f + (lane & 1);
            const uint32_t *row = kept + ((int64_t)block_of(8 * o < M ? o : 2 * f) * words + (wcol0 >> 5));
#pragma unroll
            for (int n = 0; n < FN; ++n) bits[s][n] = row[n];
        }
    };
    auto walk = [&](int n0, int b, int b2, auto use) {
        static_for<0, kDepth>([&](auto j) { ask(j, j, n0, b, b2); });
        int f0 = 0;
        for (; f0 + kDepth <= steps; f0 += kDepth)
            static_for<0, kDepth>([&](auto j) {
                use(j, f0 + j);
                ask(j, f0 + j + kDepth, n0, b, b2);
                __builtin_amdgcn_sched_barrier(0);
            });
        static_for<0, kDepth - 1>([&](auto j) {
            if (f0 + j < steps) use(j, f0 + j);  // uniform
        });
    };
    auto bit = [](uint32_t v, int i) { return (uint32_t)((int32_t)(v << (31 - i)) >> 31); };  // all ones or zeros
    auto both = [](uint4 v, const uint32_t (&mask)[4]) { return make_uint4(v.x & mask[0], v.y & mask[1], v.z & mask[2], v.w & mask[3]); };
    auto clear = [](f32x16 &v) {
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = 0.0f;
    };
    if constexpr (ROWS) {
        static_for<0, FN>([&](auto piece) {
            constexpr int n = decltype(piece)::value;
            const int m0 = wcol0 + 32 * n, last = ((m0 + 32 < N ? m0 + 32 : N) - 1) / R;
            for (int b = m0 / R; b <= last; b += 2) {  // uniform
                const int block[2] = {b, b < last ? b + 1 : b};
                f32x16 sum[2];
                clear(sum[0]);
                clear(sum[1]);
                walk(n, block[0], block[1], [&](auto slot, int f) {
                    constexpr int s = decltype(slot)::value;
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const uint32_t mine = 16 * f + 8 * kh < M ? bits[s][j] >> (16 * (f & 1) + 8 * kh) : 0u;
                        uint32_t mask[4];
#pragma unroll
                        for (int i = 0; i < 4; ++i) mask[i] = (bit(mine, 2 * i) & 0xffffu) | (bit(mine, 2 * i + 1) & 0xffff0000u);
                        sum[j] = mfma32<DT>(w[s][0], both(x[s], mask), sum[j]);
                    }
                });
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const int end = blk_ptr[block[j] + 1];
                    const float pad = end - blk_ptr[block[j]] > blk_cnt[block[j]] ? 0.0f * elem<DT>::load(u, col_idx[end - 1]) : 0.0f;
#pragma unroll
                    for (int i = 0; i < 16; ++i)
                        if ((uint32_t)(m0 + 8 * (i >> 2) + 4 * kh + (i & 3) - block[j] * R) < (uint32_t)R) acc[n][i] = sum[j][i] + pad;
                }
            }
        });
    } else {
#pragma unroll
        for (int n = 0; n < FN; ++n) clear(acc[n]);
        walk(0, 0, 0, [&](auto slot, int f) {
            constexpr int s = decltype(slot)::value;
            const bool two = 16 * f + 8 < M;  // halves
            const bool split = !two || block_of(2 * f) != block_of(2 * f + 1);
            for (int h = 0; h < (split && two ? 2 : 1); ++h) {  // uniform
                const uint32_t own = !split || kh == h ? ~0u : 0u;
                const uint32_t mask[4] = {own, own, own, own};
                f32x16 p[FN];
#pragma unroll
                for (int n = 0; n < FN; ++n) {
                    clear(p[n]);
                    p[n] = mfma32<DT>(both(w[s][n], mask), both(x[s], mask), p[n]);
                }
#pragma unroll
                for (int n = 0; n < FN; ++n) {
                    const uint32_t mine = __builtin_amdgcn_readlane(bits[s][n], h) >> (4 * kh);
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[n][i] += __uint_as_float(__float_as_uint(p[n][i]) & bit(mine, 8 * (i >> 2) + (i & 3)));
                }
            }
        });
    }
}

// ---------------------------------------------------------------------------------------
// The product.  A workgroup of NW wavefronts owns 32 FT tokens x 32 NW FN columns and walks the rows in stages of 64.  U
// goes through LDS ([token][64], 128 bytes per row, 16-byte pieces rotated so that the operand reads meet all
// banks); the expanded weights are stored as operands and every wavefront has its own columns, so it loads them
// straight into registers: through LDS as well, a stage of the 128 x 256 tile would move 144 KiB through it in the
// 1024 clocks that its products take, more than the 128 bytes per clock it has.
// While stage s is multiplied, stage s + 2 of U is written to LDS, stage s + 4 requested, and the weights of stages
// s + 1 to s + 3 are on their way.  On the 4096 x 1024 matrix a stage takes 1490 clocks, 1024 of them with the matrix
// cores busy (57 us, 1.2 PFLOP/s of dense work); with the loads of a stage issued in a row it was 2020, with 2-way bank
// conflicts in the operand reads and the weights one stage ahead 2300.
// ---------------------------------------------------------------------------------------
// ROWS: the operands are Wp's rows (the layer), U is X and M, N are the layer's columns and rows.
// (the launch bounds: workgroups of a compute unit as the products' registers allow, whatever kept_sums would like)
template <int DT, int FT, int FN, bool ROWS, int NW>
__global__ __launch_bounds__(64 * NW, FN == 2 ? 1 : (FT == 4 ? 2 : 3)) void tile_kernel(
    const uint16_t *__restrict__ U, int64_t T, int32_t M, int32_t N, int32_t R, int32_t frags_m,
    const uint8_t *__restrict__ W, const uint32_t *__restrict__ kept, const int32_t *__restrict__ blk_cnt,
    const int32_t *__restrict__ blk_ptr, const int32_t *__restrict__ col_idx, const void *__restrict__ bias,
    void *__restrict__ Z) {
    constexpr int TT = 32 * FT, NN = 32 * NW * FN, kThreads = 64 * NW;
    constexpr int kUBytes = TT * kRowBytes;
    constexpr int kPitch = NN * 2 + 16;  // bytes of a token's row in the output tile
    constexpr int kPieces = 4 * FT / NW; // 16-byte pieces of U per thread and stage
    extern __shared__ __align__(16) uint8_t smem[];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, kh = lane >> 5;
    // Workgroup ids go round the 8 XCDs, each with an L2 of its own: id % 8 names the XCD, which owns the token tiles
    // of that remainder.  It walks them for kRangeGroup column ranges at a time: the 32 workgroups of 128 x 256 that
    // it runs at once then read 8 tiles of U and 4 ranges of the weights, the least there is to read.
    const uint32_t nranges = (uint32_t)(N + NN - 1) / NN, ntiles = ((uint32_t)((T + TT - 1) / TT) + 7u) / 8u;  // per XCD
    const uint32_t place = blockIdx.x >> 3;
    const uint32_t group = place / (ntiles * kRangeGroup), in_group = place - group * ntiles * kRangeGroup;
    const uint32_t width = nranges - group * kRangeGroup < kRangeGroup ? nranges - group * kRangeGroup : kRangeGroup;
    const int64_t t0 = (int64_t)((in_group / width) * 8u + (blockIdx.x & 7u)) * TT;
    if (t0 >= T) return;  // uniform: before any barrier
    const int cr0 = (int)(group * kRangeGroup + in_group % width) * NN;
    const int stages = frags_m / 4;

    f32x16 acc[FN][FT];
#pragma unroll
    for (int n = 0; n < FN; ++n)
#pragma unroll
        for (int t = 0; t < FT; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[n][t][i] = 0.0f;

    // as a loader of U: pieces tid % 8 of token rows tid / 8 + 8 NW i; a token past T reads the last one
    const uint8_t *utile = reinterpret_cast<const uint8_t *>(U + t0 * M);
    uint32_t urow[kPieces];
#pragma unroll
    for (int i = 0; i < kPieces; ++i) {
        const int row = (tid >> 3) + 8 * NW * i;
        urow[i] = (uint32_t)(t0 + row < T ? row : (int)(T - 1 - t0)) * 2u * (uint32_t)M;
    }
    const uint32_t st_u = (tid >> 3) * kRowBytes + (((tid & 7) ^ ((tid >> 4) & 7)) << 4);
    // as a consumer: lane l reads row l % 32 of a 32-row piece, 16-byte piece 2 kk + l / 32
    const uint32_t lane_cell = l32 * kRowBytes + ((kh ^ ((l32 >> 1) & 7)) << 4);
    const uint8_t *wcol = W + (int64_t)(cr0 / 32 + wave * FN) * frags_m * kFrag;  // uniform
    const uint32_t lane16 = lane * 16;

    // The bias of the tile's columns, a column per thread, asked for before the operands and handed round through LDS at the end.  (With
    // 2-byte loads where a sum is rounded, 16 FT FN of them per lane, 3072 x 768 at 3x, 8192 tokens took 67 us, 52 without a bias.)
    static_assert(NN <= kThreads);
    float column_bias = 0.0f;
    if (bias && tid < NN) column_bias = elem<DT>::load(bias, cr0 + tid < N ? cr0 + tid : N - 1);

    u32x4 ru[2][kPieces];      // U of two stages on its way to LDS
    uint4 wf[kRing][FN][4];    // weights of this stage and the next three
    uint4 uf[2][FT];           // U of this quarter of a stage and the next
    auto ask_u = [&](auto slot, auto piece, int stage) {
        constexpr int s = decltype(slot)::value, I = decltype(piece)::value;
        if constexpr (I < kPieces) {
            const int k = stage * kStageK + 8 * (tid & 7);
            const uint32_t kb = 2u * (uint32_t)(k < M - 8 ? k : M - 8);  // past the last row: any value, times zero
            ru[s & 1][I] = *reinterpret_cast<const u32x4 *>(utile + (urow[I] + kb));
        }
    };
    auto put_u = [&](auto slot, auto piece) {
        constexpr int s = decltype(slot)::value, I = decltype(piece)::value;
        if constexpr (I < kPieces) *reinterpret_cast<u32x4 *>(smem + st_u + s * kUBytes + I * 8 * NW * kRowBytes) = ru[s & 1][I];
    };
    auto ask_w = [&](auto slot, auto n, auto quarter, int stage) {
        constexpr int s = decltype(slot)::value, NI = decltype(n)::value, KK = decltype(quarter)::value;
        const int at = stage < stages ? stage : stages - 1;
        wf[s][NI][KK] = *reinterpret_cast<const uint4 *>(wcol + ((int64_t)NI * frags_m + 4 * at) * kFrag + (lane16 + KK * kFrag));
    };
    auto fetch = [&](auto slot, auto quarter, auto t) {
        constexpr int s = decltype(slot)::value, kk = decltype(quarter)::value, TI = decltype(t)::value;
        uf[kk & 1][TI] =
            *reinterpret_cast<const uint4 *>(smem + (lane_cell ^ (kk << 5)) + s * kUBytes + TI * 32 * kRowBytes);
    };
    // every LDS write of the wavefront is done and its reads have returned; its loads stay on their way
    auto stage_end = [] { asm volatile("s_waitcnt lgkmcnt(0)\n s_barrier" ::: "memory"); };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;

    static_for<0, 2>([&](auto j) { static_for<0, kPieces>([&](auto i) { ask_u(j, i, j); }); });
    static_for<0, 3>([&](auto s) {
        static_for<0, FN>([&](auto n) { static_for<0, 4>([&](auto kk) { ask_w(s, n, kk, s); }); });
    });
    static_for<0, kPieces>([&](auto i) { put_u(I0{}, i); ask_u(I0{}, i, 2); });
    static_for<0, kPieces>([&](auto i) { put_u(I1{}, i); ask_u(I1{}, i, 3); });
    stage_end();
    static_for<0, FT>([&](auto t) { fetch(I0{}, I0{}, t); });
    // A stage is four quarters of 16 rows.  Between the products of a quarter go the reads of the next quarter's U, the
    // loads of one quarter of the weights of stage s + 3, and a piece of U: stage s + 2 to LDS, stage s + 4 asked for.
    // One at a time: the four wavefronts run in step, and loads issued in a row wait for each other with the matrix
    // cores idle.  (Left to itself the compiler moves the reads behind the products and waits for them.)
    auto stage = [&](auto j, int s) {
        constexpr int J = decltype(j)::value;
        using S2 = std::integral_constant<int, (J + 2) % kRing>;
        using S3 = std::integral_constant<int, (J + 3) % kRing>;
        static_for<0, 4>([&](auto quarter) {
            constexpr int KK = decltype(quarter)::value;
            using NextQ = std::integral_constant<int, (KK + 1) % 4>;
            using NextS = std::integral_constant<int, (J + (KK + 1) / 4) % kRing>;
            constexpr int kProducts = FN * FT, kOthers = FT + FN + 2;
            static_for<0, kProducts>([&](auto i) {
                constexpr int I = decltype(i)::value, NI = I / FT, TI = I % FT;
                acc[NI][TI] = mfma32<DT>(wf[J][NI][KK], uf[KK & 1][TI], acc[NI][TI]);
                static_for<0, kOthers>([&](auto o) {
                    constexpr int O = decltype(o)::value;
                    if constexpr (O * kProducts / kOthers == I) {
                        if constexpr (O < FT) fetch(NextS{}, NextQ{}, o);
                        else if constexpr (O < FT + FN) ask_w(S3{}, std::integral_constant<int, O - FT>{}, quarter, s + 3);
                        else if constexpr (O == FT + FN) put_u(S2{}, quarter);
                        else ask_u(S2{}, quarter, s + 4);
                    }
                });
                __builtin_amdgcn_sched_barrier(0);
            });
        });
        stage_end();
    };
    // (whole rounds apart from the rest: a round with exits in its middle would make every wait of the loop a full one)
    int s0 = 0;
    for (; s0 + kRing <= stages; s0 += kRing) static_for<0, kRing>([&](auto j) { stage(j, s0 + j); });
    static_for<0, kRing - 1>([&](auto j) {
        if (stages % kRing > j) stage(j, s0 + j);  // uniform
    });
    __syncthreads();

    const int64_t left = T - t0;
    // Round into a token-major tile in LDS (the stages' memory), bias added in fp32, then write whole rows.
    uint8_t *tile = smem;
    uint32_t *flags = reinterpret_cast<uint32_t *>(smem + TT * kPitch);  // one bit per token: non-finite sums
    float *biases = reinterpret_cast<float *>(smem + TT * kPitch + 16);
    const int ncol = N - cr0 < NN ? N - cr0 : NN;
    const int wcol0 = cr0 + wave * FN * 32;  // the wavefront's first column
    if (tid < FT) flags[tid] = 0u;
    if (bias && tid < NN) biases[tid] = column_bias;
    __syncthreads();
    auto round_tokens = [&](int t, const f32x16 &v16, int n) {  // one piece of 32 tokens x 32 columns; NaN if a sum is not finite
        float bad = 0.0f;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int c = wcol0 + n * 32 + 8 * q + 4 * kh;  // four consecutive columns of one token
            float v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                v[i] = v16[4 * q + i];
                bad = __builtin_fmaf(v[i], 0.0f, bad);
            }
            if (bias) {  // uniform
                const f32x4 b = *reinterpret_cast<const f32x4 *>(biases + (c - cr0));
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] += b[i];
            }
            *reinterpret_cast<uint2 *>(tile + (32 * t + l32) * kPitch + (c - cr0) * 2) =
                make_uint2(cvt_pk<DT>(v[0], v[1]), cvt_pk<DT>(v[2], v[3]));
        }
        return bad;
    };
#pragma unroll
    for (int t = 0; t < FT; ++t) {
        float bad = 0.0f;
#pragma unroll
        for (int n = 0; n < FN; ++n) bad += round_tokens(t, acc[n][t], n);
        if (bad != 0.0f) atomicOr(&flags[t], 1u << l32);
    }
    __syncthreads();
    uint32_t any = 0;
#pragma unroll
    for (int t = 0; t < FT; ++t) any |= flags[t];
    any = __builtin_amdgcn_readfirstlane(any);
    for (int t = 0; t < (any && wcol0 < N ? FT : 0); ++t) {  // (uniform in a wavefront; no barrier inside)
        const uint32_t flagged = __builtin_amdgcn_readfirstlane(flags[t]);
        if (!flagged) continue;
        const int64_t row = 32 * t + l32 < left ? 32 * t + l32 : left - 1;
        f32x16 sums[FN];
        kept_sums<DT, FN, ROWS>(reinterpret_cast<const uint8_t *>(U + (t0 + row) * M), M, N, R, frags_m, wcol, wcol0, kept,
                                blk_cnt, blk_ptr, col_idx, sums);
        if ((flagged >> l32) & 1u)  // the others keep what they have
#pragma unroll
            for (int n = 0; n < FN; ++n) round_tokens(t, sums[n], n);
    }
    if (any) __syncthreads();
    uint16_t *z = (uint16_t *)Z + t0 * N + cr0;
    if ((N & 7) == 0 && (reinterpret_cast<uintptr_t>(Z) & 15) == 0) {
        for (int i = tid; i < TT * (NN / 8); i += kThreads) {
            const int tok = i / (NN / 8), c = (i % (NN / 8)) * 8;
            if (tok < left && c < ncol)
                *reinterpret_cast<uint4 *>(z + (int64_t)tok * N + c) = *reinterpret_cast<const uint4 *>(tile + tok * kPitch + c * 2);
        }
    } else {
        for (int i = tid; i < TT * NN; i += kThreads) {
            const int tok = i / NN, c = i % NN;
            if (tok < left && c < ncol)
                z[(int64_t)tok * N + c] = *reinterpret_cast<const uint16_t *>(tile + tok * kPitch + c * 2);
        }
    }
}

template <int FT, int FN, int NW>
constexpr size_t tile_lds() {
    constexpr size_t stages = (size_t)kRing * 32 * FT * kRowBytes;
    constexpr size_t out = (size_t)32 * FT * (32 * NW * FN * 2 + 16) + 16 + 4 * 32 * NW * FN;
    return stages > out ? stages : out;
}

// Which tile (where few_columns names no smaller one): 128 x 256 (ft 4, fn 2), 128 x 128 (4, 1) or 64 x 128 (2, 1).  The larger a tile, the more products a
// loaded operand serves, but one workgroup of the largest fills a compute unit, so what it cannot overlap shows: its
// start and end (9 us) and the idle units of the last round.  The estimates are microseconds fitted to what was
// measured at 512 to 8192 tokens of 768 to 4096 rows and columns: per stage 0.70, 0.46 (two on a unit together 1.03)
// and 0.36 (two 0.62, four 1.25).  For example (MI355X, with the expansion): 4096 x 1024, 8192 tokens 64 / 73 / 85;
// 1024 x 4096, 8192 tokens 84 / 76 / 95; 3072 x 768, 4096 tokens 42 / 31 / 36; 2304 x 768, 509 tokens 34 / 25 / 20.
struct Tile {
    int ft, fn;
};

// (count: workgroups per compute unit)
double tile_us(const Tile &c, double count, double stages) {
    if (c.fn == 2) return __builtin_ceil(count) * (0.70 * stages + 9.0);
    if (c.ft == 4) return (count <= 1.0 ? 0.46 : 0.515 * (count < 1.8 ? 1.8 : count)) * stages + 7.0;
    return (count <= 1.0 ? 0.36 : 0.31 * (count < 2.0 ? 2.0 : count)) * stages + 6.0;
}

// us: the estimate; us_xcd: what it is with the token tiles on one XCD each, as the launch places them (less than 8
// leave XCDs without work).
Tile choose_tile(int64_t T, int64_t M, int64_t N, double *us = nullptr, double *us_xcd = nullptr) {
    const double stages = (double)((M + kStageK - 1) / kStageK);
    constexpr Tile shapes[] = {{4, 2}, {4, 1}, {2, 1}};
    Tile best = shapes[0];
    double best_us = 0.0;
    for (const Tile &c : shapes) {
        const int64_t tiles = (T + 32 * c.ft - 1) / (32 * c.ft), ranges = (N + 128 * c.fn - 1) / (128 * c.fn);
        const double t = tile_us(c, (double)tiles * (double)ranges / 256.0, stages);
        if (best_us != 0.0 && t >= best_us) continue;
        best = c;
        best_us = t;
        if (us_xcd) *us_xcd = tile_us(c, (double)((tiles + 7) / 8 * 8) * (double)ranges / 256.0, stages);
    }
    if (us) *us = best_us;
    return best;
}

// Columns of a workgroup of 32 tokens, where such a small tile is the faster one, else 0.  What bounds a stage of the tiles
// above in a launch of few workgroups is neither a load's nor an LDS read's latency (with twice the stages on their way, or the
// reads a whole stage ahead, it takes as long) but what a compute unit loads, 33 to 40 bytes per clock whatever the tile: 24 KB
// of 64 x 128 0.28 us, and 240 workgroups take as long as 6.  32 tokens x 64 columns are 12 KB and 0.2 us, 32 x 128 20 KB, on up
// to four times the compute units.  They stop paying where an XCD (token tiles go round the 8 of them) has more than its 32
// compute units' worth of workgroups, and for wide layers, whose matrix then crosses to more XCDs than the larger tiles
// need.  Measured with the expansion, us, 64 x 128 or the larger / 32 x 128 / 32 x 64: 2304 x 768, 509 tokens 19.3 / 17.7 / 15.7, 800 tokens
// 19.4 / 17.9 / 18.7, 1537 tokens 19.3 / 21.8 / 22.0; 4096 x 1024, 64 tokens 24.4 / 22.9 / 19.8, 1024 tokens 27.0 / 25.8 / 27.1; 1024 x 2048, 254
// tokens 15.4 / 16.6 / 16.1 (stays).  Over 150 drawn calls of 8 to 4096 tokens (about two thirds of them taken) the mean is 0.925 of the time.
int few_columns(int64_t T, int64_t N) {
    const int64_t per_xcd = (T + 255) / 256;  // token tiles
    if (N <= 1536 && per_xcd * ((N + 63) / 64) <= 32) return 64;
    return N <= 1280 && per_xcd * ((N + 127) / 128) <= 32 ? 128 : 0;
}

// The expanded matrix (N columns, M rows); behind it one bit per row-block and column of the pruned matrix.
size_t expanded_bytes(int64_t M, int64_t N) {
    return (size_t)((N + kColPad - 1) / kColPad * kColPad) * (size_t)((M + kStageK - 1) / kStageK * kStageK) * 2;
}
size_t kept_bytes(int64_t B, int64_t cols) { return (size_t)B * (size_t)((cols + kColPad - 1) / kColPad) * (kColPad / 8); }

struct Args {
    const uint16_t *U;
    int64_t T;
    int32_t M, N, B, R;
    const int32_t *blk_cnt, *blk_ptr, *col_idx;
    const uint16_t *vals;
    const void *bias;
    void *Z, *ws;
    hipStream_t s;
};

uint32_t *kept_bits(const Args &a) { return (uint32_t *)((uint8_t *)a.ws + expanded_bytes(a.M, a.N)); }

template <int DT, int FT, int FN, bool ROWS, int NW = 4>
int launch_tiles(const Args &a, int frags_m) {
    constexpr size_t lds = tile_lds<FT, FN, NW>();
    auto k = tile_kernel<DT, FT, FN, ROWS, NW>;
    if (lds > 65536) {  // (asking again is harmless)
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) {
            set_last_hip_error((int)e);
            return BSP_ERR_HIP;
        }
    }
    const int64_t tiles = (a.T + 32 * FT - 1) / (32 * FT), ranges = (a.N + 32 * NW * FN - 1) / (32 * NW * FN);
    const int64_t wgs = (tiles + 7) / 8 * 8 * ranges;  // whole rounds of the 8 XCDs
    if (wgs >= ((int64_t)1 << 31)) return BSP_ERR_SHAPE;
    k<<<dim3((unsigned)wgs), 64 * NW, lds, a.s>>>(a.U, a.T, a.M, a.N, a.R, frags_m, (const uint8_t *)a.ws, kept_bits(a), a.blk_cnt,
                                                    a.blk_ptr, a.col_idx, a.bias, a.Z);
    return BSP_OK;
}

template <int DT, bool ROWS>
int launch_all(const Args &a) {
    const Tile c = choose_tile(a.T, a.M, a.N);
    const int npad = (a.N + kColPad - 1) / kColPad * kColPad, frags_m = (a.M + kStageK - 1) / kStageK * 4;
    uint64_t *kept = (uint64_t *)kept_bits(a);
    if constexpr (ROWS)
        expand_rows_kernel<<<dim3((unsigned)((npad + a.R - 1) / a.R), (unsigned)((a.M + kColPad - 1) / kColPad), (unsigned)((a.R + 15) / 16)), kThreadsX, 0, a.s>>>(
            a.R, a.B, npad, frags_m, a.blk_cnt, a.blk_ptr, a.col_idx, a.vals, (uint8_t *)a.ws, kept);
    else
        expand_kernel<<<dim3((unsigned)a.B, (unsigned)(npad / kColPad), (unsigned)((a.R + 15) / 16)), kThreadsX, 0, a.s>>>(
            a.R, a.B, frags_m, a.blk_cnt, a.blk_ptr, a.col_idx, a.vals, (uint8_t *)a.ws, kept);
    const int few = few_columns(a.T, a.N);
    if (few == 64) return launch_tiles<DT, 1, 1, ROWS, 2>(a, frags_m);
    if (few == 128) return launch_tiles<DT, 1, 1, ROWS, 4>(a, frags_m);
    if (c.ft == 2) return launch_tiles<DT, 2, 1, ROWS>(a, frags_m);
    return c.fn == 2 ? launch_tiles<DT, 4, 2, ROWS>(a, frags_m) : launch_tiles<DT, 4, 1, ROWS>(a, frags_m);
}

}  // namespace

// (a tile's rows of U are addressed with 32-bit byte offsets; the expansion's grid has a row per 256 columns)
bool linear_t_expand_supported(int udt, int64_t M, int64_t N, int32_t R) {
    return udt != BSP_F32 && R % 8 == 0 && M < ((int64_t)1 << 23) && N <= 65535 * (int64_t)kColPad;
}

size_t linear_t_expand_bytes(int64_t M, int64_t N, int32_t R) { return expanded_bytes(M, N) + kept_bytes(M / R, N); }

int linear_t_expand(const void *U, int udt, int64_t T, int64_t M, int64_t N, int32_t R, const int32_t *blk_cnt,
                    const int32_t *blk_ptr, const int32_t *col_idx, const void *vals, const void *bias, void *Z,
                    void *ws, hipStream_t s) {
    const Args a = {(const uint16_t *)U, T, (int32_t)M, (int32_t)N, (int32_t)(M / R), R, blk_cnt, blk_ptr, col_idx,
                    (const uint16_t *)vals, bias, Z, ws, s};
    return udt == BSP_BF16 ? launch_all<BSP_BF16, false>(a) : launch_all<BSP_F16, false>(a);
}

size_t linear_expand_bytes(int64_t M, int64_t N, int32_t R) { return expanded_bytes(N, M) + kept_bytes(M / R, N); }

// Whether a layer on its compact storage is the shorter one as an expansion and a dense product: microseconds of both forms, fitted to 59000
// calls with a bias, each on inputs and results that were in no cache, of 256 to 60000 rows, 64 to 4096 columns, R = 1 to 64, 1 to 65536
// tokens, 1.1x to 8x; half of them 768 / 3072-like matrices at 1.43x to 5x, a third of the token counts powers of two and their like (the dense
// one to 4 to 8 % on average, the gather's to 6 to 9, 15 for more than 32 rows).  Measured, gather / dense: 1024 x 4096, R = 16 at
// 5x, 8192 tokens 125 / 71, 2048 tokens 41.3 / 37.8 (stays); 3072 x 768 at 3x, 8192 tokens 53 / 55, 4096 tokens 31 / 37; 768 x 768 at 3x,
// 8192 tokens 18.7 / 25.0; 896 x 896, R = 8 at 2x, 1752 tokens 24 / 14.
// The gather goes in whole rounds: its workgroups, a token tile and a strip of row-blocks each, fill compute units, so 8192 tokens
// of a narrow layer are one full round and 8200 are two.  An estimate by the mean (and an older one beside it that could say
// dense by itself) made 9 % of the calls of 8192 tokens more than 8 % slower than by the gather, 0.75 % of all, and beyond 8192 tokens it
// was asked for nothing, at 1.2 times the time.  Dense has to be the shorter one by 12 %: of 30000 calls that the fit has
// not seen 0.12 % are slower by more than 8 % (0.3 % at 8192 tokens; 1.26 times at worst), the loss against the faster
// form is 2 % of the time (6.5 % before), and the mean 0.80 of the gather alone.  A call of two launches and a workspace takes 10 us on the
// host, so nothing shorter is asked to be dense.  (The dense form rounds its sum once per 16 columns, the gather once per 32 kept ones; the result's
// 16 bits hide both: against 64 bits 1024 x 4096 at 5x in fp16 2.06919e-4 and 2.06919e-4, the rounding of the result alone 2.06919e-4.)
bool linear_expand_pays(int64_t T, int64_t M, int64_t N, int32_t R, int64_t capacity_cols) {
    const int64_t npad = (N + 255) / 256 * 256, tok = npad <= 1024 ? 64 : (npad <= 2048 ? 32 : 16), B = M / R;
    const double blocks = (double)B, all = blocks * (double)(N + 31);
    const double cols = (double)capacity_cols < all ? (double)capacity_cols : all, out = (double)T * (double)M * 1e-6;

    const int few = few_columns(T, M);
    const double workgroups = (double)((M + 255) / 256 * 256 / R) * (double)(npad / 256) * (double)((R + 15) / 16), MN = (double)M * (double)N;
    const double stages = (double)((N + kStageK - 1) / kStageK);
    double dense;
    if (few == 64) {
        dense = 7.83 + 0.150 * stages + 0.00070 * workgroups + 1.70e-6 * MN + 0.827 * out + 10.0e-6 * cols;
    } else if (few == 128) {
        dense = 7.61 + 0.233 * stages + 0.00077 * workgroups + 1.49e-6 * MN + 0.580 * out + 10.0e-6 * cols;
    } else {
        double tiles, tiles_xcd;
        choose_tile(T, N, M, &tiles, &tiles_xcd);
        const double idle = tiles_xcd > tiles ? tiles_xcd - tiles : 0.0;
        dense = 2.06 + 1.02 * tiles + 0.760 * idle + 0.00105 * workgroups + 0.956e-6 * MN + 0.460 * out + 12.6e-6 * cols;
    }

    // the call, a step of 32 kept columns of the workgroup that a compute unit is busy with, a step of a row-block (which one wavefront
    // walks), a round's 1000 columns, a million outputs; by the tile of X (64, 32, 16 tokens) and the rows of a row-block (to 16, 32, 64)
    constexpr double kGather[3][3][5] = {
        {{6.00, 0.0344, 0.198, 2.17, 0.941}, {6.13, 0.0505, 0.310, 2.32, 0.890}, {9.50, 0.431, 0.647, 4.33, 2.58}},
        {{2.67, 0.0269, 0.257, 2.67, 1.10}, {3.00, 0.0428, 0.293, 2.63, 0.938}, {0.0, 0.140, 0.813, 6.50, 2.48}},
        {{0.57, 0.0229, 0.278, 1.77, 2.30}, {2.88, 0.0435, 0.291, 1.22, 1.27}, {0.0, 0.124, 0.636, 3.27, 2.29}}};
    const double *k = kGather[tok == 64 ? 0 : (tok == 32 ? 1 : 2)][R <= 16 ? 0 : (R <= 32 ? 1 : 2)];
    const int64_t ntiles = (T + tok - 1) / tok, strip = canonical_strip(ntiles, B), wgs = ntiles * ((B + strip - 1) / strip);
    const int64_t together = 2 * npad * tok * 2 <= 156 * 1024 ? 2 : 1;  // workgroups that share a compute unit
    const double gather = k[0] + k[1] * (double)((wgs + 255) / 256) * cols / 32.0 * (double)strip / blocks + k[2] * cols / blocks / 32.0 +
                          k[3] * (double)((wgs + 256 * together - 1) / (256 * together)) * 1e-3 * (double)N + k[4] * out;
    return (dense < 10.0 ? 10.0 : dense) < 0.88 * gather;
}

int linear_expand(const void *X, int xdt, int64_t T, int64_t M, int64_t N, int32_t R, const int32_t *blk_cnt,
                  const int32_t *blk_ptr, const int32_t *col_idx, const void *vals, const void *bias, void *Y, void *ws,
                  hipStream_t s) {
    const Args a = {(const uint16_t *)X, T, (int32_t)N, (int32_t)M, (int32_t)(M / R), R, blk_cnt, blk_ptr, col_idx,
                    (const uint16_t *)vals, bias, Y, ws, s};
    return xdt == BSP_BF16 ? launch_all<BSP_BF16, true>(a) : launch_all<BSP_F16, true>(a);
}

}  // namespace bsp
