// The gradient of the layer's kept weights (see bsp_linear_dvals.hip) as a dense product dY^T X of which only the kept positions
// are written; bf16 / fp16, R % 8 == 0, N % 8 == 0.
//
// Why dense: the sparse form reads one kibibyte of LDS per 16 x 16 x 32 product and its partial sums fill the registers of
// the chip, so its start and its end take 20 us whatever the batch; a dense tile reads a sixth of that per product and its sums
// leave it by their kept positions alone, with few runs of the tokens (often one: no second pass).  At 1 / density times the
// products it is the faster one except where a large layer keeps little of many tokens (dvals_dense_pays).  Measured (MI355X, us, the whole
// call with its list, fp32 result, the sparse form / this one): 2304 x 768, R = 8 at 2x, 509 tokens 25.5 / 8.0; 4096 x 1024, R = 32 at 1.43x, 4099 tokens 78.9 / 43.8;
// R = 16 at 5x, 4096 tokens 39.0 / 38.6, 8192 tokens 58.2 / 64.8 (stays sparse).
//
// A workgroup owns BM rows of dY^T x BN columns of X and a run of the tokens, 32 tokens a stage, four stages in LDS.  Both
// operands are read from memory as they lie, [token][columns], straight into LDS, and the transposing LDS reads give a lane
// 4 + 4 tokens of its own column; a row's 64-byte pieces change places with the token so that these reads meet all banks.
// While stage s is multiplied, stage s + 1 is in LDS, stage s + 2 on its way and stage s + 3 asked for; the operands of the first half
// of a stage are read while the second half of the one before it is multiplied, so only the barrier is waited for.
#include "bsp_common.h"
#include "bsp_linear_internal.h"
#include "bsp_mfma_device.h"

namespace bsp {
namespace {

constexpr int kDdTok = 32;      // tokens of a stage
constexpr int kDdStages = 4;    // stages in LDS
constexpr int kDdPassPitch = 4; // floats that a row of the output tile is longer than its columns

// What is exclusive-ored onto the column's byte offset in a token's row of PITCH bytes: four tokens' pieces of 64 bytes (what
// half a transposing read takes) lie in 256 different bytes of the banks.
template <int PITCH>
__device__ __forceinline__ uint32_t dd_turn(uint32_t token) {
    return PITCH >= 256 ? (token & 3u) << 6 : ((token >> 1) & 1u) << 6;
}

// 64 lanes' 16 bytes at base + at to LDS at lds .. lds + 1023.  (Written out: for the builtin the compiler would wait for all such
// loads before any LDS read.  m0 is a reserved register, which can't be named as clobbered; nothing else in these kernels uses it.)
__device__ __forceinline__ void load_to_lds(uint32_t lds, const uint8_t *base, uint32_t at) {
    asm volatile("s_mov_b32 m0, %0\n s_nop 0\n global_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(at), "s"(base));
}
// The same at lds + PLUS.
template <int PLUS>
__device__ __forceinline__ void load_to_lds_at(uint32_t lds, const uint8_t *base, uint32_t at) {
    asm volatile("s_add_u32 m0, %0, %3\n s_nop 0\n global_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(at), "s"(base), "n"(PLUS) : "scc");
}
template <int LEFT>
__device__ __forceinline__ void wait_loads() {  // until LEFT loads are on their way
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LEFT) : "memory");
}
__device__ __forceinline__ void barrier() { asm volatile("s_barrier" ::: "memory"); }

template <int DT, int FM, int FN, int WR, int WC>
struct DdShape {
    static constexpr int kWaves = WR * WC;
    static constexpr int BM = 32 * FM * WR, BN = 32 * FN * WC;
    static constexpr int PY = 2 * BM, PX = 2 * BN;                   // bytes of a token's row
    static constexpr int kYBytes = kDdTok * PY, kStage = kYBytes + kDdTok * PX;
    static constexpr int NY = kYBytes / 1024 / kWaves, NX = kDdTok * PX / 1024 / kWaves;  // loads of a wavefront and stage
    static constexpr int kRows = 32 * WR;                            // rows of a pass of the output
    static constexpr int kPitch = BN + kDdPassPitch;
    static constexpr size_t kOut = (size_t)kRows * kPitch * 4;
    static constexpr size_t kLds = (size_t)kDdStages * kStage > kOut ? (size_t)kDdStages * kStage : kOut;
    static_assert(NY * kWaves * 1024 == kYBytes && NX * kWaves * 1024 == kDdTok * PX && BN % 128 == 0);
};

// ODT: the type that is written, fp32 for runs' sums that dvals_sum_kernel adds.  TOTALS: chains shorter than the run, which takes a second
// set of registers.
template <int DT, int ODT, int FM, int FN, int WR, int WC, bool TOTALS>
// (the launch bounds: with totals as many registers as two or three workgroups on a compute unit leave; with more of them the sums would
// lie in accumulation registers, three instructions away from an addition)
__global__ __launch_bounds__(WR *WC * 64, !TOTALS ? 1 : (FM == 1 ? 3 : 2)) void dvals_dense_kernel(
    const uint16_t *__restrict__ X, const uint16_t *__restrict__ dY, int64_t T, int32_t M, int32_t N, int32_t R,
    const int32_t *__restrict__ blk_cnt, const int32_t *__restrict__ blk_ptr, const int32_t *__restrict__ col_idx,
    const int32_t *__restrict__ colstart, int32_t max_col, int32_t per, int32_t S, int32_t chain, int64_t stride,
    void *__restrict__ sums) {
    using G = DdShape<DT, FM, FN, WR, WC>;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave / WC, wc = wave % WC;
    // Workgroup ids go round the 8 XCDs, each with an L2 of its own: an XCD's units are consecutive, tiles of one run of tokens.
    const int tn = (N + G::BN - 1) / G::BN, tiles = (M + G::BM - 1) / G::BM * tn, units = tiles * S, per_xcd = (units + 7) / 8;
    const int unit = (int)(blockIdx.x & 7u) * per_xcd + (int)(blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per_xcd || unit >= units) return;  // (whole workgroups, before any barrier)
    const int tile = unit % tiles, s0 = unit / tiles;
    const int m0 = tile / tn * G::BM, n0 = tile % tn * G::BN;
    const int nstages = (int)((T + kDdTok - 1) / kDdTok);
    const int first = s0 * per, n = (first + per < nstages ? first + per : nstages) - first;  // the unit's stages
    const int left = (int)(T - (int64_t)(first + n - 1) * kDdTok);  // tokens of its last one
    const int ragged = left < kDdTok ? n - 1 : -1;                    // (only the batch's last)

    // as a loader: wavefront w brings kibibytes w, w + kWaves, ... of a stage's rows of dY, then of X.  Columns past the
    // matrix are read from its last eight instead; tokens past the batch from its last one, and zeroed in LDS below.
    uint32_t yat[G::NY], xat[G::NX];
    auto places = [&](int last) {
#pragma unroll
        for (int i = 0; i < G::NY; ++i) {
            const uint32_t o = (uint32_t)(wave + G::kWaves * i) * 1024u + (uint32_t)lane * 16u, t = o / G::PY;
            const uint32_t c = ((o % G::PY) ^ dd_turn<G::PY>(t)) / 2;
            yat[i] = 2u * (min(t, (uint32_t)last) * (uint32_t)M + min((uint32_t)m0 + c, (uint32_t)M - 8u));
        }
#pragma unroll
        for (int i = 0; i < G::NX; ++i) {
            const uint32_t o = (uint32_t)(wave + G::kWaves * i) * 1024u + (uint32_t)lane * 16u, t = o / G::PX;
            const uint32_t c = ((o % G::PX) ^ dd_turn<G::PX>(t)) / 2;
            xat[i] = 2u * (min(t, (uint32_t)last) * (uint32_t)N + min((uint32_t)n0 + c, (uint32_t)N - 8u));
        }
    };
    auto stage_at = [&](int s) { return (uint32_t)(s & (kDdStages - 1)) * (uint32_t)G::kStage; };
    auto ask_y = [&](auto i, int s) {
        constexpr int I = decltype(i)::value;
        load_to_lds(stage_at(s) + (uint32_t)(wave + G::kWaves * I) * 1024u,
                    reinterpret_cast<const uint8_t *>(dY + (int64_t)(first + s) * kDdTok * M), yat[I]);
    };
    auto ask_x = [&](auto i, int s) {
        constexpr int I = decltype(i)::value;
        load_to_lds(stage_at(s) + (uint32_t)G::kYBytes + (uint32_t)(wave + G::kWaves * I) * 1024u,
                    reinterpret_cast<const uint8_t *>(X + (int64_t)(first + s) * kDdTok * N), xat[I]);
    };
    auto ask = [&](auto i, int s) {
        if constexpr (decltype(i)::value < G::NY) ask_y(i, s);
        else ask_x(std::integral_constant<int, decltype(i)::value - G::NY>{}, s);
    };
    constexpr int NL = G::NY + G::NX;
    auto zero_rows = [&](int s) {  // tokens past the batch in stage s (which has landed)
        uint8_t *st = smem_x + stage_at(s);
        for (int i = tid; i < (kDdTok - left) * (G::PY / 16); i += G::kWaves * 64)
            *reinterpret_cast<uint4 *>(st + left * G::PY + i * 16) = make_uint4(0u, 0u, 0u, 0u);
        for (int i = tid; i < (kDdTok - left) * (G::PX / 16); i += G::kWaves * 64)
            *reinterpret_cast<uint4 *>(st + G::kYBytes + left * G::PX + i * 16) = make_uint4(0u, 0u, 0u, 0u);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        barrier();
    };

    places(kDdTok - 1);
    for (int s = 0; s < 3 && s < n; ++s) {
        if (s == ragged) places(left - 1);
        static_for<0, NL>([&](auto i) { ask(i, s); });
    }

    // The output: a pass writes 32 rows of every row of wavefronts through LDS, and a wavefront then takes groups of 8 rows of it,
    // which belong to one row-block (R % 8 == 0).  What it needs to know of them is asked for now.
    constexpr int kGroups = G::kRows / 8 / G::kWaves, kCols = G::BN / 64;
    int gbase[FM][kGroups], gkp[FM][kGroups], gk[FM][kGroups], glo[FM][kGroups], gend[FM][kGroups];
    uint32_t gcol[FM][kGroups][kCols];
    const int tables = (N + 127) / 128 + 1;  // entries of a row of colstart
    auto group_row = [&](int f, int g) {  // first row of group g of the wavefront in pass f
        const int rr = 8 * (wave + G::kWaves * g);
        return m0 + rr / 32 * (32 * FM) + 32 * f + rr % 32;
    };
    // (each kind for all groups before the next kind, and without tests: a load behind a test is waited for before the next)
    static_for<0, FM * kGroups>([&](auto i) {
        constexpr int f = decltype(i)::value / kGroups, g = decltype(i)::value % kGroups;
        const int b = min(group_row(f, g), M - 8) / R;
        gbase[f][g] = blk_ptr[b];
        gkp[f][g] = blk_ptr[b + 1];
        gk[f][g] = blk_cnt[b];
        const int32_t *cs = colstart + (int64_t)b * tables;
        glo[f][g] = cs[n0 / 128];
        gend[f][g] = cs[min((n0 + G::BN) / 128, tables - 1)];
    });
    __builtin_amdgcn_sched_barrier(0);
    static_for<0, FM * kGroups>([&](auto i) {
        constexpr int f = decltype(i)::value / kGroups, g = decltype(i)::value % kGroups;
        gkp[f][g] -= gbase[f][g];
        if (n0 + G::BN >= N) gend[f][g] = gkp[f][g];  // (the last columns' tile writes the pads, too)
        // (kept inside the row-block's panel whatever the workspace holds)
        glo[f][g] = min(max(glo[f][g], 0), gkp[f][g]);
        gend[f][g] = min(max(gend[f][g], glo[f][g]), gkp[f][g]);
#pragma unroll
        for (int e = 0; e < kCols; ++e) {
            const int c = gbase[f][g] + min(glo[f][g] + lane + 64 * e, gend[f][g] - 1);
            gcol[f][g][e] = (uint32_t)col_idx[min(max(c, 0), max_col)];
        }
    });

    // as a reader: lane l's column of a 32-column operand is l % 32, its tokens 8 (l / 32) .. + 7 of the 16
    const uint32_t tok = 8u * (uint32_t)(lane >> 5) + (uint32_t)((lane >> 2) & 3), piece = (uint32_t)((lane >> 4) & 1) * 32u + (uint32_t)(lane & 3) * 8u;
    uint32_t ya[FM], xa[FN];
#pragma unroll
    for (int f = 0; f < FM; ++f) ya[f] = tok * G::PY + ((64u * (uint32_t)(wr * FM + f) + piece) ^ dd_turn<G::PY>(tok));
#pragma unroll
    for (int f = 0; f < FN; ++f) xa[f] = G::kYBytes + tok * G::PX + ((64u * (uint32_t)(wc * FN + f) + piece) ^ dd_turn<G::PX>(tok));
    // the stages of a round of four lie at constants from these (LDS offsets reach 64 KiB)
    constexpr bool kTwoBases = (kDdStages - 1) * G::kStage >= 65536;
    uint32_t yb[2][FM], xb[2][FN];
#pragma unroll
    for (int f = 0; f < FM; ++f) yb[0][f] = ya[f], yb[1][f] = ya[f] + 65536u;
#pragma unroll
    for (int f = 0; f < FN; ++f) xb[0][f] = xa[f], xb[1][f] = xa[f] + 65536u;
    if constexpr (kTwoBases) {  // (kept in registers, not added up again at every read)
#pragma unroll
        for (int f = 0; f < FM; ++f) asm volatile("" : "+v"(yb[1][f]));
#pragma unroll
        for (int f = 0; f < FN; ++f) asm volatile("" : "+v"(xb[1][f]));
    }
    uint4 yf[2][FM], xf[2][FN];
    auto read = [&](auto half, auto which, uint32_t at) {
        constexpr int H = decltype(half)::value, I = decltype(which)::value;
        constexpr int P = I < FN ? G::PX : G::PY;
        const uint2 lo = tr_read_at(at + 16 * H * P), hi = tr_read_at(at + 16 * H * P + 4 * P);
        if constexpr (I < FN) xf[H][I] = make_uint4(lo.x, lo.y, hi.x, hi.y);
        else yf[H][I - FN] = make_uint4(lo.x, lo.y, hi.x, hi.y);
    };
    auto fetch = [&](auto half, auto which, uint32_t st) {  // operand `which` of the 16 tokens of that half
        constexpr int I = decltype(which)::value;
        if constexpr (I < FN) read(half, which, st + xa[I]);
        else read(half, which, st + ya[I - FN]);
    };
    auto fetch_at = [&](auto half, auto which, auto slot) {  // of the stage in that slot
        constexpr int I = decltype(which)::value, kAt = decltype(slot)::value * G::kStage, kHi = kAt >= 65536 ? 1 : 0;
        if constexpr (I < FN) read(half, which, xb[kHi][I] + (kAt - 65536 * kHi));
        else read(half, which, yb[kHi][I - FN] + (kAt - 65536 * kHi));
    };
    f32x16 acc[FM][FN];
#pragma unroll
    for (int f = 0; f < FM; ++f)
#pragma unroll
        for (int g = 0; g < FN; ++g)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[f][g][i] = 0.0f;
    // What a chain of matrix instructions has added up goes to the totals when the next chain begins: see sums_chain below.
    f32x16 total[TOTALS ? FM : 1][TOTALS ? FN : 1];
    int chain_left = chain;
    if constexpr (TOTALS) {
#pragma unroll
        for (int f = 0; f < FM; ++f)
#pragma unroll
            for (int g = 0; g < FN; ++g) total[f][g] = acc[f][g];
    }

    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    if (n > 2) wait_loads<NL>();
    else wait_loads<0>();
    barrier();
    if (ragged == 0) zero_rows(0);
    static_for<0, FM + FN>([&](auto i) { fetch(I0{}, i, 0u); });
    // Between the products of a half go the reads of the next half's operands, and between the first half's the loads.
    auto products = [&](auto half, auto fetch_next, auto load) {
        constexpr int H = decltype(half)::value;
        constexpr int kProducts = FM * FN, kReads = FM + FN;
        if constexpr (TOTALS && H == 0) {
            if (chain_left == 0) {  // uniform
                chain_left = chain;
                static_for<0, kProducts>([&](auto p) {
                    constexpr int f = decltype(p)::value / FN, g = decltype(p)::value % FN;
                    total[f][g] += acc[f][g];
                    acc[f][g] = f32x16{};
                });
            }
            --chain_left;
        }
        static_for<0, kProducts>([&](auto p) {
            constexpr int P = decltype(p)::value;
            acc[P / FN][P % FN] = mfma32<DT>(xf[H][P % FN], yf[H][P / FN], acc[P / FN][P % FN]);
            static_for<0, kReads>([&](auto i) {
                if constexpr (decltype(i)::value * kProducts / kReads == P) fetch_next(i);
            });
            if constexpr (H == 0) {
                static_for<0, NL>([&](auto i) {
                    if constexpr (decltype(i)::value * kProducts / NL == P) load(i);
                });
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    int s = 0;
    {   // rounds of four stages that end before the last one is asked for: addresses are constants from a register
        const uint8_t *ynext = reinterpret_cast<const uint8_t *>(dY + (int64_t)(first + 3) * kDdTok * M);
        const uint8_t *xnext = reinterpret_cast<const uint8_t *>(X + (int64_t)(first + 3) * kDdTok * N);
        const uint32_t mine = (uint32_t)wave * 1024u;
        for (; s + 7 < n; s += 4)
            static_for<0, 4>([&](auto slot) {
                constexpr int J = decltype(slot)::value;
                products(I0{}, [&](auto i) { fetch_at(I1{}, i, slot); }, [&](auto i) {
                    constexpr int I = decltype(i)::value, kAt = (J + 3) % 4 * G::kStage;
                    if constexpr (I < G::NY) load_to_lds_at<kAt + I * G::kWaves * 1024>(mine, ynext, yat[I]);
                    else load_to_lds_at<kAt + G::kYBytes + (I - G::NY) * G::kWaves * 1024>(mine, xnext, xat[I - G::NY]);
                });
                ynext += (int64_t)(2 * kDdTok) * M;
                xnext += (int64_t)(2 * kDdTok) * N;
                products(I1{}, [&](auto i) { fetch_at(I0{}, i, std::integral_constant<int, (J + 1) % 4>{}); }, [&](auto) {});
                wait_loads<NL>();
                barrier();  // stage s + 2 is there for all, stage s has been read by all
            });
    }
    for (; s < n; ++s) {
        if (s + 1 == ragged) zero_rows(s + 1);
        const bool more = s + 3 < n;
        if (more && s + 3 == ragged) places(left - 1);
        products(I0{}, [&](auto i) { fetch(I1{}, i, stage_at(s)); }, [&](auto i) {
            if (more) ask(i, s + 3);  // uniform
        });
        products(I1{}, [&](auto i) { fetch(I0{}, i, stage_at(s + 1)); }, [&](auto) {});
        if (more) wait_loads<NL>();
        else wait_loads<0>();
        barrier();
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    barrier();  // (the last reads, of a stage past the end, are over before the tile's memory is used again)

    float *out = reinterpret_cast<float *>(smem_x);
    using Out = typename elem<ODT>::type;
    Out *to = (Out *)sums + (int64_t)s0 * stride;
    static_for<0, FM>([&](auto pass) {
        constexpr int f = decltype(pass)::value;
        if (f > 0) __syncthreads();
#pragma unroll
        for (int g = 0; g < FN; ++g)
#pragma unroll
            for (int q = 0; q < 4; ++q) {  // four consecutive columns of one row
                f32x16 v = acc[f][g];
                if constexpr (TOTALS) v += total[f][g];
                *reinterpret_cast<f32x4 *>(out + (32 * wr + (lane & 31)) * G::kPitch + 32 * (wc * FN + g) + 8 * q + 4 * (lane >> 5)) =
                    f32x4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
            }
        __syncthreads();
#pragma unroll
        for (int g = 0; g < kGroups; ++g) {
            const int m = group_row(f, g);
            if (m >= M) continue;  // uniform
            const float *row = out + 8 * (wave + G::kWaves * g) * G::kPitch;
            Out *at = to + (int64_t)R * gbase[f][g] + (int64_t)(m % R) * gkp[f][g];
            // (the kept columns of BN fit kCols rounds; the pads behind the last of them, fewer than 64, take another)
#pragma unroll
            for (int i = 0; i <= kCols; ++i) {
                const int c = glo[f][g] + lane + 64 * i;
                if (glo[f][g] + 64 * i >= gend[f][g]) break;  // uniform
                const uint32_t j = i < kCols ? min(gcol[f][g][i < kCols ? i : 0] - (uint32_t)n0, (uint32_t)G::BN - 1u) : 0u;
                float v[8];
#pragma unroll
                for (int r = 0; r < 8; ++r) v[r] = row[r * G::kPitch + j];
                if (c >= gend[f][g]) continue;
                const bool kept = i < kCols && c < gk[f][g];
#pragma unroll
                for (int r = 0; r < 8; ++r) elem<ODT>::store(at, (int64_t)r * gkp[f][g] + c, kept ? v[r] : 0.0f);
            }
        }
    });
}

// The runs' sums in their order, rounded once.
template <int GDT>
__global__ __launch_bounds__(256) void dvals_sum_kernel(int64_t B, int32_t R, const int32_t *__restrict__ blk_ptr, int32_t S,
                                                        const float *__restrict__ partial, int64_t stride, int32_t vec,
                                                        void *__restrict__ D) {
    const int64_t total = (int64_t)R * blk_ptr[B];
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
    if (i >= total) return;  // (total is a multiple of 8)
    f32x4 acc = *reinterpret_cast<const f32x4 *>(partial + i);
    for (int s = 1; s < S; ++s) acc += *reinterpret_cast<const f32x4 *>(partial + (int64_t)s * stride + i);
    if (vec) {
        if constexpr (GDT == BSP_F32) *reinterpret_cast<f32x4 *>((float *)D + i) = acc;
        else *reinterpret_cast<uint2 *>((uint16_t *)D + i) = make_uint2(cvt_pk<GDT>(acc[0], acc[1]), cvt_pk<GDT>(acc[2], acc[3]));
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) elem<GDT>::store(D, i + j, acc[j]);
    }
}

template <int DT, int ODT, int FM, int FN, int WR, int WC, bool TOTALS>
int launch_dense(const DvalsDense &a, int S, int per, int chain) {
    using G = DdShape<DT, FM, FN, WR, WC>;
    auto k = dvals_dense_kernel<DT, ODT, FM, FN, WR, WC, TOTALS>;
    if constexpr (G::kLds > 65536) {  // (asking again is harmless)
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, (int)G::kLds);
        if (e != hipSuccess) {
            set_last_hip_error((int)e);
            return BSP_ERR_HIP;
        }
    }
    const int64_t tiles = ((a.M + G::BM - 1) / G::BM) * ((a.N + G::BN - 1) / G::BN), wgs = (tiles * S + 7) / 8 * 8;
    if (wgs >= ((int64_t)1 << 31)) return BSP_ERR_SHAPE;
    const int64_t stride = ((int64_t)a.R * a.capacity_cols + 3) / 4 * 4;
    k<<<(unsigned)wgs, G::kWaves * 64, G::kLds, a.s>>>(a.X, a.dY, a.T, (int32_t)a.M, (int32_t)a.N, a.R, a.blk_cnt, a.blk_ptr, a.col_idx,
                                                       a.colstart, (int32_t)(a.capacity_cols - 1), per, S, chain, stride, S > 1 ? (void *)a.partial : a.D);
    if (S > 1) {
        const unsigned grid = (unsigned)(((int64_t)a.R * a.capacity_cols + 1023) / 1024);
        const int vec = aligned(a.D, 16) ? 1 : 0;
        BSP_DISPATCH_DTYPE(a.gdt, GDT, (dvals_sum_kernel<GDT><<<grid, 256, 0, a.s>>>(a.M / a.R, a.R, a.blk_ptr, S, a.partial, stride, vec, a.D)));
    }
    return check_launch();
}

}  // namespace

namespace {
// The square of a sum's error grows with the stages of a chain of matrix instructions, which rounds a sum that grows all along, and with the
// additions that put the chains together; a stage counts as much as 2.7 additions (dvals_sums_error).  Measured, sums of N(0, 1) products in
// fp32 against 64 bits: 1.25e-7 of the value for a chain of 16 stages, 2.7e-7 of 64, 5.8e-7 of 256; 64 stages in chains of 4 0.97e-7, of 8
// 1.03e-7, of 16 1.33e-7; 256 in chains of 8 1.36e-7.
// The longest chain for sums over `runs` runs of `per` stages that are no further off than `error`, that of the sparse form's runs: with one
// chain per run this form's were up to 2.1 times as far (4096 x 1024, R = 32 at 1.43x, 4099 tokens 4.0e-7 against 1.9e-7).  0: none is.
int64_t sums_chain(int64_t per, int64_t runs, int64_t error) {
    auto off = [&](int64_t c) { return dvals_sums_error(c, (per + c - 1) / c + runs - 1); };
    const double k = (double)(error + 20 - 10 * runs), d = k * k - 1080.0 * (double)per;
    int64_t c = per;
    if (off(c) > error) c = d < 0.0 ? 0 : (int64_t)((k + __builtin_sqrt(d)) / 54.0);
    while (c > 0 && off(c) > error) --c;
    return c < per ? c : per;
}
}  // namespace

// Which tile and how many runs of the tokens: the least estimated time of those whose sums are near enough, microseconds fitted to 17800
// launches of 605 calls of 256 to 4096 rows and columns, 16 to 16384 tokens, 1.43x to 8x (4 to 7 % off on average; on 400
// other calls, on operands in the caches and on fresh ones, the choice, the sparse form among it, costs 0.9 % against the fastest of all that was
// measured, more than 10 % in 2.3 % of them, 1.23 times at worst).  A
// workgroup of the largest tile fills a compute unit; of the others two and three share one; a stage takes longer the more of the chip
// is busy.  The largest tile has no registers for totals, so for fp32 results it is taken where its runs are as short as the sparse form's, at
// low rates.  What the chains cost: fp32 results of 150 drawn calls take 1.045 of the time of one chain per run, 0.44 of the sparse form's alone.
DvalsDenseChoice dvals_dense_choose(int64_t T, int64_t M, int64_t N, int32_t R, int64_t capacity_cols, int64_t partial_floats, int64_t error) {
    constexpr struct {
        int bm, bn;
        double fixed, alone, full, shared, end, flush, sums;  // a stage of a workgroup alone on its compute unit, more of it the fuller the
                                                              // chip is, per workgroup of several; a workgroup's end; its sums to
                                                              // the totals; a million sums of a run
    } shapes[] = {{256, 256, 5.4, 0.440, 0.220, 0.550, 3.8, 0.0, 0.9},
                  {128, 128, 5.5, 0.200, 0.056, 0.176, 1.41, 0.285, 1.37},
                  {64, 128, 4.5, 0.179, 0.030, 0.135, 0.77, 0.069, 1.37}};
    const int64_t stages = (T + kDdTok - 1) / kDdTok, stride = ((int64_t)R * capacity_cols + 3) / 4 * 4;
    DvalsDenseChoice best = {-1, 0, 0, 0, 0.0};
    for (int i = 0; i < 3; ++i) {
        const int64_t tiles = ((M + shapes[i].bm - 1) / shapes[i].bm) * ((N + shapes[i].bn - 1) / shapes[i].bn);
        for (int64_t S = 1; S <= 16 && S <= stages; ++S) {
            if ((S > 1 && S * stride > partial_floats) || tiles * S >= ((int64_t)1 << 30)) break;
            const int64_t per = (stages + S - 1) / S;
            if ((stages + per - 1) / per != S) continue;  // (runs without a stage)
            const double count = (double)(tiles * S) / 256.0, rounds = __builtin_ceil(count);  // workgroups per compute unit
            // (the largest tile's stage takes 0.44 us on up to half of the compute units, 0.60 on seven eighths, 0.66 on all: the clocks)
            const double fill = __builtin_fmin(count, 1.0), slower = i == 0 ? fill * fill * fill : fill;
            const double stage = __builtin_fmax(shapes[i].alone + shapes[i].full * slower, shapes[i].shared * rounds);
            double us = shapes[i].fixed + stage * (double)per + shapes[i].end * rounds;
            if (S > 1) us += 1.0 + 0.25 * (double)S + 1e-6 * shapes[i].sums * (double)(S + 1) * (double)stride;
            if (best.shape >= 0 && us >= best.us) continue;
            const int64_t chain = sums_chain(per, S, error);
            if (chain < 1 || (i == 0 && chain < per)) continue;
            if (chain < per) us += shapes[i].flush * (double)per / (double)chain * rounds;
            if (best.shape < 0 || us < best.us) best = {i, (int)S, (int)per, (int)chain, us};
        }
    }
    // (Large products in 128 x 128 tiles, which read each operand twice as often as the largest tile: on operands that are in no cache 1.2 to 1.36
    // of the estimate, 1.05 on cached ones.  3072 x 1024 at 5x, 6144 tokens, fp32 result 43 us by the estimate, 58 fresh; sparse 45.  Of 4200 calls
    // of more than 0.3 G products with fp32 results the choice of the form lost up to 1.32 without this, 1.09 with it.)
    if (best.shape == 1) best.us *= 1.0 + __builtin_fmin(0.3, __builtin_fmax(0.0, 0.012 * (1e-9 * (double)M * (double)N * (double)T - 8.0)));
    return best;
}

int launch_dvals_dense(const DvalsDense &a, const DvalsDenseChoice &c) {
    auto shape = [&](auto dt, auto odt) {
        constexpr int DT = decltype(dt)::value, ODT = decltype(odt)::value;
        if (c.shape == 0) return launch_dense<DT, ODT, 4, 2, 2, 4, false>(a, c.S, c.per, c.chain);
        if constexpr (ODT == BSP_F32) {  // (16-bit results of one run ask for no chains)
            if (c.chain < c.per)
                return c.shape == 1 ? launch_dense<DT, ODT, 2, 2, 2, 2, true>(a, c.S, c.per, c.chain)
                                    : launch_dense<DT, ODT, 1, 2, 2, 2, true>(a, c.S, c.per, c.chain);
        }
        if (c.shape == 1) return launch_dense<DT, ODT, 2, 2, 2, 2, false>(a, c.S, c.per, c.chain);
        return launch_dense<DT, ODT, 1, 2, 2, 2, false>(a, c.S, c.per, c.chain);
    };
    auto go = [&](auto dt) {
        if (c.S > 1 || a.gdt == BSP_F32) return shape(dt, std::integral_constant<int, BSP_F32>{});
        return a.gdt == BSP_BF16 ? shape(dt, std::integral_constant<int, BSP_BF16>{}) : shape(dt, std::integral_constant<int, BSP_F16>{});
    };
    return a.xdt == BSP_BF16 ? go(std::integral_constant<int, BSP_BF16>{}) : go(std::integral_constant<int, BSP_F16>{});
}

}  // namespace bsp
