// The planned layer for few tokens (Sec. 3.1, Sec. 4.4): row-blocks of 16 rows (and the block heights whose plans are made of
// those), bf16 / fp16 on gfx950.
//
// The kernels for many tokens give a workgroup 64 tokens and at least 32 row-blocks, and the one for wide layers
// walks the column chunks of X one after the other: with 24 tokens a 768 x 3072 layer is two workgroups of 256 compute
// units, 33 us.  Here a workgroup owns 16 NSUB tokens and NB row-blocks, and 8 / NB wavefronts share the steps of a row-block
// over all its chunks; their partial sums meet in LDS (in the order of the steps, so two calls give the same bits).
// All columns of X are in LDS ([column][16 tokens], the layout the plan's offsets are made for), which is what the
// narrow token tile buys: 16 tokens of 4096 columns are 128 KiB.
//
// It reads the same plan as the other kernels: the steps of a (row-block, chunk) are contiguous, found through the
// stream table.  A wavefront lists its steps 64 at a time, one per lane, and runs through them with the operands of
// four steps in flight.
#include "bsp_common.h"
#include "bsp_linear_internal.h"
#include "bsp_mfma_device.h"
#include "bsp_tile_device.h"

namespace bsp {
namespace {

constexpr int kSmDepth = 4;     // steps whose operands are on their way
constexpr int kSmMaxSteps = 4096 / 32 + kPlanMaxChunks;  // of a row-block

struct SmPlan {  // the plan's geometry
    const int32_t *wptr;
    const uint8_t *wfrag, *xoff;
    int32_t waves, nacc, NG, nq, paired, max_step;
};

// Copy-in of 16 NSUB token rows (past T: zeros): a unit is 4 tokens x 8 columns, see stage_x_tile64_rows16.
template <int NSUB, int NW>
__device__ __forceinline__ void small_copy_in(const uint16_t *__restrict__ X, int64_t T, int64_t N, int32_t npad,
                                              int64_t t0) {
    const int octs = (int)(N >> 3), octs_pad = npad >> 3;
    constexpr int kBatch = 3, kThreads = NW * 64;
    for (int u0 = threadIdx.x; u0 < octs_pad * 4 * NSUB; u0 += kThreads * kBatch) {
        uint4 a[kBatch][4];
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            const int u = u0 + k * kThreads;
            const int o = u % octs_pad, tq = u / octs_pad;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int64_t t = t0 + 4 * tq + i;
                a[k][i] = (tq < 4 * NSUB && o < octs && t < T) ? *reinterpret_cast<const uint4 *>(X + t * N + 8 * o)
                                                               : make_uint4(0u, 0u, 0u, 0u);
            }
        }
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            const int u = u0 + k * kThreads;
            const int o = u % octs_pad, tq = u / octs_pad;
            if (tq >= 4 * NSUB) break;
            const uint32_t c = 8u * (uint32_t)o;
            uint8_t *dst = smem_x + (c >> 9) * (NSUB * kSubStride4) + (uint32_t)(tq >> 2) * kSubStride4 +
                           lds_col_offset(c & 511u, (uint32_t)(tq & 3));
            const uint32_t w[4][4] = {{a[k][0].x, a[k][1].x, a[k][2].x, a[k][3].x},
                                      {a[k][0].y, a[k][1].y, a[k][2].y, a[k][3].y},
                                      {a[k][0].z, a[k][1].z, a[k][2].z, a[k][3].z},
                                      {a[k][0].w, a[k][1].w, a[k][2].w, a[k][3].w}};
#pragma unroll
            for (int j = 0; j < 4; ++j) {  // the column pair 2 j, 2 j + 1 of the piece
                uint2 lo, hi;
                lo.x = __builtin_amdgcn_perm(w[j][1], w[j][0], 0x05040100u);
                lo.y = __builtin_amdgcn_perm(w[j][3], w[j][2], 0x05040100u);
                hi.x = __builtin_amdgcn_perm(w[j][1], w[j][0], 0x07060302u);
                hi.y = __builtin_amdgcn_perm(w[j][3], w[j][2], 0x07060302u);
                const uint32_t at = (uint32_t)(j >> 1) * 32u + (uint32_t)(j & 1) * (16u * 32u);
                *reinterpret_cast<uint2 *>(dst + at) = lo;
                *reinterpret_cast<uint2 *>(dst + at + 8u * 32u) = hi;
            }
        }
    }
}

template <int DT, int NSUB, int NW>
__global__ __launch_bounds__(NW * 64) void linear_small16_kernel(const uint16_t *__restrict__ X, int64_t T, int64_t M,
                                                                    int64_t N, int32_t npad, SmPlan P, int32_t B,
                                                                    int32_t ntiles, int32_t nb,
                                                                    const void *__restrict__ bias,
                                                                    void *__restrict__ Y, int32_t act,
                                                                    const uint16_t *__restrict__ residual) {
    const int tile = blockIdx.x % ntiles, b0 = (int)(blockIdx.x / ntiles) * nb;
    const int64_t t0 = (int64_t)tile * (16 * NSUB);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // NW / nb wavefronts share a row-block; with nb > NW a wavefront takes row-blocks NW apart one after the other
    const int kw = nb < NW ? NW / nb : 1;
    const int part = wave % kw;
    int b = b0 + wave / kw;
    const int b_end = b0 + nb < B ? b0 + nb : B;

    // ---- the wavefront's steps: first .. first + cnt - 1 of its row-block's, chunk after chunk ----
    int start = 0, n = 0, incl = 0;  // lane q: chunk q's first step in the plan, its steps, the steps up to its end
    int first = 0, cnt = 0;
    auto locate = [&](int block, int &lo, int &hi) {  // lane q: where chunk q's steps begin and end
        lo = hi = 0;
        if (block < b_end && lane < P.nq) {
            int64_t eg;
            int ew, ei;
            plan_entry(block, P.waves, P.nacc, P.paired != 0, eg, ew, ei);
            const int32_t *my = P.wptr + (int64_t)ew * ((int64_t)P.nq * P.NG * P.nacc + 1) + ((int64_t)eg * P.nq * P.nacc + ei);
            lo = my[lane * P.nacc];
            hi = my[lane * P.nacc + 1];
        }
    };
    auto count = [&](int lo, int hi) {  // (kept inside the plan whatever it holds)
        start = min(max(lo, 0), P.max_step);
        n = min(min(max(hi, start), P.max_step) - start, kSmMaxSteps);
        incl = n;
#pragma unroll
        for (int o = 1; o < kPlanMaxChunks; o <<= 1) {
            const int up = __shfl_up(incl, o, 64);
            if (lane >= o) incl += up;
        }
        const int total = min(__builtin_amdgcn_readlane(incl, kPlanMaxChunks - 1), kSmMaxSteps);
        first = total * part / kw;
        cnt = total * (part + 1) / kw - first;
    };
    auto list_steps = [&](int from) {  // step | chunk << 28 of the row-block's step from + lane
        int e = 0;
        for (int q = 0; q < P.nq; ++q) {
            const int s = __builtin_amdgcn_readlane(start, q), c = __builtin_amdgcn_readlane(n, q);
            const int j = from + lane - (__builtin_amdgcn_readlane(incl, q) - c);
            if (j >= 0) e = (s + min(j, max(c - 1, 0))) | (q << 28);
        }
        return e;
    };
    int next_lo, next_hi;
    locate(b, next_lo, next_hi);
    count(next_lo, next_hi);
    // ---- its operands: four steps on their way before the copy-in, whose latency they share ----
    const bool chunked = P.nq > 1;
    const uint32_t quad = (uint32_t)(lane & 3) * 0x00010001u;
    const uint32_t frag_at = lane * 16, off_at = (lane >> 2) * 4;
    u32x4 rf[kSmDepth];
    uint32_t ro[kSmDepth], rq[kSmDepth];
    auto ask = [&](auto slot, int list, int k, int end) {  // the k-th step of the list, or the last one
        constexpr int s = decltype(slot)::value;
        const int e = __builtin_amdgcn_readlane(list, k < end ? k : end - 1);
        const int64_t st = e & 0x0fffffff;
        rf[s] = *reinterpret_cast<const u32x4 *>(P.wfrag + st * 1024 + frag_at);
        ro[s] = *reinterpret_cast<const uint32_t *>(P.xoff + st * 64 + off_at);
        rq[s] = (uint32_t)e >> 28;
    };
    int list = list_steps(first), listed = min(cnt, 64);
    if (cnt > 0) static_for<0, kSmDepth>([&](auto j) { ask(j, list, j, listed); });
    // Results: four rows of one token, (row-block i, sub-tile u, lane l); what is added to them at the end.
    auto extras = [&](bool in, int64_t t, int64_t m, float (&bv)[4], uint2 &res) {
#pragma unroll
        for (int v = 0; v < 4; ++v) bv[v] = (in && bias) ? elem<DT>::load(bias, m + v) : 0.0f;
        res = (in && residual) ? *reinterpret_cast<const uint2 *>(residual + t * M + m) : make_uint2(0u, 0u);
    };
    auto finish = [&](f32x4 s, int64_t t, int64_t m, const float (&bv)[4], uint2 res) {
        const uint32_t h[4] = {res.x & 0xffffu, res.x >> 16, res.y & 0xffffu, res.y >> 16};
        float y[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            y[v] = s[v] + bv[v];
            if (act == BSP_ACT_GELU) y[v] = gelu_fit(y[v]);
            if (residual) {
                if constexpr (DT == BSP_BF16) y[v] += __uint_as_float(h[v] << 16);
                else y[v] += (float)__builtin_bit_cast(_Float16, (uint16_t)h[v]);
            }
        }
        *reinterpret_cast<uint2 *>((uint16_t *)Y + t * M + m) = make_uint2(cvt_pk<DT>(y[0], y[1]), cvt_pk<DT>(y[2], y[3]));
    };
    const int outs = (nb < NW ? nb : NW) * NSUB * 64;
    auto place = [&](int idx, int64_t &t, int64_t &m) {
        const int i = idx / (NSUB * 64), u = (idx >> 6) % NSUB, l = idx & 63;
        t = t0 + 16 * u + (l & 15);
        m = (int64_t)(b0 + i) * 16 + 4 * (l >> 4);
        return idx < outs && b0 + i < B && t < T;
    };
    int64_t t_first, m_first;
    float bv[4];
    uint2 res;
    const bool in_first = place(tid, t_first, m_first);
    if (nb <= NW) extras(in_first, t_first, m_first, bv, res);

    small_copy_in<NSUB, NW>(X, T, N, npad, t0);
    __syncthreads();

    f32x4 acc[NSUB];
    auto use = [&](auto slot) {
        constexpr int s = decltype(slot)::value;
        // offsets / 8 of the lane's two reads, made for the 64-token tile: bits 0 - 13 of the byte offset are the place
        // inside a chunk of 512 columns; above them here follow the chunk and, by constant offsets, the sub-tiles
        const uint32_t o = ro[s] ^ quad;
        const uint32_t a = (o & 0xffffu) << 3, c = (o >> 16) << 3;
        const uint32_t a1 = (a & (kSubStride4 - 1)) + (chunked ? rq[s] : a >> 16) * (NSUB * kSubStride4);
        const uint32_t c1 = (c & (kSubStride4 - 1)) + (chunked ? rq[s] : c >> 16) * (NSUB * kSubStride4);
        const uint4 w = make_uint4(rf[s].x, rf[s].y, rf[s].z, rf[s].w);
#pragma unroll
        for (int u = 0; u < NSUB; ++u) {
            const uint2 x0 = tr_read_at(a1 + u * kSubStride4), x1 = tr_read_at(c1 + u * kSubStride4);
            acc[u] = mfma16<DT>(w, make_uint4(x0.x, x0.y, x1.x, x1.y), acc[u]);
        }
    };
    auto walk = [&]() {  // the steps of one row-block (its first four are on their way)
#pragma unroll
        for (int u = 0; u < NSUB; ++u) acc[u] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int from = 0; from < cnt; from += 64) {
            if (from > 0) {
                list = list_steps(first + from);
                listed = min(cnt - from, 64);
                static_for<0, kSmDepth>([&](auto j) { ask(j, list, j, listed); });
            }
            int k = 0;
            for (; k + kSmDepth <= listed; k += kSmDepth)
                static_for<0, kSmDepth>([&](auto j) {
                    use(j);
                    ask(j, list, k + j + kSmDepth, listed);
                });
            static_for<0, kSmDepth - 1>([&](auto j) {
                if (k + j < listed) use(j);
            });
        }
    };

    if (nb > NW) {  // whole row-blocks one after the other, straight from the registers
        for (; b < b_end; b += NW) {  // uniform
            const int64_t m = (int64_t)b * 16 + 4 * (lane >> 4);
            float bw[NSUB][4];
            uint2 rw[NSUB];
#pragma unroll
            for (int u = 0; u < NSUB; ++u) {
                const int64_t t = t0 + 16 * u + (lane & 15);
                extras(t < T, t, m, bw[u], rw[u]);
            }
            locate(b + NW, next_lo, next_hi);
            walk();
            count(next_lo, next_hi);
            list = list_steps(first);
            listed = min(cnt, 64);
            if (cnt > 0) static_for<0, kSmDepth>([&](auto j) { ask(j, list, j, listed); });
#pragma unroll
            for (int u = 0; u < NSUB; ++u) {
                const int64_t t = t0 + 16 * u + (lane & 15);
                if (t < T) finish(acc[u], t, m, bw[u], rw[u]);
            }
        }
        return;
    }

    walk();
    // ---- partial sums together, then bias, activation, residual, one rounding ----
    __syncthreads();  // the tile has been read
    f32x4 *red = reinterpret_cast<f32x4 *>(smem_x);
#pragma unroll
    for (int u = 0; u < NSUB; ++u) red[(wave * NSUB + u) * 64 + lane] = acc[u];
    __syncthreads();
    for (int idx = tid; idx < outs; idx += NW * 64) {
        int64_t t, m;
        const bool in = place(idx, t, m);
        if (idx != tid) extras(in, t, m, bv, res);
        const int i = idx / (NSUB * 64), in_block = idx % (NSUB * 64);
        f32x4 s = red[i * kw * NSUB * 64 + in_block];
        for (int p = 1; p < kw; ++p) s += red[(i * kw + p) * NSUB * 64 + in_block];
        if (in) finish(s, t, m, bv, res);
    }
}

template <int NSUB, int NW>
size_t small_lds(int32_t npad) {
    const int32_t chunks = (npad + 511) / 512;
    const size_t tile = (size_t)(chunks - 1) * NSUB * kSubStride4 + (size_t)(NSUB - 1) * kSubStride4 + (size_t)(npad - 512 * (chunks - 1)) * 32;
    const size_t red = (size_t)NW * NSUB * 1024;
    return tile > red ? tile : red;
}

template <int DT, int NSUB, int NW>
int launch_small(const TiledArgs &a, const SmPlan &P, int nb, hipStream_t s) {
    const int64_t ntiles = (a.T + 16 * NSUB - 1) / (16 * NSUB), groups = (a.B + nb - 1) / nb;
    if (ntiles * groups >= ((int64_t)1 << 31)) return BSP_ERR_SHAPE;
    static thread_local size_t configured = 0;
    const size_t lds = small_lds<NSUB, NW>(a.npad);
    auto kern = linear_small16_kernel<DT, NSUB, NW>;
    int st = raise_lds_limit(kern, lds, configured);
    if (st != BSP_OK) return st;
    kern<<<dim3((unsigned)(ntiles * groups)), dim3(NW * 64), lds, s>>>(
        a.X, a.T, a.M, a.N, a.npad, P, (int32_t)a.B, (int32_t)ntiles, nb, a.bias, a.Y, a.act, (const uint16_t *)a.residual);
    return check_launch();
}

}  // namespace

namespace {

// Microseconds that a call takes, launch included, by the kernels for many tokens and by this one; from layers of 256 to
// 4096 columns at 1.4x to 5x and 8 to 4099 tokens, to about 15 %.  steps: of a row-block, over all chunks.
double estimate_many(const TiledArgs &a, const SmPlan &P, int64_t T, double steps) {
    const int64_t tiles = (T + 63) / 64;
    if (P.nq > 1) {
        const int waves = stream_waves(tiles, a.B);
        // (that kernel's GELU: 512 x 2048 at 5x, 6243 tokens 13.5 us without, 15.1 with)
        const double gelu = a.act == BSP_ACT_GELU ? 2.0 : 0.0;
        return 5.0 + stream_load(tiles, a.B, waves) * (0.4 + 1.5 * P.nq + (waves == 8 ? 0.43 : 0.38) * steps + gelu);
    }
    const int64_t gps = steploop_groups(tiles, P.NG, a.N, steps);
    return 4.5 + steploop_walk_us(tiles, P.NG, gps, a.N, steps);
}

struct SmShape {
    int nw, nsub, nb;
};

double estimate_few(const TiledArgs &a, int64_t T, double steps, const SmShape &c) {
    const double wgs = (double)((T + 16 * c.nsub - 1) / (16 * c.nsub)) * (double)((a.B + c.nb - 1) / c.nb) / 256.0;
    const double mine = steps * (double)c.nb / (double)c.nw;  // steps of a wavefront
    const double one = 4.8 + 0.0003 * (double)a.N + (c.nw == 16 ? 0.20 : (c.nsub == 2 ? 0.18 : 0.11)) * mine;
    if (wgs <= 1.0) return one;
    // 8 wavefronts and less than half of the LDS: two workgroups on a compute unit
    if (c.nw == 8 && c.nsub * a.npad * 32 <= 80 * 1024) return one * (1.0 + (c.nsub == 2 ? 0.62 : 0.5) * (wgs - 1.0));
    return one * __builtin_ceil(wgs);
}

template <int DT>
int launch_shape(const TiledArgs &a, const SmPlan &P, const SmShape &c, hipStream_t s) {
    if (c.nw == 16) return launch_small<DT, 1, 16>(a, P, c.nb, s);
    return c.nsub == 2 ? launch_small<DT, 2, 8>(a, P, c.nb, s) : launch_small<DT, 1, 8>(a, P, c.nb, s);
}

// The shape with the least estimated time for T tokens, if that is below us (which becomes it).
SmShape choose_shape(const TiledArgs &a, int64_t T, double steps, double &us) {
    constexpr SmShape shapes[] = {{8, 1, 1}, {8, 1, 2}, {8, 1, 4}, {8, 1, 8}, {8, 2, 4}, {8, 2, 8}, {16, 1, 8}, {16, 1, 16}, {16, 1, 32}};
    SmShape best = {0, 0, 0};
    for (const SmShape &c : shapes) {
        if (c.nsub * a.npad > 4096) continue;  // (128 KiB of LDS)
        const double t = estimate_few(a, T, steps, c);
        if (t < us) us = t, best = c;
    }
    return best;
}

// The same call on rows first .. first + count - 1 of the batch.
TiledArgs token_rows(const TiledArgs &a, int64_t first, int64_t count) {
    TiledArgs r = a;
    r.X = a.X + first * a.N;
    r.Y = (uint16_t *)a.Y + first * a.M;
    if (a.residual) r.residual = (const uint16_t *)a.residual + first * a.M;
    r.T = count;
    return r;
}

}  // namespace

// True when this layer's call was taken (status in st).  Which kernel and which shape: the one with the least estimated
// time.  Measured, us (many tokens / this one): 2304 x 768 at 2x, 24 tokens 10.4 / 5.0, 400 tokens 10.9 / 7.6,
// 1200 tokens 11.7 / 15.3 (stays); 768 x 3072 at 2x, 24 tokens 31 / 6.3, 400 tokens 31 / 12.2, 1537 tokens 34 / 24.3
// and at 3x 26.7 / 19.2; 1024 x 4096 at 5x, 4099 tokens 29.6 / 60 (stays).  Those are from before the streaming kernel's loop of six
// steps, which is as fast as this one near the border now: 768 x 3072 at 3x, 1537 tokens 17.6 / 17.9 (fresh X 18.9 / 18.8), and the
// faster one at 5x: 1024 x 4096, 2048 tokens 16.6 / 23.0 (19.9 / 22.3), where the estimates still come here.
// A batch a little longer than a whole number of token tiles on every XCD costs the kernels for many tokens a round of
// mostly idle compute units, or the wide split that avoids it: then the tiles that are too many come here and only the others go
// there, if that is less by the estimates: whole / in two, us, 1024 x 4096 with a residual at 1.43x, 4099 tokens 57.0 / 52.7, at 2x,
// 8200 tokens 81.0 / 54.0; 4096 x 1024 with GELU at 1.43x, 4099 tokens 44.3 / 42.4; 2048 x 512 at 1.5x, 8200 tokens 28.1 / 24.3.
bool launch_linear_small16(const TiledArgs &a, int64_t max_step, hipStream_t s, int &st) {
    const PlanChunks ch = plan_chunks(a.N, a.R, a.M);
    const bool chunked = ch.n > 1;
    SmPlan P;
    P.wptr = a.wptr;
    P.wfrag = (const uint8_t *)a.wfrag;
    P.xoff = (const uint8_t *)a.xoff;
    P.waves = plan_waves(a.N, a.R, a.M);
    P.nacc = plan_nacc(1, chunked, a.R);
    P.paired = plan_paired(a.R, chunked) ? 1 : 0;
    P.NG = (int32_t)plan_groups(a.B, P.waves, P.nacc, P.paired != 0);
    P.nq = ch.n;
    P.max_step = (int32_t)max_step;
    const double steps = plan_steps(a);

    const double many_us = estimate_many(a, P, a.T, steps);
    double best_us = 0.85 * many_us;  // (the estimates' spread: near a tie the other kernels stay)
    const SmShape best = choose_shape(a, a.T, steps, best_us);
    const int64_t tiles = (a.T + 63) / 64, over = tiles % 8;
    if (best.nw == 0 && tiles > 24 && over >= 1 && over <= 4 && aligned(a.Y, 16)) {
        const int64_t head = (tiles - over) * 64;
        double tail_us = 0.95 * many_us - estimate_many(a, P, head, steps);
        const SmShape c = choose_shape(a, a.T - head, steps, tail_us);
        if (c.nw != 0) {
            const TiledArgs first = token_rows(a, 0, head), rest = token_rows(a, head, a.T - head);
            st = chunked ? launch_linear_stream16(first, max_step, s) : launch_linear_steploop16(first, max_step, s);
            if (st == BSP_OK) st = a.xdt == BSP_BF16 ? launch_shape<BSP_BF16>(rest, P, c, s) : launch_shape<BSP_F16>(rest, P, c, s);
            return true;
        }
    }
    if (best.nw == 0) return false;
    st = a.xdt == BSP_BF16 ? launch_shape<BSP_BF16>(a, P, best, s) : launch_shape<BSP_F16>(a, P, best, s);
    return true;
}

}  // namespace bsp
