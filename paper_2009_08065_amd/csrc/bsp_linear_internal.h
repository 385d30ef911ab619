// Internal interface between the layer's entry points and its tiled matrix-core kernel.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace bsp {

constexpr int kPlanWaves = 8;       // wavefronts per workgroup of a planned kernel = streams of a plan ...
constexpr int kPlanWavesWide = 16;  // ... and where the registers allow it: see plan_waves()
#define kPlanWaves16 16             // ... of the kernel for R = 16 and narrow layers (a macro: its assembly needs the literal)

struct TiledArgs {
    int xdt;
    const uint16_t *X;
    int64_t T, M, N, B;
    int32_t R;
    int32_t stored_R;         // planned source: rows of the storage's row-blocks (R: of the plan's)
    int32_t npad;             // filled by the launcher: N rounded up to 256 columns
    const int32_t *blk_ptr;
    const int32_t *col_idx;   // canonical source
    const uint16_t *vals;     // canonical source
    const int32_t *wptr;      // planned source: [waves][chunks * NG * nacc + 1] first step of (chunk q, block (g * waves + w) * nacc + i) at [w][(g * chunks + q) * nacc + i]
    const void *wfrag;        // planned source: [step][fragment][lane] 16-byte panel fragments
    const uint32_t *xoff;     // planned source: [step][lane] two 16-bit LDS byte offsets
    int64_t plan_steps;       // planned source: steps the fragment / offset regions hold (slack included)
    int64_t capacity_cols;    // planned source: the caller's bound on the padded kept columns of the storage
    const void *bias;
    void *Y;
    int act;                  // bsp_activation applied to the sums before they are rounded (the planned kernels of R = 16)
    const void *residual;     // [T, M], type of X, added after the activation (only the kernel that streams X), or null
};

// True when the tiled kernel can take this layer (16-bit floats, kp_b % 32 == 0, X tile fits in LDS).
bool tiled_supported(int xdt, int64_t N, int32_t k_align);
int launch_linear_tiled(const TiledArgs &args, bool plan, hipStream_t s);
// The planned kernel for R = 16 and layers of up to 1024 input columns (16-bit floats, a plan of 16 streams, Y
// aligned to 16 bytes); NG = groups of the plan, max_step = steps the plan holds without its read-ahead slack.
int launch_linear_steploop16(const TiledArgs &args, int64_t max_step, hipStream_t s);
// The same for R = 16 and wider layers (up to 4096 input columns), whose plans are cut into chunks of 512 columns.
int launch_linear_stream16(const TiledArgs &args, int64_t max_step, hipStream_t s);
// The kernel for few tokens, same plans: true when it is the faster one for this call and has been launched (status in st).
bool launch_linear_small16(const TiledArgs &args, int64_t max_step, hipStream_t s, int &st);
// Column chunks of a plan: layers with more than 1024 (padded) input columns are cut into chunks of
// 1024 columns, the width of X that fits in LDS next to 64 tokens; narrower layers are one chunk.
// R = 16: chunks of 512 columns, two of which are in LDS at a time -- one being used, one being filled.  Layers of
// R = 16 with few row-blocks (up to 64: the attention output projection) are planned that way from 513 columns
// on: with so few blocks the kernel for narrow layers would give a wavefront one or two pairs of row-blocks per
// workgroup, and the kernel that streams X runs them as fast and writes its output once, at its end -- which is
// where a residual can be added without a load in the step loop.
constexpr int kPlanMaxChunks = 8;
struct PlanChunks {
    int32_t n;      // number of chunks
    int32_t shift;  // column >> shift = chunk
};
inline PlanChunks plan_chunks(int64_t N, int32_t R, int64_t M) {
    const int64_t npad = (N + 255) / 256 * 256;
    if (R == 16 && (npad > 1024 || (npad > 512 && M / 16 <= 64))) return PlanChunks{(int32_t)((npad + 511) / 512), 9};
    if (npad <= 1024) return PlanChunks{1, 30};
    return PlanChunks{(int32_t)((npad + 1023) / 1024), 10};
}
// Row-blocks of 8 rows ride the kernels written for 16 when the layer's height allows it: two neighbouring row-blocks
// form one block of 16 rows that keeps the union of their columns; a step's fragment holds the first one's weights in
// rows 0-7 and the second one's in rows 8-15, with zeros where only the other one keeps the column.  Every plan
// parameter is then the one of R = 16.
inline bool plan_virtual16(int32_t R, int64_t M) { return R == 8 && M % 16 == 0; }
// Row-blocks of 32, 48 or 64 rows ride them too: a block of the plan is one 16-row slab of a stored row-block (the
// stored block's kept columns, the slab's rows of its panel), so such a layer runs as the layer of 16-row blocks with
// the same kept columns does.  (The slabs of a block gather the same columns of X from LDS once each; a kernel that
// shared the gather would need a step loop of its own per block height.)
inline int plan_split16(int32_t R) { return (R > 16 && R % 16 == 0) ? R / 16 : 1; }
// Height of the blocks a layer's plan is made of.
inline int32_t plan_block_rows(int32_t R, int64_t M) { return (plan_virtual16(R, M) || plan_split16(R) > 1) ? 16 : R; }
// Chunked plans of R = 16 give every (row-block, chunk) at least one step (of zero weights where the block keeps
// no column of the chunk), as one-chunk plans give every row-block: the assembly loops never meet an empty run.
inline bool plan_min_one_step(int32_t R, bool chunked) { return !chunked || R == 16; }
// A wavefront of the planned kernels works on runs of nacc consecutive row-blocks, so that it can write 64
// or 128 contiguous bytes per token row: 4 sixteen-row fragments' worth in the column-chunked kernel with 8
// wavefronts (which holds all their accumulators and writes once, at the end), 2 with 16 wavefronts (R = 16, 32:
// see plan_waves) and in the kernel for layers of up to 1024 columns (64 bytes per row are enough there).
// R = 8 fills half a fragment, so 4 of its row-blocks make 64 bytes.
constexpr int plan_nacc(int nfrag, bool chunked, int R) {
    if (R == 8) return 4;
    if (R == 16 && chunked) return 4;  // (8 wavefronts that hold the accumulators of 4 row-blocks each)
    const int frags = (chunked && R != 16 && R != 32) ? 4 : 2;
    return frags / nfrag > 0 ? frags / nfrag : 1;
}
// Streams of a plan = wavefronts of the workgroup that consumes it.  Layers with R = 16 or 32 run 16
// wavefronts (4 per SIMD) on a short operand ring: their kernels stay within 128 registers, and the
// per-wavefront chains of dependent instructions overlap better (measured 10-14 % faster than 8 wavefronts).
// The other R do not fit (R = 64: four fragments of accumulators; R = 8 and odd sizes: their output paths).
inline int plan_waves(int64_t N, int32_t R, int64_t M) {
    if (R == 16 && plan_chunks(N, R, M).n > 1) return kPlanWaves;  // beside them run the wavefronts that copy X in
    if (R == 16) return kPlanWaves16;
    return R == 32 ? kPlanWavesWide : kPlanWaves;
}
// Which row-block a plan's entry (group g, wavefront w, place i in the run) stands for, and back.  Plain plans deal
// runs of nacc blocks round robin: block (g * waves + w) * nacc + i.  Paired plans (R = 16, one column chunk: the
// kernel with the assembly loop) deal runs of 2 blocks so that the runs of one wavefront in groups 2 s and 2 s + 1 are
// neighbours -- four consecutive row-blocks, 128 bytes of a token's output row, which that kernel stores together as
// whole lines whenever both groups fall into its strip -- while the unit that balances the wavefronts stays a run.
inline bool plan_paired(int32_t R, bool chunked) { return R == 16 && !chunked; }
__host__ __device__ inline int64_t plan_block(int64_t g, int w, int i, int waves, int nacc, bool paired) {
    if (paired) return (g >> 1) * (4 * waves) + 4 * w + 2 * (int)(g & 1) + i;
    return (g * waves + w) * nacc + i;
}
__host__ __device__ inline void plan_entry(int64_t b, int waves, int nacc, bool paired, int64_t &g, int &w, int &i) {
    if (paired) {
        const int r = (int)(b % (4 * waves));
        g = 2 * (b / (4 * waves)) + ((r >> 1) & 1);
        w = r >> 2;
        i = r & 1;
    } else {
        const int64_t run = b / nacc;
        g = run / waves;
        w = (int)(run % waves);
        i = (int)(b % nacc);
    }
}
// Groups of a plan.
inline int64_t plan_groups(int64_t B, int waves, int nacc, bool paired) {
    if (paired) return 2 * ((B + 4 * waves - 1) / (4 * waves));
    return (B + (int64_t)waves * nacc - 1) / ((int64_t)waves * nacc);
}
// Steps of a row-block of the plan, over all its chunks, by the caller's bound on the kept columns: those of its stored
// row-block, or of the union of two that are kept independently.
inline double plan_steps(const TiledArgs &a) {
    double cols = (double)a.capacity_cols / (double)(a.M / a.stored_R);
    if (a.stored_R < a.R) cols = 2.0 * cols - (cols < (double)a.N ? cols * cols / (double)a.N : cols);
    return cols / 32.0 + 0.5 * plan_chunks(a.N, a.R, a.M).n;
}
// Workgroups of the kernels for many tokens: `units` per token tile.  Workgroup ids go round the 8 XCDs, each with an L2 and
// 32 compute units of its own, so the units of a tile, which read the same rows of X, take ids of one remainder modulo 8
// (with less than 8 tiles they spread over all XCDs).  When the units of 25 or 33
// tiles went to all XCDs, X came from memory eight times: 1024 x 4096 at 1.43x, 1537 tokens 49.8 us, now 44.1;
// 768 x 3072 in 8-row blocks at 3x, 1537 tokens 31.5 and 27.9.
// With the units of few tiles more than an XCD can hold, the XCD that has one tile more than the others decides (9 tiles: two
// on one XCD), and all XCDs are given all tiles if that saves rounds and not only the difference in memory traffic: 32768 x 1024 at 5x, 1100
// tokens 44.6 us by XCD and 38.0 spread, 32768 x 2048 at 20x, 513 tokens 45.1 and 34.0, 30528 x 768 at 20x, 513 tokens 18.6 and 15.7.
// Rounds of such a launch whose workgroups fill a compute unit each, by XCD and over all of them.
inline int64_t tile_rounds_xcd(int64_t tiles, int64_t units) { return ((tiles + 7) / 8 * units + 31) / 32; }
inline int64_t tile_rounds_all(int64_t tiles, int64_t units) { return (tiles * units + 255) / 256; }
constexpr double kTileSpread = 1.12;  // what a round takes longer when all XCDs read all tiles
inline bool tile_spread(int64_t tiles, int64_t units) {
    return tiles < 8 || kTileSpread * (double)tile_rounds_all(tiles, units) < (double)tile_rounds_xcd(tiles, units);
}
inline double tile_rounds(int64_t tiles, int64_t units) {
    if (tiles < 8) return (double)tile_rounds_all(tiles, units);
    return tile_spread(tiles, units) ? kTileSpread * (double)tile_rounds_all(tiles, units) : (double)tile_rounds_xcd(tiles, units);
}
inline int64_t tile_workgroups(int64_t tiles, int64_t units, bool spread) {
    return (spread || tiles < 8 ? tiles : (tiles + 7) / 8 * 8) * units;
}
__device__ inline void tile_place(uint32_t id, int32_t tiles, int32_t units, int32_t spread, int32_t &tile, int32_t &unit) {
    if (tiles < 8) {
        tile = (int32_t)(id / (uint32_t)units);
        unit = (int32_t)(id % (uint32_t)units);
    } else if (spread) {  // (a round's workgroups share the weights of few units)
        tile = (int32_t)(id % (uint32_t)tiles);
        unit = (int32_t)(id / (uint32_t)tiles);
    } else {
        const uint32_t at = id >> 3, rows = ((uint32_t)tiles + 7u) >> 3;
        tile = (int32_t)(at % rows * 8u + (id & 7u));  // (may lie past the last tile)
        unit = (int32_t)(at / rows);
    }
}
// Groups of the plan that a workgroup of the kernel for narrow layers walks.  A workgroup fills a compute unit, so
// what counts is the rounds that a launch takes, times a workgroup's copy-in and walk
// (microseconds fitted to measurements).  Enough strips to reach 256 workgroups was the rule once: 65 token tiles of a
// 4096 x 1024 layer were 260 workgroups in two rounds, 68 us at 1.43x, and are 195 in one, 46.
// Below 256 columns that rule stays, with the units over all XCDs: a workgroup is little more than its start and its output
// there, which the estimate does not know.  5632 x 32, 5691 tokens 25.0 us before, 29.4 by the estimate; 9792 x 40, 2363 tokens
// 15.0 and 19.5; of 3807 calls of up to 248 columns 118 were more than 8 % slower by it, for 2.6 % on average.
constexpr int64_t kNarrowColumns = 256;
inline double steploop_walk_us(int64_t tiles, int64_t NG, int64_t gps, int64_t N, double steps) {
    return tile_rounds(tiles, (NG + gps - 1) / gps) * (0.0016 * (double)N + 0.42 * steps * (double)gps);
}
inline int64_t steploop_groups(int64_t tiles, int64_t NG, int64_t N, double steps) {
    // (the fp32 bias of a strip's quads fills what LDS the tile leaves: 4 KiB per two groups, and a strip of gps groups
    // touches at most gps / 2 + 1 of them)
    constexpr int64_t max_gps = 14;
    if (N < kNarrowColumns) {
        const int64_t strips = (256 + tiles - 1) / tiles;
        const int64_t gps = strips < NG ? (NG + strips - 1) / strips : 1;
        return gps < max_gps ? gps : max_gps;
    }
    int64_t best = NG < max_gps ? NG : max_gps;
    for (int64_t gps = best - 1; gps >= 1; --gps)
        if (steploop_walk_us(tiles, NG, gps, N, steps) < steploop_walk_us(tiles, NG, best, N, steps)) best = gps;
    return best;
}
// The kernel that streams X: how many of a group's eight streams a workgroup takes, one per computing wavefront.  With
// fewer of them a wavefront's steps come sooner, and they are six deep (0.77 and 0.70 of the time with 4 and 2), so a launch
// that fits one round of 256 workgroups that way is shorter; a second round costs more than that.  Measured with 8 / 4 / 2, us:
// 1024 x 4096 at 5x, 2048 tokens 24.3 / 18.4 / 17.3, 4096 tokens 24.9 / 20.1 / 32.8 (2 rounds), 8192 tokens 28.8 / 40.6 / 69.6;
// at 1.43x, 4096 tokens 51.8 / 39.4 / 68.3; 2048 x 1536 at 3x, 1024 tokens 13.5 / 10.2 / 9.7; 768 x 768 in 8-row blocks at 3x,
// 4099 tokens 11.8 / 9.3 / 15.2.
inline double stream_load(int64_t tiles, int64_t B, int waves) {
    const int64_t streams = (B + 3) / 4;
    return tile_rounds(tiles, (streams + waves - 1) / waves) * (waves == 8 ? 1.0 : (waves == 4 ? 0.77 : 0.70));
}
inline int stream_waves(int64_t tiles, int64_t B) {
    int best = 8;
    for (int w = 4; w >= 2; w /= 2)
        if (stream_load(tiles, B, w) < stream_load(tiles, B, best)) best = w;
    return best;
}
// The kernel on the compact storage: row-blocks of a workgroup's strip.  Enough strips to give every compute unit a workgroup, none of
// fewer than 4 row-blocks or of more than its part of blk_ptr in LDS has room for.
constexpr int kMaxStripBlocks = 1024;
inline int64_t canonical_strip(int64_t ntiles, int64_t B) {
    int64_t strips = (256 + ntiles - 1) / ntiles;
    if (strips > (B + 3) / 4) strips = (B + 3) / 4;
    const int64_t blocks = (B + strips - 1) / strips;
    return blocks < kMaxStripBlocks ? blocks : kMaxStripBlocks;
}
// Steps the planned kernel may read past the last step of the storage (values unused).
int plan_slack_steps();

// Placement of X column c inside a 16-token sub-tile held in LDS, shared by the copy-in of the
// tiled kernels and by the plan builder: byte offset of token quad p (tokens 4p .. 4p+3).
__host__ __device__ inline uint32_t lds_col_offset(uint32_t c, uint32_t p) {
    const uint32_t row = (c & ~31u) | ((c >> 2) & 7u) | ((c & 3u) << 3);
    return row * 32u + ((p ^ ((c >> 5) & 3u)) << 3);
}
// The same for the 64-token tiles (four sub-tiles, up to 1024 columns) of the planned kernels: columns 0 .. 511
// fill the first 64 KiB of the tile and columns 512 .. 1023 the second, and sub-tile u of either half lies
// u * kSubStride4 bytes further on -- all four sub-tiles of a column are then within the 64 KiB that the immediate
// offset of an LDS instruction reaches, so one address register per column serves the whole tile.
constexpr uint32_t kSubStride4 = 16384u;
__host__ __device__ inline uint32_t lds_col_offset4(uint32_t c, uint32_t p) {
    return (c >> 9) * 65536u + lds_col_offset(c & 511u, p);
}
// LDS bank group (8 banks of 4 bytes = one 32-byte row) that column c lands in.
__host__ __device__ inline uint32_t lds_bank_group(uint32_t c) { return (c >> 2) & 7u; }

// The layer in single precision on its compact storage, from a tile of X in LDS (bsp_linear_f32.hip): whether these
// arguments can take it, whether it is the faster one for these sizes, and its launch.  No argument checks of its own.
bool linear_f32_tile_pays(int64_t T, int64_t M, int64_t N, int32_t R, int64_t capacity_cols);
bool linear_f32_tile_supported(int64_t N, int32_t k_align, const int32_t *col_idx, const float *vals);
int launch_linear_f32_tile(const float *X, int64_t T, int64_t M, int64_t N, int32_t R, const int32_t *blk_ptr,
                           const int32_t *col_idx, const float *vals, const float *bias, float *Y, hipStream_t s);

// The transposed product as a dense one on the expanded matrix (bsp_linear_t_expand.hip), for 16-bit types: whether
// these arguments can take it, the workspace it needs, and its launch.  No argument checks of its own.
bool linear_t_expand_supported(int udt, int64_t M, int64_t N, int32_t R);
size_t linear_t_expand_bytes(int64_t M, int64_t N, int32_t R);
int linear_t_expand(const void *U, int udt, int64_t T, int64_t M, int64_t N, int32_t R, const int32_t *blk_cnt,
                    const int32_t *blk_ptr, const int32_t *col_idx, const void *vals, const void *bias, void *Z,
                    void *ws, hipStream_t s);

// The layer as a dense product on the expanded matrix (same file), for 16-bit types, N % 8 == 0, X aligned to 16 bytes:
// the workspace it needs, whether it is the faster one for these sizes, and its launch.  No argument checks of its own.
size_t linear_expand_bytes(int64_t M, int64_t N, int32_t R);
bool linear_expand_pays(int64_t T, int64_t M, int64_t N, int32_t R, int64_t capacity_cols);
int linear_expand(const void *X, int xdt, int64_t T, int64_t M, int64_t N, int32_t R, const int32_t *blk_cnt,
                  const int32_t *blk_ptr, const int32_t *col_idx, const void *vals, const void *bias, void *Y, void *ws,
                  hipStream_t s);

// The weight gradient as a dense product of which the kept positions are written (bsp_linear_dvals_dense.hip).  colstart[b][j]: kept
// columns of row-block b below 128 j, j = 0 .. ceil(N / 128).  No argument checks of its own.
struct DvalsDense {
    const uint16_t *X, *dY;
    int xdt;
    int64_t T, M, N;
    int32_t R;
    const int32_t *blk_cnt, *blk_ptr, *col_idx, *colstart;
    int64_t capacity_cols;
    float *partial;
    void *D;
    int gdt;
    hipStream_t s;
};
struct DvalsDenseChoice {
    int shape, S, per, chain;  // tile, runs of the tokens, stages of a run, stages of a chain of its sums
    double us;                 // the estimate
};
// How far fp32 sums are from their values that chains of matrix instructions over `chain` stages of 32 tokens make, added up one after the
// other: see bsp_linear_dvals_dense.hip.
inline int64_t dvals_sums_error(int64_t chain, int64_t chains) { return 27 * chain + 10 * (chains - 1); }
// (error: what the sums may be off)
DvalsDenseChoice dvals_dense_choose(int64_t T, int64_t M, int64_t N, int32_t R, int64_t capacity_cols, int64_t partial_floats, int64_t error);
int launch_dvals_dense(const DvalsDense &a, const DvalsDenseChoice &c);

}  // namespace bsp
