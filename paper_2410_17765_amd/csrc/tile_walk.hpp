// Index maps of the GEMM launches (host and device; no HIP dependency, so that they can be checked on the CPU):
// workgroup id -> output tile, and the block-by-block operand layout.
#pragma once
#include <cstddef>
#if !defined(__HIPCC__)
#define CPH_HD inline
#else
#define CPH_HD __host__ __device__ __forceinline__
#endif

// Workgroup id -> output tile.  Consecutive workgroup ids go round-robin over the 8 XCDs: XCD x runs ids x, x+8, ...
// The tile rows are cut into bands of 8*GM rows; within a band XCD x takes rows [x*GM, (x+1)*GM) and walks them
// column by column, so that the tiles in flight on one XCD share GM + 32/GM operand panels in its L2 and all eight
// XCDs sweep the same columns at the same time whatever the number of tile rows is (the B panels, common to all of
// them, then come out of the last-level cache once for the eight; with per-XCD ranges that start at different
// columns a product with a ragged number of tile rows ran 5 % slower).  The rows left after the last whole band are
// dealt as equal contiguous ranges of the same walk.
struct TileWalk {
    int band_tiles;      // tiles one XCD takes from the whole bands
    int rest_first_m;    // first tile row after the whole bands
    int rest_per_xcd;    // tiles one XCD takes from the rest
};
CPH_HD TileWalk tile_walk(int tiles_m, int tiles_n, int GM)
{
    const int bands = tiles_m / (8 * GM);
    const int rest_rows = tiles_m - bands * 8 * GM;
    return {bands * GM * tiles_n, bands * 8 * GM, (rest_rows * tiles_n + 7) / 8};
}
CPH_HD bool tile_of_block(int bid, int tiles_m, int tiles_n, int GM, int &tm, int &tn)
{
    const TileWalk w = tile_walk(tiles_m, tiles_n, GM);
    const int x = bid & 7, j = bid >> 3;
    const int per_group = GM * tiles_n;
    if (j < w.band_tiles) {
        const int band = j / per_group, in = j - band * per_group;
        tm = (band * 8 + x) * GM + in % GM;
        tn = in / GM;
        return true;
    }
    const int lid = x * w.rest_per_xcd + (j - w.band_tiles);
    const int rest_rows = tiles_m - w.rest_first_m;
    if (j - w.band_tiles >= w.rest_per_xcd || lid >= rest_rows * tiles_n) return false;
    const int group = lid / per_group;
    const int first_m = group * GM;
    const int gsize = (rest_rows - first_m < GM ? rest_rows - first_m : GM);
    const int in = lid - group * per_group;
    tm = w.rest_first_m + first_m + in % gsize;
    tn = in / gsize;
    return true;
}
// Workgroups of a launch: a multiple of 8, at most 7 of them without a tile.
inline int gemm_grid(int tiles_m, int tiles_n, int GM)
{
    const TileWalk w = tile_walk(tiles_m, tiles_n, GM);
    return 8 * (w.band_tiles + w.rest_per_xcd);
}

// The last, partial round of a launch, split along K.  A launch of G workgroups runs in rounds of `slots` (the
// workgroups the chip holds at a time); the G % slots of the last round leave the rest of the chip idle for a whole
// tile's time (264 tiles: 8 busy of 256).  Their K-steps are dealt to `parts` workgroups each, which leave fp32 partial
// tiles in scratch, and a small launch adds those up in order and stores them.  Measured at T = 1500, d = 768, V = 50257,
// n = 3, r = 5: dY (264 tiles, 786 K-steps) 2416 -> 1336 us, dU (591 tiles) 1610 -> 1385, dH (18 tiles, 180 K-steps) 238 -> 60.
struct SplitPlan {
    int first;      // workgroups before this one compute whole tiles
    int tail;       // workgroups of the last round (a multiple of 8, as `first` is: a part stays on its tile's XCD)
    int parts;      // workgroups per tile of the last round; 1: nothing is split
};
constexpr int kMaxSplitItems = 512;
// Estimated times in us, measured on 256 x 256 tiles: a K-step 1.6, the extra launch 6, an item's partial tile written and
// read back 0.13 (256 KB each way at about 4 TB/s).  A part is at least four K-steps long.
inline SplitPlan split_plan(int grid, int slots, int k_steps, int max_items)
{
    SplitPlan best{grid / slots * slots, grid % slots, 1};
    double least = 1.6 * k_steps;
    for (int parts = 2; parts * best.tail <= max_items && parts * 4 <= k_steps && best.tail; ++parts) {
        const int items = parts * best.tail, rounds = (items + slots - 1) / slots;
        const double t = rounds * 1.6 * ((k_steps + parts - 1) / parts) + 6.0 + 0.13 * items;
        if (t < least) { least = t; best.parts = parts; }
    }
    return best;
}
// Item i of the split round -> the workgroup id whose tile it works on, and its K-steps [k0, k1).
CPH_HD void split_item(const SplitPlan &p, int i, int k_steps, int &bid, int &part, int &k0, int &k1)
{
    part = i / p.tail;
    bid = p.first + i % p.tail;
    k0 = (int)((long)part * k_steps / p.parts);
    k1 = (int)((long)(part + 1) * k_steps / p.parts);
}

// Element (row, col) of a bf16 matrix stored block by block, [rows / 256][ld / 64][256][64] (ld a multiple of 64, the
// rows allocated up to a multiple of 256): the layout of the chunk's logit gradients, which two products read as their first
// operand.  Where its rows are the product's rows (ABL), a K-step of a tile is a block, 32 KB of consecutive memory; where they are
// what the product contracts over (ABL and AKM), a K-step is 64 rows of the tile's four blocks, 8 KB of consecutive memory of each.
CPH_HD size_t blocked64_index(size_t row, int col, long ld)
{
    return ((row >> 8) * (size_t)(ld >> 6) + (size_t)(col >> 6)) * 16384 + (row & 255) * 64 + (size_t)(col & 63);
}

// Rows of logit gradients held at a time: about 4 GiB of bf16 at V = 32000, i.e. 65536 rows.  Measured on the
// headline step: 2 GiB 450.4 ms, 4 GiB 447.9, 8 GiB 448.3 (the dU product gains from fewer accumulation passes
// over its fp32 output, the dz product loses about half of that).  A larger vocabulary keeps at least 32768
// rows, up to 8 GiB of them: the rows of a chunk are the contraction length of its dU product, and at 8192 rows
// (2 GiB at V = 128256) that product ran at 1.08 PFLOP/s against 1.25 at 32768.  The count is a multiple of 16
// tiles of 256 rows where possible, so that the d-wide products of a chunk (16 tile columns at d = 4096) fill
// all 256 compute units in whole rounds.  M: all rows; Vp: the vocabulary rounded up to 64; least: one tile of rows.
inline size_t backward_chunk_rows(size_t M, size_t Vp, bool least)
{
    constexpr size_t kTile = 256;
    size_t rows = ((size_t)1 << 32) / (Vp * 2);
    if (rows < 32768) {
        const size_t cap = ((size_t)1 << 33) / (Vp * 2);
        rows = cap < 32768 ? cap : 32768;
    }
    if (rows >= 16 * kTile) rows = rows / (16 * kTile) * (16 * kTile);
    else rows = rows / kTile * kTile;
    if (rows < kTile || least) rows = kTile;
    return rows < M ? rows : (M ? M : 1);
}

// First element of a token's row in the teacher logits [tokens, V] of a chunk: in 64 bits, because the tokens of a chunk are its
// rows over r, and 32768 rows of one expert times V pass 2^31 from V = 65537 on.
CPH_HD size_t teacher_row_start(int token, int V) { return (size_t)token * (size_t)V; }
