// Which tile and how many splits along K a product of the plain path takes (host only; no HIP dependency, so that the
// choice can be checked on the CPU).
#pragma once
#include <cstddef>

namespace cph {

enum F32TileKind { kF32LargeTile = 0, kF32MidTile = 1, kF32SmallTile = 2 };

inline int f32_tile_edge(int kind) { return kind == kF32LargeTile ? 128 : kind == kF32MidTile ? 64 : 32; }
inline int f32_slots(int kind, long N)      // column slots of the statistics epilogue (tile columns times WN)
{
    const int e = f32_tile_edge(kind);
    return (int)((N + e - 1) / e) * (kind == kF32SmallTile ? 1 : 2);
}

// Tile and number of K-splits of an M x N x K contraction, or of up to three that share a launch (and then the tile).
struct F32Plan {
    int kind, splits;
    size_t scratch(long M, long N) const { return splits > 1 ? ((size_t)splits * M * N * 4 + 255) / 256 * 256 : 0; }
};
struct F32Shape {
    long M, N, K;
    long batch = 1;
};
// The choice is the one with the least time in a model with measured constants (of K-steps of 32 for the 128-wide tile): rounds of tiles over the compute units
// at the average cost of a tile, not less than the longest tile alone on its compute unit, plus, if a sum is split, the
// pass that adds the parts.  Cycles per k-value of one tile, alone and with a second tile on the compute unit,
// at 2.4 GHz: 128-wide 171 / 156, 64-wide 51 / 44, 32-wide 16 / 13.3 (at K = 4096, TFLOP/s on 128 and on 512 tiles: 59 / 125,
// 46 / 107, 29 / 80; on 2048 tiles the 64-wide reach 112 and the 32-wide 92); a launch costs about 4 us whatever it does.
inline void f32_plan(const F32Shape *shape, int count, bool may_split, F32Plan *out)
{
    constexpr double kCus = 256, kFixed[3] = {6000, 5000, 3000}, kReduceFixed = 10000, kBytesPerCycle = 2000;
    constexpr double kAlone[3] = {171, 51, 16}, kShared[3] = {156, 44, 13.3};
    constexpr int kSplits = 5;                              // 1, 2, 4, 8, 16
    constexpr double kMaxScratch = 128 << 20;               // bytes of partial sums per launch
    double best = -1;
    for (int kind = 0; kind < 3; ++kind) {
        const long e = f32_tile_edge(kind);
        int choice[3] = {0, 0, 0};
        for (;;) {
            double units = 0, work = 0, longest = 0, reduce = 0, scratch = 0;
            for (int i = 0; i < count; ++i) {
                const F32Shape &q = shape[i];
                const int s = 1 << choice[i];
                const double n = (double)((q.M + e - 1) / e) * (double)((q.N + e - 1) / e) * s * q.batch, k = (double)q.K / s;
                units += n;
                work += n * (k * kShared[kind] + kFixed[kind]);
                longest = longest > k ? longest : k;
                if (s > 1) {
                    reduce += (s + 1.0) * q.M * q.N * 4 / kBytesPerCycle;
                    scratch += (double)s * q.M * q.N * 4;
                }
            }
            const double rounds = (double)(long)((units + kCus - 1) / kCus);
            double t = rounds * work / units;
            const double alone = longest * kAlone[kind] + kFixed[kind];
            if (t < alone) t = alone;
            if (reduce > 0) t += kReduceFixed + reduce;
            if (scratch <= kMaxScratch && (best < 0 || t < best)) {
                best = t;
                for (int i = 0; i < count; ++i) out[i] = F32Plan{kind, 1 << choice[i]};
            }
            int i = 0;                                      // the next combination of splits of at least 256 k-values
            while (i < count && (!may_split || ++choice[i] == kSplits || (shape[i].K >> choice[i]) < 256)) choice[i++] = 0;
            if (i == count) break;
        }
    }
}
inline F32Plan f32_plan(long M, long N, long K, bool may_split, long batch = 1)
{
    const F32Shape q{M, N, K, batch};
    F32Plan p;
    f32_plan(&q, 1, may_split, &p);
    return p;
}

// Whether a launch of 128-wide tiles whose operands are both K-contiguous takes K-steps of 16 instead of 32: three workgroups share a
// compute unit then instead of two, so that a round is 768 tiles instead of 512.  `narrow` of the operands are bfloat16, whose rows
// are then read 32 bytes at a time; `vec`: four elements per load.  Products of K = 512 (vec) and 511 or 445 (not), us, K-step 32 / 16:
//   tiles           256        512        768       1024       1152       1280       1536       2048       2304       2560       3072       4032
//   fp32        46 / 46    82 / 79  149 / 119  157 / 208  211 / 210  220 / 212  230 / 221  305 / 312  357 / 324  377 / 397  452 / 428  594 / 573
//   not vec     47 / 46    88 / 80  158 / 122  167 / 213  201 / 216  231 / 219  243 / 230  323 / 320  375 / 335  405 / 390  482 / 443  632 / 587
//   one bf16    49 / 52    79 / 82  147 / 119  153 / 215  217 / 217  218 / 220  223 / 227  295 / 320  359 / 334  365 / 413  438 / 443  580 / 604
//   not vec     47 / 50    81 / 77  147 / 114  152 / 202  212 / 206  215 / 209  222 / 217  293 / 306  355 / 321  363 / 391  432 / 424  570 / 572
//   both bf16   49 / 51    78 / 81  147 / 119  150 / 213  216 / 218  217 / 221  220 / 226  292 / 325  358 / 336  362 / 401  433 / 444  582 / 608
// (K = 1024, fp32, 1088 to 1216 tiles: 359 to 367 / 394.)  Beyond a round the tiles that are left go to the compute units that are free
// first, three or two at a time, so that a few of them cost as much as many; rounds have smeared out after five of 512.
inline bool f32_short_steps(long tiles, int narrow, bool vec)
{
    const long by2 = 2 * ((tiles + 511) / 512), by3 = 3 * ((tiles + 767) / 768);        // rounds, in tiles of a compute unit
    if (narrow == 2 || (narrow == 1 && vec)) return tiles > 512 && 21 * by3 < 20 * by2;
    if (narrow == 0 && tiles > 2560) return true;
    return by3 < by2 || (by3 == by2 && tiles > 1216) || (tiles <= 512 && (narrow == 0 || tiles > 256));
}

}  // namespace cph
