// Logits kept by the forward pass for the backward pass (CP_HEAD_KEEP_LOGITS), matrix-core path.
//
// The forward product's epilogue writes zs[m, v] = fp16(z[m, v] - ref[m, v / 128]) with ref the maximum of row m
// over its block of 128 columns, which is also the first half of the (max, sum of exponentials) pair of that
// block in part[m, parts].  With the row's log-normaliser lse[m] the log-probability of eq. 5 is
//     log P[m, v] = zs[m, v] - (lse[m] - ref[m, v / 128]).
// Relative to the block maximum the large probabilities of a row sit near zero, where fp16 resolves 2^-12 or
// better; an overflow to -inf is the exact zero that the exponential of the true value rounds to as well.
//
// k_dz_from_kept turns a chunk of kept logits into logit gradients in bf16, stored block by block (blocked64_index), which
// is what the dY and dU products of the backward pass both read.  What the gradient is (training loss, fine-tuning loss)
// comes in as a rule.
#pragma once
#include "gemm_nt.hpp"

namespace cph {

constexpr int kKeptTile = 128;      // rows and columns of a workgroup's tile; its columns are one block of `part`
constexpr int kKeptBlock = 256;

// two fp32 values -> two 16-bit floats (IEEE binary16, round to nearest even) in one register (a in the low half)
__device__ __forceinline__ uint32_t f32x2_to_f16x2(float a, float b)
{
    typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    const f32x2_t v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, f16x2_t));
}

typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));

struct KeptLogits {
    const uint16_t *zs;      // [rows, ld] fp16 bits
    const float2 *part;      // [rows, parts] {block maximum, -}
    long ld;
    int parts;
};

// log P for 8 consecutive columns col .. col + 7 (one block of 128) of row m, given the row's log-normaliser
__device__ __forceinline__ void kept_log_probs(const KeptLogits &k, size_t m, int col, float lse, float (&lp)[8])
{
    const float off = lse - k.part[m * k.parts + col / kKeptTile].x;
    const f16x8_t z = __builtin_bit_cast(f16x8_t, *reinterpret_cast<const u32x4_t *>(k.zs + m * k.ld + col));
#pragma unroll
    for (int j = 0; j < 8; ++j) lp[j] = (float)z[j] - off;
}

// A workgroup takes 128 rows x 128 columns of the chunk.  A thread owns Rule::RT consecutive rows (2, 4 or 8) and
// 8 consecutive columns: it reads their kept logits with 16-byte loads, lets the rule turn the log-probabilities
// into gradients and writes them with 16-byte stores.  HBM bound, 4 bytes per logit.  The rows from Mc up to Mcp are zeroed.
//
// Rule: static constexpr int RT; and
//   void operator()(int row, int nrows, int col, int V, const float4 (&info)[RT], const float (&lp)[RT][8],
//                   float (&g)[RT][8]) const
// with row chunk-relative, rows row .. row + nrows - 1 valid (info = rowinfo of those rows, info.x their
// log-normaliser), g preset to zero; entries of columns >= V must stay zero.
// kept: rows of the chunk (already offset); rowinfo chunk-relative.  streamed: the gradients are written past the caches.
template <class Rule>
__global__ void __launch_bounds__(kKeptBlock) k_dz_from_kept(KeptLogits kept, const float4 *__restrict__ rowinfo,
                                                             Rule rule, int Mc, int Mcp, int V, int Vp,
                                                             bf16_t *__restrict__ dZ, int streamed, int tiles_c)
{
    constexpr int RT = Rule::RT;
    const int tc = blockIdx.x % tiles_c, tr = blockIdx.x / tiles_c;
    const int t = threadIdx.x, cg = t & 15;
    const int col = tc * kKeptTile + cg * 8;
    const bool col_in = col < Vp;                        // Vp is a multiple of 8: all eight columns or none
#pragma unroll
    for (int pass = 0; pass < kKeptTile / (16 * RT); ++pass) {
        const int rg = pass * 16 + (t >> 4);             // group of RT rows inside the tile
        const int row = tr * kKeptTile + RT * rg;
        float g[RT][8];
#pragma unroll
        for (int h = 0; h < RT; ++h)
#pragma unroll
            for (int k = 0; k < 8; ++k) g[h][k] = 0.f;
        if (!col_in || row >= Mcp) continue;
        if (row < Mc) {
            const int nrows = Mc - row < RT ? Mc - row : RT;
            float4 info[RT];
            float lp[RT][8];
#pragma unroll
            for (int h = 0; h < RT; ++h) {
                info[h] = rowinfo[row + (h < nrows ? h : 0)];
                kept_log_probs(kept, (size_t)(row + (h < nrows ? h : 0)), col, info[h].x, lp[h]);
            }
            rule(row, nrows, col, V, info, lp, g);
        }
#pragma unroll
        for (int h = 0; h < RT; ++h)
            if (row + h < Mcp) {
                u32x4_t out;
#pragma unroll
                for (int k = 0; k < 4; ++k) out[k] = f32x2_to_bf16x2(g[h][2 * k], g[h][2 * k + 1]);
                u32x4_t *at = reinterpret_cast<u32x4_t *>(dZ + blocked64_index((size_t)(row + h), col, Vp));
                if (streamed) __builtin_nontemporal_store(out, at);
                else *at = out;
            }
    }
}

// kept: all rows (not offset); the chunk is rows m0 .. m0 + Mc - 1; rowinfo chunk-relative; dZ has rows of Vp.
template <class Rule>
inline void launch_dz_from_kept(const KeptLogits &kept, size_t m0, const float4 *rowinfo, const Rule &rule, int Mc, int Mcp,
                                int V, bf16_t *dZ, int Vp, hipStream_t st)
{
    const int tiles_c = (Vp + kKeptTile - 1) / kKeptTile;
    const size_t tiles_r = ((size_t)Mcp + kKeptTile - 1) / kKeptTile;
    // algorithmic traffic: the logits read once, the gradients written once
    ProfileScope scope("dz_from_kept", (double)Mc * Vp * 4.0, st);
    const KeptLogits chunk{kept.zs + m0 * kept.ld, kept.part + m0 * kept.parts, kept.ld, kept.parts};
    k_dz_from_kept<Rule><<<(unsigned)(tiles_r * tiles_c), kKeptBlock, 0, st>>>(chunk, rowinfo, rule, Mc, Mcp, V, Vp, dZ,
                                                                               streamed_store((size_t)Mc * Vp * 2) ? 1 : 0, tiles_c);
}

}  // namespace cph
