// A 16 x 16 tile of products of bf16 rows that come straight from memory into the registers of the matrix instruction, the
// contraction shared by the wavefronts of a workgroup: for the calls that stream one operand once and meet few rows of
// the other (gate, y and segment logits of the decoding calls).
#pragma once

#include "cp_internal.hpp"

#include <type_traits>

namespace cph {

typedef __bf16 tile16_bf16x8_t __attribute__((ext_vector_type(8)));
typedef float tile16_acc_t __attribute__((ext_vector_type(4)));

// 16 bytes at any even address (one load instruction all the same): H, W, U and G are only promised to be bf16 arrays
typedef uint32_t u32x4_any_t __attribute__((ext_vector_type(4), aligned(2)));
typedef uint32_t tile16_u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ tile16_u32x4_t load16(const bf16_t *p) { return *reinterpret_cast<const u32x4_any_t *>(p); }

// acc[e] += a b[e]^T over N blocks of 64 columns, the first at element k0 and `stride` elements apart: all loads, then the
// products.  (A choice between two blocks lets the compiler move the loads of the second behind it, next to their use.)
template <int N, int NB>
__device__ __forceinline__ void tile16_blocks(const bf16_t *a, const bf16_t *const (&b)[NB], int k0, int stride, tile16_acc_t (&acc)[NB])
{
    tile16_u32x4_t av[N][2], bv[N][NB][2];
#pragma unroll
    for (int u = 0; u < N; ++u)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            av[u][c] = load16(a + k0 + u * stride + 8 * c);
#pragma unroll
            for (int e = 0; e < NB; ++e) bv[u][e][c] = load16(b[e] + k0 + u * stride + 8 * c);
        }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < N; ++u)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int e = 0; e < NB; ++e)
                acc[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(tile16_bf16x8_t, av[u][c]),
                                                                 __builtin_bit_cast(tile16_bf16x8_t, bv[u][e][c]), acc[e], 0, 0, 0);
}

// acc[e] += this wavefront's share of a b[e]^T.  Lane l passes its rows (number l % 16 of the 16 of either side) from element
// 16 (l / 16) on.  The wavefronts take blocks of 64 columns in turn, AHEAD of their own in flight; a lane loads 32
// consecutive bytes of its row per block, so that four lanes cover a cache line; the order of the columns inside a block is
// the same permutation for both operands.  d is a multiple of 64.
// AHEAD: four where the workgroups are few and walk their rows for long (arg-max counts at T = 16384, d = 4096, r = 8: the
// whole call 41.8 us with one, 34.8 with four); one where eight and more workgroups share a compute unit and hide each
// other's latency: registers for more of them in flight cost more workgroups than they bring loads (draft call at T = 1,
// n = 16, r = 1, d = 2048, V = 32000, with one / two / four: 71 / 76 / 80 us; T = 1024, n = 4, r = 8, d = 256, V = 100:
// 122 / 124 / 137 us).
template <int WAVES, int AHEAD, int NB>
__device__ __forceinline__ void tile16_products(const bf16_t *a, const bf16_t *const (&b)[NB], int d, int wave, tile16_acc_t (&acc)[NB])
{
    constexpr int kStride = WAVES * 64;
    int k = wave * 64, left = (d / 64 - wave + WAVES - 1) / WAVES;      // blocks of this wavefront
    for (; left >= AHEAD; left -= AHEAD, k += AHEAD * kStride) tile16_blocks<AHEAD>(a, b, k, kStride, acc);
    if (AHEAD > 3 && left == 3) tile16_blocks<3>(a, b, k, kStride, acc);
    else if (AHEAD > 2 && left == 2) tile16_blocks<2>(a, b, k, kStride, acc);
    else if (AHEAD > 1 && left == 1) tile16_blocks<1>(a, b, k, kStride, acc);
}
// The same for NA x NB tiles: acc[c][g] += a[c] b[g]^T, AHEAD blocks of every row in flight.
template <int WAVES, int AHEAD, int NA, int NB>
__device__ __forceinline__ void tile16_products_2d(const bf16_t *(&a)[NA], const bf16_t *(&b)[NB], int d, int wave,
                                                   tile16_acc_t (&acc)[NA][NB])
{
    constexpr int kStride = WAVES * 64;
    auto blocks = [&](int k0, auto count) {
        constexpr int N = decltype(count)::value;
        tile16_u32x4_t av[N][NA][2], bv[N][NB][2];
#pragma unroll
        for (int u = 0; u < N; ++u)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
#pragma unroll
                for (int e = 0; e < NA; ++e) av[u][e][c] = load16(a[e] + k0 + u * kStride + 8 * c);
#pragma unroll
                for (int e = 0; e < NB; ++e) bv[u][e][c] = load16(b[e] + k0 + u * kStride + 8 * c);
            }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < N; ++u)
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int e = 0; e < NA; ++e)
#pragma unroll
                    for (int f = 0; f < NB; ++f)
                        acc[e][f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(tile16_bf16x8_t, av[u][e][c]),
                                                                            __builtin_bit_cast(tile16_bf16x8_t, bv[u][f][c]), acc[e][f], 0, 0, 0);
    };
    int k = wave * 64, left = (d / 64 - wave + WAVES - 1) / WAVES;      // blocks of this wavefront
    for (; left >= AHEAD; left -= AHEAD, k += AHEAD * kStride) blocks(k, std::integral_constant<int, AHEAD>());
    for (; left > 0; --left, k += kStride) blocks(k, std::integral_constant<int, 1>());
}
// row (of a) of element v of the result in a lane; the column (of b) is l % 16
__device__ __forceinline__ int tile16_row(int v, int lane) { return 4 * (lane >> 4) + v; }

}  // namespace cph
