// Matrix-core path of the CP head loss (bf16 storage, d a multiple of 64).
//
// Forward:   gate -> Y = H W^T (hi/lo bf16) -> z = Y U^T with a running-statistics epilogue
//            (logits never stored) -> per-row log-normaliser and fp32 target logit -> mixture.
// Backward:  per bounded chunk of head rows: recompute z, epilogue writes dz in bf16 ->
//            dY = dz U and dU += dz^T Y; then dW = dY^T H, dH = dY W + G^T dg, dG = dg^T H.
// With CP_HEAD_KEEP_LOGITS the forward epilogue also keeps the logits as 16-bit floats and the backward
// pass reads them back instead of recomputing z (kept_logits.hpp).
// All products run through the one NT main loop of gemm_nt.hpp; operands that are not
// K-contiguous are transposed first (HBM-bound passes that cost a few percent of the GEMM time).
#include "gemm_nt.hpp"
#include "tile16.hpp"
#include "kept_logits.hpp"

#include <math.h>
#include <type_traits>

namespace cph {

namespace {

typedef TileCfg<256, 256, 2, 2> Cfg;
// the same tile with both operands K-major (the contraction index is their slow one)
typedef TileCfg<256, 256, 2, 2, true, true> CfgTN;
// A stored in blocks of 256 rows x 64 columns (the chunk's logit gradients as the dY product reads them)
typedef TileCfg<256, 256, 2, 2, false, false, true> CfgBlockedA;
// the same operand beside a K-major one (full heads: dH = dz F_sa)
typedef TileCfg<256, 256, 2, 2, false, true, true> CfgBlockedANN;
// and as the dU product reads it, K-major: the rows of dz are what it contracts over
typedef TileCfg<256, 256, 2, 2, true, false, true> CfgBlockedTN;
constexpr int kBlock = 256;


// ------------------------------------------------------------------------------------------
// epilogues
// ------------------------------------------------------------------------------------------

// bf16 store of the accumulators; optionally also the bf16 residual acc - bf16(acc), so that
// hi + lo carries the fp32 value to about 2^-17 relative.  N and ldc are multiples of 8.
struct EpiStoreBf16 {
    bf16_t *hi;
    bf16_t *lo;     // may be null
    long ldc;
    int M, N;
    static constexpr bool kSplittable = true;
    static __device__ __forceinline__ uint2 round4(f32x4_t a) { return make_uint2(f32x2_to_bf16x2(a[0], a[1]), f32x2_to_bf16x2(a[2], a[3])); }
    static __device__ __forceinline__ uint2 residual4(f32x4_t a, uint2 h)
    {
        return make_uint2(f32x2_to_bf16x2(a[0] - __uint_as_float(h.x << 16), a[1] - __uint_as_float(h.x & 0xFFFF0000u)),
                          f32x2_to_bf16x2(a[2] - __uint_as_float(h.y << 16), a[3] - __uint_as_float(h.y & 0xFFFF0000u)));
    }
    __device__ __forceinline__ void put(int row, int col, f32x4_t a) const
    {
        const size_t at = (size_t)row * ldc + col;
        const uint2 h = round4(a);
        *reinterpret_cast<uint2 *>(hi + at) = h;
        if (lo) *reinterpret_cast<uint2 *>(lo + at) = residual4(a, h);
    }
    template <class C>
    __device__ void run(f32x4_t (&acc)[C::TM16][C::TN16], int row0, int col0, int lane, int, int, char *) const
    {
        const RowsOut16<C, false> out(lane, row0, col0, M, N, hi, ldc), out_lo(lane, row0, col0, M, N, lo, ldc);
#pragma unroll
        for (int i = 0; i < C::TM16; ++i) {
            uint2 h[C::TN16];
#pragma unroll
            for (int j = 0; j < C::TN16; ++j) h[j] = round4(acc[i][j]);
            if (lo) {
                uint2 l[C::TN16];
#pragma unroll
                for (int j = 0; j < C::TN16; ++j) l[j] = residual4(acc[i][j], h[j]);
                out_lo.put(i, l);
            }
            out.put(i, h);
        }
    }
};

// fp32 store, optionally accumulating onto what is already there (chunked sums).  N, ldc multiples of 4.
struct EpiStoreF32 {
    float *C;
    long ldc;
    int M, N;
    int accumulate;
    static constexpr bool kSplittable = true;
    __device__ __forceinline__ void put(int row, int col, f32x4_t a) const
    {
        f32x4_t *o = reinterpret_cast<f32x4_t *>(C + (size_t)row * ldc + col);
        *o = accumulate ? a + *o : a;
    }
    template <class Cf>
    __device__ void run(f32x4_t (&acc)[Cf::TM16][Cf::TN16], int row0, int col0, int lane, int, int, char *) const
    {
        store_rows_f32<Cf>(acc, lane, row0, col0, M, N, C, ldc, accumulate != 0);
    }
};

// The logits of the columns past the vocabulary (only the last tile column has any) are set to -inf once, so that
// the statistics below need no per-element test: -inf never wins a maximum and its exponential is zero (a row with no
// valid column keeps the maximum -inf and the reference 0, as before).  Uniform for the wavefront.
template <class C>
__device__ __forceinline__ void mask_columns_past_vocabulary(f32x4_t (&acc)[C::TM16][C::TN16], int col0, int lane, int V)
{
    if (col0 + C::WTN <= V) return;
#pragma unroll
    for (int j = 0; j < C::TN16; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const bool past = col0 + acc_col(j, v, lane) >= V;
#pragma unroll
            for (int i = 0; i < C::TM16; ++i) acc[i][j][v] = past ? -INFINITY : acc[i][j][v];
        }
}

// Of block row i of a sub-tile (a lane has 4 TN16 columns of one row): the row's largest logit over the sub-tile, and the
// reference that its exponentials are taken against (the same, or 0 for a row with no valid column).
template <class C>
__device__ __forceinline__ void row_max(const f32x4_t (&acc)[C::TN16], float &mx, float &ref)
{
    mx = -INFINITY;
#pragma unroll
    for (int j = 0; j < C::TN16; ++j) mx = fmaxf(mx, fmaxf(fmaxf(acc[j][0], acc[j][1]), fmaxf(acc[j][2], acc[j][3])));
    mx = groups_max(mx);
    ref = (mx == -INFINITY) ? 0.f : mx;
}

// Running statistics of the logits (eq. 5 in log space): for every row of the wavefront's
// sub-tile the maximum and the sum of exp(z - max) over its columns.  One (max, sum) pair per
// row and per (tile column, wavefront column) goes to `part`; the logits themselves are dropped.
// A row of the sub-tile lives in the four lanes l % 16 + 16 k; the first of them writes the pair.  Where no column counts the maximum is
// -infinity and the sum 0; if the columns were NaN, which no maximum shows, it is NaN, and so is the row's log-normaliser.
struct EpiRowStats {
    float2 *part;   // [M, parts]
    int parts;      // tiles_n * WN
    int M, V;
    template <class C>
    __device__ void run(f32x4_t (&acc)[C::TM16][C::TN16], int row0, int col0, int lane, int wave, int tn, char *) const
    {
        const int slot = tn * C::WN + (wave % C::WN);
        mask_columns_past_vocabulary<C>(acc, col0, lane, V);
#pragma unroll
        for (int i = 0; i < C::TM16; ++i) {
            float mx, ref, s[4] = {0.f, 0.f, 0.f, 0.f};
            row_max<C>(acc[i], mx, ref);
#pragma unroll
            for (int j = 0; j < C::TN16; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) s[v] += __expf(acc[i][j][v] - ref);
            const float sum = groups_sum((s[0] + s[1]) + (s[2] + s[3]));
            const int r = row0 + acc_row(i, lane);
            if (lane < 16 && r < M) part[(size_t)r * parts + slot] = make_float2(mx, sum);
            __builtin_amdgcn_sched_barrier(0);      // one block row at a time: more of them spill registers
        }
    }
};

// The statistics of EpiRowStats, and the logits kept for the backward pass: zs[m, v] = fp16(z - ref) with ref
// the maximum of row m over the wavefront's 128 columns (the pair that goes to `part`).  Relative to that
// maximum the large probabilities of a row, which carry its gradient, sit near zero where fp16 resolves
// 2^-11 or better; a logit 16 below the maximum is kept to 2^-7, i.e. its probability to under one percent.
struct EpiRowStatsKeep {
    float2 *part;   // [M, parts]
    int parts;
    int M, V;
    uint16_t *zs;   // [M, ldzs]
    long ldzs;
    int Vp;         // columns of zs that are written (V rounded up to 64; those from V on hold junk)
    int streamed;   // written past the caches
    template <class C>
    __device__ void run(f32x4_t (&acc)[C::TM16][C::TN16], int row0, int col0, int lane, int wave, int tn, char *) const
    {
        static_assert(C::WTN == 128, "blocks of 128 columns");
        const int slot = tn * C::WN + (wave % C::WN);
        mask_columns_past_vocabulary<C>(acc, col0, lane, V);
        const RowsOut16<C, false> out(lane, row0, col0, M, Vp, zs, ldzs);
#pragma unroll
        for (int i = 0; i < C::TM16; ++i) {
            float mx, ref, s[4] = {0.f, 0.f, 0.f, 0.f};
            row_max<C>(acc[i], mx, ref);
            uint2 w[C::TN16];
#pragma unroll
            for (int j = 0; j < C::TN16; ++j) {
                float z[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    z[v] = acc[i][j][v] - ref;
                    s[v] += __expf(z[v]);
                }
                w[j] = make_uint2(f32x2_to_f16x2(z[0], z[1]), f32x2_to_f16x2(z[2], z[3]));
            }
            out.put(i, w, streamed != 0);
            const float sum = groups_sum((s[0] + s[1]) + (s[2] + s[3]));
            const int r = row0 + acc_row(i, lane);
            if (lane < 16 && r < M) part[(size_t)r * parts + slot] = make_float2(mx, sum);
            __builtin_amdgcn_sched_barrier(0);      // one block row at a time: more of them spill registers
        }
    }
};

// The statistics of EpiRowStats, and the fp32 logits themselves: for a pass over them while they are still a bounded chunk.
struct EpiRowStatsStore {
    float2 *part;   // [M, parts]
    int parts;
    int M, V;
    float *z;       // [M, ldz]
    long ldz;       // a multiple of 4, and the columns that are written (those from V on hold -inf)
    int streamed;   // written past the caches
    template <class C>
    __device__ void run(f32x4_t (&acc)[C::TM16][C::TN16], int row0, int col0, int lane, int wave, int tn, char *) const
    {
        const int slot = tn * C::WN + (wave % C::WN);
        mask_columns_past_vocabulary<C>(acc, col0, lane, V);
        store_lines_f32<C>(acc, lane, row0, col0, M, (int)ldz, z, ldz, streamed != 0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < C::TM16; ++i) {
            float mx, ref, s[4] = {0.f, 0.f, 0.f, 0.f};
            row_max<C>(acc[i], mx, ref);
#pragma unroll
            for (int j = 0; j < C::TN16; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) s[v] += __expf(acc[i][j][v] - ref);
            const float sum = groups_sum((s[0] + s[1]) + (s[2] + s[3]));
            const int r = row0 + acc_row(i, lane);
            if (lane < 16 && r < M) part[(size_t)r * parts + slot] = make_float2(mx, sum);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
};

// Softmax gradient (derivative of eq. 8/9 with respect to the logits), written in bf16, block by block (blocked64_index):
//   dz[m, v] = coef[m] * (exp(z - lse[m]) - 1[v = x_m]),  zero in the padding columns V..Vp-1 and the rows Mc..Mcp-1.
// One copy serves both products that read it: dY takes it as it lies and dU K-major (a second, transposed copy for dU
// was a third of this kernel's epilogue and of the HBM traffic of k_dz_from_kept, and more than the K-major loop costs).
struct EpiDz {
    bf16_t *dZ;
    long ldz;
    const float4 *rowinfo;   // chunk-relative: {lse, coef (zero for dropped factors), target as int bits, -}
    int Mc, Mcp, V, Vp;
    int streamed;            // written past the caches
    template <class C>
    __device__ void run(f32x4_t (&acc)[C::TM16][C::TN16], int row0, int col0, int lane, int, int, char *) const
    {
        // the values of the lane's eight rows in one go: loaded where they are used they were a chain of exposed cache misses
        float4 info[C::TM16];
#pragma unroll
        for (int i = 0; i < C::TM16; ++i) info[i] = rowinfo[min(row0 + acc_row(i, lane), Mc - 1)];
#pragma unroll
        for (int i = 0; i < C::TM16; ++i) asm volatile("" : "+v"(info[i].x), "+v"(info[i].y), "+v"(info[i].z));
        const RowsOut16<C, true> out(lane, row0, col0, Mcp, Vp, dZ, ldz);
        const int lcol = col0 + acc_col(0, 0, lane);
        const bool ragged = col0 + C::WTN > V;           // the same for the whole wavefront
#pragma unroll
        for (int i = 0; i < C::TM16; ++i) {
            // rows past the chunk hold zero logits: coefficient 0 and offset 0 keep their product finite
            const bool in = row0 + acc_row(i, lane) < Mc;
            const float cf = in ? info[i].y : 0.f, lse = in ? info[i].x : 0.f;
            float g[C::TN16][4];
#pragma unroll
            for (int j = 0; j < C::TN16; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v)     // z - lse first: exact where the logit is close to the log-normaliser (p close to 1)
                    g[j][v] = cf * __builtin_amdgcn_exp2f((acc[i][j][v] - lse) * kLog2e);
            // the one-hot term touches one element of a row: a branch that a wavefront takes only where a target falls into
            // its columns
            const int x = __float_as_int(info[i].z) - lcol;             // 16 j + v at the target
            if ((unsigned)x < 16u * C::TN16 && (x & 15) < 4) {
#pragma unroll
                for (int j = 0; j < C::TN16; ++j)
#pragma unroll
                    for (int v = 0; v < 4; ++v) g[j][v] -= x == 16 * j + v ? cf : 0.f;
            }
            if (ragged) {
#pragma unroll
                for (int j = 0; j < C::TN16; ++j)
#pragma unroll
                    for (int v = 0; v < 4; ++v) g[j][v] = lcol + 16 * j + v < V ? g[j][v] : 0.f;
            }
            uint2 w[C::TN16];
#pragma unroll
            for (int j = 0; j < C::TN16; ++j) w[j] = make_uint2(f32x2_to_bf16x2(g[j][0], g[j][1]), f32x2_to_bf16x2(g[j][2], g[j][3]));
            out.put(i, w, streamed != 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
};

// ------------------------------------------------------------------------------------------
// logit gradients from kept logits
// ------------------------------------------------------------------------------------------

// The gradient of EpiDz from the logits that EpiRowStatsKeep left behind instead of from a second product:
//   dz[m, v] = coef[m] * (exp(log P[m, v]) - 1[v = x_m]),  rowinfo as for EpiDz.
struct LossDzRule {
    static constexpr int RT = 2;
    __device__ __forceinline__ void operator()(int, int nrows, int col, int V, const float4 (&info)[2],
                                               const float (&lp)[2][8], float (&g)[2][8]) const
    {
#pragma unroll
        for (int h = 0; h < 2; ++h)
            if (h < nrows) {
                const float cf = info[h].y;
                const int x = __float_as_int(info[h].z) - col;
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    float v = cf * __builtin_amdgcn_exp2f(lp[h][k] * kLog2e);
                    if (x == k) v -= cf;
                    g[h][k] = (col + k < V) ? v : 0.f;
                }
            }
    }
};

// ------------------------------------------------------------------------------------------
// small kernels around the GEMMs
// ------------------------------------------------------------------------------------------

// dst[c, r] = src[r, c] (bf16); dst rows are ldd long and columns R..Rp-1 are zero-filled.
__global__ void __launch_bounds__(kBlock) k_transpose_bf16(const bf16_t *__restrict__ src, long lds_, int R, int C,
                                                           bf16_t *__restrict__ dst, long ldd, int Rp, int tiles_c)
{
    __shared__ bf16_t tile[64][66];
    const int tc = blockIdx.x % tiles_c, tr = blockIdx.x / tiles_c;
    const int r0 = tr * 64, c0 = tc * 64;
    const int lx = threadIdx.x & 63, ly = threadIdx.x >> 6;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int r = r0 + i * 4 + ly, c = c0 + lx;
        tile[i * 4 + ly][lx] = (r < R && c < C) ? src[(size_t)r * lds_ + c] : (bf16_t)0;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int c = c0 + i * 4 + ly, r = r0 + lx;
        if (c < C && r < Rp) dst[(size_t)c * ldd + r] = tile[lx][i * 4 + ly];
    }
}

// The same with 16-byte accesses on both sides, for C a multiple of 64 and lds_, ldd, Rp multiples of 8 (and
// 16-byte aligned bases): a thread loads eight columns of a row at once, the tile crosses LDS, and a thread
// gathers eight rows of one column for a 16-byte store; a wavefront store covers 8 output rows x 128 bytes.
__global__ void __launch_bounds__(kBlock) k_transpose_bf16_wide(const bf16_t *__restrict__ src, long lds_, int R,
                                                                bf16_t *__restrict__ dst, long ldd, int Rp, int tiles_c)
{
    __shared__ uint32_t tile[64][33];                   // 64 rows x 64 bf16, one dword of padding per row
    const int tc = blockIdx.x % tiles_c, tr = blockIdx.x / tiles_c;
    const int r0 = tr * 64, c0 = tc * 64;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int id = threadIdx.x + kBlock * p, row = id >> 3, ch = id & 7;
        const int r = r0 + row;
        u32x4_t v = {0u, 0u, 0u, 0u};
        if (r < R) v = *reinterpret_cast<const u32x4_t *>(src + (size_t)r * lds_ + c0 + ch * 8);
#pragma unroll
        for (int w = 0; w < 4; ++w) tile[row][ch * 4 + w] = v[w];
    }
    __syncthreads();
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int id = threadIdx.x + kBlock * p, col = id >> 3, rg = id & 7;     // source column, group of 8 rows
        const int shift = (col & 1) * 16;
        u32x4_t v;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const uint32_t a = (tile[rg * 8 + 2 * w][col >> 1] >> shift) & 0xFFFFu;
            const uint32_t b = (tile[rg * 8 + 2 * w + 1][col >> 1] >> shift) & 0xFFFFu;
            v[w] = a | (b << 16);
        }
        const int r = r0 + rg * 8;
        if (r < Rp) *reinterpret_cast<u32x4_t *>(dst + (size_t)(c0 + col) * ldd + r) = v;
    }
}

void transpose_bf16(const bf16_t *src, long lds_, int R, int C, bf16_t *dst, long ldd, int Rp, hipStream_t st)
{
    ProfileScope prof("transpose", 2.0 * ((double)R * C + (double)Rp * C), st);   // work = bytes moved
    const int tiles_c = (C + 63) / 64, tiles_r = (Rp + 63) / 64;
    const bool wide = C % 64 == 0 && lds_ % 8 == 0 && ldd % 8 == 0 && Rp % 8 == 0 &&
                      (reinterpret_cast<uintptr_t>(src) & 15u) == 0 && (reinterpret_cast<uintptr_t>(dst) & 15u) == 0;
    if (wide)
        k_transpose_bf16_wide<<<(unsigned)((size_t)tiles_c * tiles_r), kBlock, 0, st>>>(src, lds_, R, dst, ldd, Rp, tiles_c);
    else
        k_transpose_bf16<<<(unsigned)((size_t)tiles_c * tiles_r), kBlock, 0, st>>>(src, lds_, R, C, dst, ldd, Rp, tiles_c);
}

// Per head row: combine the per-tile statistics into the log-normaliser (eq. 5), take the
// target logit as an fp32 dot product of U[x] with y = hi (+ lo), and form C = z[x] - lse (eq. 8).
// One wavefront per row.  part == NULL: the log-normaliser is read from lse_io instead of being
// computed.  X == NULL: only the log-normaliser is produced.  Ylo == NULL: y = hi.
__global__ void __launch_bounds__(kBlock) k_row_finish(size_t M, int d, int r, int parts,
                                                       const float2 *__restrict__ part,
                                                       const bf16_t *__restrict__ Yhi, const bf16_t *__restrict__ Ylo,
                                                       const bf16_t *__restrict__ U, const int32_t *__restrict__ X,
                                                       float *__restrict__ lse_io, float *__restrict__ C_out)
{
    const size_t m = (size_t)blockIdx.x * (kBlock / kWave) + (threadIdx.x >> 6);
    if (m >= M) return;
    const int lane = threadIdx.x & 63;
    float lse;
    if (part) {
        float mx = -INFINITY, l = 0.f;
        for (int p = lane; p < parts; p += kWave) {
            const float2 q = part[m * parts + p];
            if (q.x > mx) { l = l * __expf(mx - q.x) + q.y; mx = q.x; }
            else if (q.x != -INFINITY) l += q.y * __expf(q.x - mx);
            else l += q.y;                                   // no valid column: 0, or the NaN it had
        }
        const float Mx = wave_max(mx);
        const float L = wave_sum(mx == -INFINITY ? l : l * __expf(mx - Mx));
        lse = Mx + logf(L);
        if (lane == 0) lse_io[m] = lse;
    } else {
        lse = lse_io[m];
    }
    if (!X) return;
    const int x = X[m / r];
    float zt = 0.f;
    if (x >= 0) {
        const bf16_t *u = U + (size_t)x * d, *yh = Yhi + m * d;
        if (Ylo) {
            const bf16_t *yl = Ylo + m * d;
            for (int k = lane; k < d; k += kWave)
                zt += bf16_to_f32(u[k]) * (bf16_to_f32(yh[k]) + bf16_to_f32(yl[k]));
        } else {
            for (int k = lane; k < d; k += kWave) zt += bf16_to_f32(u[k]) * bf16_to_f32(yh[k]);
        }
        zt = wave_sum(zt);
    }
    if (lane == 0) C_out[m] = (x >= 0) ? zt - lse : 0.f;
}

// ------------------------------------------------------------------------------------------
// draft step ("Sampling method"): small kernels around the two streaming GEMMs
// ------------------------------------------------------------------------------------------

__device__ __forceinline__ double wave_scan_inclusive(double v, int lane)
{
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const double o = __shfl_up(v, off, kWave);
        if (lane >= off) v += o;
    }
    return v;
}

// fp32 dot product of two bf16 vectors of length d (a multiple of 64) over one wavefront, 16-byte loads
__device__ __forceinline__ float wave_dot_bf16(const bf16_t *__restrict__ a, const bf16_t *__restrict__ b, int d, int lane)
{
    const u32x4_t *pa = reinterpret_cast<const u32x4_t *>(a);
    const u32x4_t *pb = reinterpret_cast<const u32x4_t *>(b);
    float acc = 0.f;
    for (int k = lane; k < d / 8; k += kWave) {
        const u32x4_t x = pa[k], y = pb[k];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            acc += __uint_as_float(x[e] << 16) * __uint_as_float(y[e] << 16);
            acc += __uint_as_float(x[e] & 0xFFFF0000u) * __uint_as_float(y[e] & 0xFFFF0000u);
        }
    }
    return wave_sum(acc);
}

// gate (eq. 7) and the expert draw: log w = log_softmax(G h); a* = first a whose running sum of w
// (fp64) exceeds u, clamped to r-1.  One block per row of the batch, a wavefront per expert at a time.
// g_s: at least r floats of LDS.  uniforms = null: log w only.
constexpr int kWideBlock = 1024;
constexpr int kMaxSegCols = 128;                // columns of a statistics segment: 64 or 128
__device__ __forceinline__ void draft_gate_pick_row(size_t b, int nwaves, float *g_s, int d, int n, int r,
                                                    const bf16_t *__restrict__ H, const bf16_t *__restrict__ G,
                                                    const float *__restrict__ uniforms, float *__restrict__ logw,
                                                    int32_t *__restrict__ alpha)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int a = wave; a < r; a += nwaves) {
        const float p = wave_dot_bf16(G + (size_t)a * d, H + b * d, d, lane);
        if (lane == 0) g_s[a] = p;
    }
    __syncthreads();
    if (wave != 0) return;
    const float mine = lane < r ? g_s[lane] : -INFINITY;
    const float mx = wave_max(mine);
    const float s = wave_sum(lane < r ? expf(mine - mx) : 0.f);
    const float lse = mx + logf(s);
    const float w = lane < r ? expf(mine - lse) : 0.f;
    if (lane < r) logw[b * r + lane] = mine - lse;
    if (!uniforms) return;                      // log w only
    // inclusive running sum of w in expert order, fp64
    const double incl = wave_scan_inclusive((double)w, lane);
    const double u = (double)uniforms[b * (1 + n)];
    const unsigned long long crossed = __ballot(lane < r && incl > u);
    if (lane == 0) alpha[b] = crossed ? __ffsll((long long)crossed) - 1 : r - 1;
}
// It runs as a side job of the y product's launch (the two are independent: both read only H and weights), which
// saves the draft-type calls a launch: workgroup `job` of the first `blocks` (B rounded up to 8) takes row `job`.
struct GatePickSide {
    static constexpr bool kActive = true;
    int blocks;
    int B, d, n, r;
    const bf16_t *H, *G;
    const float *uniforms;
    float *logw;
    int32_t *alpha;
    __device__ void run(int job, char *smem) const
    {
        if (job >= B) return;
        draft_gate_pick_row((size_t)job, (int)(blockDim.x / kWave), reinterpret_cast<float *>(smem), d, n, r, H, G,
                            uniforms, logw, alpha);
    }
};

// Log-normaliser (eq. 5) of one row from its per-segment statistics, by one wavefront.
__device__ __forceinline__ float row_lse_from_parts(const float2 *__restrict__ pm, int parts, int lane)
{
    // many independent loads per lane and step, since a step is a memory latency (32 rows of 2004 segments, the draft call's at
    // V = 128256: four loads a step 10.5 us for k_draft_lse_segment, sixteen 9.2); they are added up four at a time whatever the step is
    float mx = -INFINITY, l = 0.f;
    auto step = [&](int p0, auto loads) {
        constexpr int N = decltype(loads)::value;
        float2 qv[N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int p = p0 + i * kWave + lane;
            qv[i] = p < parts ? pm[p] : make_float2(-INFINITY, 0.f);
        }
#pragma unroll
        for (int i = 0; i < N; i += 4) {
            const float m4 = fmaxf(fmaxf(qv[i].x, qv[i + 1].x), fmaxf(qv[i + 2].x, qv[i + 3].x));
            if (m4 == -INFINITY) {                           // no valid columns: zeros, or the NaN they had
                l += (qv[i].y + qv[i + 1].y) + (qv[i + 2].y + qv[i + 3].y);
                continue;
            }
            const float mn = fmaxf(mx, m4);
            float add = 0.f;
#pragma unroll
            for (int e = i; e < i + 4; ++e) add += qv[e].y * __expf(qv[e].x - mn);     // exp(-inf) = 0 for empty segments
            l = l * __expf(mx - mn) + add;
            mx = mn;
        }
    };
    int p0 = 0;
    for (; parts - p0 > 4 * kWave; p0 += 16 * kWave) step(p0, std::integral_constant<int, 16>());
    if (p0 < parts) step(p0, std::integral_constant<int, 4>());
    const float Mx = wave_max(mx);
    const float L = wave_sum(mx == -INFINITY ? l : l * __expf(mx - Mx));
    return Mx + logf(L);
}

// Search by a workgroup for the segment of the vocabulary in which a running sum of probabilities passes u: mass(j) of
// the segments in vocabulary order, fp64, a run of consecutive segments per thread.  *seg_out is the segment, *base_out
// the sum before it; if the sum never passes u, ~(last segment) and 0.  All kWideBlock threads call it; ALONE: the first
// wavefront does it alone, where meeting 15 idle ones twice costs more than longer runs (k_draft_lse_segment of 600 draws
// over 56 segments: 8.4 -> 5.6 us).
template <bool ALONE, class F>
__device__ __forceinline__ void find_segment(int parts, int last_seg, double u, F mass, int32_t *seg_out, double *base_out)
{
    __shared__ double wave_tot[kWideBlock / kWave];
    __shared__ int first_wave[kWideBlock / kWave];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (ALONE && wave > 0) return;
    constexpr int threads = ALONE ? kWave : kWideBlock;
    const int per = (parts + threads - 1) / threads;
    const int lo = min(parts, tid * per), hi = min(parts, lo + per);
    double sum = 0.0;
    for (int j = lo; j < hi; ++j) sum += mass(j);
    double incl = wave_scan_inclusive(sum, lane);
    if (!ALONE) {
        if (lane == kWave - 1) wave_tot[wave] = incl;
        __syncthreads();
        for (int w = 0; w < wave; ++w) incl += wave_tot[w];
    }
    const unsigned long long crossed = __ballot(incl > u);
    int at = crossed ? __ffsll((long long)crossed) - 1 : -1;      // the first thread whose running sum passes u
    if (!ALONE) {
        if (lane == 0) first_wave[wave] = at;
        __syncthreads();
        at = -1;
        for (int w = kWideBlock / kWave - 1; w >= 0; --w)
            if (first_wave[w] >= 0) at = w * kWave + first_wave[w];
    }
    if (at < 0) {
        if (tid == 0) { *seg_out = ~last_seg; *base_out = 0.0; }
    } else if (tid == at) {
        double c = incl - sum;
        int seg = hi - 1;
        for (int j = lo; j < hi; ++j) {
            const double mj = mass(j);
            if (c + mj > u) { seg = j; break; }
            c += mj;
        }
        *seg_out = min(seg, last_seg);               // rounding may let the sum pass in the empty segments after it
        *base_out = c;
    }
}

// One wavefront continues that scan token by token through the `cols` tokens of the segment, prob(i) each: the first
// index whose running sum exceeds u, the last one if rounding between the two passes leaves none.
template <class F>
__device__ __forceinline__ int wave_pick_token(int seg_cols, int cols, double base, double u, int lane, F prob)
{
    const int per = (seg_cols + kWave - 1) / kWave;
    const int lo = lane * per;
    double sum = 0.0;
    for (int i = lo; i < lo + per && i < cols; ++i) sum += prob(i);
    const double incl = base + wave_scan_inclusive(sum, lane);
    const unsigned long long crossed = __ballot(incl > u);
    if (crossed == 0ull) return cols - 1;
    const int first = __ffsll((long long)crossed) - 1;
    int tok = min(cols, lo + per) - 1;
    if (lane == first) {
        double c = incl - sum;
        for (int i = lo; i < lo + per && i < cols; ++i) {
            c += prob(i);
            if (c > u) { tok = i; break; }
        }
    }
    return __shfl(tok, first, kWave);
}

// Per (b, s): the log-normalisers of its r head rows from the per-segment statistics (eq. 5), then the segment in which
// the running sum of the drawn expert's probabilities passes u.
template <bool ALONE>
__global__ void __launch_bounds__(kWideBlock) k_draft_lse_segment(int n, int r, int parts, int last_seg,
                                                                  const float2 *__restrict__ part,
                                                                  const int32_t *__restrict__ alpha,
                                                                  const float *__restrict__ uniforms,
                                                                  float *__restrict__ lse_out, int32_t *__restrict__ seg_out,
                                                                  double *__restrict__ base_out)
{
    __shared__ float lse_s[64];
    const size_t bs = blockIdx.x;                 // b*n + s
    const size_t b = bs / n;
    const int s = (int)(bs % n);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int a = wave; a < r; a += kWideBlock / kWave) {
        const float lse = row_lse_from_parts(part + (bs * r + a) * parts, parts, lane);
        if (lane == 0) { lse_out[bs * r + a] = lse; lse_s[a] = lse; }
    }
    __syncthreads();
    const int astar = alpha[b];
    const float l = lse_s[astar];
    const float2 *pm = part + (bs * r + astar) * parts;
    find_segment<ALONE>(parts, last_seg, (double)uniforms[b * (1 + n) + 1 + s],
                 [&](int j) {
                     const float2 q = pm[j];
                     return q.x == -INFINITY ? 0.0 : (double)(q.y * expf(q.x - l));
                 },
                 seg_out + bs, base_out + bs);
}

// The logits of a segment for the r head rows of a (row, draw), z[(x * r + a) * seg_cols + i] = U[v0 + i] . y[row0 + a]:
// a workgroup per (b, draw), 16 tokens and 16 experts, on the 16x16x32 matrix instruction; its eight wavefronts share
// the contraction and their partial products meet in LDS.  Bound by the latency of the cold rows of U: the rows of a segment are
// spread over 4 or 8 workgroups of eight wavefronts, where one workgroup per draw had the whole segment (0.5 or 1 MB) to
// fetch: the draft call 397 -> 371 us at B = 1, d = 4096, V = 128256, n = 4, r = 8.
// (b, s) of workgroup x is b = x / draws, s = draw0 + x % draws; its segment is seg_in[b * seg_ld + x % draws].
constexpr int kSegWaves = 8;
__global__ void __launch_bounds__(kSegWaves * kWave) k_segment_logits(int d, int V, int n, int r, int seg_cols, int draw0,
                                                                      int draws, const bf16_t *__restrict__ Y,
                                                                      const bf16_t *__restrict__ U,
                                                                      const int32_t *__restrict__ seg_in, int seg_ld,
                                                                      float *__restrict__ z)
{
    __shared__ float red[kSegWaves][16][17];
    const int x = (int)blockIdx.x, code = seg_in[(size_t)(x / draws) * seg_ld + x % draws];
    const int v0 = (code < 0 ? ~code : code) * seg_cols + (int)blockIdx.y * 16;
    if (v0 >= V) return;
    const size_t row0 = ((size_t)(x / draws) * n + draw0 + x % draws) * r;
    const int a0 = (int)blockIdx.z * 16;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row = lane & 15, q = lane >> 4;
    // tokens past V and experts past r repeat the last one: the former are never used, the latter not stored
    const bf16_t *pu = U + (size_t)min(v0 + row, V - 1) * d + q * 16;
    const bf16_t *const py[1] = {Y + (row0 + min(a0 + row, r - 1)) * d + q * 16};
    f32x4_t acc[1] = {{0.f, 0.f, 0.f, 0.f}};
    tile16_products<kSegWaves, 1>(pu, py, d, wave, acc);
#pragma unroll
    for (int v = 0; v < 4; ++v) red[wave][tile16_row(v, lane)][row] = acc[0][v];
    __syncthreads();
    const int tok = threadIdx.x & 15, e = threadIdx.x >> 4;
    if (e < 16 && a0 + e < r) {
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < kSegWaves; ++w) sum += red[w][tok][e];
        z[((size_t)x * r + a0 + e) * seg_cols + blockIdx.y * 16 + tok] = sum;
    }
}

// The same two steps for calls that want no log-probability: a workgroup per (b, s) forms the logits of the drawn expert's
// segment alone (a wavefront walks the contraction for four tokens together) and picks the token from them.  One launch
// instead of two for the numbers of draws that just fill the chip, whole calls, us, this against the two: 256 draws (d = 512,
// V = 1000) 39.5 / 44.5, 512 (d = 1024, V = 32000) 174 / 179, 600 (d = 512, V = 7000) 77.1 / 79.8; but 2000 (d = 128, V = 3000)
// 85.3 / 74.8 and 4096 (d = 256, V = 100) 134 / 124, where the matrix instruction counts, and the same from 36 draws down.
constexpr unsigned kAloneDraws = 64, kAloneDrawsMost = 1024;
__global__ void __launch_bounds__(kWideBlock) k_draft_pick_alone(int d, int V, int n, int r, int seg_cols, const float *__restrict__ lse,
                                                                 const bf16_t *__restrict__ Y, const bf16_t *__restrict__ U,
                                                                 const int32_t *__restrict__ alpha, const int32_t *__restrict__ seg,
                                                                 const double *__restrict__ base,
                                                                 const float *__restrict__ uniforms, int32_t *__restrict__ tokens)
{
    __shared__ float p_s[kMaxSegCols];
    const size_t bs = blockIdx.x;                 // b*n + s
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int code = seg[bs];
    if (code < 0) {                               // the running sum over the whole vocabulary never passes u
        if (threadIdx.x == 0) tokens[bs] = V - 1;
        return;
    }
    const size_t b = bs / n, m = bs * r + alpha[b];
    const float l = lse[m];
    const int v0 = code * seg_cols, cols = min(seg_cols, V - v0);
    constexpr int CW = 4;
    const u32x4_t *yrow = reinterpret_cast<const u32x4_t *>(Y + m * d);
    for (int c0 = wave * CW; c0 < cols; c0 += kWideBlock / kWave * CW) {
        float acc[CW] = {0.f, 0.f, 0.f, 0.f};
        const u32x4_t *urow[CW];
#pragma unroll
        for (int e = 0; e < CW; ++e)
            urow[e] = reinterpret_cast<const u32x4_t *>(U + (size_t)(v0 + min(c0 + e, cols - 1)) * d);
        for (int k = lane; k < d / 8; k += kWave) {
            const u32x4_t yv = yrow[k];
            u32x4_t uv[CW];
#pragma unroll
            for (int e = 0; e < CW; ++e) uv[e] = urow[e][k];
#pragma unroll
            for (int e = 0; e < CW; ++e)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    acc[e] += __uint_as_float(uv[e][q] << 16) * __uint_as_float(yv[q] << 16);
                    acc[e] += __uint_as_float(uv[e][q] & 0xFFFF0000u) * __uint_as_float(yv[q] & 0xFFFF0000u);
                }
        }
#pragma unroll
        for (int e = 0; e < CW; ++e) {
            const float z = wave_sum(acc[e]);
            if (lane == 0 && c0 + e < cols) p_s[c0 + e] = expf(z - l);
        }
    }
    __syncthreads();
    if (wave != 0) return;
    const int at = wave_pick_token(seg_cols, cols, base[bs], (double)uniforms[b * (1 + n) + 1 + bs % n], lane,
                                   [&](int i) { return (double)p_s[i]; });
    if (lane == 0) tokens[bs] = v0 + at;
}

// Per b: the tokens of its draws s0 .. s0 + draws - 1 from the logits of their segments (a wavefront per draw; z as
// k_segment_logits leaves it), then logq[b] = logsumexp_a( log w_a + sum_s (z_sa[tok_s] - lse_sa) ): eq. 9 at the drawn
// tuple over all experts, the sum so far in logw between launches.
__global__ void __launch_bounds__(kWideBlock) k_draft_pick(int V, int n, int r, int seg_cols, int s0, int draws, float *__restrict__ logw,
                                                           const float *__restrict__ lse, const float *__restrict__ z,
                                                           const int32_t *__restrict__ alpha,
                                                           const int32_t *__restrict__ seg, const double *__restrict__ base,
                                                           const float *__restrict__ uniforms, int32_t *__restrict__ tokens,
                                                           float *__restrict__ logq)
{
    __shared__ int at_s[64];                          // the drawn token's place in its segment
    const size_t b = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int i = wave; i < draws; i += kWideBlock / kWave) {
        const int s = s0 + i;
        const size_t bs = b * n + s;
        const int code = seg[bs], v0 = (code < 0 ? ~code : code) * seg_cols, cols = min(seg_cols, V - v0);
        const float l = lse[bs * r + alpha[b]];
        const float *zr = z + ((b * draws + i) * r + alpha[b]) * seg_cols;
        // the running sum over the whole vocabulary never passes u: the last token
        const int at = code < 0 ? cols - 1
                                : wave_pick_token(seg_cols, cols, base[bs], (double)uniforms[b * (1 + n) + 1 + s], lane,
                                                  [&](int k) { return (double)expf(zr[k] - l); });
        if (lane == 0) { tokens[bs] = v0 + at; at_s[i] = at; }
    }
    __syncthreads();
    if (!logq || wave != 0) return;
    float a = -INFINITY;
    if (lane < r) {
        a = logw[b * r + lane];
        for (int i = 0; i < draws; ++i) a += z[((b * draws + i) * r + lane) * seg_cols + at_s[i]] - lse[(b * n + s0 + i) * r + lane];
        if (s0 + draws < n) logw[b * r + lane] = a;
    }
    if (s0 + draws < n) return;
    const float mx = wave_max(a);
    const float sum = wave_sum(lane < r ? expf(a - mx) : 0.f);
    if (lane == 0) logq[b] = mx + logf(sum);
}

__global__ void __launch_bounds__(kBlock) k_lse_from_parts(size_t rows, int parts, const float2 *__restrict__ part,
                                                           float *__restrict__ lse)
{
    const int lane = threadIdx.x & 63;
    const size_t row = (size_t)blockIdx.x * (kBlock / kWave) + (threadIdx.x >> 6);
    if (row >= rows) return;
    const float v = row_lse_from_parts(part + row * parts, parts, lane);
    if (lane == 0) lse[row] = v;
}

// (max, sum of exp(z - max)) of one chunk of kStatCols columns of one row of stored fp32 logits
// (row stride ld, a multiple of 4): the per-segment statistics of eq. 5 for logits that are stored.
constexpr int kStatCols = 4096;
__global__ void __launch_bounds__(kBlock) k_row_stats_f32(int V, size_t ld, int parts, const float *__restrict__ z,
                                                          float2 *__restrict__ part)
{
    __shared__ float red_m[kBlock / kWave], red_l[kBlock / kWave];
    const size_t row = blockIdx.x;
    const int c0 = blockIdx.y * kStatCols;
    const float *zr = z + row * ld;
    float4 x[kStatCols / 4 / kBlock];
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < kStatCols / 4 / kBlock; ++i) {
        const int c = c0 + (i * kBlock + threadIdx.x) * 4;
        x[i] = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
        if (c + 3 < V) {
            x[i] = *reinterpret_cast<const float4 *>(zr + c);
        } else if (c < V) {
            x[i].x = zr[c];
            if (c + 1 < V) x[i].y = zr[c + 1];
            if (c + 2 < V) x[i].z = zr[c + 2];
        }
        mx = fmaxf(fmaxf(mx, fmaxf(x[i].x, x[i].y)), fmaxf(x[i].z, x[i].w));
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    mx = wave_max(mx);
    if (lane == 0) red_m[wave] = mx;
    __syncthreads();
    float Mx = red_m[0];
#pragma unroll
    for (int w = 1; w < kBlock / kWave; ++w) Mx = fmaxf(Mx, red_m[w]);
    const float ref = (Mx == -INFINITY) ? 0.f : Mx;
    float l = 0.f;
#pragma unroll
    for (int i = 0; i < kStatCols / 4 / kBlock; ++i)
        l += __expf(x[i].x - ref) + __expf(x[i].y - ref) + __expf(x[i].z - ref) + __expf(x[i].w - ref);
    l = wave_sum(l);
    if (lane == 0) red_l[wave] = l;
    __syncthreads();
    if (threadIdx.x == 0) {
        float L = 0.f;
#pragma unroll
        for (int w = 0; w < kBlock / kWave; ++w) L += red_l[w];
        part[row * parts + blockIdx.y] = make_float2(Mx, L);        // as EpiRowStats leaves it: a NaN stays one
    }
}

// logp[b, v] = logsumexp_a(log w_a + z[(b, a), v] - lse[(b, a)]) (eq. 11) for 256 tokens of one b, from the stored first-head logits and
// the per-segment statistics of their rows: every workgroup forms the r log-normalisers by itself, which saves the call a launch.
__global__ void __launch_bounds__(kBlock) k_first_token_from_parts(int V, int r, int parts, size_t ld, const float *__restrict__ z,
                                                                   const float2 *__restrict__ part, const float *__restrict__ logw,
                                                                   float *__restrict__ logp)
{
    __shared__ float off_s[64];                   // log w - lse per expert
    const size_t b = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int v = blockIdx.y * kBlock + threadIdx.x;
    const float *zv = z + b * r * ld + min(v, V - 1);
    float first[8];
#pragma unroll
    for (int a = 0; a < 8; ++a) first[a] = zv[min(a, r - 1) * ld];
    for (int a = wave; a < r; a += kBlock / kWave) {
        const float lse = row_lse_from_parts(part + (b * r + a) * parts, parts, lane);
        if (lane == 0) off_s[a] = logw[b * r + a] - lse;
    }
    __syncthreads();
    if (v >= V) return;
    float mx = -INFINITY, l = 0.f;
    auto add = [&](float x) {
        if (x > mx) { l = l * expf(mx - x) + 1.f; mx = x; }
        else l += expf(x - mx);
    };
#pragma unroll
    for (int a = 0; a < 8; ++a)
        if (a < r) add(first[a] + off_s[a]);
    for (int a = 8; a < r; ++a) add(zv[a * ld] + off_s[a]);
    logp[b * (size_t)V + v] = mx + logf(l);
}

// The paper's sequential scheme (eq. 11-13), one workgroup per row b of the batch.
// For step s the conditional is the mixture sum_a qhat_a P^(s)(. | a) with qhat = softmax(q),
// q_a = log w_a + sum_{k<s} log P^(k)(x_k | a).  It is sampled exactly like the single-expert draw of
// cp_head_draft_sample, with every mass replaced by its qhat-weighted sum over the r experts.
// Launch s picks the token of draw s - 1 from the logits of its segment (k_segment_logits, between the launches), adds
// its log-probabilities to q, and finds the segment of draw s; launch n only picks and writes logq.
template <bool ALONE>
__global__ void __launch_bounds__(kWideBlock) k_sequential_step(int step, int V, int n, int r, int parts, int seg_cols,
                                                                const float2 *__restrict__ part, const float *__restrict__ z,
                                                                const float *__restrict__ lse, float *__restrict__ q,
                                                                const float *__restrict__ uniforms, int32_t *__restrict__ seg,
                                                                double *__restrict__ base, int32_t *__restrict__ tokens,
                                                                float *__restrict__ logq)
{
    __shared__ float lse_s[64], q_s[64], qh_s[64];
    __shared__ double p_s[kMaxSegCols];
    const size_t b = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // weights of the mixture and log-normalisers of draw s
    auto load_draw = [&](int s) {
        if (wave == 0) {
            const float qa = lane < r ? q_s[lane] : -INFINITY;
            const float mx = wave_max(qa);
            const float qn = mx + logf(wave_sum(lane < r ? expf(qa - mx) : 0.f));
            if (lane < r) qh_s[lane] = expf(qa - qn);
        } else if (wave == 1 && lane < r) {
            lse_s[lane] = lse[(b * n + s) * r + lane];
        }
        __syncthreads();
    };
    if (tid < r) q_s[tid] = q[b * r + tid];
    __syncthreads();
    if (step > 0) {
        const int s = step - 1;
        load_draw(s);
        const int code = seg[b], v0 = (code < 0 ? ~code : code) * seg_cols, cols = min(seg_cols, V - v0);
        const float *zr = z + b * r * seg_cols;
        if (tid < cols) {
            double p = 0.0;
            for (int a = 0; a < r; ++a) p += (double)(qh_s[a] * expf(zr[a * seg_cols + tid] - lse_s[a]));
            p_s[tid] = p;
        }
        __syncthreads();
        if (wave == 0) {
            // the running sum over the whole vocabulary never passes u: the last token
            const int at = code < 0 ? cols - 1
                                    : wave_pick_token(seg_cols, cols, base[b], (double)uniforms[b * n + s], lane,
                                                      [&](int i) { return p_s[i]; });
            if (lane == 0) tokens[b * n + s] = v0 + at;
            // expert log-weights take the log-probability of the drawn token (text under eq. 12)
            if (lane < r) {
                q_s[lane] += zr[lane * seg_cols + at] - lse_s[lane];
                q[b * r + lane] = q_s[lane];
            }
        }
        __syncthreads();
    }
    if (step == n) {
        if (logq && wave == 0) {
            const float qa = lane < r ? q_s[lane] : -INFINITY;
            const float mx = wave_max(qa);
            const float sum = wave_sum(lane < r ? expf(qa - mx) : 0.f);
            if (lane == 0) logq[b] = mx + logf(sum);
        }
        return;
    }
    load_draw(step);
    const float2 *pm = part + (b * n + step) * r * parts;
    find_segment<ALONE>(parts, (V - 1) / seg_cols, (double)uniforms[b * n + step],
                 [&](int j) {
                     double m = 0.0;
                     for (int a = 0; a < r; ++a) {
                         const float2 qv = pm[(size_t)a * parts + j];
                         if (qv.x != -INFINITY) m += (double)(qh_s[a] * qv.y * expf(qv.x - lse_s[a]));
                     }
                     return m;
                 },
                 seg + b, base + b);
}

// The same for at most eight experts and PER segments per thread: a launch is a chain of memory latencies, so everything that
// does not hang on the token drawn last (the masses of the next draw's segments, the logits of the present one's) is
// requested at the start, and the logits stay in LDS for the update of the weights (11.6 -> 8.6 us a launch at B = 8, V = 128256, r = 8).
template <bool ALONE, int PER>
__global__ void __launch_bounds__(kWideBlock) k_sequential_step8(int step, int V, int n, int r, int parts, int seg_cols,
                                                                 const float2 *__restrict__ part, const float *__restrict__ z,
                                                                 const float *__restrict__ lse, float *__restrict__ q,
                                                                 const float *__restrict__ uniforms, int32_t *__restrict__ seg,
                                                                 double *__restrict__ base, int32_t *__restrict__ tokens,
                                                                 float *__restrict__ logq)
{
    __shared__ float lse_s[8], qh_s[8], lp_s[8][kMaxSegCols];
    __shared__ double p_s[kMaxSegCols];
    const size_t b = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool find = step < n;
    float2 qv[PER][8];
    if (find && (!ALONE || wave == 0)) {
        const float2 *pm = part + (b * n + step) * r * parts;
#pragma unroll
        for (int i = 0; i < PER; ++i)
#pragma unroll
            for (int a = 0; a < 8; ++a) {
                const int j = tid * PER + i;
                qv[i][a] = a < r && j < parts ? pm[(size_t)a * parts + j] : make_float2(-INFINITY, 0.f);
            }
    }
    int code = 0, v0 = 0, cols = 0;
    float zv[8];
    if (step > 0) {
        code = seg[b];
        v0 = (code < 0 ? ~code : code) * seg_cols;
        cols = min(seg_cols, V - v0);
        if (tid < cols) {
#pragma unroll
            for (int a = 0; a < 8; ++a) zv[a] = z[(b * r + min(a, r - 1)) * seg_cols + tid];
        }
        if (tid < r) lse_s[tid] = lse[(b * n + step - 1) * r + tid];
    }
    float qa = wave == 0 && lane < r ? q[b * r + lane] : -INFINITY;         // expert log-weights, lane a of wavefront 0
    auto weights = [&]() {
        if (wave != 0) return;
        const float mx = wave_max(qa);
        const float qn = mx + logf(wave_sum(lane < r ? expf(qa - mx) : 0.f));
        if (lane < r) qh_s[lane] = expf(qa - qn);
    };
    if (step > 0) {
        weights();
        __syncthreads();
        if (tid < cols) {
            double p = 0.0;
#pragma unroll
            for (int a = 0; a < 8; ++a)
                if (a < r) {
                    const float lp = zv[a] - lse_s[a];
                    lp_s[a][tid] = lp;
                    p += (double)(qh_s[a] * expf(lp));
                }
            p_s[tid] = p;
        }
        __syncthreads();
        if (wave == 0) {
            // the running sum over the whole vocabulary never passes u: the last token
            const int at = code < 0 ? cols - 1
                                    : wave_pick_token(seg_cols, cols, base[b], (double)uniforms[b * n + step - 1], lane,
                                                      [&](int i) { return p_s[i]; });
            if (lane == 0) tokens[b * n + step - 1] = v0 + at;
            // expert log-weights take the log-probability of the drawn token (text under eq. 12)
            if (lane < r) {
                qa += lp_s[lane][at];
                q[b * r + lane] = qa;
            }
        }
    }
    if (!find) {
        if (logq && wave == 0) {
            const float mx = wave_max(qa);
            const float sum = wave_sum(lane < r ? expf(qa - mx) : 0.f);
            if (lane == 0) logq[b] = mx + logf(sum);
        }
        return;
    }
    weights();
    float e[PER][8];
    if (!ALONE || wave == 0) {
#pragma unroll
        for (int a = 0; a < 8; ++a) {
            const float la = lse[(b * n + step) * r + min(a, r - 1)];
#pragma unroll
            for (int i = 0; i < PER; ++i) e[i][a] = qv[i][a].y * expf(qv[i][a].x - la);       // empty segments: 0 exp(-inf)
        }
    }
    __syncthreads();
    double mass[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        mass[i] = 0.0;
        if (!ALONE || wave == 0) {
#pragma unroll
            for (int a = 0; a < 8; ++a)
                if (a < r) mass[i] += (double)(qh_s[a] * e[i][a]);
        }
    }
    find_segment<ALONE>(parts, (V - 1) / seg_cols, (double)uniforms[b * n + step],
                        [&](int j) { return PER == 1 || j == tid * PER ? mass[0] : mass[PER - 1]; }, seg + b, base + b);
}

// Per head row {lse, coef = up_t * gamma[t, a] (zero for dropped factors), target}; dg[t, a] = up_t (w - gamma)
__global__ void k_bwd_coefficients(size_t M, int n, int r, const float *__restrict__ w, const float *__restrict__ gamma,
                                   const float *__restrict__ lse, const float *__restrict__ dloss, float scale,
                                   const int32_t *__restrict__ X, float4 *__restrict__ rowinfo, float *__restrict__ dg)
{
    const size_t m = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= M) return;
    const size_t t = m / ((size_t)n * r);
    const int a = (int)(m % r);
    const float up = dloss ? dloss[t] * scale : scale;
    const float gm = gamma[t * r + a];
    const int x = X[m / r];
    rowinfo[m] = make_float4(lse[m], (x >= 0) ? up * gm : 0.f, __int_as_float(x), 0.f);
    if ((m / r) % n == 0) dg[t * r + a] = up * (w[t * r + a] - gm);
}

// dH[t, j] += sum_a dg[t, a] G[a, j], four columns a thread (T = 16384, d = 4096, r = 8: one a
// thread 374 us, four 153 = 3.5 TB/s)
typedef uint32_t u32x2_any_t __attribute__((ext_vector_type(2), aligned(2)));
typedef float f32x4_any_t __attribute__((ext_vector_type(4), aligned(4)));
__global__ void __launch_bounds__(kBlock) k_add_gate_to_dh(size_t T, int d, int r, const bf16_t *__restrict__ G, const float *__restrict__ dg,
                                                           float *__restrict__ dH)
{
    const size_t idx = (size_t)blockIdx.x * kBlock + threadIdx.x, quads = (size_t)d / 4;       // d is a multiple of 64
    if (idx >= T * quads) return;
    const size_t t = idx / quads;
    const int j = (int)(idx % quads) * 4;
    f32x4_any_t *out = reinterpret_cast<f32x4_any_t *>(dH + t * d + j);
    f32x4_t acc = *out;
    for (int a = 0; a < r; ++a) {
        const float c = dg[t * r + a];
        const u32x2_any_t g = *reinterpret_cast<const u32x2_any_t *>(G + (size_t)a * d + j);
        acc[0] += c * __uint_as_float(g[0] << 16);
        acc[1] += c * __uint_as_float(g[0] & 0xFFFF0000u);
        acc[2] += c * __uint_as_float(g[1] << 16);
        acc[3] += c * __uint_as_float(g[1] & 0xFFFF0000u);
    }
    *out = acc;
}

// ------------------------------------------------------------------------------------------
// full heads (eq. 6 as printed: one V x d matrix F_sa per (s, a), no shared unembedding)
// Per-row quantities of this variant are kept head-major, index sa * T + t: every (s, a) runs its own
// products over the T positions, so its rows are contiguous for the epilogues above.
// ------------------------------------------------------------------------------------------

// One wavefront per (sa, t): log-normaliser from the statistics (eq. 5), target logit as an fp32 dot
// product of F_sa[x] with h (both bf16, so the products are exact), C = z[x] - lse (eq. 8).
__global__ void __launch_bounds__(kBlock) k_full_row_finish(size_t T, int d, int V, int n, int r, int parts,
                                                            const float2 *__restrict__ part,
                                                            const bf16_t *__restrict__ H, const bf16_t *__restrict__ F,
                                                            const int32_t *__restrict__ X, float *__restrict__ lse_out,
                                                            float *__restrict__ C_out)
{
    const size_t idx = (size_t)blockIdx.x * (kBlock / kWave) + (threadIdx.x >> 6);
    if (idx >= T * n * r) return;
    const int lane = threadIdx.x & 63;
    const size_t sa = idx / T, t = idx % T;
    const int s = (int)(sa / r), a = (int)(sa % r);
    const float lse = row_lse_from_parts(part + idx * parts, parts, lane);
    const int x = X[t * n + s];
    float zt = 0.f;
    if (x >= 0) zt = wave_dot_bf16(F + (sa * V + x) * d, H + t * d, d, lane);
    if (lane == 0) {
        lse_out[idx] = lse;
        C_out[(t * n + s) * r + a] = (x >= 0) ? zt - lse : 0.f;
    }
}

// Per (sa, t): {lse, coef = up_t * gamma[t, a] (zero for dropped factors), target}; dg[t, a] = up_t (w - gamma)
__global__ void k_full_bwd_coefficients(size_t T, int n, int r, const float *__restrict__ w,
                                        const float *__restrict__ gamma, const float *__restrict__ lse,
                                        const float *__restrict__ dloss, float scale, const int32_t *__restrict__ X,
                                        float4 *__restrict__ rowinfo, float *__restrict__ dg)
{
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= T * n * r) return;
    const size_t sa = idx / T, t = idx % T;
    const int s = (int)(sa / r), a = (int)(sa % r);
    const float up = dloss ? dloss[t] * scale : scale;
    const float gm = gamma[t * r + a];
    const int x = X[t * n + s];
    rowinfo[idx] = make_float4(lse[idx], (x >= 0) ? up * gm : 0.f, __int_as_float(x), 0.f);
    if (s == 0) dg[t * r + a] = up * (w[t * r + a] - gm);
}

// ------------------------------------------------------------------------------------------
// workspace layouts
// ------------------------------------------------------------------------------------------

// Scratch for splitting the last round of a call's products (the largest of them), none with CP_HEAD_MIN_WORKSPACE
struct SplitNeed {
    size_t bytes = 0;
    bool off;
    explicit SplitNeed(const cp_head_desc &ds) : off((ds.flags & CP_HEAD_MIN_WORKSPACE) != 0) {}
    template <class C>
    void product(size_t M, size_t N, size_t K)
    {
        const size_t b = off ? 0 : split_scratch_bytes<C>(M, N, K, kGroupRowsNarrow);
        if (b > bytes) bytes = b;
    }
    // the chunks of `total` rows: whole ones and the rest
    template <class F>
    static void chunks(size_t total, size_t chunk, F f)
    {
        if (total >= chunk) f(chunk);
        if (total % chunk) f(total % chunk);
    }
};
inline SplitScratch split_scratch(void *ws, size_t off, size_t bytes)
{
    SplitScratch s;
    if (bytes) { s.p = at<void>(ws, off); s.bytes = bytes; }
    return s;
}

inline size_t bwd_chunk_rows(const cp_head_desc &ds)
{
    static_assert(Cfg::BM == 256, "the tile of backward_chunk_rows");
    return backward_chunk_rows((size_t)ds.T * ds.n * ds.r, round_up((size_t)ds.V, 64), (ds.flags & CP_HEAD_MIN_WORKSPACE) != 0);
}

// The pair of loss calls and the single call add up every row's y and dY in the same order, so these two are split along K
// only where both calls make the same launches: y, which the pair forms for the whole batch, if that is one chunk;
// dY if the chunks are whole positions, as the single call's always are.
inline bool split_y(const cp_head_desc &ds) { return bwd_chunk_rows(ds) >= (size_t)ds.T * ds.n * ds.r; }
inline bool split_dy(const cp_head_desc &ds) { return bwd_chunk_rows(ds) % ((size_t)ds.n * ds.r) == 0; }

struct FwdWs {
    size_t logw, C, Ylo, part, split, split_bytes, total;
    int parts;
};
inline FwdWs fwd_ws(const cp_head_desc &ds)
{
    FwdWs f;
    const size_t M = (size_t)ds.T * ds.n * ds.r;
    f.parts = ((ds.V + Cfg::BN - 1) / Cfg::BN) * Cfg::WN;
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes); return o; };
    f.logw = take((size_t)ds.T * ds.r * 4);
    f.C = take(M * 4);
    f.Ylo = take(M * ds.d * 2);
    // with kept logits the statistics live in ctx: the backward pass needs the maxima again
    f.part = (ds.flags & CP_HEAD_KEEP_LOGITS) ? off : take(M * f.parts * sizeof(float2));
    SplitNeed need(ds);
    if (split_y(ds)) need.product<Cfg>((size_t)ds.T, (size_t)ds.n * ds.r * ds.d, (size_t)ds.d);    // y
    f.split_bytes = need.bytes;
    f.split = take(need.bytes);
    f.total = off;
    return f;
}

// the products of the backward pass below dz
inline void need_below_dz(const cp_head_desc &ds, size_t chunk, SplitNeed &need)
{
    const size_t T = (size_t)ds.T, d = (size_t)ds.d, V = (size_t)ds.V, nrd = (size_t)ds.n * ds.r * d;
    SplitNeed::chunks(T * ds.n * ds.r, chunk, [&](size_t Mc) {
        if (split_dy(ds)) need.product<CfgBlockedA>(Mc, d, round_up(V, 64));         // dY
        need.product<CfgBlockedTN>(V, d, round_up(Mc, 64));                          // dU
    });
    need.product<Cfg>(T, d, nrd);                                                    // dH
    need.product<CfgTN>(nrd, d, T);                                                  // dW
}

struct BwdWs {
    size_t coef, dg, dGpart, Ut, Wt, dY, dZ, Yt, split, split_bytes, total;
    size_t Vp, chunk, chunk_p;
    size_t ldV, ldM, ldN;   // leading dimensions of the transposed operands (K padded to 64, plus 64)
};
inline BwdWs bwd_ws(const cp_head_desc &ds)
{
    BwdWs b;
    const size_t T = (size_t)ds.T, nrd = (size_t)ds.n * ds.r * ds.d, M = T * ds.n * ds.r;
    b.Vp = round_up((size_t)ds.V, 64);
    b.chunk = bwd_chunk_rows(ds);
    b.chunk_p = round_up(b.chunk, 64);
    b.ldV = b.Vp + 64; b.ldM = b.chunk_p + 64; b.ldN = nrd + 64;
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes); return o; };
    b.coef = take(M * 16);
    b.dg = take(T * ds.r * 4);
    b.dGpart = take(gate_chunks(T) * ds.r * ds.d * 4);
    b.Ut = take((size_t)ds.d * b.ldV * 2);
    b.Wt = take((size_t)ds.d * b.ldN * 2);
    b.dY = take(M * ds.d * 2);
    b.dZ = take(round_up(b.chunk, 256) * b.Vp * 2);   // stored in blocks of 256 rows x 64 columns
    b.Yt = take((size_t)ds.d * b.ldM * 2);
    SplitNeed need(ds);
    need_below_dz(ds, b.chunk, need);
    b.split_bytes = need.bytes;
    b.split = take(need.bytes);
    b.total = off;
    return b;
}

// Saved-for-backward buffer of the full-head calls: [lse nr*T f32, head-major][w T*r][gamma T*r]
struct FullCtx {
    size_t lse, w, gamma, zpart, zs, total;
    size_t Vp;
    int parts;
    bool keep;      // CP_HEAD_KEEP_LOGITS: statistics and logits of all rows (head-major, like lse) stay in ctx
};
inline FullCtx full_ctx(const cp_head_desc &ds)
{
    FullCtx c;
    const size_t M = (size_t)ds.T * ds.n * ds.r, Tr = (size_t)ds.T * ds.r;
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes); return o; };
    c.lse = take(M * 4);
    c.w = take(Tr * 4);
    c.gamma = take(Tr * 4);
    c.keep = (ds.flags & CP_HEAD_KEEP_LOGITS) != 0 && use_fast_path(ds);
    c.Vp = round_up((size_t)ds.V, 64);
    c.parts = ((ds.V + Cfg::BN - 1) / Cfg::BN) * Cfg::WN;
    c.zpart = c.zs = off;
    if (c.keep) {
        c.zpart = take(M * c.parts * sizeof(float2));
        c.zs = take(M * c.Vp * 2);
    }
    c.total = off;
    return c;
}

struct FullFwdWs {
    size_t logw, C, part, total;
    int parts;
};
inline FullFwdWs full_fwd_ws(const cp_head_desc &ds)
{
    FullFwdWs f;
    const size_t M = (size_t)ds.T * ds.n * ds.r;
    f.parts = ((ds.V + Cfg::BN - 1) / Cfg::BN) * Cfg::WN;
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes); return o; };
    f.logw = take((size_t)ds.T * ds.r * 4);
    f.C = take(M * 4);
    f.part = (ds.flags & CP_HEAD_KEEP_LOGITS) ? off : take(M * f.parts * sizeof(float2));   // else in ctx
    f.total = off;
    return f;
}

// Positions whose logit gradients (for one head at a time) are held together: about 2 GiB of bf16
inline size_t full_chunk_rows(const cp_head_desc &ds)
{
    const size_t Vp = round_up((size_t)ds.V, 64);
    size_t rows = ((size_t)1 << 31) / (Vp * 2);
    rows = rows / Cfg::BM * Cfg::BM;
    if (rows < (size_t)Cfg::BM || (ds.flags & CP_HEAD_MIN_WORKSPACE)) rows = Cfg::BM;
    const size_t T = (size_t)ds.T;
    return rows < T ? rows : (T ? T : 1);
}

struct FullBwdWs {
    size_t coef, dg, dGpart, Ht, dZ, split, split_bytes, total;
    size_t Vp, Tp, chunk;
    size_t ldT;
};
inline FullBwdWs full_bwd_ws(const cp_head_desc &ds)
{
    FullBwdWs b;
    const size_t T = (size_t)ds.T, M = T * ds.n * ds.r;
    b.Vp = round_up((size_t)ds.V, 64);
    b.Tp = round_up(T, 64);
    b.chunk = full_chunk_rows(ds);
    b.ldT = b.Tp + 64;
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes); return o; };
    b.coef = take(M * 16);
    b.dg = take(T * ds.r * 4);
    b.dGpart = take(gate_chunks(T) * ds.r * ds.d * 4);
    b.Ht = take((size_t)ds.d * b.ldT * 2);
    b.dZ = take(round_up(b.chunk, 256) * b.Vp * 2);   // stored in blocks of 256 rows x 64 columns
    SplitNeed need(ds);
    SplitNeed::chunks(T, b.chunk, [&](size_t Tc) {
        need.product<CfgBlockedANN>(Tc, (size_t)ds.d, b.Vp);                         // dH
        need.product<CfgBlockedTN>((size_t)ds.V, (size_t)ds.d, round_up(Tc, 64));    // dF
    });
    b.split_bytes = need.bytes;
    b.split = take(need.bytes);
    b.total = off;
    return b;
}

inline bool dims_fit(const cp_head_desc &ds)
{
    // the GEMM addresses rows of a tile with 32-bit byte offsets and counts rows in int
    const size_t nrd = (size_t)ds.n * ds.r * ds.d, M = (size_t)ds.T * ds.n * ds.r;
    const size_t max_ld = (nrd > (size_t)ds.V + 64 ? nrd : (size_t)ds.V + 64) + 64;
    return M < ((size_t)1 << 31) && nrd < ((size_t)1 << 31) && max_ld * 2 * 256 < ((size_t)1 << 32) &&
           ((size_t)ds.T + 128) * 2 * 256 < ((size_t)1 << 32);
}

}  // namespace

// rows of a 64-row tile: the draft GEMMs with at most this many rows stream their big operand with
// two 80 KB workgroups per compute unit instead of one 128 KB workgroup
typedef TileCfg<64, 256, 1, 4> CfgSkinny;
// rows up to which the z product of a draft-type call uses the 64-row tile (several tile rows then share the
// slices of U through L2: their workgroups are neighbours in the tile walk)
#ifndef CPH_SKINNY_ROWS
#define CPH_SKINNY_ROWS 64
#endif
constexpr int kSkinnyRows = CPH_SKINNY_ROWS;
// y = W_sa h for at most 16 positions: W goes from memory straight into the registers that the matrix instruction
// reads.  The tiled main loop waits for a stage of LDS at every K-step, d / 64 times a memory latency, which the other
// workgroups of a compute unit hide only where there are two on each (512 tiles of 256 columns); here a workgroup has
// 16 columns of y, and eight or more workgroups, whose loads overlap, share a compute unit.
// The four wavefronts share the contraction, AHEAD blocks of 64 columns in flight each, and their partial products meet in LDS.
constexpr int kStreamRows = 16, kStreamWaves = 4, kStreamBlock = kStreamWaves * kWave;
template <int AHEAD>
__global__ void __launch_bounds__(kStreamBlock) k_stream_y(const bf16_t *__restrict__ H, int B, int d,
                                                           const bf16_t *__restrict__ W, int cols, bf16_t *__restrict__ Y,
                                                           GatePickSide side)
{
    __shared__ float sums[kStreamWaves][16][17];
    if ((int)blockIdx.x < side.blocks) {
        side.run(blockIdx.x, reinterpret_cast<char *>(sums));
        return;
    }
    const int col0 = ((int)blockIdx.x - side.blocks) * 16;       // cols is a multiple of 64
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row = lane & 15, q = lane >> 4;
    const bf16_t *const ph[1] = {H + (size_t)min(row, B - 1) * d + q * 16};     // rows past the last one repeat it, not stored
    const bf16_t *pw = W + (size_t)(col0 + row) * d + q * 16;
    f32x4_t acc[1] = {{0.f, 0.f, 0.f, 0.f}};
    tile16_products<kStreamWaves, AHEAD>(pw, ph, d, wave, acc);
#pragma unroll
    for (int v = 0; v < 4; ++v) sums[wave][tile16_row(v, lane)][row] = acc[0][v];
    __syncthreads();
    const int t = threadIdx.x >> 4, col = threadIdx.x & 15;
    if (t < B)
        Y[(size_t)t * cols + col0 + col] = f32_to_bf16((sums[0][col][t] + sums[1][col][t]) + (sums[2][col][t] + sums[3][col][t]));
}
// Where it is the faster one (whole first-token calls at V = 16000, us, this against the tiles; T positions):
//   cols 16384 (d 2048): T = 1 64 / 84, T = 16 82 / 99       cols 32768 (d 4096): T = 1 133 / 163, T = 16 174 / 185
//   cols 65536 (d 4096): T = 1 182 / 211, T = 8 223 / 232, T = 16 256 / 238
//   cols 98304 (d 4096): T = 1 228 / 246, T = 4 257 / 253, T = 16 323 / 261
// The tiles catch up where they fill the chip and where the rows of H differ: each workgroup reads all of them from L2.
// (Measured with one block in flight.)  Two in flight where fewer than two workgroups share a compute unit or the rows are long.  Draft calls at
// V = 2000, us, one / two, on cold weights:
//   T = 1: d 1536 cols 3072 26.3 / 25.2; d 4096 cols 4096 45.1 / 42.5; d 2560 cols 5120 36.1 / 35.1; d 2048 cols 8192 34.1 / 34.2, cols 32768 52.7 / 54.9;
//     d 1024 cols 32768 37.6 / 37.6; d 1536 cols 24576 38.0 / 37.3; d 2560 cols 20480 49.9 / 48.2; d 3072 cols 24576 58.5 / 56.3; d 4096 cols 32768 87.1 / 83.0
//   T = 4: d 4096 cols 4096 46.3 / 44.0; d 2048 cols 16384 50.0 / 51.1, cols 32768 76.3 / 78.1; d 4096 cols 32768 110.1 / 104.2
//   T = 16: d 4096 cols 4096 49.0 / 47.1; d 1024 cols 32768 60.5 / 60.8; d 2048 cols 32768 97.7 / 101.8; d 3072 cols 24576 121.4 / 121.6
// (the first-token call at T = 4, d 2048, cols 16384 by its vocabulary: V 2000 43.4 / 42.8 for two / one, V 32000 55.2 / 55.3) and on weights that the
// caches hold: T = 1: d 2048 cols 32768 46.8 / 51.5; d 2560 cols 20480 42.8 / 42.0; d 4096 cols 32768 76.6 / 78.7.
inline bool stream_y_two_ahead(int cols, int d) { return cols < 8192 || d > 2048; }
inline bool stream_y(int B, int cols) { return B <= kStreamRows && (cols <= 32768 || (cols <= 65536 && B <= 8)); }

// y = W_sa h for the first `heads` of the n r head matrices (bf16, rounded: part of the draft distribution's
// definition), with the gate (and the expert draw, if uniforms is given) as the launch's side job
inline void launch_y_with_gate(const char *name, const cp_head_desc &ds, const bf16_t *H, const bf16_t *W, const bf16_t *G,
                               const float *uniforms, bf16_t *Y, float *logw, int32_t *alpha, int heads, hipStream_t st)
{
    const int B = (int)ds.T, d = ds.d, cols = heads * d;
    const GatePickSide side{(B + 7) / 8 * 8, B, d, ds.n, ds.r, H, G, uniforms, logw, alpha};
    const EpiStoreBf16 epi{Y, nullptr, (long)cols, B, cols};
    if (stream_y(B, cols)) {
        ProfileScope prof(name, 2.0 * (double)B * (double)cols * (double)d, st);
        auto kernel = stream_y_two_ahead(cols, d) ? k_stream_y<2> : k_stream_y<1>;
        kernel<<<side.blocks + cols / 16, kStreamBlock, 0, st>>>(H, B, d, W, cols, Y, side);
    } else if (B <= CfgSkinny::BM) launch_gemm_nt<CfgSkinny>(name, H, d, B, W, d, cols, d, epi, st, kGroupRowsWide, side);
    else launch_gemm_nt<Cfg>(name, H, d, B, W, d, cols, d, epi, st, kGroupRowsWide, side);
}
// z = U y for at most 32 head rows, the statistics of EpiRowStats per 64 columns and, unless z is null, the fp32 logits: U goes from memory straight
// into the registers of the matrix instruction, as W does in k_stream_y.  A workgroup has 64 columns, so that there are four
// times as many as tiles of 256 (128 beyond 16 rows, since every workgroup reads all of Y from L2); its wavefronts share the contraction and their partial products meet in LDS.
constexpr int kStreamZSeg = 64, kStreamZWaves = 8, kStreamZBlock = kStreamZWaves * kWave;
template <int NG>
struct StreamZ {
    static constexpr int CG = NG == 1 ? 4 : 8, COLS = 16 * CG, AHEAD = NG == 1 ? 2 : 1, WAVES_PER_SIMD = NG == 1 ? 4 : 2;
};
template <int NG>
__global__ void __launch_bounds__(kStreamZBlock, StreamZ<NG>::WAVES_PER_SIMD) k_stream_z(const bf16_t *__restrict__ Y, int rows, int d,
                                                                                         const bf16_t *__restrict__ U, int V,
                                                                                         float *__restrict__ z, long ldz,
                                                                                         float2 *__restrict__ part, int parts)
{
    constexpr int CG = StreamZ<NG>::CG, COLS = StreamZ<NG>::COLS;
    __shared__ __attribute__((aligned(16))) float sums[kStreamZWaves][NG * 16][COLS + 4];
    const int col0 = (int)blockIdx.x * COLS;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row = lane & 15, q = lane >> 4;
    const bf16_t *pu[CG], *py[NG];                // rows past the last one repeat it; they are masked or not stored
#pragma unroll
    for (int c = 0; c < CG; ++c) pu[c] = U + (size_t)min(col0 + 16 * c + row, V - 1) * d + q * 16;
#pragma unroll
    for (int g = 0; g < NG; ++g) py[g] = Y + (size_t)min(16 * g + row, rows - 1) * d + q * 16;
    f32x4_t acc[CG][NG];
#pragma unroll
    for (int c = 0; c < CG; ++c)
#pragma unroll
        for (int g = 0; g < NG; ++g) acc[c][g] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    tile16_products_2d<kStreamZWaves, StreamZ<NG>::AHEAD>(pu, py, d, wave, acc);
#pragma unroll
    for (int c = 0; c < CG; ++c)
#pragma unroll
        for (int g = 0; g < NG; ++g) *reinterpret_cast<f32x4_t *>(&sums[wave][16 * g + row][16 * c + 4 * q]) = acc[c][g];
    __syncthreads();
    const int r = threadIdx.x >> 4;               // a row, and four columns of each segment, per thread; 16 threads per row
    if (r >= NG * 16 || r >= rows) return;        // whole groups of 16 lanes
#pragma unroll
    for (int s = 0; s < COLS / kStreamZSeg; ++s) {
        const int c4 = s * kStreamZSeg + (threadIdx.x & 15) * 4, seg = (int)blockIdx.x * (COLS / kStreamZSeg) + s;
        f32x4_t v = *reinterpret_cast<const f32x4_t *>(&sums[0][r][c4]);
#pragma unroll
        for (int w = 1; w < kStreamZWaves; ++w) v += *reinterpret_cast<const f32x4_t *>(&sums[w][r][c4]);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = col0 + c4 + e < V ? v[e] : -INFINITY;
        if (z && col0 + c4 < ldz) *reinterpret_cast<f32x4_t *>(z + (size_t)r * ldz + col0 + c4) = v;
        const float mx = row16_max(fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3])));
        const float ref = mx == -INFINITY ? 0.f : mx;
        const float sum = row16_sum((__expf(v[0] - ref) + __expf(v[1] - ref)) + (__expf(v[2] - ref) + __expf(v[3] - ref)));
        if ((threadIdx.x & 15) == 0 && seg < parts) part[(size_t)r * parts + seg] = make_float2(mx, sum);
    }
}
// Where it is the faster one (whole calls on cold weights, us, tiles / this, first token with r = 8 unless given):
//   up to 16 rows, two workgroups of 64 columns per compute unit: T = 1: d 512 V 32000 25.7 / 19.0; d 1024 V 33000 37.5 / 30.5, V 50000 39.8 / 36.4,
//     V 65000 43.6 / 40.8; d 2048 V 16000 57 / 37, V 65000 94 / 79; d 4096 V 32000 138 / 114, V 65000 186 / 168; draft T = 2, d 1024, V 33000 40.9 / 38.0
//   up to 32 rows, one workgroup of 128 columns per compute unit, so that 32768 columns are a round: T = 4: d 512 V 4000 22.0 / 17.6, V 32000 26.6 / 23.1,
//     V 33000 27.3 / 29.3, V 65000 33.2 / 34.5; d 1024 V 32000 37.3 / 31.4, V 33000 38.4 / 42.0, V 50000 42.9 / 44.5, V 65000 47.3 / 49.2; d 2048 V 32000
//     65.2 / 55.2, V 33000 65.1 / 72.8, V 50000 79.5 / 79.4, V 65000 97 / 89; d 4096 V 33000 144 / 155, V 50000 165 / 163, V 65000 193 / 179;
//     draft T = 4: d 1024 V 16000 39 / 34, V 33000 43.9 / 47.5, V 65000 50 / 53; d 2048 V 65000 98 / 93; d 4096 V 65000 200 / 185
// From about 65536 columns on the tiles have the loads in flight that the stream has, and read Y less often.  Beyond one round it needs wide
// rows, and rounds that are seven eighths full (V 50000 on weights that the caches hold: d 2048 62.4 / 67.4).
constexpr int kStreamZRows = 32, kStreamZMost = 65536;
inline bool stream_z(int rows, int V, int d)
{
    if (rows > kStreamZRows || V > kStreamZMost) return false;
    if (rows <= 16) return true;
    const int groups = (V + StreamZ<2>::COLS - 1) / StreamZ<2>::COLS, rounds = (groups + 255) / 256;
    return rounds == 1 || (d >= 2048 && groups * 8 >= rounds * 256 * 7);
}

// statistics segments (pairs per row, columns per segment) of the z product of a draft-type call
inline void z_segments(int rows, int V, int d, int &parts, int &seg_cols)
{
    if (stream_z(rows, V, d)) {
        parts = (V + kStreamZSeg - 1) / kStreamZSeg;
        seg_cols = kStreamZSeg;
    } else if (rows <= kSkinnyRows) {
        parts = ((V + CfgSkinny::BN - 1) / CfgSkinny::BN) * CfgSkinny::WN;
        seg_cols = CfgSkinny::WTN;
    } else {
        parts = ((V + Cfg::BN - 1) / Cfg::BN) * Cfg::WN;
        seg_cols = Cfg::WTN;
    }
}
// z = U y for the few rows of a draft-type call with its statistics, and the logits themselves unless z is null; streams U once
inline void launch_z_stats(const char *name, const bf16_t *Y, int d, int rows, const bf16_t *U, int V, float2 *part, int parts, float *z,
                           long ldz, hipStream_t st)
{
    auto tiles = [&](auto epi) {
        if (rows <= kSkinnyRows) launch_gemm_nt<CfgSkinny>(name, Y, d, rows, U, d, V, d, epi, st, kSkinnyRows / CfgSkinny::BM);
        else launch_gemm_nt<Cfg>(name, Y, d, rows, U, d, V, d, epi, st);
    };
    if (stream_z(rows, V, d)) {
        ProfileScope prof(name, 2.0 * (double)rows * V * d, st);
        if (rows <= 16) k_stream_z<1><<<blocks_for(V, StreamZ<1>::COLS), kStreamZBlock, 0, st>>>(Y, rows, d, U, V, z, ldz, part, parts);
        else k_stream_z<2><<<blocks_for(V, StreamZ<2>::COLS), kStreamZBlock, 0, st>>>(Y, rows, d, U, V, z, ldz, part, parts);
    } else if (z) {
        tiles(EpiRowStatsStore{part, parts, rows, V, z, ldz, 0});
    } else {
        tiles(EpiRowStats{part, parts, rows, V});
    }
}

struct DraftWs {
    size_t logw, Y, part, lse, seg, base, zseg, zseg_bytes, total;
    int parts_max;
};
// The logits of the segments that the draws fall into lie where the statistics are.  The expert-first draws are all
// found before any of those logits are formed, so the statistics have done their work then; `part` grows to what all draws
// need (256 or 512 bytes per head row, more than the statistics of vocabularies below 2048 or 4096) unless the call fits
// CP_HEAD_STATIC_SCRATCH_BYTES only without: then it takes what is left there, and the logits come a group of draws at a
// time.  The sequential draws need the statistics to the end but only one draw's logits at a time, for which the half
// of `part` that 128-column segments leave free is enough from 32 tiles of 256 columns and draws on.
inline DraftWs draft_ws(const cp_head_desc &ds, bool sequential)
{
    DraftWs f;
    const size_t rows = (size_t)ds.T * ds.r, M = rows * ds.n;
    const size_t tiles = ((size_t)ds.V + Cfg::BN - 1) / Cfg::BN;
    const size_t draw_bytes = (size_t)ds.r * (M > (size_t)kSkinnyRows ? Cfg::WTN : CfgSkinny::WTN) * 4;      // of one draw
    f.parts_max = (int)tiles * CfgSkinny::WN;   // the finer of the two segmentations
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes); return o; };
    f.logw = take(rows * 4);
    f.Y = take(M * ds.d * 2);
    f.lse = take(M * 4);
    f.seg = take((size_t)ds.T * ds.n * 4);
    f.base = take((size_t)ds.T * ds.n * 8);
    const size_t part_bytes = align_up(M * f.parts_max * sizeof(float2));
    f.part = off;
    if (!sequential) {
        f.zseg = f.part;
        const size_t all = std::max(part_bytes, align_up((size_t)ds.T * ds.n * draw_bytes)), limit = CP_HEAD_STATIC_SCRATCH_BYTES;
        f.zseg_bytes = off + part_bytes <= limit && off + all > limit ? std::max(limit - off, align_up(draw_bytes)) : all;
        off += f.zseg_bytes;
    } else {
        off += part_bytes;
        f.zseg_bytes = (size_t)ds.T * draw_bytes;
        const size_t used = M * tiles * Cfg::WN * sizeof(float2);
        if (M > (size_t)kSkinnyRows && used + f.zseg_bytes <= part_bytes) f.zseg = f.part + used;
        else f.zseg = take(f.zseg_bytes);
    }
    f.total = off;
    return f;
}

// Whether the mixture forms the log-normalisers itself: all its workgroups read all pairs of a b's statistics, kMixPairs of them at most
// (they are a chain in the workgroup) and kMixReads over the launch.  Whole calls on cold weights, us, a launch of their own / in the mixture:
//   B = 1, d = 512, r = 8: V = 4000 23.3 / 21.4, 32000 (4000 pairs, 0.5 M reads) 27.2 / 25.7, 128256 (16032 pairs) 43.6 / 44.7; r = 64, V = 32000
//   (32000 pairs) 86.8 / 101;  B = 4, d = 1024, r = 8, V = 32000 (2.0 M) 37.8 / 37.3;  B = 17, r = 1: V = 32000 (1.1 M) 48.3 / 48.3, 50000 (2.6 M)
//   52.6 / 53.2, 65000 (4.4 M) 58.4 / 60.4;  B = 64, r = 1: d = 1024, V = 32000 (4.0 M) 53.7 / 57.9, d = 64, V = 128256 (64 M) 40.3 / 75.9
// And the chain stands in front of every workgroup, so that there may not be many of them either, fewer with many experts.  d = 64, calls after one
// another: r = 1: 2016 workgroups (B = 32, V = 16000) 14.2 / 12.7, 2048 (B = 256, V = 2000) 29.1 / 28.2, 4000 (B = 500, V = 2000) 31.1 / 31.7, 4032 (B = 64)
//   17.7 / 18.3, 16000 (B = 500, V = 8000) 43.3 / 50.9, 32000 (B = 1000, V = 8000) 53.4 / 69.6;  r = 2: 2048 (B = 64, V = 8000) 24.9 / 24.0, 4032 28.2 / 28.5;
//   r = 8: 1008 (B = 16, V = 16000) 28.5 / 27.2, 1024 (B = 128, V = 2000) 32.6 / 31.3, 2016 (B = 32, V = 16000) 36.2 / 36.7, 4096 (B = 128, V = 8000) 45.9 / 47.9
constexpr long kMixPairs = 4096, kMixReads = 1 << 21, kMixGroups = 2048, kMixGroupsMany = 1024;
inline bool mix_from_parts(long B, long V, long r, long parts)
{
    const long groups = B * (long)blocks_for((size_t)V, kBlock);
    return r * parts <= kMixPairs && groups * r * parts <= kMixReads && groups <= (r <= 4 ? kMixGroups : kMixGroupsMany);
}

// Whether the statistics of the stored logits come from a pass over them instead of from the epilogue of 256-row tiles.  The epilogue forms
// them for all 256 rows of a tile, 7 us at the end of a launch of few tiles; the pass costs the logits' bytes once more.  Whole calls on cold weights, us,
// epilogue / pass:
//   72 rows (r = 8): d 64: V 8000 23.9 / 20.6, V 32000 27.8 / 25.9, V 128256 51.5 / 49.2; d 1024 V 128256 104.2 / 99.1; d 2048 V 128256 191.5 / 187.6
//   128 rows (r = 8): d 512 V 8000 33.4 / 32.0, V 16000 35.5 / 33.9, V 128256 85.7 / 86.3;   256 rows: r = 1, d 512 V 8000 55.0 / 53.5;
//     r = 8, d 64 V 8000 29.7 / 28.4, V 16000 33.6 / 34.2;   512 rows (r = 8): d 64 V 4000 30.6 / 29.0, V 8000 33.5 / 34.4
//   1024 rows (r = 8): d 64 V 2000 31.2 / 29.5, V 16000 52.0 / 58.6;   2048 rows (r = 8): d 64 V 1000 35.5 / 33.8;   8000 rows (r = 8): d 64 V 300 42.3 / 46.2
constexpr int kApartRows = 96, kApartMostRows = 2048;
constexpr long kApartLogits = 5L << 19;
inline bool stats_apart(int rows, int V)
{
    return rows > kSkinnyRows && (rows <= kApartRows || (rows <= kApartMostRows && (long)rows * V <= kApartLogits));
}

struct FirstTokenWs {
    size_t logw, Y, z, lse, part, total;
    size_t V4;
    int parts, seg_cols;
};
inline FirstTokenWs first_token_ws(const cp_head_desc &ds)
{
    FirstTokenWs f;
    const size_t rows = (size_t)ds.T * ds.r;
    f.V4 = round_up((size_t)ds.V, 4);
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes); return o; };
    f.logw = take(rows * 4);
    f.Y = take(rows * ds.d * 2);
    f.z = take(rows * f.V4 * 4);
    f.lse = take(rows * 4);
    z_segments((int)rows, ds.V, ds.d, f.parts, f.seg_cols);
    f.part = take(rows * f.parts * sizeof(float2));
    f.total = off;
    return f;
}

size_t fast_workspace_bytes(const cp_head_desc &ds, int op)
{
    if (op == CP_HEAD_OP_LOSS_FWD) return fwd_ws(ds).total;
    if (op == CP_HEAD_OP_LOSS_BWD) return bwd_ws(ds).total;
    if (op == CP_HEAD_OP_FIRST_TOKEN) return first_token_ws(ds).total;
    if (op == CP_HEAD_OP_FULL_LOSS_FWD) return full_fwd_ws(ds).total;
    if (op == CP_HEAD_OP_FULL_LOSS_BWD) return full_bwd_ws(ds).total;
    return draft_ws(ds, op == CP_HEAD_OP_DRAFT_SEQUENTIAL).total;
}

namespace {
// Where the per-row part of a forward pass has its buffers, and its two steps before the logits.
struct FwdRows {
    FwdWs f;
    CtxLayout cl;
    FastFwdBuffers b;
    bf16_t *Ylo;
    float2 *part;
    FwdRows(const cp_head_desc &ds, void *ctx, void *ws) : f(fwd_ws(ds)), cl(ctx_layout(ds, true))
    {
        b.lse = at<float>(ctx, cl.lse); b.w = at<float>(ctx, cl.w); b.gamma = at<float>(ctx, cl.gamma);
        b.Y = at<bf16_t>(ctx, cl.Y);
        b.logw = at<float>(ws, f.logw); b.C = at<float>(ws, f.C);
        Ylo = at<bf16_t>(ws, f.Ylo);
        part = cl.keep ? at<float2>(ctx, cl.zpart) : at<float2>(ws, f.part);
    }
    void gate_and_y(const cp_head_desc &ds, const bf16_t *H, const bf16_t *W, const bf16_t *G, void *ws, hipStream_t st) const
    {
        const int T = (int)ds.T, d = ds.d, nrd = ds.n * ds.r * d;
        launch_gate_bf16(ds, H, G, b.logw, b.w, st);                                                            // eq. 7
        launch_gemm_nt<Cfg>("gemm_y", H, d, T, W, d, nrd, d, EpiStoreBf16{b.Y, Ylo, (long)nrd, T, nrd}, st, kGroupRowsNarrow,
                            NoSideJob{0}, -1, -1, split_scratch(ws, f.split, f.split_bytes));                   // y = W_sa h
    }
    // log-normalisers and C of the rows m0 .. m0 + Mc - 1 (whole positions) from their statistics
    void finish(const cp_head_desc &ds, size_t m0, size_t Mc, const bf16_t *U, const int32_t *X, hipStream_t st) const
    {
        k_row_finish<<<blocks_for(Mc, kBlock / kWave), kBlock, 0, st>>>(Mc, ds.d, ds.r, f.parts, part + m0 * f.parts, b.Y + m0 * ds.d,
                                                                        Ylo + m0 * ds.d, U, X + m0 / ds.r, b.lse + m0, b.C + m0);
    }
};
}  // namespace

// Everything of the forward pass that is per head row: gate (eq. 7), y, the statistics of z, the
// log-normalisers (eq. 5) and C (eq. 8).  `out` receives where the results live in ctx and ws.
int fast_fwd_rows(const cp_head_desc &ds, const void *Hv, const void *Wv, const void *Uv, const void *Gv,
                  const int32_t *X, void *ctx, void *ws, FastFwdBuffers *out, hipStream_t st)
{
    if (!dims_fit(ds)) return CP_HEAD_ERR_UNSUPPORTED;
    const bf16_t *U = (const bf16_t *)Uv;
    const FwdRows fr(ds, ctx, ws);
    const FwdWs &f = fr.f;
    const CtxLayout &cl = fr.cl;
    const int d = ds.d, V = ds.V;
    const size_t M = (size_t)ds.T * ds.n * ds.r;
    if (cl.keep && (cl.parts != f.parts || kKeptTile != Cfg::WTN)) return CP_HEAD_ERR_UNSUPPORTED;
    fr.gate_and_y(ds, (const bf16_t *)Hv, (const bf16_t *)Wv, (const bf16_t *)Gv, ws, st);
    if (cl.keep)                                                                               // z = U y, statistics, z kept
        launch_gemm_nt<Cfg>("gemm_z_stats_keep", fr.b.Y, d, (int)M, U, d, V, d,
                            EpiRowStatsKeep{fr.part, f.parts, (int)M, V, at<uint16_t>(ctx, cl.zs), (long)cl.Vp, (int)cl.Vp,
                                            streamed_store(M * cl.Vp * 2)}, st);
    else
        launch_gemm_nt<Cfg>("gemm_z_stats", fr.b.Y, d, (int)M, U, d, V, d, EpiRowStats{fr.part, f.parts, (int)M, V}, st);  // z = U y, statistics
    fr.finish(ds, 0, M, U, X, st);
    *out = fr.b;
    return hipGetLastError() == hipSuccess ? CP_HEAD_OK : CP_HEAD_ERR_LAUNCH;
}

// The rounds of the z product's tiles leave the least of the chip idle in their last one at some number of tile rows: the
// best one among those of at most kStoredLogitsBytes of fp32 logits (at least one tile row), as whole positions.  3 GiB, less
// than the backward call's logit gradients: chunks that stay in the last-level cache (200 MB) save the pass nothing and the
// product's rounds cost more (forward call at T = 4096, d = 1024, V = 32000, n = 4, r = 8: 200 MB 16.3 ms, 1.5 GiB 14.0, 3 GiB 13.6).
constexpr size_t kStoredLogitsBytes = (size_t)3 << 30;
size_t fast_stored_positions(const cp_head_desc &ds)
{
    const size_t nr = (size_t)ds.n * ds.r, row = round_up((size_t)ds.V, 64) * 4, T = (size_t)ds.T;
    const size_t tiles_n = ((size_t)ds.V + Cfg::BN - 1) / Cfg::BN, most = std::max<size_t>(kStoredLogitsBytes / (row * Cfg::BM), 1);
    if (T * nr <= most * Cfg::BM) return T ? T : 1;
    size_t best = most;
    double least = 1e30;
    for (size_t m = most; m >= 1 && m * 2 >= most; --m) {
        const double per_tile = (double)((m * tiles_n + 255) / 256) / (double)(m * tiles_n);
        if (per_tile < least) { least = per_tile; best = m; }
    }
    const size_t pos = best * Cfg::BM / nr;
    return pos < 1 ? 1 : pos;
}

// The same with the fp32 logits of a chunk of positions in z[rows of the chunk, ldz] for `fn` to pass over, chunk by chunk.
int fast_fwd_rows_stored(const cp_head_desc &ds, const void *Hv, const void *Wv, const void *Uv, const void *Gv, const int32_t *X,
                         void *ctx, void *ws, float *z, long ldz, FastStoredRows fn, void *user, FastFwdBuffers *out, hipStream_t st)
{
    if (!dims_fit(ds)) return CP_HEAD_ERR_UNSUPPORTED;
    const bf16_t *U = (const bf16_t *)Uv;
    const FwdRows fr(ds, ctx, ws);
    const int d = ds.d, V = ds.V;
    const size_t T = (size_t)ds.T, nr = (size_t)ds.n * ds.r, pos = fast_stored_positions(ds);
    *out = fr.b;
    fr.gate_and_y(ds, (const bf16_t *)Hv, (const bf16_t *)Wv, (const bf16_t *)Gv, ws, st);
    for (size_t t0 = 0; t0 < T; t0 += pos) {
        const size_t P = T - t0 < pos ? T - t0 : pos, m0 = t0 * nr;
        const int Mc = (int)(P * nr);
        launch_gemm_nt<Cfg>("gemm_z_stats_store", fr.b.Y + m0 * d, d, Mc, U, d, V, d,
                            EpiRowStatsStore{fr.part + m0 * fr.f.parts, fr.f.parts, Mc, V, z, ldz, streamed_store((size_t)Mc * ldz * 4)}, st);
        fr.finish(ds, m0, (size_t)Mc, U, X, st);
        fn(user, fr.b, t0, P, z, ldz, st);
    }
    return hipGetLastError() == hipSuccess ? CP_HEAD_OK : CP_HEAD_ERR_LAUNCH;
}

int fast_loss_fwd(const cp_head_desc &ds, const void *Hv, const void *Wv, const void *Uv, const void *Gv,
                  const int32_t *X, float *loss, void *ctx, void *ws, size_t, hipStream_t st)
{
    if (ds.T == 0) return CP_HEAD_OK;
    FastFwdBuffers b;
    const int rc = fast_fwd_rows(ds, Hv, Wv, Uv, Gv, X, ctx, ws, &b, st);
    if (rc != CP_HEAD_OK) return rc;
    launch_mixture(ds, b.logw, b.C, loss, b.gamma, -1.f, st);                                        // eq. 9
    return hipGetLastError() == hipSuccess ? CP_HEAD_OK : CP_HEAD_ERR_LAUNCH;
}

// Which operand layout each product of the backward pass uses.  The main loop reads a K-major operand (the
// contraction index is its slow one) with gfx950's transposing LDS read, which needs no transposed copy of anything
// but costs the loop 4-5 % per K-major operand (two 64-bit reads per fragment instead of one 128-bit read: twice the
// LDS instructions and LDS busy time for the same bytes; measured at the headline size: dY 97.3 -> 101.2 ms per step
// with U K-major, dH 12.5 -> 13.0, dW 12.7 -> 13.7).  U^T, W^T and Y^T are copies: those cost less than the loop does
// (0.1, 0.5 and 1.6 ms).  dz, which dY reads as rows and dU as columns, is read K-major by dU, and so are both operands of
// dW = dY^T H: a transposed copy of a logit-sized or row-sized buffer costs more than the loop.

// The backward pass below dY: dH = dY W + G^T dg, dW = dY^T H, dG = dg^T H.  Wt: scratch for W^T [d, n r d + 64];
// dGpart: the partial sums of the two-stage gate gradient.
static int bwd_below_dy(const cp_head_desc &ds, const bf16_t *H, const bf16_t *W, const bf16_t *G, const bf16_t *dY,
                        const float *dg, float *dH, float *dW, float *dG, bf16_t *Wt, float *dGpart,
                        const SplitScratch &split, hipStream_t st)
{
    const int d = ds.d, r = ds.r;
    const size_t T = (size_t)ds.T, nrd = (size_t)ds.n * r * d;
    const long ldN = (long)nrd + 64;
    // dH = dY W + G^T dg   (contraction over (s, a, k))
    transpose_bf16(W, d, (int)nrd, d, Wt, ldN, (int)nrd, st);         // Wt[d, nrd]
    launch_gemm_nt<Cfg>("gemm_dh", dY, (long)nrd, (int)T, Wt, ldN, d, (int)nrd, EpiStoreF32{dH, (long)d, (int)T, d, 0}, st,
                        kGroupRowsNarrow, NoSideJob{0}, -1, -1, split);
    k_add_gate_to_dh<<<blocks_for(T * d / 4, kBlock), kBlock, 0, st>>>(T, d, r, G, dg, dH);
    if (dW)
        // dW_sa = dY_sa^T H   (contraction over positions: both operands K-major, any number of positions)
        launch_gemm_nt<CfgTN>("gemm_dw", dY, (long)nrd, (int)nrd, H, d, d, (int)T, EpiStoreF32{dW, (long)d, (int)nrd, d, 0}, st,
                              kGroupRowsNarrow, NoSideJob{0}, -1, -1, split);
    if (dG) launch_gate_gradient_bf16(ds, H, dg, dGpart, dG, st);
    return hipGetLastError() == hipSuccess ? CP_HEAD_OK : CP_HEAD_ERR_LAUNCH;
}

// dY = dz U and dU (+)= dz^T Y for one chunk of head rows whose dz is in place.
// dZ is stored block by block (blocked64_index, ld = Vp): its rows are 2 Vp bytes apart otherwise, a tile's K-step
// touches 256 separate cache lines of it, and the product, which streams the chunk's 4 GiB of it from HBM, runs 4 %
// slower.  Ut: U^T [d, Vp + 64]; Yt: scratch for the chunk's Y^T [d, Mcp + 64].
static void bwd_chunk_products(const cp_head_desc &ds, const bf16_t *dZ, long ldM, const bf16_t *Yc, int Mc, const bf16_t *Ut, bf16_t *Yt, bf16_t *dYc, float *dU, bool accumulate,
                               const SplitScratch &split, hipStream_t st)
{
    const int d = ds.d, V = ds.V;
    const int Vp = (int)round_up((size_t)V, 64), Mcp = (int)round_up((size_t)Mc, 64);
    const long ldV = (long)Vp + 64;
    // dY = dz U   (contraction over the vocabulary)
    launch_gemm_nt<CfgBlockedA>("gemm_dy", dZ, Vp, Mc, Ut, ldV, d, Vp, EpiStoreBf16{dYc, nullptr, (long)d, Mc, d}, st,
                                kGroupRowsNarrow, NoSideJob{0}, -1, -1, split_dy(ds) ? split : SplitScratch());
    if (dU) {
        // dU += dz^T Y   (contraction over the rows of the chunk)
        transpose_bf16(Yc, d, Mc, d, Yt, ldM, Mcp, st);               // Yt[d, Mcp]
        launch_gemm_nt<CfgBlockedTN>("gemm_du", dZ, Vp, V, Yt, ldM, d, Mcp, EpiStoreF32{dU, (long)d, V, d, accumulate ? 1 : 0}, st,
                            kGroupRowsNarrow, NoSideJob{0}, -1, -1, split);
    }
}

// The backward pass below the logit gradients: per bounded chunk of head rows `dz_launch` writes dz
// (bf16), then dY = dz U and dU += dz^T Y; afterwards
// dW = dY^T H, dH = dY W + G^T dg and dG = dg^T H.  dg[T,r] must already hold the gate gradients.
int fast_bwd_from_dz(const cp_head_desc &ds, const void *Hv, const void *Wv, const void *Uv, const void *Gv,
                     const void *Yv, const float *dg, float *dH, float *dW, float *dU, float *dG, void *ws,
                     FastDzLaunch dz_launch, void *user, hipStream_t st)
{
    const int d = ds.d, V = ds.V, r = ds.r, n = ds.n;
    const bf16_t *H = (const bf16_t *)Hv, *W = (const bf16_t *)Wv, *U = (const bf16_t *)Uv, *G = (const bf16_t *)Gv;
    const bf16_t *Y = (const bf16_t *)Yv;
    const BwdWs b = bwd_ws(ds);
    const size_t T = (size_t)ds.T, M = T * n * r;
    bf16_t *Ut = at<bf16_t>(ws, b.Ut), *Wt = at<bf16_t>(ws, b.Wt), *dY = at<bf16_t>(ws, b.dY);
    bf16_t *dZ = at<bf16_t>(ws, b.dZ), *Yt = at<bf16_t>(ws, b.Yt);
    const int Vp = (int)b.Vp;
    const SplitScratch split = split_scratch(ws, b.split, b.split_bytes);

    transpose_bf16(U, d, V, d, Ut, (long)b.ldV, Vp, st);              // Ut[d, Vp]
    int first = 1;
    for (size_t m0 = 0; m0 < M; m0 += b.chunk) {
        const int Mc = (int)((M - m0 < b.chunk) ? M - m0 : b.chunk);
        const int Mcp = (int)round_up((size_t)Mc, 64);
        const bf16_t *Yc = Y + m0 * d;
        // recompute z for the chunk; the epilogue turns it into dz (bf16); the tiles over V also
        // cover the padding columns V..Vp-1, which the epilogue zero-fills
        dz_launch(user, Yc, Mc, Mcp, m0, dZ, Vp, st);
        bwd_chunk_products(ds, dZ, (long)b.ldM, Yc, Mc, Ut, Yt, dY + m0 * d, dU, !first, split, st);
        first = 0;
    }
    return bwd_below_dy(ds, H, W, G, dY, dg, dH, dW, dG, Wt, at<float>(ws, b.dGpart), split, st);
}

bool fast_dims_fit(const cp_head_desc &ds) { return dims_fit(ds); }

namespace {
struct LossDzArgs {
    const bf16_t *U;
    const float4 *rowinfo;
    int d, V;
};
// dz of the training loss: dz[m, v] = coef[m] (exp(z - lse[m]) - 1[v = x_m])
void loss_dz_launch(void *user, const bf16_t *Yc, int Mc, int Mcp, size_t m0, bf16_t *dZ, int Vp, hipStream_t st)
{
    const LossDzArgs *a = static_cast<const LossDzArgs *>(user);
    launch_gemm_nt<Cfg>("gemm_z_dz", Yc, a->d, Mc, a->U, a->d, a->V, a->d,
                        EpiDz{dZ, (long)Vp, a->rowinfo + m0, Mc, Mcp, a->V, Vp, streamed_store((size_t)Mc * Vp * 2)}, st);
}

struct KeptDzArgs {
    KeptLogits kept;         // zs [M, Vp], part [M, parts]
    const float4 *rowinfo;
    int V;
};
// the same dz from the logits kept by the forward pass
void kept_dz_launch(void *user, const bf16_t *, int Mc, int Mcp, size_t m0, bf16_t *dZ, int Vp, hipStream_t st)
{
    const KeptDzArgs *a = static_cast<const KeptDzArgs *>(user);
    launch_dz_from_kept(a->kept, m0, a->rowinfo + m0, LossDzRule{}, Mc, Mcp, a->V, dZ, Vp, st);
}
}  // namespace

int fast_loss_bwd(const cp_head_desc &ds, const void *Hv, const void *Wv, const void *Uv, const void *Gv,
                  const int32_t *X, const float *dloss, float scale, const void *ctx, float *dH, float *dW,
                  float *dU, float *dG, void *ws, size_t, hipStream_t st)
{
    const int d = ds.d, V = ds.V, r = ds.r, n = ds.n;
    const size_t nrd = (size_t)n * r * d;
    if (ds.T == 0) {
        launch_fill_zero(dW, nrd * d, st);
        launch_fill_zero(dU, (size_t)V * d, st);
        launch_fill_zero(dG, (size_t)r * d, st);
        return hipGetLastError() == hipSuccess ? CP_HEAD_OK : CP_HEAD_ERR_LAUNCH;
    }
    if (!dims_fit(ds)) return CP_HEAD_ERR_UNSUPPORTED;
    const CtxLayout cl = ctx_layout(ds, true);
    const BwdWs b = bwd_ws(ds);
    const size_t M = (size_t)ds.T * n * r;
    const float *lse = at<float>(ctx, cl.lse), *w = at<float>(ctx, cl.w), *gamma = at<float>(ctx, cl.gamma);
    float4 *rowinfo = at<float4>(ws, b.coef);
    float *dg = at<float>(ws, b.dg);
    k_bwd_coefficients<<<blocks_for(M, kBlock), kBlock, 0, st>>>(M, n, r, w, gamma, lse, dloss, scale, X, rowinfo, dg);
    if (cl.keep) {
        KeptDzArgs kept{KeptLogits{at<uint16_t>(ctx, cl.zs), at<float2>(ctx, cl.zpart), (long)cl.Vp, cl.parts}, rowinfo, V};
        return fast_bwd_from_dz(ds, Hv, Wv, Uv, Gv, at<bf16_t>(ctx, cl.Y), dg, dH, dW, dU, dG, ws, kept_dz_launch, &kept, st);
    }
    LossDzArgs args{(const bf16_t *)Uv, rowinfo, d, V};
    return fast_bwd_from_dz(ds, Hv, Wv, Uv, Gv, at<bf16_t>(ctx, cl.Y), dg, dH, dW, dU, dG, ws, loss_dz_launch, &args, st);
}

// ------------------------------------------------------------------------------------------
// training step in one call: loss and gradients, one chunk of positions at a time
// ------------------------------------------------------------------------------------------

// Positions per chunk: whole positions whose head rows fit the backward pass's bound on logit-sized buffers.
struct StepWs {
    size_t logw, w, gamma, dg, dGpart, Ut, Wt, dY, C, lse, coef, Yc, Ylo, part, zs, dZ, Yt, split, split_bytes, total;
    size_t Vp, pos, rows, ldM;
    int parts;
};
inline StepWs step_ws(const cp_head_desc &ds)
{
    StepWs f;
    const size_t T = (size_t)ds.T, nr = (size_t)ds.n * ds.r, M = T * nr, nrd = nr * ds.d;
    f.Vp = round_up((size_t)ds.V, 64);
    f.parts = ((ds.V + Cfg::BN - 1) / Cfg::BN) * Cfg::WN;
    f.pos = bwd_chunk_rows(ds) / nr;
    if (f.pos < 1) f.pos = 1;
    if (f.pos > T) f.pos = T ? T : 1;
    f.rows = f.pos * nr;
    f.ldM = round_up(f.rows, 64) + 64;
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes); return o; };
    f.logw = take(T * ds.r * 4);
    f.w = take(T * ds.r * 4);
    f.gamma = take(T * ds.r * 4);
    f.dg = take(T * ds.r * 4);
    f.dGpart = take(gate_chunks(T) * ds.r * ds.d * 4);
    f.Ut = take((size_t)ds.d * (f.Vp + 64) * 2);
    f.Wt = take((size_t)ds.d * (nrd + 64) * 2);
    f.dY = take(M * ds.d * 2);
    f.C = take(f.rows * 4);
    f.lse = take(f.rows * 4);
    f.coef = take(f.rows * 16);
    f.Yc = take(f.rows * ds.d * 2);
    f.Ylo = take(f.rows * ds.d * 2);
    f.part = take(f.rows * f.parts * sizeof(float2));
    f.zs = take(f.rows * f.Vp * 2);
    f.dZ = take(round_up(f.rows, 256) * f.Vp * 2);   // stored in blocks of 256 rows x 64 columns
    f.Yt = take((size_t)ds.d * f.ldM * 2);
    SplitNeed need(ds);
    if (split_y(ds)) need.product<Cfg>(T, nrd, (size_t)ds.d);                        // y
    need_below_dz(ds, f.rows, need);
    f.split_bytes = need.bytes;
    f.split = take(need.bytes);
    f.total = off;
    return f;
}
size_t fast_step_workspace_bytes(const cp_head_desc &ds) { return step_ws(ds).total; }

// Forward and backward interleaved per chunk of positions.  The logits of a chunk are kept as 16-bit floats (as
// with CP_HEAD_KEEP_LOGITS, but for one chunk: the buffer does not grow with T) from the product that forms their
// statistics to the pass that turns them into gradients a few launches later, so U y is multiplied once per step.
int fast_loss_step(const cp_head_desc &ds, const void *Hv, const void *Wv, const void *Uv, const void *Gv,
                   const int32_t *X, const float *dloss, float scale, float *loss, float *dH, float *dW, float *dU,
                   float *dG, void *ws, hipStream_t st)
{
    const int d = ds.d, V = ds.V, r = ds.r, n = ds.n;
    const size_t nr = (size_t)n * r, nrd = nr * d, T = (size_t)ds.T;
    if (T == 0) {
        launch_fill_zero(dW, nrd * d, st);
        launch_fill_zero(dU, (size_t)V * d, st);
        launch_fill_zero(dG, (size_t)r * d, st);
        return hipGetLastError() == hipSuccess ? CP_HEAD_OK : CP_HEAD_ERR_LAUNCH;
    }
    if (!dims_fit(ds) || kKeptTile != Cfg::WTN) return CP_HEAD_ERR_UNSUPPORTED;
    const bf16_t *H = (const bf16_t *)Hv, *W = (const bf16_t *)Wv, *U = (const bf16_t *)Uv, *G = (const bf16_t *)Gv;
    const StepWs f = step_ws(ds);
    float *logw = at<float>(ws, f.logw), *w = at<float>(ws, f.w), *gamma = at<float>(ws, f.gamma), *dg = at<float>(ws, f.dg);
    float *C = at<float>(ws, f.C), *lse = at<float>(ws, f.lse);
    float4 *rowinfo = at<float4>(ws, f.coef);
    bf16_t *dY = at<bf16_t>(ws, f.dY), *Yc = at<bf16_t>(ws, f.Yc), *Ylo = at<bf16_t>(ws, f.Ylo), *dZ = at<bf16_t>(ws, f.dZ);
    float2 *part = at<float2>(ws, f.part);
    uint16_t *zs = at<uint16_t>(ws, f.zs);
    const int Vp = (int)f.Vp;
    const SplitScratch split = split_scratch(ws, f.split, f.split_bytes);

    bf16_t *Ut = at<bf16_t>(ws, f.Ut), *Yt = at<bf16_t>(ws, f.Yt);
    launch_gate_bf16(ds, (const bf16_t *)Hv, (const bf16_t *)Gv, logw, w, st);                                                             // eq. 7, all positions
    transpose_bf16(U, d, V, d, Ut, (long)f.Vp + 64, Vp, st);                                          // Ut[d, Vp]
    int first = 1;
    for (size_t t0 = 0; t0 < T; t0 += f.pos) {
        const size_t P = (T - t0 < f.pos) ? T - t0 : f.pos;
        const size_t m0 = t0 * nr;
        const int Mc = (int)(P * nr), Mcp = (int)round_up((size_t)Mc, 64);
        cp_head_desc sub = ds;
        sub.T = (int64_t)P;
        const int32_t *Xc = X + t0 * n;
        // forward of the chunk: y, statistics of z with the logits kept, log-normalisers and C (eq. 5, 8), mixture (eq. 9)
        launch_gemm_nt<Cfg>("gemm_y", H + t0 * d, d, (int)P, W, d, (int)nrd, d, EpiStoreBf16{Yc, Ylo, (long)nrd, (int)P, (int)nrd}, st,
                            kGroupRowsNarrow, NoSideJob{0}, -1, -1, split_y(ds) ? split : SplitScratch());
        launch_gemm_nt<Cfg>("gemm_z_stats_keep", Yc, d, Mc, U, d, V, d, EpiRowStatsKeep{part, f.parts, Mc, V, zs, (long)Vp, Vp, streamed_store((size_t)Mc * Vp * 2)},
                            st);
        k_row_finish<<<blocks_for((size_t)Mc, kBlock / kWave), kBlock, 0, st>>>((size_t)Mc, d, r, f.parts, part, Yc, Ylo, U, Xc, lse, C);
        launch_mixture(sub, logw + t0 * r, C, loss + t0, gamma + t0 * r, -1.f, st);
        // backward of the chunk down to dY and dU
        k_bwd_coefficients<<<blocks_for((size_t)Mc, kBlock), kBlock, 0, st>>>((size_t)Mc, n, r, w + t0 * r, gamma + t0 * r, lse,
                                                                            dloss ? dloss + t0 : nullptr, scale, Xc, rowinfo,
                                                                            dg + t0 * r);
        launch_dz_from_kept(KeptLogits{zs, part, (long)Vp, f.parts}, 0, rowinfo, LossDzRule{}, Mc, Mcp, V, dZ, Vp, st);
        bwd_chunk_products(ds, dZ, (long)f.ldM, Yc, Mc, Ut, Yt, dY + m0 * d, dU, !first, split, st);
        first = 0;
    }
    return bwd_below_dy(ds, H, W, G, dY, dg, dH, dW, dG, at<bf16_t>(ws, f.Wt), at<float>(ws, f.dGpart), split, st);
}

int fast_draft(const cp_head_desc &ds, const void *Hv, const void *Wv, const void *Uv, const void *Gv,
               const float *uniforms, int32_t *alpha, int32_t *tokens, float *logq, void *ws, size_t,
               hipStream_t st)
{
    if (ds.T == 0) return CP_HEAD_OK;
    if (!dims_fit(ds)) return CP_HEAD_ERR_UNSUPPORTED;
    const bf16_t *H = (const bf16_t *)Hv, *W = (const bf16_t *)Wv, *U = (const bf16_t *)Uv, *G = (const bf16_t *)Gv;
    const DraftWs f = draft_ws(ds, false);
    const int B = (int)ds.T, d = ds.d, V = ds.V, n = ds.n, r = ds.r;
    const size_t M = (size_t)B * n * r;
    float *logw = at<float>(ws, f.logw), *lse = at<float>(ws, f.lse);
    bf16_t *Y = at<bf16_t>(ws, f.Y);
    float2 *part = at<float2>(ws, f.part);
    int32_t *seg = at<int32_t>(ws, f.seg);
    double *base = at<double>(ws, f.base);
    float *zseg = at<float>(ws, f.zseg);
    const unsigned rows = (unsigned)(B * n);

    // y = W_sa h, rounded to bf16 (part of the draft distribution's definition); streams W once.  The gate and the
    // expert draw (eq. 7, a* ~ w) ride along as the launch's first workgroups.
    launch_y_with_gate("draft_gemm_y", ds, H, W, G, uniforms, Y, logw, alpha, n * r, st);
    // z = U y for all B*n*r rows with running statistics; streams U once, logits are not stored
    int parts, seg_cols;
    z_segments((int)M, V, d, parts, seg_cols);
    launch_z_stats("draft_gemm_z", Y, d, (int)M, U, V, part, parts, nullptr, 0, st);
    {
        ProfileScope prof("draft_lse_segment", (double)M * parts * 8, st);
        // one wavefront up to four segments a lane
        auto kernel = parts <= 4 * kWave ? k_draft_lse_segment<true> : k_draft_lse_segment<false>;
        kernel<<<rows, kWideBlock, 0, st>>>(n, r, parts, (V - 1) / seg_cols, part, alpha, uniforms, lse, seg, base);
    }
    if (!logq && rows >= kAloneDraws && rows <= kAloneDrawsMost) {
        ProfileScope prof("draft_pick", (double)rows * seg_cols * d * 2, st);
        k_draft_pick_alone<<<rows, kWideBlock, 0, st>>>(d, V, n, r, seg_cols, lse, Y, U, alpha, seg, base, uniforms, tokens);
        return hipGetLastError() == hipSuccess ? CP_HEAD_OK : CP_HEAD_ERR_LAUNCH;
    }
    // as many draws at a time as there is room for their logits: whole rows of the batch, or a part of one row's draws
    const int room = (int)std::min<size_t>(f.zseg_bytes / ((size_t)r * seg_cols * 4), rows);
    const int draws = std::min(n, room), group = std::max(room / n, 1);
    for (int b0 = 0; b0 < B; b0 += group)
        for (int s0 = 0; s0 < n; s0 += draws) {
            const int Bg = std::min(group, B - b0), Sg = std::min(draws, n - s0);
            const size_t bs0 = (size_t)b0 * n;
            {
                ProfileScope prof("draft_segment_logits", (double)Bg * Sg * seg_cols * d * 2, st);
                k_segment_logits<<<dim3((unsigned)(Bg * Sg), (unsigned)seg_cols / 16, (unsigned)(r + 15) / 16), kSegWaves * kWave, 0, st>>>(
                    d, V, n, r, seg_cols, s0, Sg, Y + bs0 * r * d, U, seg + bs0 + s0, n, zseg);
            }
            ProfileScope prof("draft_pick", (double)Bg * Sg * r * seg_cols * 4, st);
            k_draft_pick<<<(unsigned)Bg, kWideBlock, 0, st>>>(V, n, r, seg_cols, s0, Sg, logw + (size_t)b0 * r, lse + bs0 * r, zseg, alpha + b0,
                                                              seg + bs0, base + bs0, uniforms + (size_t)b0 * (1 + n), tokens + bs0,
                                                              logq ? logq + b0 : nullptr);
        }
    return hipGetLastError() == hipSuccess ? CP_HEAD_OK : CP_HEAD_ERR_LAUNCH;
}

int fast_first_token(const cp_head_desc &ds, const void *Hv, const void *Wv, const void *Uv, const void *Gv,
                     float *logp, void *ws, hipStream_t st)
{
    if (ds.T == 0) return CP_HEAD_OK;
    if (!dims_fit(ds)) return CP_HEAD_ERR_UNSUPPORTED;
    const bf16_t *H = (const bf16_t *)Hv, *W = (const bf16_t *)Wv, *U = (const bf16_t *)Uv, *G = (const bf16_t *)Gv;
    const FirstTokenWs f = first_token_ws(ds);
    const int B = (int)ds.T, d = ds.d, V = ds.V, r = ds.r;
    const int rows = B * r, V4 = (int)f.V4;
    float *logw = at<float>(ws, f.logw), *z = at<float>(ws, f.z), *lse = at<float>(ws, f.lse);
    bf16_t *Y = at<bf16_t>(ws, f.Y);
    // first head only: its matrices are the first r blocks of W, so y has rows (b, a); the gate (eq. 7) rides along
    launch_y_with_gate("first_gemm_y", ds, H, W, G, nullptr, Y, logw, nullptr, r, st);
    // the r rows of logits per b are the output's own size: they are stored once (fp32), with their statistics, and read once (twice: stats_apart)
    float2 *part = at<float2>(ws, f.part);
    int parts = f.parts;
    if (stats_apart(rows, V)) {
        launch_gemm_nt<Cfg>("first_gemm_z", Y, d, rows, U, d, V, d, EpiStoreF32{z, (long)V4, rows, V4, 0}, st);
        parts = (V + kStatCols - 1) / kStatCols;
        k_row_stats_f32<<<dim3((unsigned)rows, (unsigned)parts), kBlock, 0, st>>>(V, (size_t)V4, parts, z, part);
    } else {
        launch_z_stats("first_gemm_z", Y, d, rows, U, V, part, parts, z, (long)V4, st);
    }
    ProfileScope prof("first_mix", (double)rows * V * 4 + (double)B * V * 4, st);
    if (mix_from_parts(B, V, r, parts)) {
        k_first_token_from_parts<<<dim3((unsigned)B, blocks_for((size_t)V, kBlock)), kBlock, 0, st>>>(V, r, parts, (size_t)V4, z, part, logw,
                                                                                                     logp);
    } else {
        k_lse_from_parts<<<blocks_for((size_t)rows, kBlock / kWave), kBlock, 0, st>>>((size_t)rows, parts, part, lse);
        launch_first_token_mix(ds, z, (size_t)V4, lse, logw, logp, st);                     // eq. 11
    }
    return hipGetLastError() == hipSuccess ? CP_HEAD_OK : CP_HEAD_ERR_LAUNCH;
}

int fast_draft_sequential(const cp_head_desc &ds, const void *Hv, const void *Wv, const void *Uv, const void *Gv,
                          const float *uniforms, int32_t *tokens, float *logq, void *ws, hipStream_t st)
{
    if (ds.T == 0) return CP_HEAD_OK;
    if (!dims_fit(ds)) return CP_HEAD_ERR_UNSUPPORTED;
    const bf16_t *H = (const bf16_t *)Hv, *W = (const bf16_t *)Wv, *U = (const bf16_t *)Uv, *G = (const bf16_t *)Gv;
    const DraftWs f = draft_ws(ds, true);
    const int B = (int)ds.T, d = ds.d, V = ds.V, n = ds.n, r = ds.r;
    const size_t M = (size_t)B * n * r;
    float *logw = at<float>(ws, f.logw);
    bf16_t *Y = at<bf16_t>(ws, f.Y);
    float2 *part = at<float2>(ws, f.part);
    launch_y_with_gate("seq_gemm_y", ds, H, W, G, nullptr, Y, logw, nullptr, n * r, st);          // y and the gate (eq. 7)
    int parts, seg_cols;
    z_segments((int)M, V, d, parts, seg_cols);
    launch_z_stats("seq_gemm_z", Y, d, (int)M, U, V, part, parts, nullptr, 0, st);
    // A draw is two launches: a workgroup per row for everything but the logits of the segment, which many share.
    // (One launch with a workgroup per row for all draws fetched them on one
    // compute unit: the call took 691 us at B = 8, d = 4096, V = 128256, n = 4, r = 8 and takes 534 us this way.)
    ProfileScope prof("seq_draw", (double)B * n * r * seg_cols * d * 2, st);
    float *lse = at<float>(ws, f.lse), *zseg = at<float>(ws, f.zseg);
    int32_t *seg = at<int32_t>(ws, f.seg);
    double *base = at<double>(ws, f.base);
    k_lse_from_parts<<<blocks_for(M, kBlock / kWave), kBlock, 0, st>>>(M, parts, part, lse);
    for (int step = 0; step <= n; ++step) {
        // one wavefront up to a segment a lane, whose mass is a sum over r experts; find_segment's segments per thread
        auto kernel = parts <= kWave ? (r <= 8 ? k_sequential_step8<true, 1> : k_sequential_step<true>)
                    : r > 8 || parts > 2 * kWideBlock ? k_sequential_step<false>
                    : parts <= kWideBlock ? k_sequential_step8<false, 1> : k_sequential_step8<false, 2>;
        kernel<<<(unsigned)B, kWideBlock, 0, st>>>(step, V, n, r, parts, seg_cols, part, zseg, lse, logw, uniforms, seg, base, tokens,
                                                   logq);                                                      // eq. 11-13
        if (step < n)
            k_segment_logits<<<dim3((unsigned)B, (unsigned)seg_cols / 16, (unsigned)(r + 15) / 16), kSegWaves * kWave, 0, st>>>(
                d, V, n, r, seg_cols, step, 1, Y, U, seg, 1, zseg);
    }
    return hipGetLastError() == hipSuccess ? CP_HEAD_OK : CP_HEAD_ERR_LAUNCH;
}

// ------------------------------------------------------------------------------------------
// full heads: loss forward and backward
// ------------------------------------------------------------------------------------------

size_t fast_full_ctx_bytes(const cp_head_desc &ds) { return full_ctx(ds).total; }

int fast_full_loss_fwd(const cp_head_desc &ds, const void *Hv, const void *Fv, const void *Gv, const int32_t *X,
                       float *loss, void *ctx, void *ws, hipStream_t st)
{
    if (ds.T == 0) return CP_HEAD_OK;
    if (!dims_fit(ds)) return CP_HEAD_ERR_UNSUPPORTED;
    const bf16_t *H = (const bf16_t *)Hv, *F = (const bf16_t *)Fv;
    const FullCtx cl = full_ctx(ds);
    const FullFwdWs f = full_fwd_ws(ds);
    const int T = (int)ds.T, d = ds.d, V = ds.V, nr = ds.n * ds.r;
    const size_t M = (size_t)T * nr;
    float *lse = at<float>(ctx, cl.lse), *w = at<float>(ctx, cl.w), *gamma = at<float>(ctx, cl.gamma);
    float *logw = at<float>(ws, f.logw), *C = at<float>(ws, f.C);
    float2 *part = cl.keep ? at<float2>(ctx, cl.zpart) : at<float2>(ws, f.part);
    uint16_t *zs = at<uint16_t>(ctx, cl.zs);
    launch_gate_bf16(ds, (const bf16_t *)Hv, (const bf16_t *)Gv, logw, w, st);                                                       // eq. 7
    for (int sa = 0; sa < nr; ++sa) {                                                           // z_sa = F_sa h (eq. 6), statistics
        if (cl.keep)
            launch_gemm_nt<Cfg>("full_gemm_z_stats_keep", H, d, T, F + (size_t)sa * V * d, d, V, d,
                                EpiRowStatsKeep{part + (size_t)sa * T * f.parts, f.parts, T, V,
                                                zs + (size_t)sa * T * cl.Vp, (long)cl.Vp, (int)cl.Vp, streamed_store(M * cl.Vp * 2)}, st);
        else
            launch_gemm_nt<Cfg>("full_gemm_z_stats", H, d, T, F + (size_t)sa * V * d, d, V, d,
                                EpiRowStats{part + (size_t)sa * T * f.parts, f.parts, T, V}, st);
    }
    k_full_row_finish<<<blocks_for(M, kBlock / kWave), kBlock, 0, st>>>((size_t)T, d, V, ds.n, ds.r, f.parts, part, H, F, X,
                                                                        lse, C);             // eq. 5, 8
    launch_mixture(ds, logw, C, loss, gamma, -1.f, st);                                         // eq. 9
    return hipGetLastError() == hipSuccess ? CP_HEAD_OK : CP_HEAD_ERR_LAUNCH;
}

int fast_full_loss_bwd(const cp_head_desc &ds, const void *Hv, const void *Fv, const void *Gv, const int32_t *X,
                       const float *dloss, float scale, const void *ctx, float *dH, float *dF, float *dG, void *ws,
                       hipStream_t st)
{
    const int d = ds.d, V = ds.V, r = ds.r, n = ds.n, nr = n * r;
    if (ds.T == 0) {
        if (dF) launch_fill_zero(dF, (size_t)nr * V * d, st);
        if (dG) launch_fill_zero(dG, (size_t)r * d, st);
        return hipGetLastError() == hipSuccess ? CP_HEAD_OK : CP_HEAD_ERR_LAUNCH;
    }
    if (!dims_fit(ds)) return CP_HEAD_ERR_UNSUPPORTED;
    const bf16_t *H = (const bf16_t *)Hv, *F = (const bf16_t *)Fv, *G = (const bf16_t *)Gv;
    const FullCtx cl = full_ctx(ds);
    const FullBwdWs b = full_bwd_ws(ds);
    const size_t T = (size_t)ds.T, M = T * nr;
    const float *lse = at<float>(ctx, cl.lse), *w = at<float>(ctx, cl.w), *gamma = at<float>(ctx, cl.gamma);
    float4 *rowinfo = at<float4>(ws, b.coef);
    float *dg = at<float>(ws, b.dg);
    bf16_t *Ht = at<bf16_t>(ws, b.Ht);
    bf16_t *dZ = at<bf16_t>(ws, b.dZ);
    const int Vp = (int)b.Vp, Tp = (int)b.Tp;
    const long ldT = (long)b.ldT;
    const SplitScratch split = split_scratch(ws, b.split, b.split_bytes);

    k_full_bwd_coefficients<<<blocks_for(M, kBlock), kBlock, 0, st>>>(T, n, r, w, gamma, lse, dloss, scale, X, rowinfo, dg);
    if (dF) transpose_bf16(H, d, (int)T, d, Ht, ldT, Tp, st);         // Ht[d, Tp]
    int first_chunk = 1;
    for (size_t t0 = 0; t0 < T; t0 += b.chunk) {
        const int Tc = (int)((T - t0 < b.chunk) ? T - t0 : b.chunk);
        const int Tcp = (int)round_up((size_t)Tc, 64);
        const bf16_t *Hc = H + t0 * d;
        for (int sa = 0; sa < nr; ++sa) {
            const bf16_t *Fsa = F + (size_t)sa * V * d;
            // dz (bf16) from the kept logits of these positions, or from z_sa recomputed
            if (cl.keep) {
                KeptDzArgs kept{KeptLogits{at<uint16_t>(ctx, cl.zs), at<float2>(ctx, cl.zpart), (long)cl.Vp, cl.parts}, rowinfo, V};
                kept_dz_launch(&kept, nullptr, Tc, Tcp, (size_t)sa * T + t0, dZ, Vp, st);
            } else {
                launch_gemm_nt<Cfg>("full_gemm_z_dz", Hc, d, Tc, Fsa, d, V, d,
                                    EpiDz{dZ, (long)Vp, rowinfo + (size_t)sa * T + t0, Tc, Tcp, V, Vp, streamed_store((size_t)Tc * Vp * 2)}, st);
            }
            // dH += dz F_sa   (contraction over the vocabulary; F_sa as it is stored is K-major for this product, and
            // a transposed copy of every head matrix per chunk would cost more than the K-major loop does)
            launch_gemm_nt<CfgBlockedANN>("full_gemm_dh", dZ, Vp, Tc, Fsa, d, d, Vp,
                                  EpiStoreF32{dH + t0 * d, (long)d, Tc, d, sa ? 1 : 0}, st, kGroupRowsNarrow, NoSideJob{0}, -1, V, split);
            // dF_sa += dz^T H   (contraction over the positions of the chunk)
            if (dF)
                launch_gemm_nt<CfgBlockedTN>("full_gemm_df", dZ, Vp, V, Ht + t0, ldT, d, Tcp,
                                    EpiStoreF32{dF + (size_t)sa * V * d, (long)d, V, d, first_chunk ? 0 : 1}, st,
                                    kGroupRowsNarrow, NoSideJob{0}, -1, -1, split);
        }
        first_chunk = 0;
    }
    k_add_gate_to_dh<<<blocks_for(T * d / 4, kBlock), kBlock, 0, st>>>(T, d, r, G, dg, dH);       // + G^T dg
    if (dG) launch_gate_gradient_bf16(ds, H, dg, at<float>(ws, b.dGpart), dG, st);
    return hipGetLastError() == hipSuccess ? CP_HEAD_OK : CP_HEAD_ERR_LAUNCH;
}

}  // namespace cph
