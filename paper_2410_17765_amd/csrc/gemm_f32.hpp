// fp32 matrix-core GEMM for the plain path: acc[m, n] = sum_k A[m, k] B[n, k], any shape, any alignment, operands
// stored as float or bfloat16 and multiplied as fp32 (v_mfma_f32_16x16x4_f32: exact fp32 products, fp32 sums).
//
// Either operand is K-contiguous (X[row, ld], the contraction index fast) or K-major (X[k, ld], the output index
// fast), so no product of the path needs a transposed copy.  What bounds it is the matrix cores' fp32 rate (157
// TFLOP/s, 1/16 of bf16), so low that neither LDS nor global loads come close to it: tiles are staged through
// registers (which is where bfloat16 is widened and where any alignment is taken: 16-byte loads if the operand allows
// them, single elements otherwise), double-buffered in LDS, one barrier per K-step.  Two to four workgroups share a
// compute unit and fill each other's gaps.
//
// Fragments: lane l of a 16-row block takes row l % 16 and, of a chunk of 16 k-values, the four at 4 (l / 16); the
// four instructions of a chunk each use one of them.  The order inside the sum is permuted, the same way for both
// operands.  A K-contiguous tile has a row stride of BK + 4 floats (16-byte fragment reads), a K-major tile one of
// rows + 4 (single-element reads): both are free of bank conflicts.
#pragma once

#include "cp_internal.hpp"
#include "f32_plan.hpp"

namespace cph {

typedef float f32v4_t __attribute__((ext_vector_type(4)));

// BM x BN tile by WM x WN wavefronts, times WK wavefronts that share the k-values of every K-step (their sums meet in
// LDS at the end): small outputs with few tiles then still use four SIMDs per tile.
template <int BM_, int BN_, int WM_, int WN_, int WK_, int BK_>
struct F32Tile {
    static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, WK = WK_, BK = BK_;
    static constexpr int WTM = BM / WM, WTN = BN / WN, TM = WTM / 16, TN = WTN / 16;
    static constexpr int CHUNKS = BK / 16;          // chunks of 16 k-values per K-step
    static_assert(WM * WN * WK == 4 && BM % (16 * WM) == 0 && BN % (16 * WN) == 0 && CHUNKS % WK == 0, "four wavefronts");
};
typedef F32Tile<128, 128, 2, 2, 1, 32> F32Large;
// Both operands K-contiguous: a K-step of 16 lets a third workgroup share the compute unit, whose products fill more of the
// others' gaps (z, dz and y of T = 500, d = 512, V = 8191, n = r = 4: 1474 -> 1371 us); where that pays: f32_short_steps.  A K-major
// operand's fragments are four reads each, so that the shorter K-step gains nothing there (dY and dU: 1132 -> 1147 us), nor in
// the 64-wide tile (125 -> 166 us).
typedef F32Tile<128, 128, 2, 2, 1, 16> F32LargeContiguous;
typedef F32Tile<64, 64, 2, 2, 1, 32> F32Mid;
typedef F32Tile<32, 32, 1, 1, 4, 64> F32Small;
constexpr int kF32Threads = 256;

// One contraction.  The tile index runs over tiles_m * tiles_n * splits; split s takes the k-values
// [s * k_split, (s + 1) * k_split).  With batch_b, the splits are contractions of their own instead: the s-th takes all of K
// and B from s * batch_b elements on.
struct F32Problem {
    const void *A, *B;
    long lda, ldb;          // elements
    long M, N;
    long ka, kb;            // k-values that may be read of A and of B; the sum runs over the smaller number
    long k_split, batch_b;
    int tiles_m, tiles_n, splits;
    int vec;                // four consecutive elements of either operand may be loaded at once
    __host__ __device__ long tiles() const { return (long)tiles_m * tiles_n * splits; }
};

template <typename T>
__device__ __forceinline__ f32v4_t f32_load4(const T *p);
template <>
__device__ __forceinline__ f32v4_t f32_load4<float>(const float *p) { return *reinterpret_cast<const f32v4_t *>(p); }
template <>
__device__ __forceinline__ f32v4_t f32_load4<bf16_t>(const bf16_t *p)
{
    const uint2 q = *reinterpret_cast<const uint2 *>(p);
    return f32v4_t{__uint_as_float(q.x << 16), __uint_as_float(q.x & 0xFFFF0000u), __uint_as_float(q.y << 16),
                   __uint_as_float(q.y & 0xFFFF0000u)};
}

// One operand's share of a thread: QUADS groups of four consecutive elements per K-step.
template <typename T, bool KM, int ROWS, int BK>
struct F32Loader {
    static constexpr int STRIDE = KM ? ROWS + 4 : BK + 4;                 // floats between LDS rows
    static constexpr int FLOATS = (KM ? BK : ROWS) * STRIDE;
    static constexpr int PER_ROW = (KM ? ROWS : BK) / 4;                  // quads per LDS row
    static constexpr int QUADS = ROWS * BK / 4 / kF32Threads;
    static_assert(QUADS >= 1 && ROWS * BK % (4 * kF32Threads) == 0, "whole quads per thread");
    const T *base;       // K-contiguous: row 0 of the tile; K-major: column 0 of the tile
    long ld, limit;      // rows (K-contiguous) or columns (K-major) of the tile that exist
    long kend;           // k-values that exist
    int slow, fast;      // LDS row of the first quad, first element of it in that row
    f32v4_t q[QUADS];

    __device__ __forceinline__ void init(const T *X, long ld_, long row0, long rows, long kend_)
    {
        ld = ld_;
        limit = rows - row0;
        kend = kend_;
        base = KM ? X + row0 : X + row0 * ld;
        slow = (int)threadIdx.x / PER_ROW;
        fast = ((int)threadIdx.x % PER_ROW) * 4;
    }
    static constexpr int kStep = kF32Threads / PER_ROW;                   // LDS rows between a thread's quads
    // the quads of the K-step that starts at k0; elements past the end of K are zero, elements past the tile's rows
    // are any (their outputs are never stored) but their loads stay inside the operand
    template <bool WHOLE, bool VEC>
    __device__ __forceinline__ void load(long k0)
    {
#pragma unroll
        for (int i = 0; i < QUADS; ++i) {
            const int s = slow + i * kStep;
            if (KM) {
                const T *p = base + (k0 + s) * ld;
                const bool in = WHOLE || k0 + s < kend;
                if (VEC) {
                    const long c = fast < limit ? fast : (limit - 1) / 4 * 4;
                    q[i] = f32v4_t{0.f, 0.f, 0.f, 0.f};
                    if (in) q[i] = f32_load4<T>(p + c);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const long c = fast + e < limit ? fast + e : limit - 1;
                        q[i][e] = 0.f;
                        if (in) q[i][e] = ld_f32(p, (size_t)c);
                    }
                }
            } else {
                const T *p = base + (s < limit ? s : limit - 1) * ld + k0 + fast;
                if (VEC) {                              // the K extent is a multiple of 4 then, or zero-padded to one
                    q[i] = f32v4_t{0.f, 0.f, 0.f, 0.f};
                    if (WHOLE || k0 + fast < kend) q[i] = f32_load4<T>(p);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        q[i][e] = 0.f;
                        if (WHOLE || k0 + fast + e < kend) q[i][e] = ld_f32(p, e);
                    }
                }
            }
        }
    }
    __device__ __forceinline__ void store(float *lds) const
    {
#pragma unroll
        for (int i = 0; i < QUADS; ++i) *reinterpret_cast<f32v4_t *>(lds + (slow + i * kStep) * STRIDE + fast) = q[i];
    }
    // fragment of the 16-row block at `row` for the chunk at `kc`
    __device__ static __forceinline__ f32v4_t fragment(const float *lds, int row, int kc, int lane)
    {
        const int g = lane >> 4, x = row + (lane & 15);
        if (!KM) return *reinterpret_cast<const f32v4_t *>(lds + x * STRIDE + kc + 4 * g);
        f32v4_t f;
#pragma unroll
        for (int e = 0; e < 4; ++e) f[e] = lds[(kc + 4 * g + e) * STRIDE + x];
        return f;
    }
};

template <class Tile, typename TA, typename TB, bool AKM, bool BKM>
struct F32Gemm {
    typedef F32Loader<TA, AKM, Tile::BM, Tile::BK> LoadA;
    typedef F32Loader<TB, BKM, Tile::BN, Tile::BK> LoadB;
    static constexpr int STAGE = LoadA::FLOATS + LoadB::FLOATS;
    static constexpr int LDS_FLOATS = 2 * STAGE;
    static constexpr int PER_CU = Tile::BM == 128 && Tile::BK == 16 ? 3 : 2;      // workgroups that the register limit allows for

    // Tile `index` of the problem.  The epilogue is called by the wavefronts that hold results, with the origin of their
    // sub-tile, the split, and the sub-tile's column slot (tile column times WN plus wavefront column).
    template <class Epi>
    __device__ static __forceinline__ void run(const F32Problem &p, long index, const Epi &epi, float *lds)
    {
        if (p.vec) run_as<true>(p, index, epi, lds);
        else run_as<false>(p, index, epi, lds);
    }
    template <bool VEC, class Epi>
    __device__ static __forceinline__ void run_as(const F32Problem &p, long index, const Epi &epi, float *lds)
    {
        constexpr int TM = Tile::TM, TN = Tile::TN, BK = Tile::BK;
        const int lane = threadIdx.x & 63;
        const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
        const int wk = wave % Tile::WK, wn = wave / Tile::WK % Tile::WN, wm = wave / Tile::WK / Tile::WN;
        const long per_split = (long)p.tiles_m * p.tiles_n;
        const int split = (int)(index / per_split);
        const int rest = (int)(index % per_split);
        // the columns of eight tile rows together, so that the tiles in flight share operand panels in L2
        const int band = rest / (8 * p.tiles_n), in_band = rest % (8 * p.tiles_n);
        const int rows_in_band = min(8, p.tiles_m - band * 8);
        const int tm = band * 8 + in_band % rows_in_band, tn = in_band / rows_in_band;
        const long m0 = (long)tm * Tile::BM, n0 = (long)tn * Tile::BN;
        const long k_lo = p.batch_b ? 0 : split * p.k_split, k_all = p.ka < p.kb ? p.ka : p.kb;
        const long k_hi = k_lo + p.k_split < k_all ? k_lo + p.k_split : k_all;

        LoadA la;
        LoadB lb;
        la.init(static_cast<const TA *>(p.A), p.lda, m0, p.M, k_hi);
        lb.init(static_cast<const TB *>(p.B) + split * p.batch_b, p.ldb, n0, p.N, k_hi);
        f32v4_t acc[TM][TN];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = f32v4_t{0.f, 0.f, 0.f, 0.f};
        auto store = [&](int stage) {
            la.store(lds + stage * STAGE);
            lb.store(lds + stage * STAGE + LoadA::FLOATS);
        };
        auto multiply = [&](int stage) {
            const float *sa = lds + stage * STAGE, *sb = sa + LoadA::FLOATS;
#pragma unroll
            for (int c = 0; c < Tile::CHUNKS / Tile::WK; ++c) {
                const int kc = (c * Tile::WK + wk) * 16;
                f32v4_t a[TM], b[TN];
#pragma unroll
                for (int i = 0; i < TM; ++i) a[i] = LoadA::fragment(sa, wm * Tile::WTM + 16 * i, kc, lane);
#pragma unroll
                for (int j = 0; j < TN; ++j) b[j] = LoadB::fragment(sb, wn * Tile::WTN + 16 * j, kc, lane);
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int j = 0; j < TN; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][e], b[j][e], acc[i][j], 0, 0, 0);
            }
        };
        // Whole K-steps in a loop without a branch (a choice of load forms inside it makes the compiler wait for the
        // loads of one operand before it issues those of the other), then the partial one.
        const long whole = k_hi > k_lo ? (k_hi - k_lo) / BK : 0;
        const bool tail = k_lo + whole * BK < k_hi;
        int cur = 0;
        long k = k_lo;
        if (whole > 0) {
            la.template load<true, VEC>(k);
            lb.template load<true, VEC>(k);
            store(0);
            __syncthreads();
            for (long s = 1; s < whole; ++s) {
                k += BK;
                la.template load<true, VEC>(k);
                lb.template load<true, VEC>(k);
                __builtin_amdgcn_sched_barrier(0);          // keeps the loads ahead of the products that cover them
                multiply(cur);
                __builtin_amdgcn_sched_barrier(0);
                store(cur ^ 1);
                __syncthreads();
                cur ^= 1;
            }
            k += BK;
        }
        if (tail) {
            la.template load<false, VEC>(k);
            lb.template load<false, VEC>(k);
        }
        if (whole > 0) multiply(cur);
        if (tail) {
            store(cur ^ 1);
            __syncthreads();
            multiply(cur ^ 1);
        }
        if (Tile::WK > 1) {
            // the wavefronts' sums over their shares of K, added in wavefront order
            static_assert(Tile::WK == 1 || LDS_FLOATS >= Tile::WK * TM * TN * 256, "the partial sums fit the operand stages");
            __syncthreads();                                // every wavefront is done reading the stages
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    *reinterpret_cast<f32v4_t *>(lds + ((wk * TM + i) * TN + j) * 256 + lane * 4) = acc[i][j];
            __syncthreads();
            if (wk != 0) return;
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int w = 1; w < Tile::WK; ++w)
                        acc[i][j] += *reinterpret_cast<const f32v4_t *>(lds + ((w * TM + i) * TN + j) * 256 + lane * 4);
        }
        epi.template run<Tile>(acc, m0 + wm * Tile::WTM, n0 + wn * Tile::WTN, p, split, tn * Tile::WN + wn, lane);
    }
};

// row and column of accumulator element v of block (i, j), relative to the sub-tile's origin
__device__ __forceinline__ int f32_row(int i, int v, int lane) { return 16 * i + 4 * (lane >> 4) + v; }
__device__ __forceinline__ int f32_col(int j, int lane) { return 16 * j + (lane & 15); }

// ---------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------

// A[M, lda] or, K-major, A[K, lda]; B[N, ldb] or B[K, ldb].  ka, kb: k-values that may be read of either operand when
// they differ (a K-contiguous operand whose rows are zero-padded to a multiple of 4).
template <bool AKM, bool BKM, typename TA, typename TB>
inline F32Problem f32_problem(const TA *A, long lda, const TB *B, long ldb, long M, long N, long ka, long kb, F32Plan plan)
{
    F32Problem p;
    const int e = f32_tile_edge(plan.kind);
    p.A = A; p.B = B; p.lda = lda; p.ldb = ldb; p.M = M; p.N = N; p.ka = ka; p.kb = kb;
    p.tiles_m = (int)((M + e - 1) / e);
    p.tiles_n = (int)((N + e - 1) / e);
    p.splits = plan.splits;
    p.batch_b = 0;
    const long K = ka < kb ? ka : kb;
    p.k_split = (K + plan.splits - 1) / plan.splits;
    p.k_split = (p.k_split + 63) / 64 * 64;              // whole K-steps, and every split's start stays aligned
    auto four = [](const void *X, size_t elem, long ld, long extent) {
        return ld % 4 == 0 && extent % 4 == 0 && reinterpret_cast<uintptr_t>(X) % (4 * elem) == 0 ? 1 : 0;
    };
    p.vec = four(A, sizeof(TA), lda, AKM ? 0 : ka) && four(B, sizeof(TB), ldb, BKM ? 0 : kb);
    return p;
}

// `batch` contractions of one A with the matrices B, B + stride, ... in one launch; the epilogue's split is the matrix.
inline F32Problem f32_batch(F32Problem p, int batch, long stride)
{
    p.splits = batch;
    p.batch_b = stride;
    p.k_split = p.ka < p.kb ? p.ka : p.kb;
    if (stride % 4) p.vec = 0;
    return p;
}

// Up to three problems in one launch (their tiles share the compute units: two workgroups with K-steps of 32, each 59 % of the matrix
// cores' rate alone, fill one another's gaps to 80 %, three with K-steps of 16 to 86 %); a problem with zero tiles is absent.
template <class G1, class E1, class G2, class E2, class G3, class E3>
__global__ void __launch_bounds__(kF32Threads, G1::PER_CU)
     k_gemm_f32(F32Problem p1, E1 e1, F32Problem p2, E2 e2, F32Problem p3, E3 e3)
{
    constexpr int L12 = G1::LDS_FLOATS > G2::LDS_FLOATS ? G1::LDS_FLOATS : G2::LDS_FLOATS;
    constexpr int L = L12 > G3::LDS_FLOATS ? L12 : G3::LDS_FLOATS;
    __shared__ __attribute__((aligned(16))) float lds[L];
    long index = blockIdx.x;
    const long n1 = p1.tiles();
    if (index < n1) {
        G1::run(p1, index, e1, lds);
        return;
    }
    index -= n1;
    const long n2 = p2.tiles();
    if (index < n2) {
        G2::run(p2, index, e2, lds);
        return;
    }
    G3::run(p3, index - n2, e3, lds);
}
struct NoF32Problem {
    static constexpr int LDS_FLOATS = 1;
    template <class Epi>
    __device__ static void run(const F32Problem &, long, const Epi &, float *) {}
};
struct NoEpi {};

}  // namespace cph
