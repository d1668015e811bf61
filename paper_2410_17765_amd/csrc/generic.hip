// Plain fp32 path of the CP head: correct for every shape and storage type.  It serves fp32
// storage and shapes the bf16 matrix-core path does not take, and its per-position bookkeeping
// kernels (gate, mixture, expert draw) are shared with that path.  Every contraction runs on the
// fp32 matrix instruction (gemm_f32.hpp) with the row's bookkeeping in the epilogue; every sum
// runs in a fixed order, so results are reproducible.
//
// Head rows are ordered m = (t*n + s)*r + a, so X[m / r] is the row's target and
// m / (n*r) its position.
#include "cp_internal.hpp"
#include "gemm_f32.hpp"

#include <math.h>

#include <algorithm>
#include <type_traits>

namespace cph {

namespace {

constexpr int kBlock = 256;
constexpr int kWavesPerBlock = kBlock / kWave;


// ------------------------------------------------------------------------------------------
// gate: logw = log_softmax(G h), w = exp(logw)      (eq. 7)
// one wavefront per position; lane a ends up holding g_a
// ------------------------------------------------------------------------------------------
template <typename TIn>
__global__ void __launch_bounds__(kWave) k_gate(int d, int r, const TIn *__restrict__ H, const TIn *__restrict__ G,
                                                float *__restrict__ logw, float *__restrict__ w)
{
    const size_t t = blockIdx.x;
    const int lane = threadIdx.x;
    const TIn *h = H + t * d;
    float mine = -INFINITY;
    for (int a = 0; a < r; ++a) {
        float p = 0.f;
        for (int k = lane; k < d; k += kWave) p += ld_f32(G, (size_t)a * d + k) * ld_f32(h, k);
        p = wave_sum(p);
        if (lane == a) mine = p;
    }
    const float mx = wave_max(mine);
    const float s = wave_sum(lane < r ? expf(mine - mx) : 0.f);
    const float lse = mx + logf(s);
    if (lane < r) {
        logw[t * r + lane] = mine - lse;
        w[t * r + lane] = expf(mine - lse);
    }
}

// ------------------------------------------------------------------------------------------
// y = W_sa h rounded to bf16, one block per head row m = (t, s, a): the draft-type calls with bf16 storage.
// The rounding is discontinuous, so these calls keep this kernel's summation order: an element of y within fp32
// accumulation error of a rounding midpoint would otherwise fall on its other side and move a row's logits by 1e-2.
// ------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(kBlock) k_y_rounded(int d, int nr, const bf16_t *__restrict__ H, const bf16_t *__restrict__ W,
                                                      float *__restrict__ Y)
{
    extern __shared__ float hs[];
    const size_t m = blockIdx.x;
    const size_t t = m / nr;
    const int sa = (int)(m % nr);
    for (int k = threadIdx.x; k < d; k += kBlock) hs[k] = ld_f32(H, t * d + k);
    __syncthreads();
    const bf16_t *Wsa = W + (size_t)sa * d * d;
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    for (int k = wave; k < d; k += kWavesPerBlock) {
        float p = 0.f;
        for (int j = lane; j < d; j += kWave) p += ld_f32(Wsa, (size_t)k * d + j) * hs[j];
        p = wave_sum(p);
        if (lane == 0) Y[m * d + k] = bf16_to_f32(f32_to_bf16(p));
    }
}

// ------------------------------------------------------------------------------------------
// epilogues of the fp32 products.  A sub-tile's element v of block (i, j) is row f32_row, column f32_col from its origin.
// ------------------------------------------------------------------------------------------

// C[row, col] = acc (+ what is there); a split sum's parts go to partial[split, M, N].
struct EpiF32Store {
    float *C;
    long ldc;
    int accumulate;
    float *partial;
    template <class Tile>
    __device__ __forceinline__ void run(f32v4_t (&acc)[Tile::TM][Tile::TN], long row0, long col0, const F32Problem &p, int split,
                                        int, int lane) const
    {
        const bool part = p.splits > 1, add = accumulate && !part;
        float *out = part ? partial + (size_t)split * p.M * p.N : C;
        const long ld = part ? p.N : ldc;
#pragma unroll
        for (int i = 0; i < Tile::TM; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const long row = row0 + f32_row(i, v, lane);
                if (row >= p.M) continue;
#pragma unroll
                for (int j = 0; j < Tile::TN; ++j) {
                    const long col = col0 + f32_col(j, lane);
                    if (col >= p.N) continue;
                    float *o = out + row * ld + col;
                    *o = add ? *o + acc[i][j][v] : acc[i][j][v];
                }
            }
    }
};

// Sums of exponentials relative to their maximum mx, for logits that may be infinite or NaN as well: a term is
// exp(x - below(mx)), so that an infinite maximum leaves +infinity of its own kind and nothing of the rest, and a NaN stays
// one, also where it is alone and mx still -infinity; a sum moves from one maximum to a larger one with the factor shift().
__device__ __forceinline__ float below(float mx) { return fabsf(mx) == INFINITY ? 0.f : mx; }
__device__ __forceinline__ float shift(float from, float to) { return from == to ? 1.f : expf(from - to); }

// Logits of the head rows m = row * row_mul + batch: (maximum, sum of exp(z - maximum)) over the sub-tile's columns
// to part[m, slots], the target logit to zt[m] (if X is given), and the logits themselves to z[row, ldz] (if z is
// given; columns from V up to ldz become zero).
struct EpiF32Logits {
    float2 *part;
    int slots;
    long row_mul;
    const int32_t *X;       // null: no target logits
    int r;
    float *zt;
    float *z;               // null: logits are not kept
    long ldz;
    template <class Tile>
    __device__ __forceinline__ void run(f32v4_t (&acc)[Tile::TM][Tile::TN], long row0, long col0, const F32Problem &p, int batch,
                                        int slot, int lane) const
    {
#pragma unroll
        for (int i = 0; i < Tile::TM; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const long row = row0 + f32_row(i, v, lane);
                const long m = row * row_mul + batch;
                const bool in = row < p.M;
                if (z && in) {
#pragma unroll
                    for (int j = 0; j < Tile::TN; ++j) {
                        const long col = col0 + f32_col(j, lane);
                        if (col < ldz) z[row * ldz + col] = col < p.N ? acc[i][j][v] : 0.f;
                    }
                }
                if (part) {
                    float mx = -INFINITY;
#pragma unroll
                    for (int j = 0; j < Tile::TN; ++j)
                        if (col0 + f32_col(j, lane) < p.N) mx = fmaxf(mx, acc[i][j][v]);
                    mx = row16_max(mx);
                    const float base = below(mx);
                    float sum = 0.f;
#pragma unroll
                    for (int j = 0; j < Tile::TN; ++j)
                        if (col0 + f32_col(j, lane) < p.N) sum += expf(acc[i][j][v] - base);
                    sum = row16_sum(sum);
                    if (in && (lane & 15) == 0) part[m * slots + slot] = make_float2(mx, sum);
                }
                if (X && in) {
                    const long x = X[(unsigned)m / (unsigned)r];       // fewer than 2^31 head rows
#pragma unroll
                    for (int j = 0; j < Tile::TN; ++j)
                        if (x == col0 + f32_col(j, lane)) zt[m] = acc[i][j][v];
                }
            }
    }
};

// Logit gradients of the head rows m = m0 + row * row_mul + batch from their recomputed logits:
//   dz[v] = up_t gamma[t, a] (exp(z - lse[m]) - 1[v = x]),  zero for a dropped factor and from V up to ldz,
// written to dZ[row, ldz] (row-strided by ldz; the heads of a batch lie side by side in the row).  The first column slot also writes
// dg[t, a] = up_t (w - gamma), the derivative of eq. 9 with respect to the gate pre-activations, if dg is given.
struct EpiF32Dz {
    float *dZ;
    long ldz, columns;      // columns to write (V, or V rounded up to the padding)
    size_t m0;
    long row_mul;
    int n, r;
    const int32_t *X;
    const float *lse, *w, *gamma, *dloss;
    float scale;
    float *dg;
    template <class Tile>
    __device__ __forceinline__ void run(f32v4_t (&acc)[Tile::TM][Tile::TN], long row0, long col0, const F32Problem &p, int batch,
                                        int slot, int lane) const
    {
        float *out = dZ + batch * p.N;
#pragma unroll
        for (int i = 0; i < Tile::TM; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const long row = row0 + f32_row(i, v, lane);
                if (row >= p.M) continue;
                const unsigned m = (unsigned)(m0 + row * row_mul + batch), g = m / (unsigned)r;     // fewer than 2^31 head rows
                const unsigned a = m - g * r;
                const size_t t = g / (unsigned)n;
                const long x = X[g];
                const float up = dloss ? dloss[t] * scale : scale;
                const float gm = gamma[t * r + a];
                const float coef = x < 0 ? 0.f : up * gm, l = lse[m];
                if (dg && slot == 0 && (lane & 15) == 0 && g == t * n) dg[t * r + a] = up * (w[t * r + a] - gm);
#pragma unroll
                for (int j = 0; j < Tile::TN; ++j) {
                    const long col = col0 + f32_col(j, lane);
                    if (col >= columns) continue;
                    out[row * ldz + col] = x < 0 || col >= p.N ? 0.f : coef * (expf(acc[i][j][v] - l) - (col == x ? 1.f : 0.f));
                }
            }
    }
};

// dH[t, j] = acc + sum_a dg[t, a] G[a, j]; a split sum's parts go to partial[split, M, N] without the gate's term
template <typename TIn>
struct EpiF32Dh {
    float *dH;
    const float *dg;
    const TIn *G;
    int r;
    float *partial;
    template <class Tile>
    __device__ __forceinline__ void run(f32v4_t (&acc)[Tile::TM][Tile::TN], long row0, long col0, const F32Problem &p, int split,
                                        int, int lane) const
    {
        const bool part = p.splits > 1;
        float *out = part ? partial + (size_t)split * p.M * p.N : dH;
        const int terms = part ? 0 : r;
#pragma unroll
        for (int i = 0; i < Tile::TM; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const long row = row0 + f32_row(i, v, lane);
                if (row >= p.M) continue;
#pragma unroll
                for (int j = 0; j < Tile::TN; ++j) {
                    const long col = col0 + f32_col(j, lane);
                    if (col >= p.N) continue;
                    float x = acc[i][j][v];
                    for (int a = 0; a < terms; ++a) x += dg[row * r + a] * ld_f32(G, (size_t)a * p.N + col);
                    out[row * p.N + col] = x;
                }
            }
    }
};

// The split sums of a launch, added in split order: out[i] (+)= sum_s partial[s, i]; with dg, + sum_a dg[t, a] G[a, j] for
// i = t * N + j.  Job b covers the blocks from first[b] on.
struct AddSplits {
    int count;
    unsigned first[4];
    size_t size[3];
    int splits[3], accumulate[3];
    const float *partial[3];
    float *out[3];
    long N;
    int r, gate_job;
    const float *dg;
    const void *G;
    void add(const F32Plan &plan, long M, long Nn, const float *from, float *to, bool acc)
    {
        if (plan.splits == 1) return;
        size[count] = (size_t)M * Nn;
        splits[count] = plan.splits;
        accumulate[count] = acc ? 1 : 0;
        partial[count] = from;
        out[count] = to;
        first[count + 1] = first[count] + blocks_for(size[count], kBlock);
        ++count;
    }
};
template <typename TIn>
__global__ void __launch_bounds__(kBlock) k_add_splits(AddSplits job)
{
    int b = 0;
    while (b + 1 < job.count && blockIdx.x >= job.first[b + 1]) ++b;
    const size_t i = (size_t)(blockIdx.x - job.first[b]) * kBlock + threadIdx.x;
    if (i >= job.size[b]) return;
    float x = 0.f;
    for (int s = 0; s < job.splits[b]; ++s) x += job.partial[b][(size_t)s * job.size[b] + i];
    if (b == job.gate_job) {
        const size_t t = i / job.N, j = i % job.N;
        for (int a = 0; a < job.r; ++a) x += job.dg[t * job.r + a] * ld_f32((const TIn *)job.G, (size_t)a * job.N + j);
    }
    job.out[b][i] = job.accumulate[b] ? job.out[b][i] + x : x;
}

// One block per position: the log-normalisers (eq. 5) of its n r head rows from their per-slot statistics, a
// wavefront per row; C = z[x] - lse (eq. 8) in place of the target logits; the gate's log-softmax (eq. 7) in place of
// its pre-activations; and the mixture over the experts (eq. 9).  loss null: no mixture.
__global__ void __launch_bounds__(kBlock) k_position_finish(int n, int r, int slots, const float2 *__restrict__ part,
                                                            const int32_t *__restrict__ X, float *__restrict__ C,
                                                            float *__restrict__ lse_out, float *__restrict__ gate,
                                                            float *__restrict__ w_out, float *__restrict__ gamma,
                                                            float *__restrict__ loss)
{
    extern __shared__ float C_s[];                      // n r values
    const size_t t = blockIdx.x;
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave, nr = n * r;
    for (int j = wave; j < nr; j += kWavesPerBlock) {
        const size_t m = t * nr + j;
        float mx = -INFINITY, l = 0.f;
        for (int q = lane; q < slots; q += kWave) {
            const float2 v = part[m * slots + q];
            // a slot without columns is (-infinity, 0); one whose columns are all NaN is (-infinity, NaN)
            if (v.x > mx) { l = l * expf(mx - v.x) + v.y; mx = v.x; }
            else l += v.y * shift(v.x, mx);
        }
        const float Mx = wave_max(mx);
        const float L = wave_sum(l * shift(mx, Mx));
        const float lse = Mx + logf(L);
        if (lane == 0) {
            lse_out[m] = lse;
            const float c = X[m / r] >= 0 ? C[m] - lse : 0.f;
            C[m] = c;
            C_s[j] = c;
        }
    }
    __syncthreads();
    if (wave != 0) return;
    const float g = lane < r ? gate[t * r + lane] : -INFINITY;
    const float gm = wave_max(g);
    const float lw = g - (gm + logf(wave_sum(lane < r ? expf(g - gm) : 0.f)));
    if (lane < r) {
        gate[t * r + lane] = lw;
        w_out[t * r + lane] = expf(lw);
    }
    if (!loss) return;
    float a = -INFINITY;
    if (lane < r) {
        a = lw;
        for (int s = 0; s < n; ++s) a += C_s[s * r + lane];
    }
    const float mx = wave_max(a);
    const float L = mx + logf(wave_sum(lane < r ? expf(a - mx) : 0.f));
    if (lane == 0) loss[t] = -L;
    if (lane < r) gamma[t * r + lane] = expf(a - L);
}

// Log-normalisers (eq. 5) of stored rows of logits: a workgroup per row at a time, eight loads of a thread in flight.  The
// draft-type calls store their logits anyway, and reading them back costs V floats per row next to the 2 d V operations
// that made them; statistics in the product's epilogue would take room beside the logits.
__global__ void __launch_bounds__(1024) k_lse_of_rows(size_t rows, int V, const float *__restrict__ z, float *__restrict__ lse_out)
{
    __shared__ float2 red[1024 / kWave];
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave, waves = blockDim.x / kWave;
    for (size_t m = blockIdx.x; m < rows; m += gridDim.x) {
        const float *zr = z + m * V;
        float mx = -INFINITY, l = 0.f;
        for (int v0 = threadIdx.x; v0 < V; v0 += 8 * (int)blockDim.x) {
            float x[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) x[i] = zr[min(v0 + i * (int)blockDim.x, V - 1)];
            float mn = mx;
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (v0 + i * (int)blockDim.x < V) mn = fmaxf(mn, x[i]);
            l *= shift(mx, mn);
            const float base = below(mn);
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (v0 + i * (int)blockDim.x < V) l += expf(x[i] - base);
            mx = mn;
        }
        const float wm = wave_max(mx), wl = wave_sum(l * shift(mx, wm));
        if (lane == 0) red[wave] = make_float2(wm, wl);
        __syncthreads();
        if (wave == 0) {
            const float2 q = lane < waves ? red[lane] : make_float2(-INFINITY, 0.f);
            const float Mx = wave_max(q.x), L = wave_sum(q.y * shift(q.x, Mx));
            if (lane == 0) lse_out[m] = Mx + logf(L);
        }
        __syncthreads();
    }
}

// ---- launches: the plan picks the tile, and for two K-contiguous operands f32_short_steps its K-step
template <bool CONTIGUOUS, typename F>
void with_f32_tile(int kind, bool short_steps, const F &f)
{
    if (kind == kF32LargeTile && CONTIGUOUS && short_steps) f(std::conditional_t<CONTIGUOUS, F32LargeContiguous, F32Large>{});
    else if (kind == kF32LargeTile) f(F32Large{});
    else if (kind == kF32MidTile) f(F32Mid{});
    else f(F32Small{});
}
template <typename TA, typename TB, bool AKM, bool BKM, class Epi>
void launch_f32(const F32Problem &p, int kind, const Epi &e, hipStream_t st)
{
    const int narrow = (sizeof(TA) < 4) + (sizeof(TB) < 4);
    with_f32_tile<!AKM && !BKM>(kind, f32_short_steps(p.tiles(), narrow, p.vec != 0), [&](auto tile) {
        k_gemm_f32<F32Gemm<decltype(tile), TA, TB, AKM, BKM>, Epi, NoF32Problem, NoEpi, NoF32Problem, NoEpi>
            <<<(unsigned)p.tiles(), kF32Threads, 0, st>>>(p, e, F32Problem{}, NoEpi{}, F32Problem{}, NoEpi{});
    });
}
template <typename TIn>
void launch_add_splits(const AddSplits &job, hipStream_t st)
{
    if (job.count) k_add_splits<TIn><<<job.first[job.count], kBlock, 0, st>>>(job);
}
// y = W_sa h for `heads` head matrices, and unless `gate` is null its pre-activations G h
template <typename TIn>
void launch_f32_y(const cp_head_desc &ds, int heads, const TIn *H, const TIn *W, const TIn *G, float *Y, float *gate, hipStream_t st)
{
    const long d = ds.d, T = (long)ds.T, cols = (long)heads * d;
    const F32Plan plan = f32_plan(T, cols, d, false);
    const F32Problem py = f32_problem<false, false>(H, d, W, d, T, cols, d, d, plan);
    F32Problem pg{};
    if (gate) pg = f32_problem<false, false>(H, d, G, d, T, ds.r, d, d, plan);
    const bool short_steps = f32_short_steps(py.tiles() + pg.tiles(), sizeof(TIn) < 4 ? 2 : 0, py.vec != 0);
    with_f32_tile<true>(plan.kind, short_steps, [&](auto tile) {
        typedef F32Gemm<decltype(tile), TIn, TIn, false, false> Gm;
        // the few gate tiles first: they share the launch's first round
        k_gemm_f32<Gm, EpiF32Store, Gm, EpiF32Store, NoF32Problem, NoEpi><<<(unsigned)(py.tiles() + pg.tiles()), kF32Threads, 0, st>>>(
            pg, EpiF32Store{gate, ds.r, 0, nullptr}, py, EpiF32Store{Y, cols, 0, nullptr}, F32Problem{}, NoEpi{});
    });
}
// y of the draft-type calls: with bf16 storage its rounding is part of the distribution's definition
void launch_draft_y(const cp_head_desc &ds, int heads, const float *H, const float *W, float *Y, hipStream_t st)
{
    launch_f32_y<float>(ds, heads, H, W, nullptr, Y, nullptr, st);
}
void launch_draft_y(const cp_head_desc &ds, int heads, const bf16_t *H, const bf16_t *W, float *Y, hipStream_t st)
{
    k_y_rounded<<<(unsigned)(ds.T * heads), kBlock, (size_t)ds.d * sizeof(float), st>>>(ds.d, heads, H, W, Y);
}

// ------------------------------------------------------------------------------------------
// mixture over experts (eq. 9) and the posterior gamma_a = exp(a_a - L); one wavefront per position
// ------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(kWave) k_mixture(int n, int r, const float *__restrict__ logw,
                                                   const float *__restrict__ C, float *__restrict__ loss,
                                                   float *__restrict__ gamma, float sign)
{
    const size_t t = blockIdx.x;
    const int lane = threadIdx.x;
    float a = -INFINITY;
    if (lane < r) {
        a = logw[t * r + lane];
        for (int s = 0; s < n; ++s) a += C[(t * n + s) * r + lane];
    }
    const float mx = wave_max(a);
    const float sum = wave_sum(lane < r ? expf(a - mx) : 0.f);
    const float L = mx + logf(sum);
    if (lane == 0) loss[t] = sign * L;   // -L: the loss; +L: the joint log-probability
    if (gamma && lane < r) gamma[t * r + lane] = expf(a - L);
}

// ------------------------------------------------------------------------------------------
// backward pieces
// ------------------------------------------------------------------------------------------

__global__ void k_fill_zero(size_t count, float *__restrict__ p)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = 0.f;
}

// ------------------------------------------------------------------------------------------
// draft pieces
// ------------------------------------------------------------------------------------------

// expert draw: first a with cdf_w[a] > u, running sum in fp64, clamp to r-1
__global__ void k_pick_alpha(size_t B, int n, int r, const float *__restrict__ w, const float *__restrict__ uniforms,
                             int32_t *__restrict__ alpha)
{
    const size_t b = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    const double u = (double)uniforms[b * (1 + n)];
    double c = 0.0;
    int pick = r - 1;
    bool found = false;
    for (int a = 0; a < r; ++a) {
        c += (double)w[b * r + a];
        if (!found && c > u) { pick = a; found = true; }
    }
    alpha[b] = pick;
}

// token draw for (b, s) from the stored logits of row (b, s, a*): thread i owns a contiguous
// segment of the vocabulary; segment sums in fp64, then one thread walks the segment sums and
// the owner of the crossing segment walks its tokens.
__global__ void __launch_bounds__(kBlock) k_sample_generic(int V, int n, int r, const float *__restrict__ z,
                                                           const float *__restrict__ lse,
                                                           const int32_t *__restrict__ alpha,
                                                           const float *__restrict__ uniforms,
                                                           int32_t *__restrict__ tokens)
{
    __shared__ double seg_sum[kBlock];
    __shared__ double base;
    __shared__ int chosen;
    const size_t bs = blockIdx.x;            // b*n + s
    const size_t b = bs / n;
    const int s = (int)(bs % n);
    const size_t row = bs * r + alpha[b];
    const float *zr = z + row * V;
    const float l = lse[row];
    const double u = (double)uniforms[b * (1 + n) + 1 + s];
    const int seg = (V + kBlock - 1) / kBlock;
    const int lo = min(V, (int)threadIdx.x * seg), hi = min(V, lo + seg);
    double sum = 0.0;
    for (int v = lo; v < hi; ++v) sum += (double)expf(zr[v] - l);
    seg_sum[threadIdx.x] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        double c = 0.0;
        int pick = -1;
        for (int i = 0; i < kBlock; ++i) {
            if (c + seg_sum[i] > u) { pick = i; break; }
            c += seg_sum[i];
        }
        chosen = pick;
        base = c;
        if (pick < 0) tokens[bs] = V - 1;
    }
    __syncthreads();
    if ((int)threadIdx.x == chosen) {
        double c = base;
        int tok = hi - 1;
        for (int v = lo; v < hi; ++v) {
            c += (double)expf(zr[v] - l);
            if (c > u) { tok = v; break; }
        }
        tokens[bs] = tok;
    }
}

// logq[b] = logsumexp_a( logw_a + sum_s (z_sa[tok_s] - lse_sa) )    (eq. 9 at the drawn tuple)
__global__ void __launch_bounds__(kWave) k_logq_generic(int V, int n, int r, const float *__restrict__ logw,
                                                        const float *__restrict__ z, const float *__restrict__ lse,
                                                        const int32_t *__restrict__ tokens, float *__restrict__ logq)
{
    const size_t b = blockIdx.x;
    const int lane = threadIdx.x;
    float a = -INFINITY;
    if (lane < r) {
        a = logw[b * r + lane];
        for (int s = 0; s < n; ++s) {
            const size_t row = (b * n + s) * r + lane;
            a += z[row * V + tokens[b * n + s]] - lse[row];
        }
    }
    const float mx = wave_max(a);
    const float sum = wave_sum(lane < r ? expf(a - mx) : 0.f);
    if (lane == 0) logq[b] = mx + logf(sum);
}

// The paper's sequential scheme (eq. 11-13) from stored logits, one block per row b of the batch: for every
// token the conditional sum_a qhat_a P^(s)(. | a) is scanned in vocabulary order (thread i owns a contiguous
// run of tokens, run sums in fp64), then the expert log-weights take the drawn token's log-probabilities.
__global__ void __launch_bounds__(kBlock) k_sample_sequential_generic(int V, int n, int r, const float *__restrict__ z,
                                                                      const float *__restrict__ lse,
                                                                      const float *__restrict__ logw,
                                                                      const float *__restrict__ uniforms,
                                                                      int32_t *__restrict__ tokens,
                                                                      float *__restrict__ logq)
{
    __shared__ double seg_sum[kBlock];
    __shared__ double base;
    __shared__ float q_s[64], qh_s[64];
    __shared__ int chosen, tok_sh;
    const size_t b = blockIdx.x;
    const int tid = threadIdx.x;
    if (tid < r) q_s[tid] = logw[b * r + tid];
    __syncthreads();
    for (int s = 0; s < n; ++s) {
        const size_t row0 = (b * n + s) * r;
        const double u = (double)uniforms[b * n + s];
        if (tid == 0) {
            float mx = q_s[0];
            for (int a = 1; a < r; ++a) mx = fmaxf(mx, q_s[a]);
            float sm = 0.f;
            for (int a = 0; a < r; ++a) sm += expf(q_s[a] - mx);
            const float qn = mx + logf(sm);
            for (int a = 0; a < r; ++a) qh_s[a] = expf(q_s[a] - qn);
        }
        __syncthreads();
        const int seg = (V + kBlock - 1) / kBlock;
        const int lo = min(V, tid * seg), hi = min(V, lo + seg);
        double sum = 0.0;
        for (int v = lo; v < hi; ++v) {
            float p = 0.f;
            for (int a = 0; a < r; ++a) p += qh_s[a] * expf(z[(row0 + a) * V + v] - lse[row0 + a]);
            sum += (double)p;
        }
        seg_sum[tid] = sum;
        __syncthreads();
        if (tid == 0) {
            double c = 0.0;
            int pick = -1;
            for (int i = 0; i < kBlock; ++i) {
                if (c + seg_sum[i] > u) { pick = i; break; }
                c += seg_sum[i];
            }
            chosen = pick;
            base = c;
            if (pick < 0) tok_sh = V - 1;
        }
        __syncthreads();
        if (tid == chosen) {
            double c = base;
            int tok = hi - 1;
            for (int v = lo; v < hi; ++v) {
                float p = 0.f;
                for (int a = 0; a < r; ++a) p += qh_s[a] * expf(z[(row0 + a) * V + v] - lse[row0 + a]);
                c += (double)p;
                if (c > u) { tok = v; break; }
            }
            tok_sh = tok;
        }
        __syncthreads();
        const int tok = tok_sh;
        if (tid == 0) tokens[b * n + s] = tok;
        if (tid < r) q_s[tid] += z[(row0 + tid) * V + tok] - lse[row0 + tid];
        __syncthreads();
    }
    if (logq && tid == 0) {
        float mx = q_s[0];
        for (int a = 1; a < r; ++a) mx = fmaxf(mx, q_s[a]);
        float sm = 0.f;
        for (int a = 0; a < r; ++a) sm += expf(q_s[a] - mx);
        logq[b] = mx + logf(sm);
    }
}

// ------------------------------------------------------------------------------------------
// next-token distribution (eq. 11) and the balancing statistic (eq. 10)
// ------------------------------------------------------------------------------------------

// logp[b, v] = logsumexp_a( logw[b,a] + z[(b*r+a), v] - lse[b*r+a] )      (eq. 11 in log space)
__global__ void __launch_bounds__(kBlock) k_first_token_mix(int V, int r, size_t ld, const float *__restrict__ z,
                                                            const float *__restrict__ lse,
                                                            const float *__restrict__ logw, float *__restrict__ logp)
{
    const int v = blockIdx.y * kBlock + threadIdx.x;
    const size_t b = blockIdx.x;
    if (v >= V) return;
    float mx = -INFINITY, l = 0.f;
    for (int a = 0; a < r; ++a) {
        const size_t row = b * r + a;
        const float x = logw[row] + z[row * ld + v] - lse[row];
        if (x > mx) { l = l * expf(mx - x) + 1.f; mx = x; }
        else l += expf(x - mx);
    }
    logp[b * (size_t)V + v] = mx + logf(l);
}

// eq. 10, first stage: argmax_a of the gate pre-activations per position (first index on ties; the
// softmax is monotone), histogram per block in LDS, then integer atomics (exact, order-independent)
template <typename TIn>
__global__ void __launch_bounds__(kBlock) k_aux_argmax(size_t T, int d, int r, const TIn *__restrict__ H,
                                                       const TIn *__restrict__ G, unsigned long long *__restrict__ counts)
{
    __shared__ unsigned int hist[64];
    if (threadIdx.x < 64) hist[threadIdx.x] = 0;
    __syncthreads();
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    for (size_t t = (size_t)blockIdx.x * kWavesPerBlock + wave; t < T; t += (size_t)gridDim.x * kWavesPerBlock) {
        const TIn *h = H + t * d;
        float best = -INFINITY;
        int arg = 0;
        for (int a = 0; a < r; ++a) {
            float p = 0.f;
            for (int k = lane; k < d; k += kWave) p += ld_f32(G, (size_t)a * d + k) * ld_f32(h, k);
            p = wave_sum(p);
            if (p > best) { best = p; arg = a; }
        }
        if (lane == 0) atomicAdd(&hist[arg], 1u);
    }
    __syncthreads();
    if ((int)threadIdx.x < r && hist[threadIdx.x]) atomicAdd(&counts[threadIdx.x], (unsigned long long)hist[threadIdx.x]);
}

__global__ void k_aux_begin(int r, unsigned long long *__restrict__ counts, float *__restrict__ laux)
{
    const int i = threadIdx.x;
    if (i < r) counts[i] = 0ull;
    if (i == 0) *laux = 0.f;
}

// eq. 10, second stage: L_aux = sum_a (n_a / N - 1/r)^2
__global__ void __launch_bounds__(kWave) k_aux_finish(size_t T, int r, const unsigned long long *__restrict__ counts,
                                                      float *__restrict__ laux)
{
    const int lane = threadIdx.x;
    const float s = balance_statistic(T, r, lane < r ? counts[lane] : 0ull, lane);
    if (lane == 0) *laux = s;
}

// A chunk's logit gradients have rows of V rounded up to 4 floats (the rest zero): the products below read them with
// 16-byte loads whatever V is.
inline long dz_row(const cp_head_desc &ds) { return (long)round_up((size_t)ds.V, 4); }

// rows of the dZ chunk on this path: about 512 MiB of fp32 logit gradients at a time (256 rows with the
// least-workspace flag), and the r rows of one token never split over two chunks
inline size_t generic_chunk_rows(const cp_head_desc &ds)
{
    const size_t M = (size_t)ds.T * ds.n * ds.r;
    size_t rows = ((size_t)1 << 27) / (size_t)dz_row(ds);
    if (ds.flags & CP_HEAD_MIN_WORKSPACE) rows = 256;
    rows = rows / ds.r * ds.r;
    if (rows < (size_t)ds.r) rows = (size_t)ds.r;
    return rows < M ? rows : (M ? M : (size_t)ds.r);
}

// Tiles and splits of the backward products; those of a chunk are planned for a whole chunk.  The partial sums of a launch
// take at most 128 MiB; with the least-workspace flag nothing is split.
struct BwdPlans {
    F32Plan z, chunk[2], weights[3];            // {dY, dU}, {dH, dW, dG}: each set shares a launch
    size_t part_chunk[2], part_weights[3];      // where their partial sums start in the scratch
    size_t scratch;
};
inline BwdPlans bwd_plans(const cp_head_desc &ds)
{
    BwdPlans b;
    const long rows = (long)generic_chunk_rows(ds), d = ds.d, V = ds.V, T = (long)ds.T, nrd = (long)ds.n * ds.r * d;
    const F32Shape chunk[2] = {{rows, d, V}, {V, d, rows}}, weights[3] = {{T, d, nrd}, {nrd, d, T}, {ds.r, d, T}};
    b.z = f32_plan(rows, V, d, false);
    const bool may_split = !(ds.flags & CP_HEAD_MIN_WORKSPACE);
    f32_plan(chunk, 2, may_split, b.chunk);
    f32_plan(weights, 3, may_split, b.weights);
    size_t off = 0;
    for (int i = 0; i < 2; ++i) {
        b.part_chunk[i] = off;
        off += b.chunk[i].scratch(chunk[i].M, chunk[i].N);
    }
    b.scratch = off;
    off = 0;
    for (int i = 0; i < 3; ++i) {
        b.part_weights[i] = off;
        off += b.weights[i].scratch(weights[i].M, weights[i].N);
    }
    b.scratch = std::max(b.scratch, off);
    return b;
}

// The forward pass takes its logits a chunk of whole positions at a time, so that the statistics of their rows, a pair per
// row and column slot (up to a quarter of V floats per row), take at most 64 MiB however many positions there are, or
// 256 rows' worth with the least-workspace flag, or one position's.  64 MiB are 64 rounds of tiles over the compute units
// at any V, so the chunks' last rounds cost less than 2 %.
struct FwdChunk {
    size_t pos;         // positions
    F32Plan plan;
    int slots;
    size_t part_bytes;
};
inline FwdChunk fwd_chunk(const cp_head_desc &ds)
{
    FwdChunk c;
    const size_t nr = (size_t)ds.n * ds.r, T = (size_t)ds.T;
    const size_t most_slots = 2 * (((size_t)ds.V + 63) / 64);
    const size_t rows = (ds.flags & CP_HEAD_MIN_WORKSPACE) ? 256 : ((size_t)64 << 20) / (most_slots * sizeof(float2));
    c.pos = std::max<size_t>(rows / nr, 1);
    size_t step = 128;                                  // positions whose rows are whole tiles of rows
    for (size_t k = nr; k % 2 == 0 && step > 1; k /= 2) step /= 2;
    if (c.pos > step) c.pos -= c.pos % step;
    c.pos = std::min(c.pos, std::max<size_t>(T, 1));
    c.plan = f32_plan((long)(c.pos * nr), ds.V, ds.d, false);
    c.slots = f32_slots(c.plan.kind, ds.V);
    c.part_bytes = c.pos * nr * c.slots * sizeof(float2);
    return c;
}

struct GenericWs {
    size_t logw, C, part, dY, dZ, dg, partial, w, Y, z, lse, total;
};

inline GenericWs generic_ws(const cp_head_desc &ds, int op)
{
    GenericWs g = {};
    const size_t M = (size_t)ds.T * ds.n * ds.r, Tr = (size_t)ds.T * ds.r;
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes); return o; };
    if (op == CP_HEAD_OP_LOSS_FWD) {
        g.logw = take(Tr * 4);
        g.C = take(M * 4);
        g.part = take(fwd_chunk(ds).part_bytes);
    } else if (op == CP_HEAD_OP_LOSS_BWD) {
        g.dY = take(M * ds.d * 4);
        g.dZ = take(generic_chunk_rows(ds) * dz_row(ds) * 4);
        g.dg = take(Tr * 4);
        g.partial = take(bwd_plans(ds).scratch);
    } else {
        g.logw = take(Tr * 4);
        g.w = take(Tr * 4);
        g.Y = take(M * ds.d * 4);
        g.z = take(M * ds.V * 4);
        g.lse = take(M * 4);
    }
    g.total = off;
    return g;
}

// gate, y, then by chunks of positions the statistics of z and what follows per position; loss null: no mixture
template <typename TIn>
void fwd_rows_t(const cp_head_desc &ds, const TIn *H, const TIn *W, const TIn *U, const TIn *G, const int32_t *X,
                const GenericFwdBuffers &b, float2 *part, float *loss, hipStream_t st)
{
    const size_t T = (size_t)ds.T, n = (size_t)ds.n, r = (size_t)ds.r, nr = n * r;
    const long d = ds.d, V = ds.V;
    launch_f32_y<TIn>(ds, (int)nr, H, W, G, b.Y, b.logw, st);
    const FwdChunk c = fwd_chunk(ds);
    for (size_t t0 = 0; t0 < T; t0 += c.pos) {
        const size_t Tc = std::min(c.pos, T - t0), m0 = t0 * nr;
        launch_f32<float, TIn, false, false>(f32_problem<false, false>((const float *)b.Y + m0 * d, d, U, d, (long)(Tc * nr), V, d, d, c.plan),
                                             c.plan.kind, EpiF32Logits{part, c.slots, 1, X + t0 * n, ds.r, b.C + m0, nullptr, 0}, st);
        k_position_finish<<<(unsigned)Tc, kBlock, nr * sizeof(float), st>>>(ds.n, ds.r, c.slots, part, X + t0 * n, b.C + m0, b.lse + m0,
                                                                           b.logw + t0 * r, b.w + t0 * r, b.gamma + t0 * r,
                                                                           loss ? loss + t0 : nullptr);
    }
}

inline GenericFwdBuffers fwd_buffers(const cp_head_desc &ds, void *ctx, void *ws)
{
    const CtxLayout cl = ctx_layout(ds, false);
    const GenericWs g = generic_ws(ds, CP_HEAD_OP_LOSS_FWD);
    GenericFwdBuffers b;
    b.lse = at<float>(ctx, cl.lse);
    b.w = at<float>(ctx, cl.w);
    b.gamma = at<float>(ctx, cl.gamma);
    b.Y = at<float>(ctx, cl.Y);
    b.logw = at<float>(ws, g.logw);
    b.C = at<float>(ws, g.C);
    return b;
}

template <typename TIn>
int loss_fwd_t(const cp_head_desc &ds, const TIn *H, const TIn *W, const TIn *U, const TIn *G, const int32_t *X,
               float *loss, void *ctx, void *ws, hipStream_t st)
{
    const GenericWs g = generic_ws(ds, CP_HEAD_OP_LOSS_FWD);
    fwd_rows_t<TIn>(ds, H, W, U, G, X, fwd_buffers(ds, ctx, ws), at<float2>(ws, g.part), loss, st);
    return hipGetLastError() == hipSuccess ? CP_HEAD_OK : CP_HEAD_ERR_LAUNCH;
}

// Everything below the logit gradients, shared by the training loss and the fine-tuning loss: `fn` fills dZ with
// the gradients of the rows [m0, m0 + Mc) of one chunk, which is then contracted into dY and dU; dW, dH, dG follow.
template <typename TIn>
int bwd_from_dz_t(const cp_head_desc &ds, const TIn *H, const TIn *W, const TIn *U, const TIn *G, const float *Y,
                  const float *dg, float *dH, float *dW, float *dU, float *dG, void *ws, GenericDzLaunch fn, void *user,
                  hipStream_t st)
{
    const GenericWs g = generic_ws(ds, CP_HEAD_OP_LOSS_BWD);
    const BwdPlans pl = bwd_plans(ds);
    const long T = (long)ds.T, nr = (long)ds.n * ds.r, M = T * nr, d = ds.d, V = ds.V, nrd = nr * d, Vp = dz_row(ds);
    float *dY = at<float>(ws, g.dY), *dZ = at<float>(ws, g.dZ);
    auto part = [&](size_t off) { return at<float>(ws, g.partial + off); };
    const long chunk = (long)generic_chunk_rows(ds);
    for (long m0 = 0; m0 < M; m0 += chunk) {
        const long Mc = std::min(chunk, M - m0);
        fn(user, (size_t)m0, (size_t)Mc, dZ, Vp, st);
        // dY = dZ U and dU (+)= dZ^T Y
        float *py_part = part(pl.part_chunk[0]), *pu_part = part(pl.part_chunk[1]);
        const F32Problem py = f32_problem<false, true>((const float *)dZ, Vp, U, d, Mc, d, Vp, V, pl.chunk[0]);
        F32Problem pu{};
        if (dU) pu = f32_problem<true, true>((const float *)dZ, Vp, Y + m0 * d, d, V, d, Mc, Mc, pl.chunk[1]);
        with_f32_tile<false>(pl.chunk[0].kind, false, [&](auto tile) {
            typedef decltype(tile) Tile;
            k_gemm_f32<F32Gemm<Tile, float, TIn, false, true>, EpiF32Store, F32Gemm<Tile, float, float, true, true>, EpiF32Store,
                       NoF32Problem, NoEpi><<<(unsigned)(py.tiles() + pu.tiles()), kF32Threads, 0, st>>>(
                py, EpiF32Store{dY + m0 * d, d, 0, py_part}, pu, EpiF32Store{dU, d, m0 ? 1 : 0, pu_part}, F32Problem{}, NoEpi{});
        });
        AddSplits add{};
        add.gate_job = -1;
        add.add(pl.chunk[0], Mc, d, py_part, dY + m0 * d, false);
        if (dU) add.add(pl.chunk[1], V, d, pu_part, dU, m0 != 0);
        launch_add_splits<TIn>(add, st);
    }
    // dH = dY W + dg G, dW_sa = dY_sa^T H and dG = dg^T H (contractions over the positions)
    float *ph_part = part(pl.part_weights[0]), *pw_part = part(pl.part_weights[1]), *pg_part = part(pl.part_weights[2]);
    const F32Problem ph = f32_problem<false, true>((const float *)dY, nrd, W, d, T, d, nrd, nrd, pl.weights[0]);
    F32Problem pw{}, pg{};
    if (dW) pw = f32_problem<true, true>((const float *)dY, nrd, H, d, nrd, d, T, T, pl.weights[1]);
    if (dG) pg = f32_problem<true, true>(dg, ds.r, H, d, ds.r, d, T, T, pl.weights[2]);
    with_f32_tile<false>(pl.weights[0].kind, false, [&](auto tile) {
        typedef decltype(tile) Tile;
        typedef F32Gemm<Tile, float, TIn, true, true> Gw;
        k_gemm_f32<F32Gemm<Tile, float, TIn, false, true>, EpiF32Dh<TIn>, Gw, EpiF32Store, Gw, EpiF32Store>
            <<<(unsigned)(ph.tiles() + pw.tiles() + pg.tiles()), kF32Threads, 0, st>>>(
                ph, EpiF32Dh<TIn>{dH, dg, G, ds.r, ph_part}, pw, EpiF32Store{dW, d, 0, pw_part}, pg, EpiF32Store{dG, d, 0, pg_part});
    });
    AddSplits add{};
    add.N = d; add.r = ds.r; add.dg = dg; add.G = G;
    add.gate_job = pl.weights[0].splits > 1 ? 0 : -1;
    add.add(pl.weights[0], T, d, ph_part, dH, false);
    if (dW) add.add(pl.weights[1], nrd, d, pw_part, dW, false);
    if (dG) add.add(pl.weights[2], ds.r, d, pg_part, dG, false);
    launch_add_splits<TIn>(add, st);
    return hipGetLastError() == hipSuccess ? CP_HEAD_OK : CP_HEAD_ERR_LAUNCH;
}

template <typename TIn>
struct LossDzArgs {
    const cp_head_desc *ds;
    const TIn *U;
    const float *Y, *lse, *w, *gamma, *dloss;
    const int32_t *X;
    float scale;
    float *dg;
};
template <typename TIn>
void loss_dz_launch(void *user, size_t m0, size_t Mc, float *dZ, long ldz, hipStream_t st)
{
    const LossDzArgs<TIn> *a = static_cast<const LossDzArgs<TIn> *>(user);
    const cp_head_desc &ds = *a->ds;
    const long d = ds.d;
    const F32Plan plan = f32_plan((long)generic_chunk_rows(ds), ds.V, d, false);
    launch_f32<float, TIn, false, false>(f32_problem<false, false>(a->Y + m0 * d, d, a->U, d, (long)Mc, ds.V, d, d, plan), plan.kind,
                                         EpiF32Dz{dZ, ldz, ldz, m0, 1, ds.n, ds.r, a->X, a->lse, a->w, a->gamma, a->dloss, a->scale,
                                                  a->dg}, st);
}

template <typename TIn>
int loss_bwd_t(const cp_head_desc &ds, const TIn *H, const TIn *W, const TIn *U, const TIn *G, const int32_t *X,
               const float *dloss, float scale, const void *ctx, float *dH, float *dW, float *dU, float *dG,
               void *ws, hipStream_t st)
{
    const CtxLayout cl = ctx_layout(ds, false);
    const GenericWs g = generic_ws(ds, CP_HEAD_OP_LOSS_BWD);
    const float *lse = at<float>(ctx, cl.lse), *w = at<float>(ctx, cl.w), *gamma = at<float>(ctx, cl.gamma);
    const float *Y = at<float>(ctx, cl.Y);
    float *dg = at<float>(ws, g.dg);
    LossDzArgs<TIn> args{&ds, U, Y, lse, w, gamma, dloss, X, scale, dg};
    return bwd_from_dz_t<TIn>(ds, H, W, U, G, Y, dg, dH, dW, dU, dG, ws, loss_dz_launch<TIn>, &args, st);
}

// The logits of all `rows` head rows (row-major, V apart) and their log-normalisers, for the draft-type calls
template <typename TIn>
void launch_f32_kept_logits(const cp_head_desc &ds, long rows, const TIn *U, const float *Y, float *z, float *lse, hipStream_t st)
{
    const long d = ds.d, V = ds.V;
    const F32Plan plan = f32_plan(rows, V, d, false);
    launch_f32<float, TIn, false, false>(f32_problem<false, false>(Y, d, U, d, rows, V, d, d, plan), plan.kind,
                                         EpiF32Logits{nullptr, 0, 1, nullptr, 1, nullptr, z, V}, st);
    k_lse_of_rows<<<(unsigned)std::min<long>(rows, 1 << 20), V > 2048 ? 1024 : 256, 0, st>>>((size_t)rows, ds.V, z, lse);
}

template <typename TIn>
int draft_t(const cp_head_desc &ds, const TIn *H, const TIn *W, const TIn *U, const TIn *G, const float *uniforms,
            int32_t *alpha, int32_t *tokens, float *logq, void *ws, hipStream_t st)
{
    const GenericWs g = generic_ws(ds, CP_HEAD_OP_DRAFT);
    const size_t B = (size_t)ds.T, M = B * ds.n * ds.r;
    float *logw = at<float>(ws, g.logw), *w = at<float>(ws, g.w), *Y = at<float>(ws, g.Y);
    float *z = at<float>(ws, g.z), *lse = at<float>(ws, g.lse);
    k_gate<TIn><<<(unsigned)B, kWave, 0, st>>>(ds.d, ds.r, H, G, logw, w);
    k_pick_alpha<<<blocks_for(B, kWave), kWave, 0, st>>>(B, ds.n, ds.r, w, uniforms, alpha);
    launch_draft_y(ds, ds.n * ds.r, H, W, Y, st);
    launch_f32_kept_logits<TIn>(ds, (long)M, U, Y, z, lse, st);
    k_sample_generic<<<(unsigned)(B * ds.n), kBlock, 0, st>>>(ds.V, ds.n, ds.r, z, lse, alpha, uniforms, tokens);
    if (logq) k_logq_generic<<<(unsigned)B, kWave, 0, st>>>(ds.V, ds.n, ds.r, logw, z, lse, tokens, logq);
    return hipGetLastError() == hipSuccess ? CP_HEAD_OK : CP_HEAD_ERR_LAUNCH;
}

template <typename TIn>
int draft_sequential_t(const cp_head_desc &ds, const TIn *H, const TIn *W, const TIn *U, const TIn *G,
                       const float *uniforms, int32_t *tokens, float *logq, void *ws, hipStream_t st)
{
    const GenericWs g = generic_ws(ds, CP_HEAD_OP_DRAFT);
    const size_t B = (size_t)ds.T, M = B * ds.n * ds.r;
    float *logw = at<float>(ws, g.logw), *w = at<float>(ws, g.w), *Y = at<float>(ws, g.Y);
    float *z = at<float>(ws, g.z), *lse = at<float>(ws, g.lse);
    k_gate<TIn><<<(unsigned)B, kWave, 0, st>>>(ds.d, ds.r, H, G, logw, w);
    launch_draft_y(ds, ds.n * ds.r, H, W, Y, st);
    launch_f32_kept_logits<TIn>(ds, (long)M, U, Y, z, lse, st);
    k_sample_sequential_generic<<<(unsigned)B, kBlock, 0, st>>>(ds.V, ds.n, ds.r, z, lse, logw, uniforms, tokens, logq);
    return hipGetLastError() == hipSuccess ? CP_HEAD_OK : CP_HEAD_ERR_LAUNCH;
}

}  // namespace

int generic_draft_sequential(const cp_head_desc &ds, const void *H, const void *W, const void *U, const void *G,
                             const float *uniforms, int32_t *tokens, float *logq, void *ws, hipStream_t st)
{
    if (ds.T == 0) return CP_HEAD_OK;
    if (ds.dtype == CP_HEAD_FP32)
        return draft_sequential_t<float>(ds, (const float *)H, (const float *)W, (const float *)U, (const float *)G,
                                         uniforms, tokens, logq, ws, st);
    return draft_sequential_t<bf16_t>(ds, (const bf16_t *)H, (const bf16_t *)W, (const bf16_t *)U, (const bf16_t *)G,
                                      uniforms, tokens, logq, ws, st);
}

size_t generic_workspace_bytes(const cp_head_desc &ds, int op) { return generic_ws(ds, op).total; }

size_t generic_bwd_chunk_rows(const cp_head_desc &ds) { return generic_chunk_rows(ds); }
long generic_dz_row(const cp_head_desc &ds) { return dz_row(ds); }

int generic_fwd_rows(const cp_head_desc &ds, const void *H, const void *W, const void *U, const void *G,
                     const int32_t *X, void *ctx, void *ws, GenericFwdBuffers *out, hipStream_t st)
{
    const GenericFwdBuffers b = fwd_buffers(ds, ctx, ws);
    float2 *part = at<float2>(ws, generic_ws(ds, CP_HEAD_OP_LOSS_FWD).part);
    if (ds.dtype == CP_HEAD_FP32)
        fwd_rows_t<float>(ds, (const float *)H, (const float *)W, (const float *)U, (const float *)G, X, b, part, nullptr, st);
    else
        fwd_rows_t<bf16_t>(ds, (const bf16_t *)H, (const bf16_t *)W, (const bf16_t *)U, (const bf16_t *)G, X, b, part, nullptr, st);
    *out = b;
    return hipGetLastError() == hipSuccess ? CP_HEAD_OK : CP_HEAD_ERR_LAUNCH;
}

void generic_logits_rows(const cp_head_desc &ds, const void *U, const float *Y, size_t m0, size_t Mc, float *z, long ldz,
                         hipStream_t st)
{
    const long d = ds.d, V = ds.V;
    const F32Plan plan = f32_plan((long)generic_chunk_rows(ds), V, d, false);
    const EpiF32Logits epi{nullptr, 0, 1, nullptr, 1, nullptr, z, ldz};
    if (ds.dtype == CP_HEAD_FP32)
        launch_f32<float, float, false, false>(f32_problem<false, false>(Y + m0 * d, d, (const float *)U, d, (long)Mc, V, d, d, plan),
                                               plan.kind, epi, st);
    else
        launch_f32<float, bf16_t, false, false>(f32_problem<false, false>(Y + m0 * d, d, (const bf16_t *)U, d, (long)Mc, V, d, d, plan),
                                                plan.kind, epi, st);
}

int generic_bwd_from_dz(const cp_head_desc &ds, const void *H, const void *W, const void *U, const void *G,
                        const float *Y, const float *dg, float *dH, float *dW, float *dU, float *dG, void *ws,
                        GenericDzLaunch fn, void *user, hipStream_t st)
{
    if (ds.dtype == CP_HEAD_FP32)
        return bwd_from_dz_t<float>(ds, (const float *)H, (const float *)W, (const float *)U, (const float *)G, Y, dg,
                                    dH, dW, dU, dG, ws, fn, user, st);
    return bwd_from_dz_t<bf16_t>(ds, (const bf16_t *)H, (const bf16_t *)W, (const bf16_t *)U, (const bf16_t *)G, Y, dg,
                                 dH, dW, dU, dG, ws, fn, user, st);
}

int generic_loss_fwd(const cp_head_desc &ds, const void *H, const void *W, const void *U, const void *G,
                     const int32_t *X, float *loss, void *ctx, void *ws, hipStream_t st)
{
    if (ds.T == 0) return CP_HEAD_OK;
    if (ds.dtype == CP_HEAD_FP32)
        return loss_fwd_t<float>(ds, (const float *)H, (const float *)W, (const float *)U, (const float *)G, X, loss,
                                 ctx, ws, st);
    return loss_fwd_t<bf16_t>(ds, (const bf16_t *)H, (const bf16_t *)W, (const bf16_t *)U, (const bf16_t *)G, X, loss,
                              ctx, ws, st);
}

void launch_fill_zero(float *p, size_t count, hipStream_t st)
{
    if (p && count) k_fill_zero<<<blocks_for(count, kBlock), kBlock, 0, st>>>(count, p);
}

int generic_loss_bwd(const cp_head_desc &ds, const void *H, const void *W, const void *U, const void *G,
                     const int32_t *X, const float *dloss, float scale, const void *ctx, float *dH, float *dW,
                     float *dU, float *dG, void *ws, hipStream_t st)
{
    if (ds.T == 0) {   // empty batch: the weight gradients are empty sums
        launch_fill_zero(dW, (size_t)ds.n * ds.r * ds.d * ds.d, st);
        launch_fill_zero(dU, (size_t)ds.V * ds.d, st);
        launch_fill_zero(dG, (size_t)ds.r * ds.d, st);
        return hipGetLastError() == hipSuccess ? CP_HEAD_OK : CP_HEAD_ERR_LAUNCH;
    }
    if (ds.dtype == CP_HEAD_FP32)
        return loss_bwd_t<float>(ds, (const float *)H, (const float *)W, (const float *)U, (const float *)G, X, dloss,
                                 scale, ctx, dH, dW, dU, dG, ws, st);
    return loss_bwd_t<bf16_t>(ds, (const bf16_t *)H, (const bf16_t *)W, (const bf16_t *)U, (const bf16_t *)G, X,
                              dloss, scale, ctx, dH, dW, dU, dG, ws, st);
}

int generic_draft(const cp_head_desc &ds, const void *H, const void *W, const void *U, const void *G,
                  const float *uniforms, int32_t *alpha, int32_t *tokens, float *logq, void *ws, hipStream_t st)
{
    if (ds.T == 0) return CP_HEAD_OK;
    if (ds.dtype == CP_HEAD_FP32)
        return draft_t<float>(ds, (const float *)H, (const float *)W, (const float *)U, (const float *)G, uniforms,
                              alpha, tokens, logq, ws, st);
    return draft_t<bf16_t>(ds, (const bf16_t *)H, (const bf16_t *)W, (const bf16_t *)U, (const bf16_t *)G, uniforms,
                           alpha, tokens, logq, ws, st);
}

// ---- first-token marginal on the plain path: z of the r first-head rows is stored, then mixed
struct GenericFirstWs {
    size_t logw, w, Y, z, lse, total;
};
static GenericFirstWs generic_first_ws(const cp_head_desc &ds)
{
    GenericFirstWs g;
    const size_t rows = (size_t)ds.T * ds.r;
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes); return o; };
    g.logw = take(rows * 4);
    g.w = take(rows * 4);
    g.Y = take(rows * ds.d * 4);
    g.z = take(rows * ds.V * 4);
    g.lse = take(rows * 4);
    g.total = off;
    return g;
}
size_t generic_first_token_workspace_bytes(const cp_head_desc &ds) { return generic_first_ws(ds).total; }

void launch_first_token_mix(const cp_head_desc &ds, const float *z, size_t ld, const float *lse, const float *logw,
                            float *logp, hipStream_t st)
{
    if (ds.T == 0) return;
    k_first_token_mix<<<dim3((unsigned)ds.T, blocks_for((size_t)ds.V, kBlock)), kBlock, 0, st>>>(
        ds.V, ds.r, ld, z, lse, logw, logp);
}

template <typename TIn>
static int first_token_t(const cp_head_desc &ds, const TIn *H, const TIn *W, const TIn *U, const TIn *G, float *logp,
                         void *ws, hipStream_t st)
{
    const GenericFirstWs g = generic_first_ws(ds);
    const size_t rows = (size_t)ds.T * ds.r;
    float *logw = at<float>(ws, g.logw), *w = at<float>(ws, g.w), *Y = at<float>(ws, g.Y);
    float *z = at<float>(ws, g.z), *lse = at<float>(ws, g.lse);
    k_gate<TIn><<<(unsigned)ds.T, kWave, 0, st>>>(ds.d, ds.r, H, G, logw, w);
    // the first head's matrices are the first r blocks of W, so its rows are (b, a) with nr = r
    launch_draft_y(ds, ds.r, H, W, Y, st);
    launch_f32_kept_logits<TIn>(ds, (long)rows, U, Y, z, lse, st);
    launch_first_token_mix(ds, z, (size_t)ds.V, lse, logw, logp, st);
    return hipGetLastError() == hipSuccess ? CP_HEAD_OK : CP_HEAD_ERR_LAUNCH;
}

int generic_first_token(const cp_head_desc &ds, const void *H, const void *W, const void *U, const void *G,
                        float *logp, void *ws, hipStream_t st)
{
    if (ds.T == 0) return CP_HEAD_OK;
    if (ds.dtype == CP_HEAD_FP32)
        return first_token_t<float>(ds, (const float *)H, (const float *)W, (const float *)U, (const float *)G, logp, ws, st);
    return first_token_t<bf16_t>(ds, (const bf16_t *)H, (const bf16_t *)W, (const bf16_t *)U, (const bf16_t *)G, logp, ws,
                                 st);
}

int aux_balance(const cp_head_desc &ds, const void *H, const void *G, int64_t *counts, float *laux, hipStream_t st)
{
    unsigned long long *c = reinterpret_cast<unsigned long long *>(counts);
    k_aux_begin<<<1, 64, 0, st>>>(ds.r, c, laux);
    bool finished = false;
    if (ds.T > 0) {
        const unsigned blocks = (unsigned)std::min<size_t>(((size_t)ds.T + kWavesPerBlock - 1) / kWavesPerBlock, 4096);
        if (use_fast_path(ds))
            finished = launch_aux_argmax_bf16(ds, (const bf16_t *)H, (const bf16_t *)G, c, laux, st);
        else if (ds.dtype == CP_HEAD_FP32)
            k_aux_argmax<float><<<blocks, kBlock, 0, st>>>((size_t)ds.T, ds.d, ds.r, (const float *)H, (const float *)G, c);
        else
            k_aux_argmax<bf16_t><<<blocks, kBlock, 0, st>>>((size_t)ds.T, ds.d, ds.r, (const bf16_t *)H,
                                                            (const bf16_t *)G, c);
    }
    if (!finished) k_aux_finish<<<1, kWave, 0, st>>>((size_t)ds.T, ds.r, c, laux);
    return hipGetLastError() == hipSuccess ? CP_HEAD_OK : CP_HEAD_ERR_LAUNCH;
}

// ---- full heads on the plain path: the products of all (s, a) with the positions in one launch, whose head rows are
// m = t n r + sa.  A chunk's gradients are stored [positions, n r, V], so that dH and dF are one product each.
struct GenericFullWs {
    size_t logw, C, dg, dZ, partial, total;     // dZ: in the forward pass, the row statistics of a chunk
    size_t chunk_pos, fwd_pos;                  // positions per chunk of the backward and of the forward pass
    F32Plan z, zc, dh, df, dG;
};
static GenericFullWs generic_full_ws(const cp_head_desc &ds)
{
    GenericFullWs g;
    const size_t T = (size_t)ds.T, nr = (size_t)ds.n * ds.r;
    const long d = ds.d, V = ds.V, nrV = (long)nr * V;
    // whole positions per chunk: at most 512 MiB of fp32 logit gradients at a time, at least one position
    size_t pos = ((size_t)1 << 27) / ((size_t)ds.V * nr);
    if (pos < 1) pos = 1;
    g.chunk_pos = pos < T ? pos : (T ? T : 1);
    const long P = (long)g.chunk_pos;
    // the forward pass: as many positions as have room for their rows' statistics where the backward pass has its gradients
    const size_t dz_bytes = g.chunk_pos * nr * ds.V * 4, most_slots = 2 * (((size_t)ds.V + 63) / 64);
    size_t fwd = std::max<size_t>(dz_bytes / (nr * most_slots * sizeof(float2)), 1);
    if (fwd > 128) fwd -= fwd % 128;
    g.fwd_pos = std::min(fwd, std::max<size_t>(T, 1));
    g.z = f32_plan((long)g.fwd_pos, V, d, false, (long)nr);
    g.zc = f32_plan(P, V, d, false, (long)nr);
    const bool may_split = !(ds.flags & CP_HEAD_MIN_WORKSPACE);
    g.dh = f32_plan(P, d, nrV, may_split);
    g.df = f32_plan(nrV, d, P, false);
    g.dG = f32_plan(ds.r, d, (long)T, may_split);
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes); return o; };
    g.logw = take(T * ds.r * 4);
    g.C = take(T * nr * 4);
    g.dg = take(T * ds.r * 4);
    g.dZ = take(std::max(dz_bytes, g.fwd_pos * nr * f32_slots(g.z.kind, V) * sizeof(float2)));
    g.partial = take(std::max(g.dh.scratch(P, d), g.dG.scratch(ds.r, d)));
    g.total = off;
    return g;
}
size_t generic_full_workspace_bytes(const cp_head_desc &ds) { return generic_full_ws(ds).total; }

template <typename TIn>
static int full_fwd_t(const cp_head_desc &ds, const TIn *H, const TIn *F, const TIn *G, const int32_t *X, float *loss,
                      void *ctx, void *ws, hipStream_t st)
{
    const CtxLayout cl = ctx_layout(ds, false);      // lse, w, gamma at the same offsets; no y is kept
    const GenericFullWs g = generic_full_ws(ds);
    const long T = (long)ds.T, d = ds.d, V = ds.V, nr = (long)ds.n * ds.r;
    float *lse = at<float>(ctx, cl.lse), *w = at<float>(ctx, cl.w), *gamma = at<float>(ctx, cl.gamma);
    float *logw = at<float>(ws, g.logw), *C = at<float>(ws, g.C);
    float2 *part = at<float2>(ws, g.dZ);
    const int slots = f32_slots(g.z.kind, V);
    const F32Plan pg = f32_plan(T, ds.r, d, false);
    launch_f32<TIn, TIn, false, false>(f32_problem<false, false>(H, d, G, d, T, ds.r, d, d, pg), pg.kind, EpiF32Store{logw, ds.r, 0, nullptr}, st);
    for (long t0 = 0; t0 < T; t0 += (long)g.fwd_pos) {
        const long Tc = std::min((long)g.fwd_pos, T - t0), m0 = t0 * nr;
        const int32_t *Xc = X + t0 * ds.n;
        launch_f32<TIn, TIn, false, false>(f32_batch(f32_problem<false, false>(H + t0 * d, d, F, d, Tc, V, d, d, g.z), (int)nr, V * d),
                                           g.z.kind, EpiF32Logits{part, slots, nr, Xc, ds.r, C + m0, nullptr, 0}, st);
        k_position_finish<<<(unsigned)Tc, kBlock, (size_t)nr * sizeof(float), st>>>(ds.n, ds.r, slots, part, Xc, C + m0, lse + m0,
                                                                                   logw + t0 * ds.r, w + t0 * ds.r, gamma + t0 * ds.r,
                                                                                   loss + t0);
    }
    return hipGetLastError() == hipSuccess ? CP_HEAD_OK : CP_HEAD_ERR_LAUNCH;
}

template <typename TIn>
static int full_bwd_t(const cp_head_desc &ds, const TIn *H, const TIn *F, const TIn *G, const int32_t *X,
                      const float *dloss, float scale, const void *ctx, float *dH, float *dF, float *dG, void *ws,
                      hipStream_t st)
{
    const CtxLayout cl = ctx_layout(ds, false);
    const GenericFullWs g = generic_full_ws(ds);
    const long T = (long)ds.T, d = ds.d, V = ds.V, nr = (long)ds.n * ds.r, nrV = nr * V;
    const float *lse = at<float>(ctx, cl.lse), *w = at<float>(ctx, cl.w), *gamma = at<float>(ctx, cl.gamma);
    float *dg = at<float>(ws, g.dg), *dZ = at<float>(ws, g.dZ), *partial = at<float>(ws, g.partial);
    for (long t0 = 0; t0 < T; t0 += (long)g.chunk_pos) {
        const long Tc = std::min((long)g.chunk_pos, T - t0);
        launch_f32<TIn, TIn, false, false>(f32_batch(f32_problem<false, false>(H + t0 * d, d, F, d, Tc, V, d, d, g.zc), (int)nr, V * d),
                                           g.zc.kind, EpiF32Dz{dZ, nrV, V, (size_t)(t0 * nr), nr, ds.n, ds.r, X, lse, w, gamma, dloss,
                                                               scale, dg}, st);
        // dH = dZ F + dg G (contraction over heads and vocabulary), dF (+)= dZ^T H (over the chunk's positions)
        const F32Problem ph = f32_problem<false, true>((const float *)dZ, nrV, F, d, Tc, d, nrV, nrV, g.dh);
        launch_f32<float, TIn, false, true>(ph, g.dh.kind, EpiF32Dh<TIn>{dH + t0 * d, dg + t0 * ds.r, G, ds.r, partial}, st);
        AddSplits add{};
        add.N = d; add.r = ds.r; add.dg = dg + t0 * ds.r; add.G = G;
        add.add(g.dh, Tc, d, partial, dH + t0 * d, false);
        launch_add_splits<TIn>(add, st);
        if (dF)
            launch_f32<float, TIn, true, true>(f32_problem<true, true>((const float *)dZ, nrV, H + t0 * d, d, nrV, d, Tc, Tc, g.df),
                                               g.df.kind, EpiF32Store{dF, d, t0 ? 1 : 0, nullptr}, st);
    }
    if (dG) {
        launch_f32<float, TIn, true, true>(f32_problem<true, true>((const float *)dg, ds.r, H, d, ds.r, d, T, T, g.dG), g.dG.kind,
                                           EpiF32Store{dG, d, 0, partial}, st);
        AddSplits add{};
        add.gate_job = -1;
        add.add(g.dG, ds.r, d, partial, dG, false);
        launch_add_splits<TIn>(add, st);
    }
    return hipGetLastError() == hipSuccess ? CP_HEAD_OK : CP_HEAD_ERR_LAUNCH;
}

int generic_full_loss_fwd(const cp_head_desc &ds, const void *H, const void *F, const void *G, const int32_t *X,
                          float *loss, void *ctx, void *ws, hipStream_t st)
{
    if (ds.T == 0) return CP_HEAD_OK;
    if (ds.dtype == CP_HEAD_FP32)
        return full_fwd_t<float>(ds, (const float *)H, (const float *)F, (const float *)G, X, loss, ctx, ws, st);
    return full_fwd_t<bf16_t>(ds, (const bf16_t *)H, (const bf16_t *)F, (const bf16_t *)G, X, loss, ctx, ws, st);
}

int generic_full_loss_bwd(const cp_head_desc &ds, const void *H, const void *F, const void *G, const int32_t *X,
                          const float *dloss, float scale, const void *ctx, float *dH, float *dF, float *dG, void *ws,
                          hipStream_t st)
{
    if (ds.T == 0) {
        launch_fill_zero(dF, (size_t)ds.n * ds.r * ds.V * ds.d, st);
        launch_fill_zero(dG, (size_t)ds.r * ds.d, st);
        return hipGetLastError() == hipSuccess ? CP_HEAD_OK : CP_HEAD_ERR_LAUNCH;
    }
    if (ds.dtype == CP_HEAD_FP32)
        return full_bwd_t<float>(ds, (const float *)H, (const float *)F, (const float *)G, X, dloss, scale, ctx, dH, dF, dG,
                                 ws, st);
    return full_bwd_t<bf16_t>(ds, (const bf16_t *)H, (const bf16_t *)F, (const bf16_t *)G, X, dloss, scale, ctx, dH, dF,
                              dG, ws, st);
}

void launch_mixture(const cp_head_desc &ds, const float *logw, const float *C, float *out, float *gamma,
                    float sign, hipStream_t st)
{
    if (ds.T == 0) return;
    k_mixture<<<(unsigned)ds.T, kWave, 0, st>>>(ds.n, ds.r, logw, C, out, gamma, sign);
}

void launch_pick_alpha(const cp_head_desc &ds, const float *w, const float *uniforms, int32_t *alpha, hipStream_t st)
{
    if (ds.T == 0) return;
    k_pick_alpha<<<blocks_for((size_t)ds.T, kWave), kWave, 0, st>>>((size_t)ds.T, ds.n, ds.r, w, uniforms, alpha);
}

}  // namespace cph
