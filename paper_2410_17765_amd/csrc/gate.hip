// The gate of the matrix-core path (bf16 storage, d a multiple of 64): G h for all positions, as log-softmax
// (eq. 7), as arg-max counts (eq. 10), and the gate gradient dG = dg^T H.
//
// All three read H once and do little else: they are bound by that stream (T d 2 bytes).
#include "cp_internal.hpp"
#include "tile16.hpp"

#include <type_traits>

namespace cph {

namespace {

constexpr int kBlock = 256, kWaves = kBlock / kWave;

typedef float f32x4_t __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------------------------------------
// G h of 16 positions per step of a workgroup on the 16x16x32 matrix instruction, for the arg-max counts.
// The kernel it replaces walked H with 2-byte loads, once per expert, one position per wavefront: 353 us for the
// arg-max at T = 16384, d = 4096, r = 8 (0.4 TB/s); this one takes 31 us (4.4 TB/s).  Here the four wavefronts share the
// contraction, and the partial products meet in LDS.  Experts beyond r repeat the last row of G and are dropped.
// ------------------------------------------------------------------------------------------
constexpr int kRows = 16;

// out[row][expert] for the rows t0 .. t0+15 (rows past T repeat the last one); 16 NG >= r
template <int NG>
__device__ __forceinline__ void gate_rows(size_t t0, size_t T, int d, int r, const bf16_t *__restrict__ H,
                                          const bf16_t *__restrict__ G, float (&red)[kWaves][kRows][NG * 16 + 1])
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row = lane & 15, q = lane >> 4;
    const size_t t = t0 + row < T ? t0 + row : T - 1;
    const bf16_t *h = H + t * d + q * 16;
    const bf16_t *g[NG];
#pragma unroll
    for (int e = 0; e < NG; ++e) g[e] = G + (size_t)min(e * 16 + row, r - 1) * d + q * 16;
    f32x4_t acc[NG];
#pragma unroll
    for (int e = 0; e < NG; ++e) acc[e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    tile16_products<kWaves, NG == 1 ? 4 : 2>(h, g, d, wave, acc);
#pragma unroll
    for (int e = 0; e < NG; ++e)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[wave][tile16_row(v, lane)][e * 16 + row] = acc[e][v];
}

// logw = log_softmax(G h), w = exp(logw)   (eq. 7)
//
// Every sum has one order, which does not depend on the shape: lane l adds the columns l, l + 64, ... in turn, then lanes
// 32, 16, ... 1 apart add up.  The log-weights enter exponentials whose results are rounded to bf16, in the fine-tuning
// loss next to logits of magnitude ten, so that another order of the same fp32 sums moved its gradients by 1e-4 (the order
// of the matrix instruction, which the arg-max counts above keep).
// A wavefront takes four positions and up to eight experts at a time: a value of H meets eight experts and one of G four
// positions in registers, and 48 loads are in flight, where one position and one expert at a time had each load feed one
// multiplication, one latency after the other.  Bound by those latencies for few positions, by the stream of H and the
// vector units next to it for many: 8.7 us at T = 1500, d = 768, r = 5 (22 one at a time, 6.3 with the matrix instruction),
// 36 us at T = 16384, d = 4096, r = 8 (3.7 TB/s; 29 with the matrix instruction), in calls of 7 and 440 ms.
// UN blocks of 64 columns are in flight, so that the loads per wavefront stay near 48 with fewer experts.
constexpr int kGatePos = 4;

// v[i], summed over the wavefront for each of the COUNT of them, arrives in v[0] of the lanes whose upper bits are i: at
// each step a lane hands half of its values to the lane OFF away and adds what it gets for the other half.
template <int COUNT, int OFF, int N>
__device__ __forceinline__ void wave_sum_each(float (&v)[N], int lane)
{
    if constexpr (COUNT > 1) {
        const bool up = lane & OFF;
#pragma unroll
        for (int i = 0; i < COUNT / 2; ++i) {
            const float keep = up ? v[i + COUNT / 2] : v[i], give = up ? v[i] : v[i + COUNT / 2];
            v[i] = keep + __shfl_xor(give, OFF, kWave);
        }
    } else {
        v[0] += __shfl_xor(v[0], OFF, kWave);
    }
    if constexpr (OFF > 1) wave_sum_each<(COUNT > 1 ? COUNT / 2 : 1), OFF / 2>(v, lane);
}

// element at a byte offset from a pointer that all lanes share
__device__ __forceinline__ bf16_t ld_at(const bf16_t *p, unsigned bytes)
{
    return *reinterpret_cast<const bf16_t *>(reinterpret_cast<const char *>(p) + bytes);
}

template <int EXPERTS, int UN>
__global__ void __launch_bounds__(kBlock) k_gate_bf16(size_t T, int d, int r, const bf16_t *__restrict__ H, const bf16_t *__restrict__ G,
                                                      float *__restrict__ logw, float *__restrict__ w)
{
    __shared__ float g_s[kWaves][kGatePos][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const size_t t0 = ((size_t)blockIdx.x * kWaves + wave) * kGatePos;
    const bf16_t *h[kGatePos];                      // positions past T and experts past r repeat the last one, not stored
#pragma unroll
    for (int p = 0; p < kGatePos; ++p) h[p] = H + (t0 + p < T ? t0 + p : T - 1) * d;
    for (int a0 = 0; a0 < r; a0 += EXPERTS) {
        const bf16_t *g[EXPERTS];
#pragma unroll
        for (int e = 0; e < EXPERTS; ++e) g[e] = G + (size_t)min(a0 + e, r - 1) * d;
        float acc[kGatePos * EXPERTS];
#pragma unroll
        for (int i = 0; i < kGatePos * EXPERTS; ++i) acc[i] = 0.f;
        // `blocks` blocks of 64 columns, all their loads ahead of the arithmetic
        auto add = [&](int k0, auto blocks) {
            constexpr int N = decltype(blocks)::value;
            bf16_t hv[N][kGatePos], gv[N][EXPERTS];
#pragma unroll
            for (int u = 0; u < N; ++u) {
                const unsigned at = (unsigned)(k0 + u * kWave + lane) * sizeof(bf16_t);
#pragma unroll
                for (int p = 0; p < kGatePos; ++p) hv[u][p] = ld_at(h[p], at);
#pragma unroll
                for (int e = 0; e < EXPERTS; ++e) gv[u][e] = ld_at(g[e], at);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < N; ++u)
#pragma unroll
                for (int p = 0; p < kGatePos; ++p)
#pragma unroll
                    for (int e = 0; e < EXPERTS; ++e)
                        acc[p * EXPERTS + e] += bf16_to_f32(gv[u][e]) * bf16_to_f32(hv[u][p]);
        };
        int k0 = 0;
        for (; k0 + UN * kWave <= d; k0 += UN * kWave) add(k0, std::integral_constant<int, UN>());
        for (; k0 < d; k0 += kWave) add(k0, std::integral_constant<int, 1>());
        wave_sum_each<kGatePos * EXPERTS, 32>(acc, lane);
        constexpr int kLanes = kWave / (kGatePos * EXPERTS);      // that hold the same sum
        const int at = lane / kLanes;
        if (lane % kLanes == 0 && a0 + at % EXPERTS < r) g_s[wave][at / EXPERTS][a0 + at % EXPERTS] = acc[0];
    }
    __syncthreads();
    for (int p = 0; p < kGatePos && t0 + p < T; ++p) {
        const float mine = lane < r ? g_s[wave][p][lane] : -INFINITY;
        const float mx = wave_max(mine);
        const float s = wave_sum(lane < r ? expf(mine - mx) : 0.f);
        const float lse = mx + logf(s);
        if (lane < r) {
            logw[(t0 + p) * r + lane] = mine - lse;
            w[(t0 + p) * r + lane] = expf(mine - lse);
        }
    }
}

// counts[a] += positions whose largest gate is expert a, the first index on ties (eq. 10).  STATISTIC: the workgroup that
// adds its counts last also forms the statistic from the sums, which saves a launch; until then the four bytes of laux count
// the workgroups that have added theirs, and both start at zero.
template <int NG, bool STATISTIC>
__global__ void __launch_bounds__(kBlock) k_aux_argmax_bf16(size_t T, int d, int r, const bf16_t *__restrict__ H,
                                                            const bf16_t *__restrict__ G, unsigned long long *__restrict__ counts,
                                                            float *__restrict__ laux)
{
    __shared__ bool last;
    __shared__ float red[kWaves][kRows][NG * 16 + 1];
    __shared__ unsigned int hist[64];
    if (threadIdx.x < 64) hist[threadIdx.x] = 0;
    for (size_t t0 = (size_t)blockIdx.x * kRows; t0 < T; t0 += (size_t)gridDim.x * kRows) {
        gate_rows<NG>(t0, T, d, r, H, G, red);
        __syncthreads();
        const int row = threadIdx.x;
        if (row < kRows && t0 + row < T) {
            float best = -INFINITY;
            int arg = 0;
            for (int a = 0; a < r; ++a) {
                const float p = (red[0][row][a] + red[1][row][a]) + (red[2][row][a] + red[3][row][a]);
                if (p > best) { best = p; arg = a; }
            }
            atomicAdd(&hist[arg], 1u);
        }
        __syncthreads();
    }
    if ((int)threadIdx.x < r && hist[threadIdx.x]) {
        atomicAdd(&counts[threadIdx.x], (unsigned long long)hist[threadIdx.x]);
        if (STATISTIC) __threadfence();                   // before the workgroup counts as done
    }
    if (!STATISTIC) return;
    __syncthreads();
    if (threadIdx.x == 0)
        last = __hip_atomic_fetch_add(reinterpret_cast<unsigned *>(laux), 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
    __syncthreads();
    if (!last || threadIdx.x >= kWave) return;
    __threadfence();
    const int lane = threadIdx.x;
    const unsigned long long count = lane < r ? __hip_atomic_load(&counts[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0ull;
    const float s = balance_statistic(T, r, count, lane);
    if (lane == 0) *laux = s;
}

// dG[a, j] = sum_t dg[t, a] H[t, j] in two deterministic stages: partial sums over chunks of kGateChunk positions in turn,
// then the chunks in increasing order.  First stage: a wavefront takes a chunk, 64 columns and eight experts; it is bound by
// the chain of the chunk's positions, so the values of H are fetched a batch ahead of their use and dg lies in LDS.
// 26 us at T = 1500, d = 768, r = 5 (one thread per column without any prefetch: 230), 28 at T = 4096, d = 4096, r = 8,
// 50 at T = 16384; 28 at T = 2048, d = 1024, r = 64.  Chunks of 128 positions with 16-byte loads took 16 / 24 / 44 / 100 us
// and, whatever the batch, four times the workspace (134 MB at T = 16384, d = 4096, r = 64), and added up in another order.
constexpr int kGateBatch = 32, kGateStep = 16;
__global__ void __launch_bounds__(kWave) k_dgate_partial(size_t T, int d, int r, const bf16_t *__restrict__ H,
                                                         const float *__restrict__ dg, float *__restrict__ partial)
{
    __shared__ __attribute__((aligned(16))) float dg_s[kGateChunk][8];
    static_assert(kGateChunk % kGateBatch == 0 && kGateChunk * 8 % (16 * kWave) == 0, "whole batches in LDS");
    const int lane = threadIdx.x, a0 = (int)blockIdx.z * 8;
    const size_t t0 = (size_t)blockIdx.x * kGateChunk;
    const int count = (int)min((size_t)kGateChunk, T - t0);
    const int padded = (count + kGateBatch - 1) / kGateBatch * kGateBatch;      // positions past the last one add zeros
    constexpr int kFill = 16;                                                   // loads in flight
    for (int i0 = 0; i0 < padded * 8; i0 += kFill * kWave) {
        float v[kFill];
#pragma unroll
        for (int u = 0; u < kFill; ++u) {
            const int t = (i0 + u * kWave + lane) / 8, e = min(a0 + lane % 8, r - 1);
            v[u] = dg[(t0 + min(t, count - 1)) * r + e];
            if (t >= count) v[u] = 0.f;
        }
#pragma unroll
        for (int u = 0; u < kFill; ++u) dg_s[(i0 + u * kWave + lane) / 8][lane % 8] = v[u];
    }
    __syncthreads();
    const bf16_t *h = H + t0 * d + (size_t)blockIdx.y * kWave;
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    bf16_t next[kGateBatch];
    auto fetch = [&](int t) {
#pragma unroll
        for (int u = 0; u < kGateBatch; ++u) next[u] = ld_at(h + (size_t)min(t + u, count - 1) * d, lane * sizeof(bf16_t));
    };
    fetch(0);
    for (int t = 0; t < padded; t += kGateBatch) {
        float hv[kGateBatch];
#pragma unroll
        for (int u = 0; u < kGateBatch; ++u) hv[u] = t + u < count ? bf16_to_f32(next[u]) : 0.f;
        fetch(t + kGateBatch);
#pragma unroll
        for (int u0 = 0; u0 < kGateBatch; u0 += kGateStep) {
            f32x4_t g[kGateStep][2];
#pragma unroll
            for (int u = 0; u < kGateStep; ++u)
#pragma unroll
                for (int c = 0; c < 2; ++c) g[u][c] = *reinterpret_cast<const f32x4_t *>(&dg_s[t + u0 + u][4 * c]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < kGateStep; ++u)
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[e] += g[u][e / 4][e % 4] * hv[u0 + u];
        }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e)
        if (a0 + e < r) partial[((size_t)blockIdx.x * r + a0 + e) * d + blockIdx.y * kWave + lane] = acc[e];
}
__global__ void __launch_bounds__(kBlock) k_dgate_reduce(int chunks, size_t rd, const float *__restrict__ partial, float *__restrict__ dG)
{
    const size_t idx = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (idx >= rd) return;
    float acc = 0.f;
#pragma unroll 8
    for (int c = 0; c < chunks; ++c) acc += partial[(size_t)c * rd + idx];
    dG[idx] = acc;
}

}  // namespace

void launch_gate_bf16(const cp_head_desc &ds, const bf16_t *H, const bf16_t *G, float *logw, float *w, hipStream_t st)
{
    const size_t T = (size_t)ds.T;
    const unsigned blocks = blocks_for(T, kWaves * kGatePos);
    if (ds.r == 1) k_gate_bf16<1, 8><<<blocks, kBlock, 0, st>>>(T, ds.d, ds.r, H, G, logw, w);
    else if (ds.r == 2) k_gate_bf16<2, 8><<<blocks, kBlock, 0, st>>>(T, ds.d, ds.r, H, G, logw, w);
    else if (ds.r <= 4) k_gate_bf16<4, 6><<<blocks, kBlock, 0, st>>>(T, ds.d, ds.r, H, G, logw, w);
    else k_gate_bf16<8, 4><<<blocks, kBlock, 0, st>>>(T, ds.d, ds.r, H, G, logw, w);
}

// The statistic in the same launch: each workgroup orders its caches before it counts as done, one after the other, so for few
// workgroups only.  Whole calls, us, two launches / three: T = 300 (19 workgroups) 7.3 / 13.0, T = 4096 (256) 20.4 / 16.1, T = 16384 (512) 75 / 34.7.
// And only for calls that the host's launches bound, not the work of the counting kernel; calls after one another, by T d max(r, 8) / 2^20:
//   r = 2: T 1024 d 2048 (16) 8.6 / 10.6, T 1024 d 3072 (24) 9.7 / 10.6, T 1536 d 4096 (48) 11.6 / 10.8, T 2048 d 4096 (64) 13.1 / 11.2
//   r = 8: T 512 d 4096 (16) 11.1 / 11.2, T 1536 d 2048 (24) 9.8 / 10.5, T 1024 d 3072 (24) 10.5 / 10.5, T 2048 d 2048 (32) 10.7 / 10.5, T 2048 d 4096
//   (64) 14.3 / 12.4;  r = 16: T 1024 d 2048 (32) 9.8 / 10.6, T 512 d 3072 (24) 10.9 / 10.9, T 2048 d 2048 (64) 11.7 / 10.5, T 2048 d 4096 (128) 15.2 / 13.6
//   r = 17: T 512 d 4096 (34) 16.7 / 16.4, T 2048 d 2048 (68) 13.5 / 12.4;  r = 64: T 256 d 1024 (16) 11.5 / 11.6, T 2048 d 4096 (512) 27.6 / 26.7
constexpr unsigned kAuxAlone = 128;
constexpr size_t kAuxAloneWork = (size_t)24 << 20;
bool launch_aux_argmax_bf16(const cp_head_desc &ds, const bf16_t *H, const bf16_t *G, unsigned long long *counts, float *laux, hipStream_t st)
{
    const size_t T = (size_t)ds.T;
    // at most two workgroups per compute unit: each ends with up to r atomic additions to the same few counters
    const unsigned tiles = blocks_for(T, kRows), blocks = tiles < 512 ? tiles : 512;
    const bool whole = blocks <= kAuxAlone && T * ds.d * (ds.r > 8 ? ds.r : 8) <= kAuxAloneWork;
    auto kernel = ds.r <= 16 ? (whole ? k_aux_argmax_bf16<1, true> : k_aux_argmax_bf16<1, false>)
                             : (whole ? k_aux_argmax_bf16<4, true> : k_aux_argmax_bf16<4, false>);
    kernel<<<blocks, kBlock, 0, st>>>(T, ds.d, ds.r, H, G, counts, laux);
    return whole;
}

void launch_gate_gradient_bf16(const cp_head_desc &ds, const bf16_t *H, const float *dg, float *partial, float *dG, hipStream_t st)
{
    const unsigned chunks = (unsigned)gate_chunks((size_t)ds.T);
    const size_t rd = (size_t)ds.r * ds.d;
    k_dgate_partial<<<dim3(chunks, (unsigned)ds.d / kWave, blocks_for((size_t)ds.r, 8)), kWave, 0, st>>>((size_t)ds.T, ds.d, ds.r, H, dg,
                                                                                                        partial);
    k_dgate_reduce<<<blocks_for(rd, kBlock), kBlock, 0, st>>>((int)chunks, rd, partial, dG);
}

}  // namespace cph
