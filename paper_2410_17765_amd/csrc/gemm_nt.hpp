// bf16 "NT" matrix-core GEMM main loop for gfx950 with pluggable epilogues.
//
//   acc[m, n] = sum_k A[m, k] * B[n, k]        A[M, lda], B[N, ldb] bf16, both K-contiguous
//
// Every large contraction of the CP head (y = W h, z = U y, and the five products of the
// backward pass) is brought into this one form, if necessary by transposing an operand first,
// so that a single tuned main loop serves them all; what differs is the epilogue that consumes
// the fp32 accumulators (plain store, running log-sum-exp statistics, softmax gradient, ...).
//
// Tiling: a workgroup owns a BM x BN tile of the output and walks K in steps of BK = 64.
// WM x WN wavefronts split the tile; each wavefront issues 16x16x32 bf16 MFMAs on a
// (BM/WM) x (BN/WN) sub-tile whose fp32 accumulators stay in registers for the whole K loop.
// Operand tiles are fetched with 16-byte buffer loads (rows beyond M or N read as zero through
// the buffer descriptor's range check), staged through double-buffered LDS in an XOR-swizzled
// layout so that the 16-byte fragment reads of a wavefront are free of bank conflicts.
//
// K must be a multiple of 64; M and N are arbitrary.
//
// Either operand may instead be "K-major" (the contraction index is the slow one: A[K, lda] with the M output rows
// along its columns, likewise B[K, ldb]): the products of the backward pass that contract over rows (dU = dz^T Y,
// dW = dY^T H) or against a weight matrix stored the other way round (dY = dz U, dH = dY W) then need no
// transposed copy of anything.  A K-major tile is 64 k-rows of 256 columns; it is laid out in LDS so that gfx950's
// transposing LDS read (ds_read_b64_tr_b16: inside 16 lanes, 4 k-rows x 16 columns in, 4 k-values of one column
// per lane out) delivers MFMA operand fragments directly.  With both operands K-major K is arbitrary (rows past
// its end read as zero); otherwise K must still be a multiple of 64.
#pragma once

#include "cp_internal.hpp"
#include "tile_walk.hpp"

namespace cph {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4_t lds_s16x4_t;

struct GemmOperands {
    const bf16_t *A;   // [M, lda]
    const bf16_t *B;   // [N, ldb]
    long lda, ldb;     // elements
    int M, N, K;       // K % 64 == 0 unless both operands are K-major
    int ka_rows, kb_rows;   // K-major operands: rows that exist (<= K; the rest of K reads as zero); not for a blocked one
    int ka_tile;       // K-major A stored block by block: the K-tile (of 64 of its rows) that the contraction starts with
    int tiles_m, tiles_n;
    int gm;            // tile rows per group of the workgroup -> tile walk
};

// LDS layout of a K-major tile (64 k-rows x 256 columns).  Four consecutive k-rows (a quad) are interleaved in
// units of 32 bytes: the 16 columns [16 p, 16 p + 16) of the quad's rows t = 0..3 sit at p * 128 + t * 32, so the
// 4 x 32 bytes that 16 lanes hand to one transposing read are one 128-byte span; quads are 2 KB apart and every
// pair of quads is followed by 128 bytes of padding, which puts the quads of k-groups g and g + 1 (8 k-rows = two
// quads apart) into the two halves of the 256-byte bank cycle: a wavefront's read is free of bank conflicts.
// A direct global->LDS load instruction (64 lanes x 16 bytes = 1 KB, consecutive in LDS) fills half a quad: lane i
// fetches 8 columns [16 (8 e + i / 8) + 8 (i % 2), +8) of k-row (i % 8) / 2, i.e. 256 contiguous bytes of each of
// four rows; the four wavefronts of a pass fill two quads, and a pass advances by 4224 bytes.
constexpr int kKmPassBytes = 2 * 2048 + 128;
constexpr int kKmTileBytes = 8 * kKmPassBytes;

template <int BM_, int BN_, int WM_, int WN_, bool AKM_ = false, bool BKM_ = false, bool ABL_ = false, bool ROWS_IN_LANE_ = false>
struct TileCfg {
    static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, BK = 64;
    static constexpr bool AKM = AKM_, BKM = BKM_;     // operand is K-major
    // A is stored block by block, [rows/256][columns/64][256][64] (blocked64_index): its rows are the output's rows, or, if it
    // is K-major as well, the contraction's
    static constexpr bool ABL = ABL_;
    // which four neighbouring elements a lane holds of a 16x16 block of the result: one row's columns, or one column's rows
    static constexpr bool ROWS_IN_LANE = ROWS_IN_LANE_;
    static constexpr int THREADS = WM * WN * kWave;
    static constexpr int WTM = BM / WM, WTN = BN / WN;       // wavefront sub-tile
    static constexpr int TM16 = WTM / 16, TN16 = WTN / 16;   // 16x16 MFMA blocks per wavefront
    static constexpr int ROWS_PER_PASS = THREADS / 8;        // a pass moves one 16-byte chunk per thread
    static constexpr int A_PASSES = BM / ROWS_PER_PASS, B_PASSES = BN / ROWS_PER_PASS;
    static constexpr int A_BYTES = AKM_ ? kKmTileBytes : BM * BK * 2, B_BYTES = BKM_ ? kKmTileBytes : BN * BK * 2;
    static_assert(!(AKM_ || BKM_) || WM_ * WN_ == 4, "K-major operands: four wavefronts");
    static_assert((!AKM_ || BM_ == 256) && (!BKM_ || BN_ == 256), "a K-major tile has 256 columns");
    static constexpr int STAGE_BYTES = A_BYTES + B_BYTES;
    static constexpr int LDS_BYTES = 2 * STAGE_BYTES;
    static_assert(BM % (WM * 64) == 0 && BN % (WN * 32) == 0, "wave tile must be a multiple of 64 rows x 32 columns");
    static_assert(BM % ROWS_PER_PASS == 0 && BN % ROWS_PER_PASS == 0, "tile rows must divide into load passes");
};

// Raw buffer descriptor for `bytes` bytes at `base` (no stride, range-checked) as four scalar words, and a direct global->LDS load
// of 16 bytes per lane spelled out.  Fragments of K-major operands come from gfx950's transposing LDS read, and before
// every such read the compiler waits for all outstanding loads once it knows that loads into LDS are in flight (it cannot tell
// that they go to the other stage), which serialises the whole pipeline (measured: 3-5 times slower).  Loads
// issued this way are invisible to that bookkeeping; the main loop's own explicit waits (before the barrier that
// publishes a stage) are what orders them.  The kernels without a K-major operand issue theirs the same way: the
// builtin's address arithmetic between the products cost the kept-logits product 2 % (d = 2048: 7.07 -> 6.94 ms).
typedef int i32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ i32x4_t make_rsrc_words(const void *base, unsigned bytes)
{
    const unsigned long long p = reinterpret_cast<unsigned long long>(base);
    i32x4_t r;
    r[0] = __builtin_amdgcn_readfirstlane((int)(p & 0xFFFFFFFFull));
    r[1] = __builtin_amdgcn_readfirstlane((int)((p >> 32) & 0xFFFFull));
    r[2] = __builtin_amdgcn_readfirstlane((int)bytes);
    r[3] = 0x00020000;
    return r;
}
// lds_addr: LDS byte address of the wavefront's 1 KB destination (uniform); voff: per-lane byte offset (range-checked
// against the descriptor); soff: uniform byte offset (not range-checked)
__device__ __forceinline__ void load_lds_16_spelled_out(i32x4_t rsrc, unsigned lds_addr, unsigned voff, int soff)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :
                 : "s"(lds_addr), "v"(voff), "s"(rsrc), "s"(soff)
                 : "memory");
}

// Tile rows per group of that walk.  8 x 4 tiles in flight per XCD suit the vocabulary-wide products (125 or
// more tile columns; 16 rows per group cost them 10-25 %); the products with a d-wide output (16 tile columns)
// and y = W h run 2-5 % faster with 4 x 8, which re-reads their large A operand half as often (1, 2 and 8 rows per
// group cost dY 1.7-2.4 %, 2 and 8 cost dU 1.2-1.8 %).
constexpr int kGroupRowsWide = 8, kGroupRowsNarrow = 4;

// The main loop, with direct global->LDS loads (no staging registers, no LDS write instructions) and
// 16x16x32 MFMAs.  Each wavefront load instruction moves 64 x 16 bytes = 8 operand rows of 128 bytes into
// 1 KB of consecutive LDS; the XOR swizzle is realised by permuting which 16-byte chunk of its row each
// lane fetches.
// Why 16x16x32: on random bf16 data the matrix cores of this part are limited by power, not by issue rate,
// and that instruction delivers about 14 % more FLOP/s there than the 32x32x16 one (2.18 against 1.92
// PFLOP/s in a loop of nothing but MFMAs with this register tiling; the loop below gained 3-5 %).
// A K-step of 64 is two K-blocks of 32; a K-block is two phases, one per half of the wavefront's rows:
//   phase 0   rows half 0, k 0..31    + reads: A half 1 (k 0..31), B first half (k 32..63)   + 2nd half of the loads of tile kt+1
//   phase 1   rows half 1, k 0..31    + reads: B second half (k 32..63), A half 0 (k 32..63)
//   phase 2   rows half 0, k 32..63   + reads: A half 1 (k 32..63)
//   wait for tile kt+1, workgroup barrier
//   phase 3   rows half 1, k 32..63   + reads from tile kt+1: A half 0, B (k 0..31)          + 1st half of the loads of tile kt+2
// Memory instructions are issued one at a time between MFMAs (the order is pinned with scheduling
// barriers): a wavefront issues in order, so a cluster of loads would hold back its MFMAs.
// On return acc[i][j] holds the 16x16 block (i, j) of the wavefront's sub-tile.  The instruction gives lane l the
// elements 4*(l/16) + v, v = 0..3, of its first operand's rows, all at its second operand's row l%16.  With B as the first
// operand (the default) those are four columns of row l%16 of the block, so that a lane's results are consecutive in memory:
// the epilogues store straight from the registers, and a row's maximum and sum are 32 steps inside a lane and two
// across lanes.  With A first (ROWS_IN_LANE) they are four rows of column l%16, which is what the mixtures over the expert
// rows of a token need.
template <class Cfg>
__device__ __forceinline__ void gemm_nt_mainloop_direct(const GemmOperands &g, int tm, int tn, char *smem,
                                                          f32x4_t (&acc)[Cfg::TM16][Cfg::TN16])
{
    constexpr int BM = Cfg::BM, BN = Cfg::BN, BK = Cfg::BK, TM = Cfg::TM16, TN = Cfg::TN16;
    constexpr int HA = TM / 2, HB = TN / 2;                  // A fragments per row half, B fragments per read half
    constexpr int NLOAD = Cfg::A_PASSES + Cfg::B_PASSES;
    constexpr int NM = HA * TN;                              // MFMAs per phase
    // loads of a tile per phase, from the phase after the barrier that frees its stage: phases 3, 0, 1, 2.
    // Measured on the three large product shapes: 8/8/0/0 and 10/6/0/0 lead (the latter by about 1 %),
    // 12/4 loses 3-5 %, 16/0 and any load in phases 1 or 2 (less time to land) lose 10-30 %.
    constexpr int L3 = NLOAD * 5 / 8, L0 = NLOAD - L3, L1 = 0, L2 = 0;
    constexpr int NEARLY = L3;
    // The fragment reads of phase 2 are the last ones before the barrier, whose fence waits for every LDS read of the
    // wavefront: spread over the whole phase, the last of them was issued one matrix instruction before that wait and
    // the matrix pipe could run dry for an LDS latency per K-step.  They go into the first half of the phase (worth
    // 0.2-0.4 % on the three large shapes).
    constexpr int P2_SPAN = NM / 2;
    static_assert(BK == 64 && TM % 2 == 0 && TN % 2 == 0 && TN + HA <= NM && L2 >= 0, "schedule slots");
    typedef __attribute__((address_space(3))) void lds_void;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm0 = (wave / Cfg::WN) * Cfg::WTM;
    const int wn0 = (wave % Cfg::WN) * Cfg::WTN;

    const int m0 = tm * BM, n0 = tn * BN;
    const int rows_a = min(BM, g.M - m0), rows_b = min(BN, g.N - n0);
    // K-contiguous operand: one descriptor over the tile's rows, the K-step is a scalar byte offset.
    // K-major operand: a descriptor per K-step over its 64 k-rows from the tile's first column on (the whole
    // operand may exceed the 4 GiB a descriptor can address); k-rows past the operand's end are out of range and
    // read as zero, columns past M or N read whatever follows in the row and only reach accumulators that are
    // never stored.
    // bytes between two rows of the tile: the leading dimension, or 128 for a blocked operand
    const unsigned rsa = Cfg::ABL ? 128u : (unsigned)g.lda * 2u, rsb = (unsigned)g.ldb * 2u;
    // (a blocked operand's descriptor spans the whole panel of its tile row: all 256 rows of every block exist)
    const unsigned span_a = Cfg::ABL ? (unsigned)((size_t)BM * g.K * 2) : (unsigned)((size_t)rows_a * g.lda * 2);
    const unsigned span_b = (unsigned)((size_t)rows_b * g.ldb * 2);
    // A K-major operand's descriptor is kept for the K-tile whose loads are being issued and moved on by one tile
    // (64 k-rows) at a time: a 64-bit add on the base and a choice among three sizes (a full tile, the operand's
    // last, partial one, nothing past its end).  Rebuilding it from the tile index cost a dozen scalar instructions
    // in one place, four times per K-step, which held the matrix instructions up by several percent.
    struct KmWalk {
        i32x4_t d;          // descriptor of tile `tile`
        int tile;
        unsigned step;      // bytes from one K-tile to the next
        int full_tiles;     // tiles with all 64 rows
        unsigned full, tail;
        unsigned step_row;  // blocked: bytes from a row of blocks' last K-tile to the next one's first
    };
    auto km_start = [&](const bf16_t *base, long ld, int col0, int krows) {
        KmWalk w;
        w.tile = 0;
        w.step = (unsigned)(BK * ld * 2);
        w.full_tiles = krows / BK;
        w.full = (unsigned)(((long)BK * ld - col0) * 2);
        const int rest = krows % BK;
        w.tail = rest > 0 ? (unsigned)(((long)rest * ld - col0) * 2) : 0u;
        w.d = make_rsrc_words(base + col0, w.full_tiles > 0 ? w.full : w.tail);
        return w;
    };
    // A blocked operand: a row of blocks (256 k-rows, all columns) holds four K-tiles, 64 rows of every block each; the
    // descriptor spans the row of blocks, and the producer of the operand has zeroed the rows up to the contraction's end.
    auto km_start_blocked = [&](const bf16_t *base, long ld, int tile) {
        KmWalk w;
        w.tile = tile;
        w.step = BK * 128;
        w.step_row = (unsigned)(ld * 512) - 3 * BK * 128;
        w.full_tiles = 0x7FFFFFFF;
        w.full = w.tail = (unsigned)(ld * 512);
        w.d = make_rsrc_words(base + (size_t)(tile >> 2) * 256 * ld + (size_t)(tile & 3) * BK * 64, w.full);
        return w;
    };
    auto km_advance_blocked = [&](KmWalk &w) {
        ++w.tile;
        const unsigned long long at = (((unsigned long long)(unsigned)w.d[1] << 32) | (unsigned)w.d[0]) + ((w.tile & 3) ? w.step : w.step_row);
        w.d[0] = (int)(unsigned)at;
        w.d[1] = (int)(unsigned)(at >> 32);
    };
    auto km_advance = [&](KmWalk &w) {
        const unsigned long long at = (((unsigned long long)(unsigned)w.d[1] << 32) | (unsigned)w.d[0]) + w.step;
        ++w.tile;
        w.d[0] = (int)(unsigned)at;
        w.d[1] = (int)(unsigned)(at >> 32);
        w.d[2] = (int)(w.tile < w.full_tiles ? w.full : (w.tile == w.full_tiles ? w.tail : 0u));
    };
    constexpr bool kBlockedKm = Cfg::AKM && Cfg::ABL;
    KmWalk walk_a = kBlockedKm ? km_start_blocked(g.A, g.lda, g.ka_tile) : km_start(g.A, g.lda, m0, g.ka_rows);
    KmWalk walk_b = km_start(g.B, g.ldb, n0, g.kb_rows);
    auto advance_a = [&]() { if (kBlockedKm) km_advance_blocked(walk_a); else km_advance(walk_a); };
    const i32x4_t wa = make_rsrc_words(g.A + (size_t)m0 * g.lda, span_a);
    const i32x4_t wb = make_rsrc_words(g.B + (size_t)n0 * g.ldb, span_b);
    const unsigned lds_smem = __builtin_amdgcn_readfirstlane((unsigned)reinterpret_cast<unsigned long long>((lds_void *)smem));

    const int lrow = tid >> 3, pchunk = tid & 7;
    const int gchunk = pchunk ^ ((lrow >> 1) & 7);
    // K-major: k-row of the pass and first column that this thread fetches (see the layout above)
    const int km_row = (wave >> 1) * 4 + ((lane & 7) >> 1);
    const int km_col = ((wave & 1) * 8 + (lane >> 3)) * 16 + (lane & 1) * 8;
    // (blocked: columns past the last block read the last one again, they only reach accumulators that are never stored)
    const unsigned voff_a = kBlockedKm ? (unsigned)min((m0 + km_col) >> 6, (int)(g.lda >> 6) - 1) * 32768u + (unsigned)km_row * 128u + (km_col & 63) * 2u
                          : Cfg::AKM ? (unsigned)km_row * (unsigned)g.lda * 2u + km_col * 2u
                                     : (unsigned)lrow * rsa + gchunk * 16u;
    const unsigned voff_b = Cfg::BKM ? (unsigned)km_row * (unsigned)g.ldb * 2u + km_col * 2u
                                     : (unsigned)lrow * rsb + gchunk * 16u;
    const unsigned pass_a = kBlockedKm ? 8u * 128u : (unsigned)(Cfg::AKM ? 8 : Cfg::ROWS_PER_PASS) * rsa;
    const unsigned pass_b = (unsigned)(Cfg::BKM ? 8 : Cfg::ROWS_PER_PASS) * rsb;
    constexpr int lds_pass_a = Cfg::AKM ? kKmPassBytes : Cfg::ROWS_PER_PASS * 128;
    constexpr int lds_pass_b = Cfg::BKM ? kKmPassBytes : Cfg::ROWS_PER_PASS * 128;
    const int lds_wave = wave * 8 * 128;

    // fragment reads: lane l reads row l%16 of a 16-row block, 16-byte k-chunk 4*kb + l/16 of its 128-byte row
    const int frag_row = lane & 15, frag_q = lane >> 4, frag_sw = (lane >> 1) & 7;
    // K-major fragments: lane (g, s) = (lane / 16, lane % 16) of a transposing read addresses 8 bytes of k-row
    // s / 4 of a quad; k-group g is two quads (and one padding) further on; the 16-column block is a constant
    const int km_lane = frag_q * (2 * 2048 + 128) + frag_row * 8;
    const int lds_ra = Cfg::AKM ? km_lane + (wm0 / 16) * 128 : (wm0 + frag_row) * 128;
    const int lds_rb = Cfg::A_BYTES + (Cfg::BKM ? km_lane + (wn0 / 16) * 128 : (wn0 + frag_row) * 128);
    int coff[2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) coff[kb] = ((kb * 4 + frag_q) ^ frag_sw) << 4;

    bf16x8_t fa[2][HA], fb[2][TN];

    // Everything that the descriptor's range check must see is in the vector offset (the scalar offset is added to
    // the address but not checked): the pass for both layouts.  The K-step is the scalar offset of a K-contiguous
    // operand and part of the descriptor's base for a K-major one.
    auto load_one = [&](int kt, int stage, int q) {
        // the K-step: 128 bytes along the row, or one block of BM rows x 128 bytes of a blocked operand
        const int soff = q < Cfg::A_PASSES ? kt * (Cfg::ABL ? BM * 128 : BK * 2) : kt * (BK * 2);
        const unsigned lbase = lds_smem + stage * Cfg::STAGE_BYTES + lds_wave;
        if (q < Cfg::A_PASSES) {
            if (Cfg::AKM)
                load_lds_16_spelled_out(walk_a.d, lbase + q * lds_pass_a, voff_a + q * pass_a, 0);       // tile kt == walk_a.tile
            else
                load_lds_16_spelled_out(wa, lbase + q * lds_pass_a, voff_a + q * pass_a, soff);
        } else {
            const int qb = q - Cfg::A_PASSES;
            if (Cfg::BKM)
                load_lds_16_spelled_out(walk_b.d, lbase + Cfg::A_BYTES + qb * lds_pass_b, voff_b + qb * pass_b, 0);
            else
                load_lds_16_spelled_out(wb, lbase + Cfg::A_BYTES + qb * lds_pass_b, voff_b + qb * pass_b, soff);
        }
    };
    // a fragment of a K-major tile: 16-column block `blk` of the wavefront, k-block kb: two transposing reads
    // (k-rows 0..3 and 4..7 of the lane's group of 8)
    auto read_km = [&](const char *st, int lane_base, int kb, int blk) {
        const char *p = st + lane_base + kb * (4 * kKmPassBytes) + blk * 128;
#if defined(__HIP_DEVICE_COMPILE__)
        const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t *)(p));
        const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t *)(p + 2048));
#else   // the host pass only parses this function
        const s16x4_t lo = *reinterpret_cast<const s16x4_t *>(p), hi = lo;
#endif
        return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    auto read_a = [&](const char *st, int kb, int buf, int half, int q) {
        if (Cfg::AKM) fa[buf][q] = read_km(st, lds_ra, kb, half * HA + q);
        else fa[buf][q] = *reinterpret_cast<const bf16x8_t *>(st + lds_ra + (half * HA + q) * 16 * 128 + coff[kb]);
    };
    auto read_b = [&](const char *st, int kb, int buf, int q) {
        if (Cfg::BKM) fb[buf][q] = read_km(st, lds_rb, kb, q);
        else fb[buf][q] = *reinterpret_cast<const bf16x8_t *>(st + lds_rb + q * 16 * 128 + coff[kb]);
    };
    auto mfma_one = [&](int abuf, int bbuf, int half, int idx) {
        // The columns are walked there and back: every product shares a fragment with the one before it, which on these
        // power-limited matrix cores is worth 0.4-0.5 % of every large product.
        const int i = idx / TN, j = (i & 1) ? TN - 1 - idx % TN : idx % TN;
        // The instruction is spelled out with the accumulator tied to itself in the accumulation registers and the
        // fragments in vector registers.  Left to itself the register allocator rotates accumulators through copies between
        // the two register files: several hundred per K-step where fragments are assembled from two 64-bit reads (K-major
        // operands) or the columns are walked in another order (z at d = 4096 93.5 -> 106 ms), and dozens in the 64-row tile.
        // The compiler still inserts the waits for the fragments' LDS reads (it sees the operands); what it cannot see
        // is that the instruction is a matrix instruction: uses of one accumulator are TM TN instructions apart here, 64 in
        // the 256-row tile and 16 in the 64-row one, and the wait states before the accumulators are read back are added
        // after the loop (without them the epilogue read accumulators that lacked the last K-block's contribution).
        // This one takes four passes (16 cycles); even the result of one of eight may be read after 11 other instructions.
        static_assert(TM * TN >= 12, "uses of an accumulator far enough apart for instructions without wait states");
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0"
                     : "+a"(acc[half * HA + i][j])
                     : "v"(Cfg::ROWS_IN_LANE ? fa[abuf][i] : fb[bbuf][j]), "v"(Cfg::ROWS_IN_LANE ? fb[bbuf][j] : fa[abuf][i]));
    };
    // the reads of the four phases, in the order the MFMAs that follow need them
    auto reads0 = [&](const char *st, const char *, int q) {       // A half 1 of k-block 0, then B first half of k-block 1
        if (q < HA) read_a(st, 0, 1, 1, q); else read_b(st, 1, 1, q - HA);
    };
    auto reads1 = [&](const char *st, const char *, int q) {       // B second half of k-block 1, then A half 0 of k-block 1
        if (q < HB) read_b(st, 1, 1, HB + q); else read_a(st, 1, 0, 0, q - HB);
    };
    auto reads2 = [&](const char *st, const char *, int q) { read_a(st, 1, 1, 1, q); };   // A half 1 of k-block 1
    auto reads3 = [&](const char *, const char *nx, int q) {       // next tile: A0, all of B, the rest of A half 0
        if (q == 0) read_a(nx, 0, 0, 0, 0);
        else if (q <= TN) read_b(nx, 0, 0, q - 1);
        else read_a(nx, 0, 0, 0, q - TN);
    };
#define CPH_PIN() __builtin_amdgcn_sched_barrier(0)
#define CPH_PHASE16(ABUF, BBUF, HALF, READS, NREAD, READ_SPAN, DO_LOAD, LOAD_KT, LOAD_STAGE, LOAD_Q0, LOAD_CNT) \
    _Pragma("unroll") for (int m = 0; m < NM; ++m) {                                               \
        mfma_one(ABUF, BBUF, HALF, m);                                                             \
        CPH_PIN();                                                                                 \
        if ((DO_LOAD) && (LOAD_CNT) > 0) {                                                         \
            _Pragma("unroll") for (int q = 0; q < (LOAD_CNT); ++q)                                 \
                if ((q * NM) / ((LOAD_CNT) > 0 ? (LOAD_CNT) : 1) == m) { load_one(LOAD_KT, LOAD_STAGE, (LOAD_Q0) + q); CPH_PIN(); } \
        }                                                                                          \
        _Pragma("unroll") for (int q = 0; q < (NREAD); ++q)                                        \
            if (((q + 1) * (READ_SPAN)) / (NREAD) - 1 == m) { READS(st, nx, q); CPH_PIN(); }       \
    }

#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[i][j][v] = 0.f;

    // No load is ever issued for a tile past the end of K: a late arrival would land in LDS while the
    // epilogue is using it.  The last two K-steps are therefore peeled off with their loads removed.
    const int KT = (g.K + BK - 1) / BK;
#pragma unroll
    for (int q = 0; q < NLOAD; ++q) load_one(0, 0, q);
    if (KT > 1) {
        if (Cfg::AKM) advance_a();
        if (Cfg::BKM) km_advance(walk_b);
#pragma unroll
        for (int q = 0; q < NEARLY; ++q) load_one(1, 1, q);
        __builtin_amdgcn_s_waitcnt(0x0F70 | (NEARLY & 15) | ((NEARLY >> 4) << 14));   // vmcnt(NEARLY): tile 0 has landed
    } else {
        __builtin_amdgcn_s_waitcnt(0x0F70);
    }
    __syncthreads();
    {
        const char *st = smem, *nx = smem;
        (void)st;
#pragma unroll
        for (int q = 0; q < TN + HA; ++q) reads3(st, nx, q);
    }

#define CPH_K_STEP_DIRECT16(KT_, LOAD_NEXT, LOAD_AFTER)                                            \
    {                                                                                              \
        const int cur = (KT_) & 1;                                                                 \
        const char *st = smem + cur * Cfg::STAGE_BYTES;                                            \
        const char *nx = smem + (cur ^ 1) * Cfg::STAGE_BYTES;                                      \
        CPH_PHASE16(0, 0, 0, reads0, HA + HB, NM, LOAD_NEXT, (KT_) + 1, cur ^ 1, L3, L0)           \
        CPH_PHASE16(1, 0, 1, reads1, HB + HA, NM, LOAD_NEXT, (KT_) + 1, cur ^ 1, L3 + L0, L1)      \
        CPH_PHASE16(0, 1, 0, reads2, HA, P2_SPAN, LOAD_NEXT, (KT_) + 1, cur ^ 1, L3 + L0 + L1, L2) \
        __builtin_amdgcn_s_waitcnt(0x0F70); /* vmcnt(0): tile kt+1 is complete in the other stage */ \
        __syncthreads();                                                                           \
        if (LOAD_AFTER) { /* the loads from here on are tile kt+2's */                             \
            if (Cfg::AKM) advance_a();                                                             \
            if (Cfg::BKM) km_advance(walk_b);                                                      \
        }                                                                                          \
        CPH_PHASE16(1, 1, 1, reads3, TN + HA, NM, LOAD_AFTER, (KT_) + 2, cur, 0, NEARLY)           \
    }
    int kt = 0;
    for (; kt < KT - 2; ++kt) CPH_K_STEP_DIRECT16(kt, true, true)
    if (kt == KT - 2) {
        CPH_K_STEP_DIRECT16(kt, true, false)
        ++kt;
    }
    CPH_K_STEP_DIRECT16(kt, false, false)
    // The last matrix instructions above must have written their accumulators before anything reads them, and the
    // compiler does not know that they are matrix instructions: wait out their latency here, and pass every
    // accumulator through an (empty) volatile statement, which the compiler keeps behind that wait and ahead of
    // every later use of the accumulator.
    asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) asm volatile("" : "+a"(acc[i][j]));
#undef CPH_K_STEP_DIRECT16
#undef CPH_PHASE16
#undef CPH_PIN
}

// Generic kernel: main loop + epilogue functor.  Epi::run receives the accumulators of one wavefront
// together with the global row/column of its sub-tile's origin.
// One workgroup per output tile.  (A persistent variant, one workgroup per compute unit walking a fixed share
// of the tiles, was measured twice: it is no faster in isolation and slower inside the step, where a freshly
// dispatched workgroup goes to whichever compute unit is free first.)
// An epilogue that needs per-row values from global memory fetches them for the whole tile with one coalesced load
// at its start and parks them in LDS.  (Loaded where they are used they are a chain of exposed cache misses per
// tile while the matrix cores idle; requested before the main loop they cost the main loop 9 %: the registers
// they occupy across it change its schedule.)
// A side job rides along in the same launch: its `blocks` workgroups (a multiple of 8, so that the tile walk's
// view of the XCDs stays aligned) come first in the grid, run `run(job, smem)` and leave; small work that the
// launch does not depend on saves a launch of its own that way.
struct NoSideJob {
    static constexpr bool kActive = false;
    int blocks;
    __device__ void run(int, char *) const {}
};
// row / column of accumulator element v of block (i, j) for lane l, relative to the sub-tile origin
__device__ __forceinline__ int acc_row(int i, int lane) { return i * 16 + (lane & 15); }
__device__ __forceinline__ int acc_col(int j, int v, int lane) { return j * 16 + 4 * (lane >> 4) + v; }
// the column for ROWS_IN_LANE
__device__ __forceinline__ int acc_col_of_lane(int j, int lane) { return j * 16 + (lane & 15); }

// Epilogues whose result is a plain function of the sum over K (kSplittable) may have the launch's last round split along
// K (split_plan): put(row, col, values) stores four consecutive columns.
template <class Epi, class = void> struct IsSplittable { static constexpr bool value = false; };
template <class Epi> struct IsSplittable<Epi, decltype((void)Epi::kSplittable)> { static constexpr bool value = true; };

// The accumulators of a tile as they lie in the registers: element (i, j) of thread `tid` is one 16-byte piece.
template <class Cfg>
__device__ __forceinline__ size_t partial_index(int item, int i, int j, int tid)
{
    return (((size_t)item * Cfg::TM16 + i) * Cfg::TN16 + j) * Cfg::THREADS + tid;
}

template <class Cfg, class Epi, class Side>
__global__ void __launch_bounds__(Cfg::THREADS) k_gemm_nt(GemmOperands g, Epi epi, Side side)
{
    __shared__ __attribute__((aligned(16))) char smem[Cfg::LDS_BYTES];
    int bid = blockIdx.x;
    if (Side::kActive) {
        if (bid < side.blocks) {
            side.run(bid, smem);
            return;
        }
        bid -= side.blocks;
    }
    int tm, tn;
    if (!tile_of_block(bid, g.tiles_m, g.tiles_n, g.gm, tm, tn)) return;
    f32x4_t acc[Cfg::TM16][Cfg::TN16];
    gemm_nt_mainloop_direct<Cfg>(g, tm, tn, smem, acc);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int row0 = tm * Cfg::BM + (wave / Cfg::WN) * Cfg::WTM;
    const int col0 = tn * Cfg::BN + (wave % Cfg::WN) * Cfg::WTN;
    epi.template run<Cfg>(acc, row0, col0, lane, wave, tn, smem);
}

// The same for a launch whose last round is split.  A kernel of its own: with the choice inside it, k_gemm_nt took 1.3 to
// 2.2 us longer also where nothing is split (EpiStoreF32, 300 x 7000 x 512: 21.0 -> 23.2 us), a tenth of a small call.
template <class Cfg, class Epi>
__global__ void __launch_bounds__(Cfg::THREADS) k_gemm_nt_split(GemmOperands g, Epi epi, SplitPlan split, f32x4_t *partial)
{
    __shared__ __attribute__((aligned(16))) char smem[Cfg::LDS_BYTES];
    int bid = blockIdx.x, item = -1;
    if (bid >= split.first) {
        int part, k0, k1;
        item = bid - split.first;
        split_item(split, item, (g.K + Cfg::BK - 1) / Cfg::BK, bid, part, k0, k1);
        // the operands from K-step k0 on
        if (Cfg::AKM && Cfg::ABL) g.ka_tile += k0;
        else g.A += Cfg::AKM ? (size_t)k0 * Cfg::BK * g.lda : (size_t)k0 * (Cfg::ABL ? Cfg::BM * Cfg::BK : Cfg::BK);
        g.B += Cfg::BKM ? (size_t)k0 * Cfg::BK * g.ldb : (size_t)k0 * Cfg::BK;
        g.ka_rows = max(g.ka_rows - k0 * Cfg::BK, 0);
        g.kb_rows = max(g.kb_rows - k0 * Cfg::BK, 0);
        g.K = min(g.K, k1 * Cfg::BK) - k0 * Cfg::BK;
    }
    int tm, tn;
    if (!tile_of_block(bid, g.tiles_m, g.tiles_n, g.gm, tm, tn)) return;
    f32x4_t acc[Cfg::TM16][Cfg::TN16];
    gemm_nt_mainloop_direct<Cfg>(g, tm, tn, smem, acc);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int row0 = tm * Cfg::BM + (wave / Cfg::WN) * Cfg::WTM;
    const int col0 = tn * Cfg::BN + (wave % Cfg::WN) * Cfg::WTN;
    if (item >= 0) {
#pragma unroll
        for (int i = 0; i < Cfg::TM16; ++i)
            if (row0 + i * 16 < g.M) {                  // blocks past the last row are not read back either
#pragma unroll
                for (int j = 0; j < Cfg::TN16; ++j) partial[partial_index<Cfg>(item, i, j, threadIdx.x)] = acc[i][j];
            }
        return;
    }
    epi.template run<Cfg>(acc, row0, col0, lane, wave, tn, smem);
}

// Second stage of a split round: one workgroup per tile and 16-row block of its wavefronts; the parts in increasing order.
template <class Cfg, class Epi>
__global__ void __launch_bounds__(Cfg::THREADS) k_gemm_add_parts(GemmOperands g, Epi epi, SplitPlan split, const f32x4_t *__restrict__ partial)
{
    const int slot = blockIdx.x / Cfg::TM16, i = blockIdx.x % Cfg::TM16;
    int tm, tn;
    if (!tile_of_block(split.first + slot, g.tiles_m, g.tiles_n, g.gm, tm, tn)) return;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    static_assert(!Cfg::ROWS_IN_LANE, "four columns per lane");
    const int row = tm * Cfg::BM + (wave / Cfg::WN) * Cfg::WTM + acc_row(i, lane);
    const int col = tn * Cfg::BN + (wave % Cfg::WN) * Cfg::WTN + acc_col(0, 0, lane);
    if (row - (lane & 15) >= g.M) return;
    f32x4_t sum[Cfg::TN16];
#pragma unroll
    for (int j = 0; j < Cfg::TN16; ++j) sum[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
    for (int p = 0; p < split.parts; ++p)
#pragma unroll
        for (int j = 0; j < Cfg::TN16; ++j) sum[j] += partial[partial_index<Cfg>(p * split.tail + slot, i, j, threadIdx.x)];
#pragma unroll
    for (int j = 0; j < Cfg::TN16; ++j)
        if (row < g.M && col + j * 16 < g.N) epi.put(row, col + j * 16, sum[j]);
}

// Scratch for the partial tiles of a split round; none: launches are never split.
struct SplitScratch {
    void *p = nullptr;
    size_t bytes = 0;
};
template <class Cfg>
inline SplitPlan plan_split(int M, int N, int K, int gm, size_t scratch_bytes)
{
    constexpr size_t kItemBytes = (size_t)Cfg::BM * Cfg::BN * 4;
    static_assert(Cfg::BM == 256 && Cfg::BN == 256, "one workgroup per compute unit; the plan's times are this tile's");
    const int grid = gemm_grid((M + Cfg::BM - 1) / Cfg::BM, (N + Cfg::BN - 1) / Cfg::BN, gm);
    const size_t items = scratch_bytes / kItemBytes;
    return split_plan(grid, 256, (K + Cfg::BK - 1) / Cfg::BK, items < kMaxSplitItems ? (int)items : kMaxSplitItems);
}
// bytes of scratch with which the launch's last round is split as it is best; at most 128 MiB
template <class Cfg>
inline size_t split_scratch_bytes(size_t M, size_t N, size_t K, int gm)
{
    if (!M || !N || !K) return 0;
    const SplitPlan p = plan_split<Cfg>((int)M, (int)N, (int)K, gm, ~(size_t)0);
    return p.parts > 1 ? (size_t)p.parts * p.tail * Cfg::BM * Cfg::BN * 4 : 0;
}

template <class Cfg, class Epi, class Side = NoSideJob>
inline void launch_gemm_nt(const char *name, const bf16_t *A, long lda, int M, const bf16_t *B, long ldb, int N, int K,
                           const Epi &epi, hipStream_t st, int gm = kGroupRowsWide, const Side &side = Side{0},
                           int ka_rows = -1, int kb_rows = -1, const SplitScratch &scratch = SplitScratch())
{
    ProfileScope prof(name, 2.0 * (double)M * (double)N * (double)K, st);
    GemmOperands g;
    g.A = A; g.B = B; g.lda = lda; g.ldb = ldb; g.M = M; g.N = N; g.K = K;
    g.ka_rows = ka_rows < 0 ? K : ka_rows; g.kb_rows = kb_rows < 0 ? K : kb_rows; g.ka_tile = 0;
    g.tiles_m = (M + Cfg::BM - 1) / Cfg::BM;
    g.tiles_n = (N + Cfg::BN - 1) / Cfg::BN;
    g.gm = gm;
    if constexpr (IsSplittable<Epi>::value && !Side::kActive && Cfg::BM == 256 && Cfg::BN == 256) {
        const SplitPlan split = plan_split<Cfg>(M, N, K, gm, scratch.p ? scratch.bytes : 0);
        if (split.parts > 1) {
            f32x4_t *partial = static_cast<f32x4_t *>(scratch.p);
            k_gemm_nt_split<Cfg, Epi><<<split.first + split.tail * split.parts, Cfg::THREADS, 0, st>>>(g, epi, split, partial);
            k_gemm_add_parts<Cfg, Epi><<<split.tail * Cfg::TM16, Cfg::THREADS, 0, st>>>(g, epi, split, partial);
            return;
        }
    }
    const int extra = Side::kActive ? side.blocks : 0;
    k_gemm_nt<Cfg, Epi, Side><<<gemm_grid(g.tiles_m, g.tiles_n, g.gm) + extra, Cfg::THREADS, 0, st>>>(g, epi, side);
}

// ---------------------------------------------------------------------------------------------
// Output of a wavefront's sub-tile straight from the accumulators (four columns of a row per lane), no LDS and no barrier:
// a wavefront that is done leaves, whatever the others do.  (Through LDS, as store_tile_bf16 below still does for the other
// layout, a tile of 256 x 256 cost 64 16-bit LDS writes and three barriers per 32 rows.)
// ---------------------------------------------------------------------------------------------

// 16 lanes of x change places with 16 lanes of y: x = {x0, y0, x2, y2}, y = {x1, y1, x3, y3} by groups of 16 lanes
__device__ __forceinline__ void swap_groups16(uint32_t &x, uint32_t &y)
{
#if defined(__HIP_DEVICE_COMPILE__)
    const auto p = __builtin_amdgcn_permlane16_swap(x, y, false, false);
    x = p[0];
    y = p[1];
#endif
}
// largest value / sum over the four lanes l % 16 + 16 k
__device__ __forceinline__ float groups_max(float v)
{
#if defined(__HIP_DEVICE_COMPILE__)
    const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1]));
    const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(q[0]), __uint_as_float(q[1]));
#endif
    return v;
}
__device__ __forceinline__ float groups_sum(float v)
{
#if defined(__HIP_DEVICE_COMPILE__)
    const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(p[0]) + __uint_as_float(p[1]);
    const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(q[0]) + __uint_as_float(q[1]);
#endif
    return v;
}

// Rows of 16-bit elements.  A lane's two words (four columns) of block j and of block j + 1 are exchanged between
// neighbouring groups of 16 lanes so that it ends up with eight consecutive columns of one of the two: stores of 16 bytes,
// 64 consecutive bytes per row, the other half of the cache line with the next store.
// ld and col_limit are multiples of 8.  BLOCKED: dst is stored block by block (blocked64_index).
template <class Cfg, bool BLOCKED>
struct RowsOut16 {
    static_assert(!Cfg::ROWS_IN_LANE && Cfg::TN16 % 2 == 0 && (!BLOCKED || Cfg::WTN % 64 == 0), "layout");
    static_assert(Cfg::WTM <= 256 && 256 % Cfg::WTM == 0, "a wavefront's rows stay inside a block of 256");
    uint16_t *out;          // of the lane's first row
    size_t step;            // to the row 16 further on
    int row, col, row_limit, col_limit;
    bool whole;             // the sub-tile lies inside the matrix
    __device__ __forceinline__ RowsOut16(int lane, int row0, int col0, int rows, int cols, uint16_t *dst, long ld)
    {
        const int q = lane >> 4;
        row = row0 + (lane & 15);
        col = col0 + (q & 1) * 16 + (q >> 1) * 8;
        out = dst + (BLOCKED ? blocked64_index((size_t)row, col, ld) : (size_t)row * ld + col);
        step = BLOCKED ? (size_t)16 * 64 : (size_t)16 * ld;
        row_limit = rows;
        col_limit = cols;
        whole = row0 + Cfg::WTM <= rows && col0 + Cfg::WTN <= cols;
    }
    // block row i: words[j] are the lane's two words of block (i, j).  streamed (uniform): past the caches, for buffers that
    // are larger than those: the panels that the tiles in flight share stay in L2 (keep the logits of 22500 x 50257, d = 768:
    // 2204 -> 2115 us)
    __device__ __forceinline__ void put(int i, uint2 (&words)[Cfg::TN16], bool streamed = false) const
    {
        u32x4_t val[Cfg::TN16 / 2];
#pragma unroll
        for (int p = 0; p < Cfg::TN16 / 2; ++p) {
            uint2 a = words[2 * p], b = words[2 * p + 1];
            swap_groups16(a.x, b.x);
            swap_groups16(a.y, b.y);
            val[p] = u32x4_t{a.x, a.y, b.x, b.y};
        }
        uint16_t *o = out + i * step;
        if (whole && streamed) {
#pragma unroll
            for (int p = 0; p < Cfg::TN16 / 2; ++p) __builtin_nontemporal_store(val[p], reinterpret_cast<u32x4_t *>(o + place(p)));
        } else if (whole) {
#pragma unroll
            for (int p = 0; p < Cfg::TN16 / 2; ++p) *reinterpret_cast<u32x4_t *>(o + place(p)) = val[p];
        } else if (row + 16 * i < row_limit) {
#pragma unroll
            for (int p = 0; p < Cfg::TN16 / 2; ++p)
                if (col + 32 * p < col_limit) *reinterpret_cast<u32x4_t *>(o + place(p)) = val[p];
        }
    }
    static __device__ __forceinline__ constexpr int place(int p) { return BLOCKED ? (p >> 1) * 16384 + (p & 1) * 32 : 32 * p; }
};

// Buffers of this size and more are written past the caches (the last level holds 256 MB)
inline bool streamed_store(size_t bytes) { return bytes >= ((size_t)256 << 20); }

// Rows of fp32: dst = acc, or dst += acc when `accumulate` is set; 16-byte accesses, 64 consecutive bytes per row.
// ld and col_limit are multiples of 4.
template <class Cfg>
__device__ __forceinline__ void store_rows_f32(const f32x4_t (&acc)[Cfg::TM16][Cfg::TN16], int lane, int row0, int col0, int row_limit,
                                               int col_limit, float *__restrict__ dst, long ld, bool accumulate)
{
    static_assert(!Cfg::ROWS_IN_LANE, "four columns per lane");
    const int row = row0 + acc_row(0, lane), col = col0 + acc_col(0, 0, lane);
    float *out = dst + (size_t)row * ld + col;
    const bool whole = row0 + Cfg::WTM <= row_limit && col0 + Cfg::WTN <= col_limit;
#pragma unroll
    for (int i = 0; i < Cfg::TM16; ++i) {
        float *o = out + (size_t)(16 * i) * ld;
        const bool in = row + 16 * i < row_limit;
        if (accumulate) {
            f32x4_t old[Cfg::TN16];
#pragma unroll
            for (int j = 0; j < Cfg::TN16; ++j)
                old[j] = whole || (in && col + 16 * j < col_limit) ? *reinterpret_cast<const f32x4_t *>(o + 16 * j) : f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < Cfg::TN16; ++j)
                if (whole || (in && col + 16 * j < col_limit)) *reinterpret_cast<f32x4_t *>(o + 16 * j) = acc[i][j] + old[j];
        } else {
#pragma unroll
            for (int j = 0; j < Cfg::TN16; ++j)
                if (whole || (in && col + 16 * j < col_limit)) *reinterpret_cast<f32x4_t *>(o + 16 * j) = acc[i][j];
        }
    }
}

// A lane's 16 bytes of row l % 16 at one place, and at the place that follows where the four lanes of the row end, become the
// lane's 16 bytes of row l % 8 and of row 8 + l % 8: eight lanes then write a whole cache line of a row.
__device__ __forceinline__ void exchange_rows8(f32x4_t &a, f32x4_t &b, int lane)
{
    const bool low = (lane & 8) == 0;
    f32x4_t a1, b1;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const float take = dpp_move<0x128>(0.f, low ? b[w] : a[w]);     // rotated by eight of the 16 lanes
        a1[w] = low ? a[w] : take;
        b1[w] = low ? take : b[w];
    }
    a = a1;
    b = b1;
}

// The same without accumulation, 128 consecutive bytes per row: for a buffer that is written past the caches (`streamed`), where
// half lines cost (fp32 logits of 131072 x 32000, d = 4096: 29.3 -> 27.9 ms), and not where the caches join them (16-bit logits
// of 65536 x 32000, d = 2048, the same way: 7.05 -> 7.23 ms).
template <class Cfg>
__device__ __forceinline__ void store_lines_f32(const f32x4_t (&acc)[Cfg::TM16][Cfg::TN16], int lane, int row0, int col0, int row_limit,
                                                int col_limit, float *__restrict__ dst, long ld, bool streamed)
{
    static_assert(!Cfg::ROWS_IN_LANE && Cfg::TN16 % 2 == 0, "four columns per lane");
    const int row = row0 + (lane & 7), col = col0 + (lane & 8) * 2 + 4 * (lane >> 4);
    float *out = dst + (size_t)row * ld + col;
    const size_t step = (size_t)8 * ld;
    const bool whole = row0 + Cfg::WTM <= row_limit && col0 + Cfg::WTN <= col_limit;
#pragma unroll
    for (int i = 0; i < Cfg::TM16; ++i) {
        f32x4_t val[Cfg::TN16];         // [2 p] of rows 0..7 of the block row, [2 p + 1] of rows 8..15; 32 columns each
#pragma unroll
        for (int j = 0; j < Cfg::TN16; ++j) val[j] = acc[i][j];
#pragma unroll
        for (int p = 0; p < Cfg::TN16 / 2; ++p) exchange_rows8(val[2 * p], val[2 * p + 1], lane);
        float *o = out + 2 * i * step;
        auto place = [&](int j) { return reinterpret_cast<f32x4_t *>(o + (j & 1) * step + 32 * (j >> 1)); };
        if (whole && streamed) {
#pragma unroll
            for (int j = 0; j < Cfg::TN16; ++j) __builtin_nontemporal_store(val[j], place(j));
        } else {
#pragma unroll
            for (int j = 0; j < Cfg::TN16; ++j)
                if (row + 16 * i + 8 * (j & 1) < row_limit && col + 32 * (j >> 1) < col_limit) *place(j) = val[j];
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// ---------------------------------------------------------------------------------------------
// Coalesced output of a wavefront's sub-tile for ROWS_IN_LANE.  There the result layout gives each lane single
// elements of 16-column blocks, so values are first laid out row-major in a wave-private
// LDS area (32 rows at a time, the operand stages are free by then) and then written with
// 16-byte stores: a wavefront store covers whole 256-byte row segments.
// `value(i, j, v, row, col)` yields the output for accumulator element v of the 16x16 block (i, j), whose
// global coordinates are (row, col).  All loops are fully unrolled so that the accumulators are
// only ever indexed with constants and stay in registers.
// ---------------------------------------------------------------------------------------------


// P0, P1 restrict the call to the 32-row passes P0 .. P1-1 (default: all of them).  dst is stored block by block
// (blocked64_index).
template <class Cfg, class F, int P0 = 0, int P1 = Cfg::WTM / 32>
__device__ __forceinline__ void store_tile_bf16(char *smem, int wave, int lane, int row0, int col0, int row_limit,
                                                int col_limit /* multiple of 8 */, bf16_t *__restrict__ dst, long ld, F value)
{
    constexpr int RS = Cfg::WTN * 2 + 16;              // padded row stride in bytes
    constexpr int CPR = Cfg::WTN / 8;                   // 16-byte chunks per row
    constexpr int RPP = kWave / CPR;                    // rows per store pass
    static_assert(Cfg::WM * Cfg::WN * 32 * RS <= Cfg::LDS_BYTES, "staging fits");
    char *stage = smem + wave * (32 * RS);
    // a lane's first output address; every later one is a constant number of rows away
    // (the rows of one call lie in one block of 256 and an 8-column piece in one block of 64 columns)
    static_assert(Cfg::WTM <= 256 && 256 % Cfg::WTM == 0, "a wavefront's rows stay inside a block of 256");
    const size_t first_row = (size_t)(row0 + P0 * 32 + lane / CPR);
    const int first_col = col0 + (lane % CPR) * 8;
    bf16_t *out = dst + blocked64_index(first_row, first_col, ld);
    constexpr size_t step = (size_t)RPP * 64;
    __syncthreads();                                    // every wavefront is done reading operand tiles
#pragma unroll
    for (int p = P0; p < P1; ++p) {
#pragma unroll
        for (int ii = 0; ii < 2; ++ii) {
            const int i = 2 * p + ii;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int r = 16 * ii + 4 * (lane >> 4) + v;
#pragma unroll
                for (int j = 0; j < Cfg::TN16; ++j) {
                    const int c = j * 16 + (lane & 15);
                    *reinterpret_cast<bf16_t *>(stage + r * RS + c * 2) = value(i, j, v, row0 + p * 32 + r, col0 + c);
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 32 / RPP; ++q) {
            const int r = q * RPP + lane / CPR, ch = lane % CPR;
            const u32x4_t val = *reinterpret_cast<const u32x4_t *>(stage + r * RS + ch * 16);
            const int grow = row0 + p * 32 + r, gcol = col0 + ch * 8;
            if (grow < row_limit && gcol < col_limit)
                *reinterpret_cast<u32x4_t *>(out) = val;
            out += step;
        }
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);              // conversions of the next pass stay behind this one's stores
    }
}

}  // namespace cph
