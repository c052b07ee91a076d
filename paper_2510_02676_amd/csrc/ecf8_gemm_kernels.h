// Kernels and host-side launch helpers of the fused ECF8 decode + GEMM, shared by the translation units
// that export the calls (ecf8_gemm.hip: the FP8 matrix-core calls; ecf8_gemm_exact.hip: the calls that
// multiply on the F16 matrix cores).  Everything sits in an unnamed namespace: each unit instantiates
// what it launches.
#ifndef ECF8_GEMM_KERNELS_H
#define ECF8_GEMM_KERNELS_H

#include "ecf8_device.h"

#include <cstring>
#include <numeric>
#include <type_traits>

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

constexpr int GK = 4096;                        // K
constexpr int BLOCK_ROWS = 16;

// Waves of a workgroup of the any-K kernels with MT tiles of X: 4, 3 and 2 on a SIMD, which leaves 128, 168 and 256 registers to a wave.  What bounds them is
// each wave's chain of look-ups, some 10 clocks an instruction with two waves on a SIMD.  Two tiles on 8 / 12 waves, us, M = 17 and 32: 4096 x 14336 19.1 / 16.6,
// 20.0 / 17.1; 2048 x 7168 11.3 / 10.3, 11.9 / 10.8; 14336 x 9216 46.2 / 40.8, 49.7 / 46.4, with group scales 53.2 / 43.6, 58.1 / 52.2; 16384 x 256 5.6 / 5.1,
// 5.7 / 5.4; eight experts with scales of W M = 20 126.4 / 117.9, M = 32 135.4 / 126.2, without 114 / 110.5, 123.7 / 122.6.  On 16 they spill: up to twice the time.
template <int MT> constexpr int WAVES = MT == 1 ? 16 : MT == 2 ? 12 : 8;
constexpr int X_ROW = 256 + 16;                 // bytes of a row in a turn buffer: padded so that sixteen rows fall into different banks

// N symbols per lane: a chunk is 16 rows x 4N columns; NW waves per workgroup; MT blocks of 16 rows of X
template <int MT, int NW, int N>
struct GCfg {
    static constexpr int BLOCK_COLS = 4 * N;
    static constexpr int KCHUNKS = GK / BLOCK_COLS;        // chunks per block of rows
    static constexpr int KPW = KCHUNKS / NW;               // of which each wave takes this many
    static constexpr int PIECES = N / 16;
    static_assert(N == 64, "RawRuns, X_ROW");
    static constexpr bool EVEN = KPW * NW == KCHUNKS;              // what the kernels for K = 4096 ask for
    static constexpr int OFF_TBL = 0;
    static constexpr int OFF_RED = OFF_TBL + TBL_ENTRIES * 2;
    static constexpr int RED_BYTES = NW * MT * 64 * 16;            // one buffer of partial sums: one block of rows, every wave
    // Blocks per barrier.  Up to 16 columns of X with one chunk per wave and block, the workgroup's barrier per block
    // of rows is a fifth of the loop: there the waves park the partial sums of four blocks in a row in LDS and
    // meet once to add them up.  Else one block per barrier, in two buffers used in turn.
    static constexpr int BPB = (MT == 1 && KPW == 1) ? 4 : 1;
    static constexpr int RED_BUFS = BPB == 1 ? 2 : BPB;
    static constexpr int TOTAL = OFF_RED + RED_BUFS * RED_BYTES;
    // The any-K kernels have a turn buffer per wave (see turn_x) and give all that is left of the LDS to slots of 16 x 16 MT partial
    // sums (see anyk_walk).
    static constexpr int OFF_TURN = OFF_RED, ANYK_OFF_RED = OFF_TURN + NW * 16 * X_ROW;
    static constexpr uint32_t SLOTS = (160 * 1024 - 64 - ANYK_OFF_RED) / (MT * 1024);
    static constexpr int ANYK_TOTAL = ANYK_OFF_RED + (int)SLOTS * MT * 1024;
    static_assert(RED_BYTES >= 512, "table-build scratch");
    static_assert(TOTAL <= 160 * 1024 && SLOTS >= NW, "LDS of one gfx950 CU");
};

struct GArgs {
    uint64_t d_blob, d_w, d_x, d_y;       // d_blob: compressed W; d_w: raw W (raw kernel)
    uint64_t rows;
    uint64_t off_cb, off_lb, off_st, off_pl, st_bytes, off_tbl;
    uint8_t code_len[16];
    uint32_t M;
    uint64_t d_ws, d_xs;                  // SCALED kernels: per-128x128-block scales of W, scales of X (or 0)
    uint32_t xs_cols;                     // scales per row of X: 1, or K / 128 (one per 128 columns)
    uint64_t K;                           // columns of W (a multiple of 256; 4096 for the fixed-K kernels)
    uint32_t slices;                      // split K: workgroups that share a block of rows (divides K / 256), else 1
    uint64_t d_part, d_ctr;               // split K: partial sums [block][slice][MT * 256] fp32, arrival counters [block] u32
    // Quotients of the fused kernels' deals, from the host (deal_units, deal_waves): a division is some 25 instructions one behind the other at
    // 8 cycles each, at the start of every workgroup
    uint32_t units_each, units_rest;      // units (blocks of rows, times slices) of every workgroup; the first units_rest have one more
    uint32_t unit_chunks;                 // K / 256 / slices
    uint32_t hop, hop_kc;                 // the waves of a workgroup over unit_chunks, and the rest
    uint32_t groups, per_group;           // waves that keep X: groups that take a unit each, waves of a group
    uint32_t batch;                       // any K: blocks between two meetings of the workgroup
    uint32_t by_unit, by_group;           // for small_div by unit_chunks, per_group
};

// n / d where n d < 2^20, from by = small_by(d)
__device__ __forceinline__ uint32_t small_div(uint32_t n, uint32_t by) { return n * by >> 20; }
inline uint32_t small_by(uint32_t d) { return (1u << 20) / d + 1; }

constexpr int SCALE_BLOCK = 128;                // W carries one fp32 scale per 128 x 128 block

typedef float f32x2a __attribute__((ext_vector_type(2), aligned(4)));

// acc += part * (s * x-scale), element by element, where X carries one scale per row and 128 columns, first the forward runs' part
// with the scale of block kb, then the backward runs' with that of kb + 1.  The scales for the accumulator
// rows of this lane (row m = 16 mt + 4 (lane / 16) + r) are fetched one tile of 16 rows at a time, the two of a row together.
template <int MT>
__device__ __forceinline__ void add_scaled_groups(f32x4 (&acc)[MT], const f32x4 (&partA)[MT], const f32x4 (&partB)[MT], float sA, float sB,
                                                  const GArgs &a, int lane, uint32_t kb)
{
    const uint32_t row = 4 * (lane >> 4), at = row * a.xs_cols * 4;       // in bytes, below 2^20
#pragma unroll
    for (int mt = 0; mt < MT; mt++) {
        f32x2a v[4];
#pragma unroll
        for (uint32_t r = 0; r < 4; r++) {
            const GLOBAL uint8_t *xs = (const GLOBAL uint8_t *)a.d_xs + ((uint64_t)((16 * mt + r) * a.xs_cols) + kb) * 4;
            v[r] = f32x2a{0.f, 0.f};
            if (row + 16 * mt + r < a.M) v[r] = *(const GLOBAL f32x2a *)(xs + at);
        }
#pragma unroll
        for (int r = 0; r < 4; r++) acc[mt][r] = __builtin_fmaf(partA[mt][r], sA * v[r].x, acc[mt][r]);
#pragma unroll
        for (int r = 0; r < 4; r++) acc[mt][r] = __builtin_fmaf(partB[mt][r], sB * v[r].y, acc[mt][r]);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// acc += part * s, element by element, the same operation in the fused and in the raw kernel
template <int MT>
__device__ __forceinline__ void add_scaled(f32x4 (&acc)[MT], const f32x4 (&part)[MT], float s)
{
#pragma unroll
    for (int mt = 0; mt < MT; mt++)
#pragma unroll
        for (int r = 0; r < 4; r++) acc[mt][r] = __builtin_fmaf(part[mt][r], s, acc[mt][r]);
}

__device__ __forceinline__ long lo64(u32x4 v) { return (long)(((uint64_t)v.y << 32) | v.x); }
__device__ __forceinline__ long hi64(u32x4 v) { return (long)(((uint64_t)v.w << 32) | v.z); }

// A operands of a wave: for each of its chunks (K slices of 4N) and each piece q, the 16 bytes
// X[m][4N kc + 64 q + 16 g .. + 16) of lane (m = l % 16, g = l / 16), loaded once and kept for
// all blocks (X is M x K <= 256 KiB: half of the CU's register file at M = 64, but re-reading
// it for each of ~900 blocks costs more than everything else).  Lanes of the rows from M on have the last row, no output that is stored depends on
// them: loads under a condition are waited for one by one where the compiler joins their registers with zeros (64 x 4096 M = 1 7.2 us -> 6.3, 4096 x 4096 M = 32 / 64
// 10.4 / 13.7 -> 9.9 / 13.0, 14336 x 4096 M = 64 24.4 -> 23.8).
template <int MT, int NW, int N>
__device__ __forceinline__ void load_x_slice(const GArgs &a, int tid,
                                             u32x4 (&areg)[MT][GCfg<MT, NW, N>::KPW][GCfg<MT, NW, N>::PIECES])
{
    using C = GCfg<MT, NW, N>;
    const int lane = tid & 63, wave = tid >> 6;
    const int n = lane & 15, g = lane >> 4;
    const GLOBAL uint8_t *X = (const GLOBAL uint8_t *)a.d_x;
#pragma unroll
    for (int mt = 0; mt < MT; mt++)
#pragma unroll
        for (int i = 0; i < C::KPW; i++)
#pragma unroll
            for (int q = 0; q < C::PIECES; q++) {
                const uint32_t m = 16 * mt + n;
                const uint32_t k = (wave + NW * i) * C::BLOCK_COLS + 64 * q + 16 * g;
                areg[mt][i][q] = *(const GLOBAL u32x4 *)(X + (m < a.M ? m : a.M - 1) * (uint32_t)GK + k);
            }
}

// A lane's pieces Q and Q + 2 of the nibble plane (16 bytes of the matrix each; row l % 16, column 64 Q + 16 g, g = l / 16) out of one
// 16-byte load.  The four lanes of a row fetch two times 32 bytes of it, lane g the (g % 2)-th half of piece Q + 2 (g / 2) for g' = 0 .. 3, and two
// exchanges between the rows of 16 lanes give every lane what is its own.  Against 8 bytes a piece: half the load instructions, and the two of a
// chunk are adjacent in time, so that they share their 64 bytes while the first-level cache has them (hence no nontemporal loads).
// Eight experts, M = 4 / 16: 97.3 / 103.9 us with 8 bytes a piece, 87.8 / 93.5 with 16, 86.3 / 90.2 cached; 4096 x 14336, M = 16: 22.8, 19.4, 18.6.
__device__ __forceinline__ uint32_t plane_lane(int lane) { return 64u * ((uint32_t)lane >> 5) + 16u * (((uint32_t)lane >> 4) & 1u); }
__device__ __forceinline__ void deal_plane(u32x4 v, u32x2 &a, u32x2 &b)
{
    auto s0 = __builtin_amdgcn_permlane16_swap(v.x, v.z, false, false), s1 = __builtin_amdgcn_permlane16_swap(v.y, v.w, false, false);
    auto t0 = __builtin_amdgcn_permlane32_swap(s0[0], s0[1], false, false), t1 = __builtin_amdgcn_permlane32_swap(s1[0], s1[1], false, false);
    a = u32x2{t0[0], t1[0]};
    b = u32x2{t0[1], t1[1]};
}

// The pair table the encoder embedded, if it did, on its way from the blob to LDS.
constexpr int TABLE_16B = TBL_ENTRIES * 2 / 16;
template <int NW> constexpr int TABLE_UNITS = (TABLE_16B + NW * 64 - 1) / (NW * 64);     // 16-byte units per thread
template <int NW>
__device__ __forceinline__ void load_table(const GArgs &a, int tid, u32x4 (&tv)[TABLE_UNITS<NW>])
{
    if (!a.off_tbl) return;
    const GLOBAL u32x4 *src = (const GLOBAL u32x4 *)(a.d_blob + a.off_tbl);
#pragma unroll
    for (int j = 0; j < TABLE_UNITS<NW>; j++) {
        const int u = tid + j * NW * 64;
        tv[j] = src[TABLE_16B % (NW * 64) == 0 || u < TABLE_16B ? u : tid];
    }
}
template <int NW>
__device__ __forceinline__ void store_table(uint16_t *tbl, int tid, const u32x4 (&tv)[TABLE_UNITS<NW>])
{
#pragma unroll
    for (int j = 0; j < TABLE_UNITS<NW>; j++) {
        const int u = tid + j * NW * 64;
        if (TABLE_16B % (NW * 64) == 0 || u < TABLE_16B) ((u32x4 *)tbl)[u] = tv[j];
    }
    __syncthreads();
}

// The sums of one chunk (16 rows x 256 columns).  Without scales a chunk adds straight into the block's
// accumulators.  With scales its two 128-column halves -- exactly its forward and its backward run --
// are summed by the matrix cores apart and enter the block's sum through one multiply-add each, with
// the scale of their 128 x 128 block of W (times the scale of X for that row and slice, if X has those).
template <int MT, int SC>
struct ChunkSums {
    static constexpr bool SCALED = SC != 0, XGROUPS = SC == 2;
    f32x4 partA[SCALED ? MT : 1], partB[SCALED ? MT : 1];
    float sA = 1.f, sB = 1.f;
    uint32_t kbA = 0;              // the chunk's first 128-column block of K

    __device__ __forceinline__ void begin(const GArgs &a, uint64_t block, uint32_t kc)
    {
        if constexpr (SCALED) {
            const GLOBAL float *ws = (const GLOBAL float *)a.d_ws + (block * BLOCK_ROWS / SCALE_BLOCK) * (a.K / SCALE_BLOCK) + 2 * kc;
            sA = ws[0];
            sB = ws[1];
            kbA = 2 * kc;
#pragma unroll
            for (int mt = 0; mt < MT; mt++) partA[mt] = partB[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
    // where the MFMAs of the forward / backward run accumulate
    __device__ __forceinline__ auto &first(f32x4 (&acc)[MT]) { if constexpr (SCALED) return partA; else return acc; }
    __device__ __forceinline__ auto &second(f32x4 (&acc)[MT]) { if constexpr (SCALED) return partB; else return acc; }
    __device__ __forceinline__ void end(f32x4 (&acc)[MT], const GArgs &a, int lane)
    {
        if constexpr (XGROUPS) {   // the scales of X are fetched here: held over the decode they would cost it registers
            add_scaled_groups<MT>(acc, partA, partB, sA, sB, a, lane, kbA);
        } else if constexpr (SCALED) {
            add_scaled<MT>(acc, partA, sA);
            add_scaled<MT>(acc, partB, sB);
        }
    }
};

// Eight E4M3 bytes as eight halves.  Every E4M3 value, subnormals included, is a half exactly (3 mantissa
// bits, exponents 2^-9 .. 2^8), so nothing is rounded here; NaN encodings stay NaN.
__device__ __forceinline__ f16x8 e4m3x8_to_f16(uint32_t lo, uint32_t hi)
{
    const f16x2 a = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(lo, 1.0f, false);
    const f16x2 b = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(lo, 1.0f, true);
    const f16x2 c = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(hi, 1.0f, false);
    const f16x2 d = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(hi, 1.0f, true);
    return f16x8{a.x, a.y, b.x, b.y, c.x, c.y, d.x, d.y};
}

// One piece (16 K-elements of this lane's row of W, in w) times the matching 16 columns of X (A_OF_MT:
// the piece of X for tile mt_).  Two ways to multiply, chosen by the kernels' ACC parameter:
//   ACC = 0  the FP8 matrix core (v_mfma_f32_16x16x32_fp8_fp8) on the bytes as they are.  It aligns each
//            lane's 8 products to the largest of them and drops what lies more than about 13 bits below
//            it, so an output can be off by up to 7 * 2^-13 of sum |x w| (a few 1e-5 of it on
//            heavy-tailed weights);
//   ACC = 1  both operands converted to halves in registers (exact, see above) and multiplied by the F16
//            matrix core (v_mfma_f32_16x16x32_f16), which keeps the exact products' fp32 sums: outputs
//            within fp32 rounding of the true sum.  Same lanes, same K order: a lane's 8 bytes of a step
//            become its 8 halves.
#define ECF8_MFMA_OPERANDS(acc, A_OF_MT, W_PIECE)                                                        \
    do {                                                                                                 \
        const u32x4 w_ = (W_PIECE);                                                                      \
        if constexpr (ACC == 0) {                                                                        \
            _Pragma("unroll") for (int mt_ = 0; mt_ < MT; mt_++) {                                       \
                const u32x4 a_ = A_OF_MT;                                                                \
                acc[mt_] = __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(lo64(a_), lo64(w_), acc[mt_], 0, 0, 0); \
                acc[mt_] = __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(hi64(a_), hi64(w_), acc[mt_], 0, 0, 0); \
            }                                                                                            \
        } else {                                                                                         \
            const f16x8 wl_ = e4m3x8_to_f16(w_.x, w_.y), wh_ = e4m3x8_to_f16(w_.z, w_.w);                \
            _Pragma("unroll") for (int mt_ = 0; mt_ < MT; mt_++) {                                       \
                const u32x4 a_ = A_OF_MT;                                                                \
                acc[mt_] = __builtin_amdgcn_mfma_f32_16x16x32_f16(e4m3x8_to_f16(a_.x, a_.y), wl_, acc[mt_], 0, 0, 0); \
                acc[mt_] = __builtin_amdgcn_mfma_f32_16x16x32_f16(e4m3x8_to_f16(a_.z, a_.w), wh_, acc[mt_], 0, 0, 0); \
            }                                                                                            \
        }                                                                                                \
    } while (0)
#define ECF8_MFMA_PIECE(acc, areg, i, p, W_PIECE) ECF8_MFMA_OPERANDS(acc, areg[mt_][i][p], W_PIECE)

// Partial sums of the NW waves -> 16 x M outputs of block `block`.  `red` is the buffer of this
// block's parity; the one barrier also orders its reuse two blocks later (a thread passes the
// next block's barrier only after every thread has finished summing here).
template <int MT, int NW, bool SCALED = false>
__device__ __forceinline__ void reduce_block(f32x4 *red, const GArgs &a, uint64_t block, int tid, const f32x4 (&acc)[MT])
{
    const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
    for (int mt = 0; mt < MT; mt++) red[(wave * MT + mt) * 64 + lane] = acc[mt];
    __syncthreads();
    // a lane of the accumulator holds D[4*(lane>>4) + r][lane & 15], r = 0..3
    GLOBAL float *Y = (GLOBAL float *)a.d_y;
    for (int o = tid; o < MT * 256; o += NW * 64) {
        const int mt = o >> 8, l = (o >> 2) & 63, r = o & 3;
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < NW; w++) sum += ((const float *)&red[(w * MT + mt) * 64 + l])[r];
        const uint32_t m = 16 * mt + 4 * (l >> 4) + r;
        if (m < a.M) {
            if (SCALED && a.d_xs && a.xs_cols == 1) sum *= ((const GLOBAL float *)a.d_xs)[m];
            Y[(uint64_t)m * a.rows + block * BLOCK_ROWS + (l & 15)] = sum;
        }
    }
}

// reduce_block for `count` blocks of rows at once (up to 16 columns of X): the waves have parked their partial sums of
// blocks first, first + stride, ... in buffers 0, 1, ... of `red`; the caller's barrier lies between that and this.
// Every output is summed over the waves in reduce_block's order.
template <int NW, bool SCALED>
__device__ __forceinline__ void reduce_parked(const f32x4 *red, const GArgs &a, uint64_t first, uint64_t stride, uint32_t count, int tid)
{
    GLOBAL float *Y = (GLOBAL float *)a.d_y;
    for (uint32_t o = tid; o < count * 256; o += NW * 64) {
        const uint32_t j = o >> 8, l = (o >> 2) & 63, r = o & 3;
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < NW; w++) sum += ((const float *)&red[(j * NW + w) * 64 + l])[r];
        const uint32_t m = 4 * (l >> 4) + r;
        if (m < a.M) {
            if (SCALED && a.d_xs && a.xs_cols == 1) sum *= ((const GLOBAL float *)a.d_xs)[m];
            Y[(uint64_t)m * a.rows + (first + j * stride) * BLOCK_ROWS + (l & 15)] = sum;
        }
    }
}

// reduce_block for a batch of `count` blocks of rows first, first + stride, ...: the waves have parked block j's partial sums in
// slots slots * j, slots * j + 1, ... of `red`, one per place of a chunk in the deal (its number modulo PLACES), whoever had it; the
// caller's barriers lie around this.  Summed in that order, which is reduce_block's.
template <int MT, int NW, int PLACES, bool SCALED>
__device__ __forceinline__ void reduce_batch(const f32x4 *red, const GArgs &a, uint64_t first, uint64_t stride, uint32_t count, uint32_t slots, int tid)
{
    GLOBAL float *Y = (GLOBAL float *)a.d_y;
    for (uint32_t o = tid; o < count * (MT * 256); o += NW * 64) {
        const uint32_t j = o / (MT * 256), mt = (o >> 8) % MT, l = (o >> 2) & 63, r = o & 3;
        const float *p = (const float *)&red[(j * slots * MT + mt) * 64 + l] + r;
        float sum = 0.f;
        if (slots == PLACES) {
#pragma unroll
            for (int w = 0; w < PLACES; w++) sum += p[w * (MT * 256)];
        } else {
            for (uint32_t w = 0; w < slots; w++) sum += p[w * (MT * 256)];
        }
        const uint32_t m = 16 * mt + 4 * (l >> 4) + r;
        if (m < a.M) {
            if (SCALED && a.d_xs && a.xs_cols == 1) sum *= ((const GLOBAL float *)a.d_xs)[m];
            Y[(uint64_t)m * a.rows + (first + j * stride) * BLOCK_ROWS + (l & 15)] = sum;
        }
    }
}

// How the NW waves of a workgroup share the work of a unit in the any-K kernels on uncompressed W.  Long K: a unit is one
// block of rows and its chunks are dealt round-robin to all waves.  Short K (at most NW / 2 chunks per
// block): the waves form `groups` groups of `wpb`, and each group takes a block of rows of its own --
// blocks j, j + 1, ... of the workgroup's sequence -- so that no wave is left without work (at K = 2048,
// 8 chunks, half of 16 waves would be).
struct Deal {
    uint32_t groups, wpb;       // blocks per unit; waves per block
    uint32_t gi, kw;            // this wave: its group, its place in the group
    uint32_t my_chunks;         // chunks of a block (or slice) that fall to this wave
};

template <int NW>
__device__ __forceinline__ Deal deal_chunks(const GArgs &a, bool split, int wave)
{
    Deal d;
    const uint32_t w = uniform32((uint32_t)wave);       // the same for every lane: keep all of this in scalar registers
    d.groups = split ? 1u : a.groups;
    d.wpb = split ? (uint32_t)NW : a.per_group;
    d.gi = split ? 0u : small_div(w, a.by_group);
    d.kw = w - d.gi * d.wpb;
    if (d.groups > 1) d.my_chunks = d.gi < d.groups && d.kw < a.unit_chunks ? 1u : 0u;
    else d.my_chunks = a.unit_chunks > d.kw ? (a.unit_chunks - d.kw + NW - 1) / NW : 0u;
    return d;
}

// reduce_block for a unit of d.groups blocks: blocks j0 .. j0 + groups - 1 of the sequence first + j * stride
// (those below `count`), each summed over the waves of its group -- in the order reduce_block takes them,
// so that a block's result does not depend on how many blocks shared the unit.
template <int MT, int NW, bool SCALED>
__device__ __forceinline__ void reduce_groups(f32x4 *red, const GArgs &a, uint64_t first, uint64_t stride, uint64_t j0, uint64_t count,
                                              const Deal &d, int tid, const f32x4 (&acc)[MT])
{
    if (d.groups == 1) {
        reduce_block<MT, NW, SCALED>(red, a, first + j0 * stride, tid, acc);
        return;
    }
    const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
    for (int mt = 0; mt < MT; mt++) red[(wave * MT + mt) * 64 + lane] = acc[mt];
    __syncthreads();
    GLOBAL float *Y = (GLOBAL float *)a.d_y;
    for (uint32_t o = tid; o < d.groups * (MT * 256); o += NW * 64) {
        const uint32_t g = o / (MT * 256), oo = o % (MT * 256);
        const uint32_t mt = oo >> 8, l = (oo >> 2) & 63, r = oo & 3;
        if (j0 + g >= count) break;                     // the sequence ended inside this unit
        float sum = 0.f;
        for (uint32_t w = g * d.wpb; w < (g + 1) * d.wpb; w++) sum += ((const float *)&red[(w * MT + mt) * 64 + l])[r];
        const uint32_t m = 16 * mt + 4 * (l >> 4) + r;
        if (m < a.M) {
            if (SCALED && a.d_xs && a.xs_cols == 1) sum *= ((const GLOBAL float *)a.d_xs)[m];
            Y[(uint64_t)m * a.rows + (first + (j0 + g) * stride) * BLOCK_ROWS + (l & 15)] = sum;
        }
    }
}

// Split K: the partial sums of the unit (block of rows, slice of K) go to the workspace, and the
// workgroup that brings a block's last slice adds the slices up -- in slice order, so the result
// does not depend on which one that was -- and writes the outputs.  No workgroup waits for
// another; the last one leaves the counter at zero for the next call.
// Memory order.  Every thread writes its partial sums, the workgroup meets at a barrier, and ONE thread
// adds to the block's arrival counter with release and acquire order at agent scope: the barrier orders the
// other threads' stores before that add (release side) and the add before the other threads' loads in
// the workgroup that turns out to be last (acquire side), so the last workgroup's reads of the other
// slices are ordered after their writes by the memory model itself.  The agent-scope release / acquire
// writes back and invalidates caches once per workgroup (measured: about 2 us per launch).  Partial
// sums move through agent-scope atomic stores and loads, so they are never served from or left in a
// cache private to a part of the chip; each wave also waits for its own stores before the barrier.
template <int MT, int NW, bool SCALED>
__device__ __forceinline__ void reduce_split(f32x4 *red, uint32_t *s_flag, const GArgs &a, uint32_t block, uint32_t slice,
                                             int tid, const f32x4 (&acc)[MT])
{
    const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
    for (int mt = 0; mt < MT; mt++) red[(wave * MT + mt) * 64 + lane] = acc[mt];
    __syncthreads();
    GLOBAL uint32_t *part = (GLOBAL uint32_t *)a.d_part + (uint64_t)block * a.slices * (MT * 256);
    GLOBAL uint32_t *ctr = (GLOBAL uint32_t *)a.d_ctr + block;
    for (int o = tid; o < MT * 256; o += NW * 64) {
        const int mt = o >> 8, l = (o >> 2) & 63, r = o & 3;
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < NW; w++) sum += ((const float *)&red[(w * MT + mt) * 64 + l])[r];
        __hip_atomic_store(part + (uint64_t)slice * (MT * 256) + o, __float_as_uint(sum), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // this wave's stores have completed ...
    __syncthreads();                                        // ... and so have every wave's
    if (tid == 0) *s_flag = __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (*s_flag != a.slices - 1) return;          // uniform: the same LDS word for every thread
    GLOBAL float *Y = (GLOBAL float *)a.d_y;
    for (int o = tid; o < MT * 256; o += NW * 64) {
        const int mt = o >> 8, l = (o >> 2) & 63, r = o & 3;
        float sum = 0.f;
        for (uint32_t sl = 0; sl < a.slices; sl++)
            sum += __uint_as_float(__hip_atomic_load(part + (uint64_t)sl * (MT * 256) + o, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        const uint32_t m = 16 * mt + 4 * (l >> 4) + r;
        if (m < a.M) {
            if (SCALED && a.d_xs && a.xs_cols == 1) sum *= ((const GLOBAL float *)a.d_xs)[m];
            Y[(uint64_t)m * a.rows + (uint64_t)block * BLOCK_ROWS + (l & 15)] = sum;
        }
    }
    if (tid == 0) __hip_atomic_store(ctr, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// What of a chunk is needed before its bits: where it starts in the stream and the bits of this lane.
// ONE: fetched in one instruction of four bytes a lane, lanes 0 .. 31 the lanes' bits, two each, lanes 32 and 33 the position (the others that
// again); as two they are loads of 2 and 8 bytes a lane, the latter the same for all.
template <bool ONE>
struct ChunkMeta {
    uint64_t b0 = 0;
    uint32_t lb = 0;                        // ONE: as fetched
    __device__ __forceinline__ uint64_t begin() const
    {
        return ONE ? (uint32_t)__builtin_amdgcn_readlane((int)lb, 32) | (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)lb, 33) << 32 : uniform64(b0);
    }
    __device__ __forceinline__ uint32_t lane_bits(int lane) const
    {
        return ONE ? ((uint32_t)__builtin_amdgcn_ds_bpermute((lane >> 1) * 4, (int)lb) >> (16 * (lane & 1))) & 0xffffu : lb;
    }
};
template <bool ONE>
struct MetaReader {
    uint64_t at, off_lb;                    // ONE: of this lane's dword for chunk 0; else the blob's chunk_bit and lane_bits
    uint32_t step, lane;
    __device__ __forceinline__ MetaReader(const GArgs &a, int lane_)
    {
        lane = (uint32_t)lane_;
        at = a.d_blob + (!ONE ? a.off_cb : lane < 32 ? a.off_lb + 4 * lane : a.off_cb + 4 * (lane & 1));
        off_lb = a.d_blob + a.off_lb;
        step = lane < 32 ? 128u : 8u;
    }
    __device__ __forceinline__ ChunkMeta<ONE> operator()(uint64_t c) const
    {
        ChunkMeta<ONE> m;
        if constexpr (ONE) {
            m.lb = *(const GLOBAL uint32_t *)(at + (uint64_t)(uint32_t)c * step);           // a chunk's number is below 2^32
        } else {
            m.b0 = ((const GLOBAL uint64_t *)at)[c];
            m.lb = ((const GLOBAL uint16_t *)off_lb)[c * 64 + lane];
        }
        return m;
    }
};

// A lane's codewords of a chunk straight from memory to registers: the 8 dwords that hold its forward run from the first bit on and the 8 that hold its
// backward run from the last bit down.  32 codewords of at most 7 bits are 224 bits; with them come the bit next to the first one, which makes a
// masked window the byte offset of a table entry (see quad_step2), and up to 31 bits of its dword.  Positions are counted
// in bits from 16 bytes before the chunk's span.
// The chunk's span staged in LDS and the runs' windows read from there took a third of the LDS's time, which was busy for 61 % (14336 x 4096,
// M = 16) and 76 % (eight experts, M = 4) of the launch.  Now the gathers are 256 accesses to the
// first-level cache a chunk, which has the time; vector operations are as many as before.  us: 14336 x 4096, M = 1 / 16 / 32 / 64 17.8 / 19.1 / 22.1 / 29.2 -> 15.2 / 15.5 / 18.9 / 24.6, 14336 x 7168,
// M = 16 31.1 -> 25.1, six experts, scales of W, M = 4 67.7 -> 55.3, eight 86.6 -> 75.8.  Cached: the lines are a lane's neighbours' too.
typedef uint32_t u32x4a __attribute__((ext_vector_type(4), aligned(4)));
struct RawRuns {
    u32x4 a0, a1, b0, b1;
    uint32_t pa, pb;            // the bit before the forward run's first; the one behind the backward run's first

    // Positions beyond the stream (damaged metadata) read its end; what is read around it, 32 bytes at the most, belongs to the blob.
    template <bool ONE>
    __device__ __forceinline__ void fetch(const GLOBAL uint8_t *stream, uint64_t st_bytes, const ChunkMeta<ONE> &m, int lane)
    {
        const uint64_t begin = m.begin();
        uint64_t byte0 = (begin >> 3) & ~15ull;
        if (byte0 > st_bytes) byte0 = st_bytes;
        const uint64_t room = st_bytes - byte0 + 16;
        const uint32_t most = room < (1u << 28) ? (uint32_t)room : 1u << 28;
        const uint32_t lb = m.lane_bits(lane), end = wave_incl_scan(lb) + ((uint32_t)begin & 127u);
        pa = end - lb + 127;
        pb = end + 128;
        uint32_t atA = (pa >> 3) & ~3u, atB = (pb >> 3) & ~3u;
        atA = atA < most ? atA : most;
        atB = atB < most ? atB : most;
        const GLOBAL uint8_t *base = stream + byte0 - 16;
        a0 = *(const GLOBAL u32x4a *)(base + atA);
        a1 = *(const GLOBAL u32x4a *)(base + atA + 16);
        b0 = *(const GLOBAL u32x4a *)(base - 28 + atB);
        b1 = *(const GLOBAL u32x4a *)(base - 12 + atB);
    }
};

// The two runs as strings of bits in reading order, the next bit at bit 1 of the first dword.  A step takes four codewords, 28 bits at most, off
// either and shifts what may still be needed: seven dwords after the first step, one less after each.
struct ShiftedRuns {
    uint32_t a[8], b[8];

    __device__ __forceinline__ void begin(const RawRuns &r)
    {
        const uint32_t x[8] = {r.a0.x, r.a0.y, r.a0.z, r.a0.w, r.a1.x, r.a1.y, r.a1.z, r.a1.w};
        const uint32_t y[8] = {__brev(r.b1.w), __brev(r.b1.z), __brev(r.b1.y), __brev(r.b1.x), __brev(r.b0.w), __brev(r.b0.z), __brev(r.b0.y), __brev(r.b0.x)};
#pragma unroll
        for (int i = 0; i < 8; i++) {
            a[i] = __builtin_amdgcn_alignbit(i < 7 ? x[i + 1] : 0u, x[i], r.pa);
            b[i] = __builtin_amdgcn_alignbit(i < 7 ? y[i + 1] : 0u, y[i], ~r.pb);
        }
    }
    // step t = 0 .. 7: the exponent fields of four elements of each run
    __device__ __forceinline__ void step(const uint16_t *tbl, int t, uint32_t &outA, uint32_t &outB)
    {
        constexpr uint32_t OFF_MASK = TBL_MASK << 1;
        const uint8_t *tb = (const uint8_t *)tbl;
        const uint32_t eA1 = *(const uint16_t *)(tb + (a[0] & OFF_MASK)), eB1 = *(const uint16_t *)(tb + (b[0] & OFF_MASK));
        const uint32_t nA1 = (eA1 >> 7) & 15u, nB1 = (eB1 >> 7) & 15u;
        const uint32_t eA2 = *(const uint16_t *)(tb + ((a[0] >> nA1) & OFF_MASK)), eB2 = *(const uint16_t *)(tb + ((b[0] >> nB1) & OFF_MASK));
        const uint32_t nA = nA1 + ((eA2 >> 7) & 15u), nB = nB1 + ((eB2 >> 7) & 15u);
#pragma unroll
        for (int i = 0; i < 7; i++)
            if (i < 7 - t) {                                // 28 (7 - t) + 1 bits are left at most
                a[i] = __builtin_amdgcn_alignbit(a[i + 1], a[i], nA);
                b[i] = __builtin_amdgcn_alignbit(b[i + 1], b[i], nB);
            }
        outA = __builtin_amdgcn_perm(eA2, eA1, 0x05040100u);
        outB = __builtin_amdgcn_perm(eB2, eB1, 0x05040100u);
    }
};

template <int MT, int NW, int N, int SC, int ACC, class CODES>       // SC: 0 no scales, 1 scales of W (and one per row of X), 2 also one per row and 128 columns of X; ACC: see ECF8_MFMA_OPERANDS
__global__ __launch_bounds__(NW * 64) void ecf8_gemm_kernel(GArgs a, CODES codes)
{
    constexpr bool SCALED = SC != 0;
    static_assert(!SCALED || 4 * N == 2 * SCALE_BLOCK, "a chunk spans two scale blocks of K");
    using C = GCfg<MT, NW, N>;
    static_assert(C::EVEN, "waves split the chunks of a block evenly");
    constexpr int KPW = C::KPW, KCHUNKS = C::KCHUNKS, BLOCK_COLS = C::BLOCK_COLS;
    constexpr int GPIECES = C::PIECES;
    __shared__ __attribute__((aligned(16))) uint8_t smem[C::TOTAL];
    uint16_t *tbl = (uint16_t *)(smem + C::OFF_TBL);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

    const GLOBAL uint8_t *stream = (const GLOBAL uint8_t *)(a.d_blob + a.off_st);
    const GLOBAL uint8_t *plane = (const GLOBAL uint8_t *)(a.d_blob + a.off_pl);

    constexpr bool META1 = MT == 4;            // M = 64 25.0 us, 24.6 with it, scales of W 28.6, 26.6; M = 16 15.5, 15.8
    using Meta = ChunkMeta<META1>;
    const MetaReader<META1> meta(a, lane);
    const uint32_t wave_s = uniform32((uint32_t)wave);             // the same for every lane: chunk addresses stay in scalar registers
    // the wave's chunks in the order it meets them: step s = its (s % KPW)-th chunk of its (s / KPW)-th block
    typedef typename std::conditional<MT == 1, uint32_t, uint64_t>::type Step;     // M = 1 16.1 -> 15.0 us in 32 bits, M = 32 with group scales 22.2 -> 24.7
    auto block_of = [&](Step s) -> Step { return blockIdx.x + (s / KPW) * (Step)gridDim.x; };
    auto kc_of = [&](Step s) -> uint32_t { return wave_s + NW * (uint32_t)(s % KPW); };
    auto load_meta = [&](Step s) { return meta((uint64_t)block_of(s) * KCHUNKS + kc_of(s)); };
    // nibble plane of step s: this lane's part of pieces q and q + 2 at plane_of(s) + lane_plane + 32 q, see deal_plane
    const uint32_t lane_plane = (uint32_t)(lane & 15) * (GK / 2) + plane_lane(lane);
    auto plane_of = [&](Step s) -> const GLOBAL uint8_t * {
        return plane + (block_of(s) * (uint64_t)(BLOCK_ROWS * GK) + kc_of(s) * (uint64_t)BLOCK_COLS) / 2;
    };

    // start-up: the first chunks' loads and those of X are in flight while the table is set up
    const Step n_steps = (Step)(a.units_each + (blockIdx.x < a.units_rest ? 1u : 0u)) * KPW;
    Meta m_cur, m_next;
    RawRuns raw = {};
    static_assert(GPIECES == 4, "deal_plane");
    u32x4 pl[2];
#pragma unroll
    for (int q = 0; q < 2; q++) pl[q] = u32x4{0, 0, 0, 0};
    // Only the first chunk's stream has to wait for anything (its metadata): the rest is asked for before that wait, and the
    // table first, since it is what the workgroup meets for.
    u32x4 tv[TABLE_UNITS<NW>];
    uint32_t two = 0;
    constexpr bool SHORT = std::is_same<CODES, ShortCodes>::value;
    if constexpr (!SHORT) {
        load_table<NW>(a, tid, tv);
    } else {
        if (wave_s == 0) two = codes.two[lane];
    }
    if (n_steps > 0) {
        m_cur = load_meta(0);
        m_next = load_meta(n_steps > 1 ? 1 : 0);
        const GLOBAL uint8_t *pp = plane_of(0);
#pragma unroll
        for (int q = 0; q < 2; q++) pl[q] = *(const GLOBAL u32x4 *)(pp + lane_plane + 32 * q);
    }
    u32x4 areg[MT][KPW][GPIECES];
    load_x_slice<MT, NW, N>(a, tid, areg);
    if (n_steps > 0) raw.fetch(stream, a.st_bytes, m_cur, lane);

    if constexpr (SHORT) {
        build_pair_table<NW>(two, tbl, (uint32_t *)(smem + C::OFF_RED), lane, (int)wave_s);
    } else if (a.off_tbl) {
        // Always: these calls are launched with ShortCodes where the blob has no table.  The condition changes what the compiler puts first: with / without it,
        // and load_table's, us, 4096 x 4096 M = 17 / 32 8.4 / 8.5, 9.5 / 9.6, but 14336 x 4096 M = 16 15.5 / 15.25, M = 32 18.55 / 18.4; the others are as fast either way.
        store_table<NW>(tbl, tid, tv);
    }

    uint32_t parity = 0;
    for (Step s0 = 0; s0 < n_steps; s0 += KPW) {
        f32x4 acc[MT];
#pragma unroll
        for (int mt = 0; mt < MT; mt++) acc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < KPW; i++) {
            const Step s = s0 + i;
            ShiftedRuns runs;
            runs.begin(raw);
            // The raw registers are free: fetch the next chunk's runs, and the metadata of the chunk after it.
            // The last steps have nothing to fetch and no branch around the loads either: the last chunk's metadata and runs
            // again, and the plane's first chunk, which every wave then asks for.
            const bool more = s + 1 < n_steps;                 // the same for every lane
            const Step sn = more ? s + 1 : s, sn2 = s + 2 < n_steps ? s + 2 : sn;
            raw.fetch(stream, a.st_bytes, m_next, lane);
            const Meta m_next2 = load_meta(sn2);
            const GLOBAL uint8_t *pp = more ? plane_of(sn) : plane;
            ChunkSums<MT, SC> sums;
            sums.begin(a, block_of(s), kc_of(s));
            auto &dstA = sums.first(acc);
            auto &dstB = sums.second(acc);
#pragma unroll
            for (int Q = 0; Q < GPIECES / 2; Q++) {
                uint32_t dwA[4], dwB[4];
#pragma unroll
                for (int t = 0; t < 4; t++) runs.step(tbl, 4 * Q + t, dwA[t], dwB[t]);
                // two pieces of the nibble plane are merged, and their registers take the same pieces of the next chunk
                u32x2 pA, pB;
                deal_plane(pl[Q], pA, pB);
                pl[Q] = *(const GLOBAL u32x4 *)(pp + lane_plane + 32 * Q);
                const u32x4 wA = merge_piece(dwA, pA);
                ECF8_MFMA_PIECE(dstA, areg, i, Q, wA);
                const u32x4 wB = merge_piece(dwB, pB);
                ECF8_MFMA_PIECE(dstB, areg, i, Q + GPIECES / 2, wB);
            }
            sums.end(acc, a, lane);
            m_next = m_next2;
        }
        if constexpr (C::BPB == 1) {
            reduce_block<MT, NW, SCALED>((f32x4 *)(smem + C::OFF_RED + parity * C::RED_BYTES), a, block_of(s0), tid, acc);
            parity ^= 1;
        } else {
            // park this block's partial sums; the workgroup meets after every BPB-th block and after the last one
            f32x4 *red = (f32x4 *)(smem + C::OFF_RED);
            const uint32_t j = (uint32_t)(s0 / KPW % C::BPB);
            red[(j * NW + wave_s) * 64 + lane] = acc[0];
            const bool last = s0 + KPW >= n_steps;           // the same for the whole workgroup
            if (j == C::BPB - 1 || last) {
                __syncthreads();
                reduce_parked<NW, SCALED>(red, a, block_of(s0 - j * KPW), gridDim.x, j + 1, tid);
                if (!last) __syncthreads();                  // the buffers are free again
            }
        }
    }
}

// The same GEMM on uncompressed row-major W, with the fused kernel's workgroup shape, K split
// and order of accumulation, so that the two agree bit for bit.
template <int MT, int NW, int N, int SC, int ACC = 0>
__global__ __launch_bounds__(NW * 64) void ecf8_gemm_raw_kernel(GArgs a)
{
    constexpr bool SCALED = SC != 0;
    using C = GCfg<MT, NW, N>;
    static_assert(C::EVEN, "waves split the chunks of a block evenly");
    constexpr int KPW = C::KPW, BLOCK_COLS = C::BLOCK_COLS, GPIECES = C::PIECES;
    __shared__ __attribute__((aligned(16))) uint8_t smem[C::RED_BUFS * C::RED_BYTES];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const GLOBAL uint8_t *W = (const GLOBAL uint8_t *)a.d_w;
    const uint64_t lane_elem = (uint64_t)(lane & 15) * GK + (uint64_t)(lane >> 4) * 16;
    const uint64_t n_steps = (uint64_t)(a.units_each + (blockIdx.x < a.units_rest ? 1u : 0u)) * KPW;
    auto block_of = [&](uint64_t s) -> uint64_t { return blockIdx.x + (s / KPW) * (uint64_t)gridDim.x; };
    auto load_w = [&](uint64_t s, u32x4 (&w)[GPIECES]) {
        const uint64_t e0 = block_of(s) * BLOCK_ROWS * (uint64_t)GK + (wave + NW * (uint32_t)(s % KPW)) * (uint64_t)BLOCK_COLS + lane_elem;
#pragma unroll
        for (int q = 0; q < GPIECES; q++) w[q] = __builtin_nontemporal_load((const GLOBAL u32x4 *)(W + e0 + 64 * q));
    };
    u32x4 w_cur[GPIECES], w_next[GPIECES];
    if (n_steps > 0) load_w(0, w_cur);
    u32x4 areg[MT][KPW][GPIECES];
    load_x_slice<MT, NW, N>(a, tid, areg);
    uint32_t parity = 0;
    for (uint64_t s0 = 0; s0 < n_steps; s0 += KPW) {
        f32x4 acc[MT];
#pragma unroll
        for (int mt = 0; mt < MT; mt++) acc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < KPW; i++) {
            const uint64_t s = s0 + i;
#pragma unroll
            for (int q = 0; q < GPIECES; q++) w_next[q] = w_cur[q];
            if (s + 1 < n_steps) load_w(s + 1, w_next);
            ChunkSums<MT, SC> sums;
            sums.begin(a, block_of(s), wave + NW * (uint32_t)(s % KPW));
            auto &dstA = sums.first(acc);
            auto &dstB = sums.second(acc);
#pragma unroll
            for (int Q = 0; Q < GPIECES / 2; Q++) {
                ECF8_MFMA_PIECE(dstA, areg, i, Q, w_cur[Q]);
                ECF8_MFMA_PIECE(dstB, areg, i, Q + GPIECES / 2, w_cur[Q + GPIECES / 2]);
            }
            sums.end(acc, a, lane);
#pragma unroll
            for (int q = 0; q < GPIECES; q++) w_cur[q] = w_next[q];
        }
        if constexpr (C::BPB == 1) {
            reduce_block<MT, NW, SCALED>((f32x4 *)(smem + parity * C::RED_BYTES), a, block_of(s0), tid, acc);
            parity ^= 1;
        } else {
            f32x4 *red = (f32x4 *)smem;                      // as in the fused kernel
            const uint32_t j = (uint32_t)((s0 / KPW) % C::BPB);
            red[(j * NW + wave) * 64 + lane] = acc[0];
            const bool last = s0 + KPW >= n_steps;
            if (j == C::BPB - 1 || last) {
                __syncthreads();
                reduce_parked<NW, SCALED>(red, a, block_of(s0 - j * KPW), gridDim.x, j + 1, tid);
                if (!last) __syncthreads();
            }
        }
    }
}

// ---- any K (a multiple of 256) ----
// The kernels above keep the wave's slice of X in registers, which ties them to K = 4096.  These take any K: the K / 256
// chunks of a workgroup's blocks of rows are dealt to its NW waves.  With one tile of X and at most 2 NW chunks per block
// (see resident_chunks) a wave keeps the X of its one or two chunks in registers too, and where a block has at most NW / 2 chunks the
// waves form groups with a block each; else X (L2-resident: M x K bytes) is fetched for every chunk, one chunk ahead, like the
// chunk's payload.  Same decode, same MFMA order inside a chunk, and sums added in the same order.

// The table's set-up out of line (APART), for the kernels that walk over several matrices: inlined there, its registers
// cost the decode loop spills (eight experts 113.8 us inlined, 109.6 called; kernels of one matrix have the registers and
// save the call's 1 us).
template <int NW>
__device__ __noinline__ void build_pair_table_apart(uint64_t len_lo, uint64_t len_hi, uint8_t *smem, int lane, int wave)
{
    using C = GCfg<1, NW, 64>;
    build_pair_table<NW>(len_lo, len_hi, (uint16_t *)(smem + C::OFF_TBL), (uint32_t *)(smem + C::OFF_RED), lane, wave);
}

template <int MT, int N>
struct XPieces { u32x4 v[MT][N / 16]; };

// A operands for chunk kc: v[mt][q] = X[m][256 kc + 64 q + 16 g .. + 16) of lane (m = l % 16 (+ 16 mt), g = l / 16).
// Kernels that fetch X for every chunk fetch it as rows as they lie in memory, 16 lanes to a row (slot j of lane l: bytes 16 (l % 16) .. of row
// 4 j + l / 16 of each tile), and turn it into operands in LDS.  Fetched as operands, where adjacent lanes have different rows,
// every lane is an access to the first-level cache of its own, 64 for an instruction in place of 16, and those accesses bounded
// these kernels: 14336 x 7168, M = 64, 1400 of them a chunk, nine tenths of the time; 70.3 us -> 47.8, 16384 x 16384 145 -> 97.
// (The nibble plane fetched and turned in the same way: M = 1, 14336 x 7168 21.7 -> 24.4, the exchange of deal_plane is cheaper.)
// TURNED = false: slot j as the operand it is.  Rows from M on keep what they had: no output that is stored depends on them.
template <int MT, int N, bool TURNED, bool ALL = false>
__device__ __forceinline__ void load_x_slot(const GArgs &a, int lane, uint32_t kc, int j, XPieces<MT, N> &x)
{
    const uint32_t K = (uint32_t)a.K, row = TURNED ? lane >> 4 : lane & 15, at = row * K + (TURNED ? 16 * (lane & 15) : 16 * (lane >> 4));      // 64 K <= 2^26
#pragma unroll
    for (int mt = 0; mt < MT; mt++) {
        const uint32_t first = 16 * mt + (TURNED ? 4 * j : 0);      // row of X, of the instruction's lowest one
        const GLOBAL uint8_t *X = (const GLOBAL uint8_t *)a.d_x + (uint64_t)(first * K) + (uint64_t)kc * (4 * N) + (TURNED ? 0 : 64 * j);
        if constexpr (ALL) {
            const uint32_t last = a.M - 1, m = first + row < last ? first + row : last;
            x.v[mt][j] = *(const GLOBAL u32x4 *)((const GLOBAL uint8_t *)a.d_x + (uint64_t)kc * (4 * N) + (TURNED ? 0 : 64 * j) + (m * K + (TURNED ? 16 * (lane & 15) : 16 * (lane >> 4))));
        } else if (first + row < a.M) x.v[mt][j] = *(const GLOBAL u32x4 *)(X + at);
    }
}
// What a lane reads here others have written, and what it writes next others have read.  A wave's LDS operations are done in order; that the compiler
// leaves them in order is what `from` is for: it cannot tell that a lane reads other bytes than it writes.  (Fences in their place hold other
// work back as well: 14336 x 4096, F16 cores, M = 64 33.7 us -> 35.0, six experts M = 20 82.8 -> 84.4.)
template <int MT, int N>
__device__ __forceinline__ void turn_x(uint8_t *turn, int lane, XPieces<MT, N> &x)
{
    uint32_t from = (uint32_t)(lane & 15) * X_ROW + 16 * ((uint32_t)lane >> 4);
    asm("" : "+v"(from));
#pragma unroll
    for (int mt = 0; mt < MT; mt++) {
#pragma unroll
        for (int j = 0; j < N / 16; j++) *(u32x4 *)(turn + (4 * j + (lane >> 4)) * X_ROW + 16 * (lane & 15)) = x.v[mt][j];
#pragma unroll
        for (int q = 0; q < N / 16; q++) x.v[mt][q] = *(const u32x4 *)(turn + from + 64 * q);
    }
}

#define ECF8_MFMA_XPIECE(acc, xp, p, W_PIECE) ECF8_MFMA_OPERANDS(acc, xp.v[mt_][p], W_PIECE)

// Position of a wave in its sequence of chunks.  A unit is a block of 16 rows of W, or with split K one of the `slices` equal
// parts of its chunks.
struct Place {
    uint32_t b, kc;             // the workgroup's b-th unit, its kc-th chunk
    uint32_t block;             // the unit's block of rows
    uint32_t c;                 // the chunk's number in the blob (row-tiled blobs have at most 2^28)
};

// Chunks of a block whose share of X a wave keeps in registers for the whole matrix (0: it fetches X chunk by chunk).  One tile
// of X only: two chunks of it are 32 registers, and with more tiles or chunks they are not there.  Two pay from the second block of
// rows on; a workgroup with one (1024 x 7168, M = 16: 13.9 us) only waits longer for its first look-up (14.8).  Not on the F16 matrix cores
// (ACC = 1), where the converted operands beside them spill (14336 x 7168, M = 16: 45 us; fetched chunk by chunk 41).
template <int MT, int NW, int ACC>
__host__ __device__ inline uint32_t resident_chunks(uint64_t kchunks, uint64_t blocks)
{
    return MT != 1 ? 0u : kchunks <= NW ? 1u : ACC == 0 && kchunks <= 2 * NW && blocks > 1 ? 2u : 0u;
}

// The work of one workgroup on one matrix: its units first_unit, first_unit + unit_stride, ... (my_units of them), table
// set-up included.  At a block's end a wave parks its sum in LDS and goes on; the workgroup meets once per batch, as many
// blocks as there are slots for.  Which of a block's chunks are summed together (those PLACES apart) and in which order the sums are
// added does not depend on which wave has them, so every way below gives the same bits.
//  * KRES = 1, 2 (see resident_chunks): wave w has the chunks w, w + NW of every block and keeps their X; where a block has at
//    most NW / 2 chunks the waves form groups with a block each.  That leaves waves idle at times (28 chunks on 16 waves: an
//    eighth), which costs little beside the others' work.
//  * KRES = 0: the units' chunks form one sequence, and wave w takes every NW-th of it from the w-th on, across the units'
//    borders; batches are rounded down to whole rounds of the waves.
//  * PLACES != NW: the same with the chains of chunks that are summed together in place of chunks.  For the members of a group that have M <= 32 where another one
//    has more, so that they are computed as their own calls compute them; they also have two tiles of X in place of four (eight experts of M = 3 to 64 172.5 us ->
//    167.8, with scales of W 191.1 -> 187.6).
// What bounds it, eight experts of {2 x 2048 x 7168, 7168 x 2048}, scales of W: M = 4 (75.0 us), the compute unit: six of them, which the memory-side
// cache holds, take as long for a chunk (53.9 us, 449 clocks a chunk and compute unit against 454), and no unit of it is busy all of the time: vector
// operations 69 %, LDS 64 % (72 % of that bank conflicts of the table), first-level cache 62 %, address units 58 %; a wave waits for 53 % of its life.
// M = 64 (213 us): two waves on a SIMD, which is what four tiles of X leave room for, wait for look-ups and turned X in turn (LDS and
// first-level cache busy 55 % each).
template <int MT, int NW, int N, int SC, bool SPLIT, int ACC, bool APART, int KRES, bool TURNED = KRES == 0, int PLACES = NW, class CODES = TableInBlob>
__device__ __forceinline__ void anyk_walk(const GArgs &a, uint8_t *smem, uint32_t *s_flag, uint64_t first_unit, uint32_t unit_stride,
                                          uint32_t my_units, const CODES &codes = {})
{
    constexpr bool SCALED = SC != 0;
    using C = GCfg<MT, NW, N>;
    constexpr int BLOCK_COLS = C::BLOCK_COLS, GPIECES = C::PIECES;
    static_assert(!SCALED || 4 * N == 2 * SCALE_BLOCK, "a chunk spans two scale blocks of K");
    uint16_t *tbl = (uint16_t *)(smem + C::OFF_TBL);
    f32x4 *red = (f32x4 *)(smem + C::ANYK_OFF_RED);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = (int)uniform32((uint32_t)tid >> 6);           // the same for every lane: what follows from it stays in scalar registers
    uint8_t *turn = smem + C::OFF_TURN + wave * (16 * X_ROW);

    const GLOBAL uint8_t *stream = (const GLOBAL uint8_t *)(a.d_blob + a.off_st);
    const GLOBAL uint8_t *plane = (const GLOBAL uint8_t *)(a.d_blob + a.off_pl);
    const uint32_t kchunks = (uint32_t)(a.K / BLOCK_COLS), unit_chunks = a.unit_chunks;
    // split K: the grid is the units, each workgroup has one
    const uint32_t block0 = SPLIT ? (uint32_t)first_unit / a.slices : (uint32_t)first_unit;
    const uint32_t slice = SPLIT ? (uint32_t)first_unit - block0 * a.slices : 0u, k0 = slice * unit_chunks;

    using Meta = ChunkMeta<true>;
    const MetaReader<true> meta(a, lane);
    // NW chunks on: over at most this many units and so many chunks more
    constexpr bool CHAINS = PLACES != NW;
    static_assert(!CHAINS || (KRES == 0 && !SPLIT), "the ways that have chains");
    const uint32_t hop = a.hop, hop_kc = a.hop_kc;
    const uint32_t slots = unit_chunks < (uint32_t)PLACES ? unit_chunks : (uint32_t)PLACES;
    const uint32_t skip = (unit_stride - 1) * unit_chunks;         // the other workgroups' chunks between one unit and the next
    const uint32_t groups = a.groups, gi = small_div((uint32_t)wave, a.by_group), kw = (uint32_t)wave - gi * a.per_group;     // KRES
    const bool two = KRES && kw + NW < unit_chunks;
    auto first_place = [&]() {
        Place w;
        if constexpr (KRES != 0) {
            w.b = gi;
            w.kc = kw;
            if (kw >= unit_chunks || w.b >= groups) w.b = my_units;              // a wave with nothing to do
        } else {
            w.b = small_div((uint32_t)wave, a.by_unit);
            w.kc = (uint32_t)wave - w.b * (CHAINS ? slots : unit_chunks);
        }
        w.block = block0 + w.b * unit_stride;
        w.c = w.block * kchunks + k0 + w.kc;
        return w;
    };
    auto next_of = [&](Place w) {
        uint32_t kc, units;
        if constexpr (KRES != 0) {
            const bool over = w.kc + NW >= unit_chunks;
            units = over ? groups : 0u;
            kc = over ? kw : w.kc + NW;
            w.c += units * unit_stride * unit_chunks + kc - w.kc;
        } else if constexpr (CHAINS) {
            const bool over = w.kc + PLACES >= unit_chunks;        // the chain's last chunk: on to the chain NW further on
            const uint32_t to = w.kc % (uint32_t)PLACES + hop_kc;
            units = over ? hop + (to >= slots ? 1u : 0u) : 0u;
            kc = over ? (to >= slots ? to - slots : to) : w.kc + PLACES;
            w.c += units * unit_stride * unit_chunks + kc - w.kc;
        } else if constexpr (SPLIT) {                              // one unit
            const bool over = w.kc + NW >= unit_chunks;
            units = over ? 1u : 0u;
            kc = over ? 0u : w.kc + NW;
            w.c += NW;
        } else {
            const bool over = w.kc + hop_kc >= unit_chunks;
            units = hop + (over ? 1u : 0u);
            kc = over ? w.kc + hop_kc - unit_chunks : w.kc + hop_kc;
            w.c += NW + units * skip;
        }
        w.kc = kc;
        w.b += units;
        w.block += units * unit_stride;
        return w;
    };
    auto valid = [&](const Place &w) { return w.b < my_units; };
    auto load_meta = [&](const Place &w) { return meta(w.c); };
    // nibble plane of a chunk: this lane's part of pieces q and q + 2 at plane_of(w) + lane_plane + 32 q, see deal_plane.  Block and column of chunk c begin at
    // element 256 * (16 * block * kchunks + k), k = c - block * kchunks.
    const uint32_t lane_plane = (uint32_t)(lane & 15) * (uint32_t)(a.K / 2) + plane_lane(lane);
    auto plane_of = [&](const Place &w) -> const GLOBAL uint8_t * {
        return plane + ((uint64_t)(16 * w.c - 15 * (k0 + w.kc)) << 7);
    };

    // The first chunk's X without a condition, see load_x_slice, where that pays: resident X and single products of one tile or four.  With / without, us:
    // 14336 x 7168 M = 16 24.4 / 24.9, 512 x 2048 M = 16 6.0 / 6.2, two experts M = 4 24.4 / 24.8; but eight experts M = 20 with scales of W 122.8 / 120.2, split K 1024 x 7168
    // M = 16 10.4 / 10.2.
    constexpr bool FIRST_ALL = KRES != 0 || (!SPLIT && !APART && MT != 2);
    auto load_x = [&](uint32_t kc, XPieces<MT, N> &x) {
#pragma unroll
        for (int j = 0; j < GPIECES; j++) load_x_slot<MT, N, TURNED, FIRST_ALL>(a, lane, kc, j, x);
    };
    Place cur = first_place();
    Meta m_cur, m_next;
    RawRuns raw = {};
    static_assert(GPIECES == 4, "deal_plane");
    u32x4 pl[2];
#pragma unroll
    for (int q = 0; q < 2; q++) pl[q] = u32x4{0, 0, 0, 0};
    XPieces<MT, N> x_cur[KRES > 1 ? KRES : 1] = {};
    // The order of ecf8_gemm_kernel, but not in groups with two tiles of X or four and no scales.  Metadata first / this order, us: six
    // experts M = 20 81.8 / 82.9, 48 121 / 124, eight experts M = 64 192 / 200; with scales of W no difference.
    constexpr bool EARLY = !(APART && MT > 1 && SC == 0);
    u32x4 tv[TABLE_UNITS<NW>];
    constexpr bool IN_BLOB = !APART && std::is_same<CODES, TableInBlob>::value;       // APART: known for each matrix of the group
    uint32_t codes_two = 0;
    if constexpr (IN_BLOB) load_table<NW>(a, tid, tv);
    else if constexpr (!APART) {
        if (wave == 0) codes_two = codes.two[lane];
    } else if (EARLY) load_table<NW>(a, tid, tv);
    if (valid(cur)) {
        m_cur = load_meta(cur);
        const Place nxt = next_of(cur);
        m_next = meta(valid(nxt) ? nxt.c : cur.c);      // a copy of m_cur would wait for it, in front of everything below
        if constexpr (!EARLY) raw.fetch(stream, a.st_bytes, m_cur, lane);
        const GLOBAL uint8_t *pp = plane_of(cur);
#pragma unroll
        for (int q = 0; q < 2; q++) pl[q] = *(const GLOBAL u32x4 *)(pp + 32 * q + lane_plane);
        load_x(k0 + cur.kc, x_cur[0]);
    }
    if constexpr (EARLY) {
        if (valid(cur)) raw.fetch(stream, a.st_bytes, m_cur, lane);
    }
    if constexpr (KRES > 1) load_x(two ? kw + NW : kw, x_cur[1]);

    if constexpr (IN_BLOB) {
        if (a.off_tbl) store_table<NW>(tbl, tid, tv);
    } else if constexpr (!APART) {
        build_pair_table<NW>(codes_two, tbl, (uint32_t *)(smem + C::OFF_RED), lane, wave);
    } else if (a.off_tbl) {
        if constexpr (!EARLY) load_table<NW>(a, tid, tv);
        store_table<NW>(tbl, tid, tv);
    } else {
        uint64_t len_lo, len_hi;
        __builtin_memcpy(&len_lo, a.code_len, 8);
        __builtin_memcpy(&len_hi, a.code_len + 8, 8);
        build_pair_table_apart<NW>(len_lo, len_hi, smem, lane, wave);
    }

    const uint32_t batch = SPLIT ? 1u : a.batch;

    // Waves with a piece decoded go first while they multiply it, with two tiles of X and group scales, in groups also with scales of W.  Group scales, eight experts
    // M = 32 139.5 us -> 135.3; 14336 x 9216 M = 17 / 32 44.8 / 55.2 -> 43.6 / 52.2, 2048 x 7168 10.95 / 11.83 -> 11.04 / 11.70.  Scales of W, eight experts M = 20 / 32 118.1 /
    // 132.4 -> 118.3 / 126.4, single products within 2 % either way.  Without scales: eight experts M = 20 110.8 -> 113.2, 4096 x 14336 16.6 -> 16.8, 14336 x 4096 on the F16
    // cores 22.7 -> 23.6.  Four tiles and group scales: two experts M = 64 59.2 -> 57.3, but four of M = 33 97.5 -> 98.7.
    constexpr bool PRIO = MT == 2 && !SPLIT && (SC == 2 || (APART && SC == 1));
    f32x4 acc[MT];
    auto clear = [&]() {
#pragma unroll
        for (int mt = 0; mt < MT; mt++) acc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    // One chunk: decoded and multiplied by x; the wave's next one is fetched meanwhile.  KRES = 0: x are its rows, turned just before the first
    // product, and its registers take the next chunk's rows as they are used up.
    auto chunk = [&](XPieces<MT, N> &x) {
        ShiftedRuns runs;
        runs.begin(raw);
        ChunkSums<MT, SC> sums;
        sums.begin(a, cur.block, k0 + cur.kc);
        // The raw registers are free: fetch the next chunk's runs, and the metadata of the chunk after it.
        const Place nxt = next_of(cur);
        const bool more = valid(nxt);
        Meta m_next2 = m_next;
        if (more) {
            raw.fetch(stream, a.st_bytes, m_next, lane);
            const Place nxt2 = next_of(nxt);
            if (valid(nxt2)) m_next2 = load_meta(nxt2);
        }
        // Two tiles of X and scales in groups: where a lane reads X is worked out again for every chunk; kept for the whole walk, it
        // costs a spill.
        uint32_t x_lane = (uint32_t)lane;
        if constexpr (APART && MT == 2 && SC != 0) asm("" : "+v"(x_lane));
        // after the last chunk the plane pieces are fetched from the plane's first chunk (every wave's last fetch: cached)
        const GLOBAL uint8_t *pp = more ? plane_of(nxt) : plane;
        auto &dstA = sums.first(acc);
        auto &dstB = sums.second(acc);
#pragma unroll
        for (int Q = 0; Q < GPIECES / 2; Q++) {
            uint32_t dwA[4], dwB[4];
#pragma unroll
            for (int t = 0; t < 4; t++) runs.step(tbl, 4 * Q + t, dwA[t], dwB[t]);
            // two pieces of the nibble plane are merged, and their registers take the same pieces of the next chunk
            u32x2 pA, pB;
            deal_plane(pl[Q], pA, pB);
            pl[Q] = *(const GLOBAL u32x4 *)(pp + 32 * Q + lane_plane);
            if (TURNED && Q == 0) turn_x<MT, N>(turn, lane, x);
            if constexpr (PRIO) __builtin_amdgcn_s_setprio(1);
            const u32x4 wA = merge_piece(dwA, pA);
            ECF8_MFMA_XPIECE(dstA, x, Q, wA);
            const u32x4 wB = merge_piece(dwB, pB);
            ECF8_MFMA_XPIECE(dstB, x, Q + GPIECES / 2, wB);
            if constexpr (PRIO) __builtin_amdgcn_s_setprio(0);
            if (KRES == 0 && more) {
                load_x_slot<MT, N, TURNED>(a, (int)x_lane, k0 + nxt.kc, Q, x);
                load_x_slot<MT, N, TURNED>(a, (int)x_lane, k0 + nxt.kc, Q + GPIECES / 2, x);
            }
        }
        sums.end(acc, a, lane);
        m_next = m_next2;
        return nxt;
    };
    auto park = [&](uint32_t j, uint32_t place) {                  // the wave's last chunk of the batch's j-th block is done
        f32x4 *slot = red + (j * slots + place) * (MT * 64) + lane;
#pragma unroll
        for (int mt = 0; mt < MT; mt++) slot[mt * 64] = acc[mt];
    };
    clear();
    for (uint32_t b0 = 0; b0 < my_units; b0 += batch) {            // uniform for the workgroup: its barriers
        const uint32_t b1 = my_units - b0 < batch ? my_units : b0 + batch;
        if constexpr (KRES != 0) {
            while (cur.b < b1) {
                const uint32_t j = cur.b - b0, place = cur.kc;
                clear();
                cur = chunk(x_cur[0]);
                if (KRES > 1 && two) cur = chunk(x_cur[KRES - 1]);
                park(j, place);
            }
        } else {
#pragma unroll 1
            while (cur.b < b1) {
                const Place nxt = chunk(x_cur[0]);
                if (CHAINS ? cur.kc + PLACES >= unit_chunks : !SPLIT && nxt.b != cur.b) {
                    park(cur.b - b0, cur.kc % (uint32_t)PLACES);
                    clear();
                }
                cur = nxt;
            }
        }
        if constexpr (SPLIT) {
            reduce_split<MT, NW, SCALED>(red, s_flag, a, block0, slice, tid, acc);
        } else {
            __syncthreads();
            reduce_batch<MT, NW, PLACES, SCALED>(red, a, first_unit + (uint64_t)b0 * unit_stride, unit_stride, b1 - b0, slots, tid);
            if (b1 < my_units) __syncthreads();                    // the slots are free again
        }
    }
}

template <class CODES, int MT, int NW, int N, int SC, bool SPLIT = false, int ACC = 0, int KRES = 0, bool TURNED = KRES == 0>
__global__ __launch_bounds__(NW * 64) void ecf8_gemm_anyk_kernel(GArgs a, CODES codes)
{
    __shared__ __attribute__((aligned(16))) uint8_t smem[GCfg<MT, NW, N>::ANYK_TOTAL];
    __shared__ uint32_t s_flag;                   // split K: the arrival count this workgroup drew
    anyk_walk<MT, NW, N, SC, SPLIT, ACC, false, KRES, TURNED, NW, CODES>(a, smem, &s_flag, blockIdx.x, gridDim.x, a.units_each + (blockIdx.x < a.units_rest ? 1u : 0u), codes);
}

// Position of a wave in its sequence of chunks of uncompressed W: its i-th chunk of its workgroup's b-th unit.  `block` is the
// unit's block of rows, k0 its first chunk.
struct Walk {
    uint32_t b;
    uint32_t i;
    uint32_t block;
    uint32_t k0;
};

// The any-K GEMM on uncompressed W: same deal of chunks, same order of accumulation.
template <int MT, int NW, int N, int SC, bool SPLIT, int ACC = 0, int PLACES = NW>
__device__ __forceinline__ void raw_anyk_walk(const GArgs &a, uint8_t *smem, uint32_t *s_flag, uint32_t first_unit, uint32_t unit_stride,
                                              uint32_t my_units, uint32_t &parity)
{
    constexpr bool SCALED = SC != 0;
    using C = GCfg<MT, NW, N>;
    constexpr int BLOCK_COLS = C::BLOCK_COLS, GPIECES = C::PIECES;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const GLOBAL uint8_t *W = (const GLOBAL uint8_t *)a.d_w;
    const uint64_t lane_elem = (uint64_t)(lane & 15) * a.K + (uint64_t)(lane >> 4) * 16;
    const uint32_t kchunks = (uint32_t)(a.K / BLOCK_COLS);
    const uint32_t unit_chunks = SPLIT ? kchunks / a.slices : kchunks;
    Deal deal = deal_chunks<NW>(a, SPLIT, wave);
    // sums of PLACES places with fewer waves: a wave has the places kw and kw + NW, one behind the other
    static_assert(PLACES == NW || (PLACES < 2 * NW && !SPLIT), "two places a wave");
    const bool chains = PLACES != NW && unit_chunks > (uint32_t)NW;
    const uint32_t second = deal.kw + NW;
    uint32_t in_first = deal.my_chunks;
    if (chains) {
        in_first = (unit_chunks - deal.kw + PLACES - 1) / PLACES;
        deal.my_chunks = in_first + (second < PLACES && second < unit_chunks ? (unit_chunks - second + PLACES - 1) / PLACES : 0u);
    }
    const uint32_t my_chunks = deal.my_chunks;
    uint32_t my_blocks = my_units;
    if (!SPLIT && deal.groups > 1) my_blocks = (my_units + deal.groups - 1) / deal.groups;
    auto at_unit = [&](uint32_t b) {
        Walk w{b, 0, first_unit + (b * deal.groups + deal.gi) * unit_stride, 0};
        if constexpr (SPLIT) {
            const uint32_t u = w.block;
            w.block = u / a.slices;
            w.k0 = (u % a.slices) * unit_chunks;
        }
        return w;
    };
    auto block_of = [&](const Walk &w) -> uint64_t { return w.block; };
    auto kc_of = [&](const Walk &w) -> uint32_t {
        if (chains) return w.i < in_first ? deal.kw + PLACES * w.i : second + PLACES * (w.i - in_first);
        return w.k0 + deal.kw + deal.wpb * w.i;
    };
    auto valid = [&](const Walk &w) { return my_chunks != 0 && w.b * deal.groups + deal.gi < my_units; };
    auto next_of = [&](Walk w) { if (++w.i == my_chunks) w = at_unit(w.b + 1); return w; };
    auto load_w = [&](const Walk &w, u32x4 (&v)[GPIECES]) {
        const uint64_t e0 = block_of(w) * BLOCK_ROWS * a.K + kc_of(w) * (uint64_t)BLOCK_COLS + lane_elem;
#pragma unroll
        for (int q = 0; q < GPIECES; q++) v[q] = __builtin_nontemporal_load((const GLOBAL u32x4 *)(W + e0 + 64 * q));
    };
    Walk cur = at_unit(0);
    u32x4 w_cur[GPIECES], w_next[GPIECES];
    XPieces<MT, N> x_cur = {};
    if (valid(cur)) {
        load_w(cur, w_cur);
#pragma unroll
        for (int j = 0; j < GPIECES; j++) load_x_slot<MT, N, false>(a, lane, kc_of(cur), j, x_cur);
    }
    for (uint32_t b = 0; b < my_blocks; b++) {
        f32x4 *red = (f32x4 *)(smem + parity * (PLACES * MT * 1024));
        f32x4 acc[MT];
#pragma unroll
        for (int mt = 0; mt < MT; mt++) acc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
        auto park = [&](uint32_t place) {
#pragma unroll
            for (int mt = 0; mt < MT; mt++) red[(place * MT + mt) * 64 + lane] = acc[mt];
        };
        const uint32_t n_mine = valid(at_unit(b)) ? my_chunks : 0;
#pragma unroll 1
        for (uint32_t i = 0; i < n_mine; i++) {
            if (PLACES != NW && chains && i == in_first) {
                park(deal.kw);
#pragma unroll
                for (int mt = 0; mt < MT; mt++) acc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
            const XPieces<MT, N> x = x_cur;
            ChunkSums<MT, SC> sums;
            sums.begin(a, block_of(cur), kc_of(cur));
            const Walk nxt = next_of(cur);
#pragma unroll
            for (int q = 0; q < GPIECES; q++) w_next[q] = w_cur[q];
            if (valid(nxt)) {
                load_w(nxt, w_next);
#pragma unroll
                for (int j = 0; j < GPIECES; j++) load_x_slot<MT, N, false>(a, lane, kc_of(nxt), j, x_cur);
            }
            auto &dstA = sums.first(acc);
            auto &dstB = sums.second(acc);
#pragma unroll
            for (int Q = 0; Q < GPIECES / 2; Q++) {
                ECF8_MFMA_XPIECE(dstA, x, Q, w_cur[Q]);
                ECF8_MFMA_XPIECE(dstB, x, Q + GPIECES / 2, w_cur[Q + GPIECES / 2]);
            }
            sums.end(acc, a, lane);
#pragma unroll
            for (int q = 0; q < GPIECES; q++) w_cur[q] = w_next[q];
            cur = nxt;
        }
        const Walk unit = at_unit(b);
        if constexpr (SPLIT) reduce_split<MT, NW, SCALED>(red, s_flag, a, unit.block, unit.k0 / unit_chunks, tid, acc);
        else if (PLACES != NW && chains) {
            park(my_chunks > in_first ? second : deal.kw);
            __syncthreads();
            reduce_batch<MT, NW, PLACES, SCALED>(red, a, first_unit + b * unit_stride, 1, 1, unit_chunks < (uint32_t)PLACES ? unit_chunks : (uint32_t)PLACES, tid);
        } else reduce_groups<MT, NW, SCALED>(red, a, first_unit, unit_stride, b * deal.groups, my_units, deal, tid, acc);
        parity ^= 1;
    }
}

template <int MT, int NW, int N, int SC, bool SPLIT = false, int ACC = 0>
__global__ __launch_bounds__(NW * 64) void ecf8_gemm_raw_anyk_kernel(GArgs a)
{
    __shared__ __attribute__((aligned(16))) uint8_t smem[2 * GCfg<MT, NW, N>::RED_BYTES];
    __shared__ uint32_t s_flag;
    uint32_t parity = 0;
    raw_anyk_walk<MT, NW, N, SC, SPLIT, ACC>(a, smem, &s_flag, blockIdx.x, gridDim.x, a.units_each + (blockIdx.x < a.units_rest ? 1u : 0u), parity);
}

// ---- a group of matrices in one launch ----
// Many small products at once, each with its own W, X, M and Y (the experts a batch of tokens is
// routed to): a launch per matrix would be bound by launches and would leave the chip half empty
// (a 2048 x 7168 expert has 128 blocks of rows).  The blocks of all matrices form one sequence,
// weighted by their K / 256 chunks; every workgroup takes an equal share of it, a contiguous run
// of blocks that may cross from one matrix into the next, and works through it with the any-K loop,
// setting up the code again where the matrix changes.  Inside a block nothing differs from the
// single call with the same number of waves, so the results are the same bit for bit.
struct GItem {
    uint64_t first_work;        // chunks of the matrices before this one
    GArgs a;
};
static_assert(sizeof(GItem) % 8 == 0 && sizeof(GItem) <= sizeof(ecf8_gemm_group_item), "item fits its public slot");

struct GGArgs {
    uint64_t d_items;           // device array of ecf8_gemm_group_item
    uint64_t base;              // chunks of the group before this launch's (launch_grouped): what the kernel counts from, in 32 bits
    uint32_t n_items;
    uint32_t work_each, work_rest;      // chunks of every workgroup; the first work_rest have one more
};

template <int MT, int NW, int N, int SC, bool RAW>
__global__ __launch_bounds__(NW * 64) void ecf8_gemm_grouped_kernel(GGArgs g)
{
    using C = GCfg<MT, NW, N>;
    __shared__ __attribute__((aligned(16))) uint8_t smem[RAW ? 2 * C::RED_BYTES : C::ANYK_TOTAL];
    __shared__ uint32_t s_flag;
    constexpr uint32_t WORDS = sizeof(ecf8_gemm_group_item) / 8;
    const GLOBAL uint64_t *items = (const GLOBAL uint64_t *)g.d_items;
    // this workgroup takes the blocks whose first chunk lies in [pos, end) of the sequence
    uint32_t pos = g.work_each * blockIdx.x + (blockIdx.x < g.work_rest ? blockIdx.x : g.work_rest);
    const uint32_t end = pos + g.work_each + (blockIdx.x < g.work_rest ? 1u : 0u);
    uint32_t parity = 0;
    // The matrix that holds pos: lane l probes the l-th of 64 evenly spaced items, one round trip to memory for up to 64 of
    // them (a binary search took five for 24, at the start and again wherever a share crosses into the next matrix, which is
    // simply the next item).
    uint32_t lo = 0;
    for (uint32_t n = g.n_items; n > 1;) {
        const uint32_t step = (n + 63) / 64, at = (threadIdx.x & 63) * step;
        const bool begun = at < n && items[(uint64_t)(lo + (at < n ? at : 0u)) * WORDS] <= g.base + pos;
        const uint32_t k = ((uint32_t)__popcll(__ballot(begun)) - 1u) * step;       // the first one has begun
        lo += k;
        n = n - k < step ? n - k : step;
    }
    for (; pos < end; lo++) {                           // one round per matrix the share touches (uniform)
        GItem it;
        {
            uint64_t *dst = (uint64_t *)&it;
#pragma unroll
            for (int i = 0; i < (int)(sizeof(GItem) / 8); i++) dst[i] = uniform64(items[(uint64_t)lo * WORDS + i]);
        }
        const uint32_t kchunks = (uint32_t)(it.a.K / C::BLOCK_COLS), n_blocks = (uint32_t)(it.a.rows / BLOCK_ROWS), first_work = (uint32_t)(it.first_work - g.base);
        const uint32_t b0 = (pos - first_work + kchunks - 1) / kchunks;
        uint32_t b1 = (end - first_work + kchunks - 1) / kchunks;
        if (b1 > n_blocks) b1 = n_blocks;
        __syncthreads();                                // the last matrix's table and reduction buffers are out of use
        if (b0 < b1) {
            if constexpr (RAW) {
                if (MT == 4 && it.a.M <= 32) raw_anyk_walk<(MT == 4 ? 2 : MT), NW, N, SC, false, 0, (MT == 4 ? WAVES<2> : NW)>(it.a, smem, &s_flag, b0, 1, b1 - b0, parity);
                else raw_anyk_walk<MT, NW, N, SC, false>(it.a, smem, &s_flag, b0, 1, b1 - b0, parity);
            }
            else {
                // One tile of X that is fetched chunk by chunk (K > 8192, or one block) is fetched as operands, whatever its rows: one walk serves all M <= 16,
                // and with scales of W the turned one is mostly the slower one.  Operands / turned, us, M = 1 / 9 / 16: three 4096 x 14336 37.3 / 40.6 / 46.4, 40.0 / 41.1 / 42.4, scaled
                // 39.1 / 41.4 / 47.5, 45.2 / 47.6 / 48.9; two 1024 x 9216 12.1 / 12.8 / 14.0, 12.7 / 12.9 / 13.1, scaled 12.4 / 13.0 / 14.4, 15.3 / 15.9 / 16.3; two
                // 14336 x 9216 48.7 / 52.7 / 68.7, 53.4 / 55.0 / 57.3, scaled 49.9 / 58.8 / 69.8, 58.4 / 61.1 / 63.1.
                const uint32_t n = b1 - b0, kres = resident_chunks<MT, NW, 0>(kchunks, n);
                if constexpr (MT == 4) {
                    if (it.a.M <= 32) {
                        anyk_walk<2, NW, N, SC, false, 0, true, 0, true, WAVES<2>>(it.a, smem, &s_flag, b0, 1, n);
                        pos = first_work + n_blocks * kchunks;
                        continue;
                    }
                }
                if (MT == 1 && kres == 1) anyk_walk<MT, NW, N, SC, false, 0, true, MT == 1>(it.a, smem, &s_flag, b0, 1, n);
                else if (MT == 1 && kres == 2) anyk_walk<MT, NW, N, SC, false, 0, true, MT == 1 ? 2 : 0>(it.a, smem, &s_flag, b0, 1, n);
                else anyk_walk<MT, NW, N, SC, false, 0, true, 0, (MT > 1)>(it.a, smem, &s_flag, b0, 1, n);
            }
        }
        pos = first_work + n_blocks * kchunks;          // on to the next matrix (or past `end`)
    }
}

inline int grid_for(uint64_t n_blocks)
{
    int cus = device_cus();
    if (cus <= 0) return -1;
    return (int)(n_blocks < (uint64_t)cus ? n_blocks : (uint64_t)cus);
}

inline int check_gemm_args(uint64_t rows, uint64_t cols, const void *d_x, uint32_t M, const void *d_y)
{
    if (!d_x || !d_y || M == 0 || M > 64) return ECF8_E_ARG;
    if (cols == 0 || cols % 256 || cols > (1u << 20) || rows == 0 || rows % BLOCK_ROWS) return ECF8_E_ARG;
    if (rows / BLOCK_ROWS > LAUNCH_CHUNKS / (cols / 256)) return ECF8_E_ARG;         // 8 TiB
    if (((uintptr_t)d_x & 15) || ((uintptr_t)d_y & 3)) return ECF8_E_ALIGN;
    return ECF8_OK;
}

// Checks of the fused call's blob; fills the kernel arguments.
inline int fused_args(const ecf8_header *h, const void *d_blob, const void *d_x, uint32_t M, float *d_y, GArgs *out)
{
    if (!h || !d_blob) return ECF8_E_ARG;
    if (h->magic != ECF8_MAGIC || h->version != ECF8_VERSION || (h->table_bits != 0 && h->table_bits != ECF8_TB))
        return ECF8_E_FORMAT;
    uint32_t max_len = 0;
    for (int i = 0; i < 16; i++) max_len = h->code_len[i] > max_len ? h->code_len[i] : max_len;
    // row-tiled blob of 16 x 256 chunks, every pair of codewords one table hit
    if (h->lane_syms != 64 || h->tile_rows != BLOCK_ROWS || h->group_chunks != 1 || max_len == 0 ||
        2 * max_len > (uint32_t)TB)
        return ECF8_E_ARG;
    int rc = check_gemm_args(h->rows, h->cols, d_x, M, d_y);
    if (rc) return rc;
    if (h->n_elem != h->rows * h->cols || h->n_chunks != h->n_elem / (64ull * h->lane_syms)) return ECF8_E_FORMAT;
    if (h->off_plane + h->plane_bytes > h->total_size || h->off_stream + h->stream_bytes > h->off_plane ||
        h->plane_bytes != h->n_elem / 2)
        return ECF8_E_FORMAT;
    if ((uintptr_t)d_blob & 15) return ECF8_E_ALIGN;
    GArgs a{};
    a.d_blob = (uint64_t)(uintptr_t)d_blob;
    a.d_x = (uint64_t)(uintptr_t)d_x;
    a.d_y = (uint64_t)(uintptr_t)d_y;
    a.rows = h->rows;
    a.off_cb = h->off_chunk_bit;
    a.off_lb = h->off_lane_bits;
    a.off_st = h->off_stream;
    a.off_pl = h->off_plane;
    a.st_bytes = h->stream_bytes;
    a.off_tbl = h->table_bits ? 256 : 0;
    for (int i = 0; i < 16; i++) a.code_len[i] = h->code_len[i];
    a.M = M;
    a.K = h->cols;
    *out = a;
    return ECF8_OK;
}

inline int raw_args(const void *d_w, uint64_t rows, uint64_t cols, const void *d_x, uint32_t M, float *d_y, GArgs *out)
{
    if (!d_w) return ECF8_E_ARG;
    int rc = check_gemm_args(rows, cols, d_x, M, d_y);
    if (rc) return rc;
    if ((uintptr_t)d_w & 15) return ECF8_E_ALIGN;
    GArgs a{};
    a.d_w = (uint64_t)(uintptr_t)d_w;
    a.d_x = (uint64_t)(uintptr_t)d_x;
    a.d_y = (uint64_t)(uintptr_t)d_y;
    a.rows = rows;
    a.M = M;
    a.K = cols;
    *out = a;
    return ECF8_OK;
}

inline int scale_args(const float *d_w_scale, const float *d_x_scale, uint32_t x_scale_cols, GArgs *a)
{
    if (!d_w_scale) return ECF8_E_ARG;
    if (d_x_scale ? (x_scale_cols != 1 && x_scale_cols != a->K / SCALE_BLOCK) : x_scale_cols != 0) return ECF8_E_ARG;
    a->xs_cols = x_scale_cols;
    if (((uintptr_t)d_w_scale & 3) || ((uintptr_t)d_x_scale & 3)) return ECF8_E_ALIGN;
    a->d_ws = (uint64_t)(uintptr_t)d_w_scale;
    a->d_xs = (uint64_t)(uintptr_t)d_x_scale;
    return ECF8_OK;
}

// What the fused kernels' deals divide: the units among the grid's workgroups, a unit's chunks among a workgroup's NW waves with MT tiles of 16 rows of X.
inline void deal_units(GArgs *a, uint32_t grid)
{
    const uint32_t units = (uint32_t)(a->rows / BLOCK_ROWS) * (a->slices ? a->slices : 1u);
    a->units_each = units / grid;
    a->units_rest = units % grid;
}
template <int MT, int NW = WAVES<MT>, int PLACES = NW>
void deal_waves(GArgs *a)
{
    const uint32_t slices = a->slices ? a->slices : 1u, chunks = (uint32_t)(a->K / 256) / slices;
    const uint32_t slots = chunks < (uint32_t)PLACES ? chunks : (uint32_t)PLACES, dealt = PLACES == NW ? chunks : slots;     // see anyk_walk
    a->unit_chunks = chunks;
    a->hop = NW / dealt;
    a->hop_kc = NW % dealt;
    a->groups = slices == 1 && 2 * chunks <= (uint32_t)NW ? NW / chunks : 1u;
    a->per_group = NW / a->groups;
    a->by_unit = small_by(dealt);
    a->by_group = small_by(a->per_group);
    // blocks of a batch: whole rounds of the waves where there are slots for them
    const uint32_t whole = (uint32_t)NW / std::gcd((uint32_t)NW, dealt);
    a->batch = GCfg<MT, NW, 64>::SLOTS / slots;
    if (a->batch >= whole) a->batch -= a->batch % whole;
}
// Of a call whose largest M is max_M
inline void deal_waves(GArgs *a, uint32_t max_M)
{
    if (max_M <= 16) deal_waves<1>(a);
    else if (max_M <= 32) deal_waves<2>(a);
    else if (a->M <= 32) deal_waves<2, WAVES<4>, WAVES<2>>(a);
    else deal_waves<4>(a);
}

// 16 waves (one K chunk of the block each) while X fits their registers, 8 waves of two chunks
// at M > 32.
// CODES: kernels of their own where the blob holds the table and where they build it.
template <int SCALED, int ACC, class CODES>
int launch_fused_with(const GArgs &a, const CODES &codes, int grid, hipStream_t s)
{
    // The any-K kernels also take K = 4096 where X does not fit the registers beside the rest: with a scale per row and 128 columns of X at M > 32,
    // and on the F16 matrix cores, whose operands are converted, at M > 16.  Resident X / any K, us, rows 4096, 14336 and 28672: group scales M = 33 30.9 / 11.7,
    // 69.6 / 35.2, 111 / 57.9, M = 64 37.5 / 13.2, 90.7 / 39.1, 146 / 64.5; F16 cores M = 33 27.2 / 11.1, 59.6 / 32.4, 95.0 / 53.7, M = 64 30.6 / 12.2, 63.4 / 34.0, 99.4 / 56.1.
    // F16 cores at M = 17 .. 32 go with those, though there X does fit and many rows would be faster for it: M = 32 10.7 / 9.0, 20.4 / 25.0, 29.6 / 41.0.
    if (a.K != GK || (SCALED == 2 && a.M > 32) || (ACC == 1 && a.M > 16)) {
        const uint32_t kres = a.M <= 16 ? resident_chunks<1, WAVES<1>, ACC>(a.K / 256, a.rows / BLOCK_ROWS / (uint64_t)grid) : 0u;
        if (kres == 1) hipLaunchKernelGGL((ecf8_gemm_anyk_kernel<CODES, 1, WAVES<1>, 64, SCALED, false, ACC, 1>), dim3(grid), dim3(WAVES<1> * 64), 0, s, a, codes);
        else if (kres == 2) hipLaunchKernelGGL((ecf8_gemm_anyk_kernel<CODES, 1, WAVES<1>, 64, SCALED, false, ACC, ACC == 0 ? 2 : 0>), dim3(grid), dim3(WAVES<1> * 64), 0, s, a, codes);
        // a few rows of X are few accesses either way, and the turn is time.  Operands / turned, us, M = 1 / 4 / 8 / 12 / 16: 4096 x 14336
        // 14.1 / 14.7 / 15.4 / 16.2 / 16.8, 15.3 / 15.5 / 15.4 / 15.4 / 15.4; 14336 x 9216 29.7 / 29.9 / 31.3 / 33.0 / 35.4, 32.4 for all
        else if (a.M <= 8) hipLaunchKernelGGL((ecf8_gemm_anyk_kernel<CODES, 1, WAVES<1>, 64, SCALED, false, ACC, 0, false>), dim3(grid), dim3(WAVES<1> * 64), 0, s, a, codes);
        else if (a.M <= 16) hipLaunchKernelGGL((ecf8_gemm_anyk_kernel<CODES, 1, WAVES<1>, 64, SCALED, false, ACC>), dim3(grid), dim3(WAVES<1> * 64), 0, s, a, codes);
        else if (a.M <= 32) hipLaunchKernelGGL((ecf8_gemm_anyk_kernel<CODES, 2, WAVES<2>, 64, SCALED, false, ACC>), dim3(grid), dim3(WAVES<2> * 64), 0, s, a, codes);
        else hipLaunchKernelGGL((ecf8_gemm_anyk_kernel<CODES, 4, WAVES<4>, 64, SCALED, false, ACC>), dim3(grid), dim3(WAVES<4> * 64), 0, s, a, codes);
        return hipGetLastError() == hipSuccess ? ECF8_OK : ECF8_E_HIP;
    }
    if (a.M <= 16) hipLaunchKernelGGL((ecf8_gemm_kernel<1, 16, 64, SCALED, ACC, CODES>), dim3(grid), dim3(16 * 64), 0, s, a, codes);
    else if constexpr (ACC == 0) {
        if (a.M <= 32) hipLaunchKernelGGL((ecf8_gemm_kernel<2, 16, 64, SCALED, ACC, CODES>), dim3(grid), dim3(16 * 64), 0, s, a, codes);
        else if constexpr (SCALED != 2) hipLaunchKernelGGL((ecf8_gemm_kernel<4, 8, 64, SCALED, ACC, CODES>), dim3(grid), dim3(8 * 64), 0, s, a, codes);
    }
    return hipGetLastError() == hipSuccess ? ECF8_OK : ECF8_E_HIP;
}

template <int SCALED, int ACC = 0>
int launch_fused(GArgs a, void *stream)
{
    const int grid = grid_for(a.rows / BLOCK_ROWS);
    if (grid <= 0) return ECF8_E_HIP;
    a.slices = 1;
    deal_units(&a, (uint32_t)grid);
    deal_waves(&a, a.M);
    return a.off_tbl ? launch_fused_with<SCALED, ACC>(a, TableInBlob{}, grid, (hipStream_t)stream)
                     : launch_fused_with<SCALED, ACC>(a, short_codes(a.code_len), grid, (hipStream_t)stream);
}

template <int SCALED, int ACC = 0>
int launch_raw(GArgs a, void *stream)
{
    const int grid = grid_for(a.rows / BLOCK_ROWS);
    if (grid <= 0) return ECF8_E_HIP;
    a.slices = 1;
    deal_units(&a, (uint32_t)grid);
    // Two tiles of X and at most 8 chunks of a block: 8 waves, which have as many places as the fused call's.  8 / 12 waves, us, M = 17: 16384 x 512 5.95 / 6.01, with
    // scales of W 6.47 / 6.75; 512 x 2048 6.49 / 6.65
    const bool few = a.M > 16 && a.M <= 32 && a.K <= 8 * 256;
    if (few) deal_waves<2, 8>(&a);
    else deal_waves(&a, a.M);
    hipStream_t s = (hipStream_t)stream;
    if (a.K != GK || (SCALED == 2 && a.M > 32) || (ACC == 1 && a.M > 16)) {      // the same routes as the fused call: same order of accumulation
        if (a.M <= 16) hipLaunchKernelGGL((ecf8_gemm_raw_anyk_kernel<1, WAVES<1>, 64, SCALED, false, ACC>), dim3(grid), dim3(WAVES<1> * 64), 0, s, a);
        else if (few) hipLaunchKernelGGL((ecf8_gemm_raw_anyk_kernel<2, 8, 64, SCALED, false, ACC>), dim3(grid), dim3(8 * 64), 0, s, a);
        else if (a.M <= 32) hipLaunchKernelGGL((ecf8_gemm_raw_anyk_kernel<2, WAVES<2>, 64, SCALED, false, ACC>), dim3(grid), dim3(WAVES<2> * 64), 0, s, a);
        else hipLaunchKernelGGL((ecf8_gemm_raw_anyk_kernel<4, WAVES<4>, 64, SCALED, false, ACC>), dim3(grid), dim3(WAVES<4> * 64), 0, s, a);
        return hipGetLastError() == hipSuccess ? ECF8_OK : ECF8_E_HIP;
    }
    if (a.M <= 16) hipLaunchKernelGGL((ecf8_gemm_raw_kernel<1, 16, 64, SCALED, ACC>), dim3(grid), dim3(16 * 64), 0, s, a);
    else if constexpr (ACC == 0) {
        if (a.M <= 32) hipLaunchKernelGGL((ecf8_gemm_raw_kernel<2, 16, 64, SCALED, ACC>), dim3(grid), dim3(16 * 64), 0, s, a);
        else if constexpr (SCALED != 2) hipLaunchKernelGGL((ecf8_gemm_raw_kernel<4, 8, 64, SCALED, ACC>), dim3(grid), dim3(8 * 64), 0, s, a);
    }
    return hipGetLastError() == hipSuccess ? ECF8_OK : ECF8_E_HIP;
}

// The counters (one per block of rows; a split matrix has at most compute units / 2 blocks) take a fixed
// area at the start of the workspace whatever the shape, so that the partial sums of one call never
// land where another shape's call keeps its counters.
constexpr uint64_t CTR_BYTES = 4096;

// Split K.  Workgroups that share a block of rows: the largest divisor of the K / 256 chunks that
// still gives every workgroup a compute unit of its own (1 = the matrix has blocks enough).  It goes by the matrix
// alone, since the workspace and the plan do; the hand-over costs some 2 us, so that it pays for long K or many rows of X.
// Plain call / split, us, M = 1 / 16 / 64: 256 x 14336 (14 slices) 13.0 / 14.5 / 23.9, 12.8 / 13.0 / 17.5; 576 x 7168 (7) 9.0 / 9.7 / 14.3, 11.1 / 11.6 / 14.0;
// 1536 x 7168 (2) 9.0 / 9.9 / 14.5, 10.9 / 11.1 / 14.5; 1024 x 4096 (4) 7.1 / 8.2 / 13.5, 10.1 / 10.2 / 12.5.
inline uint32_t pick_slices(uint64_t rows, uint64_t cols, int cus)
{
    const uint64_t n_blocks = rows / BLOCK_ROWS, kchunks = cols / 256;
    uint32_t best = 1;
    if (n_blocks * 4 > CTR_BYTES) return 1;
    for (uint64_t sl = 2; sl <= kchunks && n_blocks * sl <= (uint64_t)cus; sl++)
        if (kchunks % sl == 0) best = (uint32_t)sl;
    return best;
}

inline int tiles_of(uint32_t M) { return M <= 16 ? 1 : M <= 32 ? 2 : 4; }
inline uint64_t workspace_bytes(uint64_t rows, uint32_t M, uint32_t slices)
{
    return slices <= 1 ? 0 : CTR_BYTES + rows / BLOCK_ROWS * slices * tiles_of(M) * 256 * 4;
}

inline int split_args(GArgs *a, void *d_workspace, uint64_t bytes, uint32_t *slices)
{
    const int cus = device_cus();
    if (cus <= 0) return ECF8_E_HIP;
    *slices = pick_slices(a->rows, a->K, cus);
    if (*slices <= 1) return ECF8_OK;
    if (!d_workspace) return ECF8_E_ARG;
    if ((uintptr_t)d_workspace & 15) return ECF8_E_ALIGN;
    if (bytes < workspace_bytes(a->rows, a->M, *slices)) return ECF8_E_CAPACITY;
    a->slices = *slices;
    a->d_ctr = (uint64_t)(uintptr_t)d_workspace;
    a->d_part = a->d_ctr + CTR_BYTES;
    return ECF8_OK;
}

template <int SCALED, class CODES>
int launch_split_with(const GArgs &a, const CODES &codes, int grid, hipStream_t s)
{
    // X turned at any M.  Turned / as operands, us, M = 1 / 8 / 16: 2048 x 7168 11.4 / 11.5 / 11.7, 11.3 / 11.9 / 12.4; 1024 x 16384 12.3 / 12.4 / 12.7, 12.2 / 13.0 / 13.6;
    // 256 x 4096, a chunk a workgroup, 16.0 / 16.1 / 16.1, 15.7 / 15.8 / 15.8
    if (a.M <= 16) hipLaunchKernelGGL((ecf8_gemm_anyk_kernel<CODES, 1, WAVES<1>, 64, SCALED, true>), dim3(grid), dim3(WAVES<1> * 64), 0, s, a, codes);
    else if (a.M <= 32) hipLaunchKernelGGL((ecf8_gemm_anyk_kernel<CODES, 2, WAVES<2>, 64, SCALED, true>), dim3(grid), dim3(WAVES<2> * 64), 0, s, a, codes);
    else hipLaunchKernelGGL((ecf8_gemm_anyk_kernel<CODES, 4, WAVES<4>, 64, SCALED, true>), dim3(grid), dim3(WAVES<4> * 64), 0, s, a, codes);
    return hipGetLastError() == hipSuccess ? ECF8_OK : ECF8_E_HIP;
}

template <int SCALED, bool RAW>
int launch_split(GArgs a, void *stream)
{
    const int grid = grid_for(a.rows / BLOCK_ROWS * a.slices);      // <= the compute units by the choice of slices
    if (grid <= 0) return ECF8_E_HIP;
    deal_units(&a, (uint32_t)grid);
    deal_waves(&a, a.M);
    hipStream_t s = (hipStream_t)stream;
    if constexpr (!RAW) return a.off_tbl ? launch_split_with<SCALED>(a, TableInBlob{}, grid, s) : launch_split_with<SCALED>(a, short_codes(a.code_len), grid, s);
    if (a.M <= 16) hipLaunchKernelGGL((ecf8_gemm_raw_anyk_kernel<1, WAVES<1>, 64, SCALED, true>), dim3(grid), dim3(WAVES<1> * 64), 0, s, a);
    else if (a.M <= 32) hipLaunchKernelGGL((ecf8_gemm_raw_anyk_kernel<2, WAVES<2>, 64, SCALED, true>), dim3(grid), dim3(WAVES<2> * 64), 0, s, a);
    else hipLaunchKernelGGL((ecf8_gemm_raw_anyk_kernel<4, WAVES<4>, 64, SCALED, true>), dim3(grid), dim3(WAVES<4> * 64), 0, s, a);
    return hipGetLastError() == hipSuccess ? ECF8_OK : ECF8_E_HIP;
}

// the common tail of the two split-K calls: scales (or none), workspace, route
template <bool RAW>
int run_split(GArgs &a, const float *d_w_scale, const float *d_x_scale, uint32_t x_scale_cols, void *d_workspace,
              uint64_t bytes, void *stream)
{
    int sc = 0;
    if (d_w_scale || d_x_scale || x_scale_cols) {
        const int rc = scale_args(d_w_scale, d_x_scale, x_scale_cols, &a);
        if (rc) return rc;
        sc = a.xs_cols > 1 ? 2 : 1;
    }
    uint32_t slices;
    const int rc = split_args(&a, d_workspace, bytes, &slices);
    if (rc) return rc;
    if (slices <= 1) {      // blocks enough: the plain kernels
        if constexpr (RAW) return sc == 0 ? launch_raw<0>(a, stream) : sc == 1 ? launch_raw<1>(a, stream) : launch_raw<2>(a, stream);
        else return sc == 0 ? launch_fused<0>(a, stream) : sc == 1 ? launch_fused<1>(a, stream) : launch_fused<2>(a, stream);
    }
    return sc == 0 ? launch_split<0, RAW>(a, stream) : sc == 1 ? launch_split<1, RAW>(a, stream) : launch_split<2, RAW>(a, stream);
}

template <int SCALED, bool RAW>
int launch_grouped(uint64_t d_items, uint32_t n_items, uint64_t total_work, uint32_t max_M, void *stream)
{
    const int cus = device_cus();
    if (cus <= 0) return ECF8_E_HIP;
    hipStream_t s = (hipStream_t)stream;
    // As many chunks a launch as 32 bits count with room for a matrix more; 2^31 are 8 TiB of weights, so nearly always one launch
    for (uint64_t base = 0; base < total_work; base += LAUNCH_CHUNKS) {
        const uint64_t work = total_work - base < LAUNCH_CHUNKS ? total_work - base : LAUNCH_CHUNKS;
        // no more workgroups than blocks of 16 chunks: below that a share is less than a block's worth of the waves' work
        uint64_t grid = (work + 15) / 16;
        if (grid > (uint64_t)cus) grid = (uint64_t)cus;
        const GGArgs g{d_items, base, n_items, (uint32_t)(work / grid), (uint32_t)(work % grid)};
        if (max_M <= 16) hipLaunchKernelGGL((ecf8_gemm_grouped_kernel<1, WAVES<1>, 64, SCALED, RAW>), dim3((unsigned)grid), dim3(WAVES<1> * 64), 0, s, g);
        else if (max_M <= 32) hipLaunchKernelGGL((ecf8_gemm_grouped_kernel<2, WAVES<2>, 64, SCALED, RAW>), dim3((unsigned)grid), dim3(WAVES<2> * 64), 0, s, g);
        else hipLaunchKernelGGL((ecf8_gemm_grouped_kernel<4, WAVES<4>, 64, SCALED, RAW>), dim3((unsigned)grid), dim3(WAVES<4> * 64), 0, s, g);
        if (hipGetLastError() != hipSuccess) return ECF8_E_HIP;
    }
    return ECF8_OK;
}

__global__ __attribute__((unused)) void gemm_fill_zero_kernel(uint64_t p, uint64_t n_dwords)
{
    const uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
    if (i < n_dwords) ((GLOBAL uint32_t *)p)[i] = 0u;
}

} // namespace

#endif
