// Wide-alphabet decode kernels (E5M2, BF16) for gfx950, wave64: Algorithm 1 of
// the paper for exponent fields of 5 and 8 bits, organised like the ECF8 decoder
// (ecf8_decode.hip): one wavefront per chunk of 64 lanes x N symbols, the lanes'
// start bits from a prefix scan over the recorded lane lengths, the chunk's span
// of the stream staged in LDS, two independent runs per lane (one read forward,
// one backward), finished 16-byte pieces held in registers and stored in one
// burst, persistent workgroups over contiguous chunk ranges with an LDS ticket
// counter among their waves.  What differs:
//  * under the encoder's default cap of 12 bits (ecfw_decode_kernel) one lookup resolves TWO codewords, as there: a
//    pair table is built from a 2^12-entry table of single codewords, with entries that fit the format (see Pairs);
//    pairs that do not fit it take a branch-free second level.  The launch of a layer of seven matrices (218 M elements)
//    with one codeword per lookup and the lanes' bits moved to bank-private LDS columns first took 107.5 us for E5M2,
//    bound by LDS and vector work; now 86 (376 MB: 4.4 TB/s; set-up of the tables, and LDS and vector work).  BF16
//    was and is at the memory wall, 139 .. 141 us (735 MB: 5.3 TB/s);
//  * codes with longer codewords (cap 13..16, ecfw_long_decode_kernel) keep one codeword per lookup and
//    a canonical first-code comparison per length, in a rarely taken branch;
//  * the remaining bits come from planes laid out so that whole output words are
//    merged with a few bit selects (BF16: a byte per element in the order
//    0 2 1 3; E5M2: mantissas sliced by output word, signs as a bit mask);
//  * one launch may cover many tensors (ecfw_decode_batched): a workgroup's
//    range of chunks runs through the batch and the code is set up again where
//    it crosses into another tensor.
#include "ecfw.h"

#include "ecf8_device.h"

#include <cstring>
#include <type_traits>

namespace {

constexpr int WTB = ECFW_TABLE_BITS;
constexpr uint32_t WMASK2 = ((1u << WTB) - 1) << 1;   // byte offset mask of a 16-bit entry

typedef ecfw_batch_item WArgs;          // one tensor, as the kernel sees it

struct BArgs {
    WArgs single;                        // used when items == nullptr
    const GLOBAL WArgs *items;           // device array for the batched call
    uint32_t n_items;
    uint64_t total_chunks;               // of the launch, at most LAUNCH_CHUNKS
    ChunkDeal deal;                      // of the launch's chunks to its workgroups
    uint64_t base;                       // FAR kernels: chunks of the batch before the launch's
};

template <int FMT> struct Fmt;
template <> struct Fmt<ECFW_FMT_E5M2> {
    static constexpr int P = 16, ELEM = 1, A = 32;
    static constexpr int SYM_SHIFT = 2, LEN_SHIFT = 7;     // entry = exponent << 2 | length << 7
};
template <> struct Fmt<ECFW_FMT_BF16> {
    static constexpr int P = 8, ELEM = 2, A = 256;
    static constexpr int SYM_SHIFT = 7, LEN_SHIFT = 0;     // entry = exponent << 7 | length
};

// The kernel for codes with codewords of more than 12 bits (ecfw_long_decode_kernel).
template <int FMT, int N, int WAVES>
struct WCfg {
    using F = Fmt<FMT>;
    static constexpr int PIECES = N / F::P;                 // 16-byte pieces per lane
    // span of a chunk whose codewords average AVG bits: uniformly random exponent fields still fit
    static constexpr int AVG = 8;
    static constexpr int STAGE = 8 * AVG * N + 64;
    static constexpr int SEGS = (STAGE / 16 + 63) / 64;
    static constexpr int OFF_TBL = 0;
    static constexpr int OFF_WCNT = OFF_TBL + (2 << WTB);   // symbols per (wavefront, length) while the code is set up
    static constexpr int OFF_SORTED = OFF_WCNT + 320;       // symbols ordered by (length, symbol)
    static constexpr int OFF_CNT = OFF_SORTED + 256;        // per length 0..16: count, first code, offset into sorted
    static constexpr int OFF_FIRST = OFF_CNT + 80;
    static constexpr int OFF_OFFS = OFF_FIRST + 80;
    static constexpr int OFF_TICKET = OFF_OFFS + 80;
    static constexpr int OFF_STAGE = OFF_TICKET + 16;
    static constexpr int TOTAL = OFF_STAGE + WAVES * STAGE;
    static_assert(STAGE % 16 == 0 && OFF_STAGE % 16 == 0, "16-byte LDS stores");
    static_assert(PIECES % 2 == 0, "two runs of whole pieces");
    static_assert(TOTAL <= 160 * 1024, "LDS of one gfx950 CU");
};

struct CodeArrays {
    const uint16_t *tbl;
    const uint8_t *sorted;
    const uint32_t *cnt, *first, *offs;
};

// Sets up, from the code lengths in the blob: the per-length canonical arrays
// (count, first code, offset into the list of symbols sorted by (length, symbol))
// and the lookup table.  All threads of the workgroup call it; it needs at least
// four wavefronts.  Symbols are ranked with wave ballots (wavefront w holds symbols
// 64w..64w+63); in every wavefront lane l stands for length l, so that first codes and offsets are two
// wave prefix sums, and an entry's length is the number of lengths whose codes all lie below its index.
template <int FMT>
__device__ void build_code(uint32_t my_len, uint32_t *wavecnt, uint8_t *sorted, uint32_t *cnt,
                           uint32_t *first, uint32_t *offs, uint16_t *tbl, int tid, int nthreads)
{
    using F = Fmt<FMT>;
    constexpr int L = (int)ECFW_MAX_CODE_LEN;
    const int lane = tid & 63, wave = (int)uniform32((uint32_t)tid >> 6);
    uint32_t my_rank = 0;
    if (wave < 4) {
        const uint64_t below = ((uint64_t)1 << lane) - 1;
        uint32_t count = 0;                                         // lane l: symbols of length l in this wavefront
#pragma unroll
        for (int l = 1; l <= L; l++) {
            const uint64_t m = __ballot(my_len == (uint32_t)l);
            if (my_len == (uint32_t)l) my_rank = (uint32_t)__popcll(m & below);
            if (lane == l) count = (uint32_t)__popcll(m);
        }
        if (lane <= L) wavecnt[wave * 20 + lane] = count;
    }
    __syncthreads();
    // lane l = 1 .. L: symbols of length l, offset of the first one in `sorted`, its code
    uint32_t c[4], total = 0;
#pragma unroll
    for (int w = 0; w < 4; w++) {
        c[w] = lane >= 1 && lane <= L ? wavecnt[w * 20 + lane] : 0u;
        total += c[w];
    }
    const uint32_t space = lane >= 1 && lane <= L ? total << (L - lane) : 0u;      // of the 2^L units of code space
    const uint32_t used = wave_incl_scan(space), off = wave_incl_scan(total) - total;
    const uint32_t code1 = lane >= 1 && lane <= L ? (used - space) >> (L - lane) : 0u;
    if (wave == 0 && lane <= L) { cnt[lane] = total; first[lane] = code1; offs[lane] = off; }
    if (wave < 4) {
        uint32_t before = off;
#pragma unroll
        for (int w = 0; w < 3; w++) before += w < wave ? c[w] : 0u;
        my_rank += (uint32_t)__builtin_amdgcn_ds_bpermute((int)(my_len * 4), (int)before);
        if (my_len) sorted[my_rank] = (uint8_t)tid;
    }
    uint32_t limit[WTB + 1];                                        // first 12-bit index past the codes of length l and below
#pragma unroll
    for (int l = 1; l <= WTB; l++) limit[l] = (uint32_t)__builtin_amdgcn_readlane((int)used, l) >> (L - WTB);
    __syncthreads();
    // entry i: the codeword spelled by the bits of i, bit 0 first
    for (int i = tid; i < (1 << WTB); i += nthreads) {
        const uint32_t v = __brev((uint32_t)i) >> (32 - WTB);       // the 12 bits, first bit most significant
        uint32_t l = 1;
#pragma unroll
        for (int k = 1; k < WTB; k++) l += v >= limit[k];
        const uint32_t at = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(l * 4), (int)(off - code1)) + (v >> (WTB - l));
        uint32_t e = 0;
        if (v < limit[WTB]) e = ((uint32_t)sorted[at & 255u] << F::SYM_SHIFT) | (l << F::LEN_SHIFT);
        tbl[i] = (uint16_t)e;
    }
    __syncthreads();
}

template <int FMT>
__device__ __forceinline__ uint32_t entry_len(uint32_t e)
{
    return (e >> Fmt<FMT>::LEN_SHIFT) & 31u;
}

// A codeword longer than the table index: compare the next bits with the first
// code of every longer length.  `bits`: >= 16 valid stream bits, next bit = bit 0.
template <int FMT>
__device__ __noinline__ uint32_t long_code(uint32_t bits, const uint8_t *sorted, const uint32_t *cnt,
                                           const uint32_t *first, const uint32_t *offs)
{
    using F = Fmt<FMT>;
    const uint32_t r = __brev(bits);
    uint32_t e = (uint32_t)ECFW_MAX_CODE_LEN << F::LEN_SHIFT;     // no match (corrupt stream): skip 16 bits
#pragma unroll 1
    for (int l = WTB + 1; l <= (int)ECFW_MAX_CODE_LEN; l++) {
        const uint32_t d = (r >> (32 - l)) - first[l];
        if (d < cnt[l]) e = ((uint32_t)sorted[offs[l] + d] << F::SYM_SHIFT) | ((uint32_t)l << F::LEN_SHIFT);
    }
    return e;
}

template <int FMT>
__device__ __forceinline__ uint32_t decode_entry(uint32_t bits, const CodeArrays &ca)
{
    uint32_t e = ca.tbl[bits & ((1u << WTB) - 1)];
    if (__builtin_expect(e == 0, 0)) e = long_code<FMT>(bits, ca.sorted, ca.cnt, ca.first, ca.offs);
    return e;
}

// Two codewords of each run.  pa = (next bit of the forward run) - 1 and
// pb = (one past the next bit of the backward run) - 31 as absolute LDS bit
// addresses: the windows read there are the stream bits shifted left by one,
// which masked is the byte offset of a table entry.
template <int FMT>
__device__ __forceinline__ void pair_step(const uint8_t *smem, const CodeArrays &ca, uint32_t &pa, uint32_t &pb,
                                          uint32_t &eA0, uint32_t &eA1, uint32_t &eB0, uint32_t &eB1)
{
    const uint8_t *tb = (const uint8_t *)ca.tbl;
    const uint32_t aA = (pa >> 3) & ~3u, aB = (pb >> 3) & ~3u;
    const uint32_t wA = __builtin_amdgcn_alignbit(*(const uint32_t *)(smem + aA + 4), *(const uint32_t *)(smem + aA), pa);
    const uint32_t wB = __brev(__builtin_amdgcn_alignbit(*(const uint32_t *)(smem + aB + 4), *(const uint32_t *)(smem + aB), pb));
    eA0 = *(const uint16_t *)(tb + (wA & WMASK2));
    eB0 = *(const uint16_t *)(tb + (wB & WMASK2));
    uint32_t lA0 = entry_len<FMT>(eA0), lB0 = entry_len<FMT>(eB0);
    eA1 = *(const uint16_t *)(tb + ((wA >> lA0) & WMASK2));      // 31 - 12 >= 12 bits left
    eB1 = *(const uint16_t *)(tb + ((wB >> lB0) & WMASK2));
    uint32_t lA1 = entry_len<FMT>(eA1), lB1 = entry_len<FMT>(eB1);
    // a miss leaves the length 0, so the second lookup repeats the first: testing the second covers both
    if (__builtin_expect(eA1 == 0 || eB1 == 0, 0)) {
        if (eA1 == 0) {
            if (eA0 == 0) { eA0 = long_code<FMT>(wA >> 1, ca.sorted, ca.cnt, ca.first, ca.offs); lA0 = entry_len<FMT>(eA0); }
            eA1 = decode_entry<FMT>(lds_window<+1>(smem, pa + 1 + lA0), ca);
            lA1 = entry_len<FMT>(eA1);
        }
        if (eB1 == 0) {
            if (eB0 == 0) { eB0 = long_code<FMT>(wB >> 1, ca.sorted, ca.cnt, ca.first, ca.offs); lB0 = entry_len<FMT>(eB0); }
            eB1 = decode_entry<FMT>(lds_window<-1>(smem, pb + 31 - lB0), ca);
            lB1 = entry_len<FMT>(eB1);
        }
    }
    pa += lA0 + lA1;
    pb -= lB0 + lB1;
}

__device__ __forceinline__ uint32_t bit_sel(uint32_t mask, uint32_t a, uint32_t b)   // (a & mask) | (b & ~mask)
{
    return __builtin_amdgcn_bitop3_b32(a, b, mask, 0xE4);
}

// One 16-byte piece from its table entries and plane words.
// BF16: e[0..7]; pl.x / pl.y hold the remainder bytes of elements 0 2 1 3 / 4 6 5 7.
__device__ __forceinline__ u32x4 merge_bf16(const uint32_t e[8], u32x2 pl)
{
    u32x4 d;
    const uint32_t x0 = __builtin_amdgcn_perm(e[1], e[0], 0x05040100u), x1 = __builtin_amdgcn_perm(e[3], e[2], 0x05040100u);
    const uint32_t x2 = __builtin_amdgcn_perm(e[5], e[4], 0x05040100u), x3 = __builtin_amdgcn_perm(e[7], e[6], 0x05040100u);
    // per 16-bit half: bit 15 sign, bits 14..7 exponent (from the entry), bits 6..0 mantissa
    d.x = bit_sel(0x7f807f80u, x0, bit_sel(0x80008000u, pl.x << 8, pl.x));
    d.y = bit_sel(0x7f807f80u, x1, bit_sel(0x80008000u, pl.x, pl.x >> 8));
    d.z = bit_sel(0x7f807f80u, x2, bit_sel(0x80008000u, pl.y << 8, pl.y));
    d.w = bit_sel(0x7f807f80u, x3, bit_sel(0x80008000u, pl.y, pl.y >> 8));
    return d;
}

// E5M2: e[0..15]: entries of the 12-bit table; mant = the piece's mantissa word, sign = its 16 sign bits.
__device__ __forceinline__ u32x4 merge_e5m2(const uint32_t e[16], uint32_t mant, uint32_t sign)
{
    uint32_t out[4];
#pragma unroll
    for (int d = 0; d < 4; d++) {
        const uint32_t lo = __builtin_amdgcn_perm(e[4 * d + 1], e[4 * d], 0x0c0c0400u);       // bytes 0, 1
        const uint32_t hi = __builtin_amdgcn_perm(e[4 * d + 3], e[4 * d + 2], 0x04000c0cu);   // bytes 2, 3
        // four sign bits -> bit 0 of each byte (the partial products do not overlap), then up to bit 7
        const uint32_t s4 = __builtin_amdgcn_ubfe(sign, 4 * d, 4);
        const uint32_t sp = __umul24(s4, 0x204081u) << 7;
        out[d] = bit_sel(0x7c7c7c7cu, lo | hi, bit_sel(0x80808080u, sp, mant >> (2 * d)));
    }
    return u32x4{out[0], out[1], out[2], out[3]};
}

// The item of a batched launch that holds chunk g, in scalar registers.  FAR: one of several launches on a batch; of a tensor that begins before it, first_chunk is
// below 0: its low 32 bits count, and wrap.
template <bool FAR = false>
__device__ __forceinline__ WArgs find_item(const BArgs &b, uint32_t g, int lane)
{
    if (!b.items) return b.single;
    const uint64_t base = FAR ? b.base : 0;
    const BatchItem item(b.items, b.n_items, base + g, lane);
    WArgs a;
    uint64_t *dst = (uint64_t *)&a;
#pragma unroll
    for (int i = 0; i < 16; i++) dst[i] = item.word(i);
    a.first_chunk -= base;
    return a;
}

// the range of a launch's chunks for this workgroup, numbered in 32 bits through all tensors from the launch's first chunk on
__device__ __forceinline__ void share_of(const BArgs &b, uint32_t &g, uint32_t &g_end)
{
    g = b.deal.begin(blockIdx.x);
    g_end = b.deal.begin(blockIdx.x + 1);
    if (g_end > (uint32_t)b.total_chunks) g_end = (uint32_t)b.total_chunks;
}

// Element layout: piece q of lane l of chunk c starts at element base(c) + q * stride(c) + l * P.
template <int FMT, int N>
struct Place {
    static constexpr uint64_t E = 64ull * N, P = Fmt<FMT>::P;
    uint32_t group, whole;                            // whole: chunks inside complete groups (group is a power of two)
    __device__ __forceinline__ Place(const WArgs &a) : group((uint32_t)a.group_chunks), whole((uint32_t)(a.n_elem / E) & ~((uint32_t)a.group_chunks - 1)) {}
    __device__ __forceinline__ uint64_t base(uint32_t c) const
    {
        const uint32_t w = c < whole ? c & (group - 1) : 0u;
        return (c - w) * E + w * (64 * P);
    }
    __device__ __forceinline__ uint32_t stride(uint32_t c) const { return c < whole ? group * (uint32_t)(64 * P) : (uint32_t)(64 * P); }
};

struct Meta { uint64_t b0, b1; uint32_t lb; };

__device__ __forceinline__ Meta load_meta(const WArgs &a, uint32_t c, int lane)
{
    const GLOBAL uint64_t *chunk_bit = (const GLOBAL uint64_t *)(a.d_blob + a.off_chunk_bit) + c;
    Meta m;
    m.b0 = chunk_bit[0];
    m.b1 = chunk_bit[1];
    m.lb = ((const GLOBAL uint16_t *)(a.d_blob + a.off_lane_bits) + (uint64_t)c * 64)[lane];
    return m;
}

// A chunk's span of the stream (16-byte aligned start, 8 bytes of look-ahead) from its two start bits: the same in every
// lane, so the arithmetic is done once, in scalar registers.
__device__ __forceinline__ uint64_t span_of(const WArgs &a, const Meta &m, uint64_t &byte0)
{
    const uint64_t b0 = uniform64(m.b0), b1 = uniform64(m.b1);
    uint64_t byte_end = ((b1 + 7) >> 3) + 8;
    if (byte_end > a.stream_bytes) byte_end = a.stream_bytes;
    byte0 = (b0 >> 3) & ~15ull;
    if (byte0 > byte_end) byte0 = byte_end;
    return byte_end - byte0;
}

// The careful way, one symbol at a time with windows straight from HBM: chunks whose span does not fit the stage.
template <int FMT, int N>
__device__ __forceinline__ void symbol_pass(const WArgs &a, const CodeArrays &ca, uint64_t c, int lane)
{
    constexpr int P = Fmt<FMT>::P;
    const GLOBAL uint8_t *blob = (const GLOBAL uint8_t *)a.d_blob;
    const GLOBAL uint8_t *stream = blob + a.off_stream, *plane = blob + a.off_plane, *signs = blob + a.off_sign;
    GLOBAL uint8_t *out = (GLOBAL uint8_t *)a.d_out;
    const Place<FMT, N> place(a);
    const Meta m = load_meta(a, c, lane);
    const uint32_t rel = wave_incl_scan(m.lb) - m.lb;
    const uint64_t limit = a.stream_bytes * 8 - 64;
    uint64_t posA = m.b0 + rel, posB = posA + m.lb;
    const uint64_t e0 = place.base(c) + (uint64_t)lane * P, stride = place.stride(c);
#pragma unroll 1
    for (int k = 0; k < N; k++) {
        const uint64_t e = e0 + (uint64_t)(k / P) * stride + (uint32_t)(k % P);
        if (e >= a.n_elem) continue;
        uint32_t en;
        if (k < N / 2) {
            if (posA > limit) posA = limit;
            en = decode_entry<FMT>(global_window<+1>(stream, posA), ca);
            posA += entry_len<FMT>(en);
        } else {
            if (posB > limit) posB = limit;
            en = decode_entry<FMT>(global_window<-1>(stream, posB), ca);
            const uint32_t l = entry_len<FMT>(en);
            posB = posB >= l ? posB - l : 0;
        }
        if (FMT == ECFW_FMT_BF16) {
            const uint32_t swap = (0x3120u >> (4 * (uint32_t)(e & 3))) & 3u;      // 0 2 1 3
            const uint32_t r = plane[(e & ~3ull) + swap];
            ((GLOBAL uint16_t *)out)[e] = (uint16_t)(((r & 0x80u) << 8) | (en & 0x7f80u) | (r & 0x7fu));
        } else {
            const uint32_t j = (uint32_t)(e & 3), d = (uint32_t)(e >> 2) & 3;
            const uint32_t mw = ((const GLOBAL uint32_t *)plane)[e / 16];
            const uint32_t sw = ((const GLOBAL uint16_t *)signs)[e / 16];
            out[e] = (uint8_t)((((sw >> (e & 15)) & 1u) << 7) | (en & 0x7cu) | ((mw >> (8 * j + 2 * d)) & 3u));
        }
    }
}

// Codes with codewords of more than 12 bits (caps 13 .. 16): one codeword per lookup, the longer ones by a canonical
// first-code comparison in a rarely taken branch.
template <int FMT, int N, int WAVES, bool FAR = false>
__global__ __launch_bounds__(WAVES * 64) void ecfw_long_decode_kernel(BArgs b)
{
    using C = WCfg<FMT, N, WAVES>;
    using F = Fmt<FMT>;
    constexpr int PIECES = C::PIECES, SEGS = C::SEGS, STAGE = C::STAGE, P = F::P;
    __shared__ __attribute__((aligned(16))) uint8_t smem[C::TOTAL];
    uint16_t *tbl = (uint16_t *)(smem + C::OFF_TBL);
    uint32_t *s_ticket = (uint32_t *)(smem + C::OFF_TICKET);
    const CodeArrays ca{tbl, smem + C::OFF_SORTED, (const uint32_t *)(smem + C::OFF_CNT),
                        (const uint32_t *)(smem + C::OFF_FIRST), (const uint32_t *)(smem + C::OFF_OFFS)};

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t stage_off = C::OFF_STAGE + wave * STAGE;
    uint8_t *stage = smem + stage_off;
    uint32_t g, g_end;
    share_of(b, g, g_end);

    while (g < g_end) {                                // one round per tensor the range touches (uniform)
    const WArgs a = find_item<FAR>(b, g, lane);
    const uint32_t c_begin = g - (uint32_t)a.first_chunk;        // chunk numbers inside the tensor
    const uint32_t c_end = g_end - (uint32_t)a.first_chunk < (uint32_t)a.n_chunks ? g_end - (uint32_t)a.first_chunk : (uint32_t)a.n_chunks;
    if (FAR && (a.first_chunk + a.n_chunks) >> 32) break;  // it ends before the launch begins
    if (c_end <= c_begin) break;                       // the item table does not cover chunk g: stop rather than spin
    const GLOBAL uint8_t *blob = (const GLOBAL uint8_t *)a.d_blob;
    const GLOBAL uint8_t *stream = blob + a.off_stream;
    const GLOBAL uint8_t *plane = blob + a.off_plane;
    const GLOBAL uint8_t *signs = blob + a.off_sign;
    GLOBAL uint8_t *out = (GLOBAL uint8_t *)a.d_out;
    const Place<FMT, N> place(a);

    if (tid == 0) *s_ticket = 0;
    static_assert(WAVES >= 4, "the code set-up ranks 256 symbols with four wavefronts");
    uint32_t my_len = tid < F::A ? (blob + a.off_code_len)[tid] : 0u;
    if (my_len > ECFW_MAX_CODE_LEN) my_len = 0;
    build_code<FMT>(my_len, (uint32_t *)(smem + C::OFF_WCNT), smem + C::OFF_SORTED, (uint32_t *)(smem + C::OFF_CNT),
                    (uint32_t *)(smem + C::OFF_FIRST), (uint32_t *)(smem + C::OFF_OFFS), tbl, tid, WAVES * 64);

    struct Payload {
        u32x4 seg[SEGS];
        u32x2 pl[FMT == ECFW_FMT_BF16 ? PIECES : 1];
        uint32_t mant[FMT == ECFW_FMT_E5M2 ? PIECES : 1];
        uint32_t sign[FMT == ECFW_FMT_E5M2 ? PIECES : 1];
    };
    auto draw = [&]() -> uint32_t {
        uint32_t t = 0;
        if (lane == 0) t = atomicAdd(s_ticket, 1u);
        return c_begin + uniform32(t);
    };
    auto load_payload = [&](uint32_t c, const Meta &m, Payload &p) {
        uint64_t byte0;
        const uint64_t span = span_of(a, m, byte0);
        const uint64_t e0 = place.base(c) + (uint64_t)lane * P, stride = place.stride(c);
#pragma unroll
        for (int q = 0; q < PIECES; q++) {
            const uint64_t e = e0 + q * stride;
            if (FMT == ECFW_FMT_BF16) {
                p.pl[q] = __builtin_nontemporal_load((const GLOBAL u32x2 *)(plane + e));
            } else {
                p.mant[q] = __builtin_nontemporal_load((const GLOBAL uint32_t *)(plane + e / 4));
                p.sign[q] = __builtin_nontemporal_load((const GLOBAL uint16_t *)(signs + e / 8));
            }
        }
#pragma unroll
        for (int k = 0; k < SEGS; k++) {
            const uint32_t i = (lane + 64 * k) * 16;
            p.seg[k] = u32x4{0, 0, 0, 0};
            if (i < (uint32_t)STAGE && i < span)
                p.seg[k] = __builtin_nontemporal_load((const GLOBAL u32x4 *)(stream + byte0 + i));
        }
    };

    uint32_t cur = draw();
    Meta m_cur{0, 0, 0}, m_next{0, 0, 0};
    Payload p_cur;
    if (cur < c_end) {
        m_cur = load_meta(a, cur, lane);
        load_payload(cur, m_cur, p_cur);
    }
    uint32_t nxt = draw();
    if (nxt < c_end) m_next = load_meta(a, nxt, lane);

    while (cur < c_end) {
        const Meta m = m_cur;
        uint64_t byte0;
        const uint64_t span = span_of(a, m, byte0);
        const uint32_t rel = wave_incl_scan(m.lb) - m.lb;
        const uint64_t start = uniform64(m.b0);
        const uint32_t first_bit = (uint32_t)(start - byte0 * 8) + rel;           // this lane's first bit, counted from byte0
        const bool careful = span > (uint64_t)STAGE || (cur + 1) * place.E > a.n_elem;    // uniform
        if (!careful) {
#pragma unroll
            for (int k = 0; k < SEGS; k++) {
                const uint32_t j = (lane + 64 * k) * 16;
                if (j < (uint32_t)STAGE) *(u32x4 *)(stage + j) = p_cur.seg[k];
            }
        }
        u32x2 pl[FMT == ECFW_FMT_BF16 ? PIECES : 1];
        uint32_t mant[FMT == ECFW_FMT_E5M2 ? PIECES : 1], sign[FMT == ECFW_FMT_E5M2 ? PIECES : 1];
#pragma unroll
        for (int q = 0; q < PIECES; q++) {
            if (FMT == ECFW_FMT_BF16) pl[q] = p_cur.pl[q];
            else { mant[q] = p_cur.mant[q]; sign[q] = p_cur.sign[q]; }
        }
        // the payload registers are free: fetch the next chunk, draw the one after and fetch its metadata
        uint64_t nn = c_end;
        Meta m_next2{0, 0, 0};
        if (nxt < c_end) {
            load_payload(nxt, m_next, p_cur);
            nn = draw();
            if (nn < c_end) m_next2 = load_meta(a, nn, lane);
        }
        if (careful) {
            symbol_pass<FMT, N>(a, ca, cur, lane);
        } else {
            uint32_t pa = stage_off * 8 + first_bit - 1;    // one bit off, see pair_step
            uint32_t pb = pa + m.lb - 30;
            GLOBAL uint8_t *dst = out + (place.base(cur) + (uint64_t)lane * P) * F::ELEM;
            const uint64_t stride_bytes = (uint64_t)place.stride(cur) * F::ELEM;
            // finished pieces wait in registers and leave in bursts of eight (8 KiB per wavefront)
            constexpr int BURST = PIECES / 2 < 4 ? PIECES / 2 : 4;
            static_assert((PIECES / 2) % BURST == 0, "whole bursts");
#pragma unroll
            for (int q0 = 0; q0 < PIECES / 2; q0 += BURST) {
                u32x4 pieceA[BURST], pieceB[BURST];
#pragma unroll
                for (int i = 0; i < BURST; i++) {
                    const int q = q0 + i;
                    uint32_t eA[P], eB[P];
#pragma unroll
                    for (int t = 0; t < P / 2; t++)
                        pair_step<FMT>(smem, ca, pa, pb, eA[2 * t], eA[2 * t + 1], eB[2 * t], eB[2 * t + 1]);
                    if constexpr (FMT == ECFW_FMT_BF16) {
                        pieceA[i] = merge_bf16(eA, pl[q]);
                        pieceB[i] = merge_bf16(eB, pl[q + PIECES / 2]);
                    } else {
                        pieceA[i] = merge_e5m2(eA, mant[q], sign[q]);
                        pieceB[i] = merge_e5m2(eB, mant[q + PIECES / 2], sign[q + PIECES / 2]);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < BURST; i++) __builtin_nontemporal_store(pieceA[i], (GLOBAL u32x4 *)(dst + (q0 + i) * stride_bytes));
#pragma unroll
                for (int i = 0; i < BURST; i++)
                    __builtin_nontemporal_store(pieceB[i], (GLOBAL u32x4 *)(dst + (q0 + i + PIECES / 2) * stride_bytes));
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        cur = nxt;
        nxt = nn;
        m_cur = m_next;
        m_next = m_next2;
    }
    g = (uint32_t)a.first_chunk + c_end;
    __syncthreads();                                   // every wave is done with this tensor's table and tickets
    }
}

// ---- codes of at most 12 bits: two codewords per lookup ----

// Pair table, indexed by the next BITS stream bits: the exponent fields of the first two codewords and the bits both
// consume, 0 if that is more than BITS.
//  * BF16: 2^13 entries of 32 bits, the fields where an output word has them (bits 7..14 of both halves), i.e. one look-up
//    per output word; the length in bits 0..4, which the merge masks off.  (2^14 entries: no faster, these launches
//    are at the memory wall.)
//  * E5M2: 2^15 entries of 16 bits: fields at 2..6 and 7..11, the length in the upper four bits.  Fifteen bits leave pairs
//    that do not fit to one step of a wave in six; thirteen, in 32-bit entries of the same size, to two in three.
// In an entry without a pair the second field's place has the first codeword's length.
template <int FMT> struct Pairs;
template <> struct Pairs<ECFW_FMT_E5M2> {
    typedef uint16_t Entry;
    static constexpr int BITS = 15, OFF = 1;               // OFF: log2 of an entry's size
    static constexpr uint32_t SYM1 = 0x7cu;
    static constexpr int SYM2_AT = 5, FIRST_AT = 7, LEN_AT = 12;       // second field: the single table's entry << SYM2_AT
    static __device__ __forceinline__ uint32_t len(uint32_t e) { return e >> LEN_AT; }
};
template <> struct Pairs<ECFW_FMT_BF16> {
    typedef uint32_t Entry;
    static constexpr int BITS = 13, OFF = 2;
    static constexpr uint32_t SYM1 = 0x7f80u;
    static constexpr int SYM2_AT = 16, FIRST_AT = 23, LEN_AT = 0;
    static __device__ __forceinline__ uint32_t len(uint32_t e) { return e & 31u; }
};

// From the table of single codewords: the codeword at the low 12 bits of the index, then the one that many bits on (zeros
// shifted in at the top can only lengthen a codeword that does not fit anyway).  A thread keeps the low bits and
// walks over the others.
template <int FMT>
__device__ __forceinline__ void build_pairs(const uint16_t *tbl, typename Pairs<FMT>::Entry *pairs, uint16_t *tmp, int tid, int nthreads)
{
    using PT = Pairs<FMT>;
    constexpr uint32_t M = (1u << WTB) - 1;
    if constexpr (FMT == ECFW_FMT_E5M2) {
        // Two entries at a time, those of low bits 2t and 2t + 1, in the halves of a dword.  A pair's entry is the sum of two parts: of the
        // first codeword its field and length, of the second the same five bits up, which `tmp` has for all 12-bit indices.  A pair that
        // does not fit goes past 16 bits and saturates, and so does one of an index without a codeword, which is all ones here.
        // (Four times the entries of BF16, per workgroup and tensor.  Made one at a time, with a sum and two compares, a launch took 0.8 us
        // more, with lengths taken apart and compared 1.5.)
        static_assert(PT::LEN_AT == Fmt<FMT>::LEN_SHIFT + 5 && PT::SYM2_AT == 5 && PT::LEN_AT + 4 == 16 && PT::SYM1 == 0x7cu, "sums of entries");
        typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
        for (uint32_t i = tid; i <= M / 2; i += nthreads) {
            const uint32_t t = ((const uint32_t *)tbl)[i], lo = t & 0xffffu, hi = t >> 16;
            ((uint32_t *)tmp)[i] = (lo ? lo << 5 : 0xffffu) | (hi ? hi << 21 : 0xffff0000u);
        }
        __syncthreads();
        for (uint32_t i = tid; i <= M / 2; i += nthreads) {
            const uint32_t t = ((const uint32_t *)tbl)[i], lo = t & 0xffffu, hi = t >> 16;
            const uint32_t l0 = entry_len<FMT>(lo), l1 = entry_len<FMT>(hi);
            const uint32_t first = (lo ? (lo & PT::SYM1) | (l0 << PT::LEN_AT) : 0xffffu) | (hi ? (hi & PT::SYM1) | (l1 << PT::LEN_AT) : 0xffffu) << 16;
            const uint32_t alone = (lo & PT::SYM1) | (l0 << PT::FIRST_AT) | ((hi & PT::SYM1) | (l1 << PT::FIRST_AT)) << 16;
            const uint32_t at0 = ((4 * i) >> l0) & ~1u, at1 = ((4 * i + 2) >> l1) & ~1u;       // bytes into tmp
#pragma unroll
            for (uint32_t h = 0; h < 1u << (PT::BITS - WTB); h++) {
                const uint32_t t0 = *(const uint16_t *)((const uint8_t *)tmp + ((((h << (WTB + 1)) >> l0) & (2 * M)) | at0));
                const uint32_t t1 = *(const uint16_t *)((const uint8_t *)tmp + ((((h << (WTB + 1)) >> l1) & (2 * M)) | at1));
                const uint32_t second = t0 | (t1 << 16);
                const u16x2 sum = __builtin_elementwise_add_sat(__builtin_bit_cast(u16x2, first), __builtin_bit_cast(u16x2, second));
                // 0xffff where it saturated: a sum that fits has its lowest two bits clear
                const u16x2 over = __builtin_elementwise_sub_sat(sum, u16x2{0xfffc, 0xfffc}) * u16x2{0x5555, 0x5555};
                ((uint32_t *)pairs)[i | (h << (WTB - 1))] = bit_sel(__builtin_bit_cast(uint32_t, over), alone, __builtin_bit_cast(uint32_t, sum));
            }
        }
    } else {
        for (uint32_t lo = tid; lo <= M; lo += nthreads) {
            const uint32_t t1 = tbl[lo], l1 = entry_len<FMT>(t1), base = t1 & PT::SYM1;
#pragma unroll
            for (uint32_t hi = 0; hi < 1u << (PT::BITS - WTB); hi++) {
                const uint32_t t2 = tbl[((lo | (hi << WTB)) >> l1) & M], l2 = entry_len<FMT>(t2), n = l1 + l2;
                const bool pair = l1 != 0 && l2 != 0 && n <= (uint32_t)PT::BITS;
                pairs[lo | (hi << WTB)] = (typename PT::Entry)(base + (pair ? ((t2 & PT::SYM1) << PT::SYM2_AT) + (n << PT::LEN_AT) : l1 << PT::FIRST_AT));
            }
        }
    }
    __syncthreads();
}

// The second level: e, n are the entry at bit `from` of W and its length, 0 where its pair did not fit.
template <int FMT>
__device__ __forceinline__ void join_pair(const uint8_t *tbl, uint64_t W, uint32_t from, uint32_t &e, uint32_t &n)
{
    using PT = Pairs<FMT>;
    const uint32_t l = (e >> PT::FIRST_AT) & 15u;           // of use only where n == 0
    const uint32_t x = *(const uint16_t *)(tbl + (((uint32_t)(W >> (from + l)) >> (PT::OFF - 1)) & WMASK2));
    if (n == 0) {
        e = (e & PT::SYM1) | ((x & PT::SYM1) << PT::SYM2_AT);
        n = l + entry_len<FMT>(x);
    }
}

// Four codewords of each run: two lookups.  pa = (next bit of the forward run) - OFF and pb = (one past the next bit of the
// backward run) - (32 - OFF) as LDS bit addresses: the windows read there are the stream bits shifted left by OFF, which
// masked is the byte offset of a table entry.  A pair that does not fit the table sends the wave through a branch-free
// second level: the pair's other codeword is the one that many bits on, and the second pair starts where the first
// now ends; 64-bit windows reach that far.
template <int FMT>
__device__ __forceinline__ void quad_step(const uint8_t *smem, const uint8_t *pairs, const uint8_t *tbl, uint32_t &pa, uint32_t &pb, uint32_t &eA1,
                                          uint32_t &eA2, uint32_t &eB1, uint32_t &eB2)
{
    using PT = Pairs<FMT>;
    auto at = [&](uint32_t w) -> uint32_t { return *(const typename PT::Entry *)(pairs + (w & (((1u << PT::BITS) - 1) << PT::OFF))); };
    const uint32_t aA = (pa >> 3) & ~3u, aB = (pb >> 3) & ~3u;
    const uint32_t dA0 = *(const uint32_t *)(smem + aA), dA1 = *(const uint32_t *)(smem + aA + 4);
    const uint32_t dB0 = *(const uint32_t *)(smem + aB), dB1 = *(const uint32_t *)(smem + aB + 4);
    const uint32_t wA = __builtin_amdgcn_alignbit(dA1, dA0, pa);
    const uint32_t wB = __brev(__builtin_amdgcn_alignbit(dB1, dB0, pb));
    eA1 = at(wA);
    eB1 = at(wB);
    uint32_t nA1 = PT::len(eA1), nB1 = PT::len(eB1);
    eA2 = at(wA >> nA1);                          // OFF + 2 BITS <= 32 valid bits in the window
    eB2 = at(wB >> nB1);
    uint32_t nA2 = PT::len(eA2), nB2 = PT::len(eB2);
    // n1 == 0 makes the second lookup repeat the first, so n2 == 0 covers both pairs of a run
    if (__builtin_expect(nA2 == 0 || nB2 == 0, 0)) {
        const uint32_t dA2 = *(const uint32_t *)(smem + aA + 8), dBm = *(const uint32_t *)(smem + aB - 4);
        const uint64_t WA = wA | ((uint64_t)__builtin_amdgcn_alignbit(dA2, dA1, pa) << 32);
        const uint64_t WB = wB | ((uint64_t)__brev(__builtin_amdgcn_alignbit(dB0, dBm, pb)) << 32);
        join_pair<FMT>(tbl, WA, 0, eA1, nA1);     // first pairs: at most 24 bits
        join_pair<FMT>(tbl, WB, 0, eB1, nB1);
        eA2 = at((uint32_t)(WA >> nA1));
        eB2 = at((uint32_t)(WB >> nB1));
        nA2 = PT::len(eA2);
        nB2 = PT::len(eB2);
        join_pair<FMT>(tbl, WA, nA1, eA2, nA2);   // at most OFF + 24 + 15 + 12 bits from the windows' start
        join_pair<FMT>(tbl, WB, nB1, eB2, nB2);
    }
    pa += nA1 + nA2;
    pb = pb - nB1 - nB2;
}

// E5M2: quad_step over windows held in registers, as in the E4M3 decoder (HeldRuns).  Pairs that fit the table move a run by 30 bits at the most, by
// one dword; where one does not, the run may move by two, and its dwords are fetched again.
__device__ __forceinline__ void quad_step_held(const uint8_t *smem, const uint8_t *pairs, const uint8_t *tbl, HeldRuns &r, uint32_t &eA1, uint32_t &eA2,
                                               uint32_t &eB1, uint32_t &eB2)
{
    using PT = Pairs<ECFW_FMT_E5M2>;
    static_assert(PT::OFF == 1, "HeldRuns are one bit off");
    auto at = [&](uint32_t w) -> uint32_t { return *(const uint16_t *)(pairs + (w & (((1u << PT::BITS) - 1) << 1))); };
    const uint32_t wA = __builtin_amdgcn_alignbit(r.a1, r.a0, r.pa);
    const uint32_t wB = __brev(__builtin_amdgcn_alignbit(r.b1, r.b0, r.pb));
    eA1 = at(wA);
    eB1 = at(wB);
    __builtin_amdgcn_sched_barrier(0x7f);           // the look-ups stay in front of the next dwords
    const uint32_t a2 = *(const uint32_t *)(smem + r.A + 8);
    const uint32_t bm = *(const uint32_t *)(smem + r.B);
    uint32_t nA1 = PT::len(eA1), nB1 = PT::len(eB1);
    eA2 = at(wA >> nA1);
    eB2 = at(wB >> nB1);
    uint32_t nA2 = PT::len(eA2), nB2 = PT::len(eB2);
    // n1 == 0 makes the second lookup repeat the first, so n2 == 0 covers both pairs of a run
    if (__builtin_expect(nA2 == 0 || nB2 == 0, 0)) {
        const uint64_t WA = wA | ((uint64_t)__builtin_amdgcn_alignbit(a2, r.a1, r.pa) << 32);
        const uint64_t WB = wB | ((uint64_t)__brev(__builtin_amdgcn_alignbit(r.b0, bm, r.pb)) << 32);
        join_pair<ECFW_FMT_E5M2>(tbl, WA, 0, eA1, nA1);
        join_pair<ECFW_FMT_E5M2>(tbl, WB, 0, eB1, nB1);
        eA2 = at((uint32_t)(WA >> nA1));
        eB2 = at((uint32_t)(WB >> nB1));
        nA2 = PT::len(eA2);
        nB2 = PT::len(eB2);
        join_pair<ECFW_FMT_E5M2>(tbl, WA, nA1, eA2, nA2);
        join_pair<ECFW_FMT_E5M2>(tbl, WB, nB1, eB2, nB2);
        r.begin(smem, r.pa + nA1 + nA2, r.pb + 32 - nB1 - nB2);
        return;
    }
    r.pa += nA1 + nA2;
    r.pb -= nB1 + nB2;
    const uint32_t A = (r.pa >> 3) & ~3u, B = (r.pb >> 3) & ~3u;
    const bool upA = A != r.A, downB = B != r.B;
    r.a0 = upA ? r.a1 : r.a0;
    r.a1 = upA ? a2 : r.a1;
    r.b1 = downB ? r.b0 : r.b1;
    r.b0 = downB ? bm : r.b0;
    r.A = A;
    r.B = B;
}

template <int FMT, int N, int WAVES>
struct PCfg {
    using F = Fmt<FMT>;
    static constexpr int PIECES = N / F::P;                 // 16-byte pieces per lane
    // span of a chunk whose codewords average AVG bits: uniformly random exponent fields still fit
    static constexpr int AVG = FMT == ECFW_FMT_BF16 ? 8 : 5;
    static constexpr int STAGE = 8 * AVG * N + 64;
    static constexpr int SEGS = (STAGE / 16 + 63) / 64;
    static constexpr int LIST_MAX = 60;                     // oversize chunks remembered per (workgroup, tensor)
    static constexpr int OFF_PAIRS = 0;
    static constexpr int OFF_TBL = OFF_PAIRS + ((int)sizeof(typename Pairs<FMT>::Entry) << Pairs<FMT>::BITS);
    static constexpr int OFF_WCNT = OFF_TBL + (2 << WTB);
    static constexpr int OFF_SORTED = OFF_WCNT + 320;
    static constexpr int OFF_CNT = OFF_SORTED + 256;
    static constexpr int OFF_FIRST = OFF_CNT + 80;
    static constexpr int OFF_OFFS = OFF_FIRST + 80;
    static constexpr int OFF_CTL = OFF_OFFS + 80;           // ticket counter, oversize count, tail flag, oversize list
    static constexpr int OFF_STAGE = OFF_CTL + 16 + 4 * LIST_MAX;
    // a lane of a ragged last chunk reads up to N / 2 codewords past its bits
    static constexpr int TOTAL = OFF_STAGE + WAVES * STAGE + N / 2 * WTB / 8 + 32;
    static_assert(STAGE % 16 == 0 && OFF_STAGE % 16 == 0, "16-byte LDS stores");
    static_assert(PIECES % 4 == 0, "two runs of whole pieces, in bursts of two or more");
    static_assert(TOTAL <= 160 * 1024, "LDS of one gfx950 CU");
    static_assert(WAVES >= 4, "the code set-up ranks 256 symbols with four wavefronts");
    static_assert(WAVES * STAGE >= 2 << WTB, "scratch of build_pairs");
};

// The loop of the E4M3 decoder (ecf8_decode.hip) over these tables: metadata two chunks ahead, payload one chunk ahead in
// registers refilled in place, full chunks only, so that the stores of a chunk are unconditional and the wait for a
// prefetch never drains them; PER: pieces of each run that leave together.
template <int FMT, int N, int WAVES, int PER>
__global__ __launch_bounds__(WAVES * 64) void ecfw_decode_kernel(BArgs b)
{
    using C = PCfg<FMT, N, WAVES>;
    using F = Fmt<FMT>;
    constexpr int PIECES = C::PIECES, SEGS = C::SEGS, STAGE = C::STAGE, P = F::P;
    constexpr bool BF = FMT == ECFW_FMT_BF16;
    __shared__ __attribute__((aligned(16))) uint8_t smem[C::TOTAL];
    uint16_t *tbl = (uint16_t *)(smem + C::OFF_TBL);
    uint32_t *s_ticket = (uint32_t *)(smem + C::OFF_CTL);
    uint32_t *s_oversize = s_ticket + 1;                  // number of oversize chunks met in the loop
    uint32_t *s_tail = s_ticket + 2;                      // set: the ragged last chunk is left to the symbol pass
    uint32_t *s_list = s_ticket + 4;                      // oversize chunks, relative to c_begin
    const CodeArrays ca{tbl, smem + C::OFF_SORTED, (const uint32_t *)(smem + C::OFF_CNT),
                        (const uint32_t *)(smem + C::OFF_FIRST), (const uint32_t *)(smem + C::OFF_OFFS)};

    const int tid = threadIdx.x, lane = tid & 63, wave = (int)uniform32((uint32_t)tid >> 6);
    const uint32_t stage_off = C::OFF_STAGE + wave * STAGE, lane16 = (uint32_t)lane * 16;
    uint8_t *stage = smem + stage_off;
    uint32_t g, g_end;
    share_of(b, g, g_end);

    while (g < g_end) {                                // one round per tensor the range touches (uniform)
        const WArgs a = find_item(b, g, lane);
        const uint32_t c_begin = g - (uint32_t)a.first_chunk;    // chunk numbers inside the tensor
        const uint32_t c_end = g_end - (uint32_t)a.first_chunk < (uint32_t)a.n_chunks ? g_end - (uint32_t)a.first_chunk : (uint32_t)a.n_chunks;
        if (c_end <= c_begin) break;                   // the item table does not cover chunk g: stop rather than spin
        const GLOBAL uint8_t *blob = (const GLOBAL uint8_t *)a.d_blob;
        const GLOBAL uint8_t *stream = blob + a.off_stream, *plane = blob + a.off_plane, *signs = blob + a.off_sign;
        GLOBAL uint8_t *out = (GLOBAL uint8_t *)a.d_out;
        const Place<FMT, N> place(a);
        const bool ragged_tail = c_end == a.n_chunks && a.n_elem % place.E != 0;
        const uint32_t fast_end = ragged_tail ? c_end - 1 : c_end;

        __syncthreads();                               // every wave is done with the previous tensor's tables
        if (tid == 0) { *s_ticket = 2 * WAVES; *s_oversize = 0; *s_tail = 0; }

        auto draw = [&]() -> uint32_t {
            uint32_t t = 0;
            if (lane == 0) t = __hip_atomic_fetch_add(s_ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            return c_begin + uniform32(t);
        };
        // the span's 16-byte units; those beyond it keep what they held
        auto load_stream = [&](const Meta &m, u32x4 (&seg)[SEGS]) {
            uint64_t byte0;
            const uint64_t span64 = span_of(a, m, byte0);
            const uint32_t span = span64 <= (uint64_t)STAGE ? (uint32_t)span64 : 0u;
            const GLOBAL uint8_t *sp = stream + byte0;
#pragma unroll
            for (int k = 0; k < SEGS; k++) {
                const uint32_t i = lane16 + 1024 * k;
                if (i < span) seg[k] = __builtin_nontemporal_load((const GLOBAL u32x4 *)(sp + i));
            }
        };
        // what a piece's elements have besides their exponents: BF16 eight bytes, E5M2 a word of mantissas and 16 signs
        struct Rest { u32x2 v; };
        auto load_rest = [&](uint64_t e) {
            Rest r;
            if constexpr (BF) r.v = __builtin_nontemporal_load((const GLOBAL u32x2 *)(plane + e));
            else r.v = u32x2{__builtin_nontemporal_load((const GLOBAL uint32_t *)(plane + e / 4)), __builtin_nontemporal_load((const GLOBAL uint16_t *)(signs + e / 8))};
            return r;
        };

        // the first two chunks of a wave are fixed, later ones are drawn
        uint32_t cur = c_begin + wave, nxt = cur + WAVES, nn = fast_end;
        Meta m_cur{0, 0, 0}, m_next{0, 0, 0};
        u32x4 seg[SEGS];
        Rest rest[PIECES];
#pragma unroll
        for (int k = 0; k < SEGS; k++) seg[k] = u32x4{0, 0, 0, 0};
#pragma unroll
        for (int q = 0; q < PIECES; q++) rest[q].v = u32x2{0, 0};
        uint32_t my_len = tid < F::A ? (blob + a.off_code_len)[tid] : 0u;
        auto load_first = [&](uint32_t c) {
            m_cur = load_meta(a, c, lane);
            m_next = load_meta(a, nxt < fast_end ? nxt : c, lane);      // a copy of m_cur would wait for it
            const uint64_t e0 = place.base(c) + (uint64_t)lane * P;
#pragma unroll
            for (int q = 0; q < PIECES; q++) rest[q] = load_rest(e0 + q * (uint64_t)place.stride(c));
            load_stream(m_cur, seg);
        };
        // the ragged last chunk goes first, to the wave it would fall to in turn, its stores cut at the tensor's end
        const bool tail_here = ragged_tail && (uint32_t)wave == (c_end - 1 - c_begin) % WAVES;
        if (tail_here) load_first(c_end - 1);
        else if (cur < fast_end) load_first(cur);
        if (my_len > ECFW_MAX_CODE_LEN) my_len = 0;
        build_code<FMT>(my_len, (uint32_t *)(smem + C::OFF_WCNT), smem + C::OFF_SORTED, (uint32_t *)(smem + C::OFF_CNT),
                        (uint32_t *)(smem + C::OFF_FIRST), (uint32_t *)(smem + C::OFF_OFFS), tbl, tid, WAVES * 64);
        build_pairs<FMT>(tbl, (typename Pairs<FMT>::Entry *)(smem + C::OFF_PAIRS), (uint16_t *)(smem + C::OFF_STAGE), tid, WAVES * 64);

        // One chunk from LDS bit `first_bit` on.  The pieces of `rest` give their registers to the chunk whose first
        // element in this lane is next_e (RELOAD); CUT: the chunk reaches past the tensor's end.
        auto decode_store = [&](auto reload, auto cut, uint32_t first_bit, uint32_t lb, uint64_t e0, uint32_t stride, uint64_t next_e,
                                uint32_t next_stride) {
            constexpr bool RELOAD = decltype(reload)::value, CUT = decltype(cut)::value;
            uint32_t pa = first_bit - Pairs<FMT>::OFF, pb = first_bit + lb - (32 - Pairs<FMT>::OFF);                 // see quad_step
            HeldRuns runs;
            if constexpr (!BF) runs.begin(smem, pa, pb);
            auto piece = [&](const uint32_t (&x)[4], const Rest &r) {
                u32x4 d;
                if constexpr (BF) {
                    d.x = bit_sel(0x7f807f80u, x[0], bit_sel(0x80008000u, r.v.x << 8, r.v.x));
                    d.y = bit_sel(0x7f807f80u, x[1], bit_sel(0x80008000u, r.v.x, r.v.x >> 8));
                    d.z = bit_sel(0x7f807f80u, x[2], bit_sel(0x80008000u, r.v.y << 8, r.v.y));
                    d.w = bit_sel(0x7f807f80u, x[3], bit_sel(0x80008000u, r.v.y, r.v.y >> 8));
                } else {
                    uint32_t o[4];
#pragma unroll
                    for (int k = 0; k < 4; k++) {
                        // four sign bits -> bit 0 of each byte (the partial products do not overlap), then up to bit 7
                        const uint32_t sp = __umul24(__builtin_amdgcn_ubfe(r.v.y, 4 * k, 4), 0x204081u) << 7;
                        o[k] = bit_sel(0x7c7c7c7cu, x[k], bit_sel(0x80808080u, sp, r.v.x >> (2 * k)));
                    }
                    d = u32x4{o[0], o[1], o[2], o[3]};
                }
                return d;
            };
            auto store_at = [&](u32x4 v, uint64_t e) {
                GLOBAL uint8_t *to = out + e * F::ELEM;
                if (!CUT || e + P <= a.n_elem) {
                    __builtin_nontemporal_store(v, (GLOBAL u32x4 *)to);
                    return;
                }
#pragma unroll 1
                for (uint64_t i = e; i < a.n_elem; i++, to += F::ELEM) {
                    if constexpr (BF) *(GLOBAL uint16_t *)to = (uint16_t)v.x;
                    else *to = (uint8_t)v.x;
                    v.x = __builtin_amdgcn_alignbit(v.y, v.x, 8 * F::ELEM);
                    v.y = __builtin_amdgcn_alignbit(v.z, v.y, 8 * F::ELEM);
                    v.z = __builtin_amdgcn_alignbit(v.w, v.z, 8 * F::ELEM);
                    v.w >>= 8 * F::ELEM;
                }
            };
            constexpr int H = PIECES / 2, BURST = CUT ? 1 : PER;
            static_assert(H % PER == 0, "whole bursts");
#pragma unroll
            for (int q0 = 0; q0 < H; q0 += BURST) {
                u32x4 oA[BURST], oB[BURST];
#pragma unroll
                for (int i = 0; i < BURST; i++) {
                    const int q = q0 + i;
                    uint32_t xA[4], xB[4];
#pragma unroll
                    for (int t = 0; t < (BF ? 2 : 4); t++) {
                        uint32_t eA1, eA2, eB1, eB2;
                        if constexpr (BF) quad_step<FMT>(smem, smem + C::OFF_PAIRS, smem + C::OFF_TBL, pa, pb, eA1, eA2, eB1, eB2);
                        else quad_step_held(smem, smem + C::OFF_PAIRS, smem + C::OFF_TBL, runs, eA1, eA2, eB1, eB2);
                        if constexpr (BF) {
                            xA[2 * t] = eA1; xA[2 * t + 1] = eA2;
                            xB[2 * t] = eB1; xB[2 * t + 1] = eB2;
                        } else {
                            const uint32_t tA = __builtin_amdgcn_perm(eA2, eA1, 0x05040100u), tB = __builtin_amdgcn_perm(eB2, eB1, 0x05040100u);
                            xA[t] = bit_sel(0x007c007cu, tA, tA << 3);
                            xB[t] = bit_sel(0x007c007cu, tB, tB << 3);
                        }
                    }
                    oA[i] = piece(xA, rest[q]);
                    oB[i] = piece(xB, rest[q + H]);
                    if constexpr (RELOAD) {
                        rest[q] = load_rest(next_e + q * (uint64_t)next_stride);
                        rest[q + H] = load_rest(next_e + (q + H) * (uint64_t)next_stride);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < BURST; i++) store_at(oA[i], e0 + (q0 + i) * (uint64_t)stride);
#pragma unroll
                for (int i = 0; i < BURST; i++) store_at(oB[i], e0 + (q0 + i + H) * (uint64_t)stride);
                __builtin_amdgcn_sched_barrier(0);
            }
        };

        if (tail_here) {
            uint64_t byte0;
            const uint64_t span64 = span_of(a, m_cur, byte0);
            if (span64 <= (uint64_t)STAGE) {
                const uint32_t rel = wave_incl_scan(m_cur.lb) - m_cur.lb;
#pragma unroll
                for (int k = 0; k < SEGS; k++)
                    if (lane16 + 1024 * k < (uint32_t)span64) *(u32x4 *)(stage + lane16 + 1024 * k) = seg[k];
                decode_store(std::false_type{}, std::true_type{}, stage_off * 8 + (uint32_t)(uniform64(m_cur.b0) - byte0 * 8) + rel, m_cur.lb,
                             place.base(c_end - 1) + (uint64_t)lane * P, place.stride(c_end - 1), 0, 0);
            } else if (lane == 0) {
                *s_tail = 1;
            }
            if (cur < fast_end) load_first(cur);
        }
        if (cur < fast_end) {
            // drain the prologue's loads here (vmcnt(0)), so that the wait at the loop head is decided by the back edge
            __builtin_amdgcn_s_waitcnt(0x0F70);
            for (;;) {
                uint64_t byte0;
                const uint64_t span64 = span_of(a, m_cur, byte0);
                const bool staged = __builtin_amdgcn_readfirstlane((uint32_t)(span64 <= (uint64_t)STAGE)) != 0;
                const uint32_t rel = wave_incl_scan(m_cur.lb) - m_cur.lb;
                const uint32_t bit_in = (uint32_t)(uniform64(m_cur.b0) - byte0 * 8) + rel;     // this lane's first bit from byte0
#pragma unroll
                for (int k = 0; k < SEGS; k++)
                    if (lane16 + 1024 * k < (uint32_t)STAGE) *(u32x4 *)(stage + lane16 + 1024 * k) = seg[k];
                const bool has_next = nxt < fast_end;
                Meta m_next2 = m_next;
                if (has_next) {
                    load_stream(m_next, seg);
                    nn = draw();
                    if (nn < fast_end) m_next2 = load_meta(a, nn, lane);
                }
                if (!staged && lane == 0) {
                    const uint32_t at = __hip_atomic_fetch_add(s_oversize, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    if (at < (uint32_t)C::LIST_MAX) s_list[at] = cur - c_begin;
                }
                // a chunk that was not staged decodes stale bits (redone after the loop), its runs pinned to the stage's start
                const uint32_t c_rest = has_next ? nxt : cur;          // after the last chunk: its own rest again, not a branch
                decode_store(std::true_type{}, std::false_type{}, stage_off * 8 + (staged ? bit_in : 64u), staged ? m_cur.lb : 0u,
                             place.base(cur) + (uint64_t)lane * P, place.stride(cur), place.base(c_rest) + (uint64_t)lane * P, place.stride(c_rest));
                if (!has_next) break;
                m_cur = m_next;
                m_next = m_next2;
                cur = nxt;
                nxt = nn;
            }
        }
        // Chunks whose span did not fit a stage, and a ragged last one of that kind: symbol by symbol.  The loop stored
        // garbage for them, from whichever wave drew them: every such store lands before any store of this pass.
        __syncthreads();
        const uint32_t n_over = *s_oversize;
        const bool tail_left = *s_tail != 0;
        if (n_over != 0 || tail_left) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            __syncthreads();
            const bool listed = n_over <= (uint32_t)C::LIST_MAX;
            const uint32_t count = listed ? n_over + (tail_left ? 1u : 0u) : c_end - c_begin;
#pragma unroll 1
            for (uint32_t k = wave; k < count; k += WAVES) {
                const uint32_t c = !listed ? c_begin + k : k < n_over ? c_begin + uniform32(s_list[k]) : c_end - 1;
                if (!listed) {
                    uint64_t byte0;
                    const bool over = c >= fast_end ? tail_left : span_of(a, load_meta(a, c, lane), byte0) > (uint64_t)STAGE;
                    if (!__builtin_amdgcn_readfirstlane((uint32_t)over)) continue;
                }
                symbol_pass<FMT, N>(a, ca, c, lane);
            }
        }
        g = (uint32_t)a.first_chunk + c_end;
    }
}

// one per compute unit, fewer where the caller or the number of chunks says so; 0: no device
uint64_t workgroups(const BArgs &a, uint32_t max_workgroups)
{
    const int cus = device_cus();
    if (cus <= 0) return 0;
    uint64_t grid = (uint64_t)cus;
    if (max_workgroups && max_workgroups < grid) grid = max_workgroups;
    return grid < a.total_chunks ? grid : a.total_chunks;
}

template <int WAVES, class K>
int launch_as(K kernel, const BArgs &a, uint32_t max_workgroups, hipStream_t stream)
{
    const uint64_t grid = workgroups(a, max_workgroups);
    if (grid == 0) return ECF8_E_HIP;
    BArgs dealt = a;
    dealt.deal = deal_chunks(a.total_chunks, (uint32_t)grid);
    hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(WAVES * 64), 0, stream, dealt);
    return hipGetLastError() == hipSuccess ? ECF8_OK : ECF8_E_HIP;
}

template <int FMT>
int launch_fmt(const BArgs &a, uint32_t N, bool fast, uint32_t max_workgroups, hipStream_t s)
{
    if (!fast)
        return N == 64 ? launch_as<8>(ecfw_long_decode_kernel<FMT, 64, 8>, a, max_workgroups, s)
                       : launch_as<8>(ecfw_long_decode_kernel<FMT, 128, 8>, a, max_workgroups, s);
    // Waves per workgroup and bursts, measured on a layer of seven matrices (218 M elements):
    //   BF16, N = 64   8 waves, a chunk's pieces in one burst 139.0 us; 10 waves 139.6, 12 waves 140.6, 6 waves 150.7; in two
    //                  bursts 8 waves 144.8, 12 waves 145, 16 waves 149
    //   E5M2, N = 128  12 waves, two bursts 84.8 us; 12 waves, one burst 94.2; 16 waves, two 99.4; 10 waves, two 88.7; 8 waves, one 92.2, two 92.4.  The same order
    //                  for one matrix of 1024 x 1024 (12.9, 15.7, 17.1, 13.6, 13.5, 13.4) up to eight of 14336 x 4096 (160.9, 166.0, 177.1, 161.1, 169.7, 169.7)
    // i.e. BF16 is at the memory wall and wants its stores together, E5M2 wants the waves to hide its look-ups.
    if constexpr (FMT == ECFW_FMT_BF16) {
        const uint64_t wgs = workgroups(a, max_workgroups), each = wgs ? (a.total_chunks + wgs - 1) / wgs : 0;
        // N = 64: 12 waves where they save one of the first four rounds of chunks.  8 / 12 waves, us, by chunks per workgroup: 9 15.9 / 13.7,
        // 12 17.0 / 15.7, 13 17.6 / 17.7, 16 19.1 / 19.6, 17 21.3 / 20.4, 20 21.3 / 21.0, 24 23.0 / 23.1, 25 24.6 / 23.7, 28 26.6 / 25.9, 30 27.5 / 27.1,
        // 32 27.7 / 27.9, 52 39.3 / 40.1
        if (N == 64 && each <= 30 && (each + 11) / 12 < (each + 7) / 8) return launch_as<12>(ecfw_decode_kernel<FMT, 64, 12, 4>, a, max_workgroups, s);
        if (N == 64) return launch_as<8>(ecfw_decode_kernel<FMT, 64, 8, 4>, a, max_workgroups, s);
        // N = 128 has registers for two bursts of a chunk, which pay from the third round of chunks on.  Four bursts / two, us, by chunks
        // per workgroup: 8 19.3 / 19.5, 16 27.9 / 28.6, 17 32.7 / 32.4, 25 44.6 / 42.6, 48 75.3 / 73.3, 104 147.3 / 139.9
        if (each <= 16) return launch_as<8>(ecfw_decode_kernel<FMT, 128, 8, 2>, a, max_workgroups, s);
        return launch_as<8>(ecfw_decode_kernel<FMT, 128, 8, 4>, a, max_workgroups, s);
    } else {
        return N == 64 ? launch_as<12>(ecfw_decode_kernel<FMT, 64, 12, 2>, a, max_workgroups, s)
                       : launch_as<12>(ecfw_decode_kernel<FMT, 128, 12, 2>, a, max_workgroups, s);
    }
}

int launch(const BArgs &a, uint32_t fmt, uint32_t N, uint32_t max_code_len, uint32_t max_workgroups, void *stream)
{
    const bool fast = max_code_len <= ECFW_TABLE_BITS;
    hipStream_t s = (hipStream_t)stream;
    return fmt == ECFW_FMT_BF16 ? launch_fmt<ECFW_FMT_BF16>(a, N, fast, max_workgroups, s)
                                : launch_fmt<ECFW_FMT_E5M2>(a, N, fast, max_workgroups, s);
}

// A batch of more chunks than a launch counts (8 TiB or more), by the kernels that take every code
int launch_far(BArgs a, uint32_t fmt, uint32_t N, uint32_t max_workgroups, hipStream_t s)
{
    const uint64_t all = a.total_chunks;
    for (a.base = 0; a.base < all; a.base += LAUNCH_CHUNKS) {
        a.total_chunks = all - a.base < LAUNCH_CHUNKS ? all - a.base : LAUNCH_CHUNKS;
        const int rc = fmt == ECFW_FMT_BF16 ? (N == 64 ? launch_as<8>(ecfw_long_decode_kernel<ECFW_FMT_BF16, 64, 8, true>, a, max_workgroups, s)
                                                       : launch_as<8>(ecfw_long_decode_kernel<ECFW_FMT_BF16, 128, 8, true>, a, max_workgroups, s))
                                            : (N == 64 ? launch_as<8>(ecfw_long_decode_kernel<ECFW_FMT_E5M2, 64, 8, true>, a, max_workgroups, s)
                                                       : launch_as<8>(ecfw_long_decode_kernel<ECFW_FMT_E5M2, 128, 8, true>, a, max_workgroups, s));
        if (rc) return rc;
    }
    return ECF8_OK;
}

// Checks of one tensor's header and buffers; fills the kernel's view of it.
int make_item(const ecfw_header *h, const void *d_blob, void *d_out, uint64_t out_capacity, WArgs *it)
{
    if (!d_blob || !h || !d_out) return ECF8_E_ARG;
    if (h->magic != ECFW_MAGIC || h->version != ECFW_VERSION) return ECF8_E_FORMAT;
    if (h->fmt != ECFW_FMT_E5M2 && h->fmt != ECFW_FMT_BF16) return ECF8_E_FORMAT;
    if (h->lane_syms != 64 && h->lane_syms != 128) return ECF8_E_FORMAT;
    const uint32_t g = h->group_chunks;
    if (g < 1 || g > 64 || (g & (g - 1))) return ECF8_E_FORMAT;
    if (h->n_elem == 0 || h->n_chunks != (h->n_elem + 64ull * h->lane_syms - 1) / (64ull * h->lane_syms)) return ECF8_E_FORMAT;
    if (h->n_chunks > LAUNCH_CHUNKS) return ECF8_E_FORMAT;
    if (h->max_code_len < 1 || h->max_code_len > ECFW_MAX_CODE_LEN || h->stream_bytes < 16 || h->stream_bytes % 16)
        return ECF8_E_FORMAT;
    const uint64_t elem = h->fmt == ECFW_FMT_BF16 ? 2 : 1;
    if (out_capacity / elem < h->n_elem) return ECF8_E_CAPACITY;
    if (((uintptr_t)d_blob & 255) || ((uintptr_t)d_out & 15)) return ECF8_E_ALIGN;
    if ((h->off_code_len | h->off_chunk_bit | h->off_lane_bits | h->off_stream | h->off_plane | h->off_sign) & 255)
        return ECF8_E_FORMAT;
    std::memset(it, 0, sizeof(*it));
    it->d_blob = (uint64_t)(uintptr_t)d_blob;
    it->d_out = (uint64_t)(uintptr_t)d_out;
    it->n_elem = h->n_elem;
    it->n_chunks = h->n_chunks;
    it->first_chunk = 0;
    it->stream_bytes = h->stream_bytes;
    it->off_code_len = h->off_code_len;
    it->off_chunk_bit = h->off_chunk_bit;
    it->off_lane_bits = h->off_lane_bits;
    it->off_stream = h->off_stream;
    it->off_plane = h->off_plane;
    it->off_sign = h->off_sign;
    it->group_chunks = g;
    return ECF8_OK;
}

} // namespace

extern "C" int ecfw_decode(const void *d_blob, const ecfw_header *h, void *d_out, uint64_t out_capacity,
                           uint32_t max_workgroups, void *stream)
{
    BArgs a;
    int rc = make_item(h, d_blob, d_out, out_capacity, &a.single);
    if (rc) return rc;
    a.items = nullptr;
    a.n_items = 1;
    a.total_chunks = h->n_chunks;
    return launch(a, h->fmt, h->lane_syms, h->max_code_len, max_workgroups, stream);
}

extern "C" int ecfw_batch_prepare(const ecfw_header *hdrs, const void *const *d_blobs, void *const *d_outs,
                                  const uint64_t *out_capacities, uint32_t n, ecfw_batch_item *items_host,
                                  ecfw_batch_info *info)
{
    if (!hdrs || !d_blobs || !d_outs || !out_capacities || !items_host || !info || n == 0) return ECF8_E_ARG;
    std::memset(info, 0, sizeof(*info));
    uint64_t chunks = 0;
    for (uint32_t i = 0; i < n; i++) {
        int rc = make_item(&hdrs[i], d_blobs[i], d_outs[i], out_capacities[i], &items_host[i]);
        if (rc) return rc;
        if (hdrs[i].fmt != hdrs[0].fmt || hdrs[i].lane_syms != hdrs[0].lane_syms) return ECF8_E_ARG;
        items_host[i].first_chunk = chunks;
        chunks += hdrs[i].n_chunks;
        if (hdrs[i].max_code_len > info->max_code_len) info->max_code_len = hdrs[i].max_code_len;
    }
    info->total_chunks = chunks;
    info->fmt = hdrs[0].fmt;
    info->lane_syms = hdrs[0].lane_syms;
    return ECF8_OK;
}

extern "C" int ecfw_decode_batched(const void *d_items, uint32_t n, const ecfw_batch_info *info, void *stream)
{
    if (!d_items || !info || n == 0 || info->total_chunks == 0) return ECF8_E_ARG;
    if (info->fmt != ECFW_FMT_E5M2 && info->fmt != ECFW_FMT_BF16) return ECF8_E_ARG;
    if (info->lane_syms != 64 && info->lane_syms != 128) return ECF8_E_ARG;
    if (info->max_code_len < 1 || info->max_code_len > ECFW_MAX_CODE_LEN) return ECF8_E_ARG;
    if ((uintptr_t)d_items & 7) return ECF8_E_ALIGN;
    BArgs a;
    std::memset(&a.single, 0, sizeof(a.single));
    a.items = (const GLOBAL WArgs *)d_items;
    a.n_items = n;
    a.total_chunks = info->total_chunks;
    if (a.total_chunks > LAUNCH_CHUNKS) return launch_far(a, info->fmt, info->lane_syms, info->max_workgroups, (hipStream_t)stream);
    return launch(a, info->fmt, info->lane_syms, info->max_code_len, info->max_workgroups, stream);
}
