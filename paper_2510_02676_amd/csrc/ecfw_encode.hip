// GPU-side encoder of the wide-alphabet codec (E5M2, BF16) for gfx950: Section 3.1 on the device
// for 5- and 8-bit exponent fields.  Writes exactly the container ecfw_encode writes, byte for byte:
// the same code under every cap, ties included, and the layout from the same routines.
//
//   histograms of ranges of chunks -> code, places of the ranges in the stream, header, code lengths, histogram (one workgroup; the host waits for the
//   header) -> everything else, as in the E4M3 encoder (encode_range).
// No scratch memory on the device: the ranges' histograms lie where the stream will.
#include "ecfw.h"

#include "ecf8_enc_device.h"
#include "ecfw_plan.h"

namespace {

struct WEncArgs {
    uint64_t x, blob;                     // device addresses
    uint64_t n, n_chunks;
    uint64_t off_cb, off_lb, off_st, off_pl, off_sg;
    uint32_t group;
};

template <int FMT> struct EFmt;
template <> struct EFmt<ECFW_FMT_E5M2> {
    static constexpr int P = 16, ELEM = 1, A = 32;
    // exponent field of element j of a piece's four dwords
    static __device__ __forceinline__ uint32_t sym(const uint32_t (&w)[4], int j) { return (w[j >> 2] >> (8 * (j & 3) + 2)) & 31u; }
};
template <> struct EFmt<ECFW_FMT_BF16> {
    static constexpr int P = 8, ELEM = 2, A = 256;
    static __device__ __forceinline__ uint32_t sym(const uint32_t (&w)[4], int j) { return (w[j >> 1] >> (16 * (j & 1) + 7)) & 255u; }
};

template <int FMT, int N>
__device__ __forceinline__ ChunkPlace place_of(const WEncArgs &a, uint64_t c, uint32_t lane)
{
    constexpr uint64_t E = 64ull * N, P = EFmt<FMT>::P;
    const uint64_t grouped = (a.n / E) & ~((uint64_t)a.group - 1);
    const uint64_t w = c & (a.group - 1);
    if (c < grouped) return {(c - w) * E + w * 64 * P, (uint64_t)a.group * 64 * P, lane * P};
    return {c * E, 64 * P, lane * P};
}

// Histogram of the exponent field of each range into a record of A u32, one workgroup of 16 waves.
//  * E5M2: bit planes.  32 elements are turned into five 32-bit words, one per exponent bit, and each of the 32 exponents
//    is one AND and one population count that also adds: four vector operations per element, no LDS.
//  * BF16: LDS counters in 64 copies, lane l of every wave in copy l = bank l, so that the lanes of a wave, most of which
//    hold one of a handful of exponents, never meet.  (16 copies: 47 us instead of 21 for 58.7 M elements.)
// 58.7 M elements in a kernel trace: E5M2 18.3 us with the counts added to one record and summed by scans, 11.6 now; BF16 21.8 and 19.4, the read.
template <int FMT, int N>
__global__ __launch_bounds__(1024) void w_histogram_kernel(WEncArgs a, Ranges rg, uint64_t records)
{
    constexpr int A = EFmt<FMT>::A, COPIES = FMT == ECFW_FMT_BF16 ? 64 : 1;
    __shared__ uint32_t s_cnt[A * COPIES];
    const GLOBAL uint8_t *x = (const GLOBAL uint8_t *)a.x;
    GLOBAL uint32_t *record = (GLOBAL uint32_t *)records + (uint64_t)blockIdx.x * A;
    const int tid = threadIdx.x, lane = tid & 63;
    for (int i = tid; i < A * COPIES; i += 1024) s_cnt[i] = 0;
    __syncthreads();
    uint32_t cnt[FMT == ECFW_FMT_E5M2 ? 32 : 1];
    if constexpr (FMT == ECFW_FMT_E5M2)
#pragma unroll
        for (int s = 0; s < 32; s++) cnt[s] = 0;
    auto count = [&](const u32x4 &va, const u32x4 &vb) {
        const uint32_t w[8] = {va.x, va.y, va.z, va.w, vb.x, vb.y, vb.z, vb.w};
        if constexpr (FMT == ECFW_FMT_E5M2) {
            uint32_t t[4], u[4];
#pragma unroll
            for (int i = 0; i < 4; i++) {
                t[i] = bit_select(0x0f0f0f0fu, w[2 * i] >> 3, w[2 * i + 1] << 1);       // the upper four exponent bits in nibbles
                u[i] = bit_select(0x0f0f0f0fu, w[2 * i] >> 2, w[2 * i + 1] << 2);       // the lowest one at the bottom of a nibble
            }
            const uint32_t a0 = bit_select(0x55555555u, t[0], t[1] << 1), a1 = bit_select(0x55555555u, t[0] >> 1, t[1]);
            const uint32_t b0 = bit_select(0x55555555u, t[2], t[3] << 1), b1 = bit_select(0x55555555u, t[2] >> 1, t[3]);
            const uint32_t p1 = bit_select(0x33333333u, a0, b0 << 2), p3 = bit_select(0x33333333u, a0 >> 2, b0);
            const uint32_t p2 = bit_select(0x33333333u, a1, b1 << 2), p4 = bit_select(0x33333333u, a1 >> 2, b1);
            const uint32_t p0 = bit_select(0x33333333u, bit_select(0x11111111u, u[0], u[1] << 1), bit_select(0x11111111u, u[2], u[3] << 1) << 2);
#pragma unroll
            for (int s = 0; s < 32; s++) {
                const uint32_t hi = (s & 16 ? p4 : ~p4) & (s & 8 ? p3 : ~p3) & (s & 4 ? p2 : ~p2);
                const uint32_t lo = (s & 2 ? p1 : ~p1) & (s & 1 ? p0 : ~p0);
                cnt[s] += (uint32_t)__builtin_popcount(hi & lo);
            }
        } else {
#pragma unroll
            for (int k = 0; k < 8; k++) {
                atomicAdd(&s_cnt[((w[k] >> 7) & 255u) * COPIES + lane], 1u);
                atomicAdd(&s_cnt[((w[k] >> 23) & 255u) * COPIES + lane], 1u);
            }
        }
    };
    // a wave takes four pieces of 1 KiB per step
    constexpr uint32_t STEPS = N / EFmt<FMT>::P / 4;
    const uint64_t first = rg.begin(blockIdx.x);
    const uint32_t size = rg.size(blockIdx.x), whole = size - ((first + size) * (64ull * N) > a.n ? 1u : 0u);
    for (uint32_t i = uniform32(tid >> 6); i < whole * STEPS; i += 16) {
        const ChunkPlace p = place_of<FMT, N>(a, first + whole - 1 - i / STEPS, (uint32_t)lane);       // the first chunks last: the next reader begins with them
        const GLOBAL uint8_t *at = x + (p.base + p.lane_off + i % STEPS * 4 * p.stride) * EFmt<FMT>::ELEM;
        u32x4 v[4];
#pragma unroll
        for (int j = 0; j < 4; j++) v[j] = *(const GLOBAL u32x4 *)(at + j * p.stride * EFmt<FMT>::ELEM);
        count(v[0], v[1]);
        count(v[2], v[3]);
    }
    if (whole != size)
        for (uint64_t i = (first + whole) * (64ull * N) + tid; i < a.n; i += 1024) {
            const uint32_t s = FMT == ECFW_FMT_E5M2 ? (x[i] >> 2) & 31u : (((const GLOBAL uint16_t *)x)[i] >> 7) & 255u;
            atomicAdd(&s_cnt[s * COPIES + (COPIES > 1 ? lane : 0)], 1u);
        }
    if constexpr (FMT == ECFW_FMT_E5M2) {
        add_counts<32>(cnt, s_cnt, lane);
        __syncthreads();
        if (tid < A) record[tid] = s_cnt[tid];
    } else {
        __syncthreads();
        // four threads per exponent, 16 copies each, started apart so that a wave's reads fall into different banks
        const int s = tid >> 2, part = tid & 3;
        uint32_t sum = 0;
#pragma unroll
        for (int k = 0; k < 16; k++) sum += s_cnt[s * COPIES + part * 16 + ((k + s) & 15)];
        sum += __shfl_xor(sum, 1, 64);
        sum += __shfl_xor(sum, 2, 64);
        if (part == 0) record[s] = sum;
    }
}

// What plan_kernel has to know of these codecs.
template <int FMT>
struct WCodec {
    static constexpr int A = EFmt<FMT>::A;
    typedef ecfw_header Header;
    static __device__ __forceinline__ uint64_t sign_bytes(const Header &h) { return h.sign_bytes; }
    static __device__ __forceinline__ void finish(Header &h, GLOBAL uint8_t *blob, uint64_t off_sign, const uint64_t *freq, const uint32_t *len, uint32_t m, uint32_t longest, bool write, int lane)
    {
        if (lane == 0) {
            h.max_code_len = longest;
            h.n_symbols = m;
            h.off_sign = off_sign;
        }
        if (!write) return;
        uint32_t four = 0;                                  // zeros behind the last
        if (4 * lane < A) four = len[4 * lane] | len[4 * lane + 1] << 8 | len[4 * lane + 2] << 16 | len[4 * lane + 3] << 24;
        ((GLOBAL uint32_t *)(blob + h.off_code_len))[lane] = four;
        for (int s = lane; s < A; s += 64) ((GLOBAL uint64_t *)(blob + h.off_freq))[s] = freq[s];
    }
};

// What of the container is neither chunk data nor stream, header or code, by the first workgroup: zeros in the gaps between sections and behind the last dword of the stream.
__device__ __forceinline__ void write_fixed(const WEncArgs &a, const __attribute__((address_space(4))) ecfw_header &h)
{
    if (blockIdx.x != 0) return;
    const uint32_t tid = threadIdx.x;
    GLOBAL uint8_t *blob = (GLOBAL uint8_t *)a.blob;
    auto zero = [&](uint64_t from, uint64_t to) {       // multiples of four
        for (uint64_t i = from + 4 * tid; i < to; i += 4 * blockDim.x) *(GLOBAL uint32_t *)(blob + i) = 0;
    };
    zero(a.off_cb + 8 * (a.n_chunks + 1), a.off_lb);
    zero(a.off_lb + 128 * a.n_chunks, a.off_st);
    zero(a.off_st + ((h.stream_bits + 31) >> 5) * 4, a.off_pl);
    zero(a.off_pl + h.plane_bytes, h.sign_bytes ? a.off_sg : h.total_size);
    if (h.sign_bytes) zero(a.off_sg + h.sign_bytes, h.total_size);
}

// A chunk on its way through encode_range, as in the E4M3 encoder.  LMAX: the longest codeword in use is at most this.  Look-ups:
//  * BF16 one symbol at a time (256 of them would make a pair table of 256 KiB), E5M2 up to 12 bits two at a time; codeword(s) and from
//    bit 27 on their length in one dword, so that joining two of them is one operation.
//  * QUADS (up to 12 bits): count joins four codewords and leaves them in the place of their elements, for pack to put them in one go.
//    They are nearly always less than 32 bits; a chunk where they are not is fetched again and packed two codewords at a time.
template <int FMT, int N, int LMAX>
struct Chunk {
    using F = EFmt<FMT>;
    static constexpr int P = F::P, A = F::A, PIECES = N / P;
    static constexpr bool ANY = LMAX > 15;                                          // two codewords may have 32 bits
    static constexpr bool QUADS = LMAX <= 12 && PIECES <= 8, PAIRS = QUADS && FMT == ECFW_FMT_E5M2;
    static constexpr uint32_t BITS = (1u << 27) - 1;                                // of a dword that holds codewords and their length
    static constexpr int PAIR_ENTRIES = PAIRS ? A * A : 1;
    static constexpr int MOST = (160 * 1024 - 4096 - 8 * (A + 1) - 256 - 8 * PAIR_ENTRIES) / (4 * WMAX) / 4 * 4;
    static constexpr int AREA = 2 * N * LMAX + 4 < MOST ? 2 * N * LMAX + 4 : MOST;   // a chunk whatever it is, if there is room
    static_assert(N * LMAX + 4 <= AREA && AREA % 4 == 0, "half a chunk");

    const WEncArgs &a;
    const uint32_t (*code)[A + 1];          // code | length << 27, first bit lowest / highest; A = no symbol
    const uint32_t (*pair)[PAIR_ENTRIES];   // two codewords and from bit 27 on their length, in order / in reverse
    const uint8_t *len;
    int lane;
    u32x4 v[PIECES];
    bool wide;                              // QUADS: there are four codewords of 32 bits or more

    __device__ __forceinline__ bool whole(uint64_t c) const { return (c + 1) * (64ull * N) <= a.n; }
    __device__ __forceinline__ void fetch(uint64_t c)
    {
        const ChunkPlace p = place_of<FMT, N>(a, c, lane);
        const GLOBAL uint8_t *x = (const GLOBAL uint8_t *)a.x + (p.base + p.lane_off) * F::ELEM;
#pragma unroll
        for (int q = 0; q < PIECES; q++) v[q] = *(const GLOBAL u32x4 *)(x + q * p.stride * F::ELEM);
    }
    // the planes of the piece at element e
    __device__ __forceinline__ void planes(uint64_t e, const u32x4 &w) const
    {
        GLOBAL uint8_t *plane = (GLOBAL uint8_t *)(a.blob + a.off_pl), *signs = (GLOBAL uint8_t *)(a.blob + a.off_sg);
        if constexpr (FMT == ECFW_FMT_BF16) {
            // sign << 7 | mantissa in bytes 0 and 2 of a dword's two elements; the bytes of four elements in the order 0 2 1 3
            const uint32_t r0 = bit_select(0x007f007fu, w.x, w.x >> 8), r1 = bit_select(0x007f007fu, w.y, w.y >> 8);
            const uint32_t r2 = bit_select(0x007f007fu, w.z, w.z >> 8), r3 = bit_select(0x007f007fu, w.w, w.w >> 8);
            *(GLOBAL u32x2 *)(plane + e) = u32x2{bit_select(0x00ff00ffu, r0, r1 << 8), bit_select(0x00ff00ffu, r2, r3 << 8)};
        } else {
            // mantissa of element 4d + j in bits 8j + 2d; sign of element i in bit i
            const uint32_t m01 = bit_select(0x03030303u, w.x, w.y << 2), m23 = bit_select(0x03030303u, w.z, w.w << 2);
            auto signs4 = [](uint32_t d) {
                uint32_t y = (d >> 7) & 0x01010101u;
                y |= y >> 7;
                return (y | (y >> 14)) & 15u;
            };
            *(GLOBAL uint32_t *)(plane + e / 4) = bit_select(0x0f0f0f0fu, m01, m23 << 4);
            *(GLOBAL uint16_t *)(signs + e / 8) = (uint16_t)(signs4(w.x) | (signs4(w.y) << 4) | (signs4(w.z) << 8) | (signs4(w.w) << 12));
        }
    }
    __device__ __forceinline__ uint32_t count(uint64_t c)
    {
        const ChunkPlace p = place_of<FMT, N>(a, c, lane);
        uint32_t lb = 0, most = 0;
#pragma unroll
        for (int i = 0; i < PIECES; i++) {
            const int q = i < PIECES / 2 ? i : PIECES - 1 - (i - PIECES / 2);       // in the order in which pack asks for them
            planes(p.base + p.lane_off + q * p.stride, v[q]);
            uint32_t w[4] = {v[q].x, v[q].y, v[q].z, v[q].w};
            const int back = i < PIECES / 2 ? 0 : 1;
            if constexpr (PAIRS) {
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    const uint32_t u = pair_index(w[k]), e0 = pair[back][u & 1023u], e1 = pair[back][(u >> 16) & 1023u];
                    const uint32_t x0 = back ? e1 : e0, x1 = back ? e0 : e1, n0 = x0 >> 27, nb = n0 + (x1 >> 27);
                    most |= nb;
                    lb += nb;
                    w[k] = (x0 & BITS) | ((x1 & BITS) << n0) | (1u << (nb & 31u));      // a one above the codewords says how many bits they are
                }
            } else if constexpr (QUADS) {
                uint32_t r[4];
#pragma unroll
                for (int k = 0; k < 2; k++) {
                    uint32_t x[4], n0, n1, nb;              // in the order in which pack puts them
#pragma unroll
                    for (int j = 0; j < 4; j++) x[j] = code[back][F::sym(w, back ? 7 - 4 * k - j : 4 * k + j)];
                    const uint32_t p0 = joined(x[0], x[1], n0), p1 = joined(x[2], x[3], n1);
                    nb = n0 + n1;
                    r[2 * k] = p0 | (p1 << (n0 & 31u));
                    r[2 * k + 1] = nb;
                    most |= nb;
                    lb += nb;
                }
#pragma unroll
                for (int k = 0; k < 4; k++) w[k] = r[k];
            } else {
#pragma unroll
                for (int j = 0; j < P; j++) lb += len[F::sym(w, j)];
            }
            if constexpr (QUADS) v[q] = u32x4{w[0], w[1], w[2], w[3]};
        }
        wide = __ballot(most & 32u) != 0;
        return lb;
    }
    // two codewords (27 bits at the most) one behind the other, and the length of both
    static __device__ __forceinline__ uint32_t joined(uint32_t x0, uint32_t x1, uint32_t &nb)
    {
        const uint32_t l0 = x0 >> 27;
        nb = l0 + (x1 >> 27);
        return (x0 | (x1 << l0)) & BITS;                    // x1's length lands above the codewords
    }
    // E5M2: exponents of a dword's elements 0 and 1 in bits 0 .. 9, of 2 and 3 in bits 16 .. 25, others not 0
    static __device__ __forceinline__ uint32_t pair_index(uint32_t w)
    {
        const uint32_t t = (w >> 2) & 0x1f1f1f1fu;
        return bit_select(0x001f001fu, t, t >> 3);
    }
    static __device__ __forceinline__ void put2(LanePacker<ANY> &out, uint32_t x0, uint32_t x1)
    {
        uint32_t nb;
        const uint32_t x = LMAX <= 13 ? joined(x0, x1, nb) : (x0 & 0xffffu) | ((x1 & 0xffffu) << (x0 >> 27));
        out.put(x, LMAX <= 13 ? nb : (x0 >> 27) + (x1 >> 27));
    }
    template <bool BACK>
    __device__ __forceinline__ void put_piece(LanePacker<ANY> &out, const u32x4 &v4) const
    {
        const uint32_t w[4] = {v4.x, v4.y, v4.z, v4.w};
#pragma unroll
        for (int j = 0; j < P; j += 2)
            put2(out, code[BACK][F::sym(w, BACK ? P - 1 - j : j)], code[BACK][F::sym(w, BACK ? P - 2 - j : j + 1)]);
    }
    // what count has left of a piece
    template <bool BACK>
    __device__ __forceinline__ void put_quads(LanePacker<ANY> &out, const u32x4 &v4) const
    {
        const uint32_t w[4] = {v4.x, v4.y, v4.z, v4.w};
        if constexpr (PAIRS) {
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const uint32_t x = w[BACK ? 3 - k : k];
                out.put(x, 31u ^ (uint32_t)__builtin_clz(x));
            }
        } else {
            out.put(w[0], w[1]);
            out.put(w[2], w[3]);
        }
    }
    __device__ __forceinline__ void pack(uint32_t *image, uint32_t at, uint64_t c, uint64_t next, bool refill)
    {
        LanePacker<ANY> out(image, at);
        if (QUADS && wide) fetch(c);
        const ChunkPlace p = place_of<FMT, N>(a, next, lane);
        const GLOBAL uint8_t *x = (const GLOBAL uint8_t *)a.x + (p.base + p.lane_off) * F::ELEM;
        if (!QUADS || wide) {
#pragma unroll
            for (int i = 0; i < PIECES; i++) {
                const int q = i < PIECES / 2 ? i : PIECES - 1 - (i - PIECES / 2);
                if (i < PIECES / 2) put_piece<false>(out, v[q]); else put_piece<true>(out, v[q]);
                if (refill) v[q] = *(const GLOBAL u32x4 *)(x + q * p.stride * F::ELEM);
            }
        } else {
#pragma unroll
            for (int i = 0; i < PIECES; i++) {
                const int q = i < PIECES / 2 ? i : PIECES - 1 - (i - PIECES / 2);
                if (i < PIECES / 2) put_quads<false>(out, v[q]); else put_quads<true>(out, v[q]);
                if (refill) v[q] = *(const GLOBAL u32x4 *)(x + q * p.stride * F::ELEM);
            }
        }
        out.finish();
    }
    // any chunk, piece by piece; symbols past the tensor's end have no bits
    __device__ __forceinline__ void piece(const u32x4 &v4, uint64_t e, uint32_t back, uint32_t (&s)[P]) const
    {
        const uint32_t w[4] = {v4.x, v4.y, v4.z, v4.w}, have = e + P <= a.n ? (uint32_t)P : e < a.n ? (uint32_t)(a.n - e) : 0u;
#pragma unroll
        for (int j = 0; j < P; j++) s[j] = code[back][(uint32_t)j < have ? F::sym(w, j) : (uint32_t)A];
    }
    __device__ __forceinline__ u32x4 slow_fetch(uint64_t e) const { return load_cut((const GLOBAL uint8_t *)a.x, e * F::ELEM, a.n * F::ELEM); }
    __device__ __forceinline__ uint32_t slow_count(uint64_t c)
    {
        const ChunkPlace p = place_of<FMT, N>(a, c, lane);
        uint32_t lb = 0;
#pragma unroll 1
        for (int q = 0; q < PIECES; q++) {
            const uint64_t e = p.base + p.lane_off + q * p.stride;
            uint32_t s[P];
            const u32x4 w = slow_fetch(e);
            piece(w, e, 0, s);
#pragma unroll
            for (int j = 0; j < P; j++) lb += s[j] >> 27;
            planes(e, w);
        }
        return lb;
    }
    __device__ __forceinline__ void slow_pack(uint32_t *image, uint32_t at, uint64_t c)
    {
        const ChunkPlace p = place_of<FMT, N>(a, c, lane);
        LanePacker<ANY> out(image, at);
        const uint64_t e0 = p.base + p.lane_off;
        const uint32_t stride = (uint32_t)p.stride;
        auto at_piece = [&](int i) { return e0 + (uint32_t)(i >= PIECES / 2 ? PIECES - 1 - (i - PIECES / 2) : i) * stride; };
#pragma unroll 1
        for (int i = 0; i < PIECES; i++) {
            const bool back = i >= PIECES / 2;
            const u32x4 w = slow_fetch(at_piece(i));
            uint32_t s[P];
            piece(w, at_piece(i), back ? 1 : 0, s);
#pragma unroll
            for (int j = 0; j < P; j += 2) put2(out, back ? s[P - 1 - j] : s[j], back ? s[P - 2 - j] : s[j + 1]);
        }
        out.finish();
    }
    // the last 32 bits of a whole chunk: those of the first codewords of lane 63's backward run, of which each lane looks up one
    __device__ __forceinline__ uint32_t tail(uint64_t c) const
    {
        const ChunkPlace p = place_of<FMT, N>(a, c, 63);
        const uint32_t s = N / 2 + ((uint32_t)lane & 31);
        const uint64_t e = p.base + p.lane_off + s / P * p.stride + s % P;
        const GLOBAL uint8_t *x = (const GLOBAL uint8_t *)a.x;
        const uint32_t v = code[1][FMT == ECFW_FMT_E5M2 ? (x[e] >> 2) & 31u : (((const GLOBAL uint16_t *)x)[e] >> 7) & 255u];
        return last_bits(v & BITS, v >> 27, lane);
    }
};

// The container behind the code.  58.7 M elements (14336 x 4096): in a kernel trace BF16 34.4 us for the 198 MB read and written, nearly a copy's rate, and E5M2 27.2,
// three quarters of it vector operations (42.7 and 35.6 when the workgroups had to find their place in the stream from one another).  The whole call,
// one input over and over, from the memory-side cache, 74.3 -> 64.6 and 63.7 -> 45.4 (BF16 from memory 84.5 -> 73.0), 14336 x 14336 252 -> 215 and 160 -> 120.
template <int FMT, int N, int LMAX>
__global__ __launch_bounds__(WMAX * 64) void w_encode_kernel(WEncArgs a, Ranges rg)
{
    using K = Chunk<FMT, N, LMAX>;
    constexpr int A = K::A;
    __shared__ struct {                                     // the tables where a look-up needs no address of theirs
        uint32_t pair[2][K::PAIR_ENTRIES];
        uint32_t code[2][A + 1];
        uint32_t len4[64];
        RangeShared range;
        __attribute__((aligned(16))) uint32_t images[WMAX][K::AREA];
    } s;
    const uint32_t tid = threadIdx.x;
    const int wave = (int)uniform32(tid >> 6), lane = (int)(tid & 63);
    // before the first chunk is asked for: loads come back in order
    const uint32_t four = wave == 0 ? ((const GLOBAL uint32_t *)(a.blob + 256))[lane] : 0u;
    K k{a, s.code, s.pair, (const uint8_t *)s.len4, lane, {}, false};
    const uint64_t c0 = rg.begin(blockIdx.x) + wave;
    if ((uint32_t)wave < rg.size(blockIdx.x) && k.whole(c0)) k.fetch(c0);
    const auto &h = planned<ecfw_header>(a.blob);
    if (h.magic == 0) return;                               // no blob
    a.off_pl = h.off_plane;
    a.off_sg = h.off_sign;
    range_begin(s.range);
    if (wave == 0) {
        s.len4[lane] = four;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        // canonical codewords: lane l has symbols l, l + 64, ..., ranked among those of their length
        constexpr int PER = (A + 63) / 64;
        uint32_t len[PER], code[PER], begin = 0;
#pragma unroll
        for (int i = 0; i < PER; i++) {
            len[i] = lane + 64 * i < A ? ((const uint8_t *)s.len4)[lane + 64 * i] : 0u;
            code[i] = 0;
        }
#pragma unroll 1
        for (uint32_t l = 1; l <= (uint32_t)LMAX; l++) {
#pragma unroll
            for (int i = 0; i < PER; i++) {
                const uint64_t there = __ballot(len[i] == l);
                code[i] = len[i] == l ? begin + (uint32_t)__builtin_popcountll(there & ((1ull << lane) - 1)) : code[i];
                begin += (uint32_t)__builtin_popcountll(there);
            }
            begin <<= 1;
        }
#pragma unroll
        for (int i = 0; i < PER; i++)
            if (lane + 64 * i < A) {
                s.code[0][lane + 64 * i] = len[i] ? (__brev(code[i]) >> (32 - len[i])) | (len[i] << 27) : 0u;
                s.code[1][lane + 64 * i] = code[i] | (len[i] << 27);
            }
        if (lane < 2) s.code[lane][A] = 0;
    }
    __syncthreads();
    if constexpr (K::PAIRS) {
        for (uint32_t i = tid; i < (uint32_t)K::PAIR_ENTRIES; i += blockDim.x) {
            const uint32_t lo = i % A, hi = i / A;          // an entry's first and second element
            uint32_t nb;
            s.pair[0][i] = K::joined(s.code[0][lo], s.code[0][hi], nb);
            s.pair[1][i] = K::joined(s.code[1][hi], s.code[1][lo], nb) | (nb << 27);
            s.pair[0][i] |= nb << 27;
        }
        __syncthreads();
    }
    write_fixed(a, h);
    encode_range(k, s.range, s.images[wave], rg, (GLOBAL uint8_t *)a.blob, a.off_cb, a.off_lb, a.off_st, h.stream_bytes / 4, lane, wave);
}

template <int FMT, int N>
bool launch(const WEncArgs &a, const ecfw_header &h, const Ranges &rg, uint64_t capacity, uint32_t lmax, Mail &mail, hipStream_t s)
{
    const uint64_t records = a.blob + h.off_stream;
    static_assert(EFmt<FMT>::A * 4 <= 16 * N, "a record is smaller than a chunk's plane");
    const dim3 waves(range_waves(rg) * 64);
    hipLaunchKernelGGL((w_histogram_kernel<FMT, N>), dim3(rg.count), dim3(1024), 0, s, a, rg, records);
    if (!launched()) return false;
    hipLaunchKernelGGL(plan_kernel<WCodec<FMT>>, dim3(1), dim3(1024), 0, s, h, rg, a.blob, capacity, records, lmax, mail.device());
    if (!launched()) return false;
    // by the cap, the code is not known yet: BF16 under cap 16 67.6 us, under 12 64.6; when the longest codeword was known at the launch 76.9 and 74.3
    if (lmax <= ECFW_TABLE_BITS) hipLaunchKernelGGL((w_encode_kernel<FMT, N, (int)ECFW_TABLE_BITS>), dim3(rg.count), waves, 0, s, a, rg);
    else hipLaunchKernelGGL((w_encode_kernel<FMT, N, (int)ECFW_MAX_CODE_LEN>), dim3(rg.count), waves, 0, s, a, rg);
    return launched();
}

template <int FMT>
int encode_on_gpu(const void *d_elems, uint64_t rows, uint64_t cols, uint32_t N, uint32_t group, uint32_t lmax, void *d_blob,
                  uint64_t blob_capacity, ecfw_header *hdr_out, hipStream_t s)
{
    ecfw_header h;
    int rc = ecfw_internal::plan_frame(FMT, rows, cols, N, group, &h);
    if (rc) return rc;
    if (blob_capacity < h.off_stream + h.plane_bytes + h.sign_bytes) return ECF8_E_CAPACITY;      // no blob of this tensor is that small, and the ranges' histograms fit
    const int cus = device_cus();
    if (cus <= 0) return ECF8_E_HIP;

    WEncArgs a{};
    a.x = (uint64_t)(uintptr_t)d_elems;
    a.blob = (uint64_t)(uintptr_t)d_blob;
    a.n = h.n_elem;
    a.n_chunks = h.n_chunks;
    a.off_cb = h.off_chunk_bit;
    a.off_lb = h.off_lane_bits;
    a.off_st = h.off_stream;
    a.group = group;
    const Ranges rg = make_ranges(h.n_chunks, (uint32_t)cus);

    if (capturing(s)) return ECF8_E_HIP;
    Mail mail;
    if (!(N == 64 ? launch<FMT, 64>(a, h, rg, blob_capacity, lmax, mail, s) : launch<FMT, 128>(a, h, rg, blob_capacity, lmax, mail, s))) return ECF8_E_HIP;
    if (!mail.read(&h, a.blob, s)) return ECF8_E_HIP;
    if (h.magic == 0) return (int)h.version;
    *hdr_out = h;
    return ECF8_OK;
}

} // namespace

extern "C" {

int ecfw_encode_bound(uint64_t rows, uint64_t cols, const ecfw_encode_opts *opts, uint64_t *bytes)
{
    if (!bytes) return ECF8_E_ARG;
    uint32_t N, group, lmax;
    int rc = ecfw_internal::check_options(opts, rows, cols, &N, &group, &lmax);
    if (rc) return rc;
    return ecfw_internal::encode_bound(opts->fmt, rows, cols, N, lmax, bytes);
}

int ecfw_encode_gpu(const void *d_elems, uint64_t rows, uint64_t cols, const ecfw_encode_opts *opts, void *d_blob,
                    uint64_t blob_capacity, ecfw_header *hdr_out, void *stream)
{
    if (!d_elems || !d_blob || !hdr_out) return ECF8_E_ARG;
    uint32_t N, group, lmax;
    int rc = ecfw_internal::check_options(opts, rows, cols, &N, &group, &lmax);
    if (rc) return rc;
    if (((uintptr_t)d_elems & 15) || ((uintptr_t)d_blob & 255)) return ECF8_E_ALIGN;
    hipStream_t s = (hipStream_t)stream;
    return opts->fmt == ECFW_FMT_BF16
               ? encode_on_gpu<ECFW_FMT_BF16>(d_elems, rows, cols, N, group, lmax, d_blob, blob_capacity, hdr_out, s)
               : encode_on_gpu<ECFW_FMT_E5M2>(d_elems, rows, cols, N, group, lmax, d_blob, blob_capacity, hdr_out, s);
}

} // extern "C"
