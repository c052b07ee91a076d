// GPU-side encoder of the wide-alphabet codec (E5M2, BF16) for gfx950: Section 3.1 on the device
// for 5- and 8-bit exponent fields.  Writes exactly the container ecfw_encode writes, byte for byte:
// the code and the layout come from the same host routine, fed with the device histogram.
//
//   fill 0 (header, code lengths, freq) -> histogram (and zeros in chunk_bit[]), written to the host by its last workgroup -> [host: code + layout]
//   -> everything else in one pass over the elements, as in the E4M3 encoder (encode_tiles).
// No scratch memory on the device: the histogram is counted into the freq section, tiles are drawn from the header's first dword, and what the
// workgroups tell one another goes through chunk_bit[], all of them part of the output.
#include "ecfw.h"

#include "ecf8_enc_device.h"
#include "ecfw_plan.h"

namespace {

struct WEncArgs {
    uint64_t x, blob;                     // device addresses
    uint64_t n, n_chunks;
    uint64_t off_len, off_cb, off_lb, off_st, off_pl, off_sg;
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

// Histogram of the exponent field into A u64 counters, one workgroup of 16 waves per compute unit.
//  * E5M2: bit planes.  32 elements are turned into five 32-bit words, one per exponent bit, and each of the 32 exponents
//    is one AND and one population count that also adds: four vector operations per element, no LDS.
//  * BF16: LDS counters in 64 copies, lane l of every wave in copy l = bank l, so that the lanes of a wave, most of which
//    hold one of a handful of exponents, never meet.  58.7 M elements: 21 us, 5.5 TB/s (16 copies: 47 us).
template <int FMT>
__global__ __launch_bounds__(1024) void w_histogram_kernel(uint64_t x_, uint64_t n, uint64_t blob, uint64_t counters_, uint64_t chunk_bit, uint64_t n_chunks, uint64_t mail)
{
    constexpr int A = EFmt<FMT>::A, COPIES = FMT == ECFW_FMT_BF16 ? 64 : 1;
    __shared__ uint32_t s_cnt[A * COPIES];
    const GLOBAL uint8_t *x = (const GLOBAL uint8_t *)x_;
    GLOBAL unsigned long long *counters = (GLOBAL unsigned long long *)counters_;
    const int tid = threadIdx.x, lane = tid & 63;
    for (int i = tid; i < A * COPIES; i += 1024) s_cnt[i] = 0;
    zero_chunk_bits(chunk_bit, n_chunks, (uint32_t)tid, 1024);
    __syncthreads();
    // a wave takes 4 KiB per step: four loads of 1 KiB, of which a lane keeps the 16 bytes at 16 * lane
    constexpr uint64_t PER = 4096 / EFmt<FMT>::ELEM;
    const uint64_t steps = n / PER, stride = (uint64_t)gridDim.x * 16;
    const GLOBAL u32x4 *p = (const GLOBAL u32x4 *)x + lane;
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
    for (uint64_t i = (uint64_t)blockIdx.x * 16 + (tid >> 6); i < steps; i += stride) {
        const u32x4 va = p[i * 256], vb = p[i * 256 + 64], vc = p[i * 256 + 128], vd = p[i * 256 + 192];
        count(va, vb);
        count(vc, vd);
    }
    if (blockIdx.x == 0)
        for (uint64_t i = steps * PER + tid; i < n; i += 1024) {
            const uint32_t s = FMT == ECFW_FMT_E5M2 ? (x[i] >> 2) & 31u : (((const GLOBAL uint16_t *)x)[i] >> 7) & 255u;
            atomicAdd(&s_cnt[s * COPIES + (COPIES > 1 ? lane : 0)], 1u);
        }
    if constexpr (FMT == ECFW_FMT_E5M2) {
#pragma unroll
        for (int s = 0; s < 32; s++) {
            const uint32_t sum = wave_incl_scan(cnt[s]);
            if (lane == 63 && sum) atomicAdd(&s_cnt[s], sum);
        }
        __syncthreads();
        if (tid < A && s_cnt[tid]) atomicAdd((unsigned long long *)(counters + tid), (unsigned long long)s_cnt[tid]);
    } else {
        __syncthreads();
        // four threads per exponent, 16 copies each, started apart so that a wave's reads fall into different banks
        const int s = tid >> 2, part = tid & 3;
        uint32_t sum = 0;
#pragma unroll
        for (int k = 0; k < 16; k++) sum += s_cnt[s * COPIES + part * 16 + ((k + s) & 15)];
        sum += __shfl_xor(sum, 1, 64);
        sum += __shfl_xor(sum, 2, 64);
        if (part == 0 && sum) atomicAdd((unsigned long long *)(counters + s), (unsigned long long)sum);
    }
    mail_histogram<A>(blob, counters_, mail);
}

struct WCodeArgs {
    ecfw_header h;
    uint16_t code[256];                   // canonical codewords, first bit most significant
    uint8_t len[256];
};

// What of the container is neither chunk data nor stream, but for the header, by the first workgroup (the freq section already
// holds the histogram): code lengths, zeros in the gaps between sections and behind the last dword of the stream.
__device__ __forceinline__ void write_fixed(const WEncArgs &a, const WCodeArgs &ca)
{
    if (blockIdx.x != 0) return;
    const uint32_t tid = threadIdx.x;
    GLOBAL uint8_t *blob = (GLOBAL uint8_t *)a.blob;
    const ecfw_header &h = ca.h;
    if (tid * 4 < h.n_alphabet) *(GLOBAL uint32_t *)(blob + a.off_len + 4 * tid) = ((const uint32_t *)ca.len)[tid];
    auto zero = [&](uint64_t from, uint64_t to) {       // multiples of four
        for (uint64_t i = from + 4 * tid; i < to; i += 4 * blockDim.x) *(GLOBAL uint32_t *)(blob + i) = 0;
    };
    zero(a.off_cb + 8 * (a.n_chunks + 1), a.off_lb);
    zero(a.off_lb + 128 * a.n_chunks, a.off_st);
    zero(a.off_st + ((h.stream_bits + 31) >> 5) * 4, a.off_pl);
    zero(a.off_pl + h.plane_bytes, h.sign_bytes ? a.off_sg : h.total_size);
    if (h.sign_bytes) zero(a.off_sg + h.sign_bytes, h.total_size);
}

// A chunk on its way through encode_tiles, as in the E4M3 encoder.  The codewords come from the host with the launch.  LMAX: the longest codeword
// in use is at most this.  Look-ups:
//  * BF16 one symbol at a time (256 of them would make a pair table of 256 KiB), E5M2 up to 12 bits two at a time; codeword(s) and from
//    bit 27 on their length in one dword, so that joining two of them is one operation.
//  * QUADS (up to 12 bits): count joins four codewords and leaves them in the place of their elements, for pack to put them in one go.
//    They are nearly always less than 32 bits; a chunk where they are not is fetched again and packed two codewords at a time.
// What bounds it: BF16, at 4.7 TB/s, nearly a copy's rate; E5M2 the vector operations (with elements looked up one by one in count and again in
// pack the kernel took 5 us more for 14336 x 4096, BF16's 1).
template <int FMT, int N, int LMAX>
struct Chunk {
    using F = EFmt<FMT>;
    static constexpr int P = F::P, A = F::A, PIECES = N / P;
    static constexpr bool QUADS = LMAX <= 12 && PIECES <= 8, PAIRS = QUADS && FMT == ECFW_FMT_E5M2;
    static constexpr uint32_t BITS = (1u << 27) - 1;                                // of a dword that holds codewords and their length
    static constexpr int PAIR_ENTRIES = PAIRS ? A * A : 1;
    static constexpr int AREA = ((160 * 1024 - 1024 - 8 * (A + 1) - 256 - 8 * PAIR_ENTRIES) / (4 * WMAX) - 4) / 4 * 4;
    static constexpr int TAIL_FROM = PIECES - 32 / P;                               // a lane's last 32 codewords
    static_assert(32 * LMAX < 32 * LATE_DWORDS && N * LMAX * LATE_LANES <= 32 * (AREA - 4), "room for late chunks");

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
    static __device__ __forceinline__ void put2(LanePacker &out, uint32_t x0, uint32_t x1)
    {
        uint32_t nb;
        const uint32_t x = LMAX <= 13 ? joined(x0, x1, nb) : (x0 & 0xffffu) | ((x1 & 0xffffu) << (x0 >> 27));
        out.put(x, LMAX <= 13 ? nb : (x0 >> 27) + (x1 >> 27));
    }
    template <bool BACK>
    __device__ __forceinline__ void put_piece(LanePacker &out, const u32x4 &v4) const
    {
        const uint32_t w[4] = {v4.x, v4.y, v4.z, v4.w};
#pragma unroll
        for (int j = 0; j < P; j += 2)
            put2(out, code[BACK][F::sym(w, BACK ? P - 1 - j : j)], code[BACK][F::sym(w, BACK ? P - 2 - j : j + 1)]);
    }
    // what count has left of a piece
    template <bool BACK>
    __device__ __forceinline__ void put_quads(LanePacker &out, const u32x4 &v4) const
    {
        const uint32_t w[4] = {v4.x, v4.y, v4.z, v4.w};
        if constexpr (PAIRS) {
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const uint32_t x = w[BACK ? 3 - k : k], nb = 31u - (uint32_t)__builtin_clz(x);
                out.put(x ^ (1u << nb), nb);
            }
        } else {
            out.put(w[0], w[1]);
            out.put(w[2], w[3]);
        }
    }
    __device__ __forceinline__ void pack(uint32_t *image, uint32_t at, uint64_t c, bool refill)
    {
        LanePacker out(image, at);
        if (QUADS && wide) fetch(c);
        const ChunkPlace p = place_of<FMT, N>(a, c + 1, lane);
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
    // from the lane's i0-th piece on; the image's bit behind the last one
    __device__ __forceinline__ uint32_t slow_pack(uint32_t *image, uint32_t at, uint64_t c, int i0)
    {
        const ChunkPlace p = place_of<FMT, N>(a, c, lane);
        LanePacker out(image, at);
        const uint64_t e0 = p.base + p.lane_off;
        const uint32_t stride = (uint32_t)p.stride;
        auto at_piece = [&](int i) { return e0 + (uint32_t)(i >= PIECES / 2 ? PIECES - 1 - (i - PIECES / 2) : i) * stride; };
#pragma unroll 1
        for (int i = i0; i < PIECES; i++) {
            const bool back = i >= PIECES / 2;
            const u32x4 w = slow_fetch(at_piece(i));
            uint32_t s[P];
            piece(w, at_piece(i), back ? 1 : 0, s);
#pragma unroll
            for (int j = 0; j < P; j += 2) put2(out, back ? s[P - 1 - j] : s[j], back ? s[P - 2 - j] : s[j + 1]);
        }
        out.finish();
        return out.end(image);
    }
};

// The container behind the code.  58.7 M elements (14336 x 4096): in a kernel trace (the last 100 of 300 calls) BF16 42 us for the 198 MB read and
// written, E5M2 35 for 101 MB (some 20 more with metadata and planes, prefix sum and packing as kernels of their own).  The whole call 108 -> 84 us and
// 85 -> 64, 16384 x 16384 454 -> 310 and 250 -> 207.
template <int FMT, int N, int LMAX>
__global__ __launch_bounds__(WMAX * 64) void w_encode_kernel(WEncArgs a, WCodeArgs ca, uint32_t per_wave)
{
    using K = Chunk<FMT, N, LMAX>;
    constexpr int A = K::A;
    __shared__ __attribute__((aligned(16))) uint32_t images[WMAX][K::AREA + 4];  // the last of the four in front is image[-1]
    __shared__ uint32_t s_code[2][A + 1];
    __shared__ uint32_t s_pair[2][K::PAIR_ENTRIES];
    __shared__ uint32_t s_len4[64];
    __shared__ TileShared sh;
    const uint32_t tid = threadIdx.x;
    const int wave = (int)uniform32(tid >> 6);
    if (tid < (uint32_t)A) {
        const uint32_t code = ca.code[tid], l = ca.len[tid];
        s_code[0][tid] = l ? (__brev(code) >> (32 - l)) | (l << 27) : 0u;
        s_code[1][tid] = code | (l << 27);
    }
    if (tid < 2) s_code[tid][A] = 0;
    if (tid < 64) s_len4[tid] = ((const uint32_t *)ca.len)[tid];
    if constexpr (K::PAIRS) {
        __syncthreads();
        for (uint32_t i = tid; i < (uint32_t)K::PAIR_ENTRIES; i += blockDim.x) {
            const uint32_t lo = i % A, hi = i / A;          // an entry's first and second element
            uint32_t nb;
            s_pair[0][i] = K::joined(s_code[0][lo], s_code[0][hi], nb);
            s_pair[1][i] = K::joined(s_code[1][hi], s_code[1][lo], nb) | (nb << 27);
            s_pair[0][i] |= nb << 27;
        }
    }
    write_fixed(a, ca);
    K k{a, s_code, s_pair, (const uint8_t *)s_len4, (int)(tid & 63), {}, false};
    encode_tiles(k, sh, images[wave] + 4, TileArgs{a.n_chunks, per_wave, (const uint32_t *)&ca.h}, (GLOBAL uint8_t *)a.blob, a.off_cb, a.off_lb, a.off_st,
                 (int)(tid & 63), wave);
}

template <int FMT, int N, int LMAX>
int launch_encode(const WEncArgs &a, const WCodeArgs &ca, hipStream_t s)
{
    const int cus = device_cus();
    if (cus <= 0) return ECF8_E_HIP;
    using K = Chunk<FMT, N, LMAX>;
    const TilePlan p = plan_tiles<K::AREA>(a.n_chunks, ca.h.stream_bits, (uint32_t)cus);
    hipLaunchKernelGGL((w_encode_kernel<FMT, N, LMAX>), dim3(p.grid), dim3(p.waves * 64), 0, s, a, ca, p.per_wave);
    return hipGetLastError() == hipSuccess ? ECF8_OK : ECF8_E_HIP;
}

template <int FMT>
int encode_on_gpu(const void *d_elems, uint64_t rows, uint64_t cols, uint32_t N, uint32_t group, uint32_t lmax, void *d_blob,
                  uint64_t blob_capacity, ecfw_header *hdr_out, hipStream_t s)
{
    constexpr int A = EFmt<FMT>::A;
    const uint64_t n = rows * cols;
    const uint64_t blob = (uint64_t)(uintptr_t)d_blob, x = (uint64_t)(uintptr_t)d_elems;
    // the sections in front of chunk_bit have fixed places: header 256, code_len 256, freq 8A rounded up
    const uint64_t off_freq = 512, fixed = off_freq + (8ull * A + 255) / 256 * 256;
    const uint64_t n_chunks = (n + 64ull * N - 1) / (64ull * N);
    if (blob_capacity < fixed + 8 * (n_chunks + 1)) return ECF8_E_CAPACITY;         // no blob of this tensor is that small

    // pass 1: histogram, counted into the blob's freq section
    const int cus = device_cus();
    if (cus <= 0) return ECF8_E_HIP;
    if (capturing(s)) return ECF8_E_HIP;
    Mail mail;
    hipLaunchKernelGGL(fill_zero_kernel, dim3(1), dim3(256), 0, s, blob, fixed);
    const uint64_t hist_blocks = (n * EFmt<FMT>::ELEM / 4096 + 15) / 16, hist_most = (uint64_t)cus;
    hipLaunchKernelGGL(w_histogram_kernel<FMT>, dim3((uint32_t)(hist_blocks < 1 ? 1 : hist_blocks < hist_most ? hist_blocks : hist_most)), dim3(1024), 0, s,
                       x, n, blob, blob + off_freq, blob + fixed, n_chunks, mail.device());
    if (hipGetLastError() != hipSuccess) return ECF8_E_HIP;
    uint64_t freq[256] = {};
    if (!mail.read(freq, A, blob + off_freq, s)) return ECF8_E_HIP;

    ecfw_internal::WPlan plan;
    int rc = ecfw_internal::plan_encode(freq, FMT, rows, cols, N, group, lmax, &plan);
    if (rc) return rc;
    const ecfw_header &h = plan.hdr;
    if (h.total_size > blob_capacity) return ECF8_E_CAPACITY;
    if (h.off_freq != off_freq || h.off_chunk_bit != fixed || h.n_chunks != n_chunks) return ECF8_E_FORMAT;

    // pass 2: the container
    WEncArgs a{};
    a.x = x;
    a.blob = blob;
    a.n = n;
    a.n_chunks = h.n_chunks;
    a.off_len = h.off_code_len;
    a.off_cb = h.off_chunk_bit;
    a.off_lb = h.off_lane_bits;
    a.off_st = h.off_stream;
    a.off_pl = h.off_plane;
    a.off_sg = h.off_sign;
    a.group = group;
    WCodeArgs ca;
    ca.h = h;
    for (int i = 0; i < 256; i++) {
        ca.len[i] = plan.len[i];
        ca.code[i] = (uint16_t)plan.code[i];
    }
    if (h.max_code_len <= ECFW_TABLE_BITS)
        rc = N == 64 ? launch_encode<FMT, 64, (int)ECFW_TABLE_BITS>(a, ca, s) : launch_encode<FMT, 128, (int)ECFW_TABLE_BITS>(a, ca, s);
    else
        rc = N == 64 ? launch_encode<FMT, 64, (int)ECFW_MAX_CODE_LEN>(a, ca, s) : launch_encode<FMT, 128, (int)ECFW_MAX_CODE_LEN>(a, ca, s);
    if (rc) return rc;
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
