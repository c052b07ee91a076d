// GPU-side ECF8 encoder for gfx950 (paper Section 3.1: histogram, code, stream, metadata and
// nibble plane, produced on the device so that FP8 checkpoints compress at load time without a
// trip through host memory).  Writes exactly the container the CPU encoder writes, byte for
// byte: the code and the layout come from the same host routine, fed with the device histogram.
//
//   fill 0 (256 bytes) -> histogram (and zeros in chunk_bit[]), written to the host by its last workgroup -> [host: code + layout]
//   -> everything else in one pass over the weights (encode_tiles): planes, lane_bits, the chunks' bits packed in LDS, their place
//   in the stream found out between the workgroups, the stream; the workgroups also write pair table and padding, the one that
//   finds no more work last the header.
// The input is read twice (histogram, the rest).  No scratch memory on the device: the histogram is counted into the header's freq[] field, tiles are
// drawn from its first dword, and what the workgroups tell one another goes through chunk_bit[], all of them part of the output.
#include "ecf8_device.h"
#include "ecf8_enc_device.h"
#include "ecf8_plan.h"

#include <type_traits>

namespace {

struct EncArgs {
    uint64_t x, blob;                     // device addresses
    uint64_t n, cols, n_chunks;
    uint64_t off_cb, off_lb, off_st, off_pl;
    uint32_t group, tiled;
    uint64_t len_packed;                  // code length of symbol s in bits 4s..4s+3
    uint32_t code[16], rcode[16];
};

template <int N>
__device__ __forceinline__ ChunkPlace place_of(const EncArgs &a, uint64_t c, uint32_t lane)
{
    constexpr uint64_t E = 64ull * N;
    if (a.tiled) {
        const uint64_t kc_per_row = a.cols / (4ull * N);
        const uint64_t rb = c / kc_per_row;
        return {rb * 16 * a.cols + (c - rb * kc_per_row) * (4ull * N), 64, (uint64_t)(lane & 15) * a.cols + 16ull * (lane >> 4)};
    }
    const uint64_t grouped = (a.n / E) & ~((uint64_t)a.group - 1);
    const uint64_t w = c & (a.group - 1);
    if (c < grouped) return {(c - w) * E + w * 1024, (uint64_t)a.group * 1024, lane * 16ull};
    return {c * E, 1024, lane * 16ull};
}

// elements of the piece at e that exist
__device__ __forceinline__ uint32_t piece_len(uint64_t e, uint64_t n) { return e + 16 <= n ? 16u : e < n ? (uint32_t)(n - e) : 0u; }

// Exponent-field histogram into 16 u64 counters.  Counted with bit planes: 32 elements are turned into four 32-bit
// words, one per exponent bit, and each of the 16 exponents is then one AND and one population count that also adds:
// two vector operations per element and no LDS.  58.7 M weights: 14.5 us (4 TB/s; counters private to a thread in LDS,
// one read-modify-write per element, 37 us).  What is left is the read and its latency.
__global__ __launch_bounds__(1024) void histogram_kernel(uint64_t x_, uint64_t n, uint64_t blob, uint64_t counters_, uint64_t chunk_bit, uint64_t n_chunks, uint64_t mail)
{
    __shared__ uint32_t s_cnt[16];
    const GLOBAL uint8_t *x = (const GLOBAL uint8_t *)x_;
    GLOBAL unsigned long long *counters = (GLOBAL unsigned long long *)counters_;
    const int tid = threadIdx.x, lane = tid & 63;
    if (tid < 16) s_cnt[tid] = 0;
    zero_chunk_bits(chunk_bit, n_chunks, (uint32_t)tid, 1024);
    __syncthreads();
    uint32_t cnt[16];
#pragma unroll
    for (int s = 0; s < 16; s++) cnt[s] = 0;
    // a wave takes 4 KiB per step: four loads of 1 KiB, of which a lane keeps the 16 bytes at 16 * lane
    const uint64_t steps = n / 4096, stride = (uint64_t)gridDim.x * 16;
    const GLOBAL u32x4 *p = (const GLOBAL u32x4 *)x + lane;
    auto count = [&](const u32x4 &va, const u32x4 &vb) {
        const uint32_t w[8] = {va.x, va.y, va.z, va.w, vb.x, vb.y, vb.z, vb.w};
        uint32_t t[4];
#pragma unroll
        for (int i = 0; i < 4; i++) t[i] = bit_select(0x0f0f0f0fu, w[2 * i] >> 3, w[2 * i + 1] << 1);      // eight exponents in nibbles
        const uint32_t a0 = bit_select(0x55555555u, t[0], t[1] << 1), a1 = bit_select(0x55555555u, t[0] >> 1, t[1]);
        const uint32_t b0 = bit_select(0x55555555u, t[2], t[3] << 1), b1 = bit_select(0x55555555u, t[2] >> 1, t[3]);
        const uint32_t p0 = bit_select(0x33333333u, a0, b0 << 2), p2 = bit_select(0x33333333u, a0 >> 2, b0);
        const uint32_t p1 = bit_select(0x33333333u, a1, b1 << 2), p3 = bit_select(0x33333333u, a1 >> 2, b1);
#pragma unroll
        for (int s = 0; s < 16; s++) {
            const uint32_t hi = (s & 8 ? p3 : ~p3) & (s & 4 ? p2 : ~p2);
            const uint32_t lo = (s & 2 ? p1 : ~p1) & (s & 1 ? p0 : ~p0);
            cnt[s] += (uint32_t)__builtin_popcount(hi & lo);
        }
    };
    for (uint64_t i = (uint64_t)blockIdx.x * 16 + (tid >> 6); i < steps; i += stride) {
        const u32x4 va = p[i * 256], vb = p[i * 256 + 64], vc = p[i * 256 + 128], vd = p[i * 256 + 192];
        count(va, vb);
        count(vc, vd);
    }
    if (blockIdx.x == 0)
        for (uint64_t i = steps * 4096 + tid; i < n; i += 1024) atomicAdd(&s_cnt[(x[i] >> 3) & 15u], 1u);
#pragma unroll
    for (int s = 0; s < 16; s++) {
        const uint32_t sum = wave_incl_scan(cnt[s]);
        if (lane == 63 && sum) atomicAdd(&s_cnt[s], sum);
    }
    __syncthreads();
    if (tid < 16 && s_cnt[tid]) atomicAdd((unsigned long long *)(counters + tid), (unsigned long long)s_cnt[tid]);
    mail_histogram<16>(blob, counters_, mail);
}

// Everything of the container that is neither chunk data nor stream, but for the header, by all workgroups: pair table, zeros in the gaps between sections and behind the last dword of the stream.
__device__ __forceinline__ void write_fixed(const EncArgs &a, const ecf8_header &h)
{
    const uint32_t tid = threadIdx.x, threads = blockDim.x;
    GLOBAL uint8_t *blob = (GLOBAL uint8_t *)a.blob;
    if (blockIdx.x == 0) {
        auto zero = [&](uint64_t from, uint64_t to) {       // multiples of four
            for (uint64_t i = from + 4 * tid; i < to; i += 4 * threads) *(GLOBAL uint32_t *)(blob + i) = 0;
        };
        zero(a.off_cb + 8 * (a.n_chunks + 1), a.off_lb);
        zero(a.off_lb + 128 * a.n_chunks, a.off_st);
        zero(a.off_st + ((h.stream_bits + 31) >> 5) * 4, a.off_pl);
        zero(a.off_pl + h.plane_bytes, h.total_size);
    }
    if (!h.table_bits) return;
    // the first codeword at the low bits of v: symbol | length << 4, 0 if it is longer than the table's index
    auto first = [&](uint32_t v) {
        uint32_t r = 0;
#pragma unroll
        for (int s = 0; s < 16; s++) {
            const uint32_t l = (uint32_t)(a.len_packed >> (4 * s)) & 15u;
            if (l != 0 && l <= (uint32_t)TB && (v & ((1u << l) - 1u)) == a.rcode[s]) r = (uint32_t)s | (l << 4);
        }
        return r;
    };
    for (uint32_t i = blockIdx.x * threads + tid; i < (uint32_t)TBL_ENTRIES; i += gridDim.x * threads) {
        const uint32_t t1 = first(i), l1 = t1 >> 4, t2 = l1 ? first(i >> l1) : 0u;
        ((GLOBAL uint16_t *)(blob + 256))[i] = ecf8_pair_entry(t1 & 15u, l1, t2 & 15u, t2 >> 4);
    }
}

// A chunk on its way through encode_tiles.
//  * Plane: 8 elements -> 4 bytes, byte j = low nibble element j, high nibble element j + 4; zeros where the last chunk reaches past
//    the tensor.
//  * Bits: a lane's are one string, the forward run's codewords in order and then the backward run's in reverse (each with its first
//    bit highest), packed one behind the other in a register; every finished dword is ORed into the image, where neighbouring lanes
//    share a dword at their borders.  Symbols are looked up in pairs: 256 entries of the two codewords joined and their
//    length, for either direction.
//  * CAP7 (no codeword over 7 bits): count joins two pairs and leaves them in their dword, a one above them, and pack has nothing to
//    look up; its OR instructions keep look-ups from moving past them.  Else count looks lengths up four at a time, by two byte
//    permutes of the 16 lengths held in four registers, selected by the exponents' top bits and summed by one v_sad_u8.
template <int N, bool CAP7>
struct Chunk {
    typedef typename std::conditional<CAP7, uint32_t, uint64_t>::type Entry;        // codewords; length from bit 28 or 32
    static constexpr int LEN_AT = CAP7 ? 28 : 32;
    static constexpr uint32_t BITS = (1u << 28) - 1;                                // CAP7: of an entry or two joined ones
    static constexpr int AREA = ((160 * 1024 - 1024 - 512 * (int)sizeof(Entry)) / (4 * WMAX) - 4) / 4 * 4;
    static constexpr int LANE_BITS = N * (CAP7 ? 7 : 15);                           // at most
    static constexpr int TAIL_FROM = N / 16 - 2;                                    // a lane's last 32 codewords
    static_assert(32 * 15 < 32 * LATE_DWORDS && LANE_BITS * LATE_LANES <= 32 * (AREA - 4), "room for late chunks");

    const EncArgs &a;
    const Entry *fwd, *bwd;                 // pairs of symbols
    const uint32_t (*one)[17];              // single symbols, code | length << 16; 16 = no symbol
    int lane;
    uint32_t len_bytes[4];                  // code lengths of symbols 4i .. 4i + 3
    u32x4 v[N / 16];

    __device__ __forceinline__ bool whole(uint64_t c) const { return (c + 1) * (64ull * N) <= a.n; }
    __device__ __forceinline__ void fetch(uint64_t c)
    {
        const ChunkPlace p = place_of<N>(a, c, lane);
        const GLOBAL uint8_t *x = (const GLOBAL uint8_t *)a.x + p.base + p.lane_off;
#pragma unroll
        for (int q = 0; q < N / 16; q++) v[q] = *(const GLOBAL u32x4 *)(x + q * p.stride);
    }
    // the nibbles of a piece
    static __device__ __forceinline__ u32x2 nibbles(const u32x4 &w)
    {
        // low nibbles; the rest is masked off
        const uint32_t a0 = bit_select(0x07070707u, w.x, w.x >> 4), a1 = bit_select(0x07070707u, w.y, w.y >> 4);
        const uint32_t a2 = bit_select(0x07070707u, w.z, w.z >> 4), a3 = bit_select(0x07070707u, w.w, w.w >> 4);
        return u32x2{bit_select(0x0f0f0f0fu, a0, a1 << 4), bit_select(0x0f0f0f0fu, a2, a3 << 4)};
    }
    __device__ __forceinline__ uint32_t count(uint64_t c)
    {
        const ChunkPlace p = place_of<N>(a, c, lane);
        GLOBAL uint8_t *plane = (GLOBAL uint8_t *)a.blob + a.off_pl + (p.base + p.lane_off) / 2;
        uint32_t lb = 0;
#pragma unroll
        for (int i = 0; i < N / 16; i++) {
            const int q = i < N / 32 ? i : N / 16 - 1 - (i - N / 32);               // in the order in which pack asks for them
            const u32x2 plane_piece = nibbles(v[q]);
            uint32_t w[4] = {v[q].x, v[q].y, v[q].z, v[q].w};
#pragma unroll
            for (int k = 0; k < 4; k++) {
                if constexpr (CAP7) {
                    uint32_t at0, at1;
                    pair_offsets(w[k], at0, at1);
                    const bool back = i >= N / 32;
                    const uint32_t e0 = entry(back ? bwd : fwd, back ? at1 : at0), e1 = entry(back ? bwd : fwd, back ? at0 : at1);
                    const uint32_t l0 = e0 >> LEN_AT, nb = l0 + (e1 >> LEN_AT);
                    lb += nb;
                    w[k] = (((e1 << l0) | e0) & BITS) | (1u << nb);                 // e1's length lands above the codewords
                } else {
                    const uint32_t low = (w[k] >> 3) & 0x07070707u;
                    const uint32_t top = ((w[k] >> 2) & 0x10101010u) - ((w[k] >> 6) & 0x01010101u);       // 0x0f in the bytes with exponents 8 .. 15
                    lb = __builtin_amdgcn_sad_u8(bit_select(top, __builtin_amdgcn_perm(len_bytes[3], len_bytes[2], low), __builtin_amdgcn_perm(len_bytes[1], len_bytes[0], low)), 0u, lb);
                }
            }
            if constexpr (CAP7) v[q] = u32x4{w[0], w[1], w[2], w[3]};
            *(GLOBAL u32x2 *)(plane + q * (p.stride / 2)) = plane_piece;
        }
        return lb;
    }
    // where the entries of a dword's two pairs of symbols are: bytes into a table of dwords
    static __device__ __forceinline__ void pair_offsets(uint32_t w, uint32_t &at0, uint32_t &at1)
    {
        const uint32_t x = (w >> 1) & 0x3c3c3c3cu, u = x | (x >> 4);
        at0 = u & 0x3fcu;
        at1 = (u >> 16) & 0x3fcu;
    }
    static __device__ __forceinline__ uint32_t entry(const Entry *tab, uint32_t at) { return *(const uint32_t *)((const uint8_t *)tab + at); }
    // any chunk, piece by piece: its symbols one by one, those past the tensor's end have no bits
    __device__ __forceinline__ void piece(const u32x4 &v4, uint64_t e, uint32_t back, uint32_t (&s)[16]) const
    {
        const uint32_t w[4] = {v4.x, v4.y, v4.z, v4.w}, have = piece_len(e, a.n);
#pragma unroll
        for (uint32_t j = 0; j < 16; j++) s[j] = one[back][j < have ? (w[j >> 2] >> (8 * (j & 3) + 3)) & 15u : 16u];
    }
    __device__ __forceinline__ u32x4 slow_fetch(uint64_t e) const { return load_cut((const GLOBAL uint8_t *)a.x, e, a.n); }
    __device__ __forceinline__ uint32_t slow_count(uint64_t c)
    {
        const ChunkPlace p = place_of<N>(a, c, lane);
        uint32_t lb = 0;
#pragma unroll 1
        for (int q = 0; q < N / 16; q++) {
            const uint64_t e = p.base + p.lane_off + q * p.stride;
            uint32_t s[16];
            const u32x4 w = slow_fetch(e);
            piece(w, e, 0, s);
#pragma unroll
            for (int j = 0; j < 16; j++) lb += s[j] >> 16;
            *(GLOBAL u32x2 *)((GLOBAL uint8_t *)a.blob + a.off_pl + e / 2) = nibbles(w);
        }
        return lb;
    }
    // from the lane's i0-th piece on; the image's bit behind the last one
    __device__ __forceinline__ uint32_t slow_pack(uint32_t *image, uint32_t at, uint64_t c, int i0)
    {
        const ChunkPlace p = place_of<N>(a, c, lane);
        LanePacker out(image, at);
        const uint64_t e0 = p.base + p.lane_off;
        const uint32_t stride = (uint32_t)p.stride;
        auto at_piece = [&](int i) { return e0 + (uint32_t)(i >= N / 32 ? N / 16 - 1 - (i - N / 32) : i) * stride; };
        u32x4 next = slow_fetch(at_piece(i0));
#pragma unroll 1
        for (int i = i0; i < N / 16; i++) {
            const bool back = i >= N / 32;
            const u32x4 w = next;
            if (i + 1 < N / 16) next = slow_fetch(at_piece(i + 1));
            uint32_t s[16];
            piece(w, at_piece(i), back ? 1 : 0, s);
#pragma unroll
            for (int j = 0; j < 16; j++) {
                const uint32_t x = back ? s[15 - j] : s[j];
                out.put(x & 0xffffu, x >> 16);
            }
        }
        out.finish();
        return out.end(image);
    }
    // the four symbols of dword w, in order (BWD = false) or in reverse
    template <bool BWD>
    __device__ __forceinline__ void put4(LanePacker &out, uint32_t w) const
    {
        if constexpr (CAP7) {                                                       // as count has left them
            const uint32_t nb = 31u - (uint32_t)__builtin_clz(w);
            out.put(w ^ (1u << nb), nb);
        } else {
            const Entry *tab = BWD ? bwd : fwd;
            const uint32_t x = (w >> 3) & 0x0f0f0f0fu, u = x | (x >> 4);            // bytes 0 and 2: two exponents each
            Entry ea = tab[u & 0xffu], eb = tab[(u >> 16) & 0xffu];
            if (BWD) { const Entry y = ea; ea = eb; eb = y; }
            out.put((uint32_t)ea, (uint32_t)(ea >> LEN_AT));
            out.put((uint32_t)eb, (uint32_t)(eb >> LEN_AT));
        }
    }
    __device__ __forceinline__ void pack(uint32_t *image, uint32_t at, uint64_t c, bool refill)
    {
        LanePacker out(image, at);
        const ChunkPlace p = place_of<N>(a, c + 1, lane);
        const GLOBAL uint8_t *x = (const GLOBAL uint8_t *)a.x + p.base + p.lane_off;
#pragma unroll
        for (int q = 0; q < N / 32; q++) {
            put4<false>(out, v[q].x); put4<false>(out, v[q].y); put4<false>(out, v[q].z); put4<false>(out, v[q].w);
            if (refill) v[q] = *(const GLOBAL u32x4 *)(x + q * p.stride);
        }
#pragma unroll
        for (int q = N / 16 - 1; q >= N / 32; q--) {
            put4<true>(out, v[q].w); put4<true>(out, v[q].z); put4<true>(out, v[q].y); put4<true>(out, v[q].x);
            if (refill) v[q] = *(const GLOBAL u32x4 *)(x + q * p.stride);
        }
        out.finish();
    }
};

// The container behind the code.  58.7 M weights (14336 x 4096): 30 us in a kernel trace (the last 100 of 300 calls) for the 111 MB read and written,
// some 17 of them bound by vector operations, the others the first loads, the exchange and the copy to the stream, when the compute unit waits.  With two
// pairs looked up again for every put it took 2 more; metadata and planes, prefix sum and packing as kernels of their own 10 to 12 more, and
// they read the weights twice.  The whole call 67.7 -> 56.4 us (53.0 since the histogram is mailed), 16384 x 16384 242 -> 190.
template <int N, bool CAP7>
__global__ __launch_bounds__(WMAX * 64) void encode_kernel(EncArgs a, ecf8_header h, uint32_t per_wave)
{
    using K = Chunk<N, CAP7>;
    typedef typename K::Entry Entry;
    __shared__ __attribute__((aligned(16))) uint32_t images[WMAX][K::AREA + 4];  // the last of the four in front is image[-1]
    __shared__ Entry s_fwd[256], s_bwd[256];
    __shared__ uint32_t s_one[2][17];
    __shared__ TileShared sh;
    const uint32_t tid = threadIdx.x;
    const int wave = (int)uniform32(tid >> 6);
    if (tid < 256) {
        const uint32_t lo = tid & 15, hi = tid >> 4;        // an entry's first and second element
        const uint32_t l0 = (uint32_t)(a.len_packed >> (4 * lo)) & 15u, l1 = (uint32_t)(a.len_packed >> (4 * hi)) & 15u;
        s_fwd[tid] = (Entry)(a.rcode[lo] | (a.rcode[hi] << l0)) | ((Entry)(l0 + l1) << K::LEN_AT);
        s_bwd[tid] = (Entry)(a.code[hi] | (a.code[lo] << l1)) | ((Entry)(l0 + l1) << K::LEN_AT);
        if (tid < 17) {
            const uint32_t l = tid < 16 ? l0 : 0u;
            s_one[0][tid] = tid < 16 ? a.rcode[lo] | (l << 16) : 0u;
            s_one[1][tid] = tid < 16 ? a.code[lo] | (l << 16) : 0u;
        }
    }
    write_fixed(a, h);
    K k{a, s_fwd, s_bwd, s_one, (int)(tid & 63), {}, {}};
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const uint32_t l = (uint32_t)(a.len_packed >> (16 * i));
        k.len_bytes[i] = (l & 15u) | ((l & 0xf0u) << 4) | ((l & 0xf00u) << 8) | ((l & 0xf000u) << 12);
    }
    encode_tiles(k, sh, images[wave] + 4, TileArgs{a.n_chunks, per_wave, (const uint32_t *)&h}, (GLOBAL uint8_t *)a.blob, a.off_cb, a.off_lb, a.off_st,
                 (int)(tid & 63), wave);
}

template <int N, bool CAP7>
int launch_encode(const EncArgs &a, const ecf8_header &h, hipStream_t s)
{
    const int cus = device_cus();
    if (cus <= 0) return ECF8_E_HIP;
    using K = Chunk<N, CAP7>;
    const TilePlan p = plan_tiles<K::AREA>(h.n_chunks, h.stream_bits, (uint32_t)cus);
    hipLaunchKernelGGL((encode_kernel<N, CAP7>), dim3(p.grid), dim3(p.waves * 64), 0, s, a, h, p.per_wave);
    return hipGetLastError() == hipSuccess ? ECF8_OK : ECF8_E_HIP;
}

} // namespace

extern "C" {

int ecf8_encode_bound(uint64_t rows, uint64_t cols, const ecf8_encode_opts *opts, uint64_t *bytes)
{
    if (!bytes) return ECF8_E_ARG;
    return ecf8_internal::encode_bound(rows, cols, opts, bytes);
}

int ecf8_encode_gpu(const void *d_fp8, uint64_t rows, uint64_t cols, const ecf8_encode_opts *opts, void *d_blob,
                    uint64_t blob_capacity, ecf8_header *hdr_out, void *stream)
{
    if (!d_fp8 || !d_blob || !hdr_out) return ECF8_E_ARG;
    uint32_t N, group, lmax, tile_rows, tmode;
    int rc = ecf8_internal::check_options(rows, cols, opts, &N, &group, &lmax, &tile_rows, &tmode);
    if (rc) return rc;
    if (((uintptr_t)d_fp8 & 15) || ((uintptr_t)d_blob & 255)) return ECF8_E_ALIGN;
    if (blob_capacity < 256) return ECF8_E_CAPACITY;
    const uint64_t n = rows * cols;
    hipStream_t s = (hipStream_t)stream;
    const uint64_t blob = (uint64_t)(uintptr_t)d_blob, x = (uint64_t)(uintptr_t)d_fp8;

    // pass 1: histogram, counted into the header's freq[] field
    const int cus = device_cus();
    if (cus <= 0) return ECF8_E_HIP;
    const uint64_t n_chunks = (n + 64ull * N - 1) / (64ull * N), off_cb = 256 + ((tmode == 1 || (tmode == 0 && n >= (1ull << 22))) ? TBL_ENTRIES * 2 : 0);
    if (blob_capacity < off_cb + 8 * (n_chunks + 1)) return ECF8_E_CAPACITY;        // no blob of this tensor is that small
    if (capturing(s)) return ECF8_E_HIP;
    Mail mail;
    hipLaunchKernelGGL(fill_zero_kernel, dim3(1), dim3(256), 0, s, blob, (uint64_t)256);
    // one workgroup per compute unit at the most: each ends with 16 atomic additions to one line
    const uint64_t hist_blocks = (n / 4096 + 15) / 16, hist_most = (uint64_t)cus;
    hipLaunchKernelGGL(histogram_kernel, dim3((uint32_t)(hist_blocks < 1 ? 1 : hist_blocks < hist_most ? hist_blocks : hist_most)), dim3(1024), 0, s, x, n,
                       blob, blob + 128, blob + off_cb, n_chunks, mail.device());
    if (hipGetLastError() != hipSuccess) return ECF8_E_HIP;
    uint64_t freq[16];
    if (!mail.read(freq, 16, blob + 128, s)) return ECF8_E_HIP;

    ecf8_internal::Plan plan;
    rc = ecf8_internal::plan_encode(freq, rows, cols, opts, &plan);
    if (rc) return rc;
    const ecf8_header &h = plan.hdr;
    if (h.total_size > blob_capacity) return ECF8_E_CAPACITY;
    if (h.off_chunk_bit != off_cb || h.n_chunks != n_chunks) return ECF8_E_FORMAT;

    EncArgs a{};
    a.x = x;
    a.blob = blob;
    a.n = n;
    a.cols = cols;
    a.n_chunks = h.n_chunks;
    a.off_cb = h.off_chunk_bit;
    a.off_lb = h.off_lane_bits;
    a.off_st = h.off_stream;
    a.off_pl = h.off_plane;
    a.group = group;
    a.tiled = tile_rows ? 1 : 0;
    for (int i = 0; i < 16; i++) {
        a.len_packed |= (uint64_t)h.code_len[i] << (4 * i);
        a.code[i] = plan.code[i];
        a.rcode[i] = plan.rcode[i];
    }
    // pass 2: the container
    uint32_t longest = 0;
    for (int i = 0; i < 16; i++) longest = h.code_len[i] > longest ? h.code_len[i] : longest;
    if (longest <= 7) rc = N == 32 ? launch_encode<32, true>(a, h, s) : N == 64 ? launch_encode<64, true>(a, h, s) : launch_encode<128, true>(a, h, s);
    else rc = N == 32 ? launch_encode<32, false>(a, h, s) : N == 64 ? launch_encode<64, false>(a, h, s) : launch_encode<128, false>(a, h, s);
    if (rc) return rc;
    *hdr_out = h;
    return ECF8_OK;
}

} // extern "C"
