// GPU-side ECF8 encoder for gfx950 (paper Section 3.1: histogram, code, stream, metadata and
// nibble plane, produced on the device so that FP8 checkpoints compress at load time without a
// trip through host memory).  Writes exactly the container the CPU encoder writes, byte for
// byte: the same code under every cap, ties included, and the layout from the same routines.
//
//   histograms of ranges of chunks -> code, places of the ranges in the stream, header (one workgroup; the host waits for the header) -> everything else:
//   planes, lane_bits, the chunks' bits packed in LDS and copied to the stream, pair table and padding (encode_range).
// The input is read twice (histogram, the rest).  No scratch memory on the device: the ranges' histograms lie where the stream will.
#include "ecf8_device.h"
#include "ecf8_enc_device.h"
#include "ecf8_plan.h"

#include <type_traits>

namespace {

struct EncArgs {
    uint64_t x, blob;                     // device addresses
    uint64_t n, cols, n_chunks;
    uint32_t kc_per_row;                  // row-tiled: chunks per block of rows
    uint64_t off_cb, off_lb, off_st, off_pl;
    uint32_t group, tiled;
};

template <int N>
__device__ __forceinline__ ChunkPlace place_of(const EncArgs &a, uint64_t c, uint32_t lane)
{
    constexpr uint64_t E = 64ull * N;
    if (a.tiled) {
        const uint32_t rb = (uint32_t)c / a.kc_per_row;     // at most 2^40 elements
        return {(uint64_t)rb * 16 * a.cols + ((uint32_t)c - rb * a.kc_per_row) * (4ull * N), 64, (uint64_t)(lane & 15) * a.cols + 16ull * (lane >> 4)};
    }
    const uint64_t grouped = (a.n / E) & ~((uint64_t)a.group - 1);
    const uint64_t w = c & (a.group - 1);
    if (c < grouped) return {(c - w) * E + w * 1024, (uint64_t)a.group * 1024, lane * 16ull};
    return {c * E, 1024, lane * 16ull};
}

// elements of the piece at e that exist
__device__ __forceinline__ uint32_t piece_len(uint64_t e, uint64_t n) { return e + 16 <= n ? 16u : e < n ? (uint32_t)(n - e) : 0u; }

// Exponent-field histogram of each range into a record of 16 u32.  Counted with bit planes: 32 elements are turned into four 32-bit
// words, one per exponent bit, and each of the 16 exponents is then one AND and one population count that also adds:
// two vector operations per element and no LDS.  A range's last chunks come first: the pass behind it begins with the first ones, and finds them in the
// second-level cache.  58.7 M weights in a kernel trace: 15.2 us when the counts were added to one record and mailed to the host by the last workgroup, each counter
// summed over the wave by a scan of its own; 10.6 now (5.5 TB/s).  What is left is the read.
template <int N>
__global__ __launch_bounds__(1024) void histogram_kernel(EncArgs a, Ranges rg, uint64_t records)
{
    __shared__ uint32_t s_cnt[16];
    const GLOBAL uint8_t *x = (const GLOBAL uint8_t *)a.x;
    const int tid = threadIdx.x, lane = tid & 63;
    if (tid < 16) s_cnt[tid] = 0;
    __syncthreads();
    uint32_t cnt[16];
#pragma unroll
    for (int s = 0; s < 16; s++) cnt[s] = 0;
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
    // a wave takes four pieces of 1 KiB per step, two with 32 symbols per lane, where they are all of a chunk
    constexpr uint32_t PIECES = N / 16, PER = PIECES < 4 ? PIECES : 4;
    const uint64_t first = rg.begin(blockIdx.x);
    const uint32_t size = rg.size(blockIdx.x), whole = size - ((first + size) * (64ull * N) > a.n ? 1u : 0u);
    for (uint32_t i = uniform32(tid >> 6); i < whole * (PIECES / PER); i += 16) {
        const uint64_t c = first + whole - 1 - i / (PIECES / PER);      // the first chunks last: the next reader begins with them
        const uint32_t q = i % (PIECES / PER) * PER;
        u32x4 v[PER];
        if (a.tiled) {
            // in the order of the rows: 256 / N of them per piece, a lane's place in them instead of the one it codes
            const ChunkPlace p = place_of<N>(a, c, 0);
            const uint32_t o = 16 * lane;
#pragma unroll
            for (uint32_t j = 0; j < PER; j++) v[j] = *(const GLOBAL u32x4 *)(x + p.base + (uint64_t)((q + j) * (256 / N) + o / (4 * N)) * a.cols + o % (4 * N));
        } else {
            const ChunkPlace p = place_of<N>(a, c, (uint32_t)lane);
#pragma unroll
            for (uint32_t j = 0; j < PER; j++) v[j] = *(const GLOBAL u32x4 *)(x + p.base + p.lane_off + (q + j) * p.stride);
        }
#pragma unroll
        for (uint32_t j = 0; j < PER; j += 2) count(v[j], v[j + 1]);
    }
    if (whole != size)
        for (uint64_t i = (first + whole) * (64ull * N) + tid; i < a.n; i += 1024) atomicAdd(&s_cnt[(x[i] >> 3) & 15u], 1u);
    add_counts<16>(cnt, s_cnt, lane);
    __syncthreads();
    if (tid < 16) ((GLOBAL uint32_t *)records)[(uint64_t)blockIdx.x * 16 + tid] = s_cnt[tid];
}

// What plan_kernel has to know of this codec.
struct E4M3Codec {
    static constexpr int A = 16;
    typedef ecf8_header Header;
    static __device__ __forceinline__ uint64_t sign_bytes(const Header &) { return 0; }
    static __device__ __forceinline__ void finish(Header &h, GLOBAL uint8_t *, uint64_t, const uint64_t *freq, const uint32_t *len, uint32_t, uint32_t, bool, int lane)
    {
        if (lane >= 16) return;
        h.code_len[lane] = (uint8_t)len[lane];
        h.freq[lane] = freq[lane];
    }
};

// Everything of the container that is neither chunk data nor stream, but for the header, by all workgroups: pair table, zeros in the gaps between sections and behind the last dword of the stream.
__device__ __forceinline__ void write_fixed(const EncArgs &a, const __attribute__((address_space(4))) ecf8_header &h, uint64_t len_packed, const uint32_t (*one)[17])
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
    uint32_t rcode[16];
#pragma unroll
    for (int s = 0; s < 16; s++) rcode[s] = uniform32(one[0][s]) & 0xffffu;
    // the first codeword at the low bits of v: symbol | length << 4, 0 if it is longer than the table's index
    auto first = [&](uint32_t v) {
        uint32_t r = 0;
#pragma unroll
        for (int s = 0; s < 16; s++) {
            const uint32_t l = (uint32_t)(len_packed >> (4 * s)) & 15u;
            if (l != 0 && l <= (uint32_t)TB && (v & ((1u << l) - 1u)) == rcode[s]) r = (uint32_t)s | (l << 4);
        }
        return r;
    };
    for (uint32_t i = blockIdx.x * threads + tid; i < (uint32_t)TBL_ENTRIES; i += gridDim.x * threads) {
        const uint32_t t1 = first(i), l1 = t1 >> 4, t2 = l1 ? first(i >> l1) : 0u;
        ((GLOBAL uint16_t *)(blob + 256))[i] = ecf8_pair_entry(t1 & 15u, l1, t2 & 15u, t2 >> 4);
    }
}

// A chunk on its way through encode_range.
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
    static constexpr int LANE_BITS = N * (CAP7 ? 7 : 15);                           // at most
    static constexpr int MOST = (160 * 1024 - 4096 - 512 * (int)sizeof(Entry)) / (4 * WMAX) / 4 * 4;
    static constexpr int AREA = 2 * LANE_BITS + 4 < MOST ? 2 * LANE_BITS + 4 : MOST;  // a chunk whatever it is, if there is room
    static_assert(LANE_BITS + 4 <= AREA && AREA % 4 == 0, "half a chunk");

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
    __device__ __forceinline__ void slow_pack(uint32_t *image, uint32_t at, uint64_t c)
    {
        const ChunkPlace p = place_of<N>(a, c, lane);
        LanePacker<false> out(image, at);
        const uint64_t e0 = p.base + p.lane_off;
        const uint32_t stride = (uint32_t)p.stride;
        auto at_piece = [&](int i) { return e0 + (uint32_t)(i >= N / 32 ? N / 16 - 1 - (i - N / 32) : i) * stride; };
        u32x4 next = slow_fetch(at_piece(0));
#pragma unroll 1
        for (int i = 0; i < N / 16; i++) {
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
    }
    // the last 32 bits of a whole chunk: those of lane 63's last codewords, of which each lane looks up one
    __device__ __forceinline__ uint32_t tail(uint64_t c) const
    {
        const ChunkPlace p = place_of<N>(a, c, 63);
        const uint32_t t = (uint32_t)lane & 31;                 // counted from the end: the backward run from its first symbol on, then the forward run from its last
        const uint32_t s = t < N / 2 ? N / 2 + t : N - 1 - t, back = t < N / 2 ? 1 : 0;
        const uint32_t e = one[back][(((const GLOBAL uint8_t *)a.x)[p.base + p.lane_off + s / 16 * p.stride + s % 16] >> 3) & 15u];
        return last_bits(e & 0xffffu, e >> 16, lane);
    }
    // the four symbols of dword w, in order (BWD = false) or in reverse
    template <bool BWD>
    __device__ __forceinline__ void put4(LanePacker<false> &out, uint32_t w) const
    {
        if constexpr (CAP7) {                                                       // as count has left them
            out.put(w, 31u ^ (uint32_t)__builtin_clz(w));
        } else {
            const Entry *tab = BWD ? bwd : fwd;
            const uint32_t x = (w >> 3) & 0x0f0f0f0fu, u = x | (x >> 4);            // bytes 0 and 2: two exponents each
            Entry ea = tab[u & 0xffu], eb = tab[(u >> 16) & 0xffu];
            if (BWD) { const Entry y = ea; ea = eb; eb = y; }
            out.put((uint32_t)ea, (uint32_t)(ea >> LEN_AT));
            out.put((uint32_t)eb, (uint32_t)(eb >> LEN_AT));
        }
    }
    __device__ __forceinline__ void pack(uint32_t *image, uint32_t at, uint64_t, uint64_t next, bool refill)
    {
        LanePacker<false> out(image, at);
        const ChunkPlace p = place_of<N>(a, next, lane);
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

// The container behind the code.  58.7 M weights (14336 x 4096): 23.0 us in a kernel trace for the 111 MB read and written; 29.8 when the workgroups had to find their
// place in the stream from one another.  Vector operations take two thirds of it, 8.7 per weight; the rest is the first fetch and the last copy, when
// the compute unit has nothing else to do.  The whole call 53.0 -> 41.4 (one input over and
// over, from the memory-side cache, 52.7 -> 39.0), 256 x 512 26.5 -> 19.2, 14336 x 14336 147 -> 114.
template <int N, bool CAP7>
__global__ __launch_bounds__(WMAX * 64) void encode_kernel(EncArgs a, Ranges rg)
{
    using K = Chunk<N, CAP7>;
    typedef typename K::Entry Entry;
    __shared__ struct {                                     // the tables where a look-up needs no address of theirs
        Entry fwd[256], bwd[256];
        uint32_t one[2][17];
        RangeShared range;
        __attribute__((aligned(16))) uint32_t images[WMAX][K::AREA];
    } s;
    const uint32_t tid = threadIdx.x;
    const int wave = (int)uniform32(tid >> 6), lane = (int)(tid & 63);
    uint64_t len_packed = 0;                                // code length of symbol s in bits 4s..4s+3
    K k{a, s.fwd, s.bwd, s.one, lane, {}, {}};
    const uint64_t c0 = rg.begin(blockIdx.x) + wave;
    if ((uint32_t)wave < rg.size(blockIdx.x) && k.whole(c0)) k.fetch(c0);
    const auto &h = planned<ecf8_header>(a.blob);
    if (h.magic == 0) return;                               // no blob
#pragma unroll
    for (int i = 0; i < 4; i++) {
        k.len_bytes[i] = ((const __attribute__((address_space(4))) uint32_t *)h.code_len)[i];
        const uint32_t l = k.len_bytes[i] | k.len_bytes[i] >> 4;
        len_packed |= (uint64_t)((l & 0xffu) | (l >> 8 & 0xff00u)) << (16 * i);
    }
    a.off_pl = h.off_plane;
    range_begin(s.range);
    if (tid < 256) {
        const uint32_t lo = tid & 15, hi = tid >> 4;        // an entry's first and second element
        // canonical codewords: behind those of shorter and of equally long, smaller exponents
        uint32_t own = (uint32_t)(len_packed >> (4 * lo)) & 15u, code = 0;
#pragma unroll
        for (uint32_t e = 0; e < 16; e++) {
            const uint32_t l = (uint32_t)(len_packed >> (4 * e)) & 15u;
            if (l && (l < own || (l == own && e < lo))) code += 1u << (15 - l);
        }
        code = own ? code >> (15 - own) : 0u;
        const uint32_t rcode = own ? __brev(code) >> (32 - own) : 0u, l0 = own, l1 = (uint32_t)(len_packed >> (4 * hi)) & 15u;
        const uint32_t code_hi = (uint32_t)__shfl((int)code, (int)hi, 64), rcode_hi = (uint32_t)__shfl((int)rcode, (int)hi, 64);
        s.fwd[tid] = (Entry)(rcode | (rcode_hi << l0)) | ((Entry)(l0 + l1) << K::LEN_AT);
        s.bwd[tid] = (Entry)(code_hi | (code << l1)) | ((Entry)(l0 + l1) << K::LEN_AT);
        if (tid < 17) {
            s.one[0][tid] = tid < 16 ? rcode | (l0 << 16) : 0u;
            s.one[1][tid] = tid < 16 ? code | (l0 << 16) : 0u;
        }
    }
    __syncthreads();
    write_fixed(a, h, len_packed, s.one);
    encode_range(k, s.range, s.images[wave], rg, (GLOBAL uint8_t *)a.blob, a.off_cb, a.off_lb, a.off_st, h.stream_bytes / 4, lane, wave);
}

template <int N, bool CAP7>
void launch_encode(const EncArgs &a, const Ranges &rg, hipStream_t s)
{
    hipLaunchKernelGGL((encode_kernel<N, CAP7>), dim3(rg.count), dim3(range_waves(rg) * 64), 0, s, a, rg);
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
    ecf8_header h;
    rc = ecf8_internal::plan_frame(rows, cols, opts, &h);
    if (rc) return rc;
    if (blob_capacity < h.off_stream + h.plane_bytes) return ECF8_E_CAPACITY;       // no blob of this tensor is that small, and the ranges' histograms fit
    hipStream_t s = (hipStream_t)stream;
    const int cus = device_cus();
    if (cus <= 0) return ECF8_E_HIP;

    EncArgs a{};
    a.x = (uint64_t)(uintptr_t)d_fp8;
    a.blob = (uint64_t)(uintptr_t)d_blob;
    a.n = h.n_elem;
    a.cols = cols;
    a.n_chunks = h.n_chunks;
    a.kc_per_row = tile_rows ? (uint32_t)(cols / (4ull * N)) : 1u;
    a.off_cb = h.off_chunk_bit;
    a.off_lb = h.off_lane_bits;
    a.off_st = h.off_stream;
    a.group = group;
    a.tiled = tile_rows ? 1 : 0;
    const Ranges rg = make_ranges(h.n_chunks, (uint32_t)cus);
    const uint64_t records = a.blob + h.off_stream;
    static_assert(16 * 4 <= 32 * 32, "a record is smaller than a chunk's plane");

    if (capturing(s)) return ECF8_E_HIP;
    Mail mail;
    if (N == 32) hipLaunchKernelGGL(histogram_kernel<32>, dim3(rg.count), dim3(1024), 0, s, a, rg, records);
    else if (N == 64) hipLaunchKernelGGL(histogram_kernel<64>, dim3(rg.count), dim3(1024), 0, s, a, rg, records);
    else hipLaunchKernelGGL(histogram_kernel<128>, dim3(rg.count), dim3(1024), 0, s, a, rg, records);
    if (!launched()) return ECF8_E_HIP;
    hipLaunchKernelGGL(plan_kernel<E4M3Codec>, dim3(1), dim3(1024), 0, s, h, rg, a.blob, blob_capacity, records, lmax, mail.device());
    if (!launched()) return ECF8_E_HIP;
    // By the cap: the code is not known yet.  Under a cap of 8 to 15 a code that needs no more than 7 bits pays for that, 14336 x 4096 with 3 bits 37.6 us under cap 7 and 42.5
    // under 15, and is faster all the same than when the host waited for the histogram and chose by the longest codeword: 50.7; 4096 x 4096 22.5, 24.8, 35.0;
    // 256 x 512 18.6, 18.8, 24.4.
    if (lmax <= 7) {
        if (N == 32) launch_encode<32, true>(a, rg, s);
        else if (N == 64) launch_encode<64, true>(a, rg, s);
        else launch_encode<128, true>(a, rg, s);
    } else {
        if (N == 32) launch_encode<32, false>(a, rg, s);
        else if (N == 64) launch_encode<64, false>(a, rg, s);
        else launch_encode<128, false>(a, rg, s);
    }
    if (!launched()) return ECF8_E_HIP;
    if (!mail.read(&h, a.blob, s)) return ECF8_E_HIP;
    if (h.magic == 0) return (int)h.version;
    *hdr_out = h;
    return ECF8_OK;
}

} // extern "C"
