// GPU-side ECF8 encoder for gfx950 (paper Section 3.1: histogram, code, stream, metadata and
// nibble plane, produced on the device so that FP8 checkpoints compress at load time without a
// trip through host memory).  Writes exactly the container the CPU encoder writes, byte for
// byte: the code and the layout come from the same host routine, fed with the device histogram.
//
//   fill 0 (256 bytes) -> histogram -> [host: 128 bytes back, code + layout]
//   -> metadata and plane (one wave per chunk: lane_bits, the chunk's total, its nibble plane; the first
//   workgroups write the header, the pair table and the padding between sections) -> prefix sum of the
//   totals (a workgroup per 1024 chunks; one in all above 65536 of them) -> stream (one wave per chunk assembles its span
//   in LDS and copies it out; the two dwords a span may share with its neighbours go out with atomic OR).
// The input is read three times (histogram, metadata, stream), the last two mostly from the memory-side cache.
// No scratch memory: the histogram is counted into the header's freq[] field and the chunk
// totals into chunk_bit[], both part of the output.
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

// A lane's pieces of a chunk; `whole`: the chunk lies entirely inside the tensor (the same for every lane).
template <int N>
__device__ __forceinline__ void load_pieces(const EncArgs &a, const ChunkPlace &p, bool whole, u32x4 (&v)[N / 16])
{
    const GLOBAL uint8_t *x = (const GLOBAL uint8_t *)a.x;
    const uint64_t e0 = p.base + p.lane_off;
    if (whole) {
#pragma unroll
        for (int q = 0; q < N / 16; q++) v[q] = *(const GLOBAL u32x4 *)(x + e0 + q * p.stride);
    } else {
#pragma unroll
        for (int q = 0; q < N / 16; q++) {
            const uint64_t e = e0 + q * p.stride;
            v[q] = e + 16 <= a.n ? *(const GLOBAL u32x4 *)(x + e) : load_cut(x, e, a.n);
        }
    }
}

// elements of the piece at e that exist
__device__ __forceinline__ uint32_t piece_len(uint64_t e, uint64_t n) { return e + 16 <= n ? 16u : e < n ? (uint32_t)(n - e) : 0u; }

// Exponent-field histogram into 16 u64 counters.  Counted with bit planes: 32 elements are turned into four 32-bit
// words, one per exponent bit, and each of the 16 exponents is then one AND and one population count that also adds:
// two vector operations per element and no LDS.  58.7 M weights: 14.5 us (4 TB/s; counters private to a thread in LDS,
// one read-modify-write per element, 37 us).  What is left is the read and its latency.
__global__ __launch_bounds__(1024) void histogram_kernel(uint64_t x_, uint64_t n, uint64_t counters_)
{
    __shared__ uint32_t s_cnt[16];
    const GLOBAL uint8_t *x = (const GLOBAL uint8_t *)x_;
    GLOBAL unsigned long long *counters = (GLOBAL unsigned long long *)counters_;
    const int tid = threadIdx.x, lane = tid & 63;
    if (tid < 16) s_cnt[tid] = 0;
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
}

// Everything of the container that is neither chunk data nor stream, by workgroup `part` of `parts` of 256 threads:
// header, pair table (256 entries per workgroup and round), zeros in the gaps between sections and in the dwords of the
// stream section from the one that holds its last bit on.
__device__ __forceinline__ void write_fixed(const EncArgs &a, const ecf8_header &h, uint32_t part, uint32_t parts, int tid)
{
    GLOBAL uint8_t *blob = (GLOBAL uint8_t *)a.blob;
    if (part == 0) {
        if (tid < 64) ((GLOBAL uint32_t *)blob)[tid] = ((const uint32_t *)&h)[tid];
        if (tid == 0) *(GLOBAL uint64_t *)(blob + a.off_cb) = 0;
        auto zero = [&](uint64_t from, uint64_t to) {       // multiples of four
            for (uint64_t i = from + 4 * tid; i < to; i += 1024) *(GLOBAL uint32_t *)(blob + i) = 0;
        };
        zero(a.off_cb + 8 * (a.n_chunks + 1), a.off_lb);
        zero(a.off_lb + 128 * a.n_chunks, a.off_st);
        zero(a.off_st + (h.stream_bits >> 5) * 4, a.off_pl);
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
    for (uint32_t i = part * 256 + tid; i < (uint32_t)TBL_ENTRIES; i += parts * 256) {
        const uint32_t t1 = first(i), l1 = t1 >> 4, t2 = l1 ? first(i >> l1) : 0u;
        ((GLOBAL uint16_t *)(blob + 256))[i] = ecf8_pair_entry(t1 & 15u, l1, t2 & 15u, t2 >> 4);
    }
}

// lane_bits[c][l] = code bits of the lane's symbols; chunk_bit[c + 1] = bits of chunk c (turned into stream positions
// by the scan below); the chunk's nibble plane (8 elements -> 4 bytes: byte j = low nibble element j, high nibble
// element j + 4), zeros where the last chunk reaches past the tensor.  One wave per chunk; the first `parts` workgroups
// write the fixed parts instead.  Code lengths are looked up four at a time: two byte permutes of the 16 lengths
// held in four registers, selected by the exponents' top bits, summed by one v_sad_u8.  58.7 M weights: 15.5 us for the
// 89 MB it reads and writes, i.e. a copy's rate (metadata and plane each in a kernel of its own, 15 + 8 .. 14 us, after a
// zero fill of the whole blob, 10 us, and the pair table by one workgroup, 8 us).
template <int N>
__global__ __launch_bounds__(256) void meta_kernel(EncArgs a, ecf8_header h, uint32_t parts, uint64_t first_block)
{
    const int tid = threadIdx.x, lane = tid & 63;
    if (blockIdx.x < parts) {
        write_fixed(a, h, blockIdx.x, parts, tid);
        return;
    }
    const uint64_t c = (first_block + (blockIdx.x - parts)) * 4 + uniform32((uint32_t)tid >> 6);
    if (c >= a.n_chunks) return;
    uint32_t len_bytes[4];                   // code lengths of symbols 4i .. 4i + 3
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const uint32_t l = (uint32_t)(a.len_packed >> (16 * i));
        len_bytes[i] = (l & 15u) | ((l & 0xf0u) << 4) | ((l & 0xf00u) << 8) | ((l & 0xf000u) << 12);
    }
    const bool whole = (c + 1) * (64ull * N) <= a.n;
    const ChunkPlace p = place_of<N>(a, c, lane);
    u32x4 v[N / 16];
    load_pieces<N>(a, p, whole, v);
    uint32_t lb = 0;
    GLOBAL uint8_t *plane = (GLOBAL uint8_t *)(a.blob + a.off_pl) + (p.base + p.lane_off) / 2;
#pragma unroll
    for (int q = 0; q < N / 16; q++) {
        const uint32_t w[4] = {v[q].x, v[q].y, v[q].z, v[q].w};
        const uint32_t have = whole ? 16u : piece_len(p.base + p.lane_off + q * p.stride, a.n);
        uint32_t nib[4];
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const uint32_t low = (w[k] >> 3) & 0x07070707u;
            const uint32_t top = ((w[k] >> 2) & 0x10101010u) - ((w[k] >> 6) & 0x01010101u);       // 0x0f in the bytes with exponents 8 .. 15
            uint32_t len = bit_select(top, __builtin_amdgcn_perm(len_bytes[3], len_bytes[2], low), __builtin_amdgcn_perm(len_bytes[1], len_bytes[0], low));
            if (!whole) {
                const uint32_t left = have > 4u * k ? have - 4u * k : 0u;
                len = left >= 4 ? len : len & ((1u << (8 * left)) - 1u);
            }
            lb = __builtin_amdgcn_sad_u8(len, 0u, lb);
            nib[k] = bit_select(0x07070707u, w[k], w[k] >> 4);                                    // low nibbles; the rest is masked off below
        }
        const u32x2 out{bit_select(0x0f0f0f0fu, nib[0], nib[1] << 4), bit_select(0x0f0f0f0fu, nib[2], nib[3] << 4)};
        *(GLOBAL u32x2 *)(plane + q * (p.stride / 2)) = out;
    }
    ((GLOBAL uint16_t *)(a.blob + a.off_lb))[c * 64 + lane] = (uint16_t)lb;
    const uint32_t total = wave_incl_scan(lb);
    if (lane == 63) ((GLOBAL uint64_t *)(a.blob + a.off_cb))[c + 1] = (uint64_t)total << TOTAL_AT;
}

// Stream: one wave per chunk.  A lane's bits are one string, the forward run's codewords in order and then the backward
// run's in reverse (each with its first bit highest), so a lane packs them one behind the other in a register and
// ORs every finished dword into the chunk's span in LDS; neighbouring lanes share a dword at their borders.  Symbols
// are looked up in pairs: 256 entries of the two codewords joined and their length, for either direction.  CAP7 (no
// codeword over 7 bits): two pairs are joined before they are packed.  58.7 M weights: 21 us, of which the 81 MB read and
// written take 16 at a copy's rate (one byte load and two LDS atomics per symbol took 105 us).
template <int N, bool CAP7>
__global__ __launch_bounds__(256) void pack_kernel(EncArgs a)
{
    constexpr int STAGE = 2 * N * (CAP7 ? 7 : 15) + 8;      // dwords: the longest span under the cap, begun anywhere in a 16-byte unit
    static_assert(STAGE % 4 == 0, "16-byte accesses");
    typedef typename std::conditional<CAP7, uint32_t, uint64_t>::type Entry;        // codewords; length from bit 26 or 32
    constexpr int LEN_AT = CAP7 ? 26 : 32;
    __shared__ __attribute__((aligned(16))) uint32_t stage_all[4][STAGE];
    __shared__ Entry s_fwd[256], s_bwd[256];
    __shared__ uint32_t s_one[2][17];                       // single symbols, code | length << 16; 16 = no symbol
    const int tid = threadIdx.x, lane = tid & 63, wave = (int)uniform32((uint32_t)tid >> 6);
    {
        const uint32_t lo = tid & 15, hi = tid >> 4;        // an entry's first and second element
        const uint32_t l0 = (uint32_t)(a.len_packed >> (4 * lo)) & 15u, l1 = (uint32_t)(a.len_packed >> (4 * hi)) & 15u;
        s_fwd[tid] = (Entry)(a.rcode[lo] | (a.rcode[hi] << l0)) | ((Entry)(l0 + l1) << LEN_AT);
        s_bwd[tid] = (Entry)(a.code[hi] | (a.code[lo] << l1)) | ((Entry)(l0 + l1) << LEN_AT);
        if (tid < 17) {
            const uint32_t l = tid < 16 ? l0 : 0u;
            s_one[0][tid] = tid < 16 ? a.rcode[lo] | (l << 16) : 0u;
            s_one[1][tid] = tid < 16 ? a.code[lo] | (l << 16) : 0u;
        }
    }
    __syncthreads();
    uint32_t *stage = stage_all[wave];
    GLOBAL uint64_t *cb = (GLOBAL uint64_t *)(a.blob + a.off_cb);
    const uint64_t mask = position_mask(a.n_chunks);
    for (uint64_t c = (uint64_t)blockIdx.x * 4 + wave; c < a.n_chunks; c += (uint64_t)gridDim.x * 4) {       // the same for the whole wave
        const bool whole = (c + 1) * (64ull * N) <= a.n;
        const ChunkPlace p = place_of<N>(a, c, lane);
        u32x4 v[N / 16];
        load_pieces<N>(a, p, whole, v);
        uint64_t b0, b1;
        chunk_positions(cb, c, mask, lane, b0, b1);
        const uint32_t lb = ((const GLOBAL uint16_t *)(a.blob + a.off_lb))[c * 64 + lane];
        const uint32_t n_units = (uint32_t)(((b1 + 127) >> 7) - (b0 >> 7));
        for (uint32_t u = lane; u < n_units && u < (uint32_t)STAGE / 4; u += 64) *(u32x4 *)(stage + 4 * u) = u32x4{0, 0, 0, 0};
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const uint32_t at = (uint32_t)(b0 & 127) + (wave_incl_scan(lb) - lb);     // stage bit of the lane's first bit
        LanePacker out(stage, at);
        // the four symbols of dword w, in order (BWD = false) or in reverse
        auto put4 = [&](auto bwd, uint32_t w) {
            constexpr bool BWD = decltype(bwd)::value;
            const Entry *tab = BWD ? s_bwd : s_fwd;
            const uint32_t t = (w >> 3) & 0x0f0f0f0fu, u = t | (t >> 4);           // bytes 0 and 2: two exponents each
            Entry ea = tab[u & 0xffu], eb = tab[(u >> 16) & 0xffu];
            if (BWD) { const Entry x = ea; ea = eb; eb = x; }
            if constexpr (CAP7) {
                const uint32_t la = ea >> LEN_AT, lb2 = eb >> LEN_AT;
                out.put((ea & ((1u << LEN_AT) - 1u)) | ((eb & ((1u << LEN_AT) - 1u)) << la), la + lb2);
            } else {
                out.put((uint32_t)ea, (uint32_t)(ea >> LEN_AT));
                out.put((uint32_t)eb, (uint32_t)(eb >> LEN_AT));
            }
        };
        if (whole) {
#pragma unroll
            for (int q = 0; q < N / 32; q++) {
                put4(std::false_type{}, v[q].x); put4(std::false_type{}, v[q].y); put4(std::false_type{}, v[q].z); put4(std::false_type{}, v[q].w);
            }
#pragma unroll
            for (int q = N / 16 - 1; q >= N / 32; q--) {
                put4(std::true_type{}, v[q].w); put4(std::true_type{}, v[q].z); put4(std::true_type{}, v[q].y); put4(std::true_type{}, v[q].x);
            }
        } else {
            // the ragged last chunk: symbol by symbol, those past the tensor's end have no bits
            auto put_piece = [&](bool back, u32x4 piece, uint32_t have) {
#pragma unroll 1
                for (uint32_t k = 0; k < 16; k++) {
                    const uint32_t j = back ? 15 - k : k, w = j < 8 ? (j < 4 ? piece.x : piece.y) : (j < 12 ? piece.z : piece.w);
                    const uint32_t s = j < have ? (w >> (8 * (j & 3) + 3)) & 15u : 16u;
                    const uint32_t e = s_one[back][s];
                    out.put(e & 0xffffu, e >> 16);
                }
            };
            const uint64_t e0 = p.base + p.lane_off;
#pragma unroll
            for (int q = 0; q < N / 32; q++) put_piece(false, v[q], piece_len(e0 + q * p.stride, a.n));
#pragma unroll
            for (int q = N / 16 - 1; q >= N / 32; q--) put_piece(true, v[q], piece_len(e0 + q * p.stride, a.n));
        }
        out.finish();
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        copy_span(stage, (GLOBAL uint32_t *)(a.blob + a.off_st), b0, b1, lane);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
}

template <int N>
int launch_pass2(const EncArgs &a, const ecf8_header &h, uint32_t lmax, hipStream_t s)
{
    const int cus = device_cus();
    if (cus <= 0) return ECF8_E_HIP;
    const uint32_t parts = h.table_bits ? 64 : 1;
    const uint64_t chunk_blocks = (h.n_chunks + 3) / 4;
    for (uint64_t b = 0; b < chunk_blocks; b += META_BLOCKS) {
        const uint32_t fixed = b == 0 ? parts : 0, blocks = (uint32_t)(chunk_blocks - b < META_BLOCKS ? chunk_blocks - b : META_BLOCKS);
        hipLaunchKernelGGL(meta_kernel<N>, dim3(blocks + fixed), dim3(256), 0, s, a, h, fixed, b);
    }
    // prefix sum and packing store where the metadata say: neither without what it reads
    if (hipGetLastError() != hipSuccess) return ECF8_E_HIP;
    launch_scan(a.blob + a.off_cb, h.n_chunks, a.blob + a.off_st, s);
    if (hipGetLastError() != hipSuccess) return ECF8_E_HIP;
    const uint64_t most = (uint64_t)cus * 8;
    const uint32_t pg = (uint32_t)(chunk_blocks < most ? chunk_blocks : most);
    if (lmax <= 7) hipLaunchKernelGGL((pack_kernel<N, true>), dim3(pg), dim3(256), 0, s, a);
    else hipLaunchKernelGGL((pack_kernel<N, false>), dim3(pg), dim3(256), 0, s, a);
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
    hipLaunchKernelGGL(fill_zero_kernel, dim3(1), dim3(256), 0, s, blob, (uint64_t)256);
    // one workgroup per compute unit at the most: each ends with 16 atomic additions to one line
    const uint64_t hist_blocks = (n / 4096 + 15) / 16, hist_most = (uint64_t)cus;
    hipLaunchKernelGGL(histogram_kernel, dim3((uint32_t)(hist_blocks < 1 ? 1 : hist_blocks < hist_most ? hist_blocks : hist_most)), dim3(1024), 0, s, x, n,
                       blob + 128);
    uint64_t freq[16];
    if (!read_back(freq, blob + 128, sizeof(freq), s)) return ECF8_E_HIP;

    ecf8_internal::Plan plan;
    rc = ecf8_internal::plan_encode(freq, rows, cols, opts, &plan);
    if (rc) return rc;
    const ecf8_header &h = plan.hdr;
    if (h.total_size > blob_capacity) return ECF8_E_CAPACITY;

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
    rc = N == 32 ? launch_pass2<32>(a, h, longest, s) : N == 64 ? launch_pass2<64>(a, h, longest, s) : launch_pass2<128>(a, h, longest, s);
    if (rc) return rc;
    *hdr_out = h;
    return ECF8_OK;
}

} // extern "C"
