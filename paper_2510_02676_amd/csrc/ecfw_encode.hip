// GPU-side encoder of the wide-alphabet codec (E5M2, BF16) for gfx950: Section 3.1 on the device
// for 5- and 8-bit exponent fields.  Writes exactly the container ecfw_encode writes, byte for byte:
// the code and the layout come from the same host routine, fed with the device histogram.
//
//   fill 0 (header, code lengths, freq) -> histogram -> [host: the histogram back, code + layout]
//   -> metadata and planes (one wave per chunk: lane_bits, the chunk's total, the remaining bits of its elements; the
//   first workgroup writes header, code lengths and the padding between sections) -> prefix sum of the
//   totals -> stream (one wave per chunk assembles its span in LDS and copies it out; the two dwords a span may share
//   with its neighbours go out with atomic OR).
// No scratch memory: the histogram is counted into the freq section and the chunk totals into
// chunk_bit[], both part of the output.
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

// A lane's pieces of a chunk; `whole`: the chunk lies entirely inside the tensor (the same for every lane).
template <int FMT, int N>
__device__ __forceinline__ void load_pieces(const WEncArgs &a, const ChunkPlace &p, bool whole, u32x4 (&v)[N / EFmt<FMT>::P])
{
    constexpr int ELEM = EFmt<FMT>::ELEM;
    const GLOBAL uint8_t *x = (const GLOBAL uint8_t *)a.x;
    const uint64_t e0 = (p.base + p.lane_off) * ELEM;
#pragma unroll
    for (int q = 0; q < N / EFmt<FMT>::P; q++) {
        const uint64_t e = e0 + q * p.stride * ELEM;
        v[q] = whole || e + 16 <= a.n * ELEM ? *(const GLOBAL u32x4 *)(x + e) : load_cut(x, e, a.n * ELEM);
    }
}

// Histogram of the exponent field into A u64 counters, one workgroup of 16 waves per compute unit.
//  * E5M2: bit planes.  32 elements are turned into five 32-bit words, one per exponent bit, and each of the 32 exponents
//    is one AND and one population count that also adds: four vector operations per element, no LDS.
//  * BF16: LDS counters in 64 copies, lane l of every wave in copy l = bank l, so that the lanes of a wave, most of which
//    hold one of a handful of exponents, never meet.  58.7 M elements: 21 us, 5.5 TB/s (16 copies: 47 us).
template <int FMT>
__global__ __launch_bounds__(1024) void w_histogram_kernel(uint64_t x_, uint64_t n, uint64_t counters_)
{
    constexpr int A = EFmt<FMT>::A, COPIES = FMT == ECFW_FMT_BF16 ? 64 : 1;
    __shared__ uint32_t s_cnt[A * COPIES];
    const GLOBAL uint8_t *x = (const GLOBAL uint8_t *)x_;
    GLOBAL unsigned long long *counters = (GLOBAL unsigned long long *)counters_;
    const int tid = threadIdx.x, lane = tid & 63;
    for (int i = tid; i < A * COPIES; i += 1024) s_cnt[i] = 0;
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
}

struct WHeadArgs {
    ecfw_header h;
    uint8_t len[256];
};

struct WCodeArgs {
    uint16_t code[256];                   // canonical codewords, first bit most significant
    uint8_t len[256];
};

// Everything of the container that is neither chunk data nor stream (the freq section already holds the histogram):
// header, code lengths, zeros in the gaps between sections and in the dwords of the stream section from the one that
// holds its last bit on.
__device__ __forceinline__ void write_fixed(const WEncArgs &a, const WHeadArgs &ha, int tid)
{
    GLOBAL uint8_t *blob = (GLOBAL uint8_t *)a.blob;
    const ecfw_header &h = ha.h;
    if (tid < 64) ((GLOBAL uint32_t *)blob)[tid] = ((const uint32_t *)&h)[tid];
    if ((uint32_t)tid * 4 < h.n_alphabet) *(GLOBAL uint32_t *)(blob + a.off_len + 4 * tid) = ((const uint32_t *)ha.len)[tid];
    if (tid == 0) *(GLOBAL uint64_t *)(blob + a.off_cb) = 0;
    auto zero = [&](uint64_t from, uint64_t to) {       // multiples of four
        for (uint64_t i = from + 4 * tid; i < to; i += 1024) *(GLOBAL uint32_t *)(blob + i) = 0;
    };
    zero(a.off_cb + 8 * (a.n_chunks + 1), a.off_lb);
    zero(a.off_lb + 128 * a.n_chunks, a.off_st);
    zero(a.off_st + (h.stream_bits >> 5) * 4, a.off_pl);
    zero(a.off_pl + h.plane_bytes, h.sign_bytes ? a.off_sg : h.total_size);
    if (h.sign_bytes) zero(a.off_sg + h.sign_bytes, h.total_size);
}

// lane_bits[c][l] = code bits of the lane's symbols; chunk_bit[c + 1] = bits of chunk c (turned into stream positions by
// the scan); the chunk's planes, zeros where the last chunk reaches past the tensor.  One wave per chunk; the
// first workgroup writes the fixed parts instead.  The code lengths sit in 256 bytes of LDS: 64 dwords, one per bank.
template <int FMT, int N>
__global__ __launch_bounds__(256) void w_meta_kernel(WEncArgs a, WHeadArgs ha, uint32_t parts, uint64_t first_block)
{
    using F = EFmt<FMT>;
    constexpr int P = F::P;
    __shared__ uint32_t s_len4[64];
    const uint8_t *s_len = (const uint8_t *)s_len4;
    const int tid = threadIdx.x, lane = tid & 63;
    if (blockIdx.x < parts) {
        write_fixed(a, ha, tid);
        return;
    }
    const uint64_t c = (first_block + (blockIdx.x - parts)) * 4 + uniform32((uint32_t)tid >> 6);
    const bool here = c < a.n_chunks;
    const bool whole = (c + 1) * (64ull * N) <= a.n;
    const ChunkPlace p = place_of<FMT, N>(a, c, lane);
    u32x4 v[N / P];
    if (here) load_pieces<FMT, N>(a, p, whole, v);
    if (tid < 64) s_len4[tid] = ((const uint32_t *)ha.len)[tid];
    __syncthreads();
    if (!here) return;
    uint32_t lb = 0;
    GLOBAL uint8_t *plane = (GLOBAL uint8_t *)(a.blob + a.off_pl), *signs = (GLOBAL uint8_t *)(a.blob + a.off_sg);
#pragma unroll
    for (int q = 0; q < N / P; q++) {
        const uint64_t e = p.base + p.lane_off + q * p.stride;
        const uint32_t w[4] = {v[q].x, v[q].y, v[q].z, v[q].w};
        if (whole) {
#pragma unroll
            for (int j = 0; j < P; j++) lb += s_len[F::sym(w, j)];
        } else {
            const uint32_t have = e + P <= a.n ? (uint32_t)P : e < a.n ? (uint32_t)(a.n - e) : 0u;
#pragma unroll
            for (int j = 0; j < P; j++) lb += (uint32_t)j < have ? s_len[F::sym(w, j)] : 0u;
        }
        if constexpr (FMT == ECFW_FMT_BF16) {
            // sign << 7 | mantissa in bytes 0 and 2 of a dword's two elements; the bytes of four elements in the order 0 2 1 3
            uint32_t r[4];
#pragma unroll
            for (int k = 0; k < 4; k++) r[k] = bit_select(0x007f007fu, w[k], w[k] >> 8);
            *(GLOBAL u32x2 *)(plane + e) = u32x2{bit_select(0x00ff00ffu, r[0], r[1] << 8), bit_select(0x00ff00ffu, r[2], r[3] << 8)};
        } else {
            // mantissa of element 4d + j in bits 8j + 2d; sign of element i in bit i
            const uint32_t m01 = bit_select(0x03030303u, w[0], w[1] << 2), m23 = bit_select(0x03030303u, w[2], w[3] << 2);
            uint32_t s = 0;
#pragma unroll
            for (int d = 0; d < 4; d++) {
                uint32_t y = (w[d] >> 7) & 0x01010101u;
                y |= y >> 7;
                s |= ((y | (y >> 14)) & 15u) << (4 * d);
            }
            *(GLOBAL uint32_t *)(plane + e / 4) = bit_select(0x0f0f0f0fu, m01, m23 << 4);
            *(GLOBAL uint16_t *)(signs + e / 8) = (uint16_t)s;
        }
    }
    ((GLOBAL uint16_t *)(a.blob + a.off_lb))[c * 64 + lane] = (uint16_t)lb;
    const uint32_t total = wave_incl_scan(lb);
    if (lane == 63) ((GLOBAL uint64_t *)(a.blob + a.off_cb))[c + 1] = (uint64_t)total << TOTAL_AT;
}

// Stream: one wave per chunk, as in the E4M3 encoder (a lane's bits are one string: the forward run's codewords in order,
// then the backward run's in reverse with their first bits highest).  The codewords come from the host with the launch;
// symbols are looked up one by one (256 of them would make a pair table of 256 KiB) and packed two at a time.  58.7 M BF16
// elements: 30 us for the 137 MB read and written (a load and two LDS atomics per symbol: 143 us).  LMAX: the longest codeword in use is at most this.
template <int FMT, int N, int LMAX>
__global__ __launch_bounds__(256) void w_pack_kernel(WEncArgs a, WCodeArgs ca)
{
    using F = EFmt<FMT>;
    constexpr int P = F::P, A = F::A;
    constexpr int STAGE = 2 * N * LMAX + 8;                 // dwords: the longest span, begun anywhere in a 16-byte unit
    static_assert(STAGE % 4 == 0, "16-byte accesses");
    __shared__ __attribute__((aligned(16))) uint32_t stage_all[4][STAGE];
    __shared__ uint32_t s_code[2][A + 1];                   // code | length << 16, first bit lowest / highest; A = no symbol
    const int tid = threadIdx.x, lane = tid & 63, wave = (int)uniform32((uint32_t)tid >> 6);
    if (tid < A) {
        const uint32_t code = ca.code[tid], l = ca.len[tid];
        s_code[0][tid] = l ? (__brev(code) >> (32 - l)) | (l << 16) : 0u;
        s_code[1][tid] = code | (l << 16);
    }
    if (tid < 2) s_code[tid][A] = 0;
    __syncthreads();
    uint32_t *stage = stage_all[wave];
    GLOBAL uint64_t *cb = (GLOBAL uint64_t *)(a.blob + a.off_cb);
    const uint64_t mask = position_mask(a.n_chunks);
    for (uint64_t c = (uint64_t)blockIdx.x * 4 + wave; c < a.n_chunks; c += (uint64_t)gridDim.x * 4) {   // the same for the whole wave
        const bool whole = (c + 1) * (64ull * N) <= a.n;
        const ChunkPlace p = place_of<FMT, N>(a, c, lane);
        u32x4 v[N / P];
        load_pieces<FMT, N>(a, p, whole, v);
        uint64_t b0, b1;
        chunk_positions(cb, c, mask, lane, b0, b1);
        const uint32_t lb = ((const GLOBAL uint16_t *)(a.blob + a.off_lb))[c * 64 + lane];
        const uint32_t n_units = (uint32_t)(((b1 + 127) >> 7) - (b0 >> 7));
        for (uint32_t u = lane; u < n_units && u < (uint32_t)STAGE / 4; u += 64) *(u32x4 *)(stage + 4 * u) = u32x4{0, 0, 0, 0};
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        LanePacker out(stage, (uint32_t)(b0 & 127) + (wave_incl_scan(lb) - lb));
        auto put2 = [&](uint32_t e0, uint32_t e1) {
            out.put((e0 & 0xffffu) | ((e1 & 0xffffu) << (e0 >> 16)), (e0 >> 16) + (e1 >> 16));
        };
        if (whole) {
#pragma unroll
            for (int q = 0; q < N / P / 2; q++) {
                const uint32_t w[4] = {v[q].x, v[q].y, v[q].z, v[q].w};
#pragma unroll
                for (int j = 0; j < P; j += 2) put2(s_code[0][F::sym(w, j)], s_code[0][F::sym(w, j + 1)]);
            }
#pragma unroll
            for (int q = N / P - 1; q >= N / P / 2; q--) {
                const uint32_t w[4] = {v[q].x, v[q].y, v[q].z, v[q].w};
#pragma unroll
                for (int j = P - 1; j > 0; j -= 2) put2(s_code[1][F::sym(w, j)], s_code[1][F::sym(w, j - 1)]);
            }
        } else {
            // the ragged last chunk: elements past the tensor's end have no bits
            auto put_piece = [&](bool back, const u32x4 &piece, uint64_t e) {
                const uint32_t have = e + P <= a.n ? (uint32_t)P : e < a.n ? (uint32_t)(a.n - e) : 0u;
#pragma unroll 1
                for (uint32_t k = 0; k < (uint32_t)P; k++) {
                    const uint32_t j = back ? P - 1 - k : k;
                    const uint32_t word = j * 4 / P, w = word < 2 ? (word ? piece.y : piece.x) : (word == 2 ? piece.z : piece.w);
                    const uint32_t at = F::ELEM == 1 ? 8 * (j & 3) + 2 : 16 * (j & 1) + 7;
                    put2(s_code[back][j < have ? (w >> at) & (uint32_t)(A - 1) : (uint32_t)A], 0u);
                }
            };
            const uint64_t e0 = p.base + p.lane_off;
#pragma unroll
            for (int q = 0; q < N / P / 2; q++) put_piece(false, v[q], e0 + q * p.stride);
#pragma unroll
            for (int q = N / P - 1; q >= N / P / 2; q--) put_piece(true, v[q], e0 + q * p.stride);
        }
        out.finish();
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        copy_span(stage, (GLOBAL uint32_t *)(a.blob + a.off_st), b0, b1, lane);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
}

template <int FMT, int N>
int launch_pass2(const WEncArgs &a, const WHeadArgs &ha, const WCodeArgs &ca, hipStream_t s)
{
    const int cus = device_cus();
    if (cus <= 0) return ECF8_E_HIP;
    const uint64_t chunk_blocks = (a.n_chunks + 3) / 4;
    for (uint64_t b = 0; b < chunk_blocks; b += META_BLOCKS) {
        const uint32_t fixed = b == 0 ? 1 : 0, blocks = (uint32_t)(chunk_blocks - b < META_BLOCKS ? chunk_blocks - b : META_BLOCKS);
        hipLaunchKernelGGL((w_meta_kernel<FMT, N>), dim3(blocks + fixed), dim3(256), 0, s, a, ha, fixed, b);
    }
    // prefix sum and packing store where the metadata say: neither without what it reads
    if (hipGetLastError() != hipSuccess) return ECF8_E_HIP;
    launch_scan(a.blob + a.off_cb, a.n_chunks, a.blob + a.off_st, s);
    if (hipGetLastError() != hipSuccess) return ECF8_E_HIP;
    const uint64_t most = (uint64_t)cus * 8;
    const uint32_t pg = (uint32_t)(chunk_blocks < most ? chunk_blocks : most);
    if (ha.h.max_code_len <= ECFW_TABLE_BITS) hipLaunchKernelGGL((w_pack_kernel<FMT, N, (int)ECFW_TABLE_BITS>), dim3(pg), dim3(256), 0, s, a, ca);
    else hipLaunchKernelGGL((w_pack_kernel<FMT, N, (int)ECFW_MAX_CODE_LEN>), dim3(pg), dim3(256), 0, s, a, ca);
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
    if (blob_capacity < fixed) return ECF8_E_CAPACITY;

    // pass 1: histogram, counted into the blob's freq section
    const int cus = device_cus();
    if (cus <= 0) return ECF8_E_HIP;
    hipLaunchKernelGGL(fill_zero_kernel, dim3(1), dim3(256), 0, s, blob, fixed);
    const uint64_t hist_blocks = (n * EFmt<FMT>::ELEM / 4096 + 15) / 16, hist_most = (uint64_t)cus;
    hipLaunchKernelGGL(w_histogram_kernel<FMT>, dim3((uint32_t)(hist_blocks < 1 ? 1 : hist_blocks < hist_most ? hist_blocks : hist_most)), dim3(1024), 0, s,
                       x, n, blob + off_freq);
    uint64_t freq[256] = {};
    if (!read_back(freq, blob + off_freq, 8ull * A, s)) return ECF8_E_HIP;

    ecfw_internal::WPlan plan;
    int rc = ecfw_internal::plan_encode(freq, FMT, rows, cols, N, group, lmax, &plan);
    if (rc) return rc;
    const ecfw_header &h = plan.hdr;
    if (h.total_size > blob_capacity) return ECF8_E_CAPACITY;
    if (h.off_freq != off_freq || h.off_chunk_bit != fixed) return ECF8_E_FORMAT;

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
    WHeadArgs ha;
    ha.h = h;
    WCodeArgs ca;
    for (int i = 0; i < 256; i++) {
        ha.len[i] = ca.len[i] = plan.len[i];
        ca.code[i] = (uint16_t)plan.code[i];
    }
    rc = N == 64 ? launch_pass2<FMT, 64>(a, ha, ca, s) : launch_pass2<FMT, 128>(a, ha, ca, s);
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
