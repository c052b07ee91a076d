// Kernels and helpers the two GPU-side encoders (ecf8_encode.hip, ecfw_encode.hip) share.
#ifndef ECF8_ENC_DEVICE_H
#define ECF8_ENC_DEVICE_H

#include "ecf8_device.h"

namespace {

__global__ __launch_bounds__(256) void fill_zero_kernel(uint64_t dst, uint64_t bytes)   // bytes % 16 == 0
{
    GLOBAL u32x4 *p = (GLOBAL u32x4 *)dst;
    const uint64_t n16 = bytes / 16;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = u32x4{0, 0, 0, 0};
}

// chunk_bit[1 .. n_chunks] on the way from chunk totals to stream positions.  The metadata kernels leave a chunk's total
// (at most 2^17 bits) in the upper bits of its entry; the prefix sum puts the position below it.
//  * Up to SLICED chunks, a workgroup per 1024 of them: each adds up the totals in front of its slice by itself (512 KiB at the
//    most) and scans the slice.  No workgroup waits for another: an entry reads the same from before and after its
//    update, because the total stays in it, and the packing kernels mask it off and write the plain position back.
//  * Above that one workgroup goes through all of them, 8192 a round: row k of a round is 1024 chunks side by side, scanned
//    by the waves, and the 128 (row, wave) totals are scanned once more by every wave.
// Where a chunk starts inside a dword of the stream, that dword holds bits of two chunks or more: it is zeroed here, and the
// packing kernels OR into it.  (One workgroup for everything: 7.0 us for 7168 chunks and 14 for 14336, half of it these
// scattered stores from one compute unit; sliced 3 .. 4 us.)
constexpr int TOTAL_AT = 46;
constexpr uint64_t SLICED = 1 << 16;
__host__ __device__ inline uint64_t position_mask(uint64_t n_chunks) { return n_chunks <= SLICED ? (1ull << TOTAL_AT) - 1 : ~0ull; }

__global__ __launch_bounds__(1024) void scan_kernel(uint64_t chunk_bit_, uint64_t n_chunks, uint64_t stream_)
{
    constexpr int ROWS = 8;
    __shared__ uint32_t totals[2][ROWS * 16];
    __shared__ uint64_t before_s[16];
    GLOBAL uint64_t *cb = (GLOBAL uint64_t *)chunk_bit_;
    GLOBAL uint32_t *stream = (GLOBAL uint32_t *)stream_;
    const int tid = threadIdx.x, lane = tid & 63, wave = (int)uniform32((uint32_t)tid >> 6);
    if (n_chunks <= SLICED) {
        const uint64_t first = 1 + 1024ull * blockIdx.x, i = first + tid;
        const uint32_t mine = i <= n_chunks ? (uint32_t)(cb[i] >> TOTAL_AT) : 0u;
        uint32_t front = 0;                               // at most 64 totals
#pragma unroll 8
        for (uint32_t k = 0; k < blockIdx.x; k++) front += (uint32_t)(cb[1 + tid + 1024ull * k] >> TOTAL_AT);
        const uint32_t incl = wave_incl_scan(mine), f = wave_incl_scan(front);      // 64 x 64 totals: 2^29
        if (lane == 63) {
            totals[0][wave] = incl;
            before_s[wave] = f;
        }
        __syncthreads();
        uint64_t at = incl;
#pragma unroll
        for (int w = 0; w < 16; w++) at += before_s[w] + (w < wave ? totals[0][w] : 0u);
        if (i <= n_chunks) {
            cb[i] = at | ((uint64_t)mine << TOTAL_AT);
            if (i < n_chunks && (at & 31)) stream[at >> 5] = 0;
        }
        return;
    }
    uint64_t carry = 0;
    int parity = 0;
    for (uint64_t base = 1; base <= n_chunks; base += 1024 * ROWS, parity ^= 1) {
        uint32_t v[ROWS];
#pragma unroll
        for (int k = 0; k < ROWS; k++) v[k] = base + 1024 * k + tid <= n_chunks ? (uint32_t)(cb[base + 1024 * k + tid] >> TOTAL_AT) : 0u;
#pragma unroll
        for (int k = 0; k < ROWS; k++) {
            v[k] = wave_incl_scan(v[k]);
            if (lane == 63) totals[parity][k * 16 + wave] = v[k];
        }
        __syncthreads();                                  // the other buffer is free again once everyone is here
        const uint32_t t0 = totals[parity][lane], t1 = totals[parity][64 + lane];
        const uint32_t s0 = wave_incl_scan(t0), half = (uint32_t)__builtin_amdgcn_readlane((int)s0, 63);
        const uint32_t s1 = half + wave_incl_scan(t1);
        const uint32_t x0 = s0 - t0, x1 = s1 - t1;        // totals before (row, wave)
#pragma unroll
        for (int k = 0; k < ROWS; k++) {
            const uint64_t i = base + 1024 * k + tid;
            const uint32_t before = (uint32_t)__builtin_amdgcn_readlane((int)(k < 4 ? x0 : x1), (k & 3) * 16 + wave);
            const uint64_t at = carry + before + v[k];
            if (i <= n_chunks) {
                cb[i] = at;
                if (i < n_chunks && (at & 31)) stream[at >> 5] = 0;
            }
        }
        carry += (uint32_t)__builtin_amdgcn_readlane((int)s1, 63);
    }
}

inline void launch_scan(uint64_t chunk_bit, uint64_t n_chunks, uint64_t stream, hipStream_t s)
{
    const uint32_t grid = n_chunks <= SLICED ? (uint32_t)((n_chunks + 1023) / 1024) : 1u;
    hipLaunchKernelGGL(scan_kernel, dim3(grid), dim3(1024), 0, s, chunk_bit, n_chunks, stream);
}

// The metadata kernels take a workgroup of 256 threads per four chunks.  A launch must stay below 2^32 work-items, which a single one
// would pass at 2^26 chunks (2^37 weights at 32 symbols per lane): they take as many as they need, of at most this many workgroups.
constexpr uint64_t META_BLOCKS = 1 << 20;

// The positions of chunk c's first and last bit, the latter written back plain.
__device__ __forceinline__ void chunk_positions(GLOBAL uint64_t *cb, uint64_t c, uint64_t mask, int lane, uint64_t &b0, uint64_t &b1)
{
    b0 = uniform64(cb[c]) & mask;
    b1 = uniform64(cb[c + 1]) & mask;
    if (~mask && lane == 0) cb[c + 1] = b1;
}

// Where chunk c's pieces lie: piece q of lane l starts at element base + q * stride + lane_off(l) (see the container's layouts).
struct ChunkPlace {
    uint64_t base, stride, lane_off;
};

// The 16 bytes at byte e of a tensor of n bytes, zeros from its end on.
__device__ __forceinline__ u32x4 load_cut(const GLOBAL uint8_t *x, uint64_t e, uint64_t n)
{
    uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < 4; k++) {
        const uint64_t d = e + 4 * k;
        if (d + 4 <= n) w[k] = *(const GLOBAL uint32_t *)(x + d);
        else
#pragma unroll
            for (int b = 0; b < 3; b++)
                if (d + b < n) w[k] |= (uint32_t)x[d + b] << (8 * b);
    }
    return u32x4{w[0], w[1], w[2], w[3]};
}

// A lane's string of bits on its way into the chunk's span in LDS (zeroed before): whole dwords are ORed in as they fill.
struct LanePacker {
    uint32_t *d;
    uint32_t fill, acc = 0;

    __device__ __forceinline__ LanePacker(uint32_t *stage, uint32_t at) : d(stage + (at >> 5)), fill(at & 31) {}
    __device__ __forceinline__ void put(uint32_t bits, uint32_t nb)          // nb <= 32, bits above nb clear
    {
        const uint64_t t = (uint64_t)bits << fill;
        acc |= (uint32_t)t;
        fill += nb;
        if (fill >= 32) {
            __hip_atomic_fetch_or(d, acc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
            d++;
            fill -= 32;
            acc = (uint32_t)(t >> 32);
        }
    }
    __device__ __forceinline__ void finish()
    {
        if (fill) __hip_atomic_fetch_or(d, acc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    }
};

// A chunk's span of the stream, assembled in LDS (`stage` = the 16-byte unit that holds stream bit b0, on), to its place:
// whole units by 16-byte stores, the units at the ends dword by dword; the first and the last dword may hold bits of
// other chunks, were zeroed by scan_kernel (or, the stream's last one, with the padding) and are ORed into.
__device__ __forceinline__ void copy_span(const uint32_t *stage, GLOBAL uint32_t *stream, uint64_t b0, uint64_t b1, int lane)
{
    const uint64_t unit0 = b0 >> 7;
    const uint32_t n_units = (uint32_t)(((b1 + 127) >> 7) - unit0);
    const uint64_t dw0 = b0 >> 5, dw1 = (b1 + 31) >> 5;                 // dwords [dw0, dw1) hold the span
    for (uint32_t u = lane; u < n_units; u += 64) {
        const u32x4 v = *(const u32x4 *)(stage + 4 * u);
        if (u != 0 && u + 1 != n_units) {
            *(GLOBAL u32x4 *)(stream + 4 * (unit0 + u)) = v;
            continue;
        }
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const uint64_t d = 4 * (unit0 + u) + k;
            if (d < dw0 || d >= dw1) continue;
            const bool shared = (d == dw0 && (b0 & 31)) || (d + 1 == dw1 && (b1 & 31));
            if (!shared) stream[d] = w[k];
            else if (w[k]) atomicOr((unsigned int *)(stream + d), w[k]);
        }
    }
}

// The encoders' one synchronisation: the histogram back to the host, when everything queued on `s` so far is done.  The
// call returns with the bytes in place; an asynchronous copy to pageable memory waits just as long, and the
// hipStreamSynchronize it needs for that to be certain adds a second round trip to the device.
inline bool read_back(void *host, uint64_t device, uint64_t bytes, hipStream_t s)
{
    return hipMemcpyWithStream(host, (const void *)(uintptr_t)device, bytes, hipMemcpyDeviceToHost, s) == hipSuccess;
}

} // namespace

#endif
