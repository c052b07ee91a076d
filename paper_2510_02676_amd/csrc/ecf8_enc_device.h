// Kernels and helpers the two GPU-side encoders (ecf8_encode.hip, ecfw_encode.hip) share.
#ifndef ECF8_ENC_DEVICE_H
#define ECF8_ENC_DEVICE_H

#include "ecf8_device.h"

#include <chrono>
#include <mutex>
#include <vector>

namespace {

// The workgroups' shares of chunk_bit[] are zeroed by the histogram kernels, which run before anything reads them.
__device__ __forceinline__ void zero_chunk_bits(uint64_t chunk_bit, uint64_t n_chunks, uint32_t tid, uint32_t threads)
{
    for (uint64_t i = (uint64_t)blockIdx.x * threads + tid; i <= n_chunks; i += (uint64_t)gridDim.x * threads) ((GLOBAL uint64_t *)chunk_bit)[i] = 0;
}

__global__ __launch_bounds__(256) void fill_zero_kernel(uint64_t dst, uint64_t bytes)   // bytes % 16 == 0
{
    GLOBAL u32x4 *p = (GLOBAL u32x4 *)dst;
    const uint64_t n16 = bytes / 16;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = u32x4{0, 0, 0, 0};
}

// Where chunk c's pieces lie: piece q of lane l starts at element base + q * stride + lane_off(l) (see the container's layouts).
struct ChunkPlace {
    uint64_t base, stride, lane_off;
};

// The 16 bytes at byte e of a tensor of n bytes, zeros from its end on.
__device__ __forceinline__ u32x4 load_cut(const GLOBAL uint8_t *x, uint64_t e, uint64_t n)
{
    if (e + 16 <= n) return *(const GLOBAL u32x4 *)(x + e);
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

// A lane's string of bits on its way into the wave's image in LDS (zeroed before): whole dwords are ORed in as they fill.
struct LanePacker {
    uint32_t *d;
    uint32_t fill, acc = 0;

    __device__ __forceinline__ LanePacker(uint32_t *image, uint32_t at) : d(image + (at >> 5)), fill(at & 31) {}
    __device__ __forceinline__ void put(uint32_t bits, uint32_t nb)          // nb <= 32, bits above nb clear
    {
        const uint64_t t = (uint64_t)bits << fill;              // (two 32-bit shifts measured slower: a BF16 matrix 80 -> 83 us)
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
    __device__ __forceinline__ uint32_t end(const uint32_t *image) const { return (uint32_t)(d - image) * 32 + fill; }     // the bit behind the last one
};

// ---- the container behind the code: one pass over the weights ----
// A wave takes a few chunks in a row, a workgroup as many times its waves, a tile.  Chunk by chunk the wave counts the code bits,
// writes the planes and packs the bits into its image in LDS, one chunk behind the other; where they go is only known when
// everything before them has been counted.  That the workgroups find out from one another, once per tile, and then copy the
// images to the stream, shifted into place.  Chunks that did not fit any more are packed after that.  Tiles are drawn from a counter, so that a workgroup waits only for tiles
// that were drawn before its own; these wait for earlier ones only, so every wait ends whatever part of the grid is running.
//
// The exchange goes through chunk_bit[], which the histogram kernel has zeroed.  Of the entries of tile t, which has T chunks,
//   [T t]      holds the tile's first bit once the tile before has written it, plain and for good (it is not 0: a chunk has a bit
//              per weight at least, and tile 0's entry is not read);
//   [T t + 1]  holds what the tile before has to say, until tile t replaces it by its plain value: SAID_TOTAL and its length from bit 32
//              on as soon as the code bits of its chunks are counted, SAID_TAIL and its last 32 bits once they are packed.
//              An entry that has been replaced reads as not said; then the first bit of tile t + 1 is on its way, and is what ends the wait.
// What bounds it: the exchange costs a tile 3 to 5 us, round trips through the memory side and waiting for the slowest wave, and the compute unit
// has nothing else to do meanwhile; hence tiles as large as the LDS holds, and one per compute unit where that is enough.
// 58.7 M E4M3 weights: tiles of eight chunks, two workgroups per compute unit, 52 us; of 16 chunks 42; of 32, one per compute unit, 32.
constexpr uint64_t SAID_TOTAL = 1ull << 63, SAID_TAIL = 1ull << 62;
constexpr int LATE_DWORDS = 20;             // end of an image: the last 32 codewords of a lane of a chunk that does not fit into the rest
constexpr int LATE_LANES = 32;              // a chunk of more bits than an image takes goes out by so many lanes at a time, whose bits fit whatever they are

__device__ __forceinline__ uint64_t agent_load(GLOBAL uint64_t *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void agent_store(GLOBAL uint64_t *p, uint64_t v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// One wave: the first bit of tile t, by adding up what the tiles before have said back to the nearest one whose first bit is known.
// WINDOWS x 64 tiles are asked for at a time, about as many as there are workgroups on the chip.
__device__ __forceinline__ uint64_t tile_begin(GLOBAL uint64_t *cb, uint32_t T, uint32_t t, int lane)
{
    constexpr int WINDOWS = 4;
    uint64_t between = 0;
    for (uint32_t s0 = t;;) {
        uint64_t at[WINDOWS], said[WINDOWS];                    // of tile s0 - 64 k - lane
#pragma unroll
        for (int k = 0; k < WINDOWS; k++) {
            at[k] = said[k] = 0;
            if ((uint32_t)lane + 64 * k < s0) {
                GLOBAL uint64_t *e = cb + (uint64_t)T * (s0 - 64 * k - lane);
                at[k] = agent_load(e);
                said[k] = agent_load(e + 1);
            }
        }
        bool again = false;
#pragma unroll
        for (int k = 0; k < WINDOWS; k++) {
            if (again) break;
            const uint64_t known = __ballot((uint32_t)lane >= s0 || at[k] != 0), there = __ballot(said[k] >> 63);
            const uint32_t f = known ? (uint32_t)__builtin_ctzll(known) : 64u;
            const uint64_t need = f < 64 ? (1ull << f) - 1 : ~0ull;
            if ((there & need) != need) {
                again = true;                                   // from this window on
                break;
            }
            const uint32_t sum = wave_incl_scan((uint32_t)lane < f ? (uint32_t)(said[k] >> 32) & 0x3fffffffu : 0u);      // at most 64 x 2^25: a tile is 16 waves of 16 chunks of 2^17 bits at the most
            between += (uint32_t)__builtin_amdgcn_readlane((int)sum, 63);
            if (f < 64)
                return between + ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(at[k] >> 32), (int)f) << 32 |
                                  (uint32_t)__builtin_amdgcn_readlane((int)at[k], (int)f));
            s0 -= 64;
        }
        if (again) __builtin_amdgcn_s_sleep(1);
    }
}

// What the waves of a workgroup tell one another about the tile they are at, in two buffers used in turn.
constexpr int WMAX = 16;                    // waves of a workgroup at the most
struct TileShared {
    uint64_t begin;
    uint64_t counted[2];                    // code bits of the waves that have counted theirs, from bit 40 on how many have
    uint32_t drawn[2];                      // the tile after it
    uint32_t total[2][WMAX], tail[2][WMAX]; // bits of a wave's chunks, the last 32 of them
};

// `bits` bits in front of bit number `bits` of an image: the last 32 of them, for bits >= 32.
__device__ __forceinline__ uint32_t last32(const uint32_t *image, uint32_t bits)
{
    return bits >= 32 ? __builtin_amdgcn_alignbit(image[bits >> 5], image[(bits >> 5) - 1], bits & 31) : 0u;
}

typedef uint32_t u32x4a __attribute__((ext_vector_type(4), aligned(4)));

// An image's bits to bits [b0, b1) of the stream: the dwords from the one that holds the first bit, whose lower bits are the last
// ones of image[-1], to the last one that the bits fill, `all`: to the last one that they reach.  `skip`: not the first one.
__device__ __forceinline__ void copy_bits(const uint32_t *image, GLOBAL uint32_t *stream, uint64_t b0, uint64_t b1, bool all, bool skip, int lane)
{
    const uint32_t n = (uint32_t)((b1 >> 5) - (b0 >> 5)) + (all && (b1 & 31) ? 1u : 0u), shift = (uint32_t)b0 & 31;
    GLOBAL uint32_t *out = stream + (b0 >> 5);
    for (uint32_t j = 4 * lane; j < n; j += 256) {
        const u32x4 w = *(const u32x4 *)(image + j);
        const uint32_t below = image[(int)j - 1];
        u32x4a v = {w.x, w.y, w.z, w.w};
        if (shift)
            v = u32x4a{__builtin_amdgcn_alignbit(w.x, below, 32 - shift), __builtin_amdgcn_alignbit(w.y, w.x, 32 - shift),
                       __builtin_amdgcn_alignbit(w.z, w.y, 32 - shift), __builtin_amdgcn_alignbit(w.w, w.z, 32 - shift)};
        if (j + 4 <= n && (j || !skip)) {
            *(GLOBAL u32x4a *)(out + j) = v;
        } else {
            if (j || !skip) out[j] = v.x;
            if (j + 1 < n) out[j + 1] = v.y;
            if (j + 2 < n) out[j + 2] = v.z;
            if (j + 3 < n) out[j + 3] = v.w;
        }
    }
}

struct TileArgs {
    uint64_t n_chunks;
    uint32_t per_wave;                      // chunks of a wave per tile, at most 16
    const uint32_t *header;                 // the blob's first 256 bytes
};

// The tiles of one workgroup.  K is a codec's chunk.  For chunks that lie entirely inside the tensor, fetch(c) asks for the weights, count(c) gives
// the lane's code bits and writes the planes, pack(image, at, c, refill) packs the lane's bits from image bit `at` on and asks for the weights of
// chunk c + 1 piece by piece as those of c are used up.  slow_count and slow_pack do the same for any chunk, from memory and rolled
// up: the code of the common way has to stay well inside the instruction cache (with the ragged chunk's code woven in, 118 KB, it took
// twice as long).  `image` is the wave's, K::AREA dwords, and image[-1] is there to be written.
template <class K>
__device__ __forceinline__ void encode_tiles(K &k, TileShared &sh, uint32_t *image, const TileArgs &ta, GLOBAL uint8_t *blob, uint64_t off_cb,
                                             uint64_t off_lb, uint64_t off_st, int lane, int wave)
{
    constexpr uint32_t ROOM = (uint32_t)(K::AREA - LATE_DWORDS - 2) * 32;       // bits an image takes, zeros behind them
    GLOBAL uint64_t *cb = (GLOBAL uint64_t *)(blob + off_cb);
    GLOBAL uint16_t *lane_bits = (GLOBAL uint16_t *)(blob + off_lb);
    GLOBAL uint32_t *stream = (GLOBAL uint32_t *)(blob + off_st);
    const uint32_t W = blockDim.x >> 6, T = W * ta.per_wave, n_tiles = (uint32_t)((ta.n_chunks + T - 1) / T);
    // The counter is the header's first dword, 0 from before the histogram; whoever draws last writes the header.
    uint32_t drawn = 0;
    auto draw = [&]() {
        if (threadIdx.x == 0) drawn = __hip_atomic_fetch_add((GLOBAL uint32_t *)blob, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    auto first_chunk = [&](uint32_t t) { return (uint64_t)T * t + (uint64_t)ta.per_wave * wave; };
    bool fetched = false;                   // the tile's first chunk
    auto zero = [&](uint32_t dwords) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // other lanes have read what this one clears
        for (uint32_t u = lane; u * 4 < dwords; u += 64) *(u32x4 *)(image + 4 * u) = u32x4{0, 0, 0, 0};
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    };
    draw();
    if (threadIdx.x == 0) {
        sh.drawn[1] = drawn;
        sh.counted[0] = sh.counted[1] = 0;
    }
    __syncthreads();
    uint32_t t = uniform32(sh.drawn[1]);
    for (uint32_t parity = 0; t < n_tiles; parity ^= 1) {
        const uint64_t first = (uint64_t)T * t, c0 = first_chunk(t);
        const bool followed = first + T < ta.n_chunks;
        const uint32_t count = c0 < ta.n_chunks ? (uint32_t)(ta.n_chunks - c0 < ta.per_wave ? ta.n_chunks - c0 : ta.per_wave) : 0u;
        uint32_t total = 0, used = 0, kept = 0, upto = 0, late_bits = 0;         // upto: lane i, bits up to the end of chunk i
        uint32_t lb = 0, incl = 0;                                               // of the chunk counted last
        if (!fetched && k.whole(c0)) k.fetch(c0);
        zero(K::AREA);
#pragma unroll 1
        for (uint32_t i = 0; i < count; i++) {
            const uint64_t c = c0 + i;
            const bool whole = k.whole(c);
            lb = whole ? k.count(c) : k.slow_count(c);
            lane_bits[c * 64 + lane] = (uint16_t)lb;
            incl = wave_incl_scan(lb);
            uint32_t bits = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
            bits = bits ? bits : 1u;                            // weights that change under the call have no codes: garbage, but no tile that begins at 0
            total += bits;
            upto = (uint32_t)lane == i ? total : upto;
            // not before: a workgroup that draws twice before others have drawn at all takes their tile from them
            if (i + 1 == count) draw();
            if (i + 1 == count && lane == 0) {
                // the last wave of the workgroup to have counted its chunks tells the next tile
                sh.total[parity][wave] = total;
                const uint64_t now = atomicAdd((unsigned long long *)&sh.counted[parity], (1ull << 40) + total) + (1ull << 40) + total;
                if ((now >> 40) == W && followed)
                    __hip_atomic_fetch_add(cb + first + T + 1, SAID_TOTAL | (now & ((1ull << 40) - 1)) << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            // A chunk that does not fit behind the others is packed when its place is known; of the last one the last bits are needed before.
            const bool fits = kept == i && used + bits <= ROOM, refill = fits && i + 1 < count && k.whole(c + 1);
            if (fits && whole) k.pack(image, used + incl - lb, c, refill);
            else if (fits || (i + 1 == count && lane == 63))
                late_bits = k.slow_pack(image + (fits ? 0 : K::AREA - LATE_DWORDS), fits ? used + incl - lb : 0u, c, fits ? 0 : K::TAIL_FROM);
            if (i + 1 < count && !refill && k.whole(c + 1)) k.fetch(c + 1);
            kept += fits ? 1u : 0u;
            used += fits ? bits : 0u;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        late_bits = (uint32_t)__builtin_amdgcn_readlane((int)late_bits, 63);
        if (lane == 0) {
            sh.tail[parity][wave] = kept == count ? last32(image, total) : last32(image + K::AREA - LATE_DWORDS, late_bits);
            if (wave == 0) sh.drawn[parity] = drawn;
        }
        __syncthreads();
        const uint32_t next = uniform32(sh.drawn[parity]);
        uint32_t before = 0, all = 0;
        for (uint32_t w = 0; w < W; w++) {
            const uint32_t v = sh.total[parity][w];
            before += w < (uint32_t)wave ? v : 0u;
            all += v;
        }
        if (wave == 0) {
            if (lane == 0) {
                sh.counted[parity] = 0;
                if (followed) __hip_atomic_fetch_add(cb + first + T + 1, SAID_TAIL | sh.tail[parity][W - 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            const uint64_t begin = tile_begin(cb, T, t, lane);
            if (lane == 0) {
                if (followed) agent_store(cb + first + T, begin + all);
                sh.begin = begin;
            }
        }
        fetched = kept == count;
        const uint64_t then = fetched ? first_chunk(next) : c0 + kept;
        if ((fetched ? next < n_tiles : kept + 1 < count) && k.whole(then)) k.fetch(then);
        __syncthreads();
        if (count) {
            const uint64_t b0 = uniform64(sh.begin) + before;
            const uint32_t shift = (uint32_t)b0 & 31;
            const bool skip = wave == 0 && shift;               // the tile's first dword comes last: it needs the end of the tile before
            if (lane == 0 && wave != 0) image[-1] = sh.tail[parity][wave - 1];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            copy_bits(image, stream, b0, b0 + used, kept == count && c0 + count == ta.n_chunks, skip, lane);
            uint32_t tail = wave ? sh.tail[parity][wave - 1] : 0u;
            if (wave == 0 && t != 0) {
                uint64_t said;                                  // all of it, before the entry is replaced
                while (((said = agent_load(cb + first + 1)) & (SAID_TOTAL | SAID_TAIL)) != (SAID_TOTAL | SAID_TAIL)) __builtin_amdgcn_s_sleep(1);
                tail = uniform32((uint32_t)said);
                if (skip && lane == 0 && (b0 >> 5 != (b0 + used) >> 5 || (kept == count && c0 + count == ta.n_chunks)))
                    stream[b0 >> 5] = __builtin_amdgcn_alignbit(image[0], tail, 32 - shift);
            }
            // all but the first bit of the tile behind, which the first wave has written
            if ((uint32_t)lane < count && !(followed && wave + 1 == (int)W && (uint32_t)lane + 1 == count)) agent_store(cb + c0 + lane + 1, b0 + upto);
            if (kept < count) {
                // The chunks that did not fit, image by image as before.  14336 x 7168 E4M3, the upper three quarters zeros: 86 us; with these chunks looked
                // up one symbol at a time by 16 lanes after the other 222 (84 with kernels of their own for counting and packing).  16384 x
                // 16384, half zeros: 193, 323, 222.
                uint64_t at = b0 + used;
                if (kept) tail = last32(image, used);
                used = 0;
                zero(K::AREA);
                auto flush = [&](bool end) {
                    if (lane == 0) image[-1] = tail;
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    copy_bits(image, stream, at, at + used, end, false, lane);
                    if (used >= 32) tail = last32(image, used);
                    else if (used) tail = (uint32_t)((((uint64_t)image[0] << 32 | tail) >> used));
                    at += used;
                    used = 0;
                    zero(K::AREA);
                };
#pragma unroll 1
                for (uint32_t i = kept; i < count; i++) {
                    const uint64_t c = c0 + i;
                    const bool whole = k.whole(c), more = i + 1 < count && k.whole(c + 1);
                    if (kept + 1 < count) {                     // else it is the chunk counted last, and as count has left it
                        lb = whole ? k.count(c) : k.slow_count(c);
                        incl = wave_incl_scan(lb);
                    }
                    const uint32_t bits = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
                    if (used + bits > ROOM) flush(false);
                    if (whole && bits <= ROOM) {
                        k.pack(image, used + incl - lb, c, false);
                        used += bits;
                    } else {
                        const int lanes = bits <= ROOM ? 64 : LATE_LANES;        // at a time, if an image does not take them all
                        for (int l0 = 0; l0 < 64; l0 += lanes) {
                            const uint32_t from = l0 ? (uint32_t)__builtin_amdgcn_readlane((int)incl, l0 - 1) : 0u;
                            if (lane >= l0 && lane < l0 + lanes) k.slow_pack(image, used + incl - lb - from, c, 0);
                            used += (uint32_t)__builtin_amdgcn_readlane((int)incl, l0 + lanes - 1) - from;
                            if (lanes != 64) flush(false);
                        }
                    }
                    if (more) k.fetch(c + 1);
                }
                flush(c0 + count == ta.n_chunks);
            }
        }
        t = next;
    }
    if (t == n_tiles + gridDim.x - 1 && threadIdx.x < 64)
        __hip_atomic_store((GLOBAL uint32_t *)blob + threadIdx.x, ta.header[threadIdx.x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Waves per workgroup, chunks per wave and tile, workgroups, for a stream of `bits` bits: a chunk on as many compute units as there are
// chunks; then more waves, up to WMAX; then as many chunks per wave as gives every compute unit the same number of tiles, up to what
// their images hold (with 15 % to spare: a chunk that does not fit is read and packed a second time).
struct TilePlan {
    uint32_t waves, per_wave, grid;
};
template <int AREA>
inline TilePlan plan_tiles(uint64_t n_chunks, uint64_t bits, uint32_t cus)
{
    TilePlan p;
    p.waves = n_chunks <= 4ull * cus ? 4u : n_chunks <= 8ull * cus ? 8u : (uint32_t)WMAX;
    const uint64_t each = (n_chunks + (uint64_t)p.waves * cus - 1) / ((uint64_t)p.waves * cus), mean = bits / n_chunks + 1;
    uint64_t hold = (uint64_t)(AREA - LATE_DWORDS - 2) * 32 * 100 / (115 * mean);
    hold = hold < 1 ? 1 : hold > 16 ? 16 : hold;
    const uint64_t rounds = (each + hold - 1) / hold;
    p.per_wave = (uint32_t)((each + rounds - 1) / rounds);
    const uint64_t tiles = (n_chunks + (uint64_t)p.waves * p.per_wave - 1) / ((uint64_t)p.waves * p.per_wave);
    p.grid = (uint32_t)(tiles < cus ? tiles : cus);
    return p;
}

// The encoders' one synchronisation: the histogram on its way to the host.  The workgroup of the histogram kernel that adds its counts last
// writes the sums to a page of pinned host memory and says so there, and the host looks at the page until it does.  A copy behind the
// kernel and the call that waits for it took longer: 14336 x 4096 E4M3 56.8 us -> 53.0, BF16 89.2 -> 84.3, 256 x 256 34 -> 25.
constexpr int MAIL_SAID = 256;              // behind the counts
constexpr uint32_t TICKET_AT = 4;           // byte of the blob: how many workgroups have added their counts, 0 from before the histogram

// By all threads of a workgroup, after their additions to `counters`.  mail: 0, or the page.  Counts, ticket and page are only touched by atomic
// operations, which no cache answers, and each wave waits for its own to be made; a release of the whole cache in their place costs 25 us.
template <int A>
__device__ __forceinline__ void mail_histogram(uint64_t blob, uint64_t counters, uint64_t mail)
{
    __shared__ uint32_t s_last;
    if (!mail) return;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // this wave's additions have been made ...
    __syncthreads();                                        // ... and so have every wave's
    if (threadIdx.x == 0) s_last = __hip_atomic_fetch_add((GLOBAL uint32_t *)(blob + TICKET_AT), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
    __syncthreads();
    if (!s_last) return;
    if (threadIdx.x < A)
        __hip_atomic_store((GLOBAL uint64_t *)mail + threadIdx.x, agent_load((GLOBAL uint64_t *)counters + threadIdx.x), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store((GLOBAL uint64_t *)mail + MAIL_SAID, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// While another thread captures a stream, some calls (to allocate, to free, to wait) fail in this one and spoil that capture, unless the thread says that
// they have nothing to do with it.  An encoder's have not: none of its pages is ever part of a graph, and it waits for no stream that is captured.
class CaptureRelaxed {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;

public:
    CaptureRelaxed() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    CaptureRelaxed(const CaptureRelaxed &) = delete;
    CaptureRelaxed &operator=(const CaptureRelaxed &) = delete;
    ~CaptureRelaxed() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
};

// A page for one call.  Pages of finished calls are kept for later ones, of any thread, stream and device: KEPT of them per encoder, others are given back.
class Mail {
    static constexpr size_t KEPT = 16;
    static std::mutex &lock() { static std::mutex m; return m; }
    static std::vector<uint64_t *> &free_pages() { static auto *v = new std::vector<uint64_t *>(); return *v; }    // outlives the runtime
    const CaptureRelaxed relaxed;           // from before the page is allocated until it is given back
    uint64_t *page = nullptr;
    void *seen = nullptr;                   // the page as a kernel sees it
    bool quiet = true;                      // no kernel may still write to it

public:
    Mail()
    {
        {
            std::lock_guard<std::mutex> lk(lock());
            if (!free_pages().empty()) {
                page = free_pages().back();
                free_pages().pop_back();
            }
        }
        if (!page && hipHostMalloc((void **)&page, 4096, hipHostMallocPortable | hipHostMallocMapped | hipHostMallocCoherent) != hipSuccess) {
            (void)hipGetLastError();
            page = nullptr;
        }
        if (page && hipHostGetDevicePointer(&seen, page, 0) != hipSuccess) {
            (void)hipGetLastError();
            (void)hipHostFree(page);
            page = nullptr;
        }
        if (page) __atomic_store_n(page + MAIL_SAID, 0ull, __ATOMIC_RELEASE);
    }
    Mail(const Mail &) = delete;
    Mail &operator=(const Mail &) = delete;
    ~Mail()
    {
        if (!page || !quiet) return;        // after a failed launch or wait: lost rather than written to in another call
        {
            std::lock_guard<std::mutex> lk(lock());
            if (free_pages().size() < KEPT) {
                if (free_pages().capacity() < KEPT) free_pages().reserve(KEPT);
                free_pages().push_back(page);
                return;
            }
        }
        (void)hipHostFree(page);
    }
    // for the kernel; 0: there is no page, and the histogram has to be copied
    uint64_t device()
    {
        quiet = !page;
        return page ? (uint64_t)(uintptr_t)seen : 0;
    }
    // The A counts, of the kernel that was given device(); without a page, from `counters`, by a copy that waits for all that is queued on s.
    bool read(uint64_t *host, int A, uint64_t counters, hipStream_t s)
    {
        if (!page) {
            if (hipMemcpyWithStream(host, (const void *)(uintptr_t)counters, 8ull * A, hipMemcpyDeviceToHost, s) == hipSuccess) return true;
            (void)hipGetLastError();
            return false;
        }
        const auto since = std::chrono::steady_clock::now();
        for (uint32_t i = 1; !__atomic_load_n(page + MAIL_SAID, __ATOMIC_ACQUIRE); i++) {
            __builtin_ia32_pause();
            // the stream has more to do, or it has failed
            if (i % 256 == 0 && std::chrono::steady_clock::now() - since > std::chrono::milliseconds(1)) {
                const bool done = hipStreamSynchronize(s) == hipSuccess;
                if (!done) (void)hipGetLastError();
                if (!done || !__atomic_load_n(page + MAIL_SAID, __ATOMIC_ACQUIRE)) return false;
                break;
            }
        }
        for (int i = 0; i < A; i++) host[i] = page[i];
        quiet = true;
        return true;
    }
};

// A stream that is being captured runs nothing: there is no histogram to wait for.  Nor is there on the null stream while one that waits for it is
// captured, which the question is answered with as an error: the caller has it from the return value, and the next launch's check is not to find it.
inline bool capturing(hipStream_t s)
{
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &st) == hipSuccess) return st != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return true;
}

} // namespace

#endif
