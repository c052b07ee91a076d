// Kernels and helpers the two GPU-side encoders (ecf8_encode.hip, ecfw_encode.hip) share.
#ifndef ECF8_ENC_DEVICE_H
#define ECF8_ENC_DEVICE_H

#include "ecf8_device.h"

#include <chrono>
#include <mutex>
#include <type_traits>
#include <vector>

namespace {

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

// A lane's string of bits on its way into the wave's image in LDS (zeroed before): whole dwords are ORed in as they fill.  `acc` holds the last 32 bits, the latest on
// top, so that a put is one funnel shift, and what a word has above its bits falls off.  ANY: puts of 32 bits occur.
template <bool ANY>
struct LanePacker {
    uint32_t *d;
    uint32_t fill, acc = 0;                 // fill: bits of the dword that is being filled, 0 .. 31

    __device__ __forceinline__ LanePacker(uint32_t *image, uint32_t at) : d(image + (at >> 5)), fill(at & 31) {}
    __device__ __forceinline__ void put(uint32_t bits, uint32_t nb)          // nb <= 31, or 32 with ANY
    {
        const uint32_t before = fill, old = acc;
        fill += nb;
        acc = __builtin_amdgcn_alignbit(bits, old, nb);
        if (ANY) acc = nb == 32 ? bits : acc;
        if (fill >= 32) {
            const uint32_t full = __builtin_amdgcn_alignbit(bits, old, 0u - before);
            __hip_atomic_fetch_or(d, ANY && before == 0 ? bits : full, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
            d++;
            fill -= 32;
        }
    }
    __device__ __forceinline__ void finish()
    {
        if (fill) __hip_atomic_fetch_or(d, acc >> (32 - fill), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    }
};

// Sums over lanes: of a half wave and the other, of a row of 16 and its neighbour (the result in both; of two values at once, a's in the lower half or the even
// rows and b's in the others), and over 4, 8 and 16 lanes in a row.
__device__ __forceinline__ uint32_t add_32(uint32_t a, uint32_t b) { const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false); return r[0] + r[1]; }
__device__ __forceinline__ uint32_t add_16(uint32_t a, uint32_t b) { const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false); return r[0] + r[1]; }
template <int DPP> __device__ __forceinline__ uint32_t add_dpp(uint32_t v) { return v + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, DPP, 0xf, 0xf, true); }
__device__ __forceinline__ uint32_t add_quad(uint32_t v) { return add_dpp<0x4e>(add_dpp<0xb1>(v)); }       // quad_perm [1 0 3 2], [2 3 0 1]
__device__ __forceinline__ uint32_t add_eight(uint32_t v) { return add_dpp<0x141>(add_quad(v)); }           // row_half_mirror
__device__ __forceinline__ uint32_t add_row(uint32_t v) { return add_dpp<0x140>(add_eight(v)); }            // row_mirror

// Counters of every lane, added up over the wave into A counters in LDS: two at a time in the wave's halves, then in its rows.
template <int A>
__device__ __forceinline__ void add_counts(const uint32_t (&cnt)[A], uint32_t *sums, int lane)
{
    uint32_t mine = 0;
#pragma unroll
    for (int i = 0; i < A / 4; i++) {
        const uint32_t v = add_row(add_16(add_32(cnt[4 * i], cnt[4 * i + 1]), add_32(cnt[4 * i + 2], cnt[4 * i + 3])));
        mine = (lane & 15) == i ? v : mine;
    }
    if ((lane & 15) < A / 4 && mine) atomicAdd(&sums[4 * (lane & 15) + (lane >> 5) + (lane >> 4 & 1) * 2], mine);
}

// A chunk's last 32 bits from its last 32 codewords, in lanes 0 .. 31 from the end on: a codeword as a number, its first bit highest in a backward run
// and lowest in a forward one, and its length.
__device__ __forceinline__ uint32_t last_bits(uint32_t code, uint32_t len, int lane)
{
    const uint32_t end = wave_incl_scan(lane < 32 ? len : 0u);              // it begins so many bits below the top
    const uint32_t start = end - len;
    uint32_t part = 0;
    if (lane < 32 && start < 32) part = end <= 32 ? code << (32 - end) : code >> (end - 32);
    part = len ? part : 0u;
    return (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan(part), 63);
}

// ---- an encode: three launches and no wait between them ----
// The chunks are dealt to the workgroups in ranges of a few to RANGE_MOST chunks in a row, the same ranges in the first and the last launch:
//   1. range_histogram (each codec's own): the counts of the exponents of each range, a record of A u32 per range, plain stores;
//   2. plan_kernel, one workgroup: the sum of the records, the code, from record and code lengths where each range begins in the stream
//      (into chunk_bit[], for good), the header, which the host gets from there;
//   3. encode_range: a workgroup knows where its range begins, its waves find out from one another in LDS where their chunks do.
// Nothing is shared between workgroups of a launch: no counters, no waits, no atomic operations on device memory.  The records lie where the stream will
// (RECORDS_AT); a range and its record are smaller than what the range has of the blob, and they are used up before the stream is begun.
// Before, the workgroups of the last launch asked one another for their places (a look-back through chunk_bit[], 3 to 5 us for every tile), and
// the host built the code between two launches.
// One range a workgroup as a rule: where chunks that are dear to pack lie together (longer than an image) few workgroups have them all.  BF16 at 128 symbols per lane
// with random bits in an eighth of 4096 x 4096 is the worst of that kind seen, 61 us; 46 at 64 symbols; 80 and 60 with tiles drawn from a counter and a code
// from the host.  More and smaller ranges would even that out and have a record each, which the plan reads through one compute unit (BF16: 3.5 us now).
constexpr uint32_t RANGE_MOST = 256;        // chunks; four per lane where a wave adds up what lies before its chunk

struct Ranges {
    uint64_t chunks, each;                  // every range has `each` chunks, the first `rest` one more
    uint32_t count, rest;
    __device__ __forceinline__ uint64_t begin(uint32_t r) const { return r * each + (r < rest ? r : rest); }
    __device__ __forceinline__ uint32_t size(uint32_t r) const { return (uint32_t)each + (r < rest ? 1u : 0u); }
};

inline Ranges make_ranges(uint64_t chunks, uint32_t cus)
{
    Ranges g;
    g.chunks = chunks;
    const uint64_t rounds = (chunks + (uint64_t)cus * RANGE_MOST - 1) / ((uint64_t)cus * RANGE_MOST);
    g.count = (uint32_t)(chunks < cus ? chunks : cus * rounds);
    g.each = chunks / g.count;
    g.rest = (uint32_t)(chunks % g.count);
    return g;
}

// No codeword over lmax bits: how many bits the i-th lightest of m symbols gets, as len[s[i]].  Package-merge as the CPU encoders have it: a level's
// list is the symbols' coins and the packages of the level below, both in order, a coin before a package of its weight.  Of a level only the coins' places are
// kept: the items taken are the first ones, so the coins among them are the first a coins, and the packages, twice as many items one level down.
// (The CPU's E4M3 encoder asks Huffman's method first and takes its lengths where the cap does not bind.  The two agree in every tie if the one takes a leaf and
// the other a coin first; so does a cap of m - 1, which binds nowhere.)
template <int A> struct CodeShared {
    __attribute__((aligned(16))) uint64_t key[A < 64 ? 64 : A];     // count << 8 | exponent, in the order of the exponents
    uint64_t w[A];
    uint32_t s[A], rank[A < 64 ? 64 : A], m;
};

// What lies in a at the lanes with bit D set changes place with what lies in b at the lanes D below.
template <int D>
__device__ __forceinline__ void exchange(uint32_t &a, uint32_t &b, int lane)
{
    auto dpp = [](uint32_t old, uint32_t v, auto ctrl, auto banks) {
        return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)v, decltype(ctrl)::value, 0xf, decltype(banks)::value, false);
    };
    uint32_t x, y;
    if constexpr (D == 32) {
        const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
        x = r[0], y = r[1];
    } else if constexpr (D == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
        x = r[0], y = r[1];
    } else if constexpr (D == 8 || D == 4) {                // row_shr, row_shl, into the banks of four lanes that change
        x = dpp(a, b, std::integral_constant<int, 0x110 + D>(), std::integral_constant<int, D == 8 ? 0xc : 0xa>());
        y = dpp(b, a, std::integral_constant<int, 0x100 + D>(), std::integral_constant<int, D == 8 ? 0x3 : 0x5>());
    } else {                                                // quad_perm [0 1 0 1], [2 3 2 3]; [0 0 2 2], [1 1 3 3]
        x = dpp(a, b, std::integral_constant<int, D == 2 ? 0x44 : 0xa0>(), std::integral_constant<int, 0xf>());
        y = dpp(b, a, std::integral_constant<int, D == 2 ? 0xee : 0xf5>(), std::integral_constant<int, 0xf>());
        x = lane & D ? x : a;
        y = lane & D ? b : y;
    }
    a = x, b = y;
}
template <int D>
__device__ __forceinline__ void exchange(uint64_t &a, uint64_t &b, int lane)
{
    uint32_t al = (uint32_t)a, ah = (uint32_t)(a >> 32), bl = (uint32_t)b, bh = (uint32_t)(b >> 32);
    exchange<D>(al, bl, lane);
    exchange<D>(ah, bh, lane);
    a = al | (uint64_t)ah << 32;
    b = bl | (uint64_t)bh << 32;
}
template <class T>
__device__ __forceinline__ void in_order(T &a, T &b)
{
    const T x = a < b ? a : b;
    b = a < b ? b : a;
    a = x;
}
// One stage of a merge: items that differ in lane bit D only, put in order.  The bit becomes the register's (a before b), the register's the lane's.
template <int D, int J, class T>
__device__ __forceinline__ void merge_lanes(T (&a)[J], T (&b)[J], int lane)
{
#pragma unroll
    for (int j = 0; j < J; j++) {
        exchange<D>(a[j], b[j], lane);
        in_order(a[j], b[j]);
    }
    if constexpr (D > 1) merge_lanes<D / 2>(a, b, lane);
}

// m <= LANES * J, by one wave, all in registers: items 2 i and 2 i + 1 of a level's list are a[j] and b[j] of lane l, i = j * LANES + l, so that package i is a sum in its
// lane.  The coins lie there in reverse, and coins and packages, both in order, are one bitonic sequence: log2(2 LANES J) stages of minimum and maximum put it
// in order, through which the lowest bit of an item's place comes to be the register's again (merge_lanes).  T: an item is its weight twice, and 1 more if it
// is a package; 32 bits take 15 levels of 2^27 weights.  Where fewer than 64 lanes are enough the others do the same once more.
// What bounds it: one wave's chain of some 8 clocks an instruction.  The plan kernel in a kernel trace, us, with coins and packages looked for in each other's list
// in LDS (up to 64 coins by all waves, five round trips and two barriers a level, more by one wave) / now: 256 x 512 BF16 of 30 exponents 11.3 / 8.6, of 70 39.7 / 11.9,
// of 256 50.6 / 16.6, E5M2 9.6 / 6.9, E4M3 6.0 / 5.4, cap 15 8.6 / 7.2.
template <int A, int LANES, int J, class T>
__device__ __forceinline__ void package_merge(const CodeShared<A> &cs, uint32_t m, uint32_t lmax, uint32_t *len, int lane)
{
    static_assert(LANES * J <= A || A < LANES, "coins");
    constexpr T NONE = (T)~(T)0;
    constexpr uint32_t N = LANES * J;
    const uint32_t l = (uint32_t)lane % LANES;
    if (lmax > m - 1) lmax = m - 1;
    T a[J], b[J], coin[J];
    uint32_t kept[J][4];                                    // lane `level`: which items of the level are coins, of a (64 lanes) and of b
#pragma unroll
    for (int j = 0; j < J; j++) {
        const uint32_t i = j * LANES + l, back = N - 1 - i;
        a[j] = 2 * i < m ? (T)cs.w[2 * i] << 1 : NONE;
        b[j] = 2 * i + 1 < m ? (T)cs.w[2 * i + 1] << 1 : NONE;
        coin[j] = back < m ? (T)cs.w[back] << 1 : NONE;
#pragma unroll
        for (int k = 0; k < 4; k++) kept[j][k] = 0;
    }
    uint32_t n = m;
#pragma unroll 1
    for (uint32_t level = 1; level < lmax; level++) {
        const uint32_t packages = n / 2;
        n = m + packages;
#pragma unroll
        for (int j = 0; j < J; j++) {
            T p = (T)(a[j] & ~(T)1) + (T)(b[j] | (T)1);
            p = j * LANES + l < packages ? p : NONE;
            a[j] = coin[j];
            b[j] = p;
            in_order(a[j], b[j]);
        }
#pragma unroll
        for (int s = J / 2; s >= 1; s /= 2)                 // the stages between registers: what merge_lanes does, without an instruction to exchange
#pragma unroll
            for (int j = 0; j < J; j++) {
                if (j & s) continue;
                in_order(a[j], a[j + s]);
                in_order(b[j], b[j + s]);
                const T t = a[j + s];
                a[j + s] = b[j];
                b[j] = t;
            }
        merge_lanes<LANES / 2>(a, b, lane);
#pragma unroll
        for (int j = 0; j < J; j++) {
            const uint64_t ca = __ballot(!(a[j] & 1)), cb = __ballot(!(b[j] & 1));
            const bool here = lane == (int)level;
            kept[j][0] = here ? (uint32_t)ca : kept[j][0];
            kept[j][1] = here ? (uint32_t)(ca >> 32) : kept[j][1];
            kept[j][2] = here ? (uint32_t)cb : kept[j][2];
            kept[j][3] = here ? (uint32_t)(cb >> 32) : kept[j][3];
        }
    }
    uint32_t bits[J], taken = 2 * m - 2;
#pragma unroll
    for (int j = 0; j < J; j++) bits[j] = 0;
#pragma unroll 1
    for (uint32_t level = lmax; level-- > 0;) {
        uint32_t coins = taken < m ? taken : m;             // the lowest level has no packages
        if (level) {
            coins = 0;
#pragma unroll
            for (int j = 0; j < J; j++)
#pragma unroll
                for (int r = 0; r < 2; r++) {
                    const uint64_t is = (uint32_t)__builtin_amdgcn_readlane((int)kept[j][2 * r], (int)level) |
                                        (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)kept[j][2 * r + 1], (int)level) << 32;
                    const int t = (int)((taken + 1 - r) / 2) - j * LANES;           // so many of a's or b's are taken
                    const uint64_t first = t <= 0 ? 0 : t >= 64 ? ~0ull : (1ull << t) - 1;
                    coins += (uint32_t)__builtin_popcountll(is & first);
                }
        }
#pragma unroll
        for (int j = 0; j < J; j++) bits[j] += j * LANES + l < coins ? 1u : 0u;
        taken = 2 * (taken - coins);
    }
#pragma unroll
    for (int j = 0; j < J; j++)
        if (lane < LANES && j * LANES + l < m) len[cs.s[j * LANES + l]] = m == 1 ? 1u : bits[j];
}
template <int A, class T>
__device__ __forceinline__ void package_merge(const CodeShared<A> &cs, uint32_t m, uint32_t lmax, uint32_t *len, int lane)
{
    if constexpr (A <= 64) package_merge<A, A, 1, T>(cs, m, lmax, len, lane);
    else if (m <= 64) package_merge<A, 64, 1, T>(cs, m, lmax, len, lane);
    else if (m <= 128) package_merge<A, 64, 2, T>(cs, m, lmax, len, lane);
    else package_merge<A, 64, A / 64, T>(cs, m, lmax, len, lane);
}

// The code and everything that follows from it.  C: a codec: A exponents, Header, sign_bytes(), finish() (what the header holds beside the sections' places, and the
// sections between header and chunk_bit[]).  `h` is the header as far as it does not depend on the code; where the blob would not fit, or no code of lmax bits
// has room for the exponents that occur, the header is 0 and the error, and nothing is written behind it but what the container has no use for: the ranges' places in
// chunk_bit[] (if there is a code), and the records, where they lie.
// What bounds it: one compute unit, a chain of barriers and round trips to LDS, while the rest of the chip waits.  In a kernel trace, 256 ranges: E4M3 5.5 us, E5M2 7.1,
// BF16 10.1, of which 3.5 are the 256 KiB of records.  On the host, between two launches, it took 8 us and, for BF16, 18.
template <class C>
__global__ __launch_bounds__(1024) void plan_kernel(typename C::Header h, Ranges rg, uint64_t blob_, uint64_t capacity, uint64_t records, uint32_t lmax, uint64_t mail)
{
    typedef typename C::Header Header;
    constexpr int A = C::A, QUADS = A / 4, SUBSETS = 1024 / QUADS, BATCH = 256, KEEP = BATCH / SUBSETS;
    static_assert(sizeof(Header) == 256 && (QUADS == 4 || QUADS == 8 || QUADS == 64), "64 dwords; sums over quads, eights or waves");
    __shared__ CodeShared<A> cs;
    __shared__ uint64_t s_part[16][A], s_freq[A], s_there[4];
    __shared__ uint32_t s_len[A];
    __shared__ __attribute__((aligned(16))) uint32_t s_bits[BATCH];
    __shared__ __attribute__((aligned(16))) uint32_t s_header[64];
    const int tid = threadIdx.x, lane = tid & 63, wave = (int)uniform32(tid >> 6);
    const uint32_t quad = tid % QUADS, subset = tid / QUADS;
    GLOBAL uint8_t *blob = (GLOBAL uint8_t *)blob_;

    const uint32_t frame = ((const uint32_t *)&h)[lane];
    // a thread has four exponents of every SUBSETS-th range
    u32x4 rec[KEEP];
    auto load = [&](uint32_t r0) {
#pragma unroll
        for (int k = 0; k < KEEP; k++) {
            const uint32_t r = r0 + subset + k * SUBSETS;
            rec[k] = r < rg.count ? ((const GLOBAL u32x4 *)records)[(uint64_t)r * QUADS + quad] : u32x4{0, 0, 0, 0};
        }
    };
    uint64_t sum[4] = {0, 0, 0, 0};
    for (uint32_t r0 = 0; r0 < rg.count; r0 += BATCH) {
        load(r0);
#pragma unroll
        for (int k = 0; k < KEEP; k++) {
            sum[0] += rec[k].x;
            sum[1] += rec[k].y;
            sum[2] += rec[k].z;
            sum[3] += rec[k].w;
        }
    }
    if (wave == 0) s_header[lane] = frame;
    if (tid < (A < 64 ? 64 : A)) {
        cs.rank[tid] = 0;
        cs.key[tid] = ~0ull;
    }
#pragma unroll
    for (int k = 0; k < 4; k++) {
        if constexpr (QUADS < 64) {
            // in two parts whose sums fit 32 bits: 24 bits, and the rest
            uint32_t part[2] = {(uint32_t)sum[k] & 0xffffffu, (uint32_t)(sum[k] >> 24)};
#pragma unroll
            for (int i = 0; i < 2; i++) {
                part[i] = add_dpp<0x128>(part[i]);                          // row_ror:8
                if (QUADS == 4) part[i] = add_dpp<0x124>(part[i]);          // row_ror:4
                part[i] = add_16(part[i], part[i]);
                part[i] = add_32(part[i], part[i]);
            }
            sum[k] = ((uint64_t)part[1] << 24) + part[0];
        }
        if (lane < QUADS) s_part[wave][4 * quad + k] = sum[k];
    }
    __syncthreads();

    // the exponents that occur, and these in order of their counts
    uint64_t f = 0, there = 0;
    if (wave < (A + 63) / 64) {
        if (tid < A) {
#pragma unroll
            for (int w = 0; w < 16; w++) f += s_part[w][tid];
            s_freq[tid] = f;
            s_len[tid] = 0;
        }
        there = __ballot(f != 0);
        if (A > 64 && lane == 0) s_there[wave] = there;
    }
    if (A > 64) __syncthreads();
    if (wave < (A + 63) / 64) {
        uint32_t before = 0, m = 0;
        if constexpr (A > 64) {
#pragma unroll
            for (int w = 0; w < A / 64; w++) {
                const uint32_t in = (uint32_t)__builtin_popcountll(s_there[w]);
                before += w < wave ? in : 0u;
                m += in;
            }
        } else
            m = (uint32_t)__builtin_popcountll(there);
        const uint32_t i = before + (uint32_t)__builtin_popcountll(there & ((1ull << lane) - 1));
        if (f) cs.key[i] = f << 8 | (uint32_t)tid;          // f <= 2^48
        if (tid == 0) cs.m = m;
    }
    __syncthreads();
    // a thread compares one of them with 4 (m <= 64: each wave with others of 4) or 64 (each four waves)
    const uint32_t m = uniform32(cs.m), spread = A <= 64 || m <= 64 ? 6 : 8, mine = tid & ((1u << spread) - 1u);
    const uint64_t key = cs.key[mine];
    const uint32_t others = spread == 6 ? 4 : 64, from = (tid >> spread) * others;
    if (from < m && mine < m) {
        uint32_t before = 0;
        for (uint32_t j = from; j < from + others; j += 4) {
#pragma unroll
            for (uint32_t k = 0; k < 4; k++) before += cs.key[j + k] < key ? 1u : 0u;
        }
        if (before) atomicAdd(&cs.rank[mine], before);
    }
    __syncthreads();
    if (tid == (int)mine && mine < m) {
        const uint32_t r = cs.rank[mine];
        cs.w[r] = key >> 8;
        cs.s[r] = (uint32_t)key & 0xffu;
    }
    __syncthreads();
    const bool code = lmax >= 1 && m <= 1u << lmax;
    if (code && wave == 0) {
        if (h.n_elem < 1ull << 27) package_merge<A, uint32_t>(cs, m, lmax, s_len, lane);
        else package_merge<A, uint64_t>(cs, m, lmax, s_len, lane);
    }
    __syncthreads();

    // where the ranges begin
    GLOBAL uint64_t *cb = (GLOBAL uint64_t *)(blob + h.off_chunk_bit);
    const uint32_t l0 = s_len[4 * quad], l1 = s_len[4 * quad + 1], l2 = s_len[4 * quad + 2], l3 = s_len[4 * quad + 3];
    uint64_t total = 0;
    for (uint32_t r0 = 0; r0 < rg.count; r0 += BATCH) {
        if (rg.count > (uint32_t)BATCH) load(r0);
        uint32_t bits[KEEP];
#pragma unroll
        for (int k = 0; k < KEEP; k++) bits[k] = rec[k].x * l0 + rec[k].y * l1 + rec[k].z * l2 + rec[k].w * l3;      // a range: at most 2^25
        if constexpr (QUADS == 64) {
            // 16 values over a wave: two at a time in its halves, then in its rows
#pragma unroll
            for (int k = 0; k < KEEP / 4; k++) {
                const uint32_t v = add_row(add_16(add_32(bits[4 * k], bits[4 * k + 1]), add_32(bits[4 * k + 2], bits[4 * k + 3])));
                if (lane % 16 == 0) s_bits[subset + (4 * k + (lane >> 5) + (lane >> 4 & 1) * 2) * SUBSETS] = v;
            }
        } else {
#pragma unroll
            for (int k = 0; k < KEEP; k++) {
                const uint32_t v = QUADS == 4 ? add_quad(bits[k]) : add_eight(bits[k]);
                if (quad == 0) s_bits[subset + k * SUBSETS] = v;
            }
        }
        __syncthreads();
        if (wave == 0) {
            const u32x4 v = *(const u32x4 *)(s_bits + 4 * lane);
            const uint32_t own = v.x + v.y + v.z + v.w;
            const uint32_t lo = wave_incl_scan(own & 0xffffu), hi = wave_incl_scan(own >> 16);  // 64 of them may need more than 32 bits
            uint64_t at = total + (((uint64_t)hi << 16) + lo) - own;
            total += ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)hi, 63) << 16) + (uint32_t)__builtin_amdgcn_readlane((int)lo, 63);
            const uint32_t each[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const uint32_t r = r0 + 4 * lane + k;
                if (r < rg.count && code) cb[rg.begin(r)] = at;
                at += each[k];
            }
        }
        if (rg.count > (uint32_t)BATCH) __syncthreads();
    }
    if (wave != 0) return;

    // the header
    Header &out = *(Header *)s_header;
    const ecf8_internal::LayoutEnd e = ecf8_internal::layout_end(h.off_stream, total, h.plane_bytes, C::sign_bytes(h));
    const int err = !code ? ECF8_E_ARG : e.total > capacity ? ECF8_E_CAPACITY : 0;
    if (lane == 0) {
        out.stream_bits = total;
        out.stream_bytes = e.stream_bytes;
        out.off_plane = e.off_plane;
        out.total_size = e.total;
    }
    C::finish(out, blob, e.off_sign, s_freq, s_len, m, s_len[cs.s[0]], err == 0, lane);     // the lightest symbol's codeword is the longest
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (err && lane < 2) s_header[lane] = lane ? (uint32_t)err : 0u;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const uint32_t dword = s_header[lane];
    if (mail) __hip_atomic_store((GLOBAL uint64_t *)mail + lane, 1ull << 32 | dword, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    ((GLOBAL uint32_t *)blob)[lane] = dword;
    if (lane == 0 && !err) cb[rg.chunks] = total;
}

// The header as the kernels behind the plan read it.
template <class Header>
__device__ __forceinline__ const __attribute__((address_space(4))) Header &planned(uint64_t blob) { return *(const __attribute__((address_space(4))) Header *)blob; }

// What the waves of a workgroup tell one another about the chunks of their range.
constexpr int WMAX = 16;                    // waves of a workgroup at the most
struct RangeShared {
    __attribute__((aligned(16))) uint32_t bits[RANGE_MOST];     // of a chunk, 0: not counted yet
    uint64_t border[RANGE_MOST + 1];        // the dword that a chunk shares with the one before: what one of the two has of it, with a 1 above
    uint32_t next;                          // the chunk to be drawn next
};
__device__ __forceinline__ void range_begin(RangeShared &sh)
{
    for (uint32_t i = threadIdx.x; i <= RANGE_MOST; i += blockDim.x) {
        if (i < RANGE_MOST) sh.bits[i] = 0;
        sh.border[i] = 0;
    }
    if (threadIdx.x == 0) sh.next = blockDim.x >> 6;
}

typedef uint32_t u32x4a __attribute__((ext_vector_type(4), aligned(4)));

// The chunks of a workgroup's range, drawn in order from an LDS counter, a wave's first one by its number (already fetched, if it is whole).  K is a codec's chunk.
// For chunks that lie entirely inside the tensor, fetch(c) asks for the weights, count(c) gives the lane's code bits and writes the planes, pack(image, at,
// c, next, refill) packs the lane's bits from image bit `at` on and asks for the weights of chunk `next` piece by piece as its own are used up.  slow_count and
// slow_pack do the same for any chunk, from memory and rolled up: the code of the common way has to stay well inside the instruction
// cache.  tail(c): the last 32 bits of chunk c.  `image` is the wave's, K::AREA dwords.
// A chunk's place is the sum of the bits of the chunks before it in the range, which are counted by the time this one is packed: a wave counts before it
// packs and waits for chunks before its own only, so every wait ends.  The dword where two chunks meet is put together in LDS and stored by
// whoever comes second.
template <class K>
__device__ __forceinline__ void encode_range(K &k, RangeShared &sh, uint32_t *image, const Ranges &rg, GLOBAL uint8_t *blob, uint64_t off_cb, uint64_t off_lb,
                                             uint64_t off_st, uint64_t stream_dwords, int lane, int wave)
{
    constexpr uint32_t ROOM = (uint32_t)(K::AREA - 4) * 32;     // bits an image takes
    GLOBAL uint64_t *cb = (GLOBAL uint64_t *)(blob + off_cb);
    GLOBAL uint16_t *lane_bits = (GLOBAL uint16_t *)(blob + off_lb);
    GLOBAL uint32_t *stream = (GLOBAL uint32_t *)(blob + off_st);
    const uint64_t first = rg.begin(blockIdx.x), begin = uniform64(cb[first]);
    const uint32_t size = rg.size(blockIdx.x), W = blockDim.x >> 6;
    auto fence = [] { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); };
    auto border = [&](uint32_t i, uint32_t part, uint64_t at) {
        const uint64_t other = atomicOr((unsigned long long *)&sh.border[i], 1ull << 32 | part);
        if (other >> 32) stream[at] = part | (uint32_t)other;
    };
    for (uint32_t u = lane; u * 4 < (uint32_t)K::AREA; u += 64) *(u32x4 *)(image + 4 * u) = u32x4{0, 0, 0, 0};
    if (wave + 1 == (int)W && begin & 31) {                     // what the range before has of the first dword
        const uint32_t last = k.tail(first - 1) >> (32 - (begin & 31));
        if (lane == 0 && begin >> 5 < stream_dwords) border(0, last, begin >> 5);
    }
    for (uint32_t i = wave; i < size;) {
        const uint64_t c = first + i;
        uint32_t drawn = 0;
        if (lane == 0) drawn = atomicAdd(&sh.next, 1u);
        const bool whole = k.whole(c);
        uint32_t lb;
        if (whole) lb = k.count(c);
        else {
            lb = k.slow_count(c);
            __builtin_amdgcn_s_waitcnt(0x0f70);                 // vmcnt(0): nothing is on its way, which the compiler does not see; in pack it would wait for count's stores
        }
        const uint32_t incl = wave_incl_scan(lb), sum = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        const uint32_t bits = sum ? sum : 1u;                   // weights that change under the call may have no codes: garbage, but every wait ends
        if (lane == 0) __hip_atomic_store(&sh.bits[i], bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        lane_bits[c * 64 + lane] = (uint16_t)lb;
        const uint32_t next = uniform32(drawn);
        const bool fits = bits <= ROOM, more = next < size && k.whole(first + next), refill = more && fits && whole;
        fence();
        if (fits && whole) k.pack(image, incl - lb, c, first + next, refill);
        else if (fits) k.slow_pack(image, incl - lb, c);
        fence();
        uint32_t before;
        for (;;) {
            const u32x4 e = *(volatile u32x4 *)(sh.bits + 4 * lane);
            const uint32_t j = 4 * lane;
            const uint32_t v0 = j < i ? e.x : 0u, v1 = j + 1 < i ? e.y : 0u, v2 = j + 2 < i ? e.z : 0u, v3 = j + 3 < i ? e.w : 0u;
            if (!__ballot((j < i && !v0) || (j + 1 < i && !v1) || (j + 2 < i && !v2) || (j + 3 < i && !v3))) {
                before = (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan(v0 + v1 + v2 + v3), 63);
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
        uint64_t b0 = begin + before;
        if (lane == 0 && i) cb[c] = b0;
        // A chunk that an image does not take goes out by half its lanes at a time, whose bits fit whatever they are.
        const uint32_t half = (uint32_t)__builtin_amdgcn_readlane((int)incl, 31);
        uint32_t lead = 0;                                      // second half: what the first one has of its first dword
#pragma unroll 1
        for (int part = 0; part < (fits ? 1 : 2); part++) {
            const uint32_t from = part ? half : 0u, here = fits ? bits : part ? bits - half : half;
            if (!fits && (lane >> 5) == part) k.slow_pack(image, incl - lb - from, c);
            fence();
            const bool last = fits || part, end = last && c + 1 == rg.chunks;
            const uint32_t shift = (uint32_t)b0 & 31, over = (uint32_t)(b0 + here) & 31, n = (uint32_t)(((b0 + here) >> 5) - (b0 >> 5));
            const bool shared = shift && !part;                 // the first dword, with the chunk before
            const uint64_t d0 = b0 >> 5, left = d0 < stream_dwords ? stream_dwords - d0 : 0;     // changing weights again: not past the section
            const uint32_t full = n < left ? n : (uint32_t)left;
            GLOBAL uint32_t *out = stream + d0;
            uint32_t carry = 0, head = 0, tail = 0;
            for (uint32_t j0 = 0; j0 < n + 1; j0 += 256) {
                const uint32_t j = j0 + 4 * lane;
                u32x4 w = {0, 0, 0, 0};
                if (j <= n) {
                    w = *(const u32x4 *)(image + j);
                    *(u32x4 *)(image + j) = u32x4{0, 0, 0, 0};
                }
                const uint32_t below = (uint32_t)__builtin_amdgcn_update_dpp((int)carry, (int)w.w, 0x138, 0xf, 0xf, false);     // wave_shr:1
                carry = (uint32_t)__builtin_amdgcn_readlane((int)w.w, 63);
                u32x4a v = {w.x, w.y, w.z, w.w};
                if (shift)
                    v = u32x4a{__builtin_amdgcn_alignbit(w.x, below, 32 - shift), __builtin_amdgcn_alignbit(w.y, w.x, 32 - shift),
                               __builtin_amdgcn_alignbit(w.z, w.y, 32 - shift), __builtin_amdgcn_alignbit(w.w, w.z, 32 - shift)};
                if (j == 0) v.x |= lead;
                if (j0 == 0) head = v.x;
                if (j + 4 <= full && (j || !shared)) {
                    *(GLOBAL u32x4a *)(out + j) = v;
                } else {
                    if (j < full && (j || !shared)) out[j] = v.x;
                    if (j + 1 < full) out[j + 1] = v.y;
                    if (j + 2 < full) out[j + 2] = v.z;
                    if (j + 3 < full) out[j + 3] = v.w;
                }
                const uint32_t t = n & 2 ? (n & 1 ? v.w : v.z) : n & 1 ? v.y : v.x;
                tail = (uint32_t)__builtin_amdgcn_readlane((int)t, (int)(n >> 2) & 63);
            }
            lead = over ? tail : 0u;
            if (lane == 0) {
                if (shared && left) border(i, head, d0);
                if (last && over && n < left && (n || !shared)) {
                    if (end) out[n] = tail;
                    else border(i + 1, tail, d0 + n);
                }
            }
            fence();
            b0 += here;
        }
        if (more && !refill) k.fetch(first + next);
        i = next;
    }
}

// Waves of a workgroup: no more than its range has chunks, as far as the tables are set up faster by more.
inline uint32_t range_waves(const Ranges &g)
{
    const uint64_t most = g.each + (g.rest ? 1 : 0);
    return most <= 4 ? 4u : most <= 8 ? 8u : (uint32_t)WMAX;
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

// The encoders' one synchronisation: the header on its way to the host, on a page of pinned host memory.  A word of it is a dword of the header with a 1 above, so that
// the host takes each as it comes and nothing has to be ordered.  (A copy behind the kernel and the call that waits for it took some 5 us longer.)
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
        if (page)
            for (int i = 0; i < 64; i++) __atomic_store_n(page + i, 0ull, i < 63 ? __ATOMIC_RELAXED : __ATOMIC_RELEASE);
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
    // for the kernel; 0: there is no page, and the header has to be copied
    uint64_t device()
    {
        quiet = !page;
        return page ? (uint64_t)(uintptr_t)seen : 0;
    }
    // The header, of the plan kernel that was given device(), dword by dword as they come; without a page, from the blob, by a copy that waits for all that is
    // queued on s.
    bool read(void *header, uint64_t blob, hipStream_t s)
    {
        if (!page) {
            if (hipMemcpyWithStream(header, (const void *)(uintptr_t)blob, 256, hipMemcpyDeviceToHost, s) == hipSuccess) return true;
            (void)hipGetLastError();
            return false;
        }
        const auto since = std::chrono::steady_clock::now();
        bool done = false;
        int got = 0;
        for (uint32_t i = 1; got < 64; i++) {
            const uint64_t v = __atomic_load_n(page + got, __ATOMIC_ACQUIRE);
            if (v >> 32) {
                ((uint32_t *)header)[got++] = (uint32_t)v;
                continue;
            }
            if (done) return false;
            __builtin_ia32_pause();
            // the stream has more to do, or it has failed
            if (i % 256 == 0 && std::chrono::steady_clock::now() - since > std::chrono::milliseconds(1)) {
                done = hipStreamSynchronize(s) == hipSuccess;
                if (!done) {
                    (void)hipGetLastError();
                    return false;
                }
            }
        }
        quiet = true;
        return true;
    }
};

// Whether the launch just made went through.  Asked after each of an encode's three: what a kernel takes from the blob, places to store at among it, is the kernel's
// before it, and behind a launch that failed it would be whatever the caller's buffer holds.
inline bool launched() { return hipGetLastError() == hipSuccess; }

// A stream that is being captured runs nothing: there is no header to wait for.  Nor is there on the null stream while one that waits for it is
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
