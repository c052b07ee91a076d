// ECF8 -> FP8 decode kernels for gfx950 (MI355X), wave64.
//
// What is computed is Algorithm 1 of the paper (block-level decompression:
// load the compressed span, locate each lane's first codeword, decode through
// a lookup table held next to the ALUs, merge the sign/mantissa nibble, write
// back coalesced).  How it is computed is specific to CDNA4:
//
//  * one wavefront decodes one chunk = 64 lanes x N elements; the encoder
//    recorded how many stream bits each lane's N codewords take, so a DPP
//    prefix scan over those 64 numbers gives every lane its start bit, and
//    output positions are fixed by construction (lane l owns the 16-byte
//    pieces l, l+64, ... of the chunk).  The paper's first decoding pass,
//    which exists only to count symbols per thread, is gone;
//  * the chunk's span of the stream is copied to LDS with dwordx4 loads, 1 KiB
//    contiguous per wave instruction; lanes pull aligned 64-bit windows from
//    LDS (unaligned LDS accesses serialise per lane on this chip, so every LDS
//    access here is naturally aligned);
//  * the code table is a 2^TB-entry LDS table of 16-bit entries indexed by the
//    next TB stream bits; one lookup yields TWO symbols, already shifted to
//    their place in the output bytes, and the bits they consume.  A lane
//    always decodes four symbols (two lookups) per step, so every lane of the
//    wave runs the same number of steps, nothing diverges, and each step ends
//    with one finished output dword in a register.  A lane's bits hold two runs,
//    one read forward from its first bit and one read backward from its last
//    bit, so every lane advances two independent dependency chains at once
//    (twice the LDS latency hidden per wave).  Pairs that do not fit in TB bits and
//    codewords longer than TB bits take a second level (per-symbol walk that
//    reuses the table's first-symbol fields, then a 16-entry canonical match);
//    a wave holds 256 pairs per step, so even a 1e-3 miss rate sends a third of
//    the steps there.  Under the encoder's default cap of TB/2 bits per codeword
//    every pair is a table hit and the PAIRFIT kernels carry no second level.
//    The 32 KiB table is copied from the blob when the encoder embedded it (one
//    L2-resident read per workgroup), else built in LDS from the 16 code lengths;
//  * after four steps a lane holds one 16-byte piece; the 64 lanes' pieces are
//    adjacent, so each dwordx4 store instruction of the wave writes 1 KiB of
//    contiguous output, merged in registers with the nibble plane that was
//    fetched (coalesced, 512 B per instruction) a whole chunk earlier.  Decoded
//    bytes never pass through LDS.  The PAIRFIT kernels hold a chunk's pieces
//    and store them in one burst; with the container's group interleave (a
//    wave's consecutive pieces G KiB apart, the workgroup's other waves in
//    between) HBM takes such bursts about 15 % faster than 1 KiB stores
//    trickling out of every wave;
//  * persistent workgroups own contiguous chunk ranges, so a table is set up
//    once per (workgroup, tensor); inside a workgroup the waves draw chunks
//    from an LDS ticket counter (the hardware favours a SIMD's oldest wave, so
//    equal static shares would finish up to 50 % apart).  No global atomics.
#include "ecf8_device.h"

#include <cstddef>
#include <type_traits>

namespace {

// Stream, plane and output are touched exactly once: nontemporal accesses keep them from
// displacing the table and the metadata in L2.
#define LD_STREAM(p) __builtin_nontemporal_load(p)
#define ST_STREAM(v, p) __builtin_nontemporal_store((v), (p))

struct KArgs {
    ecf8_batch_item single;               // used when items == nullptr
    const GLOBAL ecf8_batch_item *items;  // device array for the batched call
    uint32_t n_items;
    uint64_t total_chunks;                // of the launch, at most LAUNCH_CHUNKS
    uint32_t max_code_len;                // longest codeword of any tensor of the launch
    uint32_t max_workgroups;              // 0 = one per compute unit
    uint32_t row_tiled;                   // every tensor of the launch is in the row-tiled layout
    ChunkDeal deal;                       // of the launch's chunks to its workgroups
    uint64_t base;                        // FAR kernels: chunks of the batch before the launch's
};

template <int N, int WAVES, bool PAIRFIT, bool TILED = false>
struct Cfg {
    // bytes of stream staged per chunk: under the cap of TB/2 bits per codeword the worst case
    // (so no chunk of a PAIRFIT launch is ever oversize), else a good 4 bits per symbol
    static constexpr int STAGE = PAIRFIT ? 64 * N * (TB / 2) / 8 + 64 : N * 32 + 64;
    static constexpr int PIECES = N / 16;             // 16-byte output pieces per lane
    static constexpr int SEGS = (STAGE / 16 + 63) / 64;  // dwordx4 loads per lane that cover STAGE
    // LDS map (byte offsets into one array)
    static constexpr int OFF_TBL = 0;
    static constexpr int OFF_SYM = OFF_TBL + TBL_ENTRIES * 2;  // s_len[16], s_code[16]
    static constexpr int OFF_CTL = OFF_SYM + 128;              // ticket counter, oversize count, oversize list
    static constexpr int LIST_MAX = 60;                        // oversize chunks remembered per (workgroup, tensor)
    static constexpr int OFF_WAVES = OFF_CTL + 16 + 4 * LIST_MAX;
    // After the pipelined loop the waves' stages together serve as a few wide slots, each large
    // enough for the longest span any code can produce (15 bits per symbol), for the chunks whose
    // span did not fit a stage.
    static constexpr int SLOT = 64 * N * 15 / 8 + 64;
    static constexpr int SLOTS = (WAVES * STAGE / SLOT) < WAVES ? (WAVES * STAGE / SLOT) : WAVES;
    static_assert(PAIRFIT || SLOTS >= 1, "wide slots must fit the stage area");
    static_assert(OFF_WAVES % 16 == 0 && SLOT % 16 == 0, "16-byte LDS stores");
    static constexpr int WAVES_BYTES = WAVES * STAGE > TBL_ENTRIES * 2 ? WAVES * STAGE : TBL_ENTRIES * 2;
    // TILED: a 16 x 256-byte tile per wave in which a decoded chunk of a row-tiled blob is turned from the
    // lanes' pieces (16 bytes of row l % 16 each) into whole 256-byte row segments before it is stored
    static constexpr int OFF_TILE = OFF_WAVES + WAVES_BYTES;  // table-build scratch aliases the stages
    static constexpr int TILE_BYTES = 16 * 4 * N;
    static_assert(!TILED || (PAIRFIT && N == 64), "the tile turn is built for the fused GEMM's layout");
    // The decode steps read one dword past a window's two, and a lane of a ragged last chunk reads up to N / 2 codewords
    // past its bits (under the cap still inside the worst-case stage): the last stage is followed by a pad.
    static constexpr int TOTAL = OFF_TILE + (TILED ? WAVES * TILE_BYTES : 0) + (PAIRFIT ? 16 : (N / 2 * 15 / 8 + 15) / 16 * 16 + 32);
    static_assert(TOTAL <= 160 * 1024, "LDS of one gfx950 CU");
};

// PAIRFIT: every tensor of the launch has codewords of at most TB/2 bits (the encoder's
// default cap), so the pipelined loop needs no second level and is one straight line.
// LONG (general kernels only): some codeword of the launch is longer than TB bits.  BURST: 1 = a chunk's pieces are
// held in registers and stored together at its end, 2 = half the chunk's pieces at a time, 0 = each piece as it is decoded.
// CODES: ShortCodes for one tensor under the cap whose blob holds no table, else TableInBlob: as the tensors have it.
// FAR: one of several launches on a batch (a general kernel, whatever the codes).  The others have no scalar registers to spare: with a base of 0 in all kernels
// 4096 x 5120 took 10.9 us in place of 10.7, a layer of E5M2 85.4 in place of 84.9.
template <int N, int WAVES, bool PAIRFIT, bool TILED, bool LONG, int BURST, class CODES, bool FAR = false>
__global__ __launch_bounds__(WAVES * 64) void ecf8_decode_kernel(KArgs a, CODES codes)
{
    constexpr bool SHORT = std::is_same<CODES, ShortCodes>::value;
    using C = Cfg<N, WAVES, PAIRFIT, TILED>;
    __shared__ __attribute__((aligned(16))) uint8_t smem[C::TOTAL];
    uint16_t *tbl = (uint16_t *)(smem + C::OFF_TBL);
    uint32_t *s_len = (uint32_t *)(smem + C::OFF_SYM);
    uint32_t *s_code = s_len + 16;
    uint32_t *s_ticket = (uint32_t *)(smem + C::OFF_CTL);
    uint32_t *s_oversize = s_ticket + 1;                  // number of oversize chunks met in the loop
    uint32_t *s_tail = s_ticket + 2;                      // set: the ragged last chunk is left to the symbol pass
    uint32_t *s_list = s_ticket + 4;                      // their chunk numbers, relative to c

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = (int)uniform32((uint32_t)tid >> 6);         // the same for every lane: chunk numbers and addresses stay in scalar registers
    const uint32_t stage_off = C::OFF_WAVES + wave * C::STAGE;   // byte offset into smem
    uint8_t *stage = smem + stage_off;

    // Chunk numbers have 32 bits and count from the launch's first chunk.  FAR: of a tensor that begins before it, first_chunk is below 0, and wraps.
    const uint64_t base = FAR ? a.base : 0;
    const uint32_t c0 = a.deal.begin(blockIdx.x), c_past = a.deal.begin(blockIdx.x + 1), c_all = (uint32_t)a.total_chunks;
    const uint32_t c_end = c_past < c_all ? c_past : c_all;
    uint32_t c = c0;
    while (c < c_end) {
        // which tensor holds chunk c (uniform)
        uint32_t n_chunks, first_chunk;
        uint64_t d_blob, d_out, n_elem, off_cb, off_lb, off_st, off_pl, st_bytes;
        uint64_t len_lo, len_hi, off_tbl, group, tcols;
        if (!SHORT && a.items) {
            const BatchItem item(a.items, a.n_items, base + c, lane);
            auto field = [&](int k) -> uint64_t { return item.word(k); };
            static_assert(sizeof(ecf8_batch_item) == 128 && offsetof(ecf8_batch_item, code_len) == 80 &&
                          offsetof(ecf8_batch_item, tile_cols) == 112, "field numbers below");
            d_blob = field(0); d_out = field(1); n_elem = field(2); n_chunks = (uint32_t)field(3); first_chunk = (uint32_t)(field(4) - base);
            off_cb = field(5); off_lb = field(6); off_st = field(7); off_pl = field(8); st_bytes = field(9);
            len_lo = field(10); len_hi = field(11); off_tbl = field(12); group = field(13); tcols = field(14);
            if (FAR && (field(4) + field(3) - base) >> 32) break;      // the table ends before the launch begins
        } else {
            d_blob = a.single.d_blob; d_out = a.single.d_out; n_elem = a.single.n_elem;
            n_chunks = (uint32_t)a.single.n_chunks; first_chunk = 0; off_cb = a.single.off_chunk_bit;
            off_lb = a.single.off_lane_bits; off_st = a.single.off_stream; off_pl = a.single.off_plane;
            st_bytes = a.single.stream_bytes;
            off_tbl = a.single.off_table; group = a.single.group_chunks; tcols = a.single.tile_cols;
            __builtin_memcpy(&len_lo, a.single.code_len, 8);
            __builtin_memcpy(&len_hi, a.single.code_len + 8, 8);
        }
        const uint32_t t_end = first_chunk + n_chunks;
        const uint32_t seg_end = c_end < t_end ? c_end : t_end;
        if (seg_end <= c) break; // item table does not cover chunk c: stop rather than spin
        GLOBAL uint8_t *out = (GLOBAL uint8_t *)d_out;
        const GLOBAL uint64_t *chunk_bit = (const GLOBAL uint64_t *)(d_blob + off_cb);
        const GLOBAL uint16_t *lane_bits = (const GLOBAL uint16_t *)(d_blob + off_lb);
        const GLOBAL uint8_t *stream = (const GLOBAL uint8_t *)(d_blob + off_st);
        const GLOBAL uint8_t *plane = (const GLOBAL uint8_t *)(d_blob + off_pl);
        // Element layout: chunk cl's piece q of lane l starts at element
        // base + q*stride + l*16.  Chunks of whole groups of `group` chunks are interleaved
        // KiB by KiB (a wave's consecutive pieces lie group KiB apart, the other waves of
        // the workgroup fill the gaps: HBM serves that markedly faster than a wave
        // walking 1 KiB steps); the rest of the tensor is chunk-major.
        // Row-tiled layout (tcols != 0): chunk cl is the block of 16 rows x 4N columns number cl
        // of a tcols-wide matrix, lane l works on row l % 16, its piece q on columns
        // 64 q + 16 (l / 16) of the block.  lane_off is the lane's share of all of this.
        if (group == 0) group = 1;
        const uint32_t g32 = (uint32_t)group, grouped = (uint32_t)(n_elem / (64ull * N)) & ~(g32 - 1);   // chunks in whole groups (group is a power of two)
        const uint64_t blocks_per_row = tcols ? tcols / (4ull * N) : 1;             // a shift
        // Row-tiled: chunk number -> (block of rows, block of columns) is a division by blocks_per_row, which the
        // hardware does not have: a 64-bit one takes more instructions than the decode of a chunk.  Chunk numbers
        // and blocks_per_row fit 32 bits (n_elem <= 2^40, checked by the encoder), so the division is a
        // multiplication by a reciprocal worked out once per tensor (Granlund and Montgomery's round-up method:
        // q = (t + ((n - t) >> sh1)) >> sh2 with t = mulhi(n, mul), exact for every 32-bit n).
        const uint32_t bpr32 = (uint32_t)blocks_per_row;
        uint32_t dv_l = 0, dv_mul = 1;
        if (TILED || tcols) {
            while (dv_l < 32 && (1ull << dv_l) < bpr32) dv_l++;
            dv_mul = (uint32_t)((((1ull << dv_l) - bpr32) << 32) / bpr32 + 1);
        }
        const uint32_t dv_sh1 = dv_l < 1 ? dv_l : 1, dv_sh2 = dv_l > 1 ? dv_l - 1 : 0;
        auto chunk_base = [&](uint32_t cl) -> uint64_t {
            if (tcols) {
                const uint32_t t = __umulhi(cl, dv_mul);
                const uint32_t rb = (t + ((cl - t) >> dv_sh1)) >> dv_sh2;
                return (uint64_t)rb * 16 * tcols + (cl - rb * bpr32) * (4ull * N);
            }
            const uint32_t w = cl < grouped ? cl & (g32 - 1) : 0u;
            return (cl - w) * (64ull * N) + w * 1024;
        };
        // What a lane stores (and the nibbles it merges): piece q at chunk_base + lane_off + q * chunk_stride.  That is where the
        // lane's symbols are, except in the TILED kernel, whose decoded exponents change lanes first: there a lane
        // holds 16 columns of row 4 q + l / 16 of the block.
        typedef typename std::conditional<TILED, uint64_t, uint32_t>::type stride_t;
        auto chunk_stride = [&](uint32_t cl) -> stride_t {
            if constexpr (TILED) return 4 * tcols;
            return tcols ? 64u : cl < grouped ? g32 * 1024u : 1024u;
        };
        const uint64_t symbol_off = tcols ? (uint64_t)(lane & 15) * tcols + (uint64_t)(lane >> 4) * 16 : (uint64_t)lane * 16;
        const uint64_t lane_off = TILED ? (uint64_t)(lane >> 4) * tcols + (uint64_t)(lane & 15) * 16 : symbol_off;

        __syncthreads(); // every wave is done with the previous tensor's table and its scratch
        // the first two chunks of a wave are fixed (c + wave, c + WAVES + wave); later ones are drawn
        if (tid == 0) { *s_ticket = 2 * WAVES; *s_oversize = 0; *s_tail = 0; }

        // Per-wave software pipeline over its chunks cg = c + wave, + WAVES, ...:
        // metadata is loaded two chunks ahead, stream span and nibble plane one chunk
        // ahead (into registers), so HBM latency is covered by the decode of the
        // chunk in hand.
        struct Meta { uint64_t b0, b1; uint32_t lb; };
        auto load_meta = [&](uint32_t cl) {
            Meta m;
            const GLOBAL uint64_t *cb = chunk_bit + cl;
            m.b0 = cb[0];
            m.b1 = cb[1];
            m.lb = (lane_bits + (uint64_t)cl * 64)[lane];
            return m;
        };
        // span of the stream a chunk needs: 16-byte aligned start, 8 bytes of look-ahead.  The chunk's two
        // start bits are the same in every lane, so the arithmetic is done once, in scalar registers.
        auto span_of = [&](const Meta &m, uint64_t &byte0) {
            const uint64_t b0 = uniform64(m.b0), b1 = uniform64(m.b1);
            uint64_t byte_end = ((b1 + 7) >> 3) + 8;
            if (byte_end > st_bytes) byte_end = st_bytes;
            byte0 = (b0 >> 3) & ~15ull;
            if (byte0 > byte_end) byte0 = byte_end;
            return byte_end - byte0;
        };
        // The span's 16-byte units into `seg` (unit lane + 64 k into seg[k]).  Units beyond the span keep what
        // they held, and so does all of `seg` when the span does not fit a stage: no codeword of a chunk that the
        // loop decodes for good reaches into them.
        const uint32_t lane16 = (uint32_t)lane * 16;
        auto load_stream = [&](const Meta &m, u32x4 (&seg)[C::SEGS]) {
            uint64_t byte0;
            const uint64_t span64 = span_of(m, byte0);
            const uint32_t span = span64 <= (uint64_t)C::STAGE ? (uint32_t)span64 : 0u;
            const GLOBAL uint8_t *sp = stream + byte0;
#pragma unroll
            for (int k = 0; k < C::SEGS; k++) {
                const uint32_t i = lane16 + 1024 * k;
                if (i < span) seg[k] = LD_STREAM((const GLOBAL u32x4 *)(sp + i));
            }
        };
        // nibble plane of chunk cl: this lane's piece j at plane_of(cl) + j * (chunk_stride(cl) / 2)
        auto plane_of = [&](uint32_t cl) -> const GLOBAL uint8_t * { return plane + chunk_base(cl) / 2 + lane_off / 2; };

        // The pipelined loop takes only chunks that are entirely inside the tensor, so its
        // stores are unconditional: between the issue of a prefetch and its use every path
        // holds the same stores, and the wait for the prefetch never drains them.  A chunk
        // whose span does not fit the stage is decoded from stale LDS there (harmless garbage,
        // in bounds) and redone by the generic pass below.
        const bool ragged_tail = !TILED && (n_elem % (64ull * N)) != 0;     // row-tiled blobs are whole chunks
        const uint32_t fast_end = (ragged_tail && seg_end == t_end) ? seg_end - 1 : seg_end;
        // next chunk of this workgroup's range, drawn from the LDS ticket counter (wave-uniform)
        auto draw = [&]() -> uint32_t {
            uint32_t t = 0;
            if (lane == 0) t = __hip_atomic_fetch_add(s_ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            return c + uniform32(t);
        };

        // Start-up: the first chunks' metadata and the first chunk's nibbles, whose places are known, are asked for first, then the table; the
        // chunk's stream as soon as the metadata is there; and all of it is in flight before the table is written to LDS, so a workgroup pays
        // about two HBM round trips, not four, before its first decode step.
        uint32_t cg = c + wave;
        uint32_t cg1 = cg + WAVES;
        uint32_t cg2 = fast_end;    // drawn when cg1 is taken up
        Meta m_cur{0, 0, 0}, m_next{0, 0, 0};
        u32x4 seg[C::SEGS];
        u32x2 pl[C::PIECES];
#pragma unroll
        for (int k = 0; k < C::SEGS; k++) seg[k] = u32x4{0, 0, 0, 0};
#pragma unroll
        for (int j = 0; j < C::PIECES; j++) pl[j] = u32x2{0, 0};
        // The ragged last chunk of a tensor goes first, to the wave it would fall to in turn: decoded like any other,
        // its stores cut at the tensor's end.  (Read symbol by symbol from HBM after the loop it was a chain of N
        // round trips at the end of every such launch: 2047 x 2049 weights 55.7 -> 11.1 us, 8 x 256 22.8 -> 9.1 us.)
        // Not inside the loop: a store under a condition there would make the wait for a prefetch drain the stores.
        const bool tail_here = fast_end != seg_end && (uint32_t)wave == (seg_end - 1 - c) % WAVES;
        auto ask_first = [&](uint32_t ck) {
            m_cur = load_meta(ck - first_chunk);
            m_next = load_meta((cg1 < fast_end ? cg1 : ck) - first_chunk);      // a copy of m_cur would wait for it
            const GLOBAL uint8_t *pp = plane_of(ck - first_chunk);
            const stride_t pstride = chunk_stride(ck - first_chunk) / 2;
#pragma unroll
            for (int j = 0; j < C::PIECES; j++) pl[j] = LD_STREAM((const GLOBAL u32x2 *)(pp + j * pstride));
        };
        const bool any = tail_here || cg < fast_end;
        if (any) ask_first(tail_here ? seg_end - 1 : cg);
        u32x4 tv[(TBL_ENTRIES * 2 / 16 + WAVES * 64 - 1) / (WAVES * 64)];
        uint32_t two = 0;
        if constexpr (SHORT) {
            if (wave == 0) two = codes.two[lane];
        } else if (off_tbl) {
            // the encoder embedded the table: copy it (L2-resident after the first workgroup)
            const GLOBAL u32x4 *src = (const GLOBAL u32x4 *)(d_blob + off_tbl);
#pragma unroll
            for (int j = 0; j < (int)(sizeof(tv) / sizeof(tv[0])); j++) {
                const int i = tid + j * WAVES * 64;
                tv[j] = u32x4{0, 0, 0, 0};
                if (i < TBL_ENTRIES * 2 / 16) tv[j] = src[i];
            }
        }
        if (any) load_stream(m_cur, seg);
        if constexpr (SHORT) {
            build_pair_table<WAVES>(two, tbl, (uint32_t *)(smem + C::OFF_WAVES), lane, wave);
        } else if (off_tbl) {
#pragma unroll
            for (int j = 0; j < (int)(sizeof(tv) / sizeof(tv[0])); j++) {
                const int i = tid + j * WAVES * 64;
                if (i < TBL_ENTRIES * 2 / 16) ((u32x4 *)tbl)[i] = tv[j];
            }
            if constexpr (!PAIRFIT) build_symbol_arrays(len_lo, len_hi, s_len, s_code, tid);
            __syncthreads();
        } else if constexpr (PAIRFIT) {
            // not where the blob has the table: building it then keeps the waves from their first chunk for 3 us longer
            // than the copy does (a layer of seven matrices, 80.6 -> 83.8 us)
            build_pair_table<WAVES>(len_lo, len_hi, tbl, (uint32_t *)(smem + C::OFF_WAVES), lane, wave);
        } else {
            build_tables<WAVES * 64>(len_lo, len_hi, tbl, s_len, s_code, (uint16_t *)(smem + C::OFF_WAVES), tid);
        }

        // Decode of one full chunk whose span sits in LDS from bit `first_bit` (smem-relative) on,
        // merge with the nibble plane, stores.  With `reload` set, each piece of the nibble plane gives its
        // registers, once merged, to the same piece of the chunk whose plane starts at next_pl.  With `cut` set the
        // chunk is a ragged last one: its stores end where the tensor does.
        auto decode_store = [&](auto reload, auto cut, uint32_t first_bit, uint32_t lb, u32x2 (&pl)[C::PIECES], GLOBAL uint8_t *out_c,
                                stride_t ostride, const GLOBAL uint8_t *next_pl, stride_t next_pstride) {
            constexpr bool RELOAD = decltype(reload)::value, CUT = decltype(cut)::value;
            auto store_cut = [&](u32x4 v, uint32_t at) {
                const uint64_t el = (uint64_t)(out_c - out) + at;
                if (el + 16 <= n_elem) {
                    ST_STREAM(v, (GLOBAL u32x4 *)(out_c + at));
                    return;
                }
#pragma unroll 1
                for (uint64_t e = el; e < n_elem; e++) {
                    out[e] = (uint8_t)v.x;
                    v.x = __builtin_amdgcn_alignbit(v.y, v.x, 8);
                    v.y = __builtin_amdgcn_alignbit(v.z, v.y, 8);
                    v.z = __builtin_amdgcn_alignbit(v.w, v.z, 8);
                    v.w >>= 8;
                }
            };
            // LDS bit addresses, kept one bit off as quad_step2 wants them: bpA = the forward
            // run's next codeword - 1; bpB = one past the backward run's next codeword - 31
            uint32_t bpA = first_bit - 1;
            uint32_t bpB = bpA + lb - 30;
            HeldRuns runs;                 // PAIRFIT: the runs' windows stay in registers
            if constexpr (PAIRFIT) runs.begin(smem, bpA, bpB);
            // BURST: the chunk's pieces (or half of them) are kept in registers and stored
            // together.  With the interleaved layout the workgroup's waves then write runs of
            // adjacent KiBs close in time, which HBM takes ~15 % faster than single KiBs
            // trickling out of every wave as they are decoded.  The general kernels have the
            // registers for a full burst at N = 64 and for half bursts at N = 128.
            u32x4 ov[BURST == 1 ? C::PIECES : BURST == 2 ? 4 : 1];
#pragma unroll
            for (int Q = 0; Q < C::PIECES / 2; Q++) {
                uint32_t dwA[4], dwB[4];
#pragma unroll
                for (int t = 0; t < 4; t++) {
                    if constexpr (PAIRFIT) quad_step_held(smem, tbl, runs, dwA[t], dwB[t]);
                    else quad_step2<PAIRFIT, LONG>(smem, tbl, s_len, s_code, bpA, bpB, dwA[t], dwB[t]);
                }
                if constexpr (TILED) {      // exponents only; merged after they have changed lanes
                    ov[Q] = u32x4{dwA[0], dwA[1], dwA[2], dwA[3]};
                    ov[Q + C::PIECES / 2] = u32x4{dwB[0], dwB[1], dwB[2], dwB[3]};
                    continue;
                }
                const u32x4 oA = merge_piece(dwA, pl[Q]);
                const u32x4 oB = merge_piece(dwB, pl[Q + C::PIECES / 2]);
                if constexpr (RELOAD) {
                    pl[Q] = LD_STREAM((const GLOBAL u32x2 *)(next_pl + Q * next_pstride));
                    pl[Q + C::PIECES / 2] = LD_STREAM((const GLOBAL u32x2 *)(next_pl + (Q + C::PIECES / 2) * next_pstride));
                }
                if constexpr (CUT) {
                    store_cut(oA, Q * ostride);
                    store_cut(oB, (Q + C::PIECES / 2) * ostride);
                } else if constexpr (BURST == 1) {
                    ov[Q] = oA;
                    ov[Q + C::PIECES / 2] = oB;
                } else if constexpr (BURST == 2) {
                    // half bursts: the pieces of two steps leave together
                    ov[2 * (Q & 1)] = oA;
                    ov[2 * (Q & 1) + 1] = oB;
                    if (Q & 1) {
                        __builtin_amdgcn_sched_barrier(0);
                        ST_STREAM(ov[0], (GLOBAL u32x4 *)(out_c + (Q - 1) * ostride));
                        ST_STREAM(ov[1], (GLOBAL u32x4 *)(out_c + (Q - 1 + C::PIECES / 2) * ostride));
                        ST_STREAM(ov[2], (GLOBAL u32x4 *)(out_c + Q * ostride));
                        ST_STREAM(ov[3], (GLOBAL u32x4 *)(out_c + (Q + C::PIECES / 2) * ostride));
                        __builtin_amdgcn_sched_barrier(0);
                    }
                } else {
                    ST_STREAM(oA, (GLOBAL u32x4 *)(out_c + Q * ostride));
                    ST_STREAM(oB, (GLOBAL u32x4 *)(out_c + (Q + C::PIECES / 2) * ostride));
                }
            }
            if constexpr (CUT) {
            } else if constexpr (TILED) {
                // Row-tiled blob: lane (r = l % 16, g = l / 16) holds the exponents of columns 64 Q + 16 g of row r; stored
                // as they are a piece would cover 16 rows x 64 bytes, and its nibbles 16 rows x 32.  Through the wave's
                // tile the exponents become whole row segments (lane l: row 4 j + l / 16, columns 16 (l % 16)), are merged
                // with nibbles that were loaded in that order (4 rows x 128 bytes per instruction) and leave as 4 rows x 256
                // bytes.  The 16-byte units of a row are swizzled by the row number against bank conflicts.
                uint8_t *tile = smem + C::OFF_TILE + wave * C::TILE_BYTES;
                const uint32_t r = lane & 15, g = lane >> 4;
#pragma unroll
                for (int Q = 0; Q < C::PIECES; Q++) *(u32x4 *)(tile + r * 256 + (((4 * Q + g) ^ r) & 15) * 16) = ov[Q];
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    const u32x4 e = *(const u32x4 *)(tile + (4 * j + g) * 256 + ((r ^ (4 * j + g)) & 15) * 16);
                    const uint32_t dw[4] = {e.x, e.y, e.z, e.w};
                    ov[j] = merge_piece(dw, pl[j]);
                    if constexpr (RELOAD) pl[j] = LD_STREAM((const GLOBAL u32x2 *)(next_pl + j * next_pstride));
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < 4; j++) ST_STREAM(ov[j], (GLOBAL u32x4 *)(out_c + j * ostride));
                __builtin_amdgcn_sched_barrier(0);
            } else if constexpr (BURST == 1) {
                __builtin_amdgcn_sched_barrier(0);   // keep the stores together, after the decode
#pragma unroll
                for (int Q = 0; Q < C::PIECES; Q++) ST_STREAM(ov[Q], (GLOBAL u32x4 *)(out_c + Q * ostride));
                __builtin_amdgcn_sched_barrier(0);
            }
        };

        if constexpr (!TILED) {
            if (tail_here) {
                uint64_t byte0;
                const uint64_t span64 = span_of(m_cur, byte0);
                if (span64 <= (uint64_t)C::STAGE) {
                    const uint32_t cl = seg_end - 1 - first_chunk;
                    const uint32_t rel = wave_incl_scan(m_cur.lb) - m_cur.lb;
                    const uint64_t b0 = uniform64(m_cur.b0);
#pragma unroll
                    for (int k = 0; k < C::SEGS; k++) {
                        const uint32_t i = lane16 + 1024 * k;
                        if (i < (uint32_t)span64) *(u32x4 *)(stage + i) = seg[k];
                    }
                    // lanes with fewer symbols than N decode on past their bits: N / 2 codewords at the most, in bounds
                    decode_store(std::false_type{}, std::true_type{}, stage_off * 8 + (uint32_t)(b0 - byte0 * 8) + rel, m_cur.lb, pl,
                                 out + chunk_base(cl) + lane_off, chunk_stride(cl), plane, 0u);
                } else if (lane == 0) {
                    *s_tail = 1;          // left to the symbol pass
                }
                if (cg < fast_end) {
                    ask_first(cg);
                    load_stream(m_cur, seg);
                }
            }
        }
        if (cg < fast_end) {
            // Drain the prologue's loads here (vmcnt(0), other counters untouched), so that
            // the wait at the loop head is decided by the back edge alone, where the four
            // stores of the previous chunk are younger than the prefetch and stay in flight.
            __builtin_amdgcn_s_waitcnt(0x0F70);
            for (;;) {
                const uint32_t cl = cg - first_chunk;            // chunk index inside the tensor
                GLOBAL uint8_t *out_c = out + chunk_base(cl) + lane_off;   // this lane's piece 0
                const stride_t ostride = chunk_stride(cl);
                const uint64_t b0 = uniform64(m_cur.b0);
                uint64_t byte0;
                const uint64_t span64 = span_of(m_cur, byte0);
                const bool staged = __builtin_amdgcn_readfirstlane((uint32_t)(span64 <= (uint64_t)C::STAGE)) != 0;

                // lane start bit = chunk start + exclusive DPP scan of the lanes' bit counts
                const uint32_t rel = wave_incl_scan(m_cur.lb) - m_cur.lb;
                const uint32_t bit_in = (uint32_t)(b0 - byte0 * 8) + rel; // bits from byte0

#pragma unroll
                for (int k = 0; k < C::SEGS; k++) {
                    const uint32_t i = lane16 + 1024 * k;
                    if (i < (uint32_t)C::STAGE && (!PAIRFIT || i < (uint32_t)span64)) *(u32x4 *)(stage + i) = seg[k];
                }

                // prefetch: the next chunk's span of the stream into the registers just written out, the metadata
                // of the chunk after it; the next chunk's nibble plane follows piece by piece inside the decode
                // (after the last chunk: this chunk's plane again, not a branch around the loads)
                const bool has_next = cg1 < fast_end;
                Meta m_next2 = m_next;
                if (has_next) {
                    load_stream(m_next, seg);
                    cg2 = draw();
                    if (cg2 < fast_end) m_next2 = load_meta(cg2 - first_chunk);
                }
                const uint32_t cl_pl = (has_next ? cg1 : cg) - first_chunk;

                if (!staged && lane == 0) {
                    const uint32_t at = __hip_atomic_fetch_add(s_oversize, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    if (at < (uint32_t)C::LIST_MAX) s_list[at] = cg - c;
                }
                // a chunk whose span was not staged decodes stale bits (redone after the loop): its runs are
                // pinned to the start of the wave's stage, so that every window stays inside this kernel's LDS
                decode_store(std::true_type{}, std::false_type{}, stage_off * 8 + (staged ? bit_in : 64u), staged ? m_cur.lb : 0u, pl, out_c, ostride,
                             plane_of(cl_pl), chunk_stride(cl_pl) / 2);

                if (!has_next) break;
                m_cur = m_next;
                m_next = m_next2;
                cg = cg1;
                cg1 = cg2;
            }
        }
        __syncthreads();

        // Chunks whose span did not fit a stage (they code far worse than 4 bits per symbol; the
        // loop decoded garbage for them, in bounds): the stage area now serves as SLOTS wide slots.
        // Round by round the workgroup copies up to SLOTS such spans in, and one wave per slot
        // decodes with the loop's own steps.  PAIRFIT launches never get here with a valid blob.
        const uint32_t n_over = *s_oversize;
        const bool tail_left = *s_tail != 0;          // a ragged last chunk whose span did not fit a stage
        bool scan_all = tail_left;
        if (n_over != 0) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");   // the loop's stores land first
            if (PAIRFIT || n_over > (uint32_t)C::LIST_MAX) {
                scan_all = true;                      // too many to remember: symbol pass over everything
            } else {
                for (uint32_t r0 = 0; r0 < n_over; r0 += C::SLOTS) {
                    __syncthreads();                  // slots free (first round: every wave is out of the loop)
                    for (uint32_t k = 0; k < (uint32_t)C::SLOTS && r0 + k < n_over; k++) {
                        const uint32_t cl = c + s_list[r0 + k] - first_chunk;
                        const uint64_t sb0 = chunk_bit[cl], sb1 = chunk_bit[cl + 1];
                        uint64_t byte_end = ((sb1 + 7) >> 3) + 8;
                        if (byte_end > st_bytes) byte_end = st_bytes;
                        uint64_t byte0 = (sb0 >> 3) & ~15ull;
                        if (byte0 > byte_end) byte0 = byte_end;
                        const uint64_t span = byte_end - byte0;
                        uint8_t *slot = smem + C::OFF_WAVES + k * C::SLOT;
                        for (uint32_t i = tid * 16; i < (uint32_t)C::SLOT && i < span; i += WAVES * 64 * 16)
                            *(u32x4 *)(slot + i) = *(const GLOBAL u32x4 *)(stream + byte0 + i);
                    }
                    __syncthreads();
                    if ((uint32_t)wave < (uint32_t)C::SLOTS && r0 + wave < n_over) {
                        const uint32_t cl = c + s_list[r0 + wave] - first_chunk;
                        const Meta m = load_meta(cl);
                        uint64_t byte0;
                        const uint64_t span = span_of(m, byte0);
                        if (span <= (uint64_t)C::SLOT) {          // else: a corrupt blob, left as decoded in the loop
                            u32x2 pl_s[C::PIECES];
                            const GLOBAL uint8_t *plane_c = plane_of(cl);
                            const stride_t pstride = chunk_stride(cl) / 2;
#pragma unroll
                            for (int j = 0; j < C::PIECES; j++) pl_s[j] = *(const GLOBAL u32x2 *)(plane_c + j * pstride);
                            const uint32_t rel = wave_incl_scan(m.lb) - m.lb;
                            const uint64_t b0 = uniform64(m.b0);
                            decode_store(std::false_type{}, std::false_type{}, (C::OFF_WAVES + wave * C::SLOT) * 8 + (uint32_t)(b0 - byte0 * 8) + rel, m.lb, pl_s,
                                         out + chunk_base(cl) + lane_off, chunk_stride(cl), plane_c, 0u);
                        }
                    }
                }
            }
        }
        // Symbol pass, with windows and nibbles read straight from HBM: a ragged last chunk that did not fit a stage
        // (and everything oversize when the list above did not apply).
        if (scan_all) {
            // The chunks redone here were stored (as garbage) by whichever wave drew them in the loop, not
            // necessarily by the wave that redoes them: every wave's loop stores are complete (fence)
            // before any wave issues a store of this pass (barrier; scan_all is uniform).
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            __syncthreads();
            for (uint32_t cg2 = c + wave; cg2 < seg_end; cg2 += WAVES) {
                const uint32_t cl = cg2 - first_chunk;
                Meta m = load_meta(cl);
                uint64_t byte0;
                const uint64_t span64 = span_of(m, byte0);
                const bool redo = (tail_left && cg2 >= fast_end) || (span64 > (uint64_t)C::STAGE && (PAIRFIT || n_over > (uint32_t)C::LIST_MAX));
                if (!__builtin_amdgcn_readfirstlane((uint32_t)redo)) continue;
                const uint64_t elem0 = chunk_base(cl);
                const uint64_t estride = TILED ? 64 : chunk_stride(cl);
                const uint32_t rel = wave_incl_scan(m.lb) - m.lb;
                const GLOBAL uint8_t *sp = stream + byte0;
                uint64_t bA = (m.b0 - byte0 * 8) + rel;   // forward run: next bit
                uint64_t bB = bA + m.lb;                  // backward run: one past the next bit
#pragma unroll 1
                for (int Q = 0; Q < C::PIECES; Q++) {
                    const uint64_t o = elem0 + (uint64_t)Q * estride + symbol_off;
                    const bool fwd = Q < C::PIECES / 2;
#pragma unroll 1
                    for (uint32_t i = 0; i < 16 && o + i < n_elem; i++) {
                        const uint32_t w = fwd ? global_window<+1>(sp, bA) : global_window<-1>(sp, bB);
                        const uint32_t r = decode_one<LONG>(w, tbl, s_len, s_code);
                        if (fwd) bA += r >> 8; else bB -= r >> 8;
                        const uint64_t el = o + i;
                        const uint32_t pb = plane[(el >> 3) * 4 + (el & 3)];
                        const uint32_t nib = (el & 4) ? pb >> 4 : pb & 15u;
                        out[el] = (uint8_t)(((r & 15u) << 3) | ((nib & 8u) << 4) | (nib & 7u));
                    }
                }
            }
        }
        c = seg_end;
    }
}

template <int N, int WAVES, bool PAIRFIT, bool TILED = false, bool LONG = !PAIRFIT, int BURST = PAIRFIT, bool FAR = false>
int launch_as(const KArgs &a, int wgs_per_cu, hipStream_t s)
{
    int cus = device_cus();
    if (cus <= 0) return ECF8_E_HIP;
    // Few chunks are spread over the compute units, a workgroup each: a wave alone on its compute unit gets through a
    // chunk's steps faster, and the chunks' loads start at more places (128 chunks of 128 symbols per lane: 16 full
    // workgroups 9.8 us, 128 workgroups with one chunk each 8.4; 1024 chunks 9.1 / 8.3).  Beside a consumer on another stream, 24
    // layers decoded ahead, means of five runs, full workgroups / a chunk each: 128 chunks beside copies 823 / 752 us, 4096^3 products
    // 2832 / 2776, one product with a weight matrix 798 / 789; 512 chunks 851 / 787, 2845 / 2865, 873 / 881; 1024 chunks 867 / 817,
    // 2843 / 2872, 881 / 906.  It costs up to 3 % there beside products and gives 6 .. 9 % beside copies.
    uint64_t want = a.total_chunks;
    uint64_t cap = (uint64_t)cus * wgs_per_cu;
    if (a.max_workgroups && a.max_workgroups < cap) cap = a.max_workgroups;
    uint32_t grid = (uint32_t)(want < cap ? want : cap);
    if (grid == 0) grid = 1;
    KArgs dealt = a;
    dealt.deal = deal_chunks(a.total_chunks, grid);
    // One tensor without a table, whose code comes from the host; the kernel has no other way in, and 20 to 30 registers less.  The same kernel for all / its own, us:
    // 64 x 256 7.0 / 6.0, row-tiled 6.4 / 5.1, 1024 x 1024 7.5 / 6.7, row-tiled 6.9 / 5.9, 1000 x 3001 7.9 / 7.2.
    if constexpr (PAIRFIT) {
        if (!a.items && !a.single.off_table) {
            hipLaunchKernelGGL((ecf8_decode_kernel<N, WAVES, PAIRFIT, TILED, LONG, BURST, ShortCodes>), dim3(grid), dim3(WAVES * 64), 0, s, dealt,
                               short_codes(a.single.code_len));
            return hipGetLastError() == hipSuccess ? ECF8_OK : ECF8_E_HIP;
        }
    }
    hipLaunchKernelGGL((ecf8_decode_kernel<N, WAVES, PAIRFIT, TILED, LONG, BURST, TableInBlob, FAR>), dim3(grid), dim3(WAVES * 64), 0, s, dealt, TableInBlob{});
    return hipGetLastError() == hipSuccess ? ECF8_OK : ECF8_E_HIP;
}

// Capped codes at N = 128: 8 waves that store a chunk in one burst, or 12 that store piece by piece (no registers for a
// burst).  Up to 8 chunks per workgroup are one round of 8 waves, whose tables are smaller; beyond that 12 waves pay where they
// save a round (one instead of two; on half of the compute units two instead of three), or where the launch is confined
// to so few compute units that HBM is not the bound (not for 13 .. 16 chunks,
// two rounds either way).  Measured, us with 8 / with 12 waves, by workgroups: chunks per workgroup
//   256: 1 8.7 / 9.2, 9 13.3 / 12.1, 10 13.8 / 13.1, 11 13.7 / 13.8, 12 14.1 / 14.3, 16 16.8 / 17.5, 104 76.5 / 88.7
//   192: 11 13.3 / 12.8, 13 14.5 / 14.8, 15 14.9 / 15.5, 64 42.0 / 44.7
//   128: 14 15.2 / 15.5, 16 14.3 / 14.6, 18 16.0 / 15.8, 22 18.4 / 17.9, 24 18.8 / 18.4, 96 51.5 / 51.4, 208 100.8 / 102.4
//    96: 6 10.0 / 10.3, 19 16.9 / 16.4, 32 22.0 / 20.3, 43 28.0 / 28.3, 277 129.6 / 126.5;  64: 40 25.0 / 22.4, 416 186 / 171
//    32: 16 14.0 / 14.2, 48 29.2 / 26.5, 832 357 / 299
int pairfit_128(const KArgs &a, hipStream_t s)
{
    const int cus = device_cus();
    if (cus <= 0) return ECF8_E_HIP;
    const uint64_t wgs = a.max_workgroups && a.max_workgroups < (uint32_t)cus ? a.max_workgroups : (uint64_t)cus;
    const uint64_t each = (a.total_chunks + wgs - 1) / wgs;
    const bool few = 8 * wgs <= 3 * (uint64_t)cus, half = 2 * wgs <= (uint64_t)cus;
    if (each > 8 && (each <= 11 || (half && each > 16 && each <= 24) || (few && (each == 12 || each > 16))))
        return launch_as<128, 12, true, false, false, 0>(a, 1, s);
    return launch_as<128, 8, true>(a, 1, s);
}

// Workgroup shapes.  PAIRFIT kernels: N = 128 runs 8 waves of ~200 VGPRs, which is what holding a chunk's 8
// output pieces for the store burst takes; it has compute to spare (6 waves measured the same, 4 a sixth slower);
// N = 64 runs 12 waves (2 % faster than 16).  General kernels: 12 waves, the most that
// leaves registers for a burst (N = 64: the whole chunk; N = 128: half a chunk at a time); N = 32 runs 16 waves
// and stores piece by piece, which measured faster there.
int dispatch(const KArgs &a, uint32_t lane_syms, hipStream_t s)
{
    const bool pairfit = 2 * a.max_code_len <= (uint32_t)TB;
    const bool lng = a.max_code_len > (uint32_t)TB;      // a codeword the table cannot hold: the kernels with the out-of-line matcher
    switch (lane_syms) {
    case 32:
        if (pairfit) return launch_as<32, 16, true>(a, 1, s);
        return lng ? launch_as<32, 16, false, false, true, 0>(a, 1, s) : launch_as<32, 16, false, false, false, 0>(a, 1, s);
    case 64:
        // the fused GEMM's blobs (row-tiled, capped codes): decoded chunks leave as whole row segments.  8 waves: a layer of
        // seven matrices (418 MB) takes 87.4 us, with 10 waves 88.5, 12 88.8, 16 91.5 (merged before the exponents
        // changed lanes, nibbles read as 16 rows x 32 bytes: 16 waves 108); in the linear layout without groups, which
        // this layout cannot have, 84
        if (pairfit && a.row_tiled) return launch_as<64, 8, true, true>(a, 1, s);
        if (pairfit) return launch_as<64, 12, true>(a, 1, s);
        return lng ? launch_as<64, 12, false, false, true, 1>(a, 1, s) : launch_as<64, 12, false, false, false, 1>(a, 1, s);
    case 128:
        if (pairfit) return pairfit_128(a, s);
        return lng ? launch_as<128, 12, false, false, true, 2>(a, 1, s) : launch_as<128, 12, false, false, false, 2>(a, 1, s);
    default: return ECF8_E_ARG;
    }
}

// A batch of more chunks than a launch counts (4 TiB or more)
int dispatch_far(KArgs a, uint32_t lane_syms, hipStream_t s)
{
    const uint64_t all = a.total_chunks;
    for (; a.base < all; a.base += LAUNCH_CHUNKS) {
        a.total_chunks = all - a.base < LAUNCH_CHUNKS ? all - a.base : LAUNCH_CHUNKS;
        const int rc = lane_syms == 32 ? launch_as<32, 16, false, false, true, 0, true>(a, 1, s)
                     : lane_syms == 64 ? launch_as<64, 12, false, false, true, 1, true>(a, 1, s)
                     : lane_syms == 128 ? launch_as<128, 12, false, false, true, 2, true>(a, 1, s) : ECF8_E_ARG;
        if (rc) return rc;
    }
    return ECF8_OK;
}

} // namespace

extern "C" {

int ecf8_decode(const ecf8_header *h, const void *d_blob, void *d_out, uint64_t out_capacity, void *stream)
{
    if (!h || !d_blob || !d_out) return ECF8_E_ARG;
    if (h->magic != ECF8_MAGIC || h->version != ECF8_VERSION || h->n_elem == 0 || h->n_chunks == 0 ||
        (h->table_bits != 0 && h->table_bits != ECF8_TB) || h->group_chunks == 0 || h->group_chunks > 64 ||
        (h->group_chunks & (h->group_chunks - 1)))
        return ECF8_E_FORMAT;
    if (h->tile_rows != 0 && (h->tile_rows != 16 || h->group_chunks != 1 || h->rows % 16 != 0 || h->cols == 0 ||
                              h->cols % (4ull * h->lane_syms) != 0 || h->rows > (1ull << 40) / h->cols || h->n_elem != h->rows * h->cols))
        return ECF8_E_FORMAT;
    if (h->n_chunks != (h->n_elem + 64ull * h->lane_syms - 1) / (64ull * h->lane_syms) || h->n_chunks > LAUNCH_CHUNKS) return ECF8_E_FORMAT;
    if (h->off_plane + h->plane_bytes > h->total_size || h->off_stream + h->stream_bytes > h->off_plane ||
        h->plane_bytes != h->n_chunks * 32ull * h->lane_syms)
        return ECF8_E_FORMAT;
    if (out_capacity < h->n_elem) return ECF8_E_CAPACITY;
    if (((uintptr_t)d_blob | (uintptr_t)d_out) & 15) return ECF8_E_ALIGN;
    KArgs a{};
    a.single.d_blob = (uint64_t)(uintptr_t)d_blob;
    a.single.d_out = (uint64_t)(uintptr_t)d_out;
    a.single.n_elem = h->n_elem;
    a.single.n_chunks = h->n_chunks;
    a.single.first_chunk = 0;
    a.single.off_chunk_bit = h->off_chunk_bit;
    a.single.off_lane_bits = h->off_lane_bits;
    a.single.off_stream = h->off_stream;
    a.single.off_plane = h->off_plane;
    a.single.stream_bytes = h->stream_bytes;
    a.single.off_table = h->table_bits ? 256 : 0;
    a.single.group_chunks = h->group_chunks;
    a.single.tile_cols = h->tile_rows ? h->cols : 0;
    for (int i = 0; i < 16; i++) a.single.code_len[i] = h->code_len[i];
    a.items = nullptr;
    a.n_items = 1;
    a.total_chunks = h->n_chunks;
    a.row_tiled = h->tile_rows != 0;
    for (int i = 0; i < 16; i++) a.max_code_len = h->code_len[i] > a.max_code_len ? h->code_len[i] : a.max_code_len;
    if (a.max_code_len == 0 || a.max_code_len > 15) return ECF8_E_ARG;
    return dispatch(a, h->lane_syms, (hipStream_t)stream);
}

int ecf8_decode_batched(const ecf8_batch_item *d_items, uint32_t n_tensors, const ecf8_batch_info *info,
                        void *stream)
{
    if (!d_items || !info || n_tensors == 0 || info->total_chunks == 0) return ECF8_E_ARG;
    if ((uintptr_t)d_items & 15) return ECF8_E_ALIGN;
    KArgs a{};
    a.items = (const GLOBAL ecf8_batch_item *)(uintptr_t)d_items;
    a.n_items = n_tensors;
    a.total_chunks = info->total_chunks;
    a.max_code_len = info->max_code_len;
    a.max_workgroups = info->max_workgroups;
    a.row_tiled = info->row_tiled;
    if (a.max_code_len == 0 || a.max_code_len > 15) return ECF8_E_ARG;
    return a.total_chunks > LAUNCH_CHUNKS ? dispatch_far(a, info->lane_syms, (hipStream_t)stream) : dispatch(a, info->lane_syms, (hipStream_t)stream);
}

} // extern "C"
