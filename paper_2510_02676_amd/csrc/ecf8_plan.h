// Internal (not part of the C ABI): what the CPU encoder and the GPU encoder share on the host -- option checks, the container
// layout, limits -- and the CPU encoder's code from a histogram (the GPU encoder makes its own on the device).
#ifndef ECF8_PLAN_H
#define ECF8_PLAN_H

#include <cstdint>

#include "ecf8.h"

// A host blob: `data` comes from std::aligned_alloc(256, .) and is released by ecf8_blob_free.
struct ecf8_blob {
    uint8_t *data;
    uint64_t size;
};

namespace ecf8_internal {

// Kernels number a launch's chunks in 32 bits: this many at the most, beside a tensor of as many that begins before the launch or ends behind it.  Longer
// batches and groups are several launches; a tensor of more (4 TiB or more, the encoders take 1 TiB of E4M3) is refused.
constexpr uint64_t LAUNCH_CHUNKS = 1ull << 31;

constexpr uint64_t round_up(uint64_t v, uint64_t a) { return (v + a - 1) / a * a; }

// The part of either container's layout that depends on the code, for the host and for the kernel that makes the code: where what follows the stream lies.
// The stream ends with 8 bytes that a decoder may look ahead to; off_sign 0: no such section.
struct LayoutEnd {
    uint64_t stream_bytes, off_plane, off_sign, total;
};
constexpr LayoutEnd layout_end(uint64_t off_stream, uint64_t stream_bits, uint64_t plane_bytes, uint64_t sign_bytes)
{
    LayoutEnd e{};
    e.stream_bytes = round_up((stream_bits + 7) / 8 + 8, 16);
    e.off_plane = round_up(off_stream + e.stream_bytes, 256);
    const uint64_t behind = round_up(e.off_plane + plane_bytes, 256);
    e.off_sign = sign_bytes ? behind : 0;
    e.total = behind + round_up(sign_bytes, 256);
    return e;
}

struct Plan {
    ecf8_header hdr;              // complete header of the blob to be written
    uint32_t code[16];            // canonical codewords, first bit most significant
    uint32_t rcode[16];           // the same, bit-reversed (first bit = bit 0)
};

// Checks rows/cols/opts (ECF8_E_ARG) and returns the effective options.
int check_options(uint64_t rows, uint64_t cols, const ecf8_encode_opts *opts, uint32_t *lane_syms,
                  uint32_t *group_chunks, uint32_t *max_code_len, uint32_t *tile_rows, uint32_t *table_mode);

// The header as far as it does not depend on the weights: 0 in total_size, stream_bits, stream_bytes, off_plane, code_len and freq.
int plan_frame(uint64_t rows, uint64_t cols, const ecf8_encode_opts *opts, ecf8_header *hdr);

// From the exponent histogram of a rows x cols tensor: cheapest code under the cap, canonical
// codewords, section layout, header.  Same result for the same inputs on every path.
int plan_encode(const uint64_t freq[16], uint64_t rows, uint64_t cols, const ecf8_encode_opts *opts, Plan *out);

// Largest blob any rows x cols tensor can need under opts.
int encode_bound(uint64_t rows, uint64_t cols, const ecf8_encode_opts *opts, uint64_t *bytes);

// The decoder's pair table for a code (host builder; the kernels have their own).
void build_pair_table_host(const uint8_t len[16], uint16_t *tbl);

} // namespace ecf8_internal

#endif
