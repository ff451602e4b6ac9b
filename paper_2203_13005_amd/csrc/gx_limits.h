// Limits that follow from the width of a counter or an index, as plain host
// code: what the engines may hand to a launch.
#pragma once

#include <algorithm>
#include <cstdint>

#ifdef __HIPCC__
#define GX_LIMIT_FN __host__ __device__ inline
#else
#define GX_LIMIT_FN inline
#endif

namespace gx {

// End of the chunk of at most `chunk` entries that starts at `begin` in a row
// that ends at `end`.  Entries of the symmetric image go up to 2^31 - 513, so
// begin + chunk may not fit 32 bits.
GX_LIMIT_FN int32_t chunk_end(int32_t begin, int32_t end, int32_t chunk) {
    return end - begin < chunk ? end : begin + chunk;
}

// Batched SSSP counts a superstep's (edge, 32-lane group) units in 32 bits,
// beside the entries in the other half of one 64-bit counter, and rounds the
// count up to whole tiles of at most BS_MAX_TILE.  A pass therefore takes at
// most this many groups, so that even a superstep with every lane of every
// vertex active fits: 8 groups below 2^29 edges, 2 at the most edges a graph
// may have (2^31 - 2049).
constexpr int64_t BS_MAX_TILE = 4096;
constexpr int64_t BS_UNITS_MAX = 0xFFFFFFFFll - BS_MAX_TILE;
inline uint32_t bs_groups_max(int64_t E) {
    return (uint32_t)std::min<int64_t>(8, BS_UNITS_MAX / std::max<int64_t>(E, 1));
}
// The lanes of a pass asked to take `width` (a multiple of 32, at most 256):
// as many whole groups as fit and divide it.
inline uint32_t bs_pass_width(int64_t E, uint32_t width) {
    const uint32_t G = width / 32, most = bs_groups_max(E);
    uint32_t g = std::min(G, most);
    while (G % g) g--;
    return g * 32;
}

}  // namespace gx
