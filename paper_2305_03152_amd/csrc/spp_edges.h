// The words of the row-block layout (see spp_graph.hip) and what its read-back checks of them.
#ifndef SPP_EDGES_H
#define SPP_EDGES_H

#include <stdint.h>

namespace spp {

// Edges grouped by blocks of destination rows and sorted by source inside a block, one 32-bit word
// per edge: (source & (2^18 - 1)) << 14 | row inside the block.  The source's high bits are the
// index of its "source chunk"; bound[c] is the position inside the block of the first edge whose
// chunk is >= c (bound[0] = 0, bound[nch] = edges of the block), so the chunk of the edge at
// position p is the largest c with bound[c] <= p.
constexpr int kTileSrcLoBits = 18;
constexpr int kTileRowBits = 14;
constexpr uint32_t kTileRowMask = (1u << kTileRowBits) - 1u;
constexpr int kPartTile = 4096;          // edges of the CSR per tile of the partition that lays the words out
// The kernels that walk such tiles look at all rows between a tile's first edge and the next tile's, empty ones included; beyond
// this many (isolated vertices side by side) every edge bisects for its row instead: some twenty dependent reads, where 4M
// empty rows would be 4000 rounds of a workgroup.  Rows per tile, placing pass and general fill in us, all rows and bisected:
// 8000 (1029 tiles) 75 + 42, 106 + 76; 16000 (516) 65 + 39, 78 + 59; 32000 (258) 66 + 40, 61 + 48; 64000 (129) 58 + 52, 35 + 32.
constexpr int kTileManyRows = 32768;

__device__ __forceinline__ uint32_t tile_source(uint32_t word, int chunk) {
    return ((uint32_t)chunk << kTileSrcLoBits) | (word >> kTileRowBits);
}

// Whether the word of a block's edge in source chunk `chunk` may be walked: its source and row exist, and its source
// is not below that of the word before it in the chunk (the word itself where it is the first), which is what lets the
// dense hops read 512 edges' values of y from a stretch that the first and the last of them bound.
__device__ __forceinline__ bool tile_word_ok(uint32_t word, uint32_t before, int chunk, uint32_t N, uint32_t rows) {
    return tile_source(word, chunk) < N && (word & kTileRowMask) < rows && (before >> kTileRowBits) <= (word >> kTileRowBits);
}

// Adds a 64-bit mix of the edge v -> u to a sum; the edges of two structures are compared by their sums, each
// formed from that structure alone.  One 32-bit and one 32x32 -> 64 product: the kernels that use it are bound by
// their instructions (a wavefront's instruction occupies its SIMD for four clocks, a product for sixteen), and a
// stronger mix was half of the read-back's time.
__device__ __forceinline__ void edge_mix(unsigned long long& sum, uint32_t v, uint32_t u) {
    const uint32_t x = v * 0x9E3779B1u + u;
    sum += (unsigned long long)(x ^ (x >> 15)) * (u ^ 0x85EBCA77u ^ (v << 7));
}

}  // namespace spp
#endif
