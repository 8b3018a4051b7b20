// tile_sum.hpp -- the entry counts of a tile (512 triangles) of k_keys.  A
// triangle's cells are counted in 32 bits and scanned within its wave in 32
// bits, which a grid far too fine for its mesh can pass (512 triangles of
// 2^23 cells each are 2^32 entries).  The waves' totals and the tile's are
// therefore 64 bits: a total that wrapped would reserve too little and not
// set the overflow flag, the only guard of a workspace that is too small.
// Plain arithmetic, so that it can be tested on the host (MS_HD: the
// includer's function attributes).
#pragma once

#include <stdint.h>

namespace ms {

// From this many entries of one triangle on, its wave's total is summed in 64
// bits beside the scan.  Any bound up to 2^26 would do.
constexpr uint32_t TILE_WIDE = 1u << 16;
static_assert(64ull * (TILE_WIDE - 1) < 1ull << 32, "a wave without a wide triangle fits its scan");

// A triangle's count; one of 2^32 - 1 or more stays there (more than the
// entries of any workspace, so that the overflow is seen).
MS_HD uint32_t tile_count(uint64_t n) { return n < 0xffffffffull ? (uint32_t)n : 0xffffffffu; }

// The entries of all NW waves; `before`: of the waves before wave wv, the
// start of its output, which is meant only where the total fits 32 bits.
template <int NW>
MS_HD uint64_t tile_total(const uint64_t *waves, int wv, uint32_t &before)
{
    uint64_t total = 0;
    before = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        const uint64_t v = waves[i];
        if (i < wv) before += (uint32_t)v;
        total += v;
    }
    return total;
}

// Whether a tile's entries have places at all: a workspace holds less than
// 2^30, and the places within a tile are counted in 32 bits.
MS_HD bool tile_placed(uint64_t total) { return total <= 0xffffffffull; }

}  // namespace ms
