// Tile kernel instances (small 2D meshes): complex128.
#include "tsq_tile.hpp"

namespace tsq {

const void* tile_ptr_c128(int pairs_per_wave, bool closed, bool td, bool u4) {
    return pick_tile<C128>(pairs_per_wave, closed, td, u4);
}

}  // namespace tsq
