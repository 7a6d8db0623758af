// March kernel instances: complex64, one mesh, 64-bit addresses per lane.
#include "tsq_march.hpp"

namespace tsq {

const void* march_ptr_c64_lanes(int steps, bool last, int ppl, bool lds) {
    return pick_kernel<C64, Variant::Lanes>(steps, last, ppl, lds);
}

}  // namespace tsq
