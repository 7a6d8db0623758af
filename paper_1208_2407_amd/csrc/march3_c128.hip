// March kernel instances: complex128, three-dimensional meshes.
#include "tsq_march3.hpp"

namespace tsq {

const void* march3_ptr_c128(bool close) { return pick_kernel3<C128>(close); }
const void* close3_ptr_c128() { return pick_close3<C128>(); }
const void* slab_ptr_c128(int stages, int rp, bool close) { return pick_slab<C128>(stages, rp, close); }

}  // namespace tsq
