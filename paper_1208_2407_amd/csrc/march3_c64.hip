// March kernel instances: complex64, three-dimensional meshes.
#include "tsq_march3.hpp"

namespace tsq {

const void* march3_ptr_c64(bool close) { return pick_kernel3<C64>(close); }
const void* close3_ptr_c64() { return pick_close3<C64>(); }
const void* slab_ptr_c64(int stages, int rp, bool close) { return pick_slab<C64>(stages, rp, close); }

}  // namespace tsq
