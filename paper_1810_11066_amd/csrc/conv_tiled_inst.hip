// Instantiations of conv_generic_kernel_tiled for groups of BS_A activation
// planes (BS_A = 1..4).  The build compiles this source once per width, so
// that the widths compile in parallel.
#include "conv_tiled.h"

#ifndef BS_A
#error "BS_A (activation planes per group, 1..4) must be defined"
#endif

namespace bs {
namespace tiled {

template <>
TiledKernelFn pick_a<BS_A>(int w, int cb, int c, bool xnor, bool req) {
    return pick_for_a<BS_A>(w, cb, c, xnor, req);
}

}  // namespace tiled
}  // namespace bs
