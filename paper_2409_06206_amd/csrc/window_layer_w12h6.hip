// Instantiations of window_layer_impl.h: bf16, 60 channels in six heads, 12x12 windows, narrow queries and keys.
#include "window_layer_impl.h"

namespace gswa {

const WindowLayerOps *window_layer_bf16_w12h6(const Geom &g)
{
#define X(G, DQ) { using S = WinShape<bf16_t, 60, 6, G, 12, DQ, 120, 12>; if (matches<S>(g)) return ops_of<S>(); }
    X(1, 4) X(2, 4) X(3, 4) X(6, 4)
#undef X
    return nullptr;
}

} // namespace gswa
