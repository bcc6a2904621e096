// Instantiations of window_layer_impl.h: bf16, 60 channels in six heads, 8x8 windows, up to three groups.
#include "window_layer_impl.h"

namespace gswa {

const WindowLayerOps *window_layer_bf16_w8(const Geom &g)
{
#define X(G) { using S = WinShape<bf16_t, 60, 6, G, 8, 10, 120, G == 1 ? 12 : 16>; if (matches<S>(g)) return ops_of<S>(); }
    X(1) X(2) X(3)
#undef X
    return nullptr;
}

} // namespace gswa
