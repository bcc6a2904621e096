// Instantiations of window_layer_impl.h for fp32, and the choice among all of them.
#include "window_layer_impl.h"

namespace gswa {

// fp32 layers of 60 channels and 8x8 windows
// (one group: a wavefront holds two score-gradient tiles of 64x16, for which 128 registers are too few)
const WindowLayerOps *window_layer_f32(const Geom &g)
{
#define X(G) { using S = WinShape<float, 60, 6, G, 8, 10, 120, G == 1 ? 12 : 16>; if (matches<S>(g)) return ops_of<S>(); }
    X(1) X(2) X(3) X(6)
#undef X
    return nullptr;
}

const WindowLayerOps *window_layer_ops(const Geom &g, bool f32, int hidden)
{
    if (g.T * g.C >= (1L << 40) || (hidden != 0 && hidden != 2 * g.C)) return nullptr;
    if (f32) return window_layer_f32(g);
    if (const WindowLayerOps *o = window_layer_bf16_w12h4(g)) return o;
    return window_layer_bf16_w12h6(g);
}

} // namespace gswa
