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

// Every window of these layers is taken by a workgroup of its own, whatever their number.  us per pass (inference;
// forward + backward), the kernels that served the layer before / these:
//                                                      1 window           256               2048              16384
//   fp32, 8x8, two groups, attention layer          98 / 15  349 / 51   114 / 17  494 / 61   470 / 112  2107 / 404   3630 / 872  16096 / 3159
//   fp32, 8x8, two groups, whole layer             150 / 22  498 / 79   183 / 24  766 / 92   676 / 171  2905 / 644   5318 / 1313 21588 / 5047
//                                                      1 window           256               512               7744
//   12x12, four heads, dqk 4, two groups, attention 21 / 14   80 / 56    24 / 17  139 / 68    43 / 25    237 / 115    632 / 294   3083 / 1559
//   the same, whole layer                           35 / 22  121 / 81    47 / 26  209 / 97    75 / 46    327 / 177    846 / 645   3735 / 2609
//   six heads, dqk 4, one group, attention          30 / 16   73 / 70    35 / 19  168 / 84    64 / 34    290 / 152    928 / 450   4090 / 2180
//   six heads, dqk 4, six groups, whole layer       42 / 32  222 / 116   56 / 36  360 / 130   90 / 66    539 / 249   1080 / 966   6071 / 3736
// The other organisations lie between.  (The one call that takes longer is the backward alone of six heads in one group
// with up to 16 windows, 43 / 54: its forward gains more.  No rule looks at the number of windows: an image has to give
// the same bits alone and in a batch.)
const WindowLayerOps *window_layer_ops(const Geom &g, bool f32, int hidden)
{
    if (g.T * g.C >= (1L << 40) || (hidden != 0 && hidden != 2 * g.C)) return nullptr;
    if (f32) return window_layer_f32(g);
    if (const WindowLayerOps *o = window_layer_bf16_w12h4(g)) return o;
    return window_layer_bf16_w12h6(g);
}

} // namespace gswa
