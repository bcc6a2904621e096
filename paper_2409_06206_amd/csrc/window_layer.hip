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

// Sequences of bf16 layers with 8x8 windows.  Their other kernels take a window per wavefront (fused.h, astl_mlp.h):
// four launches per layer and forward, a dozen per backward, each as long as a wavefront takes alone with its window.
// While every window has a compute unit of its own, one workgroup per window is about twice as fast, whatever their
// number; every further round of workgroups costs as much again.  Four layers, us per pass, window per wavefront /
// per workgroup, inference and training:
//   two groups   256 windows  123 /  65   464 / 233      512 windows  136 / 120   534 / 426     768  162 / 175   643 / 620
//   one group    256          131 /  62   464 / 227      512          148 /  85   566 / 399
//   three groups 256          121 /  65   481 / 241      512          138 / 116   555 / 443
// Errors against fp64 (64 windows, one layer): 0.82 to 1.17 times those of the other kernels, most of them smaller.
// (Six groups gain least, 1.3 times up to 256 windows and a loss behind, and keep the other kernels.)
constexpr int kSmallLayerWindows = 512;

const WindowLayerOps *window_layer_ops(const Geom &g, bool f32, int hidden, bool sequence)
{
    if (g.T * g.C >= (1L << 40) || (hidden != 0 && hidden != 2 * g.C)) return nullptr;
    if (f32) return window_layer_f32(g);
    if (const WindowLayerOps *o = window_layer_bf16_w12h4(g)) return o;
    if (const WindowLayerOps *o = window_layer_bf16_w12h6(g)) return o;
    return hidden != 0 && sequence && g.nW <= kSmallLayerWindows ? window_layer_bf16_w8(g) : nullptr;
}

} // namespace gswa
