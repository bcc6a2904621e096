// Whole layers one window at a time (Sec. "Agile Swin Transformer Block", Eq. 4-8): every step of a layer acts on
// single tokens or inside one window, so a workgroup takes a window from x to y (forward) or from dy to dx
// (backward) without leaving its compute unit.
#pragma once
#include "../../include/gswa.h"
#include "common.h"

namespace gswa {

struct WindowLayerArgs {
    Geom g;
    float eps;
    // attention layer; `x` is its input, or with the whole layer the layer's input
    const void *x, *w_qkv, *b_qkv, *w_proj, *b_proj, *table;
    // whole layer only
    const void *ln1_w, *ln1_b, *ln2_w, *ln2_b, *w_fc1, *b_fc1, *w_fc2, *b_fc2;
    void *y, *attn, *x1;        // forward: outputs; attn (group outputs) and x1 may be null.  backward: attn, x1 are inputs
    const void *dy;             // backward
    void *dx;
    float *part;                // backward: one vector of parameter gradients per workgroup
};

// Gradients in the order of a workgroup's vector; the whole-layer ones behind the attention layer's.
struct WindowLayerGrads {
    float *w_qkv, *b_qkv, *w_proj, *b_proj, *table;
    float *w_fc1, *b_fc1, *w_fc2, *b_fc2, *ln1_w, *ln1_b, *ln2_w, *ln2_b;
};

// Checks a descriptor and derives its geometry (GSWA_OK or an error code).
int make_geom(const gswa_desc *d, Geom *g);

// hidden == 0 asks for the attention layer alone
bool window_layer_supported(const Geom &g, bool f32, int hidden);
// scratch of the backward: the workgroups' vectors
size_t window_layer_bwd_ws_bytes(const Geom &g, int hidden);
hipError_t launch_window_layer_fwd(const WindowLayerArgs &a, bool f32, int hidden, hipStream_t s);
hipError_t launch_window_layer_bwd(const WindowLayerArgs &a, bool f32, int hidden, const WindowLayerGrads &gr,
                                   int accumulate, hipStream_t s);

} // namespace gswa
