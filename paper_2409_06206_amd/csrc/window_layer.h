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

// gswa_forward with what a whole layer or a sequence of layers knows besides.
struct AttnLn { // LayerNorm in front of the layer
    const void *x, *w, *b;
    float eps;
};
struct AttnOpts {
    bool packed = false; // the repacked parameters are where this call would put them (kernels that read none take no notice)
    void *pack = nullptr; // (with `packed`) they are here instead
    const AttnLn *ln = nullptr; // only where attn_forward_takes_ln: the layer is applied to LayerNorm(ln->x); `x` then only
                                // names the memory that LayerNorm would have been written to
    int windows = 0;            // > 0: only the first so many windows are wanted, the other tokens of y may hold anything
};
bool attn_forward_takes_ln(const gswa_desc *d);
// Bytes of the repacked parameters of kernels that read them repacked, and where they lie in `saved`; 0: there are none.
size_t attn_pack_bytes(const gswa_desc *d, size_t *saved_offset);
int attn_forward(const gswa_desc *d, const void *x, const void *w_qkv, const void *b_qkv, const void *w_proj, const void *b_proj,
                 const void *bias_table, void *y, void *saved, void *ws, const AttnOpts &o, void *hip_stream);

// The rules of gswa_forward's and gswa_backward's arguments alone (nothing is enqueued): for callers that run the
// attention layer inside a kernel of their own.
int attn_forward_check(const gswa_desc *d, const void *x, const void *w_qkv, const void *b_qkv, const void *w_proj,
                       const void *b_proj, const void *bias_table, const void *y, const void *saved, const void *ws);
int attn_backward_check(const gswa_desc *d, const void *x, const void *dy, const void *w_qkv, const void *b_qkv,
                        const void *w_proj, const void *b_proj, const void *bias_table, const void *saved, const void *dx,
                        const void *dw_qkv, const void *db_qkv, const void *dw_proj, const void *db_proj,
                        const void *dbias_table, const void *ws);

// Vectors of parameter gradients a backward launch leaves at most (= its workgroups).
constexpr int kWindowLayerVectors = 256;

// What a shape brings; index 0: the attention layer alone, 1: the whole layer (hidden = 2 C).
struct WindowLayerOps {
    size_t vector[2]; // floats of a workgroup's vector
    hipError_t (*fwd[2])(const WindowLayerArgs &, hipStream_t);
    hipError_t (*bwd[2])(const WindowLayerArgs &, const WindowLayerGrads &, int accumulate, hipStream_t);
};
// the shapes of each file that instantiates the kernels (null: none fits)
const WindowLayerOps *window_layer_f32(const Geom &g);
const WindowLayerOps *window_layer_bf16_w12h4(const Geom &g);
const WindowLayerOps *window_layer_bf16_w12h6(const Geom &g);

// The kernels that serve a layer, or null.  hidden == 0 asks for the attention layer alone.
const WindowLayerOps *window_layer_ops(const Geom &g, bool f32, int hidden);
// scratch of the backward: the workgroups' vectors
inline size_t window_layer_bwd_ws_bytes(const WindowLayerOps &ops, const Geom &g, bool layer)
{
    return (size_t)(g.nW < kWindowLayerVectors ? g.nW : kWindowLayerVectors) * ops.vector[layer] * sizeof(float);
}

} // namespace gswa
