// Backward of a wide attention layer with two groups, a launch a group, a wavefront per head (wide_heads_bwd.hip).
#pragma once
#include "fused.h"

namespace gswa {

// C = 180, six heads, two groups, 8x8 windows, bf16; any shift.
bool wide_heads_bwd_supported(const Geom &g);
// Scratch: first wide_heads_bwd_free_bytes that are the caller's from the start, then one vector of partial gradients of a
// group per workgroup.
size_t wide_heads_bwd_ws_bytes(const Geom &g);
size_t wide_heads_bwd_free_bytes(const Geom &g);
// dx, d w_qkv, d b_qkv and d table; the sum of the first group's vectors is left to the caller (`last`).
hipError_t launch_wide_heads_bwd(const Geom &g, const bf16_t *x, const bf16_t *dy, const bf16_t *attn, const uint8_t *pack,
                                 const bf16_t *table, bf16_t *dx, float *dw_qkv, float *db_qkv, float *dtable, int accumulate,
                                 void *ws, ReduceJob &last, hipStream_t s);

} // namespace gswa
