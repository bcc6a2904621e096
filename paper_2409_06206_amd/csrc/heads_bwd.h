// Backward of a narrow attention layer in one launch, a wavefront per head (heads_bwd.hip).
#pragma once
#include "common.h"

namespace gswa {

// C = 60, six heads, 8x8 windows, bf16, one to three groups.
bool heads_bwd_supported(const Geom &g);
// Scratch: one vector of partial parameter gradients per workgroup.
size_t heads_bwd_ws_bytes(const Geom &g);
// As launch_fused_bwd (fused.h).
hipError_t launch_heads_bwd(const Geom &g, const bf16_t *x, const bf16_t *dy, const bf16_t *attn, const void *pack,
                            const bf16_t *table, bf16_t *dx, float *dw_qkv, float *db_qkv, float *dw_proj, float *db_proj,
                            float *dtable, int accumulate, void *ws, hipStream_t s);

} // namespace gswa
