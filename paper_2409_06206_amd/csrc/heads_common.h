// What the two backward kernels with a wavefront per head share (heads_bwd.hip, wide_heads_bwd.hip).
#pragma once
#include "fused.h"
#include "mfma.h"

namespace gswa {

// 1 / x for a sum of exponentials (1 .. 64): the hardware's estimate and a Newton step, within 1 ulp of the quotient
__device__ __forceinline__ float recip(float x)
{
    const float r = __builtin_amdgcn_rcpf(x);
    return fmaf(fmaf(-x, r, 1.0f), r, r);
}

// Eq. 8: F = x slice + previous group's output, rounded to bf16 as the forward kernels round it
__device__ __forceinline__ uint4 add_bf16x8(uint4 f, uint4 a)
{
    return make_uint4(add_bf16x2(f.x, a.x), add_bf16x2(f.y, a.y), add_bf16x2(f.z, a.z), add_bf16x2(f.w, a.w));
}

// K step ks of F, lane group q: the slot behind the CG channels is 1 for the bias sums, against zeros in the weights
template <int CG> __device__ __forceinline__ uint4 with_bias_slot(uint4 f, int ks, int q)
{
    if (ks == CG / 32) {
        uint32_t &w = (CG % 8 / 2) == 0 ? f.x : (CG % 8 / 2) == 1 ? f.y : (CG % 8 / 2) == 2 ? f.z : f.w;
        w = q == CG % 32 / 8 ? w | 0x3f80u : w;
    }
    return f;
}

// The bias table (N entries, N even) to LDS by TH threads; the loads are asked for first, whatever else is on its way.
template <int N, int TH> struct TableCopy {
    static_assert(N % 2 == 0, "set-up in whole pieces");
    static constexpr int PAIRS = N / 2, IT = (PAIRS + TH - 1) / TH;
    uint16_t v[IT][2];
    __device__ __forceinline__ void fetch(const bf16_t *table, int tid)
    {
#pragma unroll
        for (int k = 0; k < IT; ++k) {
            const int at = k * TH + tid < PAIRS ? k * TH + tid : PAIRS - 1;
            v[k][0] = table[2 * at].bits;
            v[k][1] = table[2 * at + 1].bits;
        }
    }
    __device__ __forceinline__ void store(bf16_t *dst, int tid) const
    {
#pragma unroll
        for (int k = 0; k < IT; ++k)
            if (k * TH + tid < PAIRS) reinterpret_cast<uint32_t *>(dst)[k * TH + tid] = v[k][0] | (uint32_t)v[k][1] << 16;
    }
};

// Gradient of entry e of a head's bias table from its seven sums of score-gradient tiles (key tile - query tile + 3, rows = keys,
// columns = queries, rows TP floats apart).  The entry of offset (dr, dc) of a query from its key: in tiles of two window rows the
// query's row is rq, the key's rk, with rq - rk - dr = 2 (dl - 3), which two of the four pairs fulfil; eight columns each, all reads
// in flight.
template <int TP> __device__ __forceinline__ float table_entry(const float *mat, int e)
{
    constexpr int M = 8;
    const int dr = e / (2 * M - 1) - (M - 1), dc = e % (2 * M - 1) - (M - 1), odd = dr & 1;
    float a = 0.f;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int rq = odd ? 1 - i : i, rk = i, d2 = rq - rk - dr;
        const bool ok = d2 >= -6 && d2 <= 6;
        const float *t = mat + (((ok ? d2 / 2 : 0) + 3) * 16 + 8 * rk) * TP + 8 * rq;
#pragma unroll
        for (int c = 0; c < M; ++c) {
            const int ck = c - dc;
            const float v = t[(ck < 0 ? 0 : ck >= M ? M - 1 : ck) * TP + c];
            a += ok && ck >= 0 && ck < M ? v : 0.f;
        }
    }
    return a;
}

} // namespace gswa
