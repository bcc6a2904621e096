// Backward of one group of a wide attention layer (C = 180, two groups of three heads, 8x8 windows, bf16) in one launch, a
// wavefront per head: what heads_bwd.hip is for narrow layers, with one group a launch and a SIMD unit a wave.
//
// Waves 0 .. 2 of a workgroup own a head of the group for all its windows.  A wave recomputes q, k, v and the probabilities of
// a window, forms dO, d(q|k|v) and its head's weight gradients (36 tiles, in registers) and leaves d(q|k|v) in LDS; behind a
// barrier it forms the head's channels of dF = d(q|k|v) Wqkv^T, which are its part of the dx slice.  Wave 3 fetches the rows
// of the next window meanwhile, and lays them down behind that barrier.  Two barriers a window.
//
// What bounds it: the chain of a head's steps, a SIMD unit having one wave (its LDS, 150 KB, and its registers, 506, leave no
// room for a second).  Of the 18 k clocks of a window q, k, v and dO take 5 k, scores to d(q|k|v) 6.5 k, the d(q|k|v) rows 1 k,
// the weight gradients 1.9 k and dF 2.9 k; eight windows a workgroup, 12 k clocks of set-up and 12 k to leave the partial sums.
// What it saves over an adjoint and a gradient launch a group (wide_bwd.hip) is memory: d(q|k|v), F and the cascade gradient
// went out and in between the two, 380 MB a group of 2048 windows against 184 (94 are what the method needs).  Forward + backward
// of 32 / 16 / 1 images of 64x64 333.2 / 202.7 / 117.0 us by those two, 273.4 / 172.0 / 81.7 by heads; with an odd shift, which
// took four launches of one or two heads with a workgroup a window, 32 images 462.2 -> 273.2, an image of 24x16 102.5 -> 73.8.
//
// For two groups: with three a group's two heads would leave half the SIMD units to row fetches, and its launches are three.
//
// Inputs of any size.  q, k, v and the scores come from the operands of the one-launch forward, log2(e) / sqrt(d) in the query
// rows.  From 2^31 elements on the forward is another one with 1 / sqrt(d) there: q is rounded once in either, but not to the
// same values (as with three groups and an odd shift, where the backward is the one with 1 / sqrt(d), fused_bwd.hip).
#include "heads_common.h"
#include "wide_heads_bwd.h"

namespace gswa {

namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kMaskLog2 = -100.0f * kLog2e; // scores are in base-2 units, as the one-launch forward forms them

template <class Cf> struct WideHeadsCfg {
    static constexpr int C = Cf::C, D = Cf::D, CG = Cf::CG, HG = Cf::HG, HEADS = Cf::HEADS, G = Cf::G;
    static constexpr int KS = Cf::KS, KSC = Cf::KSC, KF = (3 * D + 31) / 32; // K = 32 steps over a head's 3 D features
    static_assert(Cf::ET == 2 && HG == 3, "three heads of 17 .. 32 channels");
    static constexpr int THREADS = 64 * (HG + 1);
    static constexpr int NTBL = 225, NDLT = 7;
    static constexpr int CT = CG / 16 + 1, RT = (3 * D + 15) / 16;     // tiles of a head's d w_qkv; column CG carries the bias sums
    // d(q|k|v) of a head: rows of one token, 3 D features, their pitch a multiple of 16 bytes that spreads 16 rows over the
    // banks.  A result tile's padding falls on features that are written after it, or behind the last.
    static constexpr int DQ_ROW = 104, DQ_HEAD = 64 * DQ_ROW;
    static_assert(32 * KF <= DQ_ROW && 2 * D + 32 <= DQ_ROW && DQ_ROW % 8 == 0, "padding inside the row");
    static constexpr size_t OFF_WQ = 0, SZ_WQ = (size_t)HG * 3 * 2 * KS * 1024;
    static constexpr size_t OFF_F = OFF_WQ + SZ_WQ, SZ_F = (size_t)KS * 4096;
    static constexpr size_t OFF_DY = OFF_F + SZ_F, SZ_DY = (size_t)KSC * 4096;
    static constexpr size_t OFF_DQ = OFF_DY + SZ_DY, SZ_DQ = (size_t)HG * DQ_HEAD * 2;
    static constexpr size_t OFF_TURN = OFF_DQ + SZ_DQ, SZ_TURN = 12 * 512;   // a wave's tiles on their way to the other orientation
    static constexpr size_t OFF_BIAS = OFF_TURN + HG * SZ_TURN;              // fp32 [head][q, k, v][32]
    static constexpr size_t OFF_TOK = OFF_BIAS + (size_t)HG * 96 * 4;        // token of a lane, of this window and of the next
    static constexpr size_t OFF_FLAG = OFF_TOK + 2 * 64 * 4;
    static constexpr size_t OFF_END = OFF_FLAG + 16;
    static constexpr int TP = 17;
    static constexpr size_t SZ_FOLD = (size_t)HG * NDLT * 16 * TP * 4;
    static constexpr size_t LDS_BYTES = OFF_END > SZ_FOLD ? OFF_END : SZ_FOLD;
    static_assert(LDS_BYTES <= 160 * 1024, "LDS budget");
    // partial sums of a workgroup: rows of w_qkv of the group, their biases, the table of its heads
    static constexpr int L_DW = 0, L_DB = 3 * CG * CG, L_TBL = L_DB + 3 * CG, L_END = L_TBL + HG * NTBL;
    static constexpr int L_TOTAL = (L_END + 3) & ~3;
};

template <class Cf, int GI>
__global__ __launch_bounds__(WideHeadsCfg<Cf>::THREADS, 1) void wide_heads_bwd_kernel(Geom g, const bf16_t *__restrict__ x,
                                                                                     const bf16_t *__restrict__ dy,
                                                                                     const bf16_t *__restrict__ attn,
                                                                                     const uint8_t *__restrict__ pack,
                                                                                     const bf16_t *__restrict__ table, bf16_t *dx,
                                                                                     float *__restrict__ part)
{
    using P = WideHeadsCfg<Cf>;
    constexpr int C = P::C, D = P::D, CG = P::CG, HG = P::HG, HEADS = P::HEADS, KS = P::KS, KSC = P::KSC, KF = P::KF;
    constexpr int M = 8, CT = P::CT, RT = P::RT;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const uint4 *wq = reinterpret_cast<const uint4 *>(lds + P::OFF_WQ);
    uint4 *fb = reinterpret_cast<uint4 *>(lds + P::OFF_F);
    uint4 *dyb = reinterpret_cast<uint4 *>(lds + P::OFF_DY);
    uint16_t *dqb = reinterpret_cast<uint16_t *>(lds + P::OFF_DQ);
    const float *bqkv = reinterpret_cast<const float *>(lds + P::OFF_BIAS);
    uint32_t *tokb = reinterpret_cast<uint32_t *>(lds + P::OFF_TOK);
    int *flagb = reinterpret_cast<int *>(lds + P::OFF_FLAG);
    bf16_t *tbl = reinterpret_cast<bf16_t *>(lds + P::OFF_DQ); // the bias table, during the set-up

    const int tid = threadIdx.x;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int s = g.shift;
    const int cnt = (g.nW - (int)blockIdx.x + (int)gridDim.x - 1) / (int)gridDim.x; // windows blockIdx.x + m gridDim.x, m < cnt
    const bool casc_in = GI > 0 && g.cascade, casc_out = GI < Cf::G - 1 && g.cascade;

    // ---- set-up: weights, biases and the table to LDS, all loads in flight together ----
    auto setup = [&](int tid) {
        constexpr int TH = P::THREADS, NW = TH / 64, N1K = (int)(P::SZ_WQ / 1024);
        constexpr int I_B = (HG * 96 + TH - 1) / TH;
        const int lane = tid & 63;
#pragma unroll
        for (int k = 0; k < (N1K + NW - 1) / NW; ++k) {
            const int f = k * NW + wv;
            if (f < N1K) lds_dma16(pack + Cf::P_WQN + ((size_t)GI * N1K + f) * 1024 + 16 * lane, lds + P::OFF_WQ + (size_t)f * 1024);
        }
        float bv[I_B];
        TableCopy<P::NTBL * HEADS, TH> tc;
#pragma unroll
        for (int k = 0; k < I_B; ++k) {
            const int i = k * TH + tid < HG * 96 ? k * TH + tid : 0, e = i % 32, t = i / 32 % 3, hl = i / 96;
            bv[k] = reinterpret_cast<const float *>(pack + Cf::P_BIAS)[GI * 3 * CG + t * CG + hl * D + (e < D ? e : 0)];
            bv[k] = e < D ? (t == 0 ? bv[k] * kLog2e : bv[k]) : 0.f;
        }
        tc.fetch(table, tid);
#pragma unroll
        for (int k = 0; k < I_B; ++k)
            if (k * TH + tid < HG * 96) reinterpret_cast<float *>(lds + P::OFF_BIAS)[k * TH + tid] = bv[k];
        tc.store(tbl, tid);
        __builtin_amdgcn_s_waitcnt(0);
    };

    if (wv == HG) {
        int lane_h = threadIdx.x & 63; // (opaque: nothing of this branch is kept through the other)
        asm volatile("" : "+v"(lane_h));
        const int lane = lane_h, l16 = lane & 15, q = lane >> 4;
        const int per_img = g.nwi * g.nwj;
        const float r_img = 1.0f / (float)per_img, r_nwj = 1.0f / (float)g.nwj;
        uint4 rx[4][KS], ra[4][KS], rdy[4][KSC]; // as loaded: partial pieces still unshifted
        uint32_t rtok[4];
        int rflag = 0;
        auto load_rows = [&](int m) {
            const int win = (int)blockIdx.x + m * (int)gridDim.x;
            const int b = quotient(win, per_img, r_img), wr = win - b * per_img;
            const int wi = quotient(wr, g.nwj, r_nwj), wj = wr - wi * g.nwj;
            rflag = s > 0 ? (wi == g.nwi - 1 ? 1 : 0) | (wj == g.nwj - 1 ? 2 : 0) : 0;
            int sj = wj * M + (l16 & 7) + s;
            if (sj >= g.W) sj -= g.W;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                int si = wi * M + 2 * t + (l16 >> 3) + s;
                if (si >= g.H) si -= g.H;
                const long tok = ((long)b * g.H + si) * g.W + sj;
                rtok[t] = (uint32_t)tok;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    rx[t][ks] = load_piece4<CG>(x + tok * C + GI * CG, 32 * ks + 8 * q);
                    if (casc_in) ra[t][ks] = load_piece4<CG>(attn + tok * C + (GI > 0 ? GI - 1 : 0) * CG, 32 * ks + 8 * q);
                }
#pragma unroll
                for (int ks = 0; ks < KSC; ++ks) rdy[t][ks] = load_piece4<C>(dy + tok * C, 32 * ks + 8 * q);
            }
        };
        auto stage = [&](int m) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
#pragma unroll
                for (int ks = 0; ks < KSC; ++ks) dyb[(ks * 4 + t) * 64 + lane] = piece4<C>(rdy[t][ks], 32 * ks, q);
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    uint4 f = piece4<CG>(rx[t][ks], 32 * ks, q);
                    if (casc_in) f = add_bf16x8(f, piece4<CG>(ra[t][ks], 32 * ks, q));
                    f = with_bias_slot<CG>(f, ks, q);
                    fb[(ks * 4 + t) * 64 + lane] = f;
                }
                if (q == 0) tokb[(m & 1) * 64 + 16 * t + l16] = rtok[t];
            }
            if (lane == 0) flagb[m & 1] = rflag;
        };
        load_rows(0);
        setup(HG * 64 + lane);
        stage(0);
        __syncthreads();
        __syncthreads();
        for (int m = 0; m < cnt; ++m) {
            // The heads' own loads of this window go first: they are waited for at once, these rows a window later.  (Sleeping
            // 0 / 6 / 12 / 24 / 48 / 96, 64 clocks each, of a window's 18 k: 32 images of 64x64, forward + backward, 273.9 /
            // 271.4 / 270.5 / 269.1 / 268.7 / 269.2 us, 16 images 168.6 / 167.4 / 167.4 / 165.9 / 165.4 / 166.1; eight and fewer,
            // with one or two windows a workgroup, within their noise.)
            __builtin_amdgcn_s_sleep(24);
            if (m + 1 < cnt) load_rows(m + 1);
            __syncthreads();
            if (m + 1 < cnt) stage(m + 1);
            __syncthreads();
        }
        return;
    }

    setup(tid);
    __syncthreads();
    const int hl = wv, hd = GI * HG + hl;
    f32x4 bias_t[P::NDLT], tblacc[P::NDLT], dwacc[RT][CT];
    {
        const int lane = tid & 63, l16 = lane & 15, q = lane >> 4;
#pragma unroll
        for (int dl = 0; dl < P::NDLT; ++dl) {
            const int dr = (l16 >> 3) - (q >> 1) - 2 * (dl - 3);
#pragma unroll
            for (int j = 0; j < 4; ++j)
                bias_t[dl][j] = to_f32(tbl[((dr + M - 1) * (2 * M - 1) + (l16 & 7) - 4 * (q & 1) - j + M - 1) * HEADS + hd]) * kLog2e;
            tblacc[dl] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) dwacc[rt][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    __syncthreads();
    const f32x4 zero = f32x4{0.f, 0.f, 0.f, 0.f};
    uint2 *turn = reinterpret_cast<uint2 *>(lds + P::OFF_TURN + hl * P::SZ_TURN);
    uint16_t *dq = dqb + hl * P::DQ_HEAD;
    // the places behind the last tile's padding, which dF's last step reads against zeros, are written here only
    static_assert(2 * D + 32 == 92 && 32 * KF == 96, "what a row's tiles leave");
    *reinterpret_cast<uint2 *>(dq + (tid & 63) * P::DQ_ROW + 92) = make_uint2(0u, 0u);

    for (int m = 0; m < cnt; ++m) {
        int lane_n = tid & 63; // (opaque: the many per-lane addresses are made where they are used)
        asm volatile("" : "+v"(lane_n));
        const int lane = lane_n, l16 = lane & 15, q = lane >> 4;
        const int tr = (l16 & 3) * 16 + 4 * q + (l16 >> 2);
        const uint8_t *ftr = lds + P::OFF_F + ((l16 & 3) >> 1) * 256 + (l16 & 1) * 8 + (4 * q + (l16 >> 2)) * 16;
        uint32_t tok[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) tok[t] = tokb[(m & 1) * 64 + 16 * t + l16];
        const int flags = __builtin_amdgcn_readfirstlane(flagb[m & 1]);

        // ---- dO^T of the head: adjoint of Eq. 7 plus the gradient through Eq. 8, the next group's dx slice ----
        uint2 dOb[2][4], Qb[2][4], Kb[2][4], Vb[2][4];
        {
            // (taken as loaded, from where a piece ends with the head at the latest, and put right where they are used: a
            // select behind a load is a wait behind it)
            uint2 cg[2][4];
#pragma unroll
            for (int et = 0; et < 2; ++et)
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int c = 16 * et + 4 * q, at = c < D - 4 ? c : D - 4;
                    const uint32_t *src = reinterpret_cast<const uint32_t *>(dx + (size_t)tok[t] * C + (GI + 1) * CG + hl * D + at);
                    cg[et][t] = make_uint2(0u, 0u);
                    if (casc_out) cg[et][t] = make_uint2(src[0], src[1]);
                }
            const uint4 *wo = reinterpret_cast<const uint4 *>(pack + Cf::P_WPT) + (size_t)hd * 2 * KSC * 64 + lane;
            uint4 w[2][KSC];
#pragma unroll
            for (int et = 0; et < 2; ++et)
#pragma unroll
                for (int ks = 0; ks < KSC; ++ks) w[et][ks] = wo[(et * KSC + ks) * 64];
            // q, k, v while these are on their way
            uint4 f[4][KS];
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) f[t][ks] = fb[(ks * 4 + t) * 64 + lane];
            // (fragments of a step are read under the products of the step before: left alone, the compiler reads one and
            // waits for it)
            uint4 wf[2][KS];
            f32x4 bias[2];
            auto fetch_w = [&](int i) { // i = 2 t3 + et
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) wf[i & 1][ks] = wq[((hl * 6 + i) * KS + ks) * 64 + lane];
                bias[i & 1] = *reinterpret_cast<const f32x4 *>(bqkv + (hl * 3 + i / 2) * 32 + 16 * (i % 2) + 4 * q);
            };
            uint4 dyf[2][4];
            auto fetch_dy = [&](int ks) {
#pragma unroll
                for (int t = 0; t < 4; ++t) dyf[ks & 1][t] = dyb[(ks * 4 + t) * 64 + lane];
            };
            fetch_w(0);
#pragma unroll
            for (int i = 0; i < 6; ++i) {
                if (i + 1 < 6) fetch_w(i + 1);
                else fetch_dy(0);
                __builtin_amdgcn_sched_barrier(0x6);
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    f32x4 r = bias[i & 1];
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) r = mma32(wf[i & 1][ks], f[t][ks], r);
                    (i < 2 ? Qb : i < 4 ? Kb : Vb)[i % 2][t] = pack_bf16x4(r);
                }
            }
            f32x4 acc[2][4];
#pragma unroll
            for (int et = 0; et < 2; ++et)
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int c = 16 * et + 4 * q;
                    const uint32_t lo = c <= D - 4 ? cg[et][t].x : c < D ? cg[et][t].y : 0u, hi = c <= D - 4 ? cg[et][t].y : 0u;
                    acc[et][t] = f32x4{bf16_lo(lo), bf16_hi(lo), bf16_lo(hi), bf16_hi(hi)};
                }
#pragma unroll
            for (int ks = 0; ks < KSC; ++ks) {
                if (ks + 1 < KSC) fetch_dy(ks + 1);
                __builtin_amdgcn_sched_barrier(0x6);
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    acc[0][t] = mma32(w[0][ks], dyf[ks & 1][t], acc[0][t]);
                    acc[1][t] = mma32(w[1][ks], dyf[ks & 1][t], acc[1][t]);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int et = 0; et < 2; ++et)
#pragma unroll
                for (int t = 0; t < 4; ++t) dOb[et][t] = pack_bf16x4(acc[et][t]);
        }
        // a tile of d q, d k or d v (t3 = 0, 1, 2, written in this order) into the rows of its tokens
        auto put = [&](int t3, int et, int tt, f32x4 v) {
            const uint2 p = pack_bf16x4(v);
            uint32_t *dst = reinterpret_cast<uint32_t *>(dq + (16 * tt + l16) * P::DQ_ROW + t3 * D + 16 * et + 4 * q);
            dst[0] = p.x;
            dst[1] = p.y;
        };
        f32x4 dk[2][4], dv[2][4];
        auto attention = [&](auto masked) {
            constexpr bool MASK = decltype(masked)::value;
            uint2 KT[2][4];
#pragma unroll
            for (int et = 0; et < 2; ++et)
#pragma unroll
                for (int kt = 0; kt < 4; ++kt) turn[(et * 4 + kt) * 64 + lane] = Kb[et][kt];
#pragma unroll
            for (int et = 0; et < 2; ++et)
#pragma unroll
                for (int kt = 0; kt < 4; ++kt) KT[et][kt] = lds_read_tr(turn + (et * 4 + kt) * 64 + tr);
#pragma unroll
            for (int et = 0; et < 2; ++et)
#pragma unroll
                for (int kt = 0; kt < 4; ++kt) dk[et][kt] = dv[et][kt] = zero;
            // two tiles of queries at a time, every stage for both: two chains that fill each other's waits
#pragma unroll
            for (int p2 = 0; p2 < 2; ++p2) {
                uint4 qn[2], on[2];
#pragma unroll
                for (int i = 0; i < 4; ++i) turn[(8 + i) * 64 + lane] = Qb[i / 2][2 * p2 + i % 2];
#pragma unroll
                for (int et = 0; et < 2; ++et) qn[et] = cat(lds_read_tr(turn + (8 + 2 * et) * 64 + tr), lds_read_tr(turn + (9 + 2 * et) * 64 + tr));
#pragma unroll
                for (int i = 0; i < 4; ++i) turn[(8 + i) * 64 + lane] = dOb[i / 2][2 * p2 + i % 2];
#pragma unroll
                for (int et = 0; et < 2; ++et) on[et] = cat(lds_read_tr(turn + (8 + 2 * et) * 64 + tr), lds_read_tr(turn + (9 + 2 * et) * 64 + tr));
                f32x4 st[2][4], dp[2][4];
#pragma unroll
                for (int ni = 0; ni < 2; ++ni) {
                    const int qt = 2 * p2 + ni;
                    const uint4 qop = cat(Qb[0][qt], Qb[1][qt]), oop = cat(dOb[0][qt], dOb[1][qt]);
#pragma unroll
                    for (int kt = 0; kt < 4; ++kt) {
                        st[ni][kt] = mma32(cat(Kb[0][kt], Kb[1][kt]), qop, bias_t[kt - qt + 3]);
                        dp[ni][kt] = mma32(cat(Vb[0][kt], Vb[1][kt]), oop, zero);
                    }
                }
                if (MASK) {
#pragma unroll
                    for (int ni = 0; ni < 2; ++ni) {
                        const bool qr = 2 * (2 * p2 + ni) + (l16 >> 3) >= M - s, qc = (l16 & 7) >= M - s;
#pragma unroll
                        for (int kt = 0; kt < 4; ++kt) {
                            const bool row = (flags & 1) && qr != (2 * kt + (q >> 1) >= M - s);
#pragma unroll
                            for (int j = 0; j < 4; ++j)
                                st[ni][kt][j] += row || ((flags & 2) && qc != (4 * (q & 1) + j >= M - s)) ? kMaskLog2 : 0.f;
                        }
                    }
                }
                float top[2], inv[2], delta[2];
#pragma unroll
                for (int ni = 0; ni < 2; ++ni) {
                    float mx = max4f(st[ni][0]);
#pragma unroll
                    for (int kt = 1; kt < 4; ++kt) mx = max5f(mx, st[ni][kt]);
                    top[ni] = mx;
                }
#pragma unroll
                for (int ni = 0; ni < 2; ++ni) top[ni] = qgroup_max(top[ni]);
#pragma unroll
                for (int ni = 0; ni < 2; ++ni) {
                    f32x4 sum4, del4;
#pragma unroll
                    for (int kt = 0; kt < 4; ++kt) {
#pragma unroll
                        for (int j = 0; j < 4; ++j) st[ni][kt][j] = __builtin_amdgcn_exp2f(st[ni][kt][j] - top[ni]);
                        sum4 = kt == 0 ? st[ni][0] : sum4 + st[ni][kt];
                        if (kt == 0) del4 = st[ni][0] * dp[ni][0];
                        else
#pragma unroll
                            for (int j = 0; j < 4; ++j) del4[j] = fmaf(st[ni][kt][j], dp[ni][kt][j], del4[j]);
                    }
                    inv[ni] = (sum4[0] + sum4[1]) + (sum4[2] + sum4[3]);
                    delta[ni] = (del4[0] + del4[1]) + (del4[2] + del4[3]);
                }
#pragma unroll
                for (int ni = 0; ni < 2; ++ni) inv[ni] = recip(qgroup_sum(inv[ni]));
#pragma unroll
                for (int ni = 0; ni < 2; ++ni) delta[ni] = inv[ni] * qgroup_sum(delta[ni]);
                uint2 dSb[2][4], pn[2][4];
#pragma unroll
                for (int ni = 0; ni < 2; ++ni)
#pragma unroll
                    for (int kt = 0; kt < 4; ++kt) {
                        st[ni][kt] *= inv[ni];
                        turn[(ni * 4 + kt) * 64 + lane] = pack_bf16x4(st[ni][kt]);
                    }
#pragma unroll
                for (int ni = 0; ni < 2; ++ni)
#pragma unroll
                    for (int kt = 0; kt < 4; ++kt) {
                        pn[ni][kt] = lds_read_tr(turn + (ni * 4 + kt) * 64 + tr);
#pragma unroll
                        for (int j = 0; j < 4; ++j) dp[ni][kt][j] = st[ni][kt][j] * (dp[ni][kt][j] - delta[ni]);
                        dSb[ni][kt] = pack_bf16x4(dp[ni][kt]);
                        tblacc[kt - 2 * p2 - ni + 3] += dp[ni][kt];
                    }
#pragma unroll
                for (int ni = 0; ni < 2; ++ni)
#pragma unroll
                    for (int kt = 0; kt < 4; ++kt) turn[(ni * 4 + kt) * 64 + lane] = dSb[ni][kt];
                __builtin_amdgcn_sched_barrier(0);
                uint2 sn[2][4];
#pragma unroll
                for (int ni = 0; ni < 2; ++ni)
#pragma unroll
                    for (int kt = 0; kt < 4; ++kt) sn[ni][kt] = lds_read_tr(turn + (ni * 4 + kt) * 64 + tr);
#pragma unroll
                for (int ni = 0; ni < 2; ++ni)
#pragma unroll
                    for (int et = 0; et < 2; ++et)
                        put(0, et, 2 * p2 + ni, mma32(cat(KT[et][2], KT[et][3]), cat(dSb[ni][2], dSb[ni][3]), mma32(cat(KT[et][0], KT[et][1]), cat(dSb[ni][0], dSb[ni][1]), zero)));
#pragma unroll
                for (int et = 0; et < 2; ++et)
#pragma unroll
                    for (int kt = 0; kt < 4; ++kt) {
                        dv[et][kt] = mma32(on[et], cat(pn[0][kt], pn[1][kt]), dv[et][kt]);
                        dk[et][kt] = mma32(qn[et], cat(sn[0][kt], sn[1][kt]), dk[et][kt]);
                    }
            }
        };
        if (flags) attention(std::true_type{});
        else attention(std::false_type{});
        // (the padding of one tile and the features of the next are places of different lanes: only the order of the writes,
        // which a wave's LDS accesses keep, says which of them stays, so the compiler must keep it too)
        asm volatile("" ::: "memory");
#pragma unroll
        for (int et = 0; et < 2; ++et)
#pragma unroll
            for (int kt = 0; kt < 4; ++kt) put(1, et, kt, dk[et][kt] * (1.0f / kLog2e)); // (Q carries log2(e))
        asm volatile("" ::: "memory");
#pragma unroll
        for (int et = 0; et < 2; ++et)
#pragma unroll
            for (int kt = 0; kt < 4; ++kt) put(2, et, kt, dv[et][kt]);
        // this head's channels of Wqkv^T, on their way under the weight gradients
        uint4 wy[2][HG][KF];
        {
            const uint4 *src = reinterpret_cast<const uint4 *>(pack + Cf::P_WQY) + (size_t)hd * 2 * HG * KF * 64 + lane;
#pragma unroll
            for (int et = 0; et < 2; ++et)
#pragma unroll
                for (int h = 0; h < HG; ++h)
#pragma unroll
                    for (int ks = 0; ks < KF; ++ks) wy[et][h][ks] = src[((et * HG + h) * KF + ks) * 64];
        }
        // ---- d w_qkv (and d b_qkv in the spare column) ----
#pragma unroll
        for (int kp = 0; kp < 2; ++kp) {
            uint4 f[CT];
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                const uint8_t *at = ftr + (((ct >> 1) * 4 + 2 * kp) * 64 + (ct & 1) * 32) * 16;
                f[ct] = cat(lds_read_tr(at), lds_read_tr(at + 1024));
            }
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                const uint16_t *at = dq + (32 * kp + 4 * q + (l16 >> 2)) * P::DQ_ROW + 16 * rt + 4 * (l16 & 3);
                const uint4 a = cat(lds_read_tr(at), lds_read_tr(at + 16 * P::DQ_ROW));
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) dwacc[rt][ct] = mma32(a, f[ct], dwacc[rt][ct]);
            }
        }
        __syncthreads();
        // ---- dF of the group, this head's channels: the dx slice ----
        {
            const uint16_t *src = dqb + l16 * P::DQ_ROW + 8 * q;
            f32x4 acc[2][4];
#pragma unroll
            for (int et = 0; et < 2; ++et)
#pragma unroll
                for (int t = 0; t < 4; ++t) acc[et][t] = zero;
            uint4 b[2][4];
            auto fetch = [&](int i) { // i = head of the group, K step
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    b[i & 1][t] = *reinterpret_cast<const uint4 *>(src + i / KF * P::DQ_HEAD + 16 * t * P::DQ_ROW + 32 * (i % KF));
            };
            fetch(0);
#pragma unroll
            for (int i = 0; i < HG * KF; ++i) {
                if (i + 1 < HG * KF) fetch(i + 1);
                __builtin_amdgcn_sched_barrier(0x6);
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    acc[0][t] = mma32(wy[0][i / KF][i % KF], b[i & 1][t], acc[0][t]);
                    acc[1][t] = mma32(wy[1][i / KF][i % KF], b[i & 1][t], acc[1][t]);
                }
            }
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int et = 0; et < 2; ++et) {
                    const int c = 16 * et + 4 * q;
                    uint32_t *dst = reinterpret_cast<uint32_t *>(dx + (size_t)tok[t] * C + GI * CG + hl * D + c);
                    const uint2 v = pack_bf16x4(acc[et][t]);
                    if (c < D) dst[0] = v.x;
                    if (c + 2 < D) dst[1] = v.y;
                }
        }
        __syncthreads();
    }

    // ---- this workgroup's partial sums.  The packed query weights carry 1/sqrt(d), so their gradients get it back here ----
    float *mine = part + (size_t)blockIdx.x * P::L_TOTAL;
    int lane_e = tid & 63;
    asm volatile("" : "+v"(lane_e));
    const int lane = lane_e, l16 = lane & 15, q = lane >> 4;
    const float scale = 1.0f / sqrtf((float)D);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int u = 16 * rt + 4 * q + j, t3 = u / D; // feature u of the head
            const int row = t3 * CG + hl * D + u - t3 * D;
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                const int c = 16 * ct + l16;
                const float v = t3 == 0 ? dwacc[rt][ct][j] * scale : dwacc[rt][ct][j];
                if (u < 3 * D && c <= CG) mine[c < CG ? P::L_DW + row * CG + c : P::L_DB + row] = v;
            }
        }
    // the wave's own piece: no other wave reads or writes it any more (the last barrier is behind the last read of LDS)
    float *mat = reinterpret_cast<float *>(lds) + hl * P::NDLT * 16 * P::TP;
#pragma unroll
    for (int dl = 0; dl < P::NDLT; ++dl)
#pragma unroll
        for (int j = 0; j < 4; ++j) mat[(dl * 16 + 4 * q + j) * P::TP + l16] = tblacc[dl][j];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int k = 0; k < (P::NTBL + 63) / 64; ++k) {
        const int e = 64 * k + lane < P::NTBL ? 64 * k + lane : P::NTBL - 1;
        const float a = table_entry<P::TP>(mat, e);
        if (64 * k + lane < P::NTBL) mine[P::L_TBL + hl * P::NTBL + e] = a;
    }
}

template <class Cf, int GI>
hipError_t run_group(const Geom &g, int grid, const bf16_t *x, const bf16_t *dy, const bf16_t *attn, const uint8_t *pack,
                     const bf16_t *table, bf16_t *dx, float *dw_qkv, float *db_qkv, float *dtable, int accumulate, float *part,
                     ReduceJob &last, hipStream_t s)
{
    using P = WideHeadsCfg<Cf>;
    auto kern = wide_heads_bwd_kernel<Cf, GI>;
    if (hipError_t ea = allow_dynamic_lds(reinterpret_cast<const void *>(kern), P::LDS_BYTES); ea != hipSuccess) return ea;
    {
        KernelTimer kt(K_WIDE_ATTN_BWD, s);
        hipLaunchKernelGGL(kern, dim3(grid), dim3(P::THREADS), P::LDS_BYTES, s, g, x, dy, attn, pack, table, dx, part);
    }
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    ReduceOut out{};
    out.ptr[0] = dw_qkv + (size_t)GI * 3 * Cf::CG * Cf::CG; out.begin[0] = P::L_DW;
    out.ptr[1] = db_qkv + GI * 3 * Cf::CG; out.begin[1] = P::L_DB;
    out.ptr[2] = dtable; out.begin[2] = P::L_TBL;
    out.begin[3] = P::L_END;
    out.nseg = 3;
    out.tbl_heads = P::HG; out.tbl_entries = P::NTBL; out.tbl_stride = P::HEADS; out.tbl_head0 = GI * P::HG;
    if constexpr (GI > 0) { // (the first group's sum shares a launch with the projection's)
        if (hipError_t e = launch_reduce(part, grid, P::L_TOTAL, out, accumulate, s); e != hipSuccess) return e;
        return run_group<Cf, GI - 1>(g, grid, x, dy, attn, pack, table, dx, dw_qkv, db_qkv, dtable, accumulate, part, last, s);
    }
    last.part = part; last.nparts = grid; last.n = P::L_TOTAL; last.out = out; last.accumulate = accumulate;
    return hipSuccess;
}

} // namespace

using Shape = FusedCfg<180, 6, 2>;

bool wide_heads_bwd_supported(const Geom &g)
{
    return g.M == 8 && g.C == Shape::C && g.heads == Shape::HEADS && g.groups == Shape::G && g.dq == g.d;
}

// The projection's partial vectors go there where a scratch of 36 KB a window (the d(q|k|v) of a group, which the launches of
// wide_bwd.hip hand over) has room for them, from 905 windows on; fewer windows pay one more sum instead of 33 MB of scratch.
size_t wide_heads_bwd_free_bytes(const Geom &g)
{
    const size_t room = (size_t)g.nW * 4 * Shape::HG * 3 * 1024;
    const size_t wproj = ((size_t)kSizingCus * (Shape::C * Shape::C + Shape::C) * sizeof(float) + 255) & ~size_t(255);
    return room < wproj ? room : wproj;
}

size_t wide_heads_bwd_ws_bytes(const Geom &g)
{
    const int grid = g.nW < kSizingCus ? g.nW : kSizingCus;
    return wide_heads_bwd_free_bytes(g) + (((size_t)grid * WideHeadsCfg<Shape>::L_TOTAL * sizeof(float) + 255) & ~size_t(255));
}

hipError_t launch_wide_heads_bwd(const Geom &g, const bf16_t *x, const bf16_t *dy, const bf16_t *attn, const uint8_t *pack,
                                 const bf16_t *table, bf16_t *dx, float *dw_qkv, float *db_qkv, float *dtable, int accumulate,
                                 void *ws, ReduceJob &last, hipStream_t s)
{
    float *part = reinterpret_cast<float *>(static_cast<uint8_t *>(ws) + wide_heads_bwd_free_bytes(g));
    int grid = device_cu_count();
    if (grid > kSizingCus) grid = kSizingCus;
    if (grid > g.nW) grid = g.nW;
    return run_group<Shape, 1>(g, grid, x, dy, attn, pack, table, dx, dw_qkv, db_qkv, dtable, accumulate, part, last, s);
}

} // namespace gswa
