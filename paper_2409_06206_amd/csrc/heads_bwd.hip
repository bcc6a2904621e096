// Backward of a narrow attention layer (C = 60, six heads, 8x8 windows, bf16; one, two or three groups) in one launch, a
// wavefront per head.
//
// A workgroup has eight waves.  Wave h < 6 owns head h for all windows of the workgroup: it recomputes q, k, v and the
// probabilities of a window's 64 tokens, forms their gradients and keeps the head's parameter gradients in registers.
// What a step leaves for a later one in the other orientation goes through the wave's own piece of LDS and is read back
// turned (lds_read_tr), so nothing of a score waits for another wave.  Waves 6 and 7 fetch the rows a window ahead, lay them
// down as operands in LDS and form the projection's gradient and dF of the first group, each for half of the tokens.
//
// The heads of a group meet in dF = d(q|k|v) Wqkv^T only.  They leave d(q|k|v) in LDS (two buffers in turn), and one window
// later the wave of head hl in the group before forms the channels of dF that feed its own dO (Eq. 8): the groups run as a
// pipeline, group g one window behind group g + 1, with one barrier per window.
//
// T-form, N-form and the operand conventions: fused_bwd.hip, mfma.h.
#include "heads_bwd.h"
#include "heads_common.h"

namespace gswa {

namespace {

constexpr float kLog2e = 1.4426950408889634f;
// the shift mask as the forward of narrow layers adds it (fused_bwd.hip)
constexpr float kMask = -144.0f / kLog2e;

template <class Cf> struct HeadsCfg {
    static constexpr int C = Cf::C, D = Cf::D, CG = Cf::CG, HG = Cf::HG, HEADS = Cf::HEADS, G = Cf::G;
    static constexpr int KS = Cf::KS, KSC = Cf::KSC;
    static_assert(Cf::ET == 1 && HEADS == 6 && C <= 64, "narrow heads");
    static constexpr int HELPERS = 2, THREADS = 64 * (HEADS + HELPERS);
    static constexpr int NTBL = 225;
    static constexpr int NDLT = 7;                       // key tile - query tile + 3
    static constexpr int CT = CG / 16 + 1;               // column tiles of d w_qkv; the spare column CG carries the bias sums
    static constexpr int OTP = (C + 15) / 16, CTP = C / 16 + 1;
    // window m of a workgroup is written to the row buffers while window m - 1 enters the pipeline, and leaves group g
    // G - 1 - g windows later
    static constexpr int DY_SLOTS = G + 1;
    static constexpr int f_slots(int gi) { return G + 1 - gi; }
    static constexpr int f_first(int gi) { int n = 0; for (int i = 0; i < gi; ++i) n += f_slots(i); return n; }
    static constexpr int TOK_SLOTS = 8;
    static_assert(TOK_SLOTS > G + 1, "a window's tokens are needed until its dF has left");
    // d(q|k|v) of a head: rows of one token, the 3 D features, their pitch 80 bytes (16-byte pieces of 16 rows on different
    // banks).  A result tile's padding (rows D .. 15) falls on features that are written after it, or behind the last.
    static constexpr int DQ_ROW = 40, DQ_HEAD = 64 * DQ_ROW;          // entries of two bytes
    static_assert(3 * D <= 32 && 2 * D + 16 <= DQ_ROW, "padding inside the row");
    static constexpr size_t SZ_DQ = (size_t)HEADS * DQ_HEAD * 2;
    static constexpr int RT = 2;                                      // row tiles of a head's d w_qkv
    // F and dy as operands, lane by lane.  Of F's lane groups only those that hold channels are stored; the last reads the
    // place of another, against zeros in the weights.
    static constexpr int FL = KS == 1 && CG < 24 ? 48 : 64;
    static constexpr size_t SZ_F = (size_t)KS * 4 * FL * 16, SZ_DY = (size_t)KSC * 4 * 1024;
    static constexpr size_t SZ_WPT = (size_t)Cf::N_WPT * 1024;
    static constexpr size_t SZ_TURN = 6 * 512;                        // a wave's tiles on their way to the other orientation
    static constexpr size_t OFF_DQ = 0;
    static constexpr size_t OFF_F = OFF_DQ + 2 * SZ_DQ;
    static constexpr size_t OFF_DY = OFF_F + f_first(G) * SZ_F;
    static constexpr size_t OFF_WPT = OFF_DY + DY_SLOTS * SZ_DY;
    static constexpr size_t OFF_BIAS = OFF_WPT + SZ_WPT;              // fp32 [head][q, k, v][16]
    static constexpr size_t OFF_TURN = OFF_BIAS + (size_t)HEADS * 48 * 4;
    static constexpr size_t OFF_TOK = OFF_TURN + HEADS * SZ_TURN;
    static constexpr size_t OFF_FLAG = OFF_TOK + TOK_SLOTS * 64 * 4;
    static constexpr size_t OFF_TBL = OFF_DQ;                         // the bias table, during the set-up
    static constexpr size_t OFF_END = OFF_FLAG + TOK_SLOTS * 4;
    static constexpr size_t LDS_MAX = 160 * 1024;
    // after the last window: bias-table tiles per head, one half of d w_proj
    static constexpr int TP = 17;                                     // pitch of a tile's rows
    static constexpr size_t SZ_FOLD = (size_t)HEADS * NDLT * 16 * TP * 4, SZ_WP = (size_t)OTP * CTP * 1024;
    static constexpr size_t LDS_BYTES = OFF_END > SZ_FOLD + SZ_WP ? OFF_END : SZ_FOLD + SZ_WP;
    static_assert(LDS_BYTES <= LDS_MAX, "LDS budget");
    // partial sums of a workgroup, in parameter order
    static constexpr int L_DWQ = 0, L_DBQ = L_DWQ + 3 * C * CG, L_DWP = L_DBQ + 3 * C, L_DBP = L_DWP + C * C;
    static constexpr int L_TBL = L_DBP + C, L_END = L_TBL + HEADS * NTBL, L_TOTAL = (L_END + 3) & ~3;
};

constexpr bool overlap(int a0, int a1, int b0, int b1) { return a0 < b1 && b0 < a1; }

// What bounds it: six heads on four SIMD units, so two units issue the steps of two heads, 12.5 k clocks a window where a head
// alone takes 10 k (four query tiles of 1.6 k, 3 k before and 1 k behind them); most of a tile is the chain products -> softmax
// -> products.  Against launches per head group with a window in four waves and three barriers a head: 32 images of 64x64, 60
// channels, forward + backward, 1 / 2 / 3 groups 160.4 / 128.6 / 138.8 -> 97.6 / 90.7 / 95.7 us; one image, two groups, 46.4 ->
// 31.6.
template <class Cf>
__global__ __launch_bounds__(HeadsCfg<Cf>::THREADS, 2) void heads_bwd_kernel(Geom g, const bf16_t *__restrict__ x,
                                                                            const bf16_t *__restrict__ dy,
                                                                            const bf16_t *__restrict__ attn,
                                                                            const uint8_t *__restrict__ pack,
                                                                            const bf16_t *__restrict__ table, bf16_t *dx,
                                                                            float *__restrict__ part)
{
    using P = HeadsCfg<Cf>;
    constexpr int C = P::C, D = P::D, CG = P::CG, HG = P::HG, HEADS = P::HEADS, G = P::G, KS = P::KS, KSC = P::KSC;
    constexpr int M = 8, CT = P::CT, OTP = P::OTP, CTP = P::CTP;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    uint16_t *dqb = reinterpret_cast<uint16_t *>(lds + P::OFF_DQ);
    uint4 *fb = reinterpret_cast<uint4 *>(lds + P::OFF_F);
    uint4 *dyb = reinterpret_cast<uint4 *>(lds + P::OFF_DY);
    const uint4 *wq = reinterpret_cast<const uint4 *>(pack + Cf::P_WQ);
    const uint4 *wpt = reinterpret_cast<const uint4 *>(lds + P::OFF_WPT);
    bf16_t *tbl = reinterpret_cast<bf16_t *>(lds + P::OFF_TBL);
    const float *bqkv = reinterpret_cast<const float *>(lds + P::OFF_BIAS);
    uint32_t *tokb = reinterpret_cast<uint32_t *>(lds + P::OFF_TOK);
    int *flagb = reinterpret_cast<int *>(lds + P::OFF_FLAG);
    const uint4 *wqf = reinterpret_cast<const uint4 *>(pack + Cf::P_WQF);

    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, q = lane >> 4;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int s = g.shift;
    const int cnt = (g.nW - (int)blockIdx.x + (int)gridDim.x - 1) / (int)gridDim.x; // windows blockIdx.x + m gridDim.x, m < cnt

    const int hw = wv - HEADS;
    // ---- set-up: weights, biases and the table to LDS, all loads in flight together ----
    auto setup = [&](int tid) {
        constexpr int TH = P::THREADS, NW = TH / 64, N1K = (int)(P::SZ_WPT / 1024);
        static_assert(HEADS * 48 <= TH && P::SZ_WPT % 1024 == 0, "set-up in whole pieces");
        const int lane = tid & 63;
#pragma unroll
        for (int k = 0; k < (N1K + NW - 1) / NW; ++k) {
            const int f = k * NW + wv;
            if (f < N1K) lds_dma16(pack + Cf::P_WPT + (size_t)f * 1024 + 16 * lane, lds + P::OFF_WPT + (size_t)f * 1024);
        }
        const int i = tid < HEADS * 48 ? tid : 0, e = i % 16, t = i / 16 % 3, hd = i / 48;
        const float v = reinterpret_cast<const float *>(pack + Cf::P_BIAS)[hd / HG * 3 * CG + t * CG + hd % HG * D + (e < D ? e : 0)];
        TableCopy<P::NTBL * HEADS, TH> tc;
        tc.fetch(table, tid);
        if (tid < HEADS * 48) reinterpret_cast<float *>(lds + P::OFF_BIAS)[i] = e < D ? v : 0.f;
        tc.store(tbl, tid);
        __builtin_amdgcn_s_waitcnt(0);
    };
    // Wqkv^T tiles of group gn for the channels of its head hlp, a token tile of its dF (d(q|k|v) of the group's first head at
    // `src`, this lane's piece), and that tile's place in dx
    auto read_wt = [&](int gn, int hlp, int lane, uint4 (&wt)[HG]) {
#pragma unroll
        for (int h = 0; h < HG; ++h) wt[h] = wqf[((gn * HG + hlp) * HG + h) * 64 + lane];
    };
    auto make_df = [&](const uint16_t *src, int tt, const uint4 (&wt)[HG]) {
        f32x4 a = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int h = 0; h < HG; ++h)
            a = mma32(wt[h], *reinterpret_cast<const uint4 *>(src + h * P::DQ_HEAD + 16 * tt * P::DQ_ROW), a);
        return a;
    };
    auto store_dx = [&](f32x4 dF, uint32_t tok, int gn, int hlp, int q) {
        uint32_t *dst = reinterpret_cast<uint32_t *>(dx + (size_t)tok * C + gn * CG + hlp * D + 4 * q);
        const uint2 v = pack_bf16x4(dF);
        if (4 * q < D) dst[0] = v.x;
        if (4 * q + 2 < D) dst[1] = v.y;
    };
    float *mine = part + (size_t)blockIdx.x * P::L_TOTAL;
    // after the last window the row buffers make room for the bias-table tiles and for one half of d w_proj
    float *fold = reinterpret_cast<float *>(lds);
    f32x4 *wps = reinterpret_cast<f32x4 *>(lds + P::SZ_FOLD);

    if (wv >= HEADS) {
        int tid_h = threadIdx.x; // (opaque: nothing of this branch is kept through the other)
        asm volatile("" : "+v"(tid_h));
        const int lane = tid_h & 63, l16 = lane & 15, q = lane >> 4;
        // ---- rows (waves 6 and 7): token tiles 2 hw and 2 hw + 1 of a window ----
        const int per_img = g.nwi * g.nwj;
        const float r_img = 1.0f / (float)per_img, r_nwj = 1.0f / (float)g.nwj;
        uint4 rx[2][G][KS], ra[2][G][KS], rdy[2][KSC]; // as loaded: partial pieces still unshifted
        uint32_t rtok[2];
        int rflag = 0;
        auto load_rows = [&](int m) {
            const int win = (int)blockIdx.x + m * (int)gridDim.x;
            const int b = quotient(win, per_img, r_img), wr = win - b * per_img;
            const int wi = quotient(wr, g.nwj, r_nwj), wj = wr - wi * g.nwj;
            rflag = s > 0 ? (wi == g.nwi - 1 ? 1 : 0) | (wj == g.nwj - 1 ? 2 : 0) : 0;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                int si = wi * M + 2 * (2 * hw + i) + (l16 >> 3) + s, sj = wj * M + (l16 & 7) + s;
                if (si >= g.H) si -= g.H;
                if (sj >= g.W) sj -= g.W;
                const long tok = ((long)b * g.H + si) * g.W + sj;
                rtok[i] = (uint32_t)tok;
#pragma unroll
                for (int gi = 0; gi < G; ++gi)
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) {
                        rx[i][gi][ks] = load_piece4<CG>(x + tok * C + gi * CG, 32 * ks + 8 * q);
                        ra[i][gi][ks] = load_piece4<CG>(attn + tok * C + gi * CG, 32 * ks + 8 * q);
                    }
#pragma unroll
                for (int ks = 0; ks < KSC; ++ks) rdy[i][ks] = load_piece4<C>(dy + tok * C, 32 * ks + 8 * q);
            }
        };
        f32x4 wpacc[OTP][CTP];
        // window m: its operands to LDS; then its share of d w_proj | d b_proj
        uint4 dyf[2][KSC], af[2][G][KS];
        auto stage = [&](int m) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int tt = 2 * hw + i;
#pragma unroll
                for (int ks = 0; ks < KSC; ++ks) {
                    dyf[i][ks] = piece4<C>(rdy[i][ks], 32 * ks, q);
                    dyb[((m % P::DY_SLOTS) * KSC + ks) * 256 + tt * 64 + lane] = dyf[i][ks];
                }
#pragma unroll
                for (int gi = 0; gi < G; ++gi)
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) {
                        af[i][gi][ks] = piece4<CG>(ra[i][gi][ks], 32 * ks, q);
                        uint4 f = piece4<CG>(rx[i][gi][ks], 32 * ks, q);
                        if (gi > 0 && g.cascade) f = add_bf16x8(f, af[i][gi > 0 ? gi - 1 : 0][ks]);
                        f = with_bias_slot<CG>(f, ks, q);
                        if (lane < P::FL) fb[(((P::f_first(gi) + m % P::f_slots(gi)) * KS + ks) * 4 + tt) * P::FL + lane] = f;
                    }
                if (q == 0) tokb[(m % P::TOK_SLOTS) * 64 + 16 * tt + l16] = rtok[i];
            }
            if (tid == 64 * HEADS) flagb[m % P::TOK_SLOTS] = rflag;
        };
        auto project = [&] {
            // dY^T and [A | 1]^T of the two token tiles, K = 32 tokens
            uint4 aN[CTP];
#pragma unroll
            for (int ct = 0; ct < CTP; ++ct) {
                uint2 pk[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    f32x4 t = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int gi = 0; gi < G; ++gi)
#pragma unroll
                        for (int ks = 0; ks < KS; ++ks)
                            if (overlap(gi * CG + 32 * ks, gi * CG + (32 * ks + 32 < CG ? 32 * ks + 32 : CG), 16 * ct, 16 * ct + 16))
                                t = mma32(af[i][gi][ks], select_slot(16 * ct + l16, gi * CG + 32 * ks + 8 * q), t);
                    pk[i] = pack_bf16x4(t);
                    if (16 * ct + l16 == C) pk[i] = make_uint2(0x3f803f80u, 0x3f803f80u);
                }
                aN[ct] = cat(pk[0], pk[1]);
            }
#pragma unroll
            for (int ot = 0; ot < OTP; ++ot) {
                const uint4 sel = select_slot(16 * (ot & 1) + l16, 8 * q);
                const f32x4 z = f32x4{0.f, 0.f, 0.f, 0.f};
                const uint4 dyN = cat(pack_bf16x4(mma32(dyf[0][ot >> 1], sel, z)), pack_bf16x4(mma32(dyf[1][ot >> 1], sel, z)));
#pragma unroll
                for (int ct = 0; ct < CTP; ++ct) wpacc[ot][ct] = mma32(dyN, aN[ct], wpacc[ot][ct]);
            }
        };

        load_rows(0); // (a workgroup has at least one window)
        setup(tid_h);
        __syncthreads();
#pragma unroll
        for (int ot = 0; ot < OTP; ++ot)
#pragma unroll
            for (int ct = 0; ct < CTP; ++ct) wpacc[ot][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
        stage(0);
        if (cnt > 1) load_rows(1);
        __syncthreads();
        project();
        for (int n = 0; n < cnt + G; ++n) {
            if (n + 1 < cnt) {
                stage(n + 1);
                if (n + 2 < cnt) load_rows(n + 2);
                project();
            }
            // dF of the first group, whose heads were done with window n - G in the step before
            if (n >= G) {
                int at = lane; // (opaque, as above)
                asm volatile("" : "+v"(at));
                const uint16_t *src = dqb + ((n - 1) & 1) * (P::SZ_DQ / 2) + (at & 15) * P::DQ_ROW + 8 * (at >> 4);
#pragma unroll
                for (int hlp = 0; hlp < HG; ++hlp) {
                    uint4 wt[HG];
                    read_wt(0, hlp, at, wt);
#pragma unroll
                    for (int i = 0; i < 2; ++i)
                        store_dx(make_df(src, 2 * hw + i, wt), tokb[((n - G) % P::TOK_SLOTS) * 64 + 16 * (2 * hw + i) + l16], 0, hlp, q);
                }
            }
            __syncthreads();
        }
        if (hw == 1) {
#pragma unroll
            for (int ot = 0; ot < OTP; ++ot)
#pragma unroll
                for (int ct = 0; ct < CTP; ++ct) wps[(ot * CTP + ct) * 64 + lane] = wpacc[ot][ct];
        }
        __syncthreads();
        if (hw == 0) {
#pragma unroll
            for (int ot = 0; ot < OTP; ++ot)
#pragma unroll
                for (int ct = 0; ct < CTP; ++ct) {
                    const f32x4 v = wpacc[ot][ct] + wps[(ot * CTP + ct) * 64 + lane];
                    const int c = 16 * ct + l16, o = 16 * ot + 4 * q;
                    float *dst = mine + (c < C ? P::L_DWP + o * C + c : P::L_DBP + o);
                    const int step = c < C ? C : 1;
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (o + j < C && c <= C) dst[j * step] = v[j];
                }
        }
        return;
    }

    setup(tid);
    __syncthreads();
    const int hd = wv, gi = hd / HG, hl = hd % HG;
    const int lag = G - 1 - gi;
    // relative-position bias of (query l16 of tile qt, key 4q + j of tile kt) for kt - qt + 3 = dl, and the sums of its gradient.
    // (The bias rides in the upper half of the score product's K = 32, against the identity.)
    auto read_bias = [&](int dl, int l16, int q) {
        const int dr = (l16 >> 3) - (q >> 1) - 2 * (dl - 3), at = (dr + M - 1) * (2 * M - 1) + (l16 & 7) - 4 * (q & 1) + M - 1;
        return f32x4{to_f32(tbl[at * HEADS + hd]), to_f32(tbl[(at - 1) * HEADS + hd]), to_f32(tbl[(at - 2) * HEADS + hd]), to_f32(tbl[(at - 3) * HEADS + hd])};
    };
    uint2 bias_far[2]; // of the outermost tiles, used once a window: packed, turned into a tile by a product with the identity
    f32x4 bias_t[P::NDLT];
    f32x4 tblacc[P::NDLT];
    f32x4 dwacc[P::RT][CT];
    uint2 ident; // identity, K = 16
    {
#pragma unroll
        for (int dl = 0; dl < P::NDLT; ++dl) {
            if (dl == 0 || dl == P::NDLT - 1) bias_far[dl > 0] = pack_bf16x4(read_bias(dl, l16, q));
            else bias_t[dl] = read_bias(dl, l16, q);
            tblacc[dl] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int rt = 0; rt < P::RT; ++rt)
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) dwacc[rt][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
        const uint32_t one = 0x3f80u;
        const int d0 = l16 - 4 * q;
        ident.x = (d0 == 0 ? one : 0u) | (d0 == 1 ? one << 16 : 0u);
        ident.y = (d0 == 2 ? one : 0u) | (d0 == 3 ? one << 16 : 0u);
    }
    __syncthreads();

    const f32x4 zero = f32x4{0.f, 0.f, 0.f, 0.f};
    uint2 *turn = reinterpret_cast<uint2 *>(lds + P::OFF_TURN + hd * P::SZ_TURN);
    // dF of the group after this one, channels of head hl: it feeds this head's dO
    uint4 wt[HG]; // its Wqkv^T tiles
    auto load_weights = [&] {
        int at = tid & 63; // (opaque: the loads of all windows are the same, and would be kept in registers)
        asm volatile("" : "+v"(at));
        if (gi < G - 1) read_wt(gi + 1, hl, at, wt);
    };
    const int fslots = P::f_slots(gi);
    int fslot = 0;                                    // (window n - lag) % fslots
    load_weights();

    for (int n = 0; n < cnt + G; ++n) {
        // (the lane index as a window's address arithmetic sees it: opaque, so that the many per-lane addresses are made where
        // they are used instead of being kept, and spilled, across windows)
        int lane_n = tid & 63;
        asm volatile("" : "+v"(lane_n));
        const int lane = lane_n, l16 = lane & 15, q = lane >> 4;
        // a lane's place in a tile of 8-byte pieces (row group, column) that it reads turned, and in the tiles of F
        const int tr = (l16 & 3) * 16 + 4 * q + (l16 >> 2);
        const uint8_t *ftr = lds + P::OFF_F + ((l16 & 3) >> 1) * 256 + (l16 & 1) * 8 + (4 * q + (l16 >> 2)) * 16;
        const int m = n - lag; // the window of this head
        const bool active = m >= 0 && m < cnt;
        const int flags = active ? __builtin_amdgcn_readfirstlane(flagb[m % P::TOK_SLOTS]) : 0;
        f32x4 dF[4];
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) dF[tt] = zero;
        if (gi < G - 1 && active) {
            const uint16_t *src = dqb + ((n - 1) & 1) * (P::SZ_DQ / 2) + (gi + 1) * HG * P::DQ_HEAD + l16 * P::DQ_ROW + 8 * q;
#pragma unroll
            for (int tt = 0; tt < 4; ++tt) dF[tt] = make_df(src, tt, wt);
#pragma unroll
            for (int tt = 0; tt < 4; ++tt) {
                store_dx(dF[tt], tokb[(m % P::TOK_SLOTS) * 64 + 16 * tt + l16], gi + 1, hl, q);
                if (!g.cascade) dF[tt] = zero;
            }
        }
        // ---- attention of this head, window n - lag ----
        auto attention = [&](auto masked) {
            constexpr bool MASK = decltype(masked)::value;
            const int fat = (P::f_first(G) - (G - gi) * (G - gi + 3) / 2 + fslot) * KS * 4 * P::FL;
            const uint4 *F = fb + fat + (lane < P::FL ? lane : lane - 16);
            const uint4 *DY = dyb + (m % P::DY_SLOTS) * KSC * 256 + lane;
            uint16_t *dq = dqb + (n & 1) * (P::SZ_DQ / 2) + hd * P::DQ_HEAD;
            // a tile of d q, d k or d v (t = 0, 1, 2, written in this order) into the rows of its tokens
            auto put = [&](int t, int tt, f32x4 v) {
                const uint2 p = pack_bf16x4(v);
                uint32_t *dst = reinterpret_cast<uint32_t *>(dq + (16 * tt + l16) * P::DQ_ROW + t * D + 4 * q);
                dst[0] = p.x;
                dst[1] = p.y;
            };
            // q, k, v and dO (adjoint of Eq. 7 plus the gradient through Eq. 8) of all tokens.  Every read stands in front of the
            // first write to LDS: the compiler keeps the order of the two, and a read behind a write is waited for in full.
            uint2 Qb[4], Kb[4], KT[4], Vb[4];
            {
                int at = lane;
                asm volatile("" : "+v"(at)); // (opaque, as above)
                uint4 w[3][KS];
#pragma unroll
                for (int t = 0; t < 3; ++t)
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) w[t][ks] = wq[((hd * 3 + t) * KS + ks) * 64 + at];
                uint4 f[4][KS], wo[KSC], dyf[4][KSC];
                f32x4 b[3];
#pragma unroll
                for (int t = 0; t < 3; ++t) b[t] = *reinterpret_cast<const f32x4 *>(bqkv + (hd * 3 + t) * 16 + 4 * q);
#pragma unroll
                for (int tt = 0; tt < 4; ++tt)
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) f[tt][ks] = F[(ks * 4 + tt) * P::FL];
#pragma unroll
                for (int ks = 0; ks < KSC; ++ks) wo[ks] = wpt[(hd * KSC + ks) * 64 + lane];
#pragma unroll
                for (int tt = 0; tt < 4; ++tt)
#pragma unroll
                    for (int ks = 0; ks < KSC; ++ks) dyf[tt][ks] = DY[ks * 256 + tt * 64];
#pragma unroll
                for (int t = 1; t < 4; ++t) // k, v, q
#pragma unroll
                    for (int tt = 0; tt < 4; ++tt) {
                        f32x4 r = b[t % 3];
#pragma unroll
                        for (int ks = 0; ks < KS; ++ks) r = mma32(w[t % 3][ks], f[tt][ks], r);
                        (t == 1 ? Kb : t == 2 ? Vb : Qb)[tt] = pack_bf16x4(r);
                    }
#pragma unroll
                for (int tt = 0; tt < 4; ++tt)
#pragma unroll
                    for (int ks = 0; ks < KSC; ++ks) dF[tt] = mma32(wo[ks], dyf[tt][ks], dF[tt]);
#pragma unroll
                for (int kt = 0; kt < 4; ++kt) turn[kt * 64 + lane] = Kb[kt];
#pragma unroll
                for (int kt = 0; kt < 4; ++kt) KT[kt] = lds_read_tr(turn + kt * 64 + tr);
            }
            f32x4 dk[4], dv[4];
#pragma unroll
            for (int kt = 0; kt < 4; ++kt) dk[kt] = dv[kt] = zero;
#pragma unroll
            for (int qt = 0; qt < 4; ++qt) {
                turn[4 * 64 + lane] = Qb[qt];
                // scores and softmax; P stays unnormalised, 1 / sum goes into dO: P dO^T and P (dP - delta) are the same
                f32x4 st[4], dp[4];
#pragma unroll
                for (int kt = 0; kt < 4; ++kt) {
                    const int dl = kt - qt + 3;
                    const bool far = dl == 0 || dl == P::NDLT - 1;
                    st[kt] = mma16(Kb[kt], Qb[qt], far ? mma16(ident, bias_far[dl > 0], zero) : bias_t[dl]);
                }
                if (MASK) {
                    const bool qr = 2 * qt + (l16 >> 3) >= M - s, qc = (l16 & 7) >= M - s;
#pragma unroll
                    for (int kt = 0; kt < 4; ++kt) {
                        const bool row = (flags & 1) && qr != (2 * kt + (q >> 1) >= M - s);
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            st[kt][j] += row || ((flags & 2) && qc != (4 * (q & 1) + j >= M - s)) ? kMask : 0.f;
                    }
                }
                float mx = -INFINITY;
#pragma unroll
                for (int kt = 0; kt < 4; ++kt) mx = max5f(mx, st[kt]);
                const float mxl = qgroup_max(mx) * kLog2e;
                uint2 Pb[4];
                f32x4 sum4;
#pragma unroll
                for (int kt = 0; kt < 4; ++kt) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) st[kt][j] = __builtin_amdgcn_exp2f(fmaf(st[kt][j], kLog2e, -mxl));
                    turn[kt * 64 + lane] = pack_bf16x4(st[kt]);
                    sum4 = kt == 0 ? st[0] : sum4 + st[kt];
                }
                const float inv = recip(qgroup_sum((sum4[0] + sum4[1]) + (sum4[2] + sum4[3])));
                const uint2 dOb = pack_bf16x4(dF[qt] * inv);
                turn[5 * 64 + lane] = dOb;
#pragma unroll
                for (int kt = 0; kt < 4; ++kt) dp[kt] = mma16(Vb[kt], dOb, zero);
#pragma unroll
                for (int kt = 0; kt < 4; ++kt) Pb[kt] = lds_read_tr(turn + kt * 64 + tr);
                const uint2 QN = lds_read_tr(turn + 4 * 64 + tr), dON = lds_read_tr(turn + 5 * 64 + tr);
                f32x4 del4 = st[0] * dp[0];
#pragma unroll
                for (int kt = 1; kt < 4; ++kt)
#pragma unroll
                    for (int j = 0; j < 4; ++j) del4[j] = fmaf(st[kt][j], dp[kt][j], del4[j]);
                const float delta = inv * qgroup_sum((del4[0] + del4[1]) + (del4[2] + del4[3]));
                uint2 dSb[4];
#pragma unroll
                for (int kt = 0; kt < 4; ++kt) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) dp[kt][j] = st[kt][j] * (dp[kt][j] - delta);
                    dSb[kt] = pack_bf16x4(dp[kt]);
                    turn[kt * 64 + lane] = dSb[kt];
                }
#pragma unroll
                for (int kt = 0; kt < 4; ++kt) {
                    dv[kt] = mma16(dON, Pb[kt], dv[kt]);
                    tblacc[kt - qt + 3] = mma16(ident, dSb[kt], tblacc[kt - qt + 3]);
                }
                const f32x4 dq_ = mma32(cat(KT[2], KT[3]), cat(dSb[2], dSb[3]), mma32(cat(KT[0], KT[1]), cat(dSb[0], dSb[1]), zero));
                put(0, qt, dq_);
#pragma unroll
                for (int kt = 0; kt < 4; ++kt) dk[kt] = mma16(QN, lds_read_tr(turn + kt * 64 + tr), dk[kt]);
            }
            // (the padding of one tile and the features of the next are places of different lanes: only the order of the writes,
            // which a wave's LDS accesses keep, says which of them stays, so the compiler must keep it too)
            asm volatile("" ::: "memory");
#pragma unroll
            for (int kt = 0; kt < 4; ++kt) put(1, kt, dk[kt]);
            asm volatile("" ::: "memory");
#pragma unroll
            for (int kt = 0; kt < 4; ++kt) put(2, kt, dv[kt]);
            // ---- d w_qkv (and d b_qkv in the spare column) ----
#pragma unroll
            for (int kp = 0; kp < 2; ++kp) {
                uint4 f[CT];
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    const uint8_t *at = ftr + (size_t)fat * 16 + (((ct >> 1) * 4 + 2 * kp) * P::FL + (ct & 1) * 32) * 16;
                    f[ct] = cat(lds_read_tr(at), lds_read_tr(at + P::FL * 16));
                }
#pragma unroll
                for (int rt = 0; rt < P::RT; ++rt) {
                    const uint16_t *at = dq + (32 * kp + 4 * q + (l16 >> 2)) * P::DQ_ROW + 16 * rt + 4 * (l16 & 3);
                    const uint4 a = cat(lds_read_tr(at), lds_read_tr(at + 16 * P::DQ_ROW));
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct) dwacc[rt][ct] = mma32(a, f[ct], dwacc[rt][ct]);
                }
            }
        };
        if (active) {
            if (flags) attention(std::true_type{});
            else attention(std::false_type{});
            fslot = fslot + 1 < fslots ? fslot + 1 : 0;
        }
        load_weights(); // (on their way over the barrier; held through the steps above they would cost their registers)
        __syncthreads();
    }

    // ---- this workgroup's partial sums.  The packed query weights carry 1/sqrt(d), so their gradients get it back here ----
    int lane_e = tid & 63;
    asm volatile("" : "+v"(lane_e));
    const int le = lane_e;
    {
        const int lane = le, l16 = lane & 15, q = lane >> 4;
        const float scale = 1.0f / sqrtf((float)D);
#pragma unroll
        for (int rt = 0; rt < P::RT; ++rt)
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int u = 16 * rt + 4 * q + j, t = u / D, c = 16 * ct + l16; // feature u of the head
                    const int row = (gi * 3 + t) * CG + hl * D + u % D;
                    if (u < 3 * D && c <= CG)
                        mine[c < CG ? P::L_DWQ + row * CG + c : P::L_DBQ + row] = t == 0 ? dwacc[rt][ct][j] * scale : dwacc[rt][ct][j];
                }
        float *mat = fold + hd * P::NDLT * 16 * P::TP;
#pragma unroll
        for (int dl = 0; dl < P::NDLT; ++dl)
#pragma unroll
            for (int j = 0; j < 4; ++j) mat[(dl * 16 + 4 * q + j) * P::TP + l16] = tblacc[dl][j];
    }
    __syncthreads();
    const float *mat = fold + hd * P::NDLT * 16 * P::TP;
#pragma unroll
    for (int k = 0; k < (P::NTBL + 63) / 64; ++k) {
        const int e = 64 * k + le < P::NTBL ? 64 * k + le : P::NTBL - 1;
        const float a = table_entry<P::TP>(mat, e);
        if (64 * k + le < P::NTBL) mine[P::L_TBL + hd * P::NTBL + e] = a;
    }
}

template <class Cf>
hipError_t run(const Geom &g, int grid, const bf16_t *x, const bf16_t *dy, const bf16_t *attn, const uint8_t *pack,
               const bf16_t *table, bf16_t *dx, float *dw_qkv, float *db_qkv, float *dw_proj, float *db_proj, float *dtable,
               int accumulate, float *part, hipStream_t s)
{
    using P = HeadsCfg<Cf>;
    auto kern = heads_bwd_kernel<Cf>;
    if (hipError_t ea = allow_dynamic_lds(reinterpret_cast<const void *>(kern), P::LDS_BYTES); ea != hipSuccess) return ea;
    {
        KernelTimer kt(K_FUSED_BWD, s);
        hipLaunchKernelGGL(kern, dim3(grid), dim3(P::THREADS), P::LDS_BYTES, s, g, x, dy, attn, pack, table, dx, part);
    }
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    ReduceOut out{};
    float *const ptr[5] = {dw_qkv, db_qkv, dw_proj, db_proj, dtable};
    const int begin[6] = {P::L_DWQ, P::L_DBQ, P::L_DWP, P::L_DBP, P::L_TBL, P::L_END};
    for (int k = 0; k < 5; ++k) out.ptr[k] = ptr[k];
    for (int k = 0; k < 6; ++k) out.begin[k] = begin[k];
    out.nseg = 5;
    out.tbl_heads = P::HEADS; out.tbl_entries = P::NTBL; out.tbl_stride = P::HEADS; out.tbl_head0 = 0;
    return launch_reduce(part, grid, P::L_TOTAL, out, accumulate, s);
}

int heads_grid(const Geom &g, int cus)
{
    if (cus > kSizingCus) cus = kSizingCus;
    return cus > g.nW ? g.nW : cus;
}

#define GSWA_HEADS_SHAPES(X) X(60, 6, 1) X(60, 6, 2) X(60, 6, 3)

} // namespace

bool heads_bwd_supported(const Geom &g)
{
    if (g.M != 8) return false;
#define X(C_, H_, G_) \
    if (g.C == C_ && g.heads == H_ && g.groups == G_) return true;
    GSWA_HEADS_SHAPES(X)
#undef X
    return false;
}

size_t heads_bwd_ws_bytes(const Geom &g)
{
    int total = 0;
#define X(C_, H_, G_) \
    if (g.C == C_ && g.heads == H_ && g.groups == G_) total = HeadsCfg<FusedCfg<C_, H_, G_>>::L_TOTAL;
    GSWA_HEADS_SHAPES(X)
#undef X
    return (size_t)heads_grid(g, kSizingCus) * total * sizeof(float);
}

hipError_t launch_heads_bwd(const Geom &g, const bf16_t *x, const bf16_t *dy, const bf16_t *attn, const void *pack,
                            const bf16_t *table, bf16_t *dx, float *dw_qkv, float *db_qkv, float *dw_proj, float *db_proj,
                            float *dtable, int accumulate, void *ws, hipStream_t s)
{
    const int grid = heads_grid(g, device_cu_count());
#define X(C_, H_, G_)                                                                                                     \
    if (g.C == C_ && g.heads == H_ && g.groups == G_)                                                                     \
        return run<FusedCfg<C_, H_, G_>>(g, grid, x, dy, attn, static_cast<const uint8_t *>(pack), table, dx, dw_qkv,     \
                                         db_qkv, dw_proj, db_proj, dtable, accumulate, static_cast<float *>(ws), s);
    GSWA_HEADS_SHAPES(X)
#undef X
    return hipErrorInvalidValue;
}

} // namespace gswa
