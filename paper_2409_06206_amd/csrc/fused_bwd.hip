// Fused GSWA backward for 8x8 windows, bf16 storage: narrow layers of six groups, and wide layers of three with an odd shift
// (narrow layers of one to three groups: heads_bwd.hip; wide ones of two groups: wide_heads_bwd.hip, of three with an even
// shift: wide_bwd.hip).  The backward of a layer is a
// sequence of launches of fused_bwd_kernel, one per chunk of heads in reverse order; each recomputes q, k, v, the scores and the
// softmax of its heads from x and the saved group outputs, and produces the dx slices of its groups and per-workgroup partial
// sums of the parameter gradients (accumulated in registers over the windows a workgroup owns).  reduce_partials_kernel adds
// the partials in a fixed order.  wproj_grad_kernel is the projection's weight gradient for wide layers.
//
// Per window, wave w owns tokens 16w..16w+15 both as queries and as keys.  Notation for a
// matrix X[tokens x features] held as an MFMA result tile (see mfma.h):
//   T-form: rows = features 4q+j, column = token l16   (packed: B operand "k=feature,n=token"
//           or A operand "m=token,k=feature")
//   N-form: rows = tokens 4q+j,  column = feature l16  (packed: B operand "k=token,n=feature"
//           or A operand "m=feature,k=token")
// A packed tile that other waves or the other orientation need goes to LDS as it lies in the registers, and is read back
// either as it is or turned (lds_read_tr).
#include "fused.h"
#include "heads_bwd.h"
#include "mfma.h"
#include "wide_heads_bwd.h"

namespace gswa {

namespace {

constexpr float kLog2e = 1.4426950408889634f;

template <class Cf, int HB_, int HE_, bool WPROJ_> struct BwdCfg {
    static constexpr int C = Cf::C, D = Cf::D, CG = Cf::CG, HG = Cf::HG, HEADS = Cf::HEADS, G = Cf::G;
    static constexpr int ET = Cf::ET, KS = Cf::KS;
    static constexpr int KSC = (C + 31) / 32; // K=32 steps over all C channels of dy
    static constexpr int NTBL = 15 * 15;
    static constexpr int TBL_N = NTBL * HEADS;
    // weight-gradient tiling: 16x16 tiles, one spare column (index CG resp. C) carries the bias sums
    static constexpr int CT = CG / 16 + 1;          // column tiles of d w_qkv of one head
    static constexpr int NT = 3 * ET * CT;          // tiles of one head's d w_qkv rows
    static constexpr int KT = (NT + 3) / 4;         // tiles per wave
    // heads [HB, HE) of this launch: whole groups.  WPROJ: this launch also produces the columns of
    // d w_proj that belong to its heads, and the last heads' launch d b_proj (narrow layers; wide ones use a kernel of its own).
    static constexpr int HB = HB_, HE = HE_, NH = HE - HB;
    static constexpr bool WPROJ = WPROJ_, BPROJ = WPROJ_ && HE_ == Cf::HEADS;
    static constexpr int WC0 = HB * D, WCN = NH * D;  // the columns; the spare column WCN carries the bias sums
    static constexpr int OTP = (C + 15) / 16, CTP = WCN / 16 + 1;
    static constexpr int NTP = OTP * CTP, KTP = (NTP + 3) / 4;
    static constexpr int GB = HB / HG, GE = (HE - 1) / HG; // lowest and highest group of the chunk
    static_assert(NH > 0 && HB % HG == 0 && HE % HG == 0, "a chunk is whole groups");
    // packed parameters of these heads, copied from the buffer forward filled: [WQ | BIAS | WPT | WQT]
    static constexpr int N_WQ = NH * 3 * ET * KS, N_WPT = NH * ET * KSC, N_WQT = NH * 3 * ET * HG * ET;
    static constexpr size_t SRC_WQ = Cf::P_WQ + (size_t)HB * 3 * ET * KS * 1024;
    static constexpr size_t SRC_WPT = Cf::P_WPT + (size_t)HB * ET * KSC * 1024;
    static constexpr size_t SRC_WQT = Cf::P_WQT + (size_t)HB * 3 * ET * HG * ET * 512;
    static constexpr size_t OFF_WQ = 0;
    static constexpr size_t OFF_BIAS = OFF_WQ + (size_t)N_WQ * 1024;
    static constexpr size_t OFF_WPT = OFF_BIAS + (size_t)NH * 3 * ET * 64; // fp32 b_qkv [head][q, k, v][16 ET]
    static constexpr size_t OFF_WQT = OFF_WPT + (size_t)N_WPT * 1024;
    static constexpr size_t PACK_BYTES = OFF_WQT + (size_t)N_WQT * 512;
    // LDS beyond the packed weights
    static constexpr int LW = 68; // pitch (bf16) of rows read 8 at a time (as two 8-byte halves:
                                  // 34 dwords keeps every 16-lane phase on distinct banks)
    static constexpr size_t SZ_FRAG = (size_t)4 * ET * 64 * 8; // packed tiles of 64 tokens, lane by lane
    static constexpr size_t SZ_SQ = (size_t)64 * LW * 2; // P / dS, 16 such tiles (key tile, query tile); also dY operands / A^T rows
    static constexpr size_t OFF_TBLF = PACK_BYTES;             // fp32 bias table [NH][225]
    static constexpr size_t OFF_KB = OFF_TBLF + (((size_t)NH * NTBL * 4 + 15) & ~size_t(15));
    static constexpr size_t OFF_VB = OFF_KB + SZ_FRAG;
    static constexpr size_t OFF_QB = OFF_VB + SZ_FRAG;
    static constexpr size_t OFF_DOB = OFF_QB + SZ_FRAG;
    static constexpr size_t OFF_P = OFF_DOB + SZ_FRAG;
    static constexpr size_t OFF_DS = OFF_P + SZ_SQ;
    static constexpr size_t OFF_DQKV = OFF_DS + SZ_SQ;         // d(q|k|v)^T tiles (t, et, token tile)
    static constexpr size_t SZ_DQKV = 3 * SZ_FRAG;
    static constexpr size_t OFF_F = OFF_DQKV + SZ_DQKV;        // F^T rows [c][token] of the current group
    static constexpr size_t SZ_F = (size_t)16 * CT * LW * 2;
    static constexpr size_t LDS_BYTES = OFF_F + SZ_F;
    // Per-workgroup partial sums of THIS launch only (the scratch is reused from launch to launch: the
    // head-group loop bounds it).  Rows of d w_qkv: for every group of the chunk and each of q, k, v
    // CG rows, ((gi - GB) * 3 + t) * CG + hl * D + e; then the bias
    // sums in the same order, the columns of d w_proj | d b_proj where this launch produces them, and the bias-table
    // gradient head by head.
    static constexpr int NG = GE - GB + 1;
    static constexpr int L_DWQ = 0;
    static constexpr int L_DBQ = L_DWQ + NG * 3 * CG * CG;
    static constexpr int L_DWP = L_DBQ + NG * 3 * CG;
    static constexpr int L_DBP = L_DWP + (WPROJ ? C * WCN : 0);
    static constexpr int L_TBL = L_DBP + (BPROJ ? C : 0);
    static constexpr int L_END = L_TBL + NH * NTBL;
    static constexpr int L_TOTAL = (L_END + 3) & ~3; // stride of the vectors: whole 16-byte pieces (the sum reads four entries per load)
    static_assert(!WPROJ || (OTP <= 2 * KSC && SZ_SQ >= (size_t)KSC * 4096 &&
                             SZ_SQ >= (size_t)16 * CTP * LW * 2),
                  "dY operands / A^T rows alias the P / dS squares");
};

template <class Cf> __device__ __forceinline__ constexpr int fq(int hd, int t, int et, int ks)
{
    return ((hd * 3 + t) * Cf::ET + et) * Cf::KS + ks;
}
template <class Cf> __device__ __forceinline__ constexpr int fqt(int hd, int t, int et, int hlp, int etp)
{
    return ((((hd * 3 + t) * Cf::ET + et) * Cf::HG + hlp) * Cf::ET) + etp;
}

// Channels [c, c + 4) of a row, as load_piece4 and piece4 take eight of them.
struct __attribute__((packed, aligned(4))) Piece2 { uint32_t v[2]; };
template <int N> __device__ __forceinline__ uint2 load_piece2(const bf16_t *row, int c)
{
    static_assert(N >= 4 && N % 2 == 0, "whole pieces");
    const Piece2 p = *reinterpret_cast<const Piece2 *>(row + (c < N - 4 ? c : N - 4));
    return make_uint2(p.v[0], p.v[1]);
}
template <int N> __device__ __forceinline__ uint2 piece2(uint2 p, int first, int q)
{
    const int n = N - first;
    if (n >= 16) return p;
    const int part = n / 4;
    uint2 o = make_uint2(q < part ? p.x : 0u, q < part ? p.y : 0u);
    if (n % 4) o.x = q == part ? p.y : o.x;
    return o;
}

constexpr bool ranges_overlap(int a0, int a1, int b0, int b1) { return a0 < b1 && b0 < a1; }

// What bounds it: chains, not rates.  A head is three steps of four wavefronts between barriers, each a few products
// long, and a CU holds two workgroups: a read that is waited for where it is used costs more than its products.  So the
// next window's rows are loaded a head before the window ends, in pieces of 16 bytes; a head's weights, biases (whole
// padded tiles) and bias-table entries are read in front of the barrier before their use; the set-up's loads are all in
// flight together; the table gradient of as many heads as LDS takes is folded at once.  fwd + bwd, 60 channels, six groups,
// 32 images of 64x64: 143 -> 126.5 us, with packed tiles read turned 118.8; 180 channels, three groups, odd shift, 8 images:
// 180 -> 143.
template <class Cf, int HB, int HE, bool WPROJ>
__global__ __launch_bounds__(256, (BwdCfg<Cf, HB, HE, WPROJ>::LDS_BYTES <= 80 * 1024 ? 2 : 1))
void fused_bwd_kernel(Geom g, const bf16_t *__restrict__ x,
                                                        const bf16_t *__restrict__ dy,
                                                        const bf16_t *__restrict__ attn,
                                                        const uint8_t *__restrict__ pack,
                                                        const bf16_t *__restrict__ table,
                                                        bf16_t *dx, float *__restrict__ part)
{
    using B = BwdCfg<Cf, HB, HE, WPROJ>;
    constexpr int NH = B::NH, GB = B::GB, GE = B::GE;
    constexpr int C = B::C, D = B::D, CG = B::CG, HG = B::HG, HEADS = B::HEADS, G = B::G;
    constexpr int ET = B::ET, KS = B::KS, KSC = B::KSC, LW = B::LW, NTBL = B::NTBL;
    constexpr int CT = B::CT, NT = B::NT, KT = B::KT, CTP = B::CTP, NTP = B::NTP, KTP = B::KTP;
    constexpr int M = 8;
    static_assert(CG % 2 == 0 && D % 2 == 0 && C % 4 == 0, "dword-granular loads and stores");
    // The shift mask, exactly as the forward kernel of the same layer adds it: -100 for wide layers;
    // narrow layers carry it through bf16 matrix-core operands in base-2 units, where it is
    // -144 = bf16(-100 log2 e), i.e. -99.81 here.
    constexpr float kMask = Cf::SPLIT ? -100.0f : -144.0f / kLog2e;

    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const uint4 *wq = reinterpret_cast<const uint4 *>(lds + B::OFF_WQ);
    const uint4 *wpt = reinterpret_cast<const uint4 *>(lds + B::OFF_WPT);
    const uint2 *wqt = reinterpret_cast<const uint2 *>(lds + B::OFF_WQT);
    const float *bqkv = reinterpret_cast<const float *>(lds + B::OFF_BIAS);
    float *tblf = reinterpret_cast<float *>(lds + B::OFF_TBLF);
    uint2 *kb = reinterpret_cast<uint2 *>(lds + B::OFF_KB);
    uint2 *vb = reinterpret_cast<uint2 *>(lds + B::OFF_VB);
    uint2 *qb = reinterpret_cast<uint2 *>(lds + B::OFF_QB);
    uint2 *dob = reinterpret_cast<uint2 *>(lds + B::OFF_DOB);
    uint2 *pbuf = reinterpret_cast<uint2 *>(lds + B::OFF_P);
    uint2 *dsbuf = reinterpret_cast<uint2 *>(lds + B::OFF_DS);
    uint4 *dybuf = reinterpret_cast<uint4 *>(pbuf);
    uint16_t *abuf = reinterpret_cast<uint16_t *>(dsbuf); // dY operands and A^T rows live where P / dS go later in the window
    uint2 *gbuf = reinterpret_cast<uint2 *>(lds + B::OFF_DQKV);
    uint16_t *fbuf = reinterpret_cast<uint16_t *>(lds + B::OFF_F);

    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, q = lane >> 4;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6); // wave index, held in a scalar register

    // Rows of x, of the saved group outputs and of dy of this lane's token as MFMA operands (k-slots =
    // channels).  The rows of a window are fetched while the previous window is finished (the first
    // window's during the set-up), so that their latency is off the critical path.
    const int per_img = g.nwi * g.nwj;
    const int rn = 2 * wv + (l16 >> 3), cn = l16 & 7;
    const int s = g.shift;
    // window -> (image, window row, window column)
    const float r_img = 1.0f / (float)per_img, r_nwj = 1.0f / (float)g.nwj;
    auto token_of = [&](int win) {
        const int b = quotient(win, per_img, r_img);
        const int wr = win - b * per_img;
        const int wi = quotient(wr, g.nwj, r_nwj), wj = wr - wi * g.nwj;
        int si = wi * M + rn + s, sj = wj * M + cn + s;
        if (si >= g.H) si -= g.H;
        if (sj >= g.W) sj -= g.W;
        return ((long)b * g.H + si) * g.W + sj;
    };
    constexpr auto need_x = [](int gi) { return gi >= GB && gi <= GE; };
    constexpr auto need_a = [](int gi) { return gi >= GB - 1 && gi < GE + (WPROJ ? 1 : 0); };
    // dF of the next group (Eq. 8) comes from the dx slice that an earlier launch finished
    constexpr auto need_c = [](int hd) {
        const int gi = hd / HG;
        return gi < G - 1 && !(HB <= (gi + 1) * HG && HE >= (gi + 2) * HG);
    };
    constexpr int ROW_REGS = [&]() {
        int n = 4 * KSC;
        for (int gi = 0; gi < G; ++gi) n += 4 * KS * ((need_x(gi) ? 1 : 0) + (need_a(gi) ? 1 : 0));
        return n;
    }();
    uint4 xf[G][KS], af[G][KS], dyf[KSC];    // a window's operands
    uint4 rx[G][KS], ra[G][KS], rdy[KSC];    // as loaded: partial pieces still unshifted
    uint2 cgrad[NH][ET], rc[NH][ET];
    auto load_rows = [&](int win) {
        const long tok = token_of(win);
#pragma unroll
        for (int hx = 0; hx < NH; ++hx) {
            const int hd = HB + hx, gi = hd / HG, hl = hd % HG;
#pragma unroll
            for (int et = 0; et < ET; ++et) {
                rc[hx][et] = make_uint2(0u, 0u);
                if (need_c(hd) && g.cascade)
                    rc[hx][et] = load_piece2<D>(dx + tok * C + (gi + 1) * CG + hl * D, 16 * et + 4 * q);
            }
        }
#pragma unroll
        for (int gi = 0; gi < G; ++gi)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                rx[gi][ks] = ra[gi][ks] = make_uint4(0u, 0u, 0u, 0u);
                if (need_x(gi)) rx[gi][ks] = load_piece4<CG>(x + tok * C + gi * CG, 32 * ks + 8 * q);
                if (need_a(gi)) ra[gi][ks] = load_piece4<CG>(attn + tok * C + gi * CG, 32 * ks + 8 * q);
            }
#pragma unroll
        for (int ks = 0; ks < KSC; ++ks) rdy[ks] = load_piece4<C>(dy + tok * C, 32 * ks + 8 * q);
    };
    auto take_rows = [&]() {
#pragma unroll
        for (int hx = 0; hx < NH; ++hx)
#pragma unroll
            for (int et = 0; et < ET; ++et) cgrad[hx][et] = piece2<D>(rc[hx][et], 16 * et, q);
#pragma unroll
        for (int gi = 0; gi < G; ++gi)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                xf[gi][ks] = need_x(gi) ? piece4<CG>(rx[gi][ks], 32 * ks, q) : make_uint4(0u, 0u, 0u, 0u);
                af[gi][ks] = need_a(gi) ? piece4<CG>(ra[gi][ks], 32 * ks, q) : make_uint4(0u, 0u, 0u, 0u);
            }
#pragma unroll
        for (int ks = 0; ks < KSC; ++ks) dyf[ks] = piece4<C>(rdy[ks], 32 * ks, q);
    };
    // (the rows of the next window wait in registers from the last head of the window before on; where a launch needs
    // too many of them they are loaded at the start of their own window)
    constexpr bool PIPE = ROW_REGS <= 32;
    if (PIPE && (int)blockIdx.x < g.nW) load_rows(blockIdx.x);

    // set-up copies, unrolled so that a thread's loads are all in flight before its first store
    {
        constexpr int N_Q = (int)((B::OFF_BIAS - B::OFF_WQ) / 16), N_PT = (int)((B::OFF_WQT - B::OFF_WPT) / 16);
        constexpr int N_QT = (int)((B::PACK_BYTES - B::OFF_WQT) / 16), N_T = NTBL * NH, N_B = NH * 3 * ET * 16;
        constexpr int I_Q = (N_Q + 255) / 256, I_PT = (N_PT + 255) / 256, I_QT = (N_QT + 255) / 256, I_T = (N_T + 255) / 256;
        constexpr int I_B = (N_B + 255) / 256;
        uint4 vq[I_Q], vpt[I_PT], vqt[I_QT];
        uint16_t vt[I_T];
        float vb[I_B];
        // (threads behind a part's end copy its last piece once more: under a condition each load would sit, and be
        // waited for, in the branch of its store)
        auto at = [&](int k, int n) { const int i = 256 * k + tid; return i < n ? i : n - 1; };
#pragma unroll
        for (int k = 0; k < I_Q; ++k) vq[k] = reinterpret_cast<const uint4 *>(pack + B::SRC_WQ)[at(k, N_Q)];
#pragma unroll
        for (int k = 0; k < I_PT; ++k) vpt[k] = reinterpret_cast<const uint4 *>(pack + B::SRC_WPT)[at(k, N_PT)];
#pragma unroll
        for (int k = 0; k < I_QT; ++k) vqt[k] = reinterpret_cast<const uint4 *>(pack + B::SRC_WQT)[at(k, N_QT)];
#pragma unroll
        for (int k = 0; k < I_B; ++k) {
            const int i = at(k, N_B), e = i % (16 * ET), t = i / (16 * ET) % 3, hd = HB + i / (48 * ET);
            vb[k] = reinterpret_cast<const float *>(pack + Cf::P_BIAS)[hd / HG * 3 * CG + t * CG + hd % HG * D + (e < D ? e : 0)];
            if (e >= D) vb[k] = 0.f;
        }
#pragma unroll
        for (int k = 0; k < I_T; ++k) { const int i = at(k, N_T); vt[k] = table[(i % NTBL) * HEADS + HB + i / NTBL].bits; }
#pragma unroll
        for (int k = 0; k < I_Q; ++k) reinterpret_cast<uint4 *>(lds + B::OFF_WQ)[at(k, N_Q)] = vq[k];
#pragma unroll
        for (int k = 0; k < I_PT; ++k) reinterpret_cast<uint4 *>(lds + B::OFF_WPT)[at(k, N_PT)] = vpt[k];
#pragma unroll
        for (int k = 0; k < I_QT; ++k) reinterpret_cast<uint4 *>(lds + B::OFF_WQT)[at(k, N_QT)] = vqt[k];
#pragma unroll
        for (int k = 0; k < I_B; ++k) reinterpret_cast<float *>(lds + B::OFF_BIAS)[at(k, N_B)] = vb[k];
#pragma unroll
        for (int k = 0; k < I_T; ++k) tblf[at(k, N_T)] = __uint_as_float((uint32_t)vt[k] << 16);
    }

    // this lane's token inside the window, and the bias-table row of its (query, key 4q) pair:
    // the entry of key 16kt+4q+j is idx0 - 30kt - j
    const int idx0 = (rn - (q >> 1) + M - 1) * (2 * M - 1) + (cn - 4 * (q & 1) + M - 1);
    bool rmask[4], cmask[4];
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) rmask[kt] = (rn >= M - s) != ((2 * kt + (q >> 1)) >= M - s);
#pragma unroll
    for (int j = 0; j < 4; ++j) cmask[j] = (cn >= M - s) != ((4 * (q & 1) + j) >= M - s);
    uint2 ident; // identity as a K=16 A operand: row l16, k-slots 4q+j
    {
        const uint32_t one = 0x3f80u;
        const int d0 = l16 - 4 * q;
        ident.x = (d0 == 0 ? one : 0u) | (d0 == 1 ? one << 16 : 0u);
        ident.y = (d0 == 2 ? one : 0u) | (d0 == 3 ? one << 16 : 0u);
    }
    __syncthreads();

    f32x4 tblacc[NH][4], dwacc[NH][KT], wpacc[KTP];
#pragma unroll
    for (int hd = 0; hd < NH; ++hd) {
#pragma unroll
        for (int kt = 0; kt < 4; ++kt) tblacc[hd][kt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < KT; ++k) dwacc[hd][k] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int k = 0; k < KTP; ++k) wpacc[k] = f32x4{0.f, 0.f, 0.f, 0.f};

    const uint2 ones2 = make_uint2(0x3f803f80u, 0x3f803f80u);

    // A head's weights and biases.  Narrow layers read them before the barrier in front of their use, so that the
    // wait there hides the reads' latency; wide ones, short of registers, where they are used.
    constexpr bool AHEAD = !Cf::SPLIT;
    struct HeadOps {
        uint4 pt[ET][KSC], qkv[3][ET][KS];
        f32x4 bT[3][ET];   // bias of the rows 4q + j
    } ho;
    for (int win = blockIdx.x; win < g.nW; win += gridDim.x) {
        // (the lane index as this window's address arithmetic sees it: opaque, so that the many per-lane LDS and
        // memory addresses below are computed where they are used instead of being kept, and spilled, across windows)
        int lane_w = threadIdx.x & 63;
        asm volatile("" : "+v"(lane_w));
        const int lane = lane_w, l16 = lane & 15, q = lane >> 4;
        const int tr = (l16 & 3) * 16 + 4 * q + (l16 >> 2); // this lane's place in a packed tile that is read turned
        auto read_head = [&](int hx) {
#pragma unroll
            for (int et = 0; et < ET; ++et) {
#pragma unroll
                for (int ks = 0; ks < KSC; ++ks) ho.pt[et][ks] = wpt[((hx * ET + et) * KSC + ks) * 64 + lane];
#pragma unroll
                for (int t = 0; t < 3; ++t) {
                    const float *bias = bqkv + (hx * 3 + t) * (16 * ET) + 16 * et;
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) ho.qkv[t][et][ks] = wq[fq<Cf>(hx, t, et, ks) * 64 + lane];
                    ho.bT[t][et] = *reinterpret_cast<const f32x4 *>(bias + 4 * q);
                }
            }
        };
        if (!PIPE) load_rows(win);
        if (AHEAD) read_head(NH - 1);
        take_rows();
        // Eq. 8: the input of a group with a cascade term is F = x slice + previous group's output,
        // rounded to bf16 exactly as the forward kernels round it (it is the operand of their QKV
        // product), so that q, k, v and the probabilities are recomputed from the same values
        if (g.cascade) {
#pragma unroll
            for (int gi = (GB > 1 ? GB : 1); gi <= GE; ++gi)
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    uint4 &f = xf[gi][ks];
                    const uint4 a = af[gi - 1][ks];
                    f.x = pack_bf16x2(bf16_lo(f.x) + bf16_lo(a.x), bf16_hi(f.x) + bf16_hi(a.x));
                    f.y = pack_bf16x2(bf16_lo(f.y) + bf16_lo(a.y), bf16_hi(f.y) + bf16_hi(a.y));
                    f.z = pack_bf16x2(bf16_lo(f.z) + bf16_lo(a.z), bf16_hi(f.z) + bf16_hi(a.z));
                    f.w = pack_bf16x2(bf16_lo(f.w) + bf16_lo(a.w), bf16_hi(f.w) + bf16_hi(a.w));
                }
        }
        const long tok = token_of(win);
        const int wr = win - quotient(win, per_img, r_img) * per_img, wi = quotient(wr, g.nwj, r_nwj);
        const bool lastrow = s > 0 && wi == g.nwi - 1, lastcol = s > 0 && wr - wi * g.nwj == g.nwj - 1;

        // ---- d w_proj, d b_proj: dY operands (read turned) and A^T rows [channel][token] through LDS, K = 64 tokens ----
        if (WPROJ) {
#pragma unroll
        for (int ks = 0; ks < KSC; ++ks) dybuf[(ks * 4 + wv) * 64 + lane] = dyf[ks];
#pragma unroll
        for (int ct = 0; ct < CTP; ++ct) {
            f32x4 tN = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int gi = 0; gi < G; ++gi)
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
                    if (need_a(gi) && ranges_overlap(gi * CG + 32 * ks, gi * CG + (32 * ks + 32 < CG ? 32 * ks + 32 : CG),
                                                     B::WC0 + 16 * ct, B::WC0 + 16 * ct + 16))
                        tN = mma32(af[gi][ks], select_slot(B::WC0 + 16 * ct + l16, gi * CG + 32 * ks + 8 * q), tN);
            uint2 pk = pack_bf16x4(tN);
            if (16 * ct + l16 == B::WCN) pk = ones2;
            *reinterpret_cast<uint2 *>(abuf + (16 * ct + l16) * LW + 16 * wv + 4 * q) = pk;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < KTP; ++k) {
            const int ti = 4 * k + wv;
            if (4 * k + 3 < NTP || ti < NTP) {
                const int ot = ti / CTP, ct = ti - ot * CTP;
                // (k-slots: tokens 4q .. of one tile of 16, then of the next; the 16 channels of row tile ot are two lane
                // groups of an operand of dy)
                const uint8_t *ar = reinterpret_cast<const uint8_t *>(dybuf + (ot >> 1) * 256 + (2 * (ot & 1) + ((l16 & 3) >> 1)) * 16 +
                                                                      4 * q + (l16 >> 2)) + 8 * (l16 & 1);
                const uint16_t *br = abuf + (16 * ct + l16) * LW + 4 * q;
#pragma unroll
                for (int kp = 0; kp < 2; ++kp)
                    wpacc[k] = mma32(cat(lds_read_tr(ar + 2048 * kp), lds_read_tr(ar + 2048 * kp + 1024)),
                                     cat(*reinterpret_cast<const uint2 *>(br + 32 * kp),
                                         *reinterpret_cast<const uint2 *>(br + 32 * kp + 16)), wpacc[k]);
            }
        }
        }

        f32x4 dFT[HG][ET], cascT[HG][ET];
#pragma unroll
        for (int hdr = 0; hdr < NH; ++hdr) {
            const int hd = HE - 1 - hdr; // groups in reverse order
            const int hx = hd - HB;      // index into this launch's fragments and accumulators
            const int gi = hd / HG, hl = hd % HG;
            const bool casc_out = gi < G - 1 && g.cascade; // this group's output feeds the next group
            const int g_hi = (gi + 1) * HG - 1, g_lo = gi * HG; // the heads of the group, top first
            const bool next_in_regs = HB <= (gi + 1) * HG && HE >= (gi + 2) * HG; // group gi+1 done in this launch
            if (hd == g_hi) {
#pragma unroll
                for (int hlp = 0; hlp < HG; ++hlp)
#pragma unroll
                    for (int etp = 0; etp < ET; ++etp) dFT[hlp][etp] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
            if (!AHEAD) read_head(hx);
            // ---- dO^T of this head: adjoint of Eq. 7, plus the gradient arriving through Eq. 8 ----
            f32x4 dOT[ET];
#pragma unroll
            for (int et = 0; et < ET; ++et) {
                dOT[et] = f32x4{0.f, 0.f, 0.f, 0.f};
                if (casc_out) {
                    if (next_in_regs) {
                        dOT[et] = cascT[hl][et];
                    } else { // the next group was finished by earlier launches: its dF is the dx slice
                        const uint32_t lo = cgrad[hx][et].x, hi = cgrad[hx][et].y;
                        dOT[et] = f32x4{bf16_lo(lo), bf16_hi(lo), bf16_lo(hi), bf16_hi(hi)};
                    }
                }
#pragma unroll
                for (int ks = 0; ks < KSC; ++ks)
                    dOT[et] = mma32(ho.pt[et][ks], dyf[ks], dOT[et]);
            }
            // ---- recompute q, k and v of this wave's tokens ----
            f32x4 qT[ET], kT[ET], vT[ET];
#pragma unroll
            for (int et = 0; et < ET; ++et) {
                qT[et] = ho.bT[0][et];
                kT[et] = ho.bT[1][et];
                vT[et] = ho.bT[2][et];
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    qT[et] = mma32(ho.qkv[0][et][ks], xf[gi][ks], qT[et]);
                    kT[et] = mma32(ho.qkv[1][et][ks], xf[gi][ks], kT[et]);
                    vT[et] = mma32(ho.qkv[2][et][ks], xf[gi][ks], vT[et]);
                }
            }
            // ---- exchange: packed tiles, which their readers take in either orientation ----
            uint2 Qb[ET], dOb[ET];
#pragma unroll
            for (int et = 0; et < ET; ++et) {
                const int at = (wv * ET + et) * 64 + lane;
                Qb[et] = pack_bf16x4(qT[et]);
                dOb[et] = pack_bf16x4(dOT[et]);
                kb[at] = pack_bf16x4(kT[et]);
                vb[at] = pack_bf16x4(vT[et]);
                qb[at] = Qb[et];
                dob[at] = dOb[et];
            }
            float tb[4][4]; // bias of (query, key 16kt+4q+j)
            auto read_table = [&]() {
#pragma unroll
                for (int kt = 0; kt < 4; ++kt)
#pragma unroll
                    for (int j = 0; j < 4; ++j) tb[kt][j] = tblf[hx * NTBL + idx0 - 30 * kt - j];
            };
            if (AHEAD) read_table();
            __syncthreads();
            if (PIPE && hdr == NH - 1 && win + (int)gridDim.x < g.nW) load_rows(win + gridDim.x);

            // ---- query role: S^T, P^T, dP^T, dS^T for this wave's 16 queries, all 64 keys ----
            f32x4 st[4], dp[4];
#pragma unroll
            for (int kt = 0; kt < 4; ++kt) {
                st[kt] = f32x4{0.f, 0.f, 0.f, 0.f};
                dp[kt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int et = 0; et < ET; ++et) {
                    st[kt] = mma16(kb[(kt * ET + et) * 64 + lane], Qb[et], st[kt]);
                    dp[kt] = mma16(vb[(kt * ET + et) * 64 + lane], dOb[et], dp[kt]);
                }
            }
            if (!AHEAD) read_table();
#pragma unroll
            for (int kt = 0; kt < 4; ++kt)
#pragma unroll
                for (int j = 0; j < 4; ++j) st[kt][j] += tb[kt][j];
            if (lastrow || lastcol) {
#pragma unroll
                for (int kt = 0; kt < 4; ++kt)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if ((lastrow && rmask[kt]) || (lastcol && cmask[j])) st[kt][j] += kMask;
            }
            // (one by one, not in threes as max5f takes them: behind the mask that quiets half as many operands again, 216
            // for 144 in all instances.  32 images of 64x64, forward + backward, 1 / 2 / 3 / 6 groups: 161.8 / 129.4 /
            // 138.6 / 128.8 us in threes, 161.2 / 128.4 / 137.5 / 128.2 so.)
            float mx = -INFINITY;
#pragma unroll
            for (int kt = 0; kt < 4; ++kt)
#pragma unroll
                for (int j = 0; j < 4; ++j) mx = fmaxf(mx, st[kt][j]);
            mx = qgroup_max(mx);
            const float mxl = mx * kLog2e;
            float sum = 0.f;
#pragma unroll
            for (int kt = 0; kt < 4; ++kt)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    st[kt][j] = __builtin_amdgcn_exp2f(fmaf(st[kt][j], kLog2e, -mxl));
                    sum += st[kt][j];
                }
            sum = qgroup_sum(sum);
            const float inv = 1.0f / sum;
            float delta = 0.f;
#pragma unroll
            for (int kt = 0; kt < 4; ++kt)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    st[kt][j] *= inv;
                    delta = fmaf(st[kt][j], dp[kt][j], delta);
                }
            delta = qgroup_sum(delta);
            uint2 Pb[4], dSb[4];
#pragma unroll
            for (int kt = 0; kt < 4; ++kt) {
#pragma unroll
                for (int j = 0; j < 4; ++j) dp[kt][j] = st[kt][j] * (dp[kt][j] - delta);
                Pb[kt] = pack_bf16x4(st[kt]);
                dSb[kt] = pack_bf16x4(dp[kt]);
                tblacc[hx][kt] = mma16(ident, dSb[kt], tblacc[hx][kt]);
            }
            // for the key role: tiles (key tile, this wave's queries)
#pragma unroll
            for (int kt = 0; kt < 4; ++kt) {
                pbuf[(kt * 4 + wv) * 64 + lane] = Pb[kt];
                dsbuf[(kt * 4 + wv) * 64 + lane] = dSb[kt];
            }
            // dQ = scale * dS K
            uint2 gq[ET], gk[ET], gv[ET];
#pragma unroll
            for (int et = 0; et < ET; ++et) {
                f32x4 dqT = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kp = 0; kp < 2; ++kp)
                    dqT = mma32(cat(lds_read_tr(kb + (2 * kp * ET + et) * 64 + tr), lds_read_tr(kb + ((2 * kp + 1) * ET + et) * 64 + tr)),
                                cat(dSb[2 * kp], dSb[2 * kp + 1]), dqT);
                gq[et] = pack_bf16x4(dqT);
                gbuf[((0 * ET + et) * 4 + wv) * 64 + lane] = gq[et];
            }
            uint2 wx[3][ET][HG][ET]; // the head's Wqkv^T tiles
            auto read_wqt = [&]() {
#pragma unroll
                for (int t = 0; t < 3; ++t)
#pragma unroll
                    for (int et = 0; et < ET; ++et)
#pragma unroll
                        for (int hlp = 0; hlp < HG; ++hlp)
#pragma unroll
                            for (int etp = 0; etp < ET; ++etp) wx[t][et][hlp][etp] = wqt[fqt<Cf>(hx, t, et, hlp, etp) * 64 + lane];
            };
            if (AHEAD) read_wqt();
            __syncthreads();

            // ---- key role: dV = P^T dO, dK = scale * dS^T Q for this wave's 16 keys ----
            {
                uint4 pf[2], sf[2];
#pragma unroll
                for (int kp = 0; kp < 2; ++kp) {
                    const int at = (wv * 4 + 2 * kp) * 64 + tr;
                    pf[kp] = cat(lds_read_tr(pbuf + at), lds_read_tr(pbuf + at + 64));
                    sf[kp] = cat(lds_read_tr(dsbuf + at), lds_read_tr(dsbuf + at + 64));
                }
#pragma unroll
                for (int et = 0; et < ET; ++et) {
                    f32x4 dkT = f32x4{0.f, 0.f, 0.f, 0.f}, dvT = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int kp = 0; kp < 2; ++kp) {
                        const int a0 = (2 * kp * ET + et) * 64 + tr, a1 = a0 + ET * 64;
                        dkT = mma32(cat(lds_read_tr(qb + a0), lds_read_tr(qb + a1)), sf[kp], dkT);
                        dvT = mma32(cat(lds_read_tr(dob + a0), lds_read_tr(dob + a1)), pf[kp], dvT);
                    }
                    gk[et] = pack_bf16x4(dkT);
                    gv[et] = pack_bf16x4(dvT);
                    gbuf[((1 * ET + et) * 4 + wv) * 64 + lane] = gk[et];
                    gbuf[((2 * ET + et) * 4 + wv) * 64 + lane] = gv[et];
                }
            }
            // ---- first head of a group: F^T rows [channel][token] of the group input (Eq. 8) ----
            if (hd == g_hi) {
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    f32x4 tN = f32x4{0.f, 0.f, 0.f, 0.f};
                    if (2 * (ct >> 1) < 2 * KS && (ct >> 1) < KS) {
                        const uint4 sel = select_slot(16 * ct + l16, 32 * (ct >> 1) + 8 * q);
                        tN = mma32(xf[gi][(ct >> 1) < KS ? (ct >> 1) : 0], sel, tN);
                    }
                    uint2 pk = pack_bf16x4(tN);
                    if (16 * ct + l16 == CG) pk = ones2;
                    *reinterpret_cast<uint2 *>(fbuf + (16 * ct + l16) * LW + 16 * wv + 4 * q) = pk;
                }
            }
            // ---- d(q|k|v) through Wqkv^T into dF of the group ----
            auto w_at = [&](int t, int et, int hlp, int etp) {
                return AHEAD ? wx[t][et][hlp][etp] : wqt[fqt<Cf>(hx, t, et, hlp, etp) * 64 + lane];
            };
#pragma unroll
            for (int et = 0; et < ET; ++et) {
#pragma unroll
                for (int hlp = 0; hlp < HG; ++hlp)
#pragma unroll
                    for (int etp = 0; etp < ET; ++etp) {
                        dFT[hlp][etp] = mma16(w_at(0, et, hlp, etp), gq[et], dFT[hlp][etp]);
                        dFT[hlp][etp] = mma16(w_at(1, et, hlp, etp), gk[et], dFT[hlp][etp]);
                        dFT[hlp][etp] = mma16(w_at(2, et, hlp, etp), gv[et], dFT[hlp][etp]);
                    }
            }
            if (AHEAD && hdr + 1 < NH) read_head(hx - 1);
            __syncthreads();

            // ---- d w_qkv (and d b_qkv in the spare column) of this head: K = 64 tokens ----
#pragma unroll
            for (int k = 0; k < KT; ++k) {
                const int ti = 4 * k + wv;
                if (4 * k + 3 < NT || ti < NT) {
                    const int r = ti / CT, ct = ti - r * CT;
                    // (k-slots: tokens 4q .. of one tile of 16, then of the next)
                    const uint2 *ar = gbuf + r * 256 + tr;
                    const uint16_t *br = fbuf + (16 * ct + l16) * LW + 4 * q;
#pragma unroll
                    for (int kp = 0; kp < 2; ++kp)
                        dwacc[hx][k] = mma32(cat(lds_read_tr(ar + 128 * kp), lds_read_tr(ar + 128 * kp + 64)),
                                             cat(*reinterpret_cast<const uint2 *>(br + 32 * kp),
                                                 *reinterpret_cast<const uint2 *>(br + 32 * kp + 16)), dwacc[hx][k]);
                }
            }

            // ---- end of a group: dx slice; keep dF as the cascade gradient of the previous group ----
            if (hd == g_lo) {
#pragma unroll
                for (int hlp = 0; hlp < HG; ++hlp)
#pragma unroll
                    for (int etp = 0; etp < ET; ++etp) {
                        const int c0 = 16 * etp + 4 * q;
                        uint32_t *dst = reinterpret_cast<uint32_t *>(dx + tok * C + gi * CG + hlp * D + c0);
                        const uint2 v = pack_bf16x4(dFT[hlp][etp]);
                        if (c0 < D) dst[0] = v.x;
                        if (c0 + 2 < D) dst[1] = v.y;
                        cascT[hlp][etp] = dFT[hlp][etp];
                    }
            }
        }
    }

    // ---- flush: this workgroup's partial sums, in parameter order.  The packed query weights
    // carry the 1/sqrt(d) of the scores, so their gradients get it back here. ----
    const float scale = 1.0f / sqrtf((float)D);
    float *mine = part + (size_t)blockIdx.x * B::L_TOTAL;
    if (WPROJ) {
#pragma unroll
    for (int k = 0; k < KTP; ++k) {
        const int ti = 4 * k + wv;
        if (ti < NTP) {
            const int ot = ti / CTP, ct = ti - ot * CTP;
            const int c = 16 * ct + l16, o = 16 * ot + 4 * q;
            float *dst = mine + (c < B::WCN ? B::L_DWP + o * B::WCN + c : B::L_DBP + o);
            const int step = c < B::WCN ? B::WCN : 1;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (o + j < C && (c < B::WCN || (B::BPROJ && c == B::WCN))) dst[j * step] = wpacc[k][j];
        }
    }
    }
#pragma unroll
    for (int hx = 0; hx < NH; ++hx) {
        const int hd = HB + hx;
        const int gi = hd / HG, hl = hd % HG;
#pragma unroll
        for (int k = 0; k < KT; ++k) {
            const int ti = 4 * k + wv;
            if (ti < NT) {
                const int r = ti / CT, ct = ti - r * CT;
                const int t = r / ET, et = r - t * ET;
                const int c = 16 * ct + l16, e = 16 * et + 4 * q;
                const int row = ((gi - GB) * 3 + t) * CG + hl * D + e;
                float *dst = mine + (c < CG ? B::L_DWQ + row * CG + c : B::L_DBQ + row);
                const int step = c < CG ? CG : 1;
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (e + j < D && c <= CG) dst[j * step] = t == 0 ? dwacc[hx][k][j] * scale : dwacc[hx][k][j];
            }
        }
    }
    // bias-table gradient: (query, key) accumulators -> table entries, summed in a fixed order
    // [head][64 queries][64 keys], as many heads at a time as LDS takes; rows 65 floats apart (the 16 query rows a
    // store touches then fall on different banks)
    constexpr int MP = 65, SQ = 64 * MP;
    constexpr int HP = (int)(B::LDS_BYTES / (4 * SQ)) < NH ? (int)(B::LDS_BYTES / (4 * SQ)) : NH;
    static_assert(HP > 0, "the table flush takes LDS over");
    float *mats = reinterpret_cast<float *>(lds);
#pragma unroll
    for (int h0 = 0; h0 < NH; h0 += HP) {
        __syncthreads();
#pragma unroll
        for (int hx = h0; hx < h0 + HP && hx < NH; ++hx)
#pragma unroll
            for (int kt = 0; kt < 4; ++kt)
#pragma unroll
                for (int j = 0; j < 4; ++j) mats[(hx - h0) * SQ + (16 * wv + l16) * MP + 16 * kt + 4 * q + j] = tblacc[hx][kt][j];
        __syncthreads();
#pragma unroll
        for (int hx = h0; hx < h0 + HP && hx < NH; ++hx) {
            const float *mat = mats + (hx - h0) * SQ;
            // Four threads share the offsets (dr0, dc0), (dr0 - M, dc0), (dr0, dc0 - M), (dr0 - M, dc0 - M)
            // with 0 <= dr0, dc0 < M: for every query (rn, cn) exactly one of the four has its key
            // inside the window, key = ((rn - dr0) mod M, (cn - dc0) mod M), so the four entries take
            // M*M terms together and each thread sums those of two query rows: 16 reads, all in
            // flight together, the same for every thread.
            const int grp4 = tid >> 2, part = tid & 3;
            const int dr0 = grp4 >> 3, dc0 = grp4 & 7;
            float a00 = 0.f, a01 = 0.f, a10 = 0.f, a11 = 0.f; // [row wrapped][column wrapped]
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int rn = 2 * part + i;
                const bool wr = rn < dr0;
                const int rm = (rn - dr0) & (M - 1);
                float s0 = 0.f, s1 = 0.f;
#pragma unroll
                for (int cn = 0; cn < M; ++cn) {
                    const bool wc = cn < dc0;
                    const float v = mat[(rn * M + cn) * MP + rm * M + ((cn - dc0) & (M - 1))];
                    s0 += wc ? 0.f : v;
                    s1 += wc ? v : 0.f;
                }
                a00 += wr ? 0.f : s0;
                a01 += wr ? 0.f : s1;
                a10 += wr ? s0 : 0.f;
                a11 += wr ? s1 : 0.f;
            }
            a00 += __shfl_xor(a00, 1); a01 += __shfl_xor(a01, 1); a10 += __shfl_xor(a10, 1); a11 += __shfl_xor(a11, 1);
            a00 += __shfl_xor(a00, 2); a01 += __shfl_xor(a01, 2); a10 += __shfl_xor(a10, 2); a11 += __shfl_xor(a11, 2);
            // thread `part` of the four writes entry `part`
            const int e00 = (dr0 + M - 1) * (2 * M - 1) + dc0 + M - 1;
            const float val = part == 0 ? a00 : part == 1 ? a01 : part == 2 ? a10 : a11;
            const int e = e00 - ((part & 1) ? M : 0) - ((part & 2) ? M * (2 * M - 1) : 0);
            const bool ok = !((part & 1) && dc0 == 0) && !((part & 2) && dr0 == 0);
            if (ok) mine[B::L_TBL + hx * NTBL + e] = val;
        }
    }
}

// (segment table: ReduceOut, fused.h)
// A block sums 32 * V consecutive entries over all partial vectors: thread (column group, slice) adds the
// partials slice, slice + 32, ... (V entries each, one load of 4 V bytes: with V = 2 a wave half reads 256
// contiguous bytes of a partial vector), the 32 slices meet in LDS in a fixed order.
template <int V>
__device__ __forceinline__ void reduce_partials_block(const float *__restrict__ part, int nparts, int n,
                                                      const ReduceOut &out, int accumulate, int block, float *red)
{
    constexpr int SL = 32; // slices of the partials, one per wave half: few additions per thread, all loads in flight
    constexpr int RP = 32 * V + 1; // pitch of red[SL][RP]
    typedef float vec_t __attribute__((ext_vector_type(V)));
    const int col = threadIdx.x & 31, slice = threadIdx.x >> 5;
    const int i0 = (block * 32 + col) * V;
    vec_t acc = 0.f;
    if (i0 < n) {
        vec_t a[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) a[u] = 0.f;
        int w = slice;
        for (; w + 7 * SL < nparts; w += 8 * SL) {
#pragma unroll
            for (int u = 0; u < 8; ++u) a[u] += *reinterpret_cast<const vec_t *>(part + (size_t)(w + SL * u) * n + i0);
        }
        for (; w < nparts; w += SL) a[0] += *reinterpret_cast<const vec_t *>(part + (size_t)w * n + i0);
        acc = ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
    }
#pragma unroll
    for (int v = 0; v < V; ++v) red[slice * RP + col * V + v] = acc[v];
    __syncthreads();
    const int c = threadIdx.x, i = block * 32 * V + c;
    if (c < 32 * V && i < n && i < out.begin[out.nseg]) { // (entries behind the last segment pad the vectors' stride)
        float t[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            t[u] = (red[(4 * u) * RP + c] + red[(4 * u + 1) * RP + c]) + (red[(4 * u + 2) * RP + c] + red[(4 * u + 3) * RP + c]);
        const float sum = ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]));
        int seg = 0;
        while (seg < out.nseg - 1 && i >= out.begin[seg + 1]) ++seg;
        const int k = i - out.begin[seg];
        float *dst = out.ptr[seg] + k;
        if (out.tbl_heads > 0 && seg == out.nseg - 1) {
            const int hd = k / out.tbl_entries, e = k - hd * out.tbl_entries;
            dst = out.ptr[seg] + e * out.tbl_stride + out.tbl_head0 + hd;
        }
        if (out.row_len > 0 && seg == out.row_seg) dst = out.ptr[seg] + k / out.row_len * out.row_stride + k % out.row_len;
        *dst = accumulate ? *dst + sum : sum;
    }
}

template <int V>
__global__ __launch_bounds__(1024) void reduce_partials_kernel(const float *__restrict__ part, int nparts,
                                                               int n, ReduceOut out, int accumulate)
{
    __shared__ float red[32 * (32 * V + 1)];
    reduce_partials_block<V>(part, nparts, n, out, accumulate, (int)blockIdx.x, red);
}

// Two sums in one launch: blocks [0, blocks1) take the second (one entry per load: the short vectors of a bias-table
// gradient, of which there may be many, so these blocks start first), the others the first (V entries per load); blocks2
// blocks between them, if any, a third (V2 entries per load).
template <int V, int V2>
__global__ __launch_bounds__(1024) void reduce_partials_pair_kernel(ReduceJob j0, int blocks1, ReduceJob j1, int blocks2, ReduceJob j2)
{
    __shared__ float red[32 * (32 * (V > V2 ? V : V2) + 1)];
    if ((int)blockIdx.x < blocks1)
        reduce_partials_block<1>(j1.part, j1.nparts, j1.n, j1.out, j1.accumulate, (int)blockIdx.x, red);
    else if ((int)blockIdx.x < blocks1 + blocks2)
        reduce_partials_block<V2>(j2.part, j2.nparts, j2.n, j2.out, j2.accumulate, (int)blockIdx.x - blocks1, red);
    else
        reduce_partials_block<V>(j0.part, j0.nparts, j0.n, j0.out, j0.accumulate, (int)blockIdx.x - blocks1 - blocks2, red);
}

// d w_proj, d b_proj of wide layers: dY^T [A | 1] over plain token rows, 128 tokens per pass of a workgroup
// of eight waves.  Both operands are moved into [channel][token] LDS rows by selector MFMAs; wave w owns
// the output row tiles (w % 4) * RW .. + RW - 1 and half of the column tiles; the spare column C carries the
// bias sums.  The next pass's rows are fetched under the products of the pass in hand.
template <class Cf> struct WprojGradCfg {
    static constexpr int C = Cf::C, KSC = Cf::KSC;
    static constexpr int OTP = (C + 15) / 16, CTP = C / 16 + 1;
    static constexpr int NWV = 8, TOK = 16 * NWV;
    static constexpr int RW = (OTP + 3) / 4;       // row tiles per wave (four row groups)
    static constexpr int CW = (CTP + 1) / 2;       // column tiles per wave (two column halves)
    static constexpr int LW = TOK + 8;             // pitch (bf16) of the [channel][128 tokens] rows
    static constexpr size_t LDS_BYTES = (size_t)16 * (OTP + CTP) * LW * 2;
    static_assert(LDS_BYTES <= 160 * 1024, "LDS budget");
};

template <class Cf>
__global__ __launch_bounds__(512, 1) void wproj_grad_kernel(long T, const bf16_t *__restrict__ dy,
                                                            const bf16_t *__restrict__ attn,
                                                            float *__restrict__ part)
{
    using P = WprojGradCfg<Cf>;
    constexpr int C = Cf::C, KSC = Cf::KSC, OTP = P::OTP, CTP = P::CTP, LW = P::LW, RW = P::RW, CW = P::CW;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    uint16_t *dybuf = reinterpret_cast<uint16_t *>(lds);
    uint16_t *abuf = dybuf + 16 * OTP * LW;
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, q = lane >> 4;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rg = wv & 3, ch = wv >> 2;
    const uint2 ones2 = make_uint2(0x3f803f80u, 0x3f803f80u);

    f32x4 acc[RW][CW];
#pragma unroll
    for (int r = 0; r < RW; ++r)
#pragma unroll
        for (int c = 0; c < CW; ++c) acc[r][c] = f32x4{0.f, 0.f, 0.f, 0.f};

    // The rows of the next pass are on their way while this one's are computed with.  They are taken as loaded, from a
    // valid row; the row's end and rows past the last count as zero where they are used (a select behind the load is a
    // wait behind the load; 32 images of 64x64, two groups, fwd + bwd: 352.4 -> 349.0 us).
    uint4 dyn[KSC], an[KSC];
    auto load_rows = [&](long tile) {
        const long tok = tile * P::TOK + 16 * wv + l16, row = tok < T ? tok : 0;
#pragma unroll
        for (int ks = 0; ks < KSC; ++ks) {
            dyn[ks] = load_piece4<C>(dy + row * C, 32 * ks + 8 * q);
            an[ks] = load_piece4<C>(attn + row * C, 32 * ks + 8 * q);
        }
    };

    const long ntile = (T + P::TOK - 1) / P::TOK;
    if ((long)blockIdx.x < ntile) load_rows(blockIdx.x);
    for (long tile = blockIdx.x; tile < ntile; tile += gridDim.x) {
        // this lane's token of the pass as operands: channels 32 ks + 8 q .. + 7 of dy and of the saved outputs
        const bool ok = tile * P::TOK + 16 * wv + l16 < T;
        uint4 dyf[KSC], af[KSC];
#pragma unroll
        for (int ks = 0; ks < KSC; ++ks) {
            dyf[ks] = ok ? piece4<C>(dyn[ks], 32 * ks, q) : make_uint4(0u, 0u, 0u, 0u);
            af[ks] = ok ? piece4<C>(an[ks], 32 * ks, q) : make_uint4(0u, 0u, 0u, 0u);
        }
        if (tile + (long)gridDim.x < ntile) load_rows(tile + gridDim.x);
        __syncthreads(); // the previous pass's rows are consumed
#pragma unroll
        for (int ot = 0; ot < OTP; ++ot) {
            const f32x4 tN = mma32(dyf[ot >> 1], select_slot(16 * ot + l16, 32 * (ot >> 1) + 8 * q),
                                   f32x4{0.f, 0.f, 0.f, 0.f});
            *reinterpret_cast<uint2 *>(dybuf + (16 * ot + l16) * LW + 16 * wv + 4 * q) = pack_bf16x4(tN);
        }
#pragma unroll
        for (int ct = 0; ct < CTP; ++ct) {
            f32x4 tN = f32x4{0.f, 0.f, 0.f, 0.f};
            if ((ct >> 1) < KSC)
                tN = mma32(af[(ct >> 1) < KSC ? (ct >> 1) : 0], select_slot(16 * ct + l16, 32 * (ct >> 1) + 8 * q), tN);
            uint2 pk = pack_bf16x4(tN);
            if (16 * ct + l16 == C) pk = ones2; // (tokens past the end have dy = 0)
            *reinterpret_cast<uint2 *>(abuf + (16 * ct + l16) * LW + 16 * wv + 4 * q) = pk;
        }
        __syncthreads();
#pragma unroll
        for (int kp = 0; kp < P::TOK / 32; ++kp) {
            uint4 afr[RW];
#pragma unroll
            for (int r = 0; r < RW; ++r) {
                const int ot = rg * RW + r;
                const uint16_t *ar = dybuf + (16 * (ot < OTP ? ot : 0) + l16) * LW + 32 * kp + 8 * q;
                afr[r] = cat(*reinterpret_cast<const uint2 *>(ar), *reinterpret_cast<const uint2 *>(ar + 4));
            }
#pragma unroll
            for (int c = 0; c < CW; ++c) {
                const int ct = ch * CW + c;
                const uint16_t *br = abuf + (16 * (ct < CTP ? ct : 0) + l16) * LW + 32 * kp + 8 * q;
                const uint4 bf = cat(*reinterpret_cast<const uint2 *>(br), *reinterpret_cast<const uint2 *>(br + 4));
#pragma unroll
                for (int r = 0; r < RW; ++r) acc[r][c] = mma32(afr[r], bf, acc[r][c]);
            }
        }
    }
    float *mine = part + (size_t)blockIdx.x * (C * C + C); // [d w_proj | d b_proj]
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        const int ot = rg * RW + r;
        if (ot < OTP) {
#pragma unroll
            for (int c = 0; c < CW; ++c) {
                const int ct = ch * CW + c;
                const int col = 16 * ct + l16;
                if (ct < CTP) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int o = 16 * ot + 4 * q + j;
                        if (o < C) {
                            if (col < C) mine[o * C + col] = acc[r][c][j];
                            else if (col == C) mine[C * C + o] = acc[r][c][j];
                        }
                    }
                }
            }
        }
    }
}

// Head chunks of the backward, in launch order (last group first).  Chunks are whole groups, so
// the only thing one launch hands to the next is the cascade gradient, which is the dx slice it
// wrote.  Three heads per launch keep the accumulators small enough for two workgroups per CU.
// Wide layers of three groups go a group of two heads a launch (their weights and row buffers fill LDS).
template <bool SPLIT, int G> struct ChunkPlan;
template <> struct ChunkPlan<false, 6> { static constexpr int N = 2; static constexpr int B[2] = {3, 0}, E[2] = {6, 3}; };
template <> struct ChunkPlan<true, 3> { static constexpr int N = 3; static constexpr int B[3] = {4, 2, 0}, E[3] = {6, 4, 2}; };
template <> struct ChunkPlan<true, 2> { static constexpr int N = 0; }; // (wide_heads_bwd.hip)

// Workgroups of a backward launch: narrow layers run two per compute unit.
// `cus` = the device's compute units for a launch, kSizingCus for the scratch size (a launch never
// uses more workgroups than the size was computed for).
int bwd_grid(const Geom &g, int cus)
{
    if (cus > kSizingCus) cus = kSizingCus;
    const int grid = (g.C <= 64 ? 2 : 1) * cus;
    return grid > g.nW ? g.nW : grid;
}

struct GradOut {
    float *dw_qkv, *db_qkv, *dw_proj, *db_proj, *dtable;
    int accumulate;
};

} // namespace

// entries per load: two or four where every partial vector starts on such a boundary and enough workgroups
// remain to fill the chip (24570 entries, 256 vectors: 192 workgroups of four entries a load 7.9 us, 384 of two 8.8)
static int reduce_width(const float *part, int n)
{
    const uintptr_t at = reinterpret_cast<uintptr_t>(part);
    if (n % 4 == 0 && at % 16 == 0 && n >= 180 * 128) return 4;
    if (n % 2 == 0 && at % 8 == 0 && n >= 200 * 64) return 2;
    return 1;
}

hipError_t launch_reduce(const float *part, int nparts, int n, const ReduceOut &out, int accumulate, hipStream_t s)
{
    KernelTimer kt(K_REDUCE, s);
    switch (reduce_width(part, n)) {
    case 4: hipLaunchKernelGGL(reduce_partials_kernel<4>, dim3((n + 127) / 128), dim3(1024), 0, s, part, nparts, n, out, accumulate); break;
    case 2: hipLaunchKernelGGL(reduce_partials_kernel<2>, dim3((n + 63) / 64), dim3(1024), 0, s, part, nparts, n, out, accumulate); break;
    default: hipLaunchKernelGGL(reduce_partials_kernel<1>, dim3((n + 31) / 32), dim3(1024), 0, s, part, nparts, n, out, accumulate); break;
    }
    return hipGetLastError();
}

template <int V, int V2>
static hipError_t launch_reduce_jobs(const ReduceJob &a, const ReduceJob &b, const ReduceJob &c, hipStream_t s)
{
    KernelTimer kt(K_REDUCE, s);
    const int blocks0 = (a.n + 32 * V - 1) / (32 * V), blocks1 = (b.n + 31) / 32, blocks2 = (c.n + 32 * V2 - 1) / (32 * V2);
    hipLaunchKernelGGL((reduce_partials_pair_kernel<V, V2>), dim3(blocks0 + blocks1 + blocks2), dim3(1024), 0, s, a, blocks1, b, blocks2, c);
    return hipGetLastError();
}

// The third sum four entries a load where its vectors allow that, whatever the first takes.  (With three groups of 60 channels the
// first's vectors have 10980 entries, one a load, the projection's 32580: all one a load, 2048 windows of 8x8, forward +
// backward, 347.6 us, now 345.1; 1408 windows 282.5, now 280.2.)
hipError_t launch_reduce_three(const ReduceJob &a, const ReduceJob &b, const ReduceJob &c, hipStream_t s)
{
    const int v2 = c.n > 0 ? reduce_width(c.part, c.n) : 0;
    int v = reduce_width(a.part, a.n);
    if (c.n > 0 && v2 < v) v = v2;
    switch (v) {
    case 4: return launch_reduce_jobs<4, 4>(a, b, c, s);
    case 2: return v2 == 4 ? launch_reduce_jobs<2, 4>(a, b, c, s) : launch_reduce_jobs<2, 2>(a, b, c, s);
    default: return v2 == 4 ? launch_reduce_jobs<1, 4>(a, b, c, s) : launch_reduce_jobs<1, 1>(a, b, c, s);
    }
}

hipError_t launch_reduce_pair(const ReduceJob &a, const ReduceJob &b, hipStream_t s) { return launch_reduce_three(a, b, ReduceJob{}, s); }

namespace {

// One chunk of heads: the kernel, then the sum of its partials into the gradients it owns.  The
// scratch is free again afterwards, so every chunk (and the projection's weight gradient of wide
// layers) uses the same buffer: its size is the largest chunk's, not the sum.
template <class Cf, int HB, int HE, bool WPROJ>
hipError_t launch_chunk(const Geom &g, int grid, const bf16_t *x, const bf16_t *dy, const bf16_t *attn,
                        const uint8_t *pack, const bf16_t *table, bf16_t *dx, float *part, const GradOut &go,
                        hipStream_t s)
{
    using B = BwdCfg<Cf, HB, HE, WPROJ>;
    static_assert(B::LDS_BYTES <= 160 * 1024, "LDS budget");
    auto kern = fused_bwd_kernel<Cf, HB, HE, WPROJ>;
    if (hipError_t ea = allow_dynamic_lds(reinterpret_cast<const void *>(kern), B::LDS_BYTES); ea != hipSuccess) return ea;
    {
        KernelTimer kt(K_FUSED_BWD, s);
        hipLaunchKernelGGL(kern, dim3(grid), dim3(256), B::LDS_BYTES, s, g, x, dy, attn, pack, table, dx, part);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    constexpr int CG = Cf::CG;
    ReduceOut out{};
    int k = 0;
    static_assert(2 * B::NG * 3 + 3 <= ReduceOut::MAXSEG, "segment table");
    for (int gi = 0; gi < B::NG; ++gi)
        for (int t = 0; t < 3; ++t) { // d w_qkv rows of (group, q|k|v) owned by the chunk's heads
            out.ptr[k] = go.dw_qkv + (size_t)((B::GB + gi) * 3 * CG + t * CG) * CG;
            out.begin[k++] = B::L_DWQ + (gi * 3 + t) * CG * CG;
        }
    for (int gi = 0; gi < B::NG; ++gi)
        for (int t = 0; t < 3; ++t) {
            out.ptr[k] = go.db_qkv + (B::GB + gi) * 3 * CG + t * CG;
            out.begin[k++] = B::L_DBQ + (gi * 3 + t) * CG;
        }
    if (WPROJ) {
        out.row_seg = k; out.row_len = B::WCN; out.row_stride = Cf::C;
        out.ptr[k] = go.dw_proj + B::WC0; out.begin[k++] = B::L_DWP;
    }
    if (B::BPROJ) { out.ptr[k] = go.db_proj; out.begin[k++] = B::L_DBP; }
    out.ptr[k] = go.dtable; out.begin[k++] = B::L_TBL;
    out.begin[k] = B::L_END;
    out.nseg = k;
    out.tbl_heads = B::NH; out.tbl_entries = B::NTBL; out.tbl_stride = Cf::HEADS; out.tbl_head0 = HB;
    return launch_reduce(part, grid, B::L_TOTAL, out, go.accumulate, s);
}

template <class Cf, int I = 0>
hipError_t launch_chunks(const Geom &g, int grid, const bf16_t *x, const bf16_t *dy, const bf16_t *attn,
                         const uint8_t *pack, const bf16_t *table, bf16_t *dx, float *part, const GradOut &go,
                         hipStream_t s)
{
    using Plan = ChunkPlan<Cf::SPLIT, Cf::G>;
    if constexpr (I < Plan::N) {
        hipError_t e = launch_chunk<Cf, Plan::B[I], Plan::E[I], !Cf::SPLIT>(
            g, grid, x, dy, attn, pack, table, dx, part, go, s);
        if (e != hipSuccess) return e;
        return launch_chunks<Cf, I + 1>(g, grid, x, dy, attn, pack, table, dx, part, go, s);
    }
    return hipSuccess;
}

// floats of the largest per-workgroup partial vector over the launches of a layer
template <class Cf, int I = 0> constexpr int max_partial()
{
    using Plan = ChunkPlan<Cf::SPLIT, Cf::G>;
    if constexpr (I < Plan::N) {
        constexpr int mine = BwdCfg<Cf, Plan::B[I], Plan::E[I], !Cf::SPLIT>::L_TOTAL;
        constexpr int rest = max_partial<Cf, I + 1>();
        return mine > rest ? mine : rest;
    } else {
        return Cf::SPLIT ? Cf::C * Cf::C + Cf::C : 0;
    }
}

// d w_proj, d b_proj of a wide layer: the kernel, then the sum of its partials, in the launch of `sums` where there are any.
template <class Cf>
hipError_t run_wproj_grad(const Geom &g, int grid, const bf16_t *dy, const bf16_t *attn, float *part, float *dw_proj,
                          float *db_proj, int accumulate, const ReduceJob *sums, hipStream_t s)
{
    using P = WprojGradCfg<Cf>;
    constexpr size_t lds = P::LDS_BYTES;
    auto kern = wproj_grad_kernel<Cf>;
    if (hipError_t ea = allow_dynamic_lds(reinterpret_cast<const void *>(kern), lds); ea != hipSuccess) return ea;
    {
        KernelTimer kt(K_WPROJ_GRAD, s);
        hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * P::NWV), lds, s, g.T, dy, attn, part);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    ReduceJob j{};
    j.part = part; j.nparts = grid; j.n = Cf::C * Cf::C + Cf::C; j.accumulate = accumulate;
    j.out.ptr[0] = dw_proj; j.out.begin[0] = 0;
    j.out.ptr[1] = db_proj; j.out.begin[1] = Cf::C * Cf::C;
    j.out.begin[2] = Cf::C * Cf::C + Cf::C;
    j.out.nseg = 2;
    return sums ? launch_reduce_three(sums[0], sums[1], j, s) : launch_reduce(part, grid, j.n, j.out, accumulate, s);
}

template <class Cf>
hipError_t run_bwd(const Geom &g, const bf16_t *x, const bf16_t *dy, const bf16_t *attn,
                   const void *pack_, const bf16_t *table, bf16_t *dx, float *dw_qkv, float *db_qkv,
                   float *dw_proj, float *db_proj, float *dtable, int accumulate, void *ws, hipStream_t s)
{
    const uint8_t *pack = static_cast<const uint8_t *>(pack_);
    float *part = static_cast<float *>(ws);
    const int grid = bwd_grid(g, device_cu_count());
    if constexpr (Cf::SPLIT) {
        if (Cf::WIDE_HEADS || wide_bwd_supported(g)) { // (16-byte aligned tensors: the entry points check)
            ReduceJob sums[2]{};
            hipError_t e = Cf::WIDE_HEADS ? launch_wide_heads_bwd(g, x, dy, attn, pack, table, dx, dw_qkv, db_qkv, dtable, accumulate, ws, sums[0], s)
                                          : launch_wide_bwd(g, x, dy, attn, pack, dx, dw_qkv, db_qkv, dtable, accumulate, ws, sums, s);
            if (e != hipSuccess) return e;
            // The projection's partial vectors take the free part of the scratch.  Where that is too small for them (few
            // windows for the compute units) the sums before have to run first: a launch more.  (One launch for the last
            // three sums and the wider loads of reduce_width: 32 images of 64x64, three groups, forward + backward, 5 us.)
            const size_t room = Cf::WIDE_HEADS ? wide_heads_bwd_free_bytes(g) : wide_bwd_free_bytes(g);
            const bool fits = (size_t)grid * (Cf::C * Cf::C + Cf::C) * sizeof(float) <= room;
            if (!fits && (e = launch_reduce_pair(sums[0], sums[1], s)) != hipSuccess) return e;
            return run_wproj_grad<Cf>(g, grid, dy, attn, part, dw_proj, db_proj, accumulate, fits ? sums : nullptr, s);
        }
    }
    if constexpr (!Cf::WIDE_HEADS) {
        const GradOut go{dw_qkv, db_qkv, dw_proj, db_proj, dtable, accumulate};
        hipError_t e = launch_chunks<Cf>(g, grid, x, dy, attn, pack, table, dx, part, go, s);
        if (e != hipSuccess) return e;
        if constexpr (Cf::SPLIT) return run_wproj_grad<Cf>(g, grid, dy, attn, part, dw_proj, db_proj, accumulate, nullptr, s);
    }
    return hipSuccess;
}

#define GSWA_FUSED_SHAPES(X) X(60, 6, 6) X(180, 6, 2) X(180, 6, 3)

} // namespace

// One launch with a wavefront per head, or the launches per head group of this file.  Narrow layers of one to three groups take
// the former: 32 images of 64x64, forward + backward, 1 / 2 / 3 groups 160.4 / 128.6 / 138.8 us by head groups, 97.6 / 90.7 /
// 95.7 by heads; one image of 64x64 42.6 / 46.4 / 51.3 and 35.5 / 31.6 / 35.4; two of 16x16, two groups, 42.0 and 31.1.  Six
// groups would be a pipeline of six steps whose rows LDS has no room for.
bool fused_bwd_supported(const Geom &g)
{
    if (g.M != 8) return false;
    if (heads_bwd_supported(g)) return true;
#define X(C_, H_, G_) \
    if (g.C == C_ && g.heads == H_ && g.groups == G_) return true;
    GSWA_FUSED_SHAPES(X)
#undef X
    return false;
}

size_t fused_bwd_ws_bytes(const Geom &g)
{
    if (heads_bwd_supported(g)) return (heads_bwd_ws_bytes(g) + 255) & ~size_t(255);
    int total = 0;
#define X(C_, H_, G_) \
    if (g.C == C_ && g.heads == H_ && g.groups == G_) total = max_partial<FusedCfg<C_, H_, G_>>();
    GSWA_FUSED_SHAPES(X)
#undef X
    const size_t chunks = ((size_t)bwd_grid(g, kSizingCus) * total * 4 + 255) & ~size_t(255);
    const size_t wide = wide_heads_bwd_supported(g) ? wide_heads_bwd_ws_bytes(g) : wide_bwd_supported(g) ? wide_bwd_ws_bytes(g) : 0;
    return wide > chunks ? wide : chunks;
}

hipError_t launch_fused_bwd(const Geom &g, const bf16_t *x, const bf16_t *dy, const bf16_t *attn,
                            const void *pack, const bf16_t *table, bf16_t *dx, float *dw_qkv,
                            float *db_qkv, float *dw_proj, float *db_proj, float *dtable, int accumulate,
                            void *ws, hipStream_t s)
{
    if (heads_bwd_supported(g))
        return launch_heads_bwd(g, x, dy, attn, pack, table, dx, dw_qkv, db_qkv, dw_proj, db_proj, dtable, accumulate, ws, s);
#define X(C_, H_, G_)                                                   \
    if (g.C == C_ && g.heads == H_ && g.groups == G_)                   \
        return run_bwd<FusedCfg<C_, H_, G_>>(g, x, dy, attn, pack, table, dx, dw_qkv, db_qkv, dw_proj,      \
                                             db_proj, dtable, accumulate, ws, s);
    GSWA_FUSED_SHAPES(X)
#undef X
    return hipErrorInvalidValue;
}

} // namespace gswa
