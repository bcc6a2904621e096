// Forward of wide GSWA layers (C = 180, six heads of 30 channels, 8x8 or 16x16 windows) in one launch:
// shift + partition + per-group QKV projection (Eq. 6) with the cascade add (Eq. 8) + scores with
// relative bias and shift mask + softmax + PV + output projection (Eq. 7) + merge + reverse shift.
//
// A wavefront owns two 16-token tiles: two waves share an 8x8 window, eight a 16x16 one (few 8x8 windows: one tile, four
// waves).  x of all groups and all head outputs of its tokens stay in its registers, so do its probabilities; K and V of
// a head cross the waves of a window through LDS, already in the operand layout of the products that read them (one
// 16-byte write and read per lane and tile).  A workgroup is eight waves, two per SIMD (256 registers): one
// wave's vector instructions run under the other's products, which one wave per SIMD with a whole window
// (the organisation before, 512 registers) could not offer.  The weights of a wide layer (108 KB of QKV
// fragments, 72 KB of projection fragments) do not fit LDS together, so they pass through it as a stream of
// equal units: the QKV fragments of one head, then the projection in pieces of the same size.
//
// What bounds it: with 8x8 windows the steps between barriers, 1.4 to 2.2 k clocks of which 0.6 k are
// products and 0.6 k the LDS reads of the fragments (each serves two tiles); with 16x16 windows the vector
// instructions of the softmax.  Measured (one image of 512x512, two groups; a pass is the packing and this launch, passes
// one after the other, both organisations in turn on one card): 8x8 windows 134.8 -> 97.7 us, 16x16 windows 305.6 -> 154.0
// us (there two attention launches and one of the projection before); one image of 96x64 29.7 -> 20.2 us.  Steps at 8x8, as
// they were taken, on another card: two waves per window 130 -> 115 us, the next window's rows loaded under the projection,
// a few per step (in one go they stall the wave for 8 k clocks while memory serves the whole chip) and padded bias tables
// -> 111, windows of half the waves one step late -> 100, operands of the next products read under the present ones -> 94.
// The price is memory: 8x8 windows read 1.22 and write 1.31 times the map (1.12 and 1.26 with one wave per window), 239 MB
// for 225.
//
// The softmax's denominator is the sum of the probabilities as they were rounded to bf16 for the PV product (fp32 sums;
// row D of that product), and its reciprocal v_rcp_f32's; the organisation that 16x16 windows had before summed them
// unrounded and divided.  Error of y against fp64 over three maps, one to three groups, 12 seeds: 0.5 to 1.2 % smaller
// than that, or the same (64x64, two groups 3.904 -> 3.886e-3).
//
// Everything is kept with rows = features and column = token (T-form, see fused_bwd.hip), and a
// head of 30 channels is two 16-row tiles, i.e. exactly the 32 k-slots of one K=32 MFMA step in
// "head-padded order" (lane group q: features 4q..4q+3 and 16+4q..16+4q+3).  A packed pair of
// output tiles of a head therefore is, as it lies in registers, the operand of the next group's
// QKV projection (after the cascade add onto the x operand, rounded to bf16 like a stored
// activation) and of the output projection.
#include "fused.h"
#include "mfma.h"

namespace gswa {

namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kMaskLog2 = -100.0f * kLog2e; // the additive -100 of the shift mask, in base-2 units

// M: window side, TW: 16-token tiles a wave owns
template <class Cf, int M_, int TW_> struct WideFwdCfg {
    static constexpr int M = M_, TW = TW_, NT = M * M / 16; // tiles of a window
    static constexpr int NWAVES = 8, NTHREADS = 64 * NWAVES;
    static constexpr int WPW = NT / TW, WINS = NWAVES / WPW; // waves of a window, windows of a workgroup
    static constexpr int RPT = 16 / M;                       // window rows a tile covers
    static constexpr int NTBL = (2 * M - 1) * (2 * M - 1), TP = (NTBL + 7) & ~3; // bias table of a head, its pitch
    static constexpr int NTB = M == 8 ? TW : 1;              // query tiles taken through the softmax together
    // The weights pass through LDS as a stream of equal units: the QKV fragments of one head, then the projection
    // fragments in pieces of the same size (whole output tiles).
    static constexpr int FR_UNIT = 3 * Cf::ET * Cf::KSX;           // fragments (1 KB) of one unit
    static constexpr size_t UNIT_BYTES = (size_t)FR_UNIT * 1024;
    static constexpr int OT_UNIT = FR_UNIT / Cf::HEADS;            // output tiles of one projection unit
    static constexpr int NPU = Cf::OT / OT_UNIT;                   // projection units
    static constexpr int NU = Cf::HEADS + NPU;                     // units per window
    // A round (one window per slot) is a sequence of steps: q, k, v of head 0, its scores .. PV, the same of head 1, ...,
    // then the projection unit by unit.  Steps are grouped into times; a barrier ends a time.
    //   LATE   windows of the second half of the workgroup's waves run one time behind the others, so that on every SIMD
    //          one wave is in the vector instructions of a softmax while the other is in the products and LDS reads of
    //          its q, k, v: needs windows that share no wave between the halves
    //   MERGE  the scores of head h and q, k, v of head h + 1 make one time (k and v then need two buffers)
    static constexpr int LATE = WINS > 1 ? 1 : 0;
    static constexpr bool MERGE = !LATE && Cf::G > 1;
    static constexpr int NS = 2 * Cf::HEADS + NPU;                 // steps
    static constexpr int time_of(int step) { return !MERGE ? step : step < 2 * Cf::HEADS ? (step + 1) / 2 : step - Cf::HEADS; }
    static constexpr int NTIME = time_of(NS - 1) + 1;
    static constexpr int unit_time(int u) { return time_of(u < Cf::HEADS ? 2 * u : u + Cf::HEADS); } // first time unit u is read
    static constexpr int unit_at(int time) // the unit first read at this time (its loads leave one time before), or -1
    {
        for (int u = 0; u < NU; ++u)
            if (unit_time(u) == time) return u;
        return -1;
    }
    // LDS buffer of a unit: read at times unit_time .. unit_time + LATE, written from one time before
    static constexpr int NSLOT = 2 + LATE;
    static constexpr int unit_slot(int u)
    {
        constexpr int late[3][12] = {{0, 1, 2, 0, 1, 2, 1, 2}, {0, 1, 0, 1, 0, 2, 1, 0, 2, 1}, {0, 1, 2, 0, 1, 2, 0, 1, 2, 0, 1, 2}};
        return LATE ? late[Cf::G - 1][u] : u % 2;
    }
    // The rows of the next window are loaded a few operands at a time behind the steps of scores and projection (a burst
    // stalls the wave until memory has served the whole chip's), into the registers of a group whose q, k, v are done:
    // first operand of group gi that step `step` loads, or -1
    static constexpr int KPM = Cf::G == 1 ? 2 : 1; // operands per step and tile
    static constexpr int load_at(int step, int gi)
    {
        const int m = step < 2 * Cf::HEADS ? (step % 2 ? step / 2 : -1) : step - Cf::HEADS;
        const int k = (m - ((gi + 1) * Cf::HG - 1)) * KPM;
        return m >= 0 && k >= 0 && k < Cf::KSX ? k : -1;
    }
    // vector-memory instructions a wave issues in a step at least: loads of the next window, stores of y, of `attn`
    static constexpr int loads_in(int step)
    {
        int n = 0;
        for (int gi = 0; gi < Cf::G; ++gi) n += load_at(step, gi) >= 0 ? 2 * KPM * TW : 0;
        return n;
    }
    static constexpr int stores_in(int step) { return step < 2 * Cf::HEADS ? 0 : (OT_UNIT / 2 + OT_UNIT % 2) * TW; }
    static constexpr int keeps_in(int step) { return step < 2 * Cf::HEADS && step % 2 && step / 2 % Cf::HG == Cf::HG - 1 ? Cf::HG * TW : 0; }
    static constexpr bool slots_free()
    {
        for (int u = 0; u < 2 * NU; ++u) // (u: this round's and the next one's)
            for (int v = 0; v < u; ++v) {
                const int tu = unit_time(u % NU) + u / NU * NTIME, tv = unit_time(v % NU) + v / NU * NTIME;
                if (unit_slot(u % NU) == unit_slot(v % NU) && tu - 1 <= tv + LATE) return false;
            }
        return true;
    }
    // K and V of a head, all windows of the workgroup, as the operands they are read as (1 KB per tile and kind)
    static constexpr int KVBUF = MERGE ? 2 : 1;
    static constexpr size_t KV_WIN = (size_t)2 * NT * 1024, KV_BYTES = WINS * KV_WIN;
    // fp32 linear biases padded to whole tiles: [HEADS][q, k, v][32] (q in the scores' base-2 units; v of feature D: 1,
    // see below), then b_proj [16 OT]
    static constexpr int N_BQKV = Cf::HEADS * 3 * 32;
    static constexpr size_t OFF_BIAS = 0;
    static constexpr size_t OFF_TBL = (size_t)(N_BQKV + 16 * Cf::OT) * 4; // fp32 [HEADS][TP]
    static constexpr size_t OFF_LN = OFF_TBL + (size_t)Cf::HEADS * TP * 4; // fp32 [HEADS][32][gamma, beta], head-padded
    static constexpr size_t OFF_KV = OFF_LN + (size_t)Cf::HEADS * 32 * 8;
    static constexpr size_t OFF_W = OFF_KV + KVBUF * KV_BYTES;
    static constexpr size_t LDS_BYTES = OFF_W + NSLOT * UNIT_BYTES;
    static_assert(OFF_LN % 16 == 0 && OFF_KV % 16 == 0 && OFF_W % 16 == 0 && LDS_BYTES <= 160 * 1024, "LDS budget");
    static_assert(FR_UNIT % Cf::HEADS == 0 && Cf::OT % OT_UNIT == 0 && NU % 2 == 0 && NU <= 12,
                  "units tile the projection");
    static_assert(!LATE || (NWAVES / 2) % WPW == 0, "a window's waves run at the same time");
    static_assert(Cf::ET == 2 && Cf::D + 1 <= 32 && Cf::CG % Cf::D == 0, "heads of 17..31 channels: two tiles, a spare row");
    static_assert(NT % TW == 0 && NWAVES % WPW == 0, "whole windows per workgroup");
    static_assert(TW == 1 || TW == 2, "tiles of a wave");
};

// waits until at most N vector-memory operations are outstanding, and for everything in LDS
template <int N> __device__ __forceinline__ void wait_vm()
{
    static_assert(N < 64, "six bits");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4));
}

template <int Q0> __device__ __forceinline__ float qgroup_bcast(float v)
{
    const unsigned u = __float_as_uint(v);
    u32x2 r = __builtin_amdgcn_permlane32_swap(u, u, false, false); // {groups 0,1,0,1; groups 2,3,2,3}
    const unsigned h = r[Q0 >> 1];
    r = __builtin_amdgcn_permlane16_swap(h, h, false, false);       // {even group of each pair; odd group}
    return __uint_as_float(r[Q0 & 1]);
}

// LayerNorm of the wave's rows, held as operands in head-padded order (xh[group][step][tile]; zero beyond a head's
// D features), in place: a row is spread over the four lanes that share l16.  Mean first, then the squared distances
// from it, result rounded to bf16, as the LayerNorm kernels do it (which sum a row in another order).  gb: (gamma, beta) pairs [head][32], zero beyond D.
template <int G, int KSX, int TW, int C, int D>
__device__ __forceinline__ void layer_norm_operands(uint4 (&xh)[G][KSX][TW], const float4 *gb, int q, float eps)
{
    const bool hx = 16 + 4 * q < D, hy = 16 + 4 * q + 2 < D;
    float mean[TW], rstd[TW];
#pragma unroll
    for (int t = 0; t < TW; ++t) {
        float sum = 0.f;
#pragma unroll
        for (int k = 0; k < G * KSX; ++k) {
            const uint4 v = xh[k / KSX][k % KSX][t];
            sum += (bf16_lo(v.x) + bf16_hi(v.x)) + (bf16_lo(v.y) + bf16_hi(v.y));
            sum += (bf16_lo(v.z) + bf16_hi(v.z)) + (bf16_lo(v.w) + bf16_hi(v.w));
        }
        mean[t] = qgroup_sum(sum) / (float)C;
        float dev = 0.f;
#pragma unroll
        for (int k = 0; k < G * KSX; ++k) {
            const uint4 v = xh[k / KSX][k % KSX][t];
            auto sq = [&](uint32_t u) {
                const float a = bf16_lo(u) - mean[t], b = bf16_hi(u) - mean[t];
                return a * a + b * b;
            };
            dev += sq(v.x) + sq(v.y);
            dev += (hx ? sq(v.z) : 0.f) + (hy ? sq(v.w) : 0.f);
        }
        rstd[t] = rsqrtf(qgroup_sum(dev) / (float)C + eps);
    }
#pragma unroll
    for (int k = 0; k < G * KSX; ++k) {
        const float4 *p = gb + k * 16 + 2 * q;
        const float4 g0 = p[0], g1 = p[1], g2 = p[8], g3 = p[9];
#pragma unroll
        for (int t = 0; t < TW; ++t) {
            uint4 &v = xh[k / KSX][k % KSX][t];
            auto norm = [&](uint32_t u, const float4 &g) {
                return pack_bf16x2((bf16_lo(u) - mean[t]) * rstd[t] * g.x + g.y, (bf16_hi(u) - mean[t]) * rstd[t] * g.z + g.w);
            };
            v = make_uint4(norm(v.x, g0), norm(v.y, g1), norm(v.z, g2), norm(v.w, g3));
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

template <class Cf, int M, int TW>
__global__ __launch_bounds__(512, 2) void wide_fwd_kernel(Geom g, const bf16_t *__restrict__ x,
                                                          const uint8_t *__restrict__ pack,
                                                          const bf16_t *__restrict__ table,
                                                          bf16_t *__restrict__ y, bf16_t *__restrict__ attn,
                                                          const bf16_t *__restrict__ ln_w, const bf16_t *__restrict__ ln_b,
                                                          float ln_eps)
{
    using W = WideFwdCfg<Cf, M, TW>;
    constexpr int C = Cf::C, D = Cf::D, CG = Cf::CG, HG = Cf::HG, HEADS = Cf::HEADS, G = Cf::G;
    constexpr int KSX = Cf::KSX, TP = W::TP, OT_UNIT = W::OT_UNIT, NT = W::NT, NTB = W::NTB;
    constexpr int NTHREADS = W::NTHREADS, RPT = W::RPT, STEP = RPT * (2 * M - 1);
    constexpr int FPW = (W::FR_UNIT + W::NWAVES - 1) / W::NWAVES; // fragments a wave moves per unit
    static_assert(W::slots_free(), "no unit is overwritten while it is read");

    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];

    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, q = lane >> 4;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wslot = wv / W::WPW;          // window of the workgroup this wave works on
    const int t0 = (wv % W::WPW) * TW;      // its first tile in the window
    const int s = g.shift;
    const int cn = l16 % M, rsub = l16 / M;
    const int per_img = g.nwi * g.nwj;
    const uint32_t tbytes = (uint32_t)g.T * (2u * C);
    const buf_t xbuf = make_buf(x, tbytes), ybuf = make_buf(y, tbytes), abuf = make_buf(attn, attn ? tbytes : 0u);
    const uint32_t c8 = 8u * q;

    const bool late = W::LATE && wv >= W::NWAVES / 2;

    // ---- weight stream ----
    // (the lane index as a round's address arithmetic sees it: opaque, re-made every round, so that per-lane
    // addresses are computed where they are used instead of being kept, and spilled, across the kernel)
    int lane_r = lane, wv_r = wv;
    // second half of a head's k-slots: features 16+4q..16+4q+3, of which only those below D exist
    auto keep_hi = [&](uint4 &v) {
        if (16 + 4 * (lane_r >> 4) >= D) v.z = 0u;
        if (16 + 4 * (lane_r >> 4) + 2 >= D) v.w = 0u;
    };
    // Loads that write LDS directly: one instruction moves one fragment (64 lanes x 16 bytes land at
    // the wave-uniform LDS address + 16 * lane).  Wave w moves fragments w, w + 8, ... of the unit.
    const uint32_t lds_w = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)lds + (uint32_t)W::OFF_W;
    auto stream_unit = [&](int u) {
        const uint8_t *src = pack + (u < HEADS ? Cf::P_WQW + (size_t)u * W::UNIT_BYTES
                                               : Cf::P_WPW + (size_t)(u - HEADS) * W::UNIT_BYTES) +
                             16 * lane_r + 1024 * wv_r;
        const uint32_t dst = __builtin_amdgcn_readfirstlane(lds_w + (uint32_t)(W::unit_slot(u) * W::UNIT_BYTES) + 1024 * wv_r);
#pragma unroll
        for (int k = 0; k < FPW; ++k)
            if (k * W::NWAVES + wv_r < W::FR_UNIT) lds_dma16_at(src + k * W::NWAVES * 1024, dst + k * W::NWAVES * 1024);
    };

    // ---- the tokens of this wave: byte offsets (tile t, this lane's column) and their x as MFMA
    // operands (all groups, head-padded order: step ks of group gi, tile t) ----
    const int stride = W::WINS * (int)gridDim.x;
    const int rounds = (g.nW + stride - 1) / stride;
    uint32_t tok[TW], tokn[TW]; // of the window in hand, of the one whose rows are on their way
    bool lastrow = false, lastcol = false, lastrow_n = false, lastcol_n = false;
    uint4 xh[G][KSX][TW];
    auto window_tokens = [&](int win) {
        const int b = win / per_img;
        const int wr = win - b * per_img;
        const int wi = wr / g.nwj, wj = wr - wi * g.nwj;
        lastrow_n = s > 0 && wi == g.nwi - 1;
        lastcol_n = s > 0 && wj == g.nwj - 1;
        int sj = wj * M + cn + s;
        if (sj >= g.W) sj -= g.W;
#pragma unroll
        for (int t = 0; t < TW; ++t) {
            int si = wi * M + RPT * (t0 + t) + rsub + s;
            if (si >= g.H) si -= g.H;
            tokn[t] = (uint32_t)((((b * g.H + si) * g.W) + sj) * C) * 2u;
        }
    };
    auto load_x = [&](int gi, int ks) {
#pragma unroll
        for (int t = 0; t < TW; ++t) {
            const uint32_t off = tokn[t] + c8 + 2u * (gi * CG + ks * D);
            xh[gi][ks][t] = cat(bload64(xbuf, off, 0u), bload64(xbuf, off + 32u, 0u));
        }
    };
    int win = wslot * (int)gridDim.x + (int)blockIdx.x;
    bool active = win < g.nW;
    if (active) {
        window_tokens(win);
#pragma unroll
        for (int gi = 0; gi < G; ++gi)
#pragma unroll
            for (int ks = 0; ks < KSX; ++ks) load_x(gi, ks);
    }

    // set-up: linear biases, bias table (base-2 units; last entry first, so that a lane's four key rows are four
    // consecutive floats), LayerNorm's vectors, first unit
    stream_unit(0);
    {
        const float *pb = reinterpret_cast<const float *>(pack + Cf::P_BIAS); // b_qkv [3C], b_proj [C]
        float *bias = reinterpret_cast<float *>(lds + W::OFF_BIAS);
        for (int i = tid; i < W::N_BQKV; i += NTHREADS) {
            const int e = i & 31, t3 = (i >> 5) % 3, hd = i / 96;
            float v = e < D ? pb[(hd / HG) * 3 * CG + t3 * CG + (hd % HG) * D + e] : 0.f;
            if (t3 == 0) v *= kLog2e;
            if (t3 == 2 && e == D) v = 1.f;
            bias[i] = v;
        }
        for (int i = tid; i < 16 * Cf::OT; i += NTHREADS) bias[W::N_BQKV + i] = i < C ? pb[3 * C + i] : 0.f;
    }
    for (int i = tid; i < W::NTBL * HEADS; i += NTHREADS)
        reinterpret_cast<float *>(lds + W::OFF_TBL)[(i % HEADS) * TP + W::NTBL - 1 - i / HEADS] = to_f32(table[i]) * kLog2e;
    if (ln_w)
        for (int i = tid; i < HEADS * 32; i += NTHREADS) {
            const int e = i & 31, c = (i >> 5) * D + e;
            reinterpret_cast<float2 *>(lds + W::OFF_LN)[i] = e < D ? make_float2(to_f32(ln_w[c]), to_f32(ln_b[c])) : make_float2(0.f, 0.f);
        }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();

    // this lane's query column (rn = RPT (t0 + ni) + rsub, cn) against key rows 4q+j of key tile kt: key
    // (RPT kt + 4q/M, 4q%M + j); reversed table entry = tb0 + STEP (kt + TW-1 - ni) + j
    const int key_r0 = (4 * q) / M, key_c0 = (4 * q) % M;
    const int tb0 = W::NTBL - 1 - STEP * (TW - 1) -
                    ((RPT * t0 + rsub - key_r0 + M - 1) * (2 * M - 1) + (cn - key_c0 + M - 1));
    const f32x4 zero4 = f32x4{0.f, 0.f, 0.f, 0.f};

    // (a late wave's share of the unit its first step's time would have sent off)
    if (late) {
        if (W::unit_at(1) >= 0) stream_unit(W::unit_at(1));
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
    }
    for (int round = 0; round < rounds; ++round) {
        const bool more = round + 1 < rounds;
        const bool next = win + stride < g.nW;
        // head outputs, packed tile pairs [head][token tile]: operand of the cascade and of the projection
        uint4 Ob[HEADS][TW];
        uint2 Qb[2][TW]; // q of the head whose scores come next

        uint32_t lds0 = 0;
        asm volatile("" : "+v"(lds0)); // keeps the LDS reads of a round inside the round
        lane_r = lane;
        wv_r = wv;
        asm volatile("" : "+v"(lane_r), "+s"(wv_r));
        const float *bqkv = reinterpret_cast<const float *>(lds + lds0 + W::OFF_BIAS);
        const float *bproj = bqkv + W::N_BQKV;
        const float *tbl = reinterpret_cast<const float *>(lds + lds0 + W::OFF_TBL);
        uint4 *kv = reinterpret_cast<uint4 *>(lds + lds0 + W::OFF_KV + (size_t)wslot * W::KV_WIN);
        if (active) {
#pragma unroll
            for (int t = 0; t < TW; ++t) tok[t] = tokn[t];
            lastrow = lastrow_n;
            lastcol = lastcol_n;
#pragma unroll
            for (int gi = 0; gi < G; ++gi)
#pragma unroll
                for (int ks = 0; ks < KSX; ++ks)
#pragma unroll
                    for (int t = 0; t < TW; ++t) keep_hi(xh[gi][ks][t]);
            if (ln_w)
                layer_norm_operands<G, KSX, TW, C, D>(xh, reinterpret_cast<const float4 *>(lds + lds0 + W::OFF_LN), q, ln_eps);
        }

        // scores, softmax and PV of head hd (K and V of all tiles of the window from LDS)
        auto attention = [&](auto hd_) {
            constexpr int hd = decltype(hd_)::value, gi = hd / HG, hl = hd % HG;
            const uint4 *kvh = kv + (size_t)(hd % W::KVBUF) * (W::KV_BYTES / 16);
            const float *tb = tbl + hd * TP + tb0;
#pragma unroll
            for (int n0 = 0; n0 < TW; n0 += NTB) {
                // S^T tiles (base-2 units), accumulated onto the relative bias: rows = keys 16kt+4q+j, column = query
                f32x4 st[NTB][NT];
                constexpr int KC = NT == 4 ? 4 : 1; // key tiles whose operands are read together, one chunk ahead of the products
                uint4 kop[2][KC];
                auto fetch = [&](int c) {
#pragma unroll
                    for (int k = 0; k < KC; ++k) {
                        const int kt = c * KC + k;
                        kop[c & 1][k] = kvh[kt * 64 + lane];
#pragma unroll
                        for (int ni = 0; ni < NTB; ++ni)
#pragma unroll
                            for (int j = 0; j < 4; ++j) st[ni][kt][j] = tb[STEP * (kt + TW - 1 - (n0 + ni)) + j];
                    }
                };
                fetch(0);
#pragma unroll
                for (int c = 0; c < NT / KC; ++c) {
                    if (c + 1 < NT / KC) fetch(c + 1);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int k = 0; k < KC; ++k)
#pragma unroll
                        for (int ni = 0; ni < NTB; ++ni) {
                            const int kt = c * KC + k;
                            st[ni][kt] = mma32(kop[c & 1][k], cat(Qb[0][n0 + ni], Qb[1][n0 + ni]), st[ni][kt]);
                        }
                }
                constexpr int VC = NT == 4 ? 2 : 1; // (V the same way, in pairs of tiles; with few tiles the first under the softmax)
                uint4 vop[2][2 * VC];
                auto fetch_v = [&](int c) {
#pragma unroll
                    for (int k = 0; k < 2 * VC; ++k) vop[c & 1][k] = kvh[(NT + 2 * VC * c + k) * 64 + lane];
                };
                if (NT == 4) fetch_v(0);
                if (lastrow || lastcol) {
                    int s_ = s; // (opaque: the conditions are made here, not kept over the head)
                    asm volatile("" : "+s"(s_));
                    float cm[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) cm[j] = (lastcol && (cn >= M - s_) != (key_c0 + j >= M - s_)) ? kMaskLog2 : 0.f;
#pragma unroll
                    for (int ni = 0; ni < NTB; ++ni) {
                        const bool qr_w = RPT * (t0 + n0 + ni) + rsub >= M - s_;
#pragma unroll
                        for (int kt = 0; kt < NT; ++kt) {
                            const bool rm = lastrow && qr_w != (RPT * kt + key_r0 >= M - s_);
#pragma unroll
                            for (int j = 0; j < 4; ++j) st[ni][kt][j] += rm ? kMaskLog2 : cm[j];
                        }
                    }
                }
                float mx[NTB];
#pragma unroll
                for (int ni = 0; ni < NTB; ++ni) {
                    float m0 = max4f(st[ni][0]);
#pragma unroll
                    for (int kt = 1; kt < NT; ++kt) m0 = max5f(m0, st[ni][kt]);
                    mx[ni] = m0;
                }
#pragma unroll
                for (int ni = 0; ni < NTB; ++ni) mx[ni] = qgroup_max(mx[ni]);
                uint2 Pb[NTB][NT];
#pragma unroll
                for (int ni = 0; ni < NTB; ++ni)
#pragma unroll
                    for (int kt = 0; kt < NT; ++kt) {
#pragma unroll
                        for (int j = 0; j < 4; ++j) st[ni][kt][j] = __builtin_amdgcn_exp2f(st[ni][kt][j] - mx[ni]);
                        Pb[ni][kt] = pack_bf16x4(st[ni][kt]);
                    }
                // O^T = V^T P^T: rows = head features (row D = sum of the probabilities)
                f32x4 o0[NTB], o1[NTB];
#pragma unroll
                for (int ni = 0; ni < NTB; ++ni) o0[ni] = o1[ni] = zero4;
#pragma unroll
                for (int c = 0; c < NT / (2 * VC); ++c) {
                    if (NT > 4 && c == 0) fetch_v(0);
                    if (c + 1 < NT / (2 * VC)) fetch_v(c + 1);
                    if (NT > 4) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int k = 0; k < VC; ++k)
#pragma unroll
                        for (int ni = 0; ni < NTB; ++ni) {
                            const int kt = 2 * (VC * c + k);
                            const uint4 p = cat(Pb[ni][kt], Pb[ni][kt + 1]);
                            o0[ni] = mma32(vop[c & 1][2 * k], p, o0[ni]);
                            o1[ni] = mma32(vop[c & 1][2 * k + 1], p, o1[ni]);
                        }
                }
#pragma unroll
                for (int ni = 0; ni < NTB; ++ni) {
                    const float inv = __builtin_amdgcn_rcpf(qgroup_bcast<(D - 16) / 4>(o1[ni][(D - 16) % 4]));
                    o0[ni] *= inv;
                    o1[ni] *= inv;
                    Ob[hd][n0 + ni] = cat(pack_bf16x4(o0[ni]), pack_bf16x4(o1[ni]));
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            // the outputs of a group leave together when the caller keeps them for the backward
            // pass (pieces of a row then fill whole cache lines)
            if (attn && hl == HG - 1) {
#pragma unroll
                for (int nt = 0; nt < TW; ++nt)
#pragma unroll
                    for (int h2 = gi * HG; h2 <= hd; ++h2) {
                        // lane group q: features 8q .. 8q+7 of the head (16 contiguous bytes)
                        const uint32_t off = tok[nt] + 16u * q + 2u * (h2 * D);
                        const uint4 o = pair_rows(make_uint2(Ob[h2][nt].x, Ob[h2][nt].y),
                                                  make_uint2(Ob[h2][nt].z, Ob[h2][nt].w));
                        if (8 * q + 8 <= D) {
                            bstore128(abuf, off, 0u, o);
                        } else {
                            if (8 * q + 4 <= D) bstore64(abuf, off, 0u, make_uint2(o.x, o.y));
                            if (8 * q + 6 <= D) bstore32(abuf, off + 8u, 0u, o.z);
                        }
                    }
            }
        };

        static_for<W::NS>([&](auto i_) {
            constexpr int i = decltype(i_)::value, time = W::time_of(i);
            constexpr bool first = i == 0 || W::time_of(i - 1) != time, last = i == W::NS - 1 || W::time_of(i + 1) != time;
            // the unit that the next time reads first, on its way into a buffer that every wave has finished reading
            // (late waves are one time further on)
            constexpr int ue = W::unit_at((time + 1) % W::NTIME), ul = W::unit_at((time + 1 + W::LATE) % W::NTIME);
            constexpr bool we = time + 1 >= W::NTIME, wl = time + 1 + W::LATE >= W::NTIME; // (of the next round)
            if constexpr (first) {
                if (!late) {
                    if (ue >= 0 && (!we || more)) stream_unit(ue);
                } else {
                    if (ul >= 0 && (!wl || more)) stream_unit(ul);
                }
            }
            if (next) {
                static_for<G>([&](auto g_) {
                    constexpr int gi = decltype(g_)::value, k0 = W::load_at(i, gi);
                    if constexpr (k0 >= 0) {
                        if constexpr (gi == 0 && k0 == 0) window_tokens(win + stride);
#pragma unroll
                        for (int ks = k0; ks < k0 + W::KPM; ++ks) load_x(gi, ks);
                    }
                });
            }
            const uint4 *wu;
            if constexpr (i < 2 * HEADS) {
                constexpr int hd = i / 2, gi = hd / HG, hl = hd % HG;
                if constexpr (i % 2) {
                    if (active) attention(std::integral_constant<int, hd>{});
                } else if (active) {
                    wu = reinterpret_cast<const uint4 *>(lds + lds0 + W::OFF_W + (size_t)W::unit_slot(hd) * W::UNIT_BYTES);
                    if (G > 1 && hl == 0 && gi > 0 && g.cascade) { // Eq. 8
#pragma unroll
                        for (int ks = 0; ks < KSX; ++ks)
#pragma unroll
                            for (int t = 0; t < TW; ++t) {
                                uint4 p = Ob[(gi > 0 ? gi - 1 : 0) * HG + ks][t];
                                keep_hi(p);
                                uint4 &xv = xh[gi][ks][t];
                                xv.x = add_bf16x2(xv.x, p.x);
                                xv.y = add_bf16x2(xv.y, p.y);
                                xv.z = add_bf16x2(xv.z, p.z);
                                xv.w = add_bf16x2(xv.w, p.w);
                            }
                    }
                    // ---- Q^T, K^T (rows = head features) and V (rows = tokens) ----
                    uint4 *kvw = kv + (size_t)(hd % W::KVBUF) * (W::KV_BYTES / 16);
                    // (fragments and bias of the next kind are read under the products of the one in hand: left alone the
                    // compiler keeps two reads in flight and waits for each pair)
                    constexpr int KH = KSX > 3 ? KSX / 2 : KSX, NC = KSX / KH; // K steps of a chunk, chunks of a kind
                    uint4 fr[2][2 * KH];
                    f32x4 acc[2][TW];
                    f32x4 b4[2];
                    auto fetch = [&](int c) {
                        const int t3 = c / NC, k0 = c % NC * KH;
                        if (k0 == 0) {
                            const float *bh = bqkv + (hd * 3 + t3) * 32;
#pragma unroll
                            for (int et = 0; et < 2; ++et) {
                                if (t3 < 2) {
                                    b4[et] = *reinterpret_cast<const f32x4 *>(bh + 16 * et + 4 * q);
                                } else { // (column D of V is one: row D of the PV product is the sum of the probabilities)
                                    const float bv = bh[16 * et + l16];
                                    b4[et] = f32x4{bv, bv, bv, bv};
                                }
                            }
                        }
#pragma unroll
                        for (int ks = 0; ks < KH; ++ks)
#pragma unroll
                            for (int et = 0; et < 2; ++et) fr[c & 1][2 * ks + et] = wu[((t3 * 2 + et) * KSX + k0 + ks) * 64 + lane];
                    };
                    fetch(0);
#pragma unroll
                    for (int c = 0; c < 3 * NC; ++c) {
                        const int t3 = c / NC, k0 = c % NC * KH;
                        if (k0 == 0) {
#pragma unroll
                            for (int et = 0; et < 2; ++et)
#pragma unroll
                                for (int t = 0; t < TW; ++t) acc[et][t] = b4[et];
                        }
                        if (c + 1 < 3 * NC) fetch(c + 1);
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int ks = 0; ks < KH; ++ks)
#pragma unroll
                            for (int et = 0; et < 2; ++et) {
                                const uint4 f = fr[c & 1][2 * ks + et];
#pragma unroll
                                for (int t = 0; t < TW; ++t) {
                                    const uint4 xv = xh[gi][k0 + ks][t];
                                    acc[et][t] = t3 < 2 ? mma32(f, xv, acc[et][t]) : mma32(xv, f, acc[et][t]);
                                }
                            }
                        if (k0 + KH < KSX) continue;
                        // q stays with the wave; k and v go to LDS as the operands the scores and PV read:
                        // k tile by tile, v by pairs of tiles and per half of the features
#pragma unroll
                        for (int t = 0; t < TW; ++t) {
                            const uint2 p0 = pack_bf16x4(acc[0][t]), p1 = pack_bf16x4(acc[1][t]);
                            if (t3 == 0) {
                                Qb[0][t] = p0;
                                Qb[1][t] = p1;
                            } else if (t3 == 1) {
                                kvw[(t0 + t) * 64 + lane] = cat(p0, p1);
                            } else {
                                uint2 *vw = reinterpret_cast<uint2 *>(kvw + (NT + ((t0 + t) & ~1)) * 64 + lane) + ((t0 + t) & 1);
                                vw[0] = p0;
                                vw[128] = p1;
                            }
                        }
                    }
                }
            } else {
                constexpr int pu = i - 2 * HEADS;
                wu = reinterpret_cast<const uint4 *>(lds + lds0 + W::OFF_W + (size_t)W::unit_slot(HEADS + pu) * W::UNIT_BYTES);
                // ---- Y^T = Wproj A^T + b for OT_UNIT output tiles: rows = output channels, column = token ----
                if (active) {
                    // two output tiles at a time: their packed results are regrouped so that a lane holds 16
                    // contiguous bytes of its token's row (a tile left over at the end goes out in 8-byte pieces)
                    uint4 wf[2][HEADS]; // (fragments of the next tile are read under the products of the one in hand)
                    auto fetch = [&](int oi) {
#pragma unroll
                        for (int hd = 0; hd < HEADS; ++hd) wf[oi & 1][hd] = wu[(oi * HEADS + hd) * 64 + lane];
                    };
                    auto project = [&](int oi, f32x4(&acc)[TW]) {
                        const f32x4 b4 = *reinterpret_cast<const f32x4 *>(bproj + 16 * (pu * OT_UNIT + oi) + 4 * q);
                        if (oi + 1 < OT_UNIT) fetch(oi + 1);
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int t = 0; t < TW; ++t) acc[t] = b4;
#pragma unroll
                        for (int hd = 0; hd < HEADS; ++hd)
#pragma unroll
                            for (int t = 0; t < TW; ++t) acc[t] = mma32(wf[oi & 1][hd], Ob[hd][t], acc[t]);
                    };
                    fetch(0);
#pragma unroll
                    for (int oi = 0; oi + 1 < OT_UNIT; oi += 2) {
                        const int ot = pu * OT_UNIT + oi;
                        f32x4 acc0[TW], acc1[TW];
                        project(oi, acc0);
                        project(oi + 1, acc1);
                        const int o0 = 16 * ot + 8 * q; // first channel of this lane's eight
#pragma unroll
                        for (int t = 0; t < TW; ++t) {
                            const uint4 v = pair_rows(pack_bf16x4(acc0[t]), pack_bf16x4(acc1[t]));
                            const uint32_t off = tok[t] + 2u * o0;
                            if (o0 + 8 <= C) bstore128(ybuf, off, 0u, v);
                            else if (o0 + 4 <= C) bstore64(ybuf, off, 0u, make_uint2(v.x, v.y));
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (OT_UNIT % 2 == 1) {
                        const int ot = pu * OT_UNIT + OT_UNIT - 1;
                        f32x4 acc[TW];
                        project(OT_UNIT - 1, acc);
                        const int o0 = 16 * ot + 4 * q;
#pragma unroll
                        for (int t = 0; t < TW; ++t)
                            if (o0 < C) bstore64(ybuf, tok[t] + c8 + 32u * ot, 0u, pack_bf16x4(acc[t]));
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
            // Before the barrier: the wave's share of the next unit has landed in LDS, its k and v are written and read.
            // Vector-memory operations complete in the order they were issued: "at most n outstanding" covers the
            // stream loads when at least n were issued behind them.
            if constexpr (last) {
                constexpr int p = first ? i : i - 1; // the other step of this time
                constexpr int NY = W::stores_in(i) + (first ? 0 : W::stores_in(p)), NX = W::loads_in(i) + (first ? 0 : W::loads_in(p)),
                              NA = W::keeps_in(i) + (first ? 0 : W::keeps_in(p));
                __builtin_amdgcn_sched_barrier(0);
                if ((late ? ul : ue) < 0) wait_vm<63>();
                else if (!active) wait_vm<0>();
                else if (NA && attn) { if (next) wait_vm<NX + NY + NA>(); else wait_vm<NY + NA>(); }
                else if (NX && next) wait_vm<NX + NY>();
                else wait_vm<NY>();
                __syncthreads();
            }
        });
        win += stride;
        active = next;
    }
    if (W::LATE && !late) __syncthreads(); // (as many barriers for every wave)
}

#define GSWA_WIDE_SHAPES(X) X(180, 6, 1) X(180, 6, 2) X(180, 6, 3)

template <class Cf, int M, int TW>
hipError_t run_wide_fwd(const Geom &g, const bf16_t *x, const uint8_t *pack, const bf16_t *table, bf16_t *y, bf16_t *attn,
                        const FusedLn &ln, hipStream_t s)
{
    using W = WideFwdCfg<Cf, M, TW>;
    auto kern = wide_fwd_kernel<Cf, M, TW>;
    if (hipError_t ea = allow_dynamic_lds(reinterpret_cast<const void *>(kern), W::LDS_BYTES); ea != hipSuccess) return ea;
    // spread the windows over the compute units before filling a workgroup
    int grid = device_cu_count();
    if (grid > g.nW) grid = g.nW;
    KernelTimer kt(K_FUSED_FWD, s);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(W::NTHREADS), W::LDS_BYTES, s, g, x, pack, table, y, attn, ln.w, ln.b, ln.eps);
    return hipGetLastError();
}

} // namespace

bool wide_fwd_supported(const Geom &g)
{
    if ((g.M != 8 && g.M != 16) || g.dq != g.d || (long)g.T * g.C >= (1L << 31)) return false;
#define X(C_, H_, G_) \
    if (g.C == C_ && g.heads == H_ && g.groups == G_) return true;
    GSWA_WIDE_SHAPES(X)
#undef X
    return false;
}

hipError_t launch_wide_fwd(const Geom &g, const bf16_t *x, const void *pack, const bf16_t *table, bf16_t *y, bf16_t *attn,
                           int training, const FusedLn &ln, hipStream_t s)
{
    if (training && !attn) return hipErrorInvalidValue;
    // (8x8 windows, up to two a compute unit: four waves a window, which shortens the chain of steps: one window 19.6 -> 17.1
    // us, 99 windows 19.6 -> 17.0, 512 windows 22.7 -> 22.1; more windows are better off with each fragment read from LDS
    // serving two tiles.  The same bits.)
    const uint8_t *p = static_cast<const uint8_t *>(pack);
    bf16_t *at = training ? attn : nullptr;
#define X(C_, H_, G_)                                                                             \
    if (g.C == C_ && g.heads == H_ && g.groups == G_) {                                           \
        using Cf = FusedCfg<C_, H_, G_>;                                                          \
        if (g.M == 16) return run_wide_fwd<Cf, 16, 2>(g, x, p, table, y, at, ln, s);              \
        return g.nW <= 2 * device_cu_count() ? run_wide_fwd<Cf, 8, 1>(g, x, p, table, y, at, ln, s)  \
                                             : run_wide_fwd<Cf, 8, 2>(g, x, p, table, y, at, ln, s); \
    }
    GSWA_WIDE_SHAPES(X)
#undef X
    return hipErrorInvalidValue;
}

} // namespace gswa
