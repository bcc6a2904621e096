// Kernels of window_layer.h, included by the files that instantiate them.
//
// What bounds the layers this file serves (60 channels, 8x8 windows in fp32 or 12x12 in bf16, any number of windows) is
// not bandwidth and, with few windows, hardly arithmetic but the chain of launches: one kernel per step of Eq. 4-8 and
// head group is 40 launches of 5-70 us per training step, each a trip of every activation through memory.  (Figures
// against those kernels, from 1 to 16384 windows: window_layer.hip.)  Here a layer is one launch per
// direction (plus the sum of the parameter gradients): the window's rows, its q|k|v, its hidden layer and all their
// gradients stay in the 160 KB of LDS, and the weights are read as matrix-core operands straight from L2 (every
// workgroup reads the same few tens of KB).
//
// All products run on the matrix cores, in fp32 as 16x16x4 products (exact products, fp32 accumulation: nothing is
// rounded that the vector ALUs would keep).  With l16 = lane & 15 and q = lane >> 4, an operand of 16 k-slots is four
// values of one row l16, slots 4q .. 4q+3; a result tile holds column l16, rows 4q .. 4q+3.  A result tile is
// therefore the right-hand operand of a product that reduces over its rows (mfma.h has the same rule for bf16), and
// the two orientations of every product cost the same:
//   [features x tokens] results are stored as four consecutive features of a token (rows of LDS are token-major);
//   products that reduce over features read four consecutive features of a token (ld_n),
//   products that reduce over tokens read one feature of four consecutive tokens (ld_t).
// Rows q|k|v hold every head at a stride rounded up to four features (zeros in between, because the weight rows
// that belong there are taken as zero), rows of C channels end in pad columns; the first pad column of the operands
// of weight-gradient products is one, so a bias gradient is one more column of its weight gradient.
#pragma once
#include "window_layer.h"
#include "fused.h"
#include "mfma.h"
#include "staged_kernels.h"

namespace gswa {

namespace {

constexpr float kLog2e = 1.4426950408889634f;
// Scores: in bf16 base 2, with the factor and the scale in q and in the bias table.  In fp32 the roundings of these would
// show, and so would the order of the sums: there a score is taken times the scale and with its bias at the end, the
// exponentials are summed on the vector ALU, and the backward keeps maximum and denominator apart.  Against all of these
// the bf16 way, error against fp64 over the one-kernel-per-step path's (attention layer, two groups, 16 layers): y 1.13 ->
// 1.00, dx 1.12 -> 1.01, dtable 1.15 -> 0.99; a whole layer takes 86 us either way (three 48x56 patches).
template <typename E> constexpr float score_unit = sizeof(E) == 2 ? kLog2e : 1.f; // (of bias and mask)
template <typename E> __device__ __forceinline__ float prob(float d) { return __builtin_amdgcn_exp2f(sizeof(E) == 2 ? d : d * kLog2e); }

// The lane's place in an operand, made afresh where it is used: otherwise the compiler computes the lane's addresses
// of every phase at the start of the kernel, runs out of registers and spills them.
#define FRESH_LANE                            \
    int fresh_ = (int)threadIdx.x;            \
    asm volatile("" : "+v"(fresh_));          \
    [[maybe_unused]] const int l16 = fresh_ & 15, q = (fresh_ >> 4) & 3

// Row pitch (elements): a multiple of four that is not a multiple of eight, so that 16 rows read at the same column
// fall on different banks.
constexpr int pitch_of(int n) { return (n + 3) / 8 * 8 + 4; }
constexpr int up(int a, int b) { return (a + b - 1) / b; }
constexpr int imax(int a, int b) { return a > b ? a : b; }

template <typename T_, int C_, int HEADS_, int G_, int M_, int DQ_, int HID_, int WAVES_> struct WinShape {
    using T = T_;
    using E = T_;
    static constexpr int C = C_, HEADS = HEADS_, G = G_, M = M_, DQ = DQ_, HID = HID_, WAVES = WAVES_;
    static constexpr int NTH = 64 * WAVES;
    static constexpr int N = M * M, NT = N / 16, CG = C / G, HG = HEADS / G, D = C / HEADS, QG = HG * DQ, RG = 2 * QG + CG;
    static constexpr int HSQ = (DQ + 3) & ~3, HSV = (D + 3) & ~3;  // stride of a head in the q, k and in the v rows
    static constexpr int RQ = HG * HSQ, RV = HG * HSV, RP = 2 * RQ + RV;
    static constexpr int NFT = up(RP, 16), KUG = up(CG, 16), KUC = up(C, 16), KUR = up(RP, 16), CTC = up(C, 16), CTG = up(CG, 16);
    static constexpr int HFT = up(HID, 16), NVT = up(RV, 16);
    // token tiles that share one reading of the weights: the loads of weights, 16 short pieces of rows each, are
    // what the vector memory pipe of a compute unit spends its time on otherwise
    static constexpr int TT = NT % 3 == 0 ? 3 : 2, TU = NT / TT;
    static constexpr int TP = NT % 3 == 0 ? 3 : 1, PU = NT / TP; // (products with C outputs: as many units as wavefronts)
    // Rows of C channels that group slices are read from keep every group at a stride of a multiple of four channels
    // (CGP), so that slices are aligned; OC is their first pad column.
    static constexpr int CGP = (CG + 3) & ~3, XW = G * CGP, OC = CG < CGP ? CG : XW;
    static constexpr int KUX = up(XW, 16), CTX = up(OC < XW ? XW : XW + 1, 16);
    static __device__ __forceinline__ int xcol(int c) { return CGP == CG ? c : c / CG * CGP + c % CG; }
    // (a slice's last k-slots and column tiles may run into the next row: numbers that meet zero weights or are dropped)
    static constexpr int PC = pitch_of(imax(16 * up(C + 1, 16), XW)), PR = pitch_of(sizeof(E) == 2 ? RP + 12 : RP), PD = pitch_of(RV), PH = pitch_of(16 * up(HID + 1, 16));
    // (behind q|k|v a row holds its token's part of the shift mask: as a key; as a query, the rounded factor and the rest)
    static constexpr int MK = RP, MQ = RP + 4;
    static constexpr int PF = N + 4; // pitch of a head's matrix of score gradients
    static constexpr int NTB = 2 * M - 1, NTBL = NTB * NTB, TBP = (NTBL + 3) & ~3;
    static_assert(M * M % 16 == 0 && C % 4 == 0 && D <= 16 && DQ <= 16 && C % 16 != 0 && CG % 16 != 0 && HID % 16 != 0, "shape");
    // a workgroup's vector of parameter gradients
    static constexpr int P_WQ = 0, P_BQ = P_WQ + G * RG * CG, P_WP = P_BQ + G * RG, P_BP = P_WP + C * C, P_TB = P_BP + C;
    static constexpr int P_ATTN = P_TB + NTBL * HEADS;
    static constexpr int P_W1 = P_ATTN, P_B1 = P_W1 + HID * C, P_W2 = P_B1 + HID, P_B2 = P_W2 + C * HID, P_G1 = P_B2 + C;
    static constexpr int P_E1 = P_G1 + C, P_G2 = P_E1 + C, P_E2 = P_G2 + C, P_ALL = P_E2 + C;
    static constexpr int stride(bool layer) { return ((layer ? P_ALL : P_ATTN) + 3) & ~3; }
    // LDS (bytes).  Forward: X | A | R (q|k|v of a group, or the hidden layer) | tables
    static constexpr size_t SZ_ROW = sizeof(E) * N * PC, SZ_R = sizeof(E) * N * PR, SZ_H = sizeof(E) * N * PH;
    static constexpr size_t SZ_TB = sizeof(float) * HEADS * TBP;
    static constexpr size_t F_X = 0, F_A = SZ_ROW, F_R = 2 * SZ_ROW;
    static constexpr size_t fwd_tb(bool layer) { return F_R + (layer && SZ_H > SZ_R ? SZ_H : SZ_R); }
    static constexpr size_t fwd_lds(bool layer) { return fwd_tb(layer) + SZ_TB; }
    // Backward: X | A | DX | R | dO of a group | score gradients of NF heads | tables | statistics (and row sums).  The
    // heads of a group are taken NF at a time; where a group is the whole layer and has more, the score gradients lie
    // over DX, whose last use (but for the skip, which goes by memory) is over by then.  The MLP's hidden layer and its
    // gradient lie over what follows DX.
    static constexpr size_t SZ_DO = sizeof(E) * N * PD, SZ_F = sizeof(E) * N * PF;
    static constexpr size_t SZ_ST = sizeof(float) * (sizeof(E) == 4 ? 3 : 2) * HG * N, SZ_RED = sizeof(float) * WAVES * 2 * 16 * up(C, 16);
    static constexpr size_t SZ_SR = SZ_ST > SZ_RED ? SZ_ST : SZ_RED; // (row sums and softmax statistics take turns)
    static constexpr size_t FIXED = 2 * SZ_ROW + SZ_R + SZ_DO + SZ_TB + SZ_SR;
    static constexpr bool fits(int n, bool over) { return FIXED + (over ? (n * SZ_F > SZ_ROW ? n * SZ_F : SZ_ROW) : SZ_ROW + n * SZ_F) <= 160 * 1024; }
    static constexpr bool OVER = G == 1 && !fits(HG, false);
    static constexpr int fit_heads()
    {
        int n = HG;
        while (n > 1 && !fits(n, OVER)) --n;
        return n;
    }
    static constexpr int NF = fit_heads(), ROUNDS = up(HG, NF);
    static constexpr size_t SZ_DX = OVER && NF * SZ_F > SZ_ROW ? NF * SZ_F : SZ_ROW;
    static constexpr size_t B_DX = 2 * SZ_ROW, B_R = B_DX + SZ_DX, B_DO = B_R + SZ_R, B_FO = OVER ? B_DX : B_DO + SZ_DO;
    static constexpr size_t B_H = 3 * SZ_ROW, B_END = B_DO + SZ_DO + (OVER ? 0 : NF * SZ_F);
    // Where there is room: sums of a head's score gradients over pairs of window rows at the same distance (see fold_blocks)
    static constexpr size_t SZ_S = sizeof(float) * NTB * N;
    static constexpr size_t tb_at(bool layer, bool blocks)
    {
        const size_t end = B_END + (blocks ? NF * SZ_S : 0);
        return layer && B_H + 2 * SZ_H > end ? B_H + 2 * SZ_H : end;
    }
    static constexpr bool BLOCKS = sizeof(E) == 2 && tb_at(false, true) + SZ_TB + SZ_SR <= 160 * 1024 && tb_at(true, true) + SZ_TB + SZ_SR <= 160 * 1024;
    static constexpr size_t bwd_tb(bool layer) { return tb_at(layer, BLOCKS); }
    static constexpr size_t bwd_lds(bool layer) { return bwd_tb(layer) + SZ_TB + SZ_SR; }
    static_assert(fwd_lds(true) <= 160 * 1024 && bwd_lds(true) <= 160 * 1024, "LDS budget");
};

__device__ __forceinline__ f32x4 zero4() { return f32x4{0.f, 0.f, 0.f, 0.f}; }

// ---- operands of 16 k-slots --------------------------------------------------------------------------------
// fp32: four 16x16x4 products; slot 4q + i of an operand is k-slot q of product i
__device__ __forceinline__ f32x4 mma(f32x4 a, f32x4 b, f32x4 c)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[i], c, 0, 0, 0);
    return c;
}
__device__ __forceinline__ f32x4 mma(uint2 a, uint2 b, f32x4 c) { return mma16(a, b, c); }
template <typename E> struct Op;
template <> struct Op<float> {
    using F = f32x4;
    static __device__ __forceinline__ F ones() { return f32x4{1.f, 1.f, 1.f, 1.f}; }
    static __device__ __forceinline__ F ld(const float *p) { return *reinterpret_cast<const f32x4 *>(p); }
    // element (row 4q + i, column l16), i < 4: `p` points at row 0, column 0; ld_tr: row 15 - 4q - i
    static __device__ __forceinline__ F ld_t(const float *p, int pitch, int q, int l16)
    {
        const float *r = p + 4 * q * pitch + l16;
        return f32x4{r[0], r[pitch], r[2 * pitch], r[3 * pitch]};
    }
    static __device__ __forceinline__ F ld_tr(const float *p, int pitch, int q, int l16)
    {
        const float *r = p + (12 - 4 * q) * pitch + l16;
        return f32x4{r[3 * pitch], r[2 * pitch], r[pitch], r[0]};
    }
    static __device__ __forceinline__ F gather(float a, float b, float c, float d) { return f32x4{a, b, c, d}; }
    static __device__ __forceinline__ F from(f32x4 v) { return v; }
    static __device__ __forceinline__ f32x4 wide(F v) { return v; }
    static __device__ __forceinline__ F add(F a, F b) { return a + b; }
    static __device__ __forceinline__ void st(float *p, f32x4 v) { *reinterpret_cast<f32x4 *>(p) = v; }
    static __device__ __forceinline__ F pick(bool ok, F v)
    {
        return f32x4{ok ? v[0] : 0.f, ok ? v[1] : 0.f, ok ? v[2] : 0.f, ok ? v[3] : 0.f};
    }
    static __device__ __forceinline__ float get(const float *p) { return *p; }
    static __device__ __forceinline__ void put(float *p, float v) { *p = v; }
    static __device__ __forceinline__ void gelu(float t, float &h, float &dh)
    {
        const float Phi = gauss_cdf(t);
        h = t * Phi;
        dh = fmaf(t, 0.39894228040143268f * __builtin_amdgcn_exp2f(t * t * -0.72134752044448170f), Phi);
    }
};
template <> struct Op<bf16_t> {
    using F = uint2;
    static __device__ __forceinline__ F ones() { return make_uint2(0x3f803f80u, 0x3f803f80u); }
    static __device__ __forceinline__ F ld(const bf16_t *p) { return *reinterpret_cast<const uint2 *>(p); }
    // The four rows 4q .. 4q+3 of 16 columns are 128 bytes for the 16 lanes of a q; each lane names eight of them (row
    // 4q + l16 / 4, columns 4 (l16 % 4) ..) and the read hands out columns.
    static __device__ __forceinline__ F ld_t(const bf16_t *p, int pitch, int q, int l16)
    {
        const bf16_t *r = p + (4 * q + (l16 >> 2)) * pitch + 4 * (l16 & 3);
        const s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(r));
        return __builtin_bit_cast(uint2, v);
    }
    static __device__ __forceinline__ F ld_tr(const bf16_t *p, int pitch, int q, int l16)
    {
        const bf16_t *r = p + (15 - 4 * q - (l16 >> 2)) * pitch + 4 * (l16 & 3);
        const s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(r));
        return __builtin_bit_cast(uint2, v);
    }
    static __device__ __forceinline__ F gather(float a, float b, float c, float d) { return make_uint2(pack_bf16x2(a, b), pack_bf16x2(c, d)); }
    static __device__ __forceinline__ F from(f32x4 v) { return pack_bf16x4(v); }
    static __device__ __forceinline__ f32x4 wide(F v) { return f32x4{bf16_lo(v.x), bf16_hi(v.x), bf16_lo(v.y), bf16_hi(v.y)}; }
    static __device__ __forceinline__ F add(F a, F b) { return make_uint2(add_bf16x2(a.x, b.x), add_bf16x2(a.y, b.y)); }
    static __device__ __forceinline__ void st(bf16_t *p, f32x4 v) { *reinterpret_cast<uint2 *>(p) = pack_bf16x4(v); }
    static __device__ __forceinline__ F pick(bool ok, F v) { return make_uint2(ok ? v.x : 0u, ok ? v.y : 0u); }
    static __device__ __forceinline__ float get(const bf16_t *p) { return to_f32(*p); }
    static __device__ __forceinline__ void put(bf16_t *p, float v) { p->bits = (uint16_t)pack_bf16x2(v, 0.f); }
    static __device__ __forceinline__ void gelu(float t, float &h, float &dh)
    {
        float Phi, phi;
        gauss(t, Phi, phi);
        h = t * Phi;
        dh = Phi + t * phi;
    }
};

// One head's slice of a row as an operand: HS channels (a multiple of four, at most 16).
//
// Q and K operands (HS <= 8) carry the shift mask with them.  With r, c = "past the wrap in the last window row, column"
// of a token, [regions of n and m differ] = (r_n|c_n) + (1-2 r_n)(1-c_n) r_m + (1-2 c_n)(1-r_n) c_m
// - (1-2 r_n)(1-2 c_n) r_m c_m: four more k-slots, (1, r, c, rc) of the key against those coefficients of the query
// times -100 log2(e).  In bf16 they take the slots 12 .. 15 that no head uses, with the factor rounded to bf16 (144), and
// the slots 8 .. 11 with what the rounding left (0.2695): together -100.00002, at no cost.  In fp32, where adding and
// taking away 144 would cost the scores their last bits, masked windows add the mask on the vector ALU.
template <typename E, int HS> struct HeadOp;
// `at`: where in the head's slice a lane's part begins, `load` reads it from there
template <int HS> struct HeadOp<float, HS> { // product i takes channels 4i .. 4i+3: HS / 4 products instead of four
    float v[HS / 4];
    static __device__ __forceinline__ int at(int q) { return q; }
    __device__ __forceinline__ void load(const float *p)
    {
#pragma unroll
        for (int i = 0; i < HS / 4; ++i) v[i] = p[4 * i];
    }
    __device__ __forceinline__ void mask(int) {}
};
template <int HS> __device__ __forceinline__ f32x4 mma(const HeadOp<float, HS> &a, const HeadOp<float, HS> &b, f32x4 c)
{
#pragma unroll
    for (int i = 0; i < HS / 4; ++i) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v[i], b.v[i], c, 0, 0, 0);
    return c;
}
template <int HS> struct HeadOp<bf16_t, HS> { // (slots beyond the head: any number on one side, zeros on the masked one)
    uint2 v;
    static __device__ __forceinline__ int at(int q) { return 4 * q < HS ? 4 * q : 0; }
    __device__ __forceinline__ void load(const bf16_t *p) { v = *reinterpret_cast<const uint2 *>(p); }
    __device__ __forceinline__ void mask(int q) { v = make_uint2(4 * q < HS ? v.x : 0u, 4 * q < HS ? v.y : 0u); }
};
template <int HS> __device__ __forceinline__ f32x4 mma(const HeadOp<bf16_t, HS> &a, const HeadOp<bf16_t, HS> &b, f32x4 c) { return mma16(a.v, b.v, c); }
// q (`query`) or k of a head: `at` is where in a token's row the lane's part of the head at column `col` lies
template <class S> struct QkOp : HeadOp<typename S::E, S::HSQ> {
    static constexpr bool SLOTS = sizeof(typename S::E) == 2;
    static_assert(!SLOTS || S::HSQ <= 8, "slots 8 .. 15 are the mask's");
    static __device__ __forceinline__ int at(int col, bool query, int q)
    {
        if constexpr (SLOTS) return q < 2 ? col + (4 * q < S::HSQ ? 4 * q : 0) : query ? S::MQ + 4 * (3 - q) : S::MK;
        return col + HeadOp<typename S::E, S::HSQ>::at(q);
    }
    __device__ __forceinline__ void mask(int q)
    {
        if constexpr (SLOTS) { // (which of the four slot groups count, as bits)
            const uint32_t m = 0u - (((12u | ((1u << S::HSQ / 4) - 1u)) >> q) & 1u);
            this->v = make_uint2(this->v.x & m, this->v.y & m);
        }
    }
};
// a tile of scores, from the four bias entries of the lane on: in bf16 they start the sum
template <class S> __device__ __forceinline__ f32x4 scores(const QkOp<S> &a, const QkOp<S> &b, f32x4 t)
{
    if constexpr (sizeof(typename S::E) == 2) return mma(a, b, t);
    f32x4 d = mma(a, b, zero4());
#pragma unroll
    for (int i = 0; i < 4; ++i) d[i] = fmaf(d[i], 1.f / sqrtf((float)S::DQ), t[i]);
    return d;
}
// sum over the 16 lanes of a row, left in all of them
__device__ __forceinline__ float row16_sum(float v)
{
    auto dpp = [](float x, auto ctrl) {
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value, 0xF, 0xF, true));
    };
    v += dpp(v, std::integral_constant<int, 0xB1>{});  // quad_perm [1,0,3,2]
    v += dpp(v, std::integral_constant<int, 0x4E>{});  // quad_perm [2,3,0,1]
    v += dpp(v, std::integral_constant<int, 0x141>{}); // row_half_mirror
    v += dpp(v, std::integral_constant<int, 0x140>{}); // row_mirror
    return v;
}

// Where the window's tokens lie and which mask region they belong to.
template <class S> struct Window {
    int b, wi, wj, H, W, s;
    bool last_r, last_c;
    __device__ __forceinline__ Window(const Geom &g, int w)
    {
        const int per = g.nwi * g.nwj;
        b = __builtin_amdgcn_readfirstlane(w / per); // (uniform, but divided on the vector ALU)
        const int r = w - b * per;
        wi = __builtin_amdgcn_readfirstlane(r / g.nwj);
        wj = r - wi * g.nwj;
        H = g.H; W = g.W; s = g.shift;
        last_r = s > 0 && wi == g.nwi - 1;
        last_c = s > 0 && wj == g.nwj - 1;
    }
    __device__ __forceinline__ long token(int n) const
    {
        const int r = n / S::M, c = n - r * S::M;
        int i = wi * S::M + r + s, j = wj * S::M + c + s;
        if (i >= H) i -= H;
        if (j >= W) j -= W;
        return ((long)b * H + i) * W + j;
    }
    // tokens of different regions do not attend to each other
    __device__ __forceinline__ int region(int n) const
    {
        const int r = n / S::M, c = n - r * S::M;
        return ((last_r && r >= S::M - s) ? 1 : 0) | ((last_c && c >= S::M - s) ? 2 : 0);
    }
};
// offset of a token in the bias table: the entry of (query, key) is key_offset(query) - key_offset(key) + a constant;
// of tokens 16 tile + 4q + i, which are neighbours in a window row (M is a multiple of four), it is that of i = 0 plus i
template <class S> __device__ __forceinline__ int key_offset(int n) { const int r = n / S::M; return r * S::NTB + (n - r * S::M); }
template <class S> __device__ __forceinline__ int key_offset4(int tile, int q)
{
    if (S::M == 8) return 2 * S::NTB * tile + S::NTB * (q >> 1) + 4 * (q & 1);
    static_assert(S::M == 8 || S::M == 12, "window size");
    return 4 * S::NTB * (tile / 3) + key_offset<S>(16 * (tile % 3) + 4 * q); // (12: three tiles are four window rows)
}

// A lane's place in LDS, kept in a register of its own: what a loop over tiles adds to it is then an offset of the read
// instruction (two or three instructions per read otherwise, with which the units of scores spent a quarter of their
// vector instructions).
template <typename E> __device__ __forceinline__ const E *lane_base(const E *p, int off)
{
    asm volatile("" : "+v"(off));
    return p + off;
}
// The lane's four bias entries of a score tile: with a query per column (keys of the tile in descending order), with a key
// per column.  Tiles KB apart differ by KSTEP entries.
template <class S> struct BiasOf {
    static constexpr int KB = S::M == 8 ? 1 : 3, KSTEP = S::M == 8 ? 2 * S::NTB : 4 * S::NTB, KN = S::NT / KB;
    static_assert(S::NT % KB == 0, "whole turns");
    const float *p[KB];
    bool query;
    __device__ __forceinline__ BiasOf(const float *tbh, int token, bool query_, int q) : query(query_)
    {
        const int o = key_offset<S>(token), mid = (S::M - 1) * (S::NTB + 1);
#pragma unroll
        for (int r = 0; r < KB; ++r)
            p[r] = lane_base(tbh, query ? mid + o - key_offset4<S>(r, 3 - q) - 3 - KSTEP * (KN - 1) : mid - o + key_offset4<S>(r, q));
    }
    __device__ __forceinline__ f32x4 tile(int t) const
    {
        const float *b = p[t % KB] + KSTEP * (query ? KN - 1 - t / KB : t / KB);
        return f32x4{b[0], b[1], b[2], b[3]};
    }
};

// feature of the padded q|k|v rows -> row of the group's weight block [q: QG | k: QG | v: CG], -1 for padding
template <class S> __device__ __forceinline__ int weight_row(int f)
{
    if (f < 2 * S::RQ) {
        const int part = f >= S::RQ ? 1 : 0, r = f - part * S::RQ, h = r / S::HSQ, e = r - h * S::HSQ;
        return e < S::DQ ? part * S::QG + h * S::DQ + e : -1;
    }
    const int r = f - 2 * S::RQ, h = r / S::HSV, e = r - h * S::HSV;
    return (r < S::RV && e < S::D) ? 2 * S::QG + h * S::D + e : -1;
}
// the same for features f .. f + 3, f a multiple of four (all in one head): rows row .. row + n - 1, the rest is padding
struct Rows4 { int row, n; };
template <class S> __device__ __forceinline__ Rows4 weight_rows4(int f)
{
    const bool v = f >= 2 * S::RQ;
    const int part = f >= S::RQ ? 1 : 0;
    const int rq = f - part * S::RQ, hq = rq / S::HSQ, eq = rq - hq * S::HSQ;
    const int rv = f - 2 * S::RQ, hv = (v ? rv : 0) / S::HSV, ev = rv - hv * S::HSV;
    Rows4 r;
    r.row = v ? 2 * S::QG + hv * S::D + ev : part * S::QG + hq * S::DQ + eq;
    r.n = v ? S::D - ev : S::DQ - eq;
    if (f >= S::RP) r.row = r.n = 0;
    return r;
}

// Weights as operands, straight from memory.  All loads of a tile are issued before the first product (the compiler,
// left alone, keeps four in flight: five trips to L2 per tile of 16 loads instead of one), so the values are masked
// where they are used.  Only the k-slots beyond the matrix are masked; rows beyond it are the caller's to drop.
// WeightsN: row `row` of a row-major matrix, k-slots along it (K and ld even).  WeightsT: column, k-slots down it.
template <typename E, int K> struct WeightsN;
template <typename E, int K> struct WeightsT;
template <int K> struct WeightsN<float, K> {
    static constexpr int KU = up(K, 16);
    f32x4 v[KU];
    __device__ __forceinline__ void load(const float *row, int q)
    {
#pragma unroll
        for (int s = 0; s < KU; ++s) {
            const int k = 16 * s + 4 * q;
            if (K % 4 == 0) { // (rows of a multiple of 16 bytes)
                v[s] = *reinterpret_cast<const f32x4 *>(row + (16 * s + 16 <= K || k < K ? k : 0));
            } else {
                const f32x2 lo = *reinterpret_cast<const f32x2 *>(row + (16 * s + 16 <= K || k < K ? k : 0));
                const f32x2 hi = *reinterpret_cast<const f32x2 *>(row + (16 * s + 16 <= K || k + 2 < K ? k + 2 : 0));
                v[s] = f32x4{lo[0], lo[1], hi[0], hi[1]};
            }
        }
    }
    __device__ __forceinline__ f32x4 op(int s, int q) const
    {
        const int k = 16 * s + 4 * q;
        if (16 * s + 16 <= K) return v[s];
        return f32x4{k < K ? v[s][0] : 0.f, k < K ? v[s][1] : 0.f, k + 2 < K ? v[s][2] : 0.f, k + 2 < K ? v[s][3] : 0.f};
    }
};
template <int K> struct WeightsT<float, K> {
    static constexpr int KU = up(K, 16);
    float v[KU][4];
    __device__ __forceinline__ void load(const float *col, int ld, int q)
    {
#pragma unroll
        for (int s = 0; s < KU; ++s)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int k = 16 * s + 4 * q + i;
                v[s][i] = col[(16 * s + 16 <= K || k < K ? k : 0) * ld];
            }
    }
    __device__ __forceinline__ f32x4 op(int s, int q) const
    {
        f32x4 r;
#pragma unroll
        for (int i = 0; i < 4; ++i) r[i] = (16 * s + 16 <= K || 16 * s + 4 * q + i < K) ? v[s][i] : 0.f;
        return r;
    }
};
template <int K> struct WeightsN<bf16_t, K> {
    static constexpr int KU = up(K, 16);
    uint2 v[KU];
    __device__ __forceinline__ void load(const bf16_t *row, int q)
    {
#pragma unroll
        for (int s = 0; s < KU; ++s) {
            const int k = 16 * s + 4 * q;
            if (K % 4 == 0) {
                v[s] = *reinterpret_cast<const uint2 *>(row + (16 * s + 16 <= K || k < K ? k : 0));
            } else if (K % 2 == 0) {
                v[s].x = *reinterpret_cast<const uint32_t *>(row + (16 * s + 16 <= K || k < K ? k : 0));
                v[s].y = *reinterpret_cast<const uint32_t *>(row + (16 * s + 16 <= K || k + 2 < K ? k + 2 : 0));
            } else { // (rows of an odd number of channels start anywhere)
                uint32_t e[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) e[i] = row[16 * s + 16 <= K || k + i < K ? k + i : 0].bits;
                v[s] = make_uint2(e[0] | e[1] << 16, e[2] | e[3] << 16);
            }
        }
    }
    __device__ __forceinline__ uint2 op(int s, int q) const
    {
        const int k = 16 * s + 4 * q;
        if (16 * s + 16 <= K) return v[s];
        if (K % 2 == 0) return make_uint2(k < K ? v[s].x : 0u, k + 2 < K ? v[s].y : 0u);
        return make_uint2((k < K ? v[s].x & 0xffffu : 0u) | (k + 1 < K ? v[s].x & 0xffff0000u : 0u),
                          (k + 2 < K ? v[s].y & 0xffffu : 0u) | (k + 3 < K ? v[s].y & 0xffff0000u : 0u));
    }
};
template <int K> struct WeightsT<bf16_t, K> {
    static constexpr int KU = up(K, 16);
    uint16_t v[KU][4];
    __device__ __forceinline__ void load(const bf16_t *col, int ld, int q)
    {
#pragma unroll
        for (int s = 0; s < KU; ++s)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int k = 16 * s + 4 * q + i;
                v[s][i] = col[(16 * s + 16 <= K || k < K ? k : 0) * ld].bits;
            }
    }
    __device__ __forceinline__ uint2 op(int s, int q) const
    {
        uint32_t e[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) e[i] = (16 * s + 16 <= K || 16 * s + 4 * q + i < K) ? v[s][i] : 0u;
        return make_uint2(e[0] | e[1] << 16, e[2] | e[3] << 16);
    }
};
// A row of the output projection, k-slots along the group-strided columns of the rows it multiplies.
template <class S> struct WeightsX {
    typename S::T v[S::KUX][4];
    WeightsN<typename S::T, S::C> n;
    __device__ __forceinline__ void load(const typename S::T *row, int q)
    {
        if (S::CGP == S::CG) { n.load(row, q); return; }
#pragma unroll
        for (int s = 0; s < S::KUX; ++s) {
            const int k = 16 * s + 4 * q, g = k / S::CGP, o = k - g * S::CGP;
#pragma unroll
            for (int i = 0; i < 4; ++i) v[s][i] = row[g < S::G && o + i < S::CG ? g * S::CG + o + i : 0];
        }
    }
    __device__ __forceinline__ typename Op<typename S::E>::F op(int s, int q) const
    {
        if (S::CGP == S::CG) return n.op(s, q);
        const int k = 16 * s + 4 * q, g = k / S::CGP, o = k - g * S::CGP;
        float e[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) e[i] = g < S::G && o + i < S::CG ? to_f32(v[s][i]) : 0.f;
        return Op<typename S::E>::gather(e[0], e[1], e[2], e[3]);
    }
};
__device__ __forceinline__ void loads_issued() { __builtin_amdgcn_sched_barrier(0); }

// Scores with a query per column are taken of the keys of a tile in descending order (row 4q + i is key 15 - 4q - i), so
// that a lane's four bias entries ascend in memory and enter the product as they are read.

// The row phases: 16 lanes hold a token, four channels each; a wave takes four tokens at a time.
template <class S> struct Rows {
    static constexpr int UNITS = S::N / 4, PER = up(UNITS, S::WAVES);
};
__device__ __forceinline__ f32x4 load4(const float *p) { return *reinterpret_cast<const f32x4 *>(p); }
__device__ __forceinline__ f32x4 load4(const bf16_t *p) { return Op<bf16_t>::wide(*reinterpret_cast<const uint2 *>(p)); }
// the same, or zeros (a load that no branch guards is not waited for before its value is used)
template <typename T> __device__ __forceinline__ f32x4 load4_if(bool ok, const T *base, long at)
{
    const f32x4 v = load4(base + (ok ? at : 0));
    return f32x4{ok ? v[0] : 0.f, ok ? v[1] : 0.f, ok ? v[2] : 0.f, ok ? v[3] : 0.f};
}
__device__ __forceinline__ void store4(float *p, f32x4 v) { *reinterpret_cast<f32x4 *>(p) = v; }

__device__ __forceinline__ void store4(bf16_t *p, f32x4 v) { *reinterpret_cast<uint2 *>(p) = pack_bf16x4(v); }
// four channels of a group-strided row; lane 15 (which holds no channels) clears the pad columns
template <class S> __device__ __forceinline__ void put_row(typename S::E *row, int l16, f32x4 v)
{
    using O = Op<typename S::E>;
    if (4 * l16 < S::C) {
        if (S::CGP == S::CG) O::st(row + 4 * l16, v);
        else {
#pragma unroll
            for (int i = 0; i < 4; ++i) O::put(row + S::xcol(4 * l16 + i), v[i]);
        }
    } else if (l16 == 15) {
#pragma unroll
        for (int g = 0; g < S::G; ++g)
#pragma unroll
            for (int c = S::CG; c < S::CGP; ++c) O::put(row + g * S::CGP + c, 0.f);
#pragma unroll
        for (int c = S::XW; c < S::PC; c += 4) O::st(row + c, zero4());
    }
}
template <class S> __device__ __forceinline__ f32x4 get_row(const typename S::E *row, int l16)
{
    using O = Op<typename S::E>;
    if (S::CGP == S::CG) return O::wide(O::ld(row + 4 * l16));
    f32x4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = O::get(row + S::xcol(4 * l16 + i < S::C ? 4 * l16 + i : 0));
    return v;
}

// fp32: the mask on top of scores; the lane's column is token `col`, its rows are tokens row0 + i (`up`) or row0 + 3 - i,
// row0 a multiple of four
template <class S> __device__ __forceinline__ f32x4 add_mask(const Window<S> &win, f32x4 s, int row0, bool up, int col)
{
    const int reg = win.region(col), r = row0 / S::M, c = row0 - r * S::M;
    const bool rows = ((reg & 1) != 0) != (win.last_r && r >= S::M - win.s);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const bool cols = ((reg & 2) != 0) != (win.last_c && c + (up ? i : 3 - i) >= S::M - win.s);
        s[i] += (rows || cols) ? -100.f * score_unit<float> : 0.f;
    }
    return s;
}

// the shift mask's parts of a token, behind its q|k|v
template <class S> __device__ __forceinline__ void put_mask(const Window<S> &win, typename S::E *R)
{
    using O = Op<typename S::E>;
    if (!QkOp<S>::SLOTS) return;
    for (int t = threadIdx.x; t < S::N; t += S::NTH) {
        const int reg = win.region(t);
        const float r = reg & 1 ? 1.f : 0.f, c = reg & 2 ? 1.f : 0.f, hi = -144.f, lo = -100.f * kLog2e - hi;
        const f32x4 coef = {r + c - r * c, (1.f - 2.f * r) * (1.f - c), (1.f - 2.f * c) * (1.f - r), -(1.f - 2.f * r) * (1.f - 2.f * c)};
        O::st(R + t * S::PR + S::MK, f32x4{1.f, r, c, r * c});
        O::st(R + t * S::PR + S::MQ, hi * coef);
        O::st(R + t * S::PR + S::MQ + 4, lo * coef);
    }
}

// v / C.  fp32: rounded once (1 / 60 alone is 5e-8 off, and with it every token's mean and variance, which cost a whole
// layer 2 to 5 % of its precision; no time)
template <class S> __device__ __forceinline__ float over_channels(float v)
{
    const float r = v * (1.f / S::C);
    return sizeof(typename S::E) == 2 ? r : fmaf(fmaf(-(float)S::C, r, v), 1.f / S::C, r);
}
// mean and 1 / sqrt(var + eps) of a token; lanes beyond the channels hold zeros
template <class S> __device__ __forceinline__ void stats(f32x4 f, bool in, float eps, float &mean, float &rstd)
{
    mean = over_channels<S>(row16_sum((f[0] + f[1]) + (f[2] + f[3])));
    float qs = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) { const float d = in ? f[i] - mean : 0.f; qs += d * d; }
    rstd = rsqrtf(over_channels<S>(row16_sum(qs)) + eps);
}

template <class S> __device__ __forceinline__ void load_table(float *tb, const typename S::T *table)
{
    constexpr int PER = up(S::NTBL * S::HEADS, S::NTH);
    typename S::T v[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int e = threadIdx.x + k * S::NTH;
        v[k] = table[e < S::NTBL * S::HEADS ? e : 0];
    }
    loads_issued();
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int e = threadIdx.x + k * S::NTH, i = e / S::HEADS, h = e - i * S::HEADS;
        if (e < S::NTBL * S::HEADS) tb[h * S::TBP + i] = to_f32(v[k]) * score_unit<typename S::E>;
    }
}

// q|k|v of group gi from X (+ the output of the group before it, A) into the padded rows R; q times log2(e) / sqrt(d)
template <class S> __device__ __forceinline__ void qkv_unit(const WindowLayerArgs &a, int gi, int ft, int tu, const typename S::E *X,
                                                            const typename S::E *A, typename S::E *R)
{
    FRESH_LANE;
    using O = Op<typename S::E>;
    const auto *w = static_cast<const typename S::T *>(a.w_qkv) + (long)gi * S::RG * S::CG;
    const auto *bias = static_cast<const typename S::T *>(a.b_qkv) + gi * S::RG;
    const int row = weight_row<S>(16 * ft + l16);
    WeightsN<typename S::E, S::CG> wf;
    wf.load(w + (row < 0 ? 0 : row) * S::CG, q);
    const Rows4 rows = weight_rows4<S>(16 * ft + 4 * q);
    float bf[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) bf[i] = to_f32(bias[i < rows.n ? rows.row + i : 0]);
    loads_issued();
    const bool casc = gi > 0 && a.g.cascade;
    const float pad = sizeof(typename S::E) == 2 && 16 * ft + 4 * q >= 2 * S::RQ ? 1.f : 0.f; // (bf16: v is one in the first pad feature: see window_layer_fwd_kernel)
    const float sc = 16 * ft + 4 * q < S::RQ && sizeof(typename S::E) == 2 ? kLog2e / sqrtf((float)S::DQ) : 1.f;
#pragma unroll
    for (int tt = 0; tt < S::TT; ++tt) {
        const int t = 16 * (tu * S::TT + tt) + l16;
        typename O::F f[S::KUG];
#pragma unroll
        for (int s = 0; s < S::KUG; ++s) f[s] = O::ld(X + t * S::PC + gi * S::CGP + 16 * s + 4 * q);
        f32x4 acc = zero4();
        if (casc) {
            // (Groups of an odd number of channels: W x + W o instead of W (x + o), whose sum would be rounded.  The
            // one-kernel-per-step path adds these in fp32; with the sum rounded four groups lose a fifth of their digits.)
#pragma unroll
            for (int s = 0; s < S::KUG; ++s) {
                const typename O::F o = O::ld(A + t * S::PC + (gi - 1) * S::CGP + 16 * s + 4 * q);
                if (sizeof(typename S::E) == 2 && S::CG % 2 != 0) acc = mma(wf.op(s, q), o, acc);
                else f[s] = O::add(f[s], o);
            }
        }
#pragma unroll
        for (int s = 0; s < S::KUG; ++s) acc = mma(wf.op(s, q), f[s], acc);
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] = i < rows.n ? (acc[i] + bf[i]) * sc : (i == rows.n ? pad : 0.f);
        if (16 * ft + 4 * q < S::RP) O::st(R + t * S::PR + 16 * ft + 4 * q, acc);
    }
}

template <class S, bool LAYER>
__global__ __launch_bounds__(S::NTH) void window_layer_fwd_kernel(WindowLayerArgs a)
{
    using E = typename S::E;
    using T = typename S::T;
    using O = Op<E>;
    using F = typename O::F;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    E *X = reinterpret_cast<E *>(lds + S::F_X), *A = reinterpret_cast<E *>(lds + S::F_A), *R = reinterpret_cast<E *>(lds + S::F_R);
    float *tb = reinterpret_cast<float *>(lds + S::fwd_tb(LAYER));
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const T *x = static_cast<const T *>(a.x);

    for (int w = blockIdx.x; w < a.g.nW; w += gridDim.x) {
        const Window<S> win(a.g, w);
        [[maybe_unused]] const bool masked = win.last_r || win.last_c;
        // ---- the window's rows (through LN_1) ----
        {
            FRESH_LANE;
            const bool in = 4 * l16 < S::C;
            f32x4 gam, bet;
            if (LAYER) {
                gam = load4_if(in, static_cast<const T *>(a.ln1_w), 4 * l16);
                bet = load4_if(in, static_cast<const T *>(a.ln1_b), 4 * l16);
            }
            typename O::F raw[Rows<S>::PER];
#pragma unroll
            for (int k = 0; k < Rows<S>::PER; ++k) {
                FRESH_LANE;
                const int t = 4 * (wv + k * S::WAVES) + q;
                raw[k] = O::ld(x + win.token(t < S::N ? t : 0) * S::C + (4 * l16 < S::C ? 4 * l16 : 0));
            }
            loads_issued();
            if (w == (int)blockIdx.x) load_table<S>(tb, static_cast<const T *>(a.table));
#pragma unroll
            for (int k = 0; k < Rows<S>::PER; ++k) {
                FRESH_LANE;
                const int t = 4 * (wv + k * S::WAVES) + q;
                f32x4 f = O::wide(O::pick(in, raw[k]));
                if (LAYER) {
                    float mean, rstd;
                    stats<S>(f, in, a.eps, mean, rstd);
#pragma unroll
                    for (int i = 0; i < 4; ++i) f[i] = in ? (f[i] - mean) * rstd * gam[i] + bet[i] : 0.f;
                }
                if (t < S::N) put_row<S>(X + t * S::PC, l16, f);
            }
        }
        // (columns of the group outputs that no head has written yet meet zero weights, but must be numbers)
        for (int e = 4 * threadIdx.x; e < S::N * S::PC; e += 4 * S::NTH) O::st(A + e, zero4());
        put_mask<S>(win, R);
        __syncthreads();
#pragma unroll 1
        for (int gi = 0; gi < S::G; ++gi) {
#pragma unroll 1
            for (int u = wv; u < S::NFT * S::TU; u += S::WAVES) qkv_unit<S>(a, gi, u / S::TU, u % S::TU, X, A, R);
            __syncthreads();
#pragma unroll 1
            for (int u = wv; u < S::HG * S::NT; u += S::WAVES) {
                FRESH_LANE;
                const int hl = u / S::NT, nt = u - hl * S::NT, tq = 16 * nt + l16;
                const BiasOf<S> bias(tb + (gi * S::HG + hl) * S::TBP, tq, true, q);
                const E *krow = lane_base(R, (15 - l16) * S::PR + QkOp<S>::at(S::RQ + hl * S::HSQ, false, q));
                QkOp<S> qf;
                qf.load(R + tq * S::PR + QkOp<S>::at(hl * S::HSQ, true, q));
                qf.mask(q);
                f32x4 st[S::NT];
#pragma unroll
                for (int kt = 0; kt < S::NT; ++kt) {
                    QkOp<S> kf;
                    kf.load(krow + 16 * kt * S::PR);
                    st[kt] = scores<S>(kf, qf, bias.tile(kt));
                }
                if (sizeof(E) == 4 && masked) {
#pragma unroll
                    for (int kt = 0; kt < S::NT; ++kt) st[kt] = add_mask<S>(win, st[kt], 16 * kt + 12 - 4 * q, false, tq);
                }
                float mx = max4f(st[0]);
#pragma unroll
                for (int kt = 1; kt < S::NT; ++kt) mx = max5f(mx, st[kt]);
                mx = qgroup_max(mx);
                f32x4 sum = zero4();
#pragma unroll
                for (int kt = 0; kt < S::NT; ++kt) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) st[kt][i] = prob<E>(st[kt][i] - mx);
                    if (sizeof(E) == 4) sum += st[kt];
                }
                f32x4 o = zero4();
#pragma unroll
                for (int kt = 0; kt < S::NT; ++kt)
                    o = mma(O::ld_tr(R + 16 * kt * S::PR + 2 * S::RQ + hl * S::HSV, S::PR, q, l16), O::from(st[kt]), o);
                // The softmax's denominator.  In bf16 v is one in feature D, so it is row D of the product: the sum of the
                // exponentials as rounded for the product; numerator and denominator share the roundings.  (Against the sum
                // of the fp32 exponentials, error of y over 48 layers each: (heads, groups, dqk) = (4, 1, 4) 3.64e-3 either
                // way, (6, 3, 4) 4.52e-3 and 4.53e-3, (6, 6, 4) 6.15e-3 and 6.21e-3.)
                static_assert(S::D % 4 != 0, "a pad feature");
                const float inv = 1.f / qgroup_sum(sizeof(E) == 4 ? (sum[0] + sum[1]) + (sum[2] + sum[3]) : q == S::D / 4 ? o[S::D % 4] : 0.f);
                E *ar = A + tq * S::PC + gi * S::CGP + hl * S::D;
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (4 * q + i < S::D) O::put(ar + 4 * q + i, o[i] * inv);
            }
            __syncthreads();
        }
        // ---- projection (Eq. 7), the skip of Eq. 4; the group outputs for the backward pass ----
        if (a.attn) {
#pragma unroll
            for (int k = 0; k < Rows<S>::PER; ++k) {
                FRESH_LANE;
                const int t = 4 * (wv + k * S::WAVES) + q;
                if (t < S::N && 4 * l16 < S::C) store4(static_cast<T *>(a.attn) + win.token(t) * S::C + 4 * l16, get_row<S>(A + t * S::PC, l16));
            }
        }
#pragma unroll 1
        for (int u = wv; u < S::CTC * S::PU; u += S::WAVES) {
            FRESH_LANE;
            const int ct = u / S::PU, tu = u - ct * S::PU, c = 16 * ct + 4 * q;
            const bool in = c < S::C;
            WeightsX<S> wf;
            wf.load(static_cast<const T *>(a.w_proj) + (16 * ct + l16 < S::C ? 16 * ct + l16 : 0) * S::C, q);
            const f32x4 b = load4(static_cast<const T *>(a.b_proj) + (in ? c : 0));
            F skip[S::TP];
            if (LAYER) {
#pragma unroll
                for (int tt = 0; tt < S::TP; ++tt) skip[tt] = O::ld(x + win.token(16 * (tu * S::TP + tt) + l16) * S::C + (in ? c : 0));
            }
            loads_issued();
#pragma unroll
            for (int tt = 0; tt < S::TP; ++tt) {
                const int t = 16 * (tu * S::TP + tt) + l16;
                f32x4 acc = zero4();
#pragma unroll
                for (int s = 0; s < S::KUX; ++s) acc = mma(wf.op(s, q), O::ld(A + t * S::PC + 16 * s + 4 * q), acc);
                acc += b;
                if (LAYER) acc += O::wide(skip[tt]);
                if (in) {
                    const long at = win.token(t) * S::C + c;
                    if (LAYER) {
                        O::st(X + t * S::PC + c, acc);
                        if (a.x1) store4(static_cast<T *>(a.x1) + at, acc);
                    } else {
                        store4(static_cast<T *>(a.y) + at, acc);
                    }
                }
            }
        }
        if (LAYER) {
            __syncthreads();
            // ---- LN_2 (over the group outputs), the MLP and its skip (Eq. 5) ----
            {
                FRESH_LANE;
                const bool in = 4 * l16 < S::C;
                const f32x4 gam = load4_if(in, static_cast<const T *>(a.ln2_w), 4 * l16);
                const f32x4 bet = load4_if(in, static_cast<const T *>(a.ln2_b), 4 * l16);
#pragma unroll
                for (int k = 0; k < Rows<S>::PER; ++k) {
                    FRESH_LANE;
                    const int t = 4 * (wv + k * S::WAVES) + q;
                    if (t < S::N) {
                        f32x4 f = in ? O::wide(O::ld(X + t * S::PC + 4 * l16)) : zero4();
                        float mean, rstd;
                        stats<S>(f, in, a.eps, mean, rstd);
#pragma unroll
                        for (int i = 0; i < 4; ++i) f[i] = in ? (f[i] - mean) * rstd * gam[i] + bet[i] : 0.f;
                        O::st(A + t * S::PC + 4 * l16, f);
                    }
                }
            }
            __syncthreads();
#pragma unroll 1
            for (int u = wv; u < S::HFT * S::TU; u += S::WAVES) {
                FRESH_LANE;
                const int ft = u / S::TU, tu = u - ft * S::TU;
                const bool in = 16 * ft + 4 * q < S::HID;
                WeightsN<E, S::C> wf;
                wf.load(static_cast<const T *>(a.w_fc1) + (16 * ft + l16 < S::HID ? 16 * ft + l16 : 0) * S::C, q);
                const f32x4 b = load4(static_cast<const T *>(a.b_fc1) + (in ? 16 * ft + 4 * q : 0));
                loads_issued();
#pragma unroll
                for (int tt = 0; tt < S::TT; ++tt) {
                    const int t = 16 * (tu * S::TT + tt) + l16;
                    f32x4 acc = zero4();
#pragma unroll
                    for (int s = 0; s < S::KUC; ++s) acc = mma(wf.op(s, q), O::ld(A + t * S::PC + 16 * s + 4 * q), acc);
#pragma unroll
                    for (int i = 0; i < 4; ++i) { float h, d; O::gelu(acc[i] + b[i], h, d); acc[i] = in ? h : 0.f; }
                    O::st(R + t * S::PH + 16 * ft + 4 * q, acc);
                }
            }
            __syncthreads();
#pragma unroll 1
            for (int u = wv; u < S::CTC * S::PU; u += S::WAVES) {
                FRESH_LANE;
                const int ct = u / S::PU, tu = u - ct * S::PU, c = 16 * ct + 4 * q;
                const bool in = c < S::C;
                WeightsN<E, S::HID> wf;
                wf.load(static_cast<const T *>(a.w_fc2) + (16 * ct + l16 < S::C ? 16 * ct + l16 : 0) * S::HID, q);
                const f32x4 b = load4(static_cast<const T *>(a.b_fc2) + (in ? c : 0));
                loads_issued();
#pragma unroll
                for (int tt = 0; tt < S::TP; ++tt) {
                    const int t = 16 * (tu * S::TP + tt) + l16;
                    f32x4 acc = zero4();
#pragma unroll
                    for (int s = 0; s < S::HFT; ++s) acc = mma(wf.op(s, q), O::ld(R + t * S::PH + 16 * s + 4 * q), acc);
                    acc += b + O::wide(O::ld(X + t * S::PC + c));
                    if (in) store4(static_cast<T *>(a.y) + win.token(t) * S::C + c, acc);
                }
            }
        }
        if (w + (int)gridDim.x < a.g.nW) __syncthreads(); // (the next window's rows go where this one's are read)
    }
}

// adds to (or, for the workgroup's first window, sets) an entry of the workgroup's vector of parameter gradients
__device__ __forceinline__ void put_grad(float *p, float v, bool first) { *p = first ? v : *p + v; }

// Four entries of the workgroup's vector of parameter gradients, `step` apart, the first n of them in use.  What earlier
// windows left there is read ahead of the products whose sums are added (read behind them, every tile of the second window
// of a workgroup waited for memory: 11 k of its 92 k clocks).
struct GradTile {
    float *p;
    int step, n;
    f32x4 old;
    __device__ __forceinline__ void load(bool first)
    {
        old = zero4();
        if (first) return;
#pragma unroll
        for (int i = 0; i < 4; ++i) old[i] = i < n ? p[i * step] : 0.f;
    }
    // (all sums before the first store: a wait for a load behind it waits for the store as well)
    __device__ __forceinline__ f32x4 sum(f32x4 v, bool first) const
    {
        f32x4 r = first ? v : old + v;
        asm volatile("" : "+v"(r));
        return r;
    }
    __device__ __forceinline__ void store(f32x4 r) const
    {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (i < n) p[i * step] = r[i];
    }
};
// result tile [16 rows of `rows`][16 columns] of a weight gradient: column `cols` is the bias gradient
__device__ __forceinline__ GradTile grad_tile(float *dw, float *db, int ld, int row0, int rows, int col, int cols, bool first)
{
    GradTile t;
    t.n = row0 >= rows || col > cols ? 0 : 4; // (rows is a multiple of four)
    t.p = t.n == 0 ? dw : col < cols ? dw + row0 * ld + col : db + row0;
    t.step = col < cols ? ld : 1;
    t.load(first);
    return t;
}

// four channels (piece k of 16) of a token's row of dn, fp32; the pieces of a row are exchanged so that 16 rows written at
// the same channels fall on different banks
template <class S> __device__ __forceinline__ float *dn_piece(float *dn, int t, int k)
{
    static_assert(S::CTC == 4, "16 pieces a row");
    return dn + (sizeof(typename S::E) == 4 ? S::PC : 64) * t + 4 * (k ^ (t & 15));
}

template <class S, bool LAYER>
__global__ __launch_bounds__(S::NTH) void window_layer_bwd_kernel(WindowLayerArgs a)
{
    using E = typename S::E;
    using T = typename S::T;
    using O = Op<E>;
    using F = typename O::F;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    E *X = reinterpret_cast<E *>(lds), *A = reinterpret_cast<E *>(lds + S::SZ_ROW), *DX = reinterpret_cast<E *>(lds + 2 * S::SZ_ROW);
    E *R = reinterpret_cast<E *>(lds + S::B_R), *DO = reinterpret_cast<E *>(lds + S::B_DO), *FO = reinterpret_cast<E *>(lds + S::B_FO);
    E *Hh = reinterpret_cast<E *>(lds + S::B_H), *DP = reinterpret_cast<E *>(lds + S::B_H + S::SZ_H);
    constexpr bool DN_IN_X = sizeof(E) == 4;
    float *DN = reinterpret_cast<float *>(DN_IN_X ? X : Hh);
    static_assert(DN_IN_X || sizeof(float) * S::N * 16 * S::CTC <= S::SZ_H, "dn in the hidden layer's place");
    float *tb = reinterpret_cast<float *>(lds + S::bwd_tb(LAYER));
    // of every query: bf16 its base-2 log-sum-exp, fp32 its largest score and 1 / the sum of exponentials; minus sum P dP
    float *lse = tb + S::HEADS * S::TBP, *delta = lse + S::HG * S::N, *rsum = delta + S::HG * S::N;
    float *red = lse;  // [WAVES][2][CP]
    constexpr int CP = 16 * up(S::C, 16);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const T *x = static_cast<const T *>(a.x);
    const float qscale = 1.f / sqrtf((float)S::DQ);
    float *part = a.part + (long)blockIdx.x * S::stride(LAYER);
    if (S::stride(LAYER) > (LAYER ? S::P_ALL : S::P_ATTN) && threadIdx.x < 4u) {
        const int e = (LAYER ? S::P_ALL : S::P_ATTN) + threadIdx.x;
        if (e < S::stride(LAYER)) part[e] = 0.f;
    }

    // gamma / beta sums over the tokens of a row phase: the four tokens of a wave here, the waves by finish_row_sums
    auto leave_row_sums = [&](f32x4 sg, f32x4 sb) {
        FRESH_LANE;
#pragma unroll
        for (int i = 0; i < 4; ++i) { sg[i] = qgroup_sum(sg[i]); sb[i] = qgroup_sum(sb[i]); }
        if (q == 0) {
            *reinterpret_cast<f32x4 *>(red + (wv * 2 + 0) * CP + 4 * l16) = sg;
            *reinterpret_cast<f32x4 *>(red + (wv * 2 + 1) * CP + 4 * l16) = sb;
        }
    };
    auto finish_row_sums = [&](int pg, int pb, bool first) { // behind a barrier
        for (int e = threadIdx.x; e < 2 * CP; e += S::NTH) {
            const int which = e / CP, c = e - which * CP;
            if (c >= S::C) continue;
            float s = 0.f;
#pragma unroll
            for (int k = 0; k < S::WAVES; ++k) s += red[(k * 2 + which) * CP + c];
            put_grad(part + (which ? pb : pg) + c, s, first);
        }
    };

    for (int w = blockIdx.x; w < a.g.nW; w += gridDim.x) {
        const Window<S> win(a.g, w);
        const bool first = w == (int)blockIdx.x;
        [[maybe_unused]] const bool masked = win.last_r || win.last_c;
        const f32x4 one_pad = {1.f, 0.f, 0.f, 0.f};
        if (!first) __syncthreads();
        if (LAYER) {
            // ---- Eq. 5 backwards.  A: LN_2(x1), DX: dy ----
            {
                FRESH_LANE;
                const bool in = 4 * l16 < S::C;
                const f32x4 gam = load4_if(in, static_cast<const T *>(a.ln2_w), 4 * l16);
                const f32x4 bet = load4_if(in, static_cast<const T *>(a.ln2_b), 4 * l16);
                F rx[Rows<S>::PER], rd[Rows<S>::PER];
#pragma unroll
                for (int k = 0; k < Rows<S>::PER; ++k) {
                    FRESH_LANE;
                    const int t = 4 * (wv + k * S::WAVES) + q;
                    const long tok = win.token(t < S::N ? t : 0) * S::C + (4 * l16 < S::C ? 4 * l16 : 0);
                    rx[k] = O::ld(static_cast<const T *>(a.x1) + tok);
                    rd[k] = O::ld(static_cast<const T *>(a.dy) + tok);
                }
                loads_issued();
                if (first) load_table<S>(tb, static_cast<const T *>(a.table));
#pragma unroll
                for (int k = 0; k < Rows<S>::PER; ++k) {
                    FRESH_LANE;
                    const int t = 4 * (wv + k * S::WAVES) + q;
                    if (t < S::N) {
                        f32x4 f = O::wide(O::pick(in, rx[k]));
                        const f32x4 d = O::wide(O::pick(in, rd[k]));
                        float mean, rstd;
                        stats<S>(f, in, a.eps, mean, rstd);
#pragma unroll
                        for (int i = 0; i < 4; ++i) f[i] = (f[i] - mean) * rstd * gam[i] + bet[i];
                        O::st(A + t * S::PC + 4 * l16, in ? f : (4 * l16 == S::C ? one_pad : zero4()));
                        O::st(DX + t * S::PC + 4 * l16, d);
                    }
                }
            }
            __syncthreads();
            // ---- hidden layer, its gradient through the GELU ----
#pragma unroll 1
            for (int u = wv; u < S::HFT * S::TU; u += S::WAVES) {
                FRESH_LANE;
                const int ft = u / S::TU, tu = u - ft * S::TU, f = 16 * ft + l16;
                const bool inf = 16 * ft + 4 * q < S::HID;
                WeightsN<E, S::C> w1;
                WeightsT<E, S::C> w2;
                w1.load(static_cast<const T *>(a.w_fc1) + (f < S::HID ? f : 0) * S::C, q);
                w2.load(static_cast<const T *>(a.w_fc2) + (f < S::HID ? f : 0), S::HID, q);
                const f32x4 b = load4(static_cast<const T *>(a.b_fc1) + (inf ? 16 * ft + 4 * q : 0));
                loads_issued();
#pragma unroll
                for (int tt = 0; tt < S::TT; ++tt) {
                    const int t = 16 * (tu * S::TT + tt) + l16;
                    f32x4 pre = zero4(), dh = zero4();
#pragma unroll
                    for (int s = 0; s < S::KUC; ++s) {
                        pre = mma(w1.op(s, q), O::ld(A + t * S::PC + 16 * s + 4 * q), pre);
                        dh = mma(w2.op(s, q), O::ld(DX + t * S::PC + 16 * s + 4 * q), dh);
                    }
                    f32x4 h;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        float hv, dv;
                        O::gelu(pre[i] + b[i], hv, dv);
                        h[i] = inf ? hv : 0.f;
                        dh[i] = inf ? dh[i] * dv : 0.f;
                    }
                    if (16 * ft + 4 * q == S::HID) h = one_pad;
                    O::st(Hh + t * S::PH + 16 * ft + 4 * q, h);
                    O::st(DP + t * S::PH + 16 * ft + 4 * q, dh);
                }
            }
            __syncthreads();
            // ---- d Wfc1 = dpre^T LN_2(x1);  d Wfc2 = dy^T h;  dn = dpre W1 ----
            // (weight gradients two column tiles at a time: they share the reading of the row tile)
            // dn is the start of LN_2's adjoint and its gamma / beta sums and stays in fp32.  X has the place for it where
            // rows are fp32; otherwise it goes where the hidden layer was, when that has been read.
            constexpr int U0 = S::CTC * S::TU, U1 = U0 + S::HFT * up(S::CTC, 2), U2 = U1 + S::CTC * up(S::HFT, 2);
            static_assert(S::CTC % 2 == 0 && S::HFT % 2 == 0, "pairs of column tiles");
            auto dn_unit = [&](int u) {
                FRESH_LANE;
                const int ct = u / S::TU, tu = u - ct * S::TU, c = 16 * ct + l16;
                WeightsT<E, S::HID> wf;
                wf.load(static_cast<const T *>(a.w_fc1) + (c < S::C ? c : 0), S::C, q);
                loads_issued();
#pragma unroll
                for (int tt = 0; tt < S::TT; ++tt) {
                    const int t = 16 * (tu * S::TT + tt) + l16;
                    f32x4 acc = zero4();
#pragma unroll
                    for (int s = 0; s < S::HFT; ++s) acc = mma(wf.op(s, q), O::ld(DP + t * S::PH + 16 * s + 4 * q), acc);
                    *reinterpret_cast<f32x4 *>(dn_piece<S>(DN, t, 4 * ct + q)) = acc;
                }
            };
#pragma unroll 1
            for (int u = DN_IN_X ? wv : U0 + wv; u < U2; u += S::WAVES) {
                FRESH_LANE;
                if (u < U0) {
                    dn_unit(u);
                } else if (u < U1) {
                    const int v = u - U0, ft = v / (S::CTC / 2), ct = 2 * (v - ft * (S::CTC / 2));
                    GradTile gt[2];
#pragma unroll
                    for (int p = 0; p < 2; ++p) gt[p] = grad_tile(part + S::P_W1, part + S::P_B1, S::C, 16 * ft + 4 * q, S::HID, 16 * (ct + p) + l16, S::C, first);
                    f32x4 acc[2] = {zero4(), zero4()};
#pragma unroll
                    for (int s = 0; s < S::NT; ++s) {
                        const F r = O::ld_t(DP + 16 * s * S::PH + 16 * ft, S::PH, q, l16);
#pragma unroll
                        for (int p = 0; p < 2; ++p) acc[p] = mma(r, O::ld_t(A + 16 * s * S::PC + 16 * (ct + p), S::PC, q, l16), acc[p]);
                    }
#pragma unroll
                    for (int p = 0; p < 2; ++p) acc[p] = gt[p].sum(acc[p], first);
#pragma unroll
                    for (int p = 0; p < 2; ++p) gt[p].store(acc[p]);
                } else {
                    const int v = u - U1, ct = v / (S::HFT / 2), ft = 2 * (v - ct * (S::HFT / 2));
                    GradTile gt[2];
#pragma unroll
                    for (int p = 0; p < 2; ++p) gt[p] = grad_tile(part + S::P_W2, part + S::P_B2, S::HID, 16 * ct + 4 * q, S::C, 16 * (ft + p) + l16, S::HID, first);
                    f32x4 acc[2] = {zero4(), zero4()};
#pragma unroll
                    for (int s = 0; s < S::NT; ++s) {
                        const F r = O::ld_t(DX + 16 * s * S::PC + 16 * ct, S::PC, q, l16);
#pragma unroll
                        for (int p = 0; p < 2; ++p) acc[p] = mma(r, O::ld_t(Hh + 16 * s * S::PH + 16 * (ft + p), S::PH, q, l16), acc[p]);
                    }
#pragma unroll
                    for (int p = 0; p < 2; ++p) acc[p] = gt[p].sum(acc[p], first);
#pragma unroll
                    for (int p = 0; p < 2; ++p) gt[p].store(acc[p]);
                }
            }
            __syncthreads();
            if (!DN_IN_X) {
#pragma unroll 1
                for (int u = wv; u < U0; u += S::WAVES) dn_unit(u);
                __syncthreads();
            }
        }
        // ---- rows: with the whole layer LN_2's adjoint and the skip of Eq. 5 (DX: dx1), LN_1(x) (X); A: group outputs ----
        {
            FRESH_LANE;
            const bool in = 4 * l16 < S::C;
            f32x4 gam1, bet1, gam2, sg = zero4(), sb = zero4();
            if (LAYER) {
                gam1 = load4_if(in, static_cast<const T *>(a.ln1_w), 4 * l16);
                bet1 = load4_if(in, static_cast<const T *>(a.ln1_b), 4 * l16);
                gam2 = load4_if(in, static_cast<const T *>(a.ln2_w), 4 * l16);
            }
            F rx[Rows<S>::PER], ra[Rows<S>::PER], ru[Rows<S>::PER]; // x, group outputs, and x1 or dy
#pragma unroll
            for (int k = 0; k < Rows<S>::PER; ++k) {
                FRESH_LANE;
                const int t = 4 * (wv + k * S::WAVES) + q;
                const long tok = win.token(t < S::N ? t : 0) * S::C + (4 * l16 < S::C ? 4 * l16 : 0);
                rx[k] = O::ld(x + tok);
                ra[k] = O::ld(static_cast<const T *>(a.attn) + tok);
                ru[k] = O::ld(static_cast<const T *>(LAYER ? a.x1 : a.dy) + tok);
            }
            loads_issued();
            if (!LAYER && first) load_table<S>(tb, static_cast<const T *>(a.table));
#pragma unroll
            for (int k = 0; k < Rows<S>::PER; ++k) {
                FRESH_LANE;
                const int t = 4 * (wv + k * S::WAVES) + q;
                if (t < S::N) {
                    const long tok = win.token(t) * S::C + 4 * l16;
                    f32x4 f = O::wide(O::pick(in, rx[k]));
                    const f32x4 at = O::wide(O::pick(in, ra[k]));
                    E *dr = DX + t * S::PC + 4 * l16;
                    float mean, rstd;
                    if (LAYER) {
                        const f32x4 u = O::wide(O::pick(in, ru[k]));
                        stats<S>(u, in, a.eps, mean, rstd);
                        f32x4 d = *reinterpret_cast<const f32x4 *>(dn_piece<S>(DN, t, l16)), xh;
                        float s1 = 0.f, s2 = 0.f;
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            d[i] = in ? d[i] : 0.f;
                            xh[i] = in ? (u[i] - mean) * rstd : 0.f;
                            sg[i] += d[i] * xh[i];
                            sb[i] += d[i];
                            d[i] *= gam2[i];
                            s1 += d[i];
                            s2 += d[i] * xh[i];
                        }
                        s1 = over_channels<S>(row16_sum(s1));
                        s2 = over_channels<S>(row16_sum(s2));
                        const f32x4 r = O::wide(O::ld(dr));
#pragma unroll
                        for (int i = 0; i < 4; ++i) d[i] = in ? rstd * (d[i] - s1 - xh[i] * s2) + r[i] : 0.f;
                        O::st(dr, d);
                        if (S::OVER && in) store4(static_cast<T *>(a.dx) + tok, d); // (read back by this lane at the end)
                        stats<S>(f, in, a.eps, mean, rstd);
#pragma unroll
                        for (int i = 0; i < 4; ++i) f[i] = in ? (f[i] - mean) * rstd * gam1[i] + bet1[i] : 0.f;
                    } else {
                        O::st(dr, O::wide(O::pick(in, ru[k])));
                    }
                    put_row<S>(X + t * S::PC, l16, f);
                    put_row<S>(A + t * S::PC, l16, at);
                }
            }
            if (LAYER) leave_row_sums(sg, sb);
        }
        __syncthreads();
        put_mask<S>(win, R); // (not before: dn lies there)
        if (LAYER) finish_row_sums(S::P_G2, S::P_E2, first);

#pragma unroll 1
        for (int gi = S::G - 1; gi >= 0; --gi) {
            const bool casc = gi > 0 && a.g.cascade;
            // ---- q|k|v of the group, dO = dY Wproj slice + the cascade gradient; once: d Wproj ----
            constexpr int U0 = S::NVT * S::TU, U1 = U0 + S::NFT * S::TU;
            constexpr int CX2 = up(S::CTX, 2);
            const int U2 = gi == S::G - 1 ? U1 + S::CTC * CX2 : U1;
#pragma unroll 1
            for (int u = wv; u < U2; u += S::WAVES) {
                FRESH_LANE;
                if (u < U0) {
                    const int vt = u / S::TU, tu = u - vt * S::TU;
                    const int fr = 16 * vt + l16, hr = fr / S::HSV, er = fr - hr * S::HSV;
                    const bool okr = fr < S::RV && er < S::D;
                    WeightsT<E, S::C> wf;
                    wf.load(static_cast<const T *>(a.w_proj) + (okr ? gi * S::CG + hr * S::D + er : 0), S::C, q);
                    loads_issued();
                    const int fo = 16 * vt + 4 * q, h = fo / S::HSV, e = fo - h * S::HSV; // (four features of one head)
                    const bool prev = gi < S::G - 1 && a.g.cascade;
#pragma unroll
                    for (int tt = 0; tt < S::TT; ++tt) {
                        const int t = 16 * (tu * S::TT + tt) + l16;
                        f32x4 acc = zero4();
#pragma unroll
                        for (int s = 0; s < S::KUC; ++s) acc = mma(wf.op(s, q), O::ld(DX + t * S::PC + 16 * s + 4 * q), acc);
                        const E *xp = X + t * S::PC + (gi + 1) * S::CGP + h * S::D + e;
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            if (prev) acc[i] += O::get(xp + i);
                            acc[i] = e + i < S::D ? acc[i] : 0.f;
                        }
                        if (fo < S::RV) O::st(DO + t * S::PD + fo, acc);
                    }
                } else if (u < U1) {
                    qkv_unit<S>(a, gi, (u - U0) / S::TU, (u - U0) % S::TU, X, A, R);
                } else {
                    const int v = u - U1, ot = v / CX2, ct = 2 * (v - ot * CX2);
                    GradTile gt[2];
#pragma unroll
                    for (int p = 0; p < 2; ++p) {
                        const int col = 16 * (ct + p) + l16, g = col / S::CGP, o = col - g * S::CGP;
                        const int c = col == S::OC ? S::C : (g < S::G && o < S::CG ? g * S::CG + o : S::C + 1);
                        gt[p] = grad_tile(part + S::P_WP, part + S::P_BP, S::C, 16 * ot + 4 * q, S::C, c, S::C, first);
                    }
                    f32x4 acc[2] = {zero4(), zero4()};
#pragma unroll
                    for (int s = 0; s < S::NT; ++s) {
                        const F r = O::ld_t(DX + 16 * s * S::PC + 16 * ot, S::PC, q, l16);
#pragma unroll
                        for (int p = 0; p < 2; ++p) {
                            if (S::CTX % 2 && ct + p >= S::CTX) continue;
                            F b = O::ld_t(A + 16 * s * S::PC + 16 * (ct + p), S::PC, q, l16);
                            if (16 * (ct + p) + l16 == S::OC) b = O::ones();
                            acc[p] = mma(r, b, acc[p]);
                        }
                    }
#pragma unroll
                    for (int p = 0; p < 2; ++p) acc[p] = gt[p].sum(acc[p], first);
#pragma unroll
                    for (int p = 0; p < 2; ++p) gt[p].store(acc[p]);
                }
            }
            __syncthreads();
            constexpr int UA = S::HG * S::NT, PA = up(UA, S::WAVES);
            // ---- query role: softmax, delta, dQ ----
            F dq[PA]; // (held as what LDS gets of them: a wave of a layer with one group holds five, and six dK and dV)
#pragma unroll
            for (int k = 0; k < PA; ++k) {
                __builtin_amdgcn_sched_barrier(0);
                FRESH_LANE;
                dq[k] = F{};
                f32x4 acc = zero4();
                const int u = wv + k * S::WAVES;
                if (u >= UA) continue;
                const int hl = u / S::NT, nt = u - hl * S::NT, tq = 16 * nt + l16;
                const BiasOf<S> bias(tb + (gi * S::HG + hl) * S::TBP, tq, true, q);
                const E *krow = lane_base(R, (15 - l16) * S::PR + QkOp<S>::at(S::RQ + hl * S::HSQ, false, q));
                const E *vrow = lane_base(R, (15 - l16) * S::PR + 2 * S::RQ + hl * S::HSV + HeadOp<E, S::HSV>::at(q));
                QkOp<S> qf;
                HeadOp<E, S::HSV> of;
                qf.load(R + tq * S::PR + QkOp<S>::at(hl * S::HSQ, true, q));
                of.load(DO + tq * S::PD + hl * S::HSV + HeadOp<E, S::HSV>::at(q));
                qf.mask(q);
                of.mask(q);
                f32x4 st[S::NT], dp[S::NT];
#pragma unroll
                for (int kt = 0; kt < S::NT; ++kt) {
                    QkOp<S> kf;
                    HeadOp<E, S::HSV> vf;
                    kf.load(krow + 16 * kt * S::PR);
                    vf.load(vrow + 16 * kt * S::PR);
                    st[kt] = scores<S>(kf, qf, bias.tile(kt));
                    dp[kt] = mma(vf, of, zero4());
                }
                if (sizeof(E) == 4 && masked) {
#pragma unroll
                    for (int kt = 0; kt < S::NT; ++kt) st[kt] = add_mask<S>(win, st[kt], 16 * kt + 12 - 4 * q, false, tq);
                }
                float mx = max4f(st[0]);
#pragma unroll
                for (int kt = 1; kt < S::NT; ++kt) mx = max5f(mx, st[kt]);
                mx = qgroup_max(mx);
                float sum = 0.f, dl = 0.f;
#pragma unroll
                for (int kt = 0; kt < S::NT; ++kt)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        st[kt][i] = prob<E>(st[kt][i] - mx);
                        sum += st[kt][i];
                        dl += st[kt][i] * dp[kt][i];
                    }
                sum = qgroup_sum(sum);
                const float inv = 1.f / sum;
                dl = qgroup_sum(dl) * inv;
                if (q == 0) {
                    lse[hl * S::N + tq] = sizeof(E) == 4 ? mx : mx + __log2f(sum);
                    if (sizeof(E) == 4) rsum[hl * S::N + tq] = inv;
                    delta[hl * S::N + tq] = -dl;
                }
#pragma unroll
                for (int kt = 0; kt < S::NT; ++kt) {
                    f32x4 ds;
#pragma unroll
                    for (int i = 0; i < 4; ++i) ds[i] = st[kt][i] * (dp[kt][i] - dl);
                    acc = mma(O::ld_tr(R + 16 * kt * S::PR + S::RQ + hl * S::HSQ, S::PR, q, l16), O::from(ds), acc);
                }
                dq[k] = O::from(acc * (inv * qscale));
            }
            __syncthreads();
            // The bias-table gradient of a head.  A lane owns the offset (dr, dc), 0 <= dr, dc < M, of a query from its key,
            // and the three that differ from it by M in either direction: for every key exactly one of the four has its
            // query inside the window (query = key + offset mod M), so a lane takes one term per key.
            constexpr int FP = up(S::N, 64); // wavefronts a head's fold takes
            auto fold = [&](int hl, int slot, int part0) {
                FRESH_LANE;
                const int pair = part0 * 64 + 16 * q + l16;
                if (pair >= S::N) return;
                const int dr = pair / S::M, dc = pair - dr * S::M;
                const E *fo = FO + slot * S::N * S::PF;
                float t00 = 0.f, t01 = 0.f, t10 = 0.f, t11 = 0.f; // (row wraps, column wraps)
                float keep[S::M], wrap[S::M];
                int off[S::M];
#pragma unroll
                for (int c = 0; c < S::M; ++c) {
                    const bool wc = c + dc >= S::M;
                    keep[c] = wc ? 0.f : 1.f;
                    wrap[c] = wc ? 1.f : 0.f;
                    off[c] = c * S::PF + (wc ? c + dc - S::M : c + dc);
                }
#pragma unroll 1
                for (int r = 0; r < S::M; ++r) {
                    const bool wr = r + dr >= S::M;
                    const E *row = fo + r * S::M * S::PF + (wr ? r + dr - S::M : r + dr) * S::M;
                    float v[S::M], s0 = 0.f, s1 = 0.f;
#pragma unroll
                    for (int c = 0; c < S::M; ++c) v[c] = O::get(row + off[c]);
#pragma unroll
                    for (int c = 0; c < S::M; ++c) {
                        s0 = fmaf(v[c], keep[c], s0);
                        s1 = fmaf(v[c], wrap[c], s1);
                    }
                    t00 += wr ? 0.f : s0; t01 += wr ? 0.f : s1;
                    t10 += wr ? s0 : 0.f; t11 += wr ? s1 : 0.f;
                }
                float *tg = part + S::P_TB + gi * S::HG + hl;
                const int e = ((dr + S::M - 1) * S::NTB + dc + S::M - 1) * S::HEADS;
                float *pt[4] = {tg + e, dc > 0 ? tg + e - S::M * S::HEADS : tg + e, dr > 0 ? tg + e - S::M * S::NTB * S::HEADS : tg + e,
                                dr > 0 && dc > 0 ? tg + e - S::M * (S::NTB + 1) * S::HEADS : tg + e};
                f32x4 t = {t00, t01, t10, t11};
                if (!first) t += f32x4{*pt[0], *pt[1], *pt[2], *pt[3]};
                asm volatile("" : "+v"(t)); // (as GradTile)
                *pt[0] = t[0];
                if (dc > 0) *pt[1] = t[1];
                if (dr > 0) *pt[2] = t[2];
                if (dr > 0 && dc > 0) *pt[3] = t[3];
            };
            // The same in two steps where LDS has room for what lies between (BLOCKS).  First the blocks [keys of a window row]
            // x [queries of a window row] at the same distance dr of the two rows are added up: a lane owns four
            // neighbouring queries of one column of keys and the distances dr and dr - M, M blocks in all, read eight
            // bytes at a time.  Then the diagonals of each sum.  `fold` reads two bytes at a time and is three wavefronts'
            // work that the others wait for (8.2 k clocks under the second head's key role, 5.5 k behind the last head's);
            // this is seven units of 2 k and nine of 1 k (32 48x48 patches, two groups, fwd + bwd: 113.0 -> 109.1 us; six
            // groups of six heads, 4 patches: 94 -> 87).
            constexpr int FB = up(S::M * S::M * S::M / 4, 64), FS = up(S::NTBL, 64);
            float *SB = reinterpret_cast<float *>(lds + S::B_END);
            auto fold_blocks = [&](int slot, int unit) {
                FRESH_LANE;
                const int task = unit * 64 + 16 * q + l16;
                if (task >= S::M * S::M * S::M / 4) return;
                const int cq = task % (S::M / 4), c = task / (S::M / 4) % S::M, dr = task / (S::M / 4 * S::M);
                const E *fo = FO + slot * S::N * S::PF + c * S::PF + 4 * cq;
                F v[S::M];
#pragma unroll
                for (int r = 0; r < S::M; ++r) v[r] = O::ld(fo + r * S::M * S::PF + (r + dr >= S::M ? r + dr - S::M : r + dr) * S::M);
                loads_issued();
                f32x4 near = zero4(), wrap = zero4(); // dr, dr - M
#pragma unroll
                for (int r = 0; r < S::M; ++r) {
                    const f32x4 x = O::wide(v[r]);
                    const float w = r + dr >= S::M ? 1.f : 0.f, n = 1.f - w;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        near[i] = fmaf(x[i], n, near[i]);
                        wrap[i] = fmaf(x[i], w, wrap[i]);
                    }
                }
                float *sb = SB + slot * S::NTB * S::N + c * S::M + 4 * cq;
                *reinterpret_cast<f32x4 *>(sb + (dr + S::M - 1) * S::N) = near;
                if (dr > 0) *reinterpret_cast<f32x4 *>(sb + (dr - 1) * S::N) = wrap;
            };
            auto fold_sums = [&](int hl, int slot, int unit) {
                FRESH_LANE;
                const int e = unit * 64 + 16 * q + l16;
                if (e >= S::NTBL) return;
                const int dri = e / S::NTB, dc = e - dri * S::NTB - (S::M - 1);
                const float *sb = SB + slot * S::NTB * S::N + dri * S::N;
                float *pt = part + S::P_TB + e * S::HEADS + gi * S::HG + hl;
                const float old = first ? 0.f : *pt; // (as GradTile)
                float v[S::M], sum = 0.f;
#pragma unroll
                for (int c = 0; c < S::M; ++c) v[c] = sb[c * S::M + (c + dc < 0 ? 0 : c + dc >= S::M ? S::M - 1 : c + dc)];
                loads_issued();
#pragma unroll
                for (int c = 0; c < S::M; ++c) sum += c + dc >= 0 && c + dc < S::M ? v[c] : 0.f;
                *pt = first ? sum : old + sum;
            };
            // ---- key role, NF heads at a time: dV, dK, and the score gradients for the table gradient.  With one round they
            // go to LDS as they come; with more they wait in registers until the heads before have been folded, which the
            // wavefronts without a tile do meanwhile. ----
            constexpr int UR = S::NF * S::NT, PR_ = up(UR, S::WAVES), SPARE = UR < S::WAVES ? S::WAVES - UR : S::WAVES;
            constexpr bool DIRECT = S::ROUNDS == 1;
            F dk[S::ROUNDS * PR_], dv[S::ROUNDS * PR_];
#pragma unroll
            for (int round = 0; round < S::ROUNDS; ++round) {
                F ds[PR_][S::NT];
#pragma unroll
            for (int j = 0; j < PR_; ++j) {
                __builtin_amdgcn_sched_barrier(0);
                FRESH_LANE;
                const int k = round * PR_ + j;
                dk[k] = dv[k] = F{};
                f32x4 ak = zero4(), av = zero4();
                const int u = wv + j * S::WAVES, slot = u / S::NT, hl = round * S::NF + slot;
                if (u >= UR || hl >= S::HG) continue;
                const int kt = u - slot * S::NT, tk = 16 * kt + l16;
                E *fo = FO + (slot * S::N + tk) * S::PF;
                const BiasOf<S> bias(tb + (gi * S::HG + hl) * S::TBP, tk, false, q);
                const E *qrow = lane_base(R, l16 * S::PR + QkOp<S>::at(hl * S::HSQ, true, q));
                const E *orow = lane_base(DO, l16 * S::PD + hl * S::HSV + HeadOp<E, S::HSV>::at(q));
                const float *srow = lane_base(lse, hl * S::N + 4 * q); // (statistics: base-2 log-sum-exp or maximum; minus sum P dP; 1 / sum)
                QkOp<S> kf;
                HeadOp<E, S::HSV> vf;
                kf.load(R + tk * S::PR + QkOp<S>::at(S::RQ + hl * S::HSQ, false, q));
                vf.load(R + tk * S::PR + 2 * S::RQ + hl * S::HSV + HeadOp<E, S::HSV>::at(q));
                kf.mask(q);
                vf.mask(q);
#pragma unroll
                for (int nt = 0; nt < S::NT; ++nt) {
                    QkOp<S> qf;
                    HeadOp<E, S::HSV> of;
                    qf.load(qrow + 16 * nt * S::PR);
                    of.load(orow + 16 * nt * S::PD);
                    const f32x4 ls = *reinterpret_cast<const f32x4 *>(srow + 16 * nt);
                    const f32x4 dl = *reinterpret_cast<const f32x4 *>(srow + S::HG * S::N + 16 * nt);
                    f32x4 p = scores<S>(qf, kf, bias.tile(nt)), d;
                    f32x4 dp = mma(of, vf, sizeof(E) == 4 ? zero4() : dl), rs; // dP - delta
                    if (sizeof(E) == 4) { dp += dl; rs = *reinterpret_cast<const f32x4 *>(srow + 2 * S::HG * S::N + 16 * nt); }
                    if (sizeof(E) == 4 && masked) p = add_mask<S>(win, p, 16 * nt + 4 * q, true, tk);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        p[i] = prob<E>(p[i] - ls[i]);
                        if (sizeof(E) == 4) p[i] *= rs[i];
                        d[i] = p[i] * dp[i];
                    }
                    ds[j][nt] = O::from(d);
                    if (DIRECT) *reinterpret_cast<F *>(fo + 16 * nt + 4 * q) = ds[j][nt]; // [key][query]: four queries of a key
                    av = mma(O::ld_t(DO + 16 * nt * S::PD + hl * S::HSV, S::PD, q, l16), O::from(p), av);
                    ak = mma(O::ld_t(R + 16 * nt * S::PR + hl * S::HSQ, S::PR, q, l16), ds[j][nt], ak);
                }
                dk[k] = O::from(ak * (sizeof(E) == 4 ? qscale : 1.f / kLog2e));
                dv[k] = O::from(av);
            }
                if (!DIRECT) {
                    if (round > 0)
#pragma unroll 1
                        for (int u = UR < S::WAVES ? wv - UR : wv; u >= 0 && u < S::NF * (S::BLOCKS ? FB : FP); u += SPARE) {
                            if constexpr (S::BLOCKS) fold_blocks(u / FB, u % FB);
                            else fold((round - 1) * S::NF + u / FP, u / FP, u % FP);
                        }
                    __syncthreads();
                    if (S::BLOCKS && round > 0)
#pragma unroll 1
                        for (int u = S::WAVES - 1 - wv; u < S::NF * FS; u += S::WAVES) fold_sums((round - 1) * S::NF + u / FS, u / FS, u % FS);
#pragma unroll
                    for (int j = 0; j < PR_; ++j) {
                        FRESH_LANE;
                        const int u = wv + j * S::WAVES, slot = u / S::NT;
                        if (u >= UR || round * S::NF + slot >= S::HG) continue;
                        E *fo = FO + (slot * S::N + 16 * (u - slot * S::NT) + l16) * S::PF;
#pragma unroll
                        for (int nt = 0; nt < S::NT; ++nt) *reinterpret_cast<F *>(fo + 16 * nt + 4 * q) = ds[j][nt];
                    }
                    if (round + 1 < S::ROUNDS) __syncthreads();
                }
            }
            if (DIRECT) __syncthreads();
            // ---- gradients over q|k|v ----
#pragma unroll
            for (int k = 0; k < PA; ++k) {
                FRESH_LANE;
                const int u = wv + k * S::WAVES, hl = u / S::NT, tt = u - hl * S::NT, t = 16 * tt + l16;
                if (u >= UA) continue;
                if (4 * q < S::HSQ) *reinterpret_cast<F *>(R + t * S::PR + hl * S::HSQ + 4 * q) = dq[k];
            }
#pragma unroll
            for (int k = 0; k < S::ROUNDS * PR_; ++k) {
                FRESH_LANE;
                const int round = k / PR_, u = wv + (k - round * PR_) * S::WAVES, slot = u / S::NT, hl = round * S::NF + slot;
                if (u >= UR || hl >= S::HG) continue;
                const int t = 16 * (u - slot * S::NT) + l16;
                if (4 * q < S::HSQ) *reinterpret_cast<F *>(R + t * S::PR + S::RQ + hl * S::HSQ + 4 * q) = dk[k];
                if (4 * q < S::HSV) *reinterpret_cast<F *>(R + t * S::PR + 2 * S::RQ + hl * S::HSV + 4 * q) = dv[k];
            }
            __syncthreads();
            // ---- table gradient, dF = d(q|k|v) Wqkv, d Wqkv = d(q|k|v)^T F ----
            constexpr int UF = S::CTG * S::TU, PX = up(UF, S::WAVES), CP2 = up(S::CTG, 2), V0 = S::NF * (S::BLOCKS ? FB : FP), V1 = V0 + S::NFT * CP2;
            f32x4 df[PX][S::TT];
            const T *wq = static_cast<const T *>(a.w_qkv) + (long)gi * S::RG * S::CG;
#pragma unroll
            for (int k = 0; k < PX; ++k) {
                FRESH_LANE;
                const int u = wv + k * S::WAVES;
#pragma unroll
                for (int tt = 0; tt < S::TT; ++tt) df[k][tt] = zero4();
                if (u >= UF) continue;
                const int ct = u / S::TU, tu = u - ct * S::TU, c = 16 * ct + l16;
                const T *wc = wq + (c < S::CG ? c : 0);
                constexpr int KB = S::KUR > 8 ? up(S::KUR, 2) : S::KUR; // (in two batches where the registers ask for it)
#pragma unroll
                for (int s0 = 0; s0 < S::KUR; s0 += KB) {
                    T v[KB][4];
#pragma unroll
                    for (int s = s0; s < s0 + KB && s < S::KUR; ++s) {
                        const Rows4 rows = weight_rows4<S>(16 * s + 4 * q);
                        const T *wr = wc + rows.row * S::CG;
#pragma unroll
                        for (int i = 0; i < 4; ++i) v[s - s0][i] = wr[i < rows.n ? i * S::CG : 0];
                    }
                    loads_issued();
#pragma unroll
                    for (int s = s0; s < s0 + KB && s < S::KUR; ++s) {
                        const Rows4 rows = weight_rows4<S>(16 * s + 4 * q);
                        const bool okk = 16 * s + 16 <= S::RP || 16 * s + 4 * q < S::RP;
                        float m[4];
#pragma unroll
                        for (int i = 0; i < 4; ++i) m[i] = i < rows.n ? to_f32(v[s - s0][i]) : 0.f;
                        const F wf = O::gather(m[0], m[1], m[2], m[3]);
#pragma unroll
                        for (int tt = 0; tt < S::TT; ++tt) {
                            const E *r = R + (16 * (tu * S::TT + tt) + l16) * S::PR;
                            df[k][tt] = mma(wf, O::pick(okk, O::ld(r + (okk ? 16 * s + 4 * q : 0))), df[k][tt]);
                        }
                    }
                    loads_issued();
                }
            }
            // (the wavefronts without tiles of dF take the first of the other units)
#pragma unroll 1
            for (int u = (wv + S::WAVES - UF % S::WAVES) % S::WAVES; u < V1; u += S::WAVES) {
                FRESH_LANE;
                if (u < V0) {
                    if constexpr (S::BLOCKS) { if ((S::ROUNDS - 1) * S::NF + u / FB < S::HG) fold_blocks(u / FB, u % FB); }
                    else { if ((S::ROUNDS - 1) * S::NF + u / FP < S::HG) fold((S::ROUNDS - 1) * S::NF + u / FP, u / FP, u % FP); }
                } else {
                    constexpr int P = S::CTG > 1 ? 2 : 1;
                    const int ft = (u - V0) / CP2, ct = P * ((u - V0) - ft * CP2);
                    const Rows4 rows = weight_rows4<S>(16 * ft + 4 * q);
                    GradTile gt[P];
#pragma unroll
                    for (int p = 0; p < P; ++p) {
                        const int c = 16 * (ct + p) + l16;
                        gt[p].n = c > S::CG ? 0 : rows.n < 4 ? rows.n : 4;
                        gt[p].p = c < S::CG ? part + S::P_WQ + (gi * S::RG + rows.row) * S::CG + c : part + S::P_BQ + gi * S::RG + rows.row;
                        gt[p].step = c < S::CG ? S::CG : 1;
                        gt[p].load(first);
                    }
                    f32x4 acc[P];
#pragma unroll
                    for (int p = 0; p < P; ++p) acc[p] = zero4();
#pragma unroll
                    for (int s = 0; s < S::NT; ++s) {
                        const F r = O::ld_t(R + 16 * s * S::PR + 16 * ft, S::PR, q, l16);
#pragma unroll
                        for (int p = 0; p < P; ++p) {
                            F b = O::ld_t(X + 16 * s * S::PC + gi * S::CGP + 16 * (ct + p), S::PC, q, l16);
                            if (casc) b = O::add(b, O::ld_t(A + 16 * s * S::PC + (gi - 1) * S::CGP + 16 * (ct + p), S::PC, q, l16));
                            if (16 * (ct + p) + l16 == S::CG) b = O::ones();
                            acc[p] = mma(r, b, acc[p]);
                        }
                    }
#pragma unroll
                    for (int p = 0; p < P; ++p) acc[p] = gt[p].sum(acc[p], first);
#pragma unroll
                    for (int p = 0; p < P; ++p) gt[p].store(acc[p]);
                }
            }
            __syncthreads();
            if (S::BLOCKS)
#pragma unroll 1
                for (int u = (wv + S::WAVES - UF % S::WAVES) % S::WAVES; u < S::NF * FS; u += S::WAVES)
                    if ((S::ROUNDS - 1) * S::NF + u / FS < S::HG) fold_sums((S::ROUNDS - 1) * S::NF + u / FS, u / FS, u % FS);
#pragma unroll
            for (int k = 0; k < PX; ++k) {
                FRESH_LANE;
                const int u = wv + k * S::WAVES;
                if (u >= UF) continue;
                const int ct = u / S::TU, tu = u - ct * S::TU;
#pragma unroll
                for (int tt = 0; tt < S::TT; ++tt) {
                    E *xr = X + (16 * (tu * S::TT + tt) + l16) * S::PC + gi * S::CGP + 16 * ct + 4 * q;
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (16 * ct + 4 * q + i < S::CG) O::put(xr + i, df[k][tt][i]);
                }
            }
            __syncthreads();
        }
        // ---- X is the gradient of the attention layer's input: out, or through LN_1's adjoint and the skip of Eq. 4 ----
        {
            FRESH_LANE;
            const bool in = 4 * l16 < S::C;
            f32x4 gam1, sg = zero4(), sb = zero4();
            if (LAYER) gam1 = load4_if(in, static_cast<const T *>(a.ln1_w), 4 * l16);
#pragma unroll
            for (int k = 0; k < Rows<S>::PER; ++k) {
                FRESH_LANE;
                const int t = 4 * (wv + k * S::WAVES) + q;
                if (t < S::N) {
                    const long tok = win.token(t) * S::C + 4 * l16;
                    f32x4 d = get_row<S>(X + t * S::PC, l16);
                    if (!in) d = zero4();
                    if (LAYER) {
                        const f32x4 f = load4_if(in, x, tok), r = S::OVER ? load4_if(in, static_cast<const T *>(a.dx), tok) : O::wide(O::ld(DX + t * S::PC + 4 * l16));
                        float mean, rstd, s1 = 0.f, s2 = 0.f;
                        stats<S>(f, in, a.eps, mean, rstd);
                        f32x4 xh;
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            xh[i] = in ? (f[i] - mean) * rstd : 0.f;
                            sg[i] += d[i] * xh[i];
                            sb[i] += d[i];
                            d[i] *= gam1[i];
                            s1 += d[i];
                            s2 += d[i] * xh[i];
                        }
                        s1 = over_channels<S>(row16_sum(s1));
                        s2 = over_channels<S>(row16_sum(s2));
#pragma unroll
                        for (int i = 0; i < 4; ++i) d[i] = rstd * (d[i] - s1 - xh[i] * s2) + r[i];
                    }
                    if (in) store4(static_cast<T *>(a.dx) + tok, d);
                }
            }
            if (LAYER) {
                leave_row_sums(sg, sb);
                __syncthreads();
                finish_row_sums(S::P_G1, S::P_E1, first);
            }
        }
    }
}

template <class S> bool matches(const Geom &g)
{
    return g.C == S::C && g.heads == S::HEADS && g.groups == S::G && g.M == S::M && g.dq == S::DQ;
}

template <class S, bool LAYER> hipError_t launch_fwd(const WindowLayerArgs &a, hipStream_t s)
{
    auto kern = window_layer_fwd_kernel<S, LAYER>;
    if (hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(kern), S::fwd_lds(LAYER)); e != hipSuccess) return e;
    const int grid = a.g.nW < 4096 ? a.g.nW : 4096;
    KernelTimer kt(LAYER ? K_LAYER_FWD : K_WINDOW_ATTN_FWD, s);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(S::NTH), S::fwd_lds(LAYER), s, a);
    return hipGetLastError();
}

template <class S, bool LAYER>
hipError_t launch_bwd(const WindowLayerArgs &a, const WindowLayerGrads &gr, int accumulate, hipStream_t s)
{
    auto kern = window_layer_bwd_kernel<S, LAYER>;
    if (hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(kern), S::bwd_lds(LAYER)); e != hipSuccess) return e;
    const int grid = a.g.nW < kWindowLayerVectors ? a.g.nW : kWindowLayerVectors;
    {
        KernelTimer kt(LAYER ? K_LAYER_BWD : K_WINDOW_BWD, s);
        hipLaunchKernelGGL(kern, dim3(grid), dim3(S::NTH), S::bwd_lds(LAYER), s, a);
    }
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    ReduceOut out{};
    float *ptr[13] = {gr.w_qkv, gr.b_qkv, gr.w_proj, gr.b_proj, gr.table, gr.w_fc1, gr.b_fc1, gr.w_fc2, gr.b_fc2, gr.ln1_w, gr.ln1_b, gr.ln2_w, gr.ln2_b};
    const int begin[14] = {S::P_WQ, S::P_BQ, S::P_WP, S::P_BP, S::P_TB, S::P_W1, S::P_B1, S::P_W2, S::P_B2, S::P_G1, S::P_E1, S::P_G2, S::P_E2, S::P_ALL};
    out.nseg = LAYER ? 13 : 5;
    for (int k = 0; k < out.nseg; ++k) out.ptr[k] = ptr[k];
    for (int k = 0; k <= out.nseg; ++k) out.begin[k] = begin[k];
    return launch_reduce(a.part, grid, S::stride(LAYER), out, accumulate, s);
}

template <class S> const WindowLayerOps *ops_of()
{
    static const WindowLayerOps ops = {{(size_t)S::stride(false), (size_t)S::stride(true)},
                                       {launch_fwd<S, false>, launch_fwd<S, true>},
                                       {launch_bwd<S, false>, launch_bwd<S, true>}};
    return &ops;
}

} // namespace

} // namespace gswa
