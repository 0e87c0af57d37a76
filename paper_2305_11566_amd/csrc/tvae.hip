// The refinement network exactly in the shape of Table I (Sec. III-B1):
// feature extraction, encoder with residual blocks, the one-channel mu /
// sigma head with the shifts of Eq. (8), decoder with 5x5 stride-2
// deconvolutions and skip connections, and the final upsampling layer; plus
// the loss of Eqs. (9)-(11).
//
// Layout: each level keeps one NHWC map whose channel ranges are the maps the
// table concatenates, in the table's order, so every "A & B & C" input is one
// contiguous channel range read by one convolution source:
//   level 1 (h1 x w1 = the coarse map): [D 16 | FE_1 32 | FE_2 32]        80 ch
//   level 2 (h1/2):                     [D_2 16 | EN_1 16 | EN_1_R 8 | D_2_R 8] 48 ch
//   level 3 (h1/4):                     [D_1 32 | EN_2 32 | EN_2_R 16 | D_1_R 16] 96 ch
// A stride-2 deconvolution is a stride-1 convolution with the flipped kernel
// over its input seen with zeros inserted between samples, cut to the size of
// the level it feeds (tconv.hip computes it without the zeros).  FE_1 and FE_2 run as one layer over the two
// input channels with block-diagonal weights.  The final upsampling layer
// (5x5, stride f, one output channel) is a 1x1 projection of the level-1 map and
// X_0 onto its 25 taps (MFMA) and a gather that adds, for each full-resolution
// pixel, the taps that land on it, in one kernel.
#include <algorithm>
#include <array>
#include <atomic>
#include <map>
#include <mutex>
#include <tuple>

#include "mfma.h"

namespace sv {

namespace {

#define SV_TRY_STATUS(x)            \
    do {                            \
        sv_status r_ = (x);         \
        if (r_ != SV_OK) return r_; \
    } while (0)

constexpr int TV_K = 5, TV_TAPS = 25;
constexpr int L1C = 80, L2C = 48, L3C = 96, ZC = 8, TC = 32;

// canonical layers, in the table's order: weights [out][in][k][k], then bias
struct CanonLayer { int cout, cin, k; };
constexpr CanonLayer kCanon[] = {
    {32, 1, 5},   // FE_1
    {32, 1, 5},   // FE_2
    {16, 64, 5},  // EN_1
    {8, 16, 5},   // EN_1_R
    {32, 24, 5},  // EN_2
    {16, 32, 5},  // EN_2_R
    {2, 48, 1},   // mu & sigma
    {32, 1, 1},   // D_1 (1x1 deconvolution)
    {16, 80, 5},  // D_1_R
    {16, 96, 5},  // D_2 (deconvolution, stride 2)
    {8, 40, 5},   // D_2_R
    {16, 48, 5},  // D (deconvolution, stride 2)
    {1, 81, 5},   // Y (upsampling layer, stride f)
};
constexpr int NCANON = 13;
enum { C_FE1 = 0, C_FE2, C_EN1, C_EN1R, C_EN2, C_EN2R, C_MS, C_D1, C_D1R, C_D2, C_D2R, C_D, C_Y };

// launched layers (FE_1 and FE_2 fused; Y as its tap projection)
enum { T_FE = 0, T_EN1, T_EN1R, T_EN2, T_EN2R, T_MS, T_D1, T_D1R, T_D2, T_D2R, T_D, T_YP, T_NL };
struct TvLayer { int cout, cin, k, stride; };  // stride of the launched convolution
constexpr TvLayer kLayers[T_NL] = {
    {64, 2, 5, 1}, {16, 64, 5, 2}, {8, 16, 5, 1}, {32, 24, 5, 2}, {16, 32, 5, 1}, {2, 48, 1, 1},
    {32, 1, 1, 1}, {16, 80, 5, 1}, {16, 96, 5, 1}, {8, 40, 5, 1}, {16, 48, 5, 1}, {TV_TAPS, 82, 1, 1},
};

int64_t canon_off(int i) {
    int64_t o = 0;
    for (int j = 0; j < i; ++j) o += (int64_t)kCanon[j].cout * kCanon[j].cin * kCanon[j].k * kCanon[j].k + kCanon[j].cout;
    return o;
}

inline int rup(int v, int m) { return (v + m - 1) / m * m; }

struct TvShape {
    int dtype, es;
    int n_pad[T_NL], cin_pad[T_NL];
    size_t w_off[T_NL], b_off[T_NL], bytes;
    // adjoint packs of the input gradient: rows = the layer's inputs (Y's
    // projection: the 80 level-1 channels), columns = its outputs; 0 for FE
    int bn_pad[T_NL], bcin_pad[T_NL];
    size_t bw_off[T_NL];
    // stride-2 deconvolutions (D_2, D) in polyphase form: per output parity
    // class a 3x3 kernel [9][n_pad][cin_pad] over the un-inserted input
    size_t ph_off[T_NL][4];
};

// Launched layers' input rows of the adjoint pack (0: no input gradient).
constexpr int kAdjRows[T_NL] = {0, 64, 16, 24, 32, 48, 1, 80, 96, 40, 48, 80};

TvShape tv_shape(int dtype) {
    TvShape s{};
    s.dtype = dtype;
    s.es = dtype_bytes(dtype);
    size_t off = 0;
    for (int i = 0; i < T_NL; ++i) {
        const TvLayer &l = kLayers[i];
        s.n_pad[i] = rup(l.cout, 16);
        s.cin_pad[i] = rup(l.cin, 8);
        // the tap projection stays FP32 in every mode, like the other network's
        // final layer: its few weights dominate the reduced-precision error
        const int les = i == T_YP ? 4 : s.es;
        s.w_off[i] = off;
        off = align256(off + (size_t)l.k * l.k * s.n_pad[i] * s.cin_pad[i] * les);
        s.b_off[i] = off;
        off = align256(off + (size_t)s.n_pad[i] * sizeof(float));
    }
    for (int i = 0; i < T_NL; ++i) {
        s.bw_off[i] = 0;
        s.bn_pad[i] = s.bcin_pad[i] = 0;
        if (!kAdjRows[i]) continue;
        s.bn_pad[i] = rup(kAdjRows[i], 16);
        s.bcin_pad[i] = rup(kLayers[i].cout, 8);
        const int les = i == T_YP ? 4 : s.es;
        s.bw_off[i] = off;
        off = align256(off + (size_t)kLayers[i].k * kLayers[i].k * s.bn_pad[i] * s.bcin_pad[i] * les);
    }
    for (int i = 0; i < T_NL; ++i)
        for (int ph = 0; ph < 4; ++ph) {
            s.ph_off[i][ph] = 0;
            if (i != T_D2 && i != T_D) continue;
            s.ph_off[i][ph] = off;
            off = align256(off + (size_t)9 * s.n_pad[i] * s.cin_pad[i] * s.es);
        }
    s.bytes = off;
    return s;
}

struct TvLevels { int H, W, h[4], w[4]; };  // h[1..3]: levels 1..3

TvLevels tv_levels(int f, int H, int W) {
    TvLevels lv{};
    lv.H = H; lv.W = W;
    lv.h[1] = cdiv(H, f); lv.w[1] = cdiv(W, f);
    for (int k = 2; k < 4; ++k) { lv.h[k] = cdiv(lv.h[k - 1], 2); lv.w[k] = cdiv(lv.w[k - 1], 2); }
    return lv;
}

struct TvAct { size_t L1, L2, L3, Z, ML, part, part_bytes, total; };

// output level of each launched layer
constexpr int kOutLevel[T_NL] = {1, 2, 2, 3, 3, 3, 3, 3, 2, 2, 1, 1};

TvAct tv_act(int es, const TvLevels &lv, int B) {
    auto px = [&](int k) { return (size_t)B * lv.h[k] * lv.w[k]; };
    TvAct a{};
    size_t o = 0;
    // partial sums of split-reduction launches (small grids): room for the
    // largest layer output at the maximum split, capped
    size_t part = 0;
    for (int i = 0; i < T_NL; ++i)
        part = std::max(part, (size_t)CONV_MAX_SPLIT * px(kOutLevel[i]) * rup(kLayers[i].cout, 16) * sizeof(float));
    a.part_bytes = std::min(part, CONV_PART_CAP);
    a.L1 = o; o = align256(o + px(1) * L1C * es);
    a.L2 = o; o = align256(o + px(2) * L2C * es);
    a.L3 = o; o = align256(o + px(3) * L3C * es);
    a.Z = o;  o = align256(o + px(3) * ZC * es);
    a.ML = o; o = align256(o + px(3) * 2 * sizeof(float));
    a.part = o; o = align256(o + a.part_bytes);
    a.total = o;
    return a;
}

std::atomic<int> g_tv_cfg[T_NL];
struct TvCfgInit {
    TvCfgInit() { for (auto &v : g_tv_cfg) v.store(-1); }
} g_tv_cfg_init;

// Configurations sv_tvae_autotune chose, per (dtype, factor, B, H, W), for
// this process.
std::mutex g_tv_mu;
std::map<std::tuple<int, int, int, int, int>, std::array<int, T_NL>> g_tv_tuned;

// Default: tile th4_tn16 / th4_tn32 by output width (EN_2, whose 32 outputs
// leave half the workgroups of the other coarse layers: th4_tn16 below 256
// workgroups, 4.7 us of a 163 us pass at batch 1, th8_tn32 where that still
// gives 200, 5 us at batch 16); grids of fewer than 256
// workgroups (the coarse levels of small batches) split the reduction over
// up to four channel ranges so that more CUs take part.
int tv_heuristic_cfg(int layer, int B, int Ho, int Wo) {
    const int tn = kLayers[layer].cout <= 16 ? 16 : 32;
    const int tile = tn == 16 ? T4_16 : T4_32;
    const long long nwg = (long long)cdiv(Wo, 16) * cdiv(Ho, 4) * B * cdiv(kLayers[layer].cout, tn);
    int split = 1;
    while (split < CONV_MAX_SPLIT && nwg * split < 256) ++split;
    if (layer == T_EN2) {
        if (nwg < 256) return T4_16 + conv_num_tiles() * (split - 1);
        if ((long long)cdiv(Wo, 16) * cdiv(Ho, 8) * B >= 200) return T8_32;
    }
    return tile + conv_num_tiles() * (split - 1);
}

// Per launched layer: an explicit override, else the tuned choice for this
// shape, else the heuristic.
void tv_layer_cfgs(int dtype, int f, int B, int H, int W, int *cfg) {
    const TvLevels lv = tv_levels(f, H, W);
    std::array<int, T_NL> tuned{};
    bool have = false;
    {
        std::lock_guard<std::mutex> g(g_tv_mu);
        auto it = g_tv_tuned.find(std::make_tuple(dtype, f, B, H, W));
        if (it != g_tv_tuned.end()) { tuned = it->second; have = true; }
    }
    for (int i = 0; i < T_NL; ++i) {
        const int ov = g_tv_cfg[i].load();
        const int k = kOutLevel[i];
        cfg[i] = (ov >= 0 && ov < conv_num_cfgs()) ? ov : (have ? tuned[i] : tv_heuristic_cfg(i, B, lv.h[k], lv.w[k]));
    }
}

// ---- packing ------------------------------------------------------------------------
__global__ void k_zero_bytes(uint32_t *__restrict__ p, size_t n_words) {
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < n_words; e += (size_t)gridDim.x * blockDim.x)
        p[e] = 0u;
}

// A deconvolution's stride-1 form over the zero-inserted input is the
// correlation with the flipped kernel; its polyphase packs keep the kernel.  A
// convolution's input gradient correlates the output gradient with the flipped
// kernel (over the zero-inserted gradient for stride 2); a deconvolution's is
// the stride-2 correlation with the kernel as it is.
sv_status tv_pack(const TvShape &s, const float *params, void *packed, hipStream_t st) {
    static constexpr int kCanonOf[T_NL] = {C_FE1, C_EN1, C_EN1R, C_EN2, C_EN2R, C_MS, C_D1, C_D1R, C_D2, C_D2R, C_D, C_Y};
    PackList list{};
    char *P = (char *)packed;
    for (int li = 0; li < T_NL; ++li) {
        const CanonLayer &c = kCanon[kCanonOf[li]];
        const float *w = params + canon_off(kCanonOf[li]);
        const float *bias = w + (size_t)c.cout * c.cin * c.k * c.k;
        const bool deconv = li == T_D2 || li == T_D, proj = li == T_YP;
        const int dt = proj ? SV_F32 : s.dtype;
        list.add(li == T_FE ? PK_FE : (proj ? PK_Y : PK_FWD), dt, w, c.cout, c.cin, c.k, s.n_pad[li], s.cin_pad[li],
                 deconv, P + s.w_off[li]);
        // the projection has no bias of its own: Y's, in its slot, is read by the gather
        float *bd = (float *)(P + s.b_off[li]);
        list.add(PK_BIAS, SV_F32, bias, c.cout, 0, 1, li == T_FE ? 32 : s.n_pad[li], 1, 0, bd);
        if (li == T_FE)
            list.add(PK_BIAS, SV_F32, params + canon_off(C_FE2) + 32 * TV_TAPS, 32, 0, 1, 32, 1, 0, bd + 32);
        if (kAdjRows[li])
            list.add(proj ? PK_YADJ : PK_ADJ, dt, w, c.cout, c.cin, c.k, s.bn_pad[li], s.bcin_pad[li],
                     !deconv && c.k > 1, P + s.bw_off[li]);
        if (deconv)
            for (int ph = 0; ph < 4; ++ph)
                list.add(PK_PHASE, dt, w, c.cout, c.cin, c.k, s.n_pad[li], s.cin_pad[li], ph, P + s.ph_off[li][ph]);
    }
    return launch_pack(list, st);
}

// ---- Eq. (8) and the final gather ------------------------------------------------
// z = (mu - 1) + eps * exp(sigma - 1) (eps NULL: z = mu - 1), stored as channel 0
// of an 8-channel row (channels 1..7 zero) so that the 1x1 deconvolution reads
// whole channel groups.
template <int DT>
__global__ void k_tv_reparam(const float *__restrict__ ml, const float *__restrict__ eps, int n,
                             typename Elem<DT>::T *__restrict__ z) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    float v = ml[2 * i] - 1.0f;
    if (eps) v += eps[i] * expf(ml[2 * i + 1] - 1.0f);
    typename Elem<DT>::T *o = z + (size_t)i * ZC;
    o[0] = Elem<DT>::make(v);
#pragma unroll
    for (int c = 1; c < ZC; ++c) o[c] = Elem<DT>::make(0.f);
}

// The upsampling layer: the 25 tap projections T[t] = w[t] . [D | FE | x0] of
// each level-1 pixel (FP32 weights, FP32 matrix steps, the map as stored) and
//   out[b][y][x] = 256 * (bias + sum over level-1 pixels (i, j) and taps (u, v)
//   with f*i + u - 2 = y, f*j + v - 2 = x of T[i][j][5u + v]), rows i and
//   columns j ascending,
// in one kernel.  It is bound by reading the map (160 bytes a pixel in 16 bits)
// and writing the result; the projections stay in LDS, where storing them cost
// 128 bytes a pixel written and read again.  A workgroup makes the outputs of
// 16 x 8 level-1 pixels from the projections of these and of the HL before /
// HH after them that an output's five taps reach, 16 pixels at a time on a wave:
// lane group g multiplies channels 20 g .. 20 g + 19, five loads of four channels
// straight from the map, and the weights stay in registers for all of a
// workgroup's tiles.  BF16 maps take three BF16 steps of 32 channels in place of
// eight FP32 steps of 4, the weight as the sum of three parts (24 bits; against
// 64 bits its error is below the FP32 steps'): 52 -> 33 us.
// Two kernels before: 16 BF16 images of 1242x375 125 -> 33 us, one in FP32 14.3
// -> 9.2, 4 of 512x256 at factor 2 in FP32 34 -> 20.
constexpr int TF_TW = 16, TF_TH = 8;

template <int F>  // the factor; 0: any from 3
struct FinalTile {
    static constexpr int HL = F == 1 ? 2 : F == 2 ? 1 : 0, HH = F == 1 ? 2 : 1;
    static constexpr int PW = TF_TW + HL + HH, PH = TF_TH + HL + HH, NPIX = PW * PH;
    static constexpr int NG = (NPIX + 15) / 16;
    // plane pitch: a step's four lane groups write 16 banks apart
    static constexpr int PITCH = (NG * 16 + 43) / 64 * 64 + 20;
};

// An output's sum straight from the maps in FP32 products, for one that the weight's
// parts leave not finite: a part that is zero or of the other sign makes NaN of an
// infinity of the map, and the first part of a weight past the largest BF16 value is
// an infinity itself.
template <int DT>
__device__ __forceinline__ float tv_final_sum(const typename Elem<DT>::T *__restrict__ L1, const uint8_t *__restrict__ disp,
                                              const uint8_t *__restrict__ img, float scale0, const float *__restrict__ wpk,
                                              int cin_pad, size_t ib, int h, int w, int f, int y, int x) {
    float s = 0.f;
    for (int i = max(0, (y - 2 + 3 * f - 1) / f - 2); i <= min(h - 1, (y + 2) / f); ++i)
        for (int j = max(0, (x - 2 + 3 * f - 1) / f - 2); j <= min(w - 1, (x + 2) / f); ++j) {
            const size_t q = ib + (size_t)i * w + j;
            const float *wr = wpk + ((y + 2 - f * i) * TV_K + x + 2 - f * j) * cin_pad;
            float t = fmaf(wr[81], (float)img[q] * (1.0f / 256.0f), wr[80] * (scale0 * (float)disp[q]));
#pragma unroll 1
            for (int c = 0; c < L1C; ++c) t = fmaf(wr[c], Elem<DT>::load(L1 + q * L1C + c), t);
            s += t;
        }
    return s;
}

template <int DT, int F>
__global__ void __launch_bounds__(256, 4)
k_tv_final(const typename Elem<DT>::T *__restrict__ L1, const uint8_t *__restrict__ disp,
           const uint8_t *__restrict__ img, float scale0, const float *__restrict__ wpk, int cin_pad,
           const float *__restrict__ bias, int h, int w, int f_any, int H, int W, int tiles_x, int tiles_y, int tiles,
           float *__restrict__ out) {
    using G = FinalTile<F>;
    using ST = typename Elem<DT>::T;
    typedef ST S4 __attribute__((ext_vector_type(4)));
    // BF16: the FP32 weight is the sum of three BF16 parts (24 bits)
    constexpr bool SPLIT = DT == SV_BF16;
    const int f = F ? F : f_any;
    __shared__ float T[TV_TAPS * G::PITCH];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int g = lane >> 4, r16 = lane & 15;
    // this lane's weights: tap 16 n + r16, channels 20 g .. 20 g + 19; x0's two (groups 0, 1)
    float ax[2];
    float af[SPLIT ? 1 : 2][20];
    u16x8 as[SPLIT ? 2 : 1][3][3];  // [block][eight channels][part]
#pragma unroll
    for (int n = 0; n < 2; ++n) {
        const float *wr = wpk + (size_t)(16 * n + r16) * cin_pad;
        ax[n] = g < 2 ? wr[80 + g] : 0.f;
#pragma unroll
        for (int i = 0; i < (SPLIT ? 24 : 20); ++i) {
            if constexpr (!SPLIT) {
                af[n][i] = wr[20 * g + i];
            } else {
                float v = i < 20 ? wr[20 * g + i] : 0.f;
#pragma unroll
                for (int p = 0; p < 3; ++p) {
                    const ST q = Elem<DT>::make(v);
                    as[n][i / 8][p][i % 8] = q;
                    const float qf = Elem<DT>::load(&q);
                    v = fabsf(qf) < INFINITY ? v - qf : 0.f;
                }
            }
        }
    }
    bool odd = false;  // (BF16) one of this thread's sums is not finite
    for (int t = blockIdx.x; t < tiles; t += gridDim.x) {
        const int b = t / (tiles_x * tiles_y), r = t - b * tiles_x * tiles_y;
        const int i0 = r / tiles_x * TF_TH, j0 = r % tiles_x * TF_TW;
        const size_t ib = (size_t)b * h * w;
        // ---- projections ------------------------------------------------------
        S4 x[5];
        float x0 = 0.f;
        auto load = [&](int grp) {
            // (pixels outside the map are read at its edge and not used)
            const int px = min(grp * 16 + r16, G::NPIX - 1), py = px / G::PW;
            const int i = min(max(i0 - G::HL + py, 0), h - 1), j = min(max(j0 - G::HL + px - py * G::PW, 0), w - 1);
            const size_t q = ib + (size_t)i * w + j;
            const ST *s = L1 + q * L1C + 20 * g;
#pragma unroll
            for (int k = 0; k < 5; ++k) x[k] = *(const S4 *)(s + 4 * k);
            const float v = (float)(g == 0 ? disp : img)[q];
            x0 = g == 0 ? scale0 * v : v * (1.0f / 256.0f);
        };
        load(wave);
        for (int grp = wave; grp < G::NG; grp += 4) {
            // NS sums a block (shorter chains, of steps and of roundings)
            constexpr int NS = SPLIT ? 2 : 4;
            f32x4 c[2][NS];
#pragma unroll
            for (int k = 0; k < 2 * NS; ++k) c[k % 2][k / 2] = f32x4{0.f, 0.f, 0.f, 0.f};
            const float x0c = x0;
            if constexpr (SPLIT) {
                u16x8 xb[3];
#pragma unroll
                for (int k = 0; k < 6; ++k)
#pragma unroll
                    for (int e = 0; e < 4; ++e) xb[k / 2][k % 2 * 4 + e] = k < 5 ? (uint16_t)x[k < 5 ? k : 0][e] : (uint16_t)0;
                if (grp + 4 < G::NG) load(grp + 4);
#pragma unroll
                for (int k = 0; k < 3; ++k)
#pragma unroll
                    for (int p = 2; p >= 0; --p)
#pragma unroll
                        for (int n = 0; n < 2; ++n) {
                            f32x4 &a = c[n][p == 0];
                            a = Mfma<DT>::run(as[n][k][p], xb[k], a);
                        }
            } else {
                float xv[20];
#pragma unroll
                for (int k = 0; k < 5; ++k)
#pragma unroll
                    for (int e = 0; e < 4; ++e) xv[4 * k + e] = Elem<DT>::load((const ST *)&x[k] + e);
                if (grp + 4 < G::NG) load(grp + 4);
#pragma unroll
                for (int i = 0; i < 20; ++i)
#pragma unroll
                    for (int n = 0; n < 2; ++n) {
                        f32x4 &a = c[n][i % NS];
                        a = __builtin_amdgcn_mfma_f32_16x16x4f32(af[n][i], xv[i], a, 0, 0, 0);
                    }
            }
#pragma unroll
            for (int n = 0; n < 2; ++n) {
                f32x4 s = c[n][0] + c[n][1];
                if constexpr (NS == 4) s += c[n][2] + c[n][3];
                s = __builtin_amdgcn_mfma_f32_16x16x4f32(ax[n], x0c, s, 0, 0, 0);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int tap = 16 * n + 4 * g + e;
                    if (tap < TV_TAPS) T[tap * G::PITCH + grp * 16 + r16] = s[e];
                }
            }
        }
        __syncthreads();
        // ---- gather -------------------------------------------------------------
        const int ow = TF_TW * f, oh = TF_TH * f;
        const float bv = bias[0];
        for (int e = threadIdx.x; e < ow * oh; e += 256) {
            const int oy = e / ow, ox = e - oy * ow;
            const int y = i0 * f + oy, xx = j0 * f + ox;
            if (y >= H || xx >= W) continue;
            // i with 0 <= y + 2 - f i <= 4
            const int ilo = max(0, (y - 2 + f - 1 + 2 * f) / f - 2), ihi = min(h - 1, (y + 2) / f);
            const int jlo = max(0, (xx - 2 + f - 1 + 2 * f) / f - 2), jhi = min(w - 1, (xx + 2) / f);
            float s = 0.f;
            for (int i = ilo; i <= ihi; ++i) {
                const int u = y + 2 - f * i;
                for (int j = jlo; j <= jhi; ++j) {
                    const int v = xx + 2 - f * j;
                    s += T[(u * TV_K + v) * G::PITCH + (i - i0 + G::HL) * G::PW + j - j0 + G::HL];
                }
            }
            if (SPLIT) odd |= !(fabsf(s) < INFINITY);
            out[((size_t)b * H + y) * W + xx] = 256.0f * (s + bv);
        }
        __syncthreads();
    }
    if constexpr (SPLIT) {
        if (!odd) return;
        // every thread's own outputs again (here, where the weights' registers are free)
        for (int t = blockIdx.x; t < tiles; t += gridDim.x) {
            const int b = t / (tiles_x * tiles_y), r = t - b * tiles_x * tiles_y;
            const int i0 = r / tiles_x * TF_TH, j0 = r % tiles_x * TF_TW;
            const int ow = TF_TW * f, oh = TF_TH * f;
            for (int e = threadIdx.x; e < ow * oh; e += 256) {
                const int y = i0 * f + e / ow, x = j0 * f + e % ow;
                if (y >= H || x >= W) continue;
                float *o = out + ((size_t)b * H + y) * W + x;
                if (fabsf(*o) < INFINITY) continue;
                *o = 256.0f * (tv_final_sum<DT>(L1, disp, img, scale0, wpk, cin_pad, (size_t)b * h * w, h, w, f, y, x) + bias[0]);
            }
        }
    }
}

template <int DT>
sv_status tv_final(const TvShape &s, const void *packed, const void *L1, const uint8_t *disp, const uint8_t *img,
                   int B, int h, int w, int f, int H, int W, float *out, hipStream_t st) {
    using ST = typename Elem<DT>::T;
    const int tx = cdiv(w, TF_TW), ty = cdiv(h, TF_TH), tiles = B * tx * ty;
    auto run = [&](auto *fn) {
        const long long n = resident_grid((const void *)fn, 0, tiles);
        hipLaunchKernelGGL(fn, dim3((unsigned)n), dim3(256), 0, st, (const ST *)L1, disp, img, (float)f / 256.0f,
                           (const float *)((const char *)packed + s.w_off[T_YP]), s.cin_pad[T_YP],
                           (const float *)((const char *)packed + s.b_off[T_YP]), h, w, f, H, W, tx, ty, tiles, out);
    };
    switch (f) {
    case 1: run(k_tv_final<DT, 1>); break;
    case 2: run(k_tv_final<DT, 2>); break;
    case 4: run(k_tv_final<DT, 4>); break;
    default: run(k_tv_final<DT, 0>); break;
    }
    SV_LAUNCH_CHECK("k_tv_final");
    return SV_OK;
}

__global__ void k_tv_copy(const float *__restrict__ src, int n, float *__restrict__ dst) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

ConvSrc tsrc(const void *p, int C, int pitch, int coff, int hs, int ws, int kind, int sdt) {
    ConvSrc s{};
    s.ptr = p; s.kind = kind; s.C = C; s.pitch = pitch; s.coff = coff; s.hs = hs; s.ws = ws; s.sdt = sdt;
    return s;
}

// Form of the stride-2 deconvolutions: -1 their own kernel (k_tconv; tv_deconv2 has
// the exceptions), 0 the general convolution over the zero-inserted grid, 1 as four
// polyphase ones (a
// pass of 16 BF16 images of 1242x375 261 us by the first against 341 by the
// faster of the others for each layer, of one in FP32 136 against 148).
std::atomic<int> g_tv_deconv_form{-1};

// Feature extraction (FE_1 = conv5x5(X_0), FE_2 = conv5x5(X_1), 32 outputs
// each, leaky ReLU) into channels 16..79 of the level-1 map.  Bound by writing
// these (128 bytes a pixel in 16 bits); as a stencil on the vector units it was
// bound by its 25 products an output and their weight reads instead, so the
// FP32 matrix steps take them, in every type: rows = outputs, columns = 16
// pixels of a row, k = four taps in order, so that a sum is the same chain of
// fused products, tap by tap from the bias, as a loop over the taps has.  A
// workgroup owns 16 x TH pixels, its wave TH / 4 rows; the patch with its 2-pixel
// halo is built in LDS from the uint8 maps.  Row 4 i + r of the two blocks of a
// branch is output 8 i + r and 8 i + 4 + r: a lane ends up with eight neighbouring
// outputs of one pixel and stores them at once.
// Measured (us): 16 BF16 images of 1242x375 41.8 -> 31.3,
// one in FP32 12.2 -> 9.6, 4 of 512x256 at factor 2 in FP32 23.2 -> 13.6.
constexpr int FE_TW = 16, FE_PW = FE_TW + 4;

template <int DT, int TH>
__global__ void __launch_bounds__(256)
k_tv_fe(const uint8_t *__restrict__ disp, const uint8_t *__restrict__ img, int h, int w, float scale0,
        const typename Elem<DT>::T *__restrict__ wpk, int n_pad, int cin_pad, const float *__restrict__ bias,
        typename Elem<DT>::T *__restrict__ out) {
    using T = typename Elem<DT>::T;
    constexpr int NK = (TV_TAPS + 3) / 4, PH = TH + 4, WP = 65;
    typedef T V __attribute__((ext_vector_type(16 / sizeof(T))));
    __shared__ float xs[2][PH * FE_PW];
    __shared__ float ws[NK * 4 * WP];  // [tap][output], taps 25..27 zero
    const int b = blockIdx.z;
    const int x0 = blockIdx.x * FE_TW, y0 = blockIdx.y * TH;
    const size_t ib = (size_t)b * h * w;
    for (int e = threadIdx.x; e < 64 * NK * 4; e += 256) {
        const int t = e >> 6, o = e & 63;
        ws[t * WP + o] = t < TV_TAPS ? Elem<DT>::load(wpk + ((size_t)t * n_pad + o) * cin_pad + (o >> 5)) : 0.f;
    }
    for (int e = threadIdx.x; e < PH * FE_PW; e += 256) {
        const int py = e / FE_PW, px = e - py * FE_PW;
        const int y = y0 + py - 2, x = x0 + px - 2;
        float a = 0.f, c = 0.f;
        if (y >= 0 && y < h && x >= 0 && x < w) {
            a = scale0 * (float)disp[ib + (size_t)y * w + x];
            c = (float)img[ib + (size_t)y * w + x] * (1.0f / 256.0f);
        }
        xs[0][e] = a;
        xs[1][e] = c;
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int g = lane >> 4, r16 = lane & 15;
    float a[2][2][NK];  // [branch][block][step]
    f32x4 bi[2][2];
    int off[NK];  // this lane's taps in the patch (any pixel for the zero weights)
#pragma unroll
    for (int k = 0; k < NK; ++k) {
        const int t = min(k * 4 + g, TV_TAPS - 1);
        off[k] = t / TV_K * FE_PW + t % TV_K;
    }
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int n = 0; n < 2; ++n) {
            const int o = 32 * c + 8 * (r16 / 4) + 4 * n + r16 % 4;
#pragma unroll
            for (int k = 0; k < NK; ++k) a[c][n][k] = ws[(k * 4 + g) * WP + o];
#pragma unroll
            for (int i = 0; i < 4; ++i) bi[c][n][i] = bias[32 * c + 8 * g + 4 * n + i];
        }
#pragma unroll
    for (int m = 0; m < TH / 4; ++m) {
        const int row = wave * (TH / 4) + m;
        const int y = y0 + row, x = x0 + r16;
        if (y >= h) break;
        f32x4 acc[2][2];
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int n = 0; n < 2; ++n) acc[c][n] = bi[c][n];
#pragma unroll
        for (int k = 0; k < NK; ++k)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const float xv = xs[c][row * FE_PW + r16 + off[k]];
#pragma unroll
                for (int n = 0; n < 2; ++n) acc[c][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[c][n][k], xv, acc[c][n], 0, 0, 0);
            }
        if (x >= w) continue;
        T *op = out + ((ib + (size_t)y * w + x) * L1C + 16 + 8 * g);
        constexpr int VN = 16 / sizeof(T);
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int i = 0; i < 8; i += VN) {
                V q;
#pragma unroll
                for (int k = 0; k < VN; ++k) {
                    const float r = acc[c][(i + k) / 4][(i + k) % 4];
                    q[k] = Elem<DT>::make(r > 0.f ? r : 0.1f * r);
                }
                *(V *)(op + 32 * c + i) = q;
            }
    }
}

template <int DT>
sv_status tv_fe_launch(const TvShape &s, const void *packed, const uint8_t *disp, const uint8_t *img, int B, int h,
                       int w, int f, void *L1, hipStream_t st) {
    using T = typename Elem<DT>::T;
    const float sc = (float)f / 256.0f;
    const float *bias = (const float *)((const char *)packed + s.b_off[T_FE]);
    const T *wp = (const T *)((const char *)packed + s.w_off[T_FE]);
    // 16 rows a workgroup spread the weights' staging and the halo; four where
    // that would leave CUs without one
    const bool tall = (long long)cdiv(w, FE_TW) * cdiv(h, 16) * B >= 512;
    const dim3 grid(cdiv(w, FE_TW), cdiv(h, tall ? 16 : 4), B);
    if (tall) hipLaunchKernelGGL((k_tv_fe<DT, 16>), grid, dim3(256), 0, st, disp, img, h, w, sc, wp, s.n_pad[T_FE], s.cin_pad[T_FE], bias, (T *)L1);
    else hipLaunchKernelGGL((k_tv_fe<DT, 4>), grid, dim3(256), 0, st, disp, img, h, w, sc, wp, s.n_pad[T_FE], s.cin_pad[T_FE], bias, (T *)L1);
    SV_LAUNCH_CHECK("k_tv_fe");
    return SV_OK;
}

sv_status tv_fe(const TvShape &s, const void *packed, const uint8_t *disp, const uint8_t *img, int B, int h, int w,
                int f, void *L1, int only, hipStream_t st) {
    if (only >= 0 && only != T_FE) return SV_OK;
    switch (s.dtype) {
    case SV_F32: return tv_fe_launch<SV_F32>(s, packed, disp, img, B, h, w, f, L1, st);
    case SV_BF16: return tv_fe_launch<SV_BF16>(s, packed, disp, img, B, h, w, f, L1, st);
    default: return tv_fe_launch<SV_F16>(s, packed, disp, img, B, h, w, f, L1, st);
    }
}

// One launched layer with configuration cfg[li]; with only >= 0 every other
// layer is skipped (the autotuner times one layer at a time).
sv_status tv_layer(const TvShape &s, const void *packed, int li, ConvSrc s0, ConvSrc s1, int B, int Hi,
                   int Wi, int Ho, int Wo, void *out, int out_pitch, int out_coff, int out_f32, int act,
                   float *part, size_t part_bytes, const int *cfg, int only, hipStream_t st) {
    if (only >= 0 && only != li) return SV_OK;
    ConvParams p{};
    p.part = part;
    p.part_bytes = part_bytes;
    p.src[0] = s0; p.src[1] = s1;
    p.B = B; p.Hi = Hi; p.Wi = Wi; p.Ho = Ho; p.Wo = Wo;
    p.Cin = s0.C + (s1.kind ? s1.C : 0);
    p.Cout = kLayers[li].cout;
    p.cin_pad = s.cin_pad[li];
    p.n_pad = s.n_pad[li];
    p.wpk = (const char *)packed + s.w_off[li];
    p.bias = (const float *)((const char *)packed + s.b_off[li]);
    p.out = out; p.out_pitch = out_pitch; p.out_coff = out_coff;
    p.act = act; p.out_f32 = out_f32;
    return launch_conv(s.dtype, kLayers[li].k, kLayers[li].stride, cfg[li], p, st);
}

// A stride-2 deconvolution (D_2 or D) by the form that is set; the polyphase
// one is four 3x3 correlations over its input, one per output parity class,
// each writing its pixels of the interleaved Ho x Wo output.
sv_status tv_deconv2(const TvShape &s, const void *packed, int li, ConvSrc src, int B, int Hi, int Wi, int Ho,
                     int Wo, void *out, int out_pitch, int out_coff, float *part, size_t part_bytes, const int *cfg,
                     int only, hipStream_t st) {
    if (only >= 0 && only != li) return SV_OK;
    int form = g_tv_deconv_form.load();
    // 16-bit maps of small grids, whose zero-inserted launch splits its reduction,
    // keep it: without the split the FP32 sums round otherwise, and the stored maps
    // with them (3e-5 of the refined map of one 228x218 image)
    if (form < 0 && s.dtype != SV_F32 &&
        conv_effective_split(s.dtype, conv_resolve_cfg(s.dtype, kLayers[li].k, 1, cfg[li]), src.C,
                             (long long)B * Ho * Wo, s.n_pad[li], part, part_bytes) > 1)
        form = 0;
    if (form < 0) {
        ConvParams p{};
        p.src[0] = src;
        p.B = B; p.Hi = 2 * Hi - 1; p.Wi = 2 * Wi - 1; p.Ho = Ho; p.Wo = Wo;
        p.Cin = src.C;
        p.Cout = kLayers[li].cout;
        p.cin_pad = s.cin_pad[li];
        p.n_pad = s.n_pad[li];
        p.wpk = (const char *)packed + s.w_off[li];
        p.bias = (const float *)((const char *)packed + s.b_off[li]);
        p.out = out; p.out_pitch = out_pitch; p.out_coff = out_coff;
        p.act = 1;
        if (tconv_fits(s.dtype, kLayers[li].k, p)) return launch_tconv(s.dtype, kLayers[li].k, p, st);
        form = 0;
    }
    if (form == 0) {
        src.kind = SRC_ZINS;
        return tv_layer(s, packed, li, src, ConvSrc{}, B, 2 * Hi - 1, 2 * Wi - 1, Ho, Wo, out, out_pitch, out_coff, 0,
                        1, part, part_bytes, cfg, only, st);
    }
    for (int ph = 0; ph < 4; ++ph) {
        const int py = ph >> 1, px = ph & 1;
        ConvParams p{};
        p.src[0] = src;
        p.B = B; p.Hi = Hi; p.Wi = Wi;
        p.Ho = (Ho - py + 1) / 2; p.Wo = (Wo - px + 1) / 2;
        if (p.Ho <= 0 || p.Wo <= 0) continue;
        p.ophase = 1 + ph; p.Ho_full = Ho; p.Wo_full = Wo;
        p.Cin = src.C;
        p.Cout = kLayers[li].cout;
        p.cin_pad = s.cin_pad[li];
        p.n_pad = s.n_pad[li];
        p.wpk = (const char *)packed + s.ph_off[li][ph];
        p.bias = (const float *)((const char *)packed + s.b_off[li]);
        p.out = out; p.out_pitch = out_pitch; p.out_coff = out_coff;
        p.act = 1;
        SV_TRY_STATUS(launch_conv(s.dtype, 3, 1, cfg[li] % conv_num_tiles(), p, st));
    }
    return SV_OK;
}

sv_status tv_forward(const TvShape &s, int f, const void *packed, const uint8_t *disp, const uint8_t *img,
                     int B, int H, int W, const float *eps, float *out, float *ml_user, void *ws,
                     hipStream_t st, int only = -1, const int *cfg_in = nullptr) {
    // cfg_in (nullable): this call's configurations (the autotuner's candidates)
    int cfg[T_NL];
    if (cfg_in) {
        for (int i = 0; i < T_NL; ++i) cfg[i] = cfg_in[i];
    } else {
        tv_layer_cfgs(s.dtype, f, B, H, W, cfg);
    }
    const TvLevels lv = tv_levels(f, H, W);
    const TvAct a = tv_act(s.es, lv, B);
    char *w = (char *)ws;
    void *L1 = w + a.L1, *L2 = w + a.L2, *L3 = w + a.L3, *Z = w + a.Z;
    // mu / sigma stay in the workspace (the backward reads them there); the
    // caller's buffer gets a copy
    float *ML = (float *)(w + a.ML);
    float *part = (float *)(w + a.part);
    const int h1 = lv.h[1], w1 = lv.w[1], h2 = lv.h[2], w2 = lv.w[2], h3 = lv.h[3], w3 = lv.w[3];
    const ConvSrc none{};
    // feature extraction: [FE_1 | FE_2] into level 1, channels 16..79
    SV_TRY_STATUS(tv_fe(s, packed, disp, img, B, h1, w1, f, L1, only, st));
    // encoder
    SV_TRY_STATUS(tv_layer(s, packed, T_EN1, tsrc(L1, 64, L1C, 16, h1, w1, SRC_TENSOR, 0), none, B, h1, w1, h2, w2,
                           L2, L2C, 16, 0, 1, part, a.part_bytes, cfg, only, st));
    SV_TRY_STATUS(tv_layer(s, packed, T_EN1R, tsrc(L2, 16, L2C, 16, h2, w2, SRC_TENSOR, 0), none, B, h2, w2, h2, w2,
                           L2, L2C, 32, 0, 1, part, a.part_bytes, cfg, only, st));
    SV_TRY_STATUS(tv_layer(s, packed, T_EN2, tsrc(L2, 24, L2C, 16, h2, w2, SRC_TENSOR, 0), none, B, h2, w2, h3, w3,
                           L3, L3C, 32, 0, 1, part, a.part_bytes, cfg, only, st));
    SV_TRY_STATUS(tv_layer(s, packed, T_EN2R, tsrc(L3, 32, L3C, 32, h3, w3, SRC_TENSOR, 0), none, B, h3, w3, h3, w3,
                           L3, L3C, 64, 0, 1, part, a.part_bytes, cfg, only, st));
    // mu & sigma (FP32), then Eq. (8)
    SV_TRY_STATUS(tv_layer(s, packed, T_MS, tsrc(L3, 48, L3C, 32, h3, w3, SRC_TENSOR, 0), none, B, h3, w3, h3, w3,
                           ML, 2, 0, 1, 0, part, a.part_bytes, cfg, only, st));
    const int nl = B * h3 * w3;
    if (ml_user && only < 0) {
        hipLaunchKernelGGL(k_tv_copy, dim3(cdiv(2 * nl, 256)), dim3(256), 0, st, ML, 2 * nl, ml_user);
        SV_LAUNCH_CHECK("k_tv_copy");
    }
    if (only < 0) switch (s.dtype) {
    case SV_F32: hipLaunchKernelGGL(k_tv_reparam<SV_F32>, dim3(cdiv(nl, 256)), dim3(256), 0, st, ML, eps, nl, (float *)Z); break;
    case SV_BF16: hipLaunchKernelGGL(k_tv_reparam<SV_BF16>, dim3(cdiv(nl, 256)), dim3(256), 0, st, ML, eps, nl, (uint16_t *)Z); break;
    default: hipLaunchKernelGGL(k_tv_reparam<SV_F16>, dim3(cdiv(nl, 256)), dim3(256), 0, st, ML, eps, nl, (uint16_t *)Z); break;
    }
    SV_LAUNCH_CHECK("k_tv_reparam");
    // decoder
    SV_TRY_STATUS(tv_layer(s, packed, T_D1, tsrc(Z, 1, ZC, 0, h3, w3, SRC_TENSOR, 0), none, B, h3, w3, h3, w3,
                           L3, L3C, 0, 0, 1, part, a.part_bytes, cfg, only, st));
    SV_TRY_STATUS(tv_layer(s, packed, T_D1R, tsrc(L3, 80, L3C, 0, h3, w3, SRC_TENSOR, 0), none, B, h3, w3, h3, w3,
                           L3, L3C, 80, 0, 1, part, a.part_bytes, cfg, only, st));
    // stride-2 deconvolutions
    SV_TRY_STATUS(tv_deconv2(s, packed, T_D2, tsrc(L3, 96, L3C, 0, h3, w3, SRC_TENSOR, 0), B, h3, w3, h2, w2,
                             L2, L2C, 0, part, a.part_bytes, cfg, only, st));
    SV_TRY_STATUS(tv_layer(s, packed, T_D2R, tsrc(L2, 40, L2C, 0, h2, w2, SRC_TENSOR, 0), none, B, h2, w2, h2, w2,
                           L2, L2C, 40, 0, 1, part, a.part_bytes, cfg, only, st));
    SV_TRY_STATUS(tv_deconv2(s, packed, T_D, tsrc(L2, 48, L2C, 0, h2, w2, SRC_TENSOR, 0), B, h2, w2, h1, w1,
                             L1, L1C, 0, part, a.part_bytes, cfg, only, st));
    if (only >= 0) return SV_OK;
    switch (s.dtype) {
    case SV_F32: return tv_final<SV_F32>(s, packed, L1, disp, img, B, h1, w1, f, H, W, out, st);
    case SV_BF16: return tv_final<SV_BF16>(s, packed, L1, disp, img, B, h1, w1, f, H, W, out, st);
    default: return tv_final<SV_F16>(s, packed, L1, disp, img, B, h1, w1, f, H, W, out, st);
    }
}

// ---- backward ----------------------------------------------------------------------
// Gradient maps (FP32 NHWC): one per level, channel ranges as in the forward
// maps; dZ [px3]; d(mu, sigma) [px3][8] (channels 2..7 zero, so that the 1x1
// input-gradient convolution reads whole channel groups); the tap gradients
// of the upsampling layer [px1][32] (taps 25..31 zero).
constexpr int DMLC = 8;
struct TvBwd { size_t dL1, dL2, dL3, dZ, dML, dT, part, sum, total; };

// The weight gradient of launched layer li: its shape and dtype (the caller
// fills in the sources and the gradient).  The two stride-2 deconvolutions
// exchange the roles of input and output gradient (see WgradJob): a quarter of
// the products of the zero-inserted form, whose other three quarters are zeros.
WgradJob tv_wgrad_job(int dtype, const TvLevels &lv, int B, int li) {
    static constexpr int kInLevel[T_NL] = {1, 1, 2, 2, 3, 3, 3, 3, 3, 2, 2, 1};
    const bool deconv = li == T_D2 || li == T_D;
    const int ki = deconv ? kOutLevel[li] : kInLevel[li], ko = deconv ? kInLevel[li] : kOutLevel[li];
    WgradJob j{};
    j.dtype = li == T_YP ? SV_F32 : dtype;
    j.ks = kLayers[li].k;
    j.stride = deconv ? 2 : kLayers[li].stride;
    j.B = B;
    j.Hi = lv.h[ki]; j.Wi = lv.w[ki];
    j.Ho = lv.h[ko]; j.Wo = lv.w[ko];
    j.Cout = deconv ? kLayers[li].cin : kLayers[li].cout;
    j.s0.C = deconv ? kLayers[li].cout : kLayers[li].cin;
    j.s0.kind = li == T_FE ? SRC_X0 : SRC_TENSOR;
    j.dy_sdt = SV_F32;
    j.bias_src = deconv;
    return j;
}

TvBwd tv_bwd_layout(const TvShape &s, const TvLevels &lv, int B) {
    auto px = [&](int k) { return (size_t)B * lv.h[k] * lv.w[k]; };
    TvBwd l{};
    size_t o = 0;
    auto take = [&](size_t floats) { size_t r = o; o = align256(o + floats * sizeof(float)); return r; };
    l.dL1 = take(px(1) * L1C);
    l.dL2 = take(px(2) * L2C);
    l.dL3 = take(px(3) * L3C);
    l.dZ = take(px(3));
    l.dML = take(px(3) * DMLC);
    l.dT = take(px(1) * TC);
    // weight-gradient partial sums of the largest layer (layers run one after another)
    size_t mx = 0;
    for (int i = 0; i < T_NL; ++i) mx = std::max(mx, wgrad_part_floats(tv_wgrad_job(s.dtype, lv, B, i)));
    l.part = take(mx);
    l.sum = take(256 + 1);
    l.total = o;
    return l;
}

// dT[b][i][j][t] = 256 * dout[b][f i + u - 2][f j + v - 2] (t = 5u + v; 0 where
// that pixel is outside the image, and for t >= 25): each tap of a coarse
// pixel lands on exactly one full-resolution pixel.
__global__ void k_tv_final_bwd(const float *__restrict__ dout, int B, int h, int w, int f, int H, int W,
                               float *__restrict__ dT) {
    const size_t n = (size_t)B * h * w * TC;
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < n; e += (size_t)gridDim.x * blockDim.x) {
        const int t = (int)(e % TC);
        const size_t pix = e / TC;
        const int j = (int)(pix % w), i = (int)((pix / w) % h), b = (int)(pix / ((size_t)w * h));
        float v = 0.f;
        if (t < TV_TAPS) {
            const int y = f * i + t / TV_K - 2, x = f * j + t % TV_K - 2;
            if (y >= 0 && y < H && x >= 0 && x < W) v = 256.0f * dout[((size_t)b * H + y) * W + x];
        }
        dT[e] = v;
    }
}

// sum of 256 * dout (Y's bias), two fixed-order passes
__global__ void __launch_bounds__(256) k_tv_sum_partial(const float *__restrict__ x, int64_t n, float *__restrict__ part) {
    __shared__ double sh[256];
    const int64_t per = (n + gridDim.x - 1) / gridDim.x;
    const int64_t lo = blockIdx.x * per, hi = lo + per < n ? lo + per : n;
    double acc = 0.0;
    for (int64_t i = lo + threadIdx.x; i < hi; i += 256) acc += (double)x[i];
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if ((int)threadIdx.x < k) sh[threadIdx.x] += sh[threadIdx.x + k];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = (float)sh[0];
}

__global__ void __launch_bounds__(256) k_tv_sum_final(const float *__restrict__ part, float scale, float *__restrict__ out) {
    __shared__ double sh[256];
    sh[threadIdx.x] = (double)part[threadIdx.x];
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if ((int)threadIdx.x < k) sh[threadIdx.x] += sh[threadIdx.x + k];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = (float)(scale * sh[0]);
}

// The upsampling layer's input gradient: dL1[pixel][c] = sum over the 25 taps of
// w[c][t] dT[pixel][t] for the 80 level-1 channels, D's (0..15) then through its
// leaky ReLU.  Bound by writing the gradient map (320 bytes a pixel): 16 pixels
// at a time on a wave, their taps (eight to a lane group) straight from memory
// into FP32 matrix steps, all 80 channels of a pixel from one read, the weights
// in registers for all of a wave's pixels.  4 maps of 256x128: 28 us, where the
// general kernel took 36 (three channel tiles, each staging the taps again).
template <int DT>
__global__ void __launch_bounds__(256)
k_tv_final_dgrad(const float *__restrict__ dT, const float *__restrict__ wpk, int cin_pad,
                 const typename Elem<DT>::T *__restrict__ L1, int64_t npix, float *__restrict__ dL1) {
    typedef typename Elem<DT>::T T4 __attribute__((ext_vector_type(4)));
    constexpr int NB = L1C / 16;
    const int lane = threadIdx.x & 63, g = lane >> 4, r16 = lane & 15;
    float a[NB][8];  // channel 16 n + r16, tap 8 g + i
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
        for (int i = 0; i < 8; ++i)
            a[n][i] = 8 * g + i < TV_TAPS ? wpk[(16 * n + r16) * cin_pad + 8 * g + i] : 0.f;
    const int64_t step = (int64_t)gridDim.x * 4 * 16;
    for (int64_t p0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 16; p0 < npix; p0 += step) {
        const int64_t px = p0 + r16, q = px < npix ? px : npix - 1;
        const f32x4 x0 = *(const f32x4 *)(dT + q * TC + 8 * g), x1 = *(const f32x4 *)(dT + q * TC + 8 * g + 4);
        const T4 act = *(const T4 *)(L1 + q * L1C + 4 * g);
        f32x4 c[NB];
#pragma unroll
        for (int n = 0; n < NB; ++n) c[n] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int n = 0; n < NB; ++n)
                c[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[n][i], i < 4 ? x0[i % 4] : x1[i % 4], c[n], 0, 0, 0);
        if (px >= npix) continue;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float v = Elem<DT>::load((const typename Elem<DT>::T *)&act + i);
            c[0][i] *= v > 0.f ? 1.0f : 0.1f;
        }
#pragma unroll
        for (int n = 0; n < NB; ++n) *(f32x4 *)(dL1 + px * L1C + 16 * n + 4 * g) = c[n];
    }
}

// Eq. (8) backward: d mu = dz (+ the loss's), d sigma = dz * eps * exp(sigma - 1) (+ the loss's)
__global__ void k_tv_reparam_bwd(const float *__restrict__ dz, const float *__restrict__ ml, const float *__restrict__ eps,
                                 const float *__restrict__ dms, int n, float *__restrict__ dml) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    float dm = dz[i], ds = eps ? dz[i] * eps[i] * expf(ml[2 * i + 1] - 1.0f) : 0.f;
    if (dms) { dm += dms[2 * i]; ds += dms[2 * i + 1]; }
    float *o = dml + (size_t)i * DMLC;
    o[0] = dm;
    o[1] = ds;
#pragma unroll
    for (int c = 2; c < DMLC; ++c) o[c] = 0.f;
}

ConvSrc fsrc(const float *p, int C, int pitch, int coff, int hs, int ws, int kind) {
    return tsrc(p, C, pitch, coff, hs, ws, kind, SDT_F32);
}

// Input gradient of launched layer li through the forward convolution kernel
// and the adjoint pack: `dy` is the output gradient as a source (plain, or
// zero-inserted for a stride-2 convolution); out / add give the target range.
// Channels mask_lo .. mask_hi - 1 of the range, complete with this term, are taken
// through the leaky ReLU of the stored map act (its range at the same offset): ten
// passes over the gradient maps less, 66 us of the 820 of a step of 4 512x256 in FP32.
sv_status tv_dgrad(const TvShape &s, const void *packed, int li, ConvSrc dy, int stride, int B, int Hi, int Wi,
                   int Ho, int Wo, float *out, int out_pitch, int out_coff, bool add, const void *act, int mask_lo, int mask_hi,
                   hipStream_t st) {
    ConvParams p{};
    p.src[0] = dy;
    p.B = B; p.Hi = Hi; p.Wi = Wi; p.Ho = Ho; p.Wo = Wo;
    p.Cin = dy.C;
    p.Cout = kAdjRows[li];
    p.cin_pad = s.bcin_pad[li];
    p.n_pad = s.bn_pad[li];
    p.wpk = (const char *)packed + s.bw_off[li];
    p.out = out; p.out_pitch = out_pitch; p.out_coff = out_coff; p.out_f32 = 1;
    if (add) { p.add = out; p.add_pitch = out_pitch; p.add_coff = out_coff; }
    p.mask = mask_hi ? (const char *)act + (size_t)out_coff * s.es : nullptr;
    p.mask_pitch = out_pitch; p.mask_lo = mask_lo; p.mask_hi = mask_hi;
    if (dy.kind == SRC_ZINS && tconv_fits(s.dtype, kLayers[li].k, p)) return launch_tconv(s.dtype, kLayers[li].k, p, st);
    const int cfg = p.Cout <= 16 ? T4_16 : T4_32;
    return launch_conv(s.dtype, kLayers[li].k, stride, cfg, p, st);
}

sv_status tv_backward(const TvShape &s, int f, const void *packed, const uint8_t *disp, const uint8_t *img, int B,
                      int H, int W, const float *eps, const void *fws, const float *dout, const float *dms,
                      float *grad, void *ws, hipStream_t st) {
    const TvLevels lv = tv_levels(f, H, W);
    const TvAct a = tv_act(s.es, lv, B);
    const TvBwd l = tv_bwd_layout(s, lv, B);
    const char *fw = (const char *)fws;
    const void *L1 = fw + a.L1, *L2 = fw + a.L2, *L3 = fw + a.L3, *Z = fw + a.Z;
    const float *ML = (const float *)(fw + a.ML);
    char *bw = (char *)ws;
    float *dL1 = (float *)(bw + l.dL1), *dL2 = (float *)(bw + l.dL2), *dL3 = (float *)(bw + l.dL3);
    float *dZ = (float *)(bw + l.dZ), *dML = (float *)(bw + l.dML), *dT = (float *)(bw + l.dT);
    float *part = (float *)(bw + l.part), *sum = (float *)(bw + l.sum);
    const int h1 = lv.h[1], w1 = lv.w[1], h2 = lv.h[2], w2 = lv.w[2], h3 = lv.h[3], w3 = lv.w[3];
    const size_t p1 = (size_t)B * h1 * w1, p3 = (size_t)B * h3 * w3;
    const int sdt = s.dtype == SV_F32 ? 0 : 1 + s.dtype;  // the maps' storage, seen from an FP32 launch
    const ConvSrc none{};
    ConvSrc x0{};
    x0.ptr = disp; x0.img = img; x0.kind = SRC_X0; x0.C = 2; x0.hs = h1; x0.ws = w1;
    x0.scale0 = (float)f / 256.0f;
    auto blocks = [](size_t n) { return (unsigned)std::min<size_t>((n + 255) / 256, 4096); };

    // weight and bias gradient of launched layer li into its canonical slice
    auto wgrad = [&](int li, int canon, ConvSrc s0, ConvSrc s1, const void *dy, int dy_pitch) -> sv_status {
        WgradJob j = tv_wgrad_job(s.dtype, lv, B, li);
        j.s0 = s0; j.s1 = s1;
        j.dy = dy; j.dy_pitch = dy_pitch;
        const CanonLayer &c = kCanon[canon];
        GradMap m{};
        m.kind = j.bias_src ? GM_SWAP : (li == T_YP ? GM_Y : (li == T_FE ? GM_FE : GM_OIHW));
        m.cin = c.cin;
        m.kk = c.k * c.k;
        m.nbias = li == T_YP ? 0 : c.cout;
        if (j.bias_src) j.dy_sdt = s.dtype;  // the deconvolution's input, as it is stored
        if (li == T_FE) {
            m.nbias = kLayers[T_FE].cout;
            m.off1 = m.off2 = (int)(canon_off(C_FE2) - canon_off(C_FE1));
        }
        float *gw = grad + canon_off(canon);
        return launch_wgrad(j, m, part, gw, gw + (size_t)c.cout * c.cin * c.k * c.k, st);
    };
    // upsampling layer: tap gradients, Y's bias, its projection's weights and input gradient
    hipLaunchKernelGGL(k_tv_final_bwd, dim3(blocks(p1 * TC)), dim3(256), 0, st, dout, B, h1, w1, f, H, W, dT);
    SV_LAUNCH_CHECK("k_tv_final_bwd");
    hipLaunchKernelGGL(k_tv_sum_partial, dim3(256), dim3(256), 0, st, dout, (int64_t)B * H * W, sum);
    hipLaunchKernelGGL(k_tv_sum_final, dim3(1), dim3(256), 0, st, sum, 256.0f, grad + canon_off(C_Y) + 81 * 25);
    SV_LAUNCH_CHECK("k_tv_sum");
    SV_TRY_STATUS(wgrad(T_YP, C_Y, tsrc(L1, 80, L1C, 0, h1, w1, SRC_TENSOR, sdt), x0, dT, TC));
    {
        const float *wy = (const float *)((const char *)packed + s.bw_off[T_YP]);
        auto run = [&](auto *fn, auto *act) {
            const long long n = resident_grid((const void *)fn, 0, (long long)((p1 + 63) / 64));
            hipLaunchKernelGGL(fn, dim3((unsigned)n), dim3(256), 0, st, dT, wy, s.bcin_pad[T_YP], act, (int64_t)p1, dL1);
        };
        switch (s.dtype) {
        case SV_F32: run(k_tv_final_dgrad<SV_F32>, (const float *)L1); break;
        case SV_BF16: run(k_tv_final_dgrad<SV_BF16>, (const uint16_t *)L1); break;
        default: run(k_tv_final_dgrad<SV_F16>, (const uint16_t *)L1); break;
        }
        SV_LAUNCH_CHECK("k_tv_final_dgrad");
    }
    // D (deconvolution into level 1)
    SV_TRY_STATUS(wgrad(T_D, C_D, fsrc(dL1, 16, L1C, 0, h1, w1, SRC_TENSOR), none, L2, L2C));
    SV_TRY_STATUS(tv_dgrad(s, packed, T_D, fsrc(dL1, 16, L1C, 0, h1, w1, SRC_TENSOR), 2, B, h1, w1, h2, w2,
                           dL2, L2C, 0, false, L2, 40, 48, st));
    // D_2_R
    SV_TRY_STATUS(wgrad(T_D2R, C_D2R, tsrc(L2, 40, L2C, 0, h2, w2, SRC_TENSOR, 0), none, dL2 + 40, L2C));
    SV_TRY_STATUS(tv_dgrad(s, packed, T_D2R, fsrc(dL2, 8, L2C, 40, h2, w2, SRC_TENSOR), 1, B, h2, w2, h2, w2,
                           dL2, L2C, 0, true, L2, 0, 16, st));
    // D_2 (deconvolution into level 2)
    SV_TRY_STATUS(wgrad(T_D2, C_D2, fsrc(dL2, 16, L2C, 0, h2, w2, SRC_TENSOR), none, L3, L3C));
    SV_TRY_STATUS(tv_dgrad(s, packed, T_D2, fsrc(dL2, 16, L2C, 0, h2, w2, SRC_TENSOR), 2, B, h2, w2, h3, w3,
                           dL3, L3C, 0, false, L3, 80, 96, st));
    // D_1_R
    SV_TRY_STATUS(wgrad(T_D1R, C_D1R, tsrc(L3, 80, L3C, 0, h3, w3, SRC_TENSOR, 0), none, dL3 + 80, L3C));
    SV_TRY_STATUS(tv_dgrad(s, packed, T_D1R, fsrc(dL3, 16, L3C, 80, h3, w3, SRC_TENSOR), 1, B, h3, w3, h3, w3,
                           dL3, L3C, 0, true, L3, 0, 32, st));
    // D_1 (1x1 deconvolution of z)
    SV_TRY_STATUS(wgrad(T_D1, C_D1, tsrc(Z, 1, ZC, 0, h3, w3, SRC_TENSOR, 0), none, dL3, L3C));
    SV_TRY_STATUS(tv_dgrad(s, packed, T_D1, fsrc(dL3, 32, L3C, 0, h3, w3, SRC_TENSOR), 1, B, h3, w3, h3, w3,
                           dZ, 1, 0, false, nullptr, 0, 0, st));
    // Eq. (8), then the head
    hipLaunchKernelGGL(k_tv_reparam_bwd, dim3(cdiv((int)p3, 256)), dim3(256), 0, st, dZ, ML, eps, dms, (int)p3, dML);
    SV_LAUNCH_CHECK("k_tv_reparam_bwd");
    SV_TRY_STATUS(wgrad(T_MS, C_MS, tsrc(L3, 48, L3C, 32, h3, w3, SRC_TENSOR, 0), none, dML, DMLC));
    SV_TRY_STATUS(tv_dgrad(s, packed, T_MS, fsrc(dML, 2, DMLC, 0, h3, w3, SRC_TENSOR), 1, B, h3, w3, h3, w3,
                           dL3, L3C, 32, true, L3, 32, 48, st));
    // EN_2_R
    SV_TRY_STATUS(wgrad(T_EN2R, C_EN2R, tsrc(L3, 32, L3C, 32, h3, w3, SRC_TENSOR, 0), none, dL3 + 64, L3C));
    SV_TRY_STATUS(tv_dgrad(s, packed, T_EN2R, fsrc(dL3, 16, L3C, 64, h3, w3, SRC_TENSOR), 1, B, h3, w3, h3, w3,
                           dL3, L3C, 32, true, L3, 0, 32, st));
    // EN_2 (stride 2: its input gradient is a transposed convolution)
    SV_TRY_STATUS(wgrad(T_EN2, C_EN2, tsrc(L2, 24, L2C, 16, h2, w2, SRC_TENSOR, 0), none, dL3 + 32, L3C));
    SV_TRY_STATUS(tv_dgrad(s, packed, T_EN2, fsrc(dL3, 32, L3C, 32, h3, w3, SRC_ZINS), 1, B, 2 * h3 - 1, 2 * w3 - 1,
                           h2, w2, dL2, L2C, 16, true, L2, 16, 24, st));
    // EN_1_R
    SV_TRY_STATUS(wgrad(T_EN1R, C_EN1R, tsrc(L2, 16, L2C, 16, h2, w2, SRC_TENSOR, 0), none, dL2 + 32, L2C));
    SV_TRY_STATUS(tv_dgrad(s, packed, T_EN1R, fsrc(dL2, 8, L2C, 32, h2, w2, SRC_TENSOR), 1, B, h2, w2, h2, w2,
                           dL2, L2C, 16, true, L2, 0, 16, st));
    // EN_1
    SV_TRY_STATUS(wgrad(T_EN1, C_EN1, tsrc(L1, 64, L1C, 16, h1, w1, SRC_TENSOR, 0), none, dL2 + 16, L2C));
    SV_TRY_STATUS(tv_dgrad(s, packed, T_EN1, fsrc(dL2, 16, L2C, 16, h2, w2, SRC_ZINS), 1, B, 2 * h2 - 1, 2 * w2 - 1,
                           h1, w1, dL1, L1C, 16, true, L1, 0, 64, st));
    // FE_1 (rows 0..31, input channel 0) and FE_2 (rows 32..63, channel 1)
    SV_TRY_STATUS(wgrad(T_FE, C_FE1, x0, none, dL1 + 16, L1C));
    return SV_OK;
}

// ---- loss (Eqs. (9)-(11)) -----------------------------------------------------------
constexpr int TL_BLOCKS = 256, TL_THREADS = 256;

__device__ __forceinline__ double tl_block_sum(double v, double *sh) {
    const int t = threadIdx.x;
    sh[t] = v;
    __syncthreads();
    for (int k = TL_THREADS / 2; k > 0; k >>= 1) {
        if (t < k) sh[t] += sh[t + k];
        __syncthreads();
    }
    const double r = sh[0];
    __syncthreads();
    return r;
}

// per block: sum |out - gt| (noc + occ), the occ count and the KL sum
__global__ void __launch_bounds__(TL_THREADS)
k_tv_loss_partial(const float *__restrict__ out, const float *__restrict__ gt, const uint8_t *__restrict__ noc,
                  const uint8_t *__restrict__ occ, int64_t n, const float *__restrict__ ml, int64_t nl,
                  double *__restrict__ part) {
    __shared__ double sh[TL_THREADS];
    const int64_t per = (n + gridDim.x - 1) / gridDim.x;
    const int64_t lo = blockIdx.x * per, hi = lo + per < n ? lo + per : n;
    double s = 0.0, cnt = 0.0;
    for (int64_t i = lo + threadIdx.x; i < hi; i += TL_THREADS) {
        const double a = fabs((double)out[i] - (double)gt[i]);
        const int m = (noc[i] ? 1 : 0) + (occ[i] ? 1 : 0);
        s += a * m;
        cnt += occ[i] ? 1.0 : 0.0;
    }
    const int64_t perl = (nl + gridDim.x - 1) / gridDim.x;
    const int64_t llo = blockIdx.x * perl, lhi = llo + perl < nl ? llo + perl : nl;
    double k = 0.0;
    for (int64_t i = llo + threadIdx.x; i < lhi; i += TL_THREADS) {
        const double m = (double)ml[2 * i] - 1.0, sg = (double)ml[2 * i + 1] - 1.0;
        k += 0.5 * (m * m - 1.0 + exp(2.0 * sg) - 2.0 * sg);
    }
    s = tl_block_sum(s, sh);
    cnt = tl_block_sum(cnt, sh);
    k = tl_block_sum(k, sh);
    if (threadIdx.x == 0) {
        part[3 * blockIdx.x] = s;
        part[3 * blockIdx.x + 1] = cnt;
        part[3 * blockIdx.x + 2] = k;
    }
}

// loss_out = [total, 256 * Loss_1, 256 * Loss_2]; part[3 * TL_BLOCKS] keeps the
// ground-truth count for the gradient kernel
__global__ void __launch_bounds__(TL_THREADS)
k_tv_loss_final(double *__restrict__ part, int64_t nl, float *__restrict__ loss_out) {
    __shared__ double sh[TL_THREADS];
    double s = 0.0, c = 0.0, k = 0.0;
    for (int i = threadIdx.x; i < TL_BLOCKS; i += TL_THREADS) {
        s += part[3 * i];
        c += part[3 * i + 1];
        k += part[3 * i + 2];
    }
    s = tl_block_sum(s, sh);
    c = tl_block_sum(c, sh);
    k = tl_block_sum(k, sh);
    if (threadIdx.x == 0) {
        const double nn = c > 1.0 ? c : 1.0;
        const double l1 = s / nn, l2 = nl > 0 ? 256.0 * k / (double)nl : 0.0;
        loss_out[0] = (float)(l1 + l2);
        loss_out[1] = (float)l1;
        loss_out[2] = (float)l2;
        part[3 * TL_BLOCKS] = nn;
    }
}

__global__ void k_tv_loss_grad(const float *__restrict__ out, const float *__restrict__ gt,
                               const uint8_t *__restrict__ noc, const uint8_t *__restrict__ occ, int64_t n,
                               const float *__restrict__ ml, int64_t nl, const double *__restrict__ part,
                               float *__restrict__ dout, float *__restrict__ dml) {
    const double inv = 1.0 / part[3 * TL_BLOCKS];
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        if (!dout) break;
        const float e = out[i] - gt[i];
        const int sg = (e > 0.f) - (e < 0.f);
        const int m = (noc[i] ? 1 : 0) + (occ[i] ? 1 : 0);
        dout[i] = (float)((double)(sg * m) * inv);
    }
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < nl; i += (int64_t)gridDim.x * blockDim.x) {
        if (!dml) break;
        const double m = (double)ml[2 * i] - 1.0, sgm = (double)ml[2 * i + 1] - 1.0;
        dml[2 * i] = (float)(256.0 * m / (double)nl);
        dml[2 * i + 1] = (float)(256.0 * (exp(2.0 * sgm) - 1.0) / (double)nl);
    }
}

}  // namespace

}  // namespace sv

using namespace sv;

extern "C" {

int64_t sv_tvae_param_count(void) { return canon_off(NCANON); }

size_t sv_tvae_packed_bytes(int dtype) {
    if (dtype != SV_F32 && dtype != SV_BF16 && dtype != SV_F16) return 0;
    return tv_shape(dtype).bytes;
}

sv_status sv_tvae_pack_weights(int dtype, const float *params, void *packed_out, void *stream) {
    if (!params || !packed_out) return SV_ERR_NULL;
    if (dtype != SV_F32 && dtype != SV_BF16 && dtype != SV_F16) return SV_ERR_DTYPE;
    if ((uintptr_t)packed_out % 256) return SV_ERR_RANGE;
    return tv_pack(tv_shape(dtype), params, packed_out, (hipStream_t)stream);
}

static bool tv_shape_ok(int factor, int B, int H, int W) {
    if (factor < 1 || factor > 8 || B < 1 || H < 1 || W < 1) return false;
    if ((int64_t)B * H * W >= ((int64_t)1 << 31)) return false;
    // one workgroup row per 4 images in z for the widest layer
    return (int64_t)B * 4 <= 65535;
}

size_t sv_tvae_workspace_bytes(int dtype, int factor, int B, int H, int W) {
    if (dtype != SV_F32 && dtype != SV_BF16 && dtype != SV_F16) return 0;
    if (!tv_shape_ok(factor, B, H, W)) return 0;
    return tv_act(dtype_bytes(dtype), tv_levels(factor, H, W), B).total;
}

sv_status sv_tvae_forward(int dtype, int factor, const void *packed_w, const uint8_t *disp_low,
                          const uint8_t *img_low, int B, int H, int W, const float *eps, float *out,
                          float *mu_sigma, void *workspace, size_t ws_bytes, void *stream) {
    if (!packed_w || !disp_low || !img_low || !out || !workspace) return SV_ERR_NULL;
    if (dtype != SV_F32 && dtype != SV_BF16 && dtype != SV_F16) return SV_ERR_DTYPE;
    if (factor < 1 || factor > 8) return SV_ERR_RANGE;
    if (!tv_shape_ok(factor, B, H, W)) return SV_ERR_SHAPE;
    if (ws_bytes < sv_tvae_workspace_bytes(dtype, factor, B, H, W)) return SV_ERR_WORKSPACE;
    if ((uintptr_t)workspace % 256 || (uintptr_t)packed_w % 256) return SV_ERR_RANGE;
    return tv_forward(tv_shape(dtype), factor, packed_w, disp_low, img_low, B, H, W, eps, out, mu_sigma,
                      workspace, (hipStream_t)stream);
}

size_t sv_tvae_loss_workspace_bytes(void) { return sizeof(double) * (3 * TL_BLOCKS + 1); }

sv_status sv_tvae_loss(const float *out, const float *gt, const uint8_t *noc, const uint8_t *occ, int64_t n,
                       const float *mu_sigma, int64_t n_lat, float *loss_out, float *dout, float *dmu_sigma,
                       void *workspace, size_t ws_bytes, void *stream) {
    if (!out || !gt || !noc || !occ || !mu_sigma || !loss_out || !workspace) return SV_ERR_NULL;
    if (n <= 0 || n_lat <= 0) return SV_ERR_SHAPE;
    if (ws_bytes < sv_tvae_loss_workspace_bytes()) return SV_ERR_WORKSPACE;
    if ((uintptr_t)workspace % 8) return SV_ERR_RANGE;
    hipStream_t st = (hipStream_t)stream;
    double *part = (double *)workspace;
    hipLaunchKernelGGL(k_tv_loss_partial, dim3(TL_BLOCKS), dim3(TL_THREADS), 0, st, out, gt, noc, occ, n, mu_sigma,
                       n_lat, part);
    SV_LAUNCH_CHECK("k_tv_loss_partial");
    hipLaunchKernelGGL(k_tv_loss_final, dim3(1), dim3(TL_THREADS), 0, st, part, n_lat, loss_out);
    SV_LAUNCH_CHECK("k_tv_loss_final");
    if (dout || dmu_sigma) {
        const int64_t m = n > n_lat ? n : n_lat;
        const int blocks = (int)std::min<int64_t>((m + 255) / 256, 4096);
        hipLaunchKernelGGL(k_tv_loss_grad, dim3(blocks), dim3(256), 0, st, out, gt, noc, occ, n, mu_sigma, n_lat,
                           (const double *)part, dout, dmu_sigma);
        SV_LAUNCH_CHECK("k_tv_loss_grad");
    }
    return SV_OK;
}

sv_status sv_tvae_set_layer_cfg(int layer, int cfg) {
    if (layer < 0 || layer >= T_NL) return SV_ERR_RANGE;
    if (cfg < -1 || cfg >= conv_num_cfgs()) return SV_ERR_RANGE;
    g_tv_cfg[layer].store(cfg);
    return SV_OK;
}

int sv_tvae_num_layers(void) { return T_NL; }

sv_status sv_tvae_set_deconv_form(int form) {
    if (form < -1 || form > 1) return SV_ERR_RANGE;
    g_tv_deconv_form.store(form);
    return SV_OK;
}

size_t sv_tvae_backward_workspace_bytes(int dtype, int factor, int B, int H, int W) {
    if (dtype != SV_F32 && dtype != SV_BF16 && dtype != SV_F16) return 0;
    if (!tv_shape_ok(factor, B, H, W)) return 0;
    return tv_bwd_layout(tv_shape(dtype), tv_levels(factor, H, W), B).total;
}

sv_status sv_tvae_backward(int dtype, int factor, const void *packed_w, const uint8_t *disp_low,
                           const uint8_t *img_low, int B, int H, int W, const float *eps,
                           const void *fwd_workspace, const float *dout, const float *dmu_sigma, float *grad_out,
                           void *workspace, size_t ws_bytes, void *stream) {
    if (!packed_w || !disp_low || !img_low || !fwd_workspace || !dout || !grad_out || !workspace) return SV_ERR_NULL;
    if (dtype != SV_F32 && dtype != SV_BF16 && dtype != SV_F16) return SV_ERR_DTYPE;
    if (factor < 1 || factor > 8) return SV_ERR_RANGE;
    if (!tv_shape_ok(factor, B, H, W)) return SV_ERR_SHAPE;
    if (ws_bytes < sv_tvae_backward_workspace_bytes(dtype, factor, B, H, W)) return SV_ERR_WORKSPACE;
    if ((uintptr_t)workspace % 256 || (uintptr_t)fwd_workspace % 256 || (uintptr_t)packed_w % 256) return SV_ERR_RANGE;
    return tv_backward(tv_shape(dtype), factor, packed_w, disp_low, img_low, B, H, W, eps, fwd_workspace, dout,
                       dmu_sigma, grad_out, workspace, (hipStream_t)stream);
}

sv_status sv_tvae_autotune(int dtype, int factor, int B, int H, int W) {
    if (dtype != SV_F32 && dtype != SV_BF16 && dtype != SV_F16) return SV_ERR_DTYPE;
    if (factor < 1 || factor > 8) return SV_ERR_RANGE;
    if (!tv_shape_ok(factor, B, H, W)) return SV_ERR_SHAPE;
    const TvShape s = tv_shape(dtype);
    const TvLevels lv = tv_levels(factor, H, W);
    const size_t ws = sv_tvae_workspace_bytes(dtype, factor, B, H, W);
    const size_t nlow = (size_t)B * lv.h[1] * lv.w[1];
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = align256(off + bytes); return o; };
    const size_t o_pk = take(s.bytes), o_par = take((size_t)canon_off(NCANON) * 4), o_ws = take(ws);
    const size_t o_in = take(2 * nlow), o_out = take((size_t)B * H * W * 4);
    void *mem = nullptr;
    SV_HIP(hipMalloc(&mem, off));
    char *d = (char *)mem;
    hipStream_t st = nullptr;
    // zero parameters and inputs: timing does not depend on the values
    hipLaunchKernelGGL(k_zero_bytes, dim3(4096), dim3(256), 0, st, (uint32_t *)d, off / 4);
    sv_status r = tv_pack(s, (const float *)(d + o_par), d + o_pk, st);
    const uint8_t *disp = (const uint8_t *)(d + o_in), *img = disp + nlow;
    // the configurations under test travel with each call (cur): tuning
    // changes no process-wide setting, so other threads' calls are unaffected
    int cur[T_NL], base[T_NL], best[T_NL];
    auto run = [&](int only) {
        return tv_forward(s, factor, d + o_pk, disp, img, B, H, W, nullptr, (float *)(d + o_out), nullptr,
                          d + o_ws, st, only, cur);
    };
    auto timed = [&](int only, int reps) {
        hipEvent_t a, b;
        float t = 1e30f;
        if (hipEventCreate(&a) != hipSuccess) return t;
        if (hipEventCreate(&b) != hipSuccess) { (void)hipEventDestroy(a); return t; }
        for (int i = 0; i < 2 && r == SV_OK; ++i) r = run(only);
        (void)hipEventRecord(a, st);
        for (int i = 0; i < reps && r == SV_OK; ++i) r = run(only);
        (void)hipEventRecord(b, st);
        (void)hipEventSynchronize(b);
        (void)hipEventElapsedTime(&t, a, b);
        (void)hipEventDestroy(a);
        (void)hipEventDestroy(b);
        return t / reps;
    };
    for (int i = 0; i < T_NL; ++i) {
        const int k = kOutLevel[i];
        base[i] = tv_heuristic_cfg(i, B, lv.h[k], lv.w[k]);
        best[i] = cur[i] = base[i];
    }
    const int reps = B >= 16 ? 4 : 12;
    for (int li = 0; li < T_NL && r == SV_OK; ++li) {
        // kernels of their own, no tile configuration; the default form's deconvolutions
        // but for 16-bit ones that run split over the zero-inserted input (see
        // tv_deconv2), which keep their split: without it they would be another kernel
        // and other bits
        const bool deconv = (li == T_D2 || li == T_D) && g_tv_deconv_form.load() < 0;
        const int keep = deconv ? base[li] / conv_num_tiles() + 1 : 0;
        if (li == T_FE || li == T_YP || (deconv && (dtype == SV_F32 || keep == 1))) continue;
        const int k = kOutLevel[li];
        const long long npix = (long long)B * lv.h[k] * lv.w[k];
        float bt = 1e30f;
        best[li] = base[li];
        for (int c = 0; c < conv_num_cfgs() && r == SV_OK; ++c) {
            if (conv_resolve_cfg(dtype, kLayers[li].k, kLayers[li].stride, c) != c) continue;
            // a split the launch would not take duplicates a smaller one
            const int want = c / conv_num_tiles() + 1;
            static float dummy;
            const TvAct a = tv_act(s.es, lv, B);
            if (conv_effective_split(dtype, c, kLayers[li].cin, npix, s.n_pad[li], &dummy, a.part_bytes) != want) continue;
            if (keep && want != keep) continue;
            cur[li] = c;
            const float t = timed(li, reps);
            if (t < bt) { bt = t; best[li] = c; }
        }
        cur[li] = base[li];
    }
    if (r == SV_OK) {
        // keep the tuned set only if the whole pass is faster than the defaults
        const float t0 = timed(-1, reps);
        for (int i = 0; i < T_NL; ++i) cur[i] = best[i];
        const float t1 = timed(-1, reps);
        std::lock_guard<std::mutex> g(g_tv_mu);
        if (t1 < t0) {
            std::array<int, T_NL> a;
            for (int i = 0; i < T_NL; ++i) a[i] = best[i];
            g_tv_tuned[std::make_tuple(dtype, factor, B, H, W)] = a;
        } else {
            g_tv_tuned.erase(std::make_tuple(dtype, factor, B, H, W));
        }
    }
    const hipError_t e = hipFree(mem);
    if (r == SV_OK && e != hipSuccess) r = hip_fail(e, "hipFree");
    return r;
}

sv_status sv_tvae_layer_cfgs(int dtype, int factor, int B, int H, int W, int *cfg_out) {
    if (!cfg_out) return SV_ERR_NULL;
    if (dtype != SV_F32 && dtype != SV_BF16 && dtype != SV_F16) return SV_ERR_DTYPE;
    if (factor < 1 || factor > 8) return SV_ERR_RANGE;
    if (!tv_shape_ok(factor, B, H, W)) return SV_ERR_SHAPE;
    tv_layer_cfgs(dtype, factor, B, H, W, cfg_out);
    return SV_OK;
}

}  // extern "C"
