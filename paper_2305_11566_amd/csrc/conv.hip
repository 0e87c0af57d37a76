// Convolutions of the refinement network (Table I) as implicit GEMM on MFMA.
//
// GEMM view: rows = output channels n, columns = output pixels m, reduction
// over k = (tap, input channel).  The MFMA A operand is a 16 x k slice of the
// weights and B a k x 16 slice of the input, so each lane of the 16x16
// result holds four consecutive output channels of one pixel, which the
// epilogue stores as one NHWC vector.
//
// A workgroup (4 waves) owns an output tile of TH rows x 16 columns of one
// image and TN output channels.  For each chunk of KC input channels it
// stages into LDS
//   * the input patch (tile plus halo), gathered from up to two sources:
//     a same-level NHWC map, a map bilinearly resized on the fly from a
//     coarser level (the decoder's upsampling), or the network input x0 built
//     from the uint8 coarse disparity and reduced left image; out-of-image
//     pixels and channels past Cin are zeros (the zero padding);
//   * the chunk of packed weights for all taps and the tile's TN channels.
// The reduction then runs over (tap, channel group) pairs straight out of
// LDS: lane group g (lanes 16g..16g+15) takes pair 4*step + g, so a step
// covers four pairs whatever the tap count, and Cin = 2 (the first layer)
// wastes little.  Accumulation is FP32 for every storage type.  The order of
// the reduction is fixed by the base chunk and the step, not by the tile
// shape, so every tile shape gives bitwise-identical results.  The kernel
// templates live in conv_impl.h and are instantiated per compute dtype in
// conv_f32.hip / conv_bf16.hip / conv_f16.hip / conv_i8.hip; this file holds the
// tile table, the dispatch and the INT8 weight packing (pack.hip the others').
#include <algorithm>
#include <cstdio>
#include <mutex>

#include "conv_impl.h"

namespace sv {

// ---- tile configurations ---------------------------------------------------------
// A configuration id is a tile shape plus a reduction split:
// id = tile + kNumTiles * (ksplit - 1), ksplit = 1 .. kMaxSplit.  A split only
// applies to uniform launches that bring a partial-sum buffer.
struct CfgDesc { int TH, TN, WM, KCM; const char *name; };
static constexpr CfgDesc kCfgs[] = {
#define SV_CFG(i, TH, TN, WM, KCM, name) {TH, TN, WM, KCM, name},
    SV_CONV_CFGS(SV_CFG)
#undef SV_CFG
};
static constexpr int kNumTiles = (int)(sizeof(kCfgs) / sizeof(kCfgs[0]));
static constexpr int kMaxSplit = CONV_MAX_SPLIT;
static constexpr bool is_tile(int t, int th, int tn, int kcm) {
    return kCfgs[t].TH == th && kCfgs[t].TN == tn && kCfgs[t].KCM == kcm;
}
static_assert(is_tile(T4_64, 4, 64, 1) && is_tile(T8_64, 8, 64, 1) && is_tile(T4_32, 4, 32, 1) &&
                  is_tile(T8_32, 8, 32, 1) && is_tile(T2_64, 2, 64, 1) && is_tile(T4_16, 4, 16, 1) &&
                  is_tile(T4_16_K4, 4, 16, 4) && is_tile(T4_32_K2, 4, 32, 2) && is_tile(T4_16_K2, 4, 16, 2) &&
                  is_tile(T2_32_K2, 2, 32, 2) && is_tile(T16_32, 16, 32, 1),
              "ConvTileId names the table's rows");
static constexpr int kFallbackTile = T4_16;
int conv_num_tiles() { return kNumTiles; }
int conv_num_cfgs() { return kNumTiles * kMaxSplit; }

const char *conv_cfg_name(int cfg) {
    static char names[kNumTiles * kMaxSplit][32];
    static std::once_flag once;
    std::call_once(once, [] {
        for (int i = 0; i < kNumTiles * kMaxSplit; ++i) {
            const int t = i % kNumTiles, sp = i / kNumTiles + 1;
            if (sp == 1) snprintf(names[i], sizeof names[i], "%s", kCfgs[t].name);
            else snprintf(names[i], sizeof names[i], "%s_s%d", kCfgs[t].name, sp);
        }
    });
    return (cfg >= 0 && cfg < conv_num_cfgs()) ? names[cfg] : "?";
}

sv_status launch_conv_f32(int ks, int stride, int cfg, const ConvParams &p, int pg, hipStream_t st);
sv_status launch_split_sum_f32(const ConvParams &p, hipStream_t st);
sv_status launch_split_sum_bf16(const ConvParams &p, hipStream_t st);
sv_status launch_split_sum_f16(const ConvParams &p, hipStream_t st);
sv_status launch_conv_bf16(int ks, int stride, int cfg, const ConvParams &p, int pg, hipStream_t st);
sv_status launch_conv_f16(int ks, int stride, int cfg, const ConvParams &p, int pg, hipStream_t st);
bool conv_fits_f32(int ks, int stride, int tile);
bool conv_fits_bf16(int ks, int stride, int tile);
bool conv_fits_f16(int ks, int stride, int tile);
sv_status launch_conv_i8(int ks, int stride, int cfg, const ConvParams &p, int pg, hipStream_t st);
bool conv_fits_i8(int ks, int stride, int tile);
#define SV_CONV5_DECL(S, dt)                                                                      \
    sv_status launch_conv5_s##S##_##dt(int cfg, const ConvParams &p, int pg, hipStream_t st); \
    bool conv5_fits_s##S##_##dt(int tile);
SV_CONV5_DECL(1, f32) SV_CONV5_DECL(2, f32) SV_CONV5_DECL(1, bf16) SV_CONV5_DECL(2, bf16)
SV_CONV5_DECL(1, f16) SV_CONV5_DECL(2, f16)
#undef SV_CONV5_DECL

static bool fits_any(int dtype, int ks, int stride, int tile) {
    if (ks == 5) {
        if (stride != 1 && stride != 2) return false;
        switch (dtype) {
        case SV_F32: return stride == 1 ? conv5_fits_s1_f32(tile) : conv5_fits_s2_f32(tile);
        case SV_BF16: return stride == 1 ? conv5_fits_s1_bf16(tile) : conv5_fits_s2_bf16(tile);
        case SV_F16: return stride == 1 ? conv5_fits_s1_f16(tile) : conv5_fits_s2_f16(tile);
        default: return false;
        }
    }
    switch (dtype) {
    case SV_F32: return conv_fits_f32(ks, stride, tile);
    case SV_BF16: return conv_fits_bf16(ks, stride, tile);
    case SV_F16: return conv_fits_f16(ks, stride, tile);
    case SV_I8: return conv_fits_i8(ks, stride, tile);
    default: return false;
    }
}

// A configuration whose tile shape does not fit the LDS for this kernel size
// and stride runs as th4_tn16 (which fits every case) with the same split;
// the tile shape does not change results.
int conv_resolve_cfg(int dtype, int ks, int stride, int cfg) {
    if (cfg < 0 || cfg >= conv_num_cfgs()) return cfg;
    if (dtype != SV_F32 && dtype != SV_BF16 && dtype != SV_F16 && dtype != SV_I8) return cfg;
    const int tile = cfg % kNumTiles;
    return fits_any(dtype, ks, stride, tile) ? cfg : cfg - tile + kFallbackTile;
}

static sv_status launch_any(int dtype, int ks, int stride, int tile, const ConvParams &p, int pg,
                            hipStream_t st) {
    if (ks == 5) {
        if (stride != 1 && stride != 2) return SV_ERR_UNSUPPORTED;
        switch (dtype) {
        case SV_F32:
            return stride == 1 ? launch_conv5_s1_f32(tile, p, pg, st) : launch_conv5_s2_f32(tile, p, pg, st);
        case SV_BF16:
            return stride == 1 ? launch_conv5_s1_bf16(tile, p, pg, st) : launch_conv5_s2_bf16(tile, p, pg, st);
        case SV_F16:
            return stride == 1 ? launch_conv5_s1_f16(tile, p, pg, st) : launch_conv5_s2_f16(tile, p, pg, st);
        default: return SV_ERR_DTYPE;
        }
    }
    switch (dtype) {
    case SV_F32: return launch_conv_f32(ks, stride, tile, p, pg, st);
    case SV_BF16: return launch_conv_bf16(ks, stride, tile, p, pg, st);
    case SV_F16: return launch_conv_f16(ks, stride, tile, p, pg, st);
    case SV_I8:
        if (ks == 5) return SV_ERR_UNSUPPORTED;
        return launch_conv_i8(ks, stride, tile, p, pg, st);
    default: return SV_ERR_DTYPE;
    }
}

int conv_effective_split(int dtype, int cfg, int Cin, long long npix, int n_pad, const float *part,
                         size_t part_bytes) {
    if (dtype == SV_I8) return 1;  // integer sums are kept whole
    int ksplit = cfg / kNumTiles + 1;
    // at most one split per base chunk of input channels, and only when the
    // partial sums fit the caller's buffer; otherwise one pass
    const int kcb = dtype == SV_F32 ? 16 : 32;
    ksplit = std::min(ksplit, cdiv(Cin, kcb));
    const size_t need = (size_t)ksplit * (size_t)npix * n_pad * sizeof(float);
    if (!part || need > part_bytes) ksplit = 1;
    return ksplit;
}

sv_status launch_conv_split(int dtype, int ks, int stride, int cfg, const ConvParams &p0, hipStream_t st,
                            int *ksplit_used) {
    if (cfg < 0 || cfg >= conv_num_cfgs()) return SV_ERR_RANGE;
    cfg = conv_resolve_cfg(dtype, ks, stride, cfg);
    ConvParams p = p0;
    p.ksplit = conv_effective_split(dtype, cfg, p.Cin, (long long)p.B * p.Ho * p.Wo, p.n_pad, p.part,
                                    p.part_bytes);
    if (p.ophase) p.ksplit = 1;  // a phase launch writes its pixels straight into the full map
    if (p.proj_out) {
        // the projection epilogue needs whole sums and every channel in each wave
        if (!conv_cfg_projects(cfg % kNumTiles, p.Cout)) return SV_ERR_UNSUPPORTED;
        p.ksplit = 1;
    }
    if (ksplit_used) *ksplit_used = p.ksplit > 1 ? p.ksplit : 1;
    // the row kernel stands for the default tiles; any other is the general kernel's, so
    // that the autotuners time what a later call with their choice runs
    const int tile = cfg % kNumTiles;
    const bool deflt = ks == 5 ? tile == T4_16 || tile == T4_32
                               : tile == conv_resolve_cfg(dtype, ks, stride, conv_default_tile(dtype, stride, p.Cin, p.Cout,
                                                                                              p.B, p.Ho, p.Wo));
    if (deflt && conv_rows_fits(dtype, ks, stride, p)) return launch_conv_rows(dtype, ks, stride, p, st);
    return launch_any(dtype, ks, stride, tile, p, 0, st);
}

sv_status launch_split_sum(int dtype, const ConvParams &p0, int ksplit, hipStream_t st) {
    if (ksplit <= 1) return SV_OK;
    ConvParams p = p0;
    p.ksplit = ksplit;
    p.defer_sum = 0;
    switch (dtype) {
    case SV_F32: return launch_split_sum_f32(p, st);
    case SV_BF16: return launch_split_sum_bf16(p, st);
    case SV_F16: return launch_split_sum_f16(p, st);
    default: return SV_ERR_DTYPE;  // INT8 never splits
    }
}

sv_status launch_conv(int dtype, int ks, int stride, int cfg, const ConvParams &p0, hipStream_t st) {
    return launch_conv_split(dtype, ks, stride, cfg, p0, st, nullptr);
}

sv_status launch_conv_tab(int dtype, int ks, int stride, int cfg, const ConvParams &p0, int grid,
                          hipStream_t st) {
    if (!p0.tab || grid <= 0) return SV_ERR_RANGE;
    if (cfg < 0 || cfg >= conv_num_cfgs()) return SV_ERR_RANGE;
    cfg = conv_resolve_cfg(dtype, ks, stride, cfg);
    if (p0.proj_out && !conv_cfg_projects(cfg % kNumTiles, p0.Cout))
        return SV_ERR_UNSUPPORTED;
    ConvParams p = p0;
    p.ksplit = 1;  // the persistent path never splits
    return launch_any(dtype, ks, stride, cfg % kNumTiles, p, grid, st);
}

// The tile shape a persistent pair-table launch uses for configuration cfg:
// 16-row tiles (tuned on uniform batches) become the 8-row tile of the same
// width, which runs faster there (twice the resident workgroups and twice
// the tiles to balance over uneven pairs).
int conv_persistent_cfg(int cfg) {
    if (cfg < 0 || cfg >= conv_num_cfgs()) return cfg;
    const CfgDesc &c = kCfgs[cfg % kNumTiles];
    if (c.TH != 16) return cfg;
    for (int t = 0; t < kNumTiles; ++t)
        if (kCfgs[t].TH == 8 && kCfgs[t].TN == c.TN && kCfgs[t].WM == c.WM && kCfgs[t].KCM == c.KCM)
            return t + (cfg / kNumTiles) * kNumTiles;
    return cfg;
}

// The tile shape for a 3x3 layer without an entry in the autotune cache (the
// tile does not change results, so this is a matter of speed alone).
//
// A taller or wider tile spends less on staging its halo, its pixel table and
// the weights, until the chip is left with idle CUs: two workgroups a CU are
// resident, so the lines lie between one workgroup a CU (256) and somewhat past
// the first full wave (512, 700).  They are fitted to 5900 timings of every tile
// at 4 to 74112 output pixels a map, 1 to 64 maps, 8 to 256 channels and each
// type, and are within 2.2 % of the best tile on average (the one tile per width
// that stood here first, four rows of 16, 32 or 64 channels: 34 %).  By group,
// this rule against those tiles:
//   16-bit, stride 1:  32 channels 0.88, 64 0.72, wider 0.68; INT8 0.85, 0.74, 0.76;
//   FP32 0.84, 0.65, 0.64; stride 2 past 32 channels 0.50 to 0.71 in every type.
// 16 channels keep four rows: a 32-channel tile would compute half its products
// for padding, at the same time or up to 1.38 of it (61 F16 maps 19x88 23.5 us
// against 15.5).
//   - A tall tile may pad at most a fifth more rows than the low one: 24 BF16 maps of
//     10x44, 96 -> 40 channels, in 16-row tiles compute 16 rows for 10.
//   - INT8 past 32 channels: eight rows only within one full wave (4 maps 28x85, 448 ->
//     192 channels, 576 workgroups: 80 us, T4_64 52; 12 maps 32x29, 256 -> 96, 288
//     workgroups: T8_32 31.9, T4_64 32.1, T4_32_K2 40.5).
//   - FP32 turns to tall tiles last: its matrix steps are longer, so the last wave costs
//     more (28 maps 82x52 to 32 channels in 16 rows 131 us, in four 100).
//   - Below the last line the reduction is shared between wavefronts (_K2, _K4): one
//     workgroup a CU or less, whose own chain is the time.
static int rule_tile(int dtype, int stride, int cin, int cout, int B, int Ho, int Wo) {
    auto wgs = [&](int th, int tn) { return (long long)B * cdiv(Ho, th) * cdiv(Wo, 16) * cdiv(cout, tn); };
    const int low = stride == 1 ? 4 : 2;
    auto tall = [&](int th, int tn, int from, int pad = 20) {  // pad: most added rows, in percent
        return wgs(th, tn) >= from && 100ll * cdiv(Ho, th) * th <= (100ll + pad) * cdiv(Ho, low) * low;
    };
    const bool f32 = dtype == SV_F32, i8 = dtype == SV_I8;
    if (cout <= 16) return T4_16;
    if (stride == 2) {
        if (cout <= 32) return wgs(4, 32) >= 256 ? T4_32 : T4_16;
        if (i8 && tall(8, 32, 300)) return T8_32;
        if (f32 && wgs(4, 32) >= 1600) return T4_32;
        if (wgs(2, 64) >= 256) return T2_64;
        return f32 || cin >= 64 ? T2_32_K2 : T4_16;
    }
    if (f32) {
        if (cout <= 32) {
            if (tall(16, 32, 700)) return T16_32;
            if (tall(8, 32, 700)) return T8_32;
            if (wgs(4, 32) >= 400) return T4_32;
            return wgs(4, 16) >= 300 ? T4_16 : T4_16_K2;
        }
        if (tall(8, 64, 700)) return T8_64;
        if (cout > 64 && tall(8, 32, 400)) return T8_32;
        if (wgs(4, 32) >= (cout <= 64 ? 1024 : 400)) return T4_32;
        return wgs(4, 16) >= 512 ? T4_16 : T4_16_K4;
    }
    if (cout <= 32) {
        if (tall(16, 32, 400)) return T16_32;
        if (tall(8, 32, i8 ? 300 : (cin > 32 ? 400 : 700))) return T8_32;
        return wgs(4, 32) >= 400 ? T4_32 : T4_16;
    }
    if (i8) {
        if (tall(16, 32, 320)) return T16_32;
        if (tall(8, 32, 256) && wgs(8, 32) <= 512) return T8_32;
        if (wgs(4, 64) >= 256) return T4_64;
        return wgs(4, 32) >= 256 ? T4_32_K2 : T2_32_K2;
    }
    if (tall(8, 64, 256, cout > 64 ? 34 : 20)) return T8_64;
    if (tall(8, 32, 300)) return T8_32;
    if (wgs(4, 32) >= 512) return T4_32;
    return wgs(4, 32) >= 256 ? T4_32_K2 : T4_16_K2;
}

// Batches whose images times channel tiles pass a grid's 65535 planes in a narrow
// tile take the widest.
int conv_default_tile(int dtype, int stride, int cin, int cout, int B, int Ho, int Wo) {
    const int t = rule_tile(dtype, stride, cin, cout, B, Ho, Wo);
    if ((long long)B * cdiv(cout, kCfgs[t].TN) <= CONV_MAX_PLANES) return t;
    return cout <= 16 ? T4_16 : (cout <= 32 ? T4_32 : T4_64);
}

bool conv_cfg_projects(int cfg, int cout) {
    if (cfg < 0) return false;
    const CfgDesc &c = kCfgs[cfg % kNumTiles];
    return c.TN >= cout && c.WM == 4;  // one channel tile; WN = 4 / WM = 1
}

void conv_cfg_tile(int cfg, int &TH, int &TN) {
    if (cfg < 0 || cfg >= conv_num_cfgs()) cfg = 0;
    TH = kCfgs[cfg % kNumTiles].TH;
    TN = kCfgs[cfg % kNumTiles].TN;
}

// ---- INT8: weight packing and the activations' maxima -------------------------------
// INT8 packing: one workgroup per output row n.  a = max |w[n]| over its
// inputs and taps (FP32), code = clamp(rint(w * (127 / a)), -127, 127),
// scale = a / 127; rows past Cout and columns past Cin are 0.
__global__ void __launch_bounds__(256)
k_pack_i8(const float *__restrict__ w, int Cout, int Cin, int k, int n_pad, int cin_pad, int8_t *__restrict__ dst,
          float *__restrict__ scale) {
    __shared__ float red[256];
    const int n = blockIdx.x;
    const int taps = k * k, len = Cin * taps;
    float m = 0.f;
    if (n < Cout)
        for (int e = threadIdx.x; e < len; e += 256) m = fmaxf(m, fabsf(w[(size_t)n * len + e]));
    red[threadIdx.x] = m;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + s]);
        __syncthreads();
    }
    const float a = red[0];
    const float inv = a > 0.f ? 127.0f / a : 0.f;
    if (threadIdx.x == 0) scale[n] = n < Cout ? a / 127.0f : 0.f;
    for (int e = threadIdx.x; e < taps * cin_pad; e += 256) {
        const int tap = e / cin_pad, c = e - tap * cin_pad;
        const float v = (n < Cout && c < Cin) ? w[((size_t)n * Cin + c) * taps + tap] : 0.f;
        dst[((size_t)tap * n_pad + n) * cin_pad + c] = quant_i8(v, inv);
    }
}

sv_status launch_pack_i8(const float *w, int Cout, int Cin, int k, int n_pad, int cin_pad, int8_t *dst,
                         float *scale, hipStream_t s) {
    hipLaunchKernelGGL(k_pack_i8, dim3(n_pad), dim3(256), 0, s, w, Cout, Cin, k, n_pad, cin_pad, dst, scale);
    SV_LAUNCH_CHECK("k_pack_i8");
    return SV_OK;
}

__global__ void k_amax_zero(uint32_t *__restrict__ amax, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) amax[i] = 0u;
}

// max(scale0 * d, img / 256) over the coarse pixels, one slot word per workgroup
__global__ void __launch_bounds__(256)
k_amax_x0(uint32_t *__restrict__ slot, const uint8_t *__restrict__ disp, const uint8_t *__restrict__ img,
          long long n, float scale0) {
    float m = 0.f;
    for (long long i = blockIdx.x * 256ll + threadIdx.x; i < n; i += (long long)gridDim.x * 256)
        m = fmaxf(m, fmaxf(scale0 * (float)disp[i], (float)img[i] * (1.0f / 256.0f)));
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    if ((threadIdx.x & 63) == 0) atomicMax(slot + (blockIdx.x & (AMAX_SUB - 1)), __float_as_uint(m));
}

sv_status launch_amax_prologue(uint32_t *amax, int nslots, int x0_slot, const uint8_t *disp,
                               const uint8_t *img, long long n, float scale0, hipStream_t s) {
    const int nw = nslots * AMAX_SUB;
    hipLaunchKernelGGL(k_amax_zero, dim3(cdiv(nw, 256)), dim3(256), 0, s, amax, nw);
    SV_LAUNCH_CHECK("k_amax_zero");
    const int blocks = (int)std::min<long long>((n + 255) / 256, 256);
    hipLaunchKernelGGL(k_amax_x0, dim3(blocks), dim3(256), 0, s, amax + (size_t)x0_slot * AMAX_SUB, disp, img, n,
                       scale0);
    SV_LAUNCH_CHECK("k_amax_x0");
    return SV_OK;
}

}  // namespace sv
