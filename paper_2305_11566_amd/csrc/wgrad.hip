// Weight and bias gradients of the convolutions (both networks), an MFMA
// product that reduces over pixels, and the ordered sum of its partials.
#include <algorithm>

#include "mfma.h"

namespace sv {

// ---------------------------------------------------------------------------
// dW[o][tap][c] = sum over output pixels m of dY[m][o] X[m shifted by tap][c],
// db[o] = sum over m of dY[m][o].
//
// Workgroup = (split, chunk of CC input channels, chunk of OC rows); it visits
// tiles of TH x 16 output pixels, tile = split, split + splits, ...  Per tile
// the output gradient ([pixel][o]) and the input patch with its halo
// ([pixel][c]) are staged in LDS once, and every (tap, 16 x 16) block of the
// workgroup is accumulated from them: the pixel (= reduction) index of both
// operands is a row of LDS, so a tap is only an address offset and nothing is
// unfolded.  FP32 reads one value per lane and 4-pixel step; 16-bit types read
// their eight pixels per lane with the transposing LDS read
// (ds_read_b64_tr_b16: of four 16-value rows, lane l gets column l).  The four
// waves take different rows of the tile, so a wave reads no operand that
// another one reads, and all blocks share the row operand; the waves' sums
// meet in LDS once, at the end.  LDS row pitches keep the four (eight) pixels
// a read touches in different banks.
//
// XP: the input is x0 alone (two channels).  Its columns are the (tap,
// channel) pairs, 2 taps of them, instead of 16 channels a tap of which 14
// would be zeros (E1: 2 column blocks instead of 9; FE: 4 instead of 25).  It
// runs the FP32 instruction on the values rounded to the compute dtype.
//
// Measured on a training pass: all layers of the BF16 network on 16 512x256
// crops 200 us, of the FP32 Table I network on four 255 us (610 and 1373 us with
// a kernel that unfolded each tile tap by tap in LDS, gave every wave its own
// blocks, and ran the deconvolutions over the zero-inserted input).  Staging
// bounds the large 16-bit layers: a tile's loads are issued together, one kind
// of source at a time (per element, with the kinds' branches between them,
// they cost a memory latency each: G0 132 us instead of 71).  The FP32 matrix
// rate bounds the 5x5 ones.
// ---------------------------------------------------------------------------
struct WgradParams {
    ConvSrc src[2];
    int B, Hi, Wi, Ho, Wo, Cin, Cout;
    const void *dy;
    int dy_pitch, dy_sdt;  // storage SV_F32 / SV_BF16 / SV_F16 of dy
    int bias_src;          // 1: the bias sums are those of src[0]'s pixels (see WgradJob)
    float *part;           // [split][o_pad][taps][cinp], XP: [split][o_pad][cinp]
    float *part_b;         // [split][b_pad]
    int o_pad, cinp, b_pad;
    int ntiles, tiles_x, tiles_y;
};

// elements of an LDS row of C channels whose neighbours a read takes S rows
// apart: four rows of 16 FP32 (eight of 16 16-bit values) then start in
// different groups of banks
constexpr int wg_pitch(int C, int S) { return S == 1 ? (C == 16 ? 16 : C + 16) : C + 8; }

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

// Pixels k = 0..7 of this lane's column: two transposing reads of four rows.
__device__ __forceinline__ u16x8 tr_frag(const uint16_t *p0, const uint16_t *p1) {
    const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)p0);
    const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)p1);
    u16x8 r;
#pragma unroll
    for (int i = 0; i < 4; ++i) { r[i] = (uint16_t)a[i]; r[4 + i] = (uint16_t)b[i]; }
    return r;
}

// N consecutive values of U places of a map stored in sdt, as FP32: every load
// is issued before the first conversion (a branch or conversion between them
// would wait for each in turn)
template <int N, int U>
__device__ __forceinline__ void ld_vals(const void *base, const size_t (&off)[U], int sdt, float (&v)[U][N]) {
    if (sdt == SV_F32) {
        f32x4 q[U][N / 4];
#pragma unroll
        for (int k = 0; k < U; ++k)
#pragma unroll
            for (int i = 0; i < N / 4; ++i) q[k][i] = *(const f32x4 *)((const float *)base + off[k] + 4 * i);
#pragma unroll
        for (int k = 0; k < U; ++k)
#pragma unroll
            for (int i = 0; i < N; ++i) v[k][i] = q[k][i / 4][i % 4];
    } else {
        typedef uint16_t hvec __attribute__((ext_vector_type(N)));
        hvec q[U];
#pragma unroll
        for (int k = 0; k < U; ++k) q[k] = *(const hvec *)((const uint16_t *)base + off[k]);
#pragma unroll
        for (int k = 0; k < U; ++k)
#pragma unroll
            for (int i = 0; i < N; ++i) v[k][i] = sdt == SV_BF16 ? bf16_bits_to_f32(q[k][i]) : f16_bits_to_f32(q[k][i]);
    }
}

template <int DT, int KS, int S, int OB, int CB, bool XP>
struct WgTile {
    static constexpr bool F32M = DT == SV_F32 || XP;      // FP32 operands in LDS
    typedef typename Elem<F32M ? (int)SV_F32 : DT>::T T;
    static constexpr int TAPS = KS * KS, PAD = (KS - 1) / 2;
    static constexpr int TH = (F32M && S == 2) ? 4 : 8, TW = 16, MT = TH * TW, RW = TH / 4;
    static constexpr int PH = (TH - 1) * S + KS, PW = (TW - 1) * S + KS, NPIX = PH * PW;
    static constexpr int OC = OB * 16, CC = XP ? 2 : CB * 16;
    static constexpr int OP = wg_pitch(OC, 1), CP = XP ? 2 : wg_pitch(CC, S);
    static constexpr int NB = XP ? (2 * TAPS + 15) / 16 : TAPS * CB;  // column blocks
    static constexpr int GS = F32M ? 4 : 8, KCG = CC / GS;            // channel groups of the patch
    static constexpr int JB = 4;                                      // blocks the waves combine at once
    struct Smem {
        union {
            struct { T dy[MT * OP]; T xp[NPIX * CP + (XP ? 64 : 0)]; } t;
            float red[4][JB * 256];
            float bsum[256 * 8];
        };
    };
};

template <int DT, int KS, int S, int OB, int CB, bool XP>
__global__ void __launch_bounds__(256, 2) k_wgrad(const WgradParams p)
{
    using W = WgTile<DT, KS, S, OB, CB, XP>;
    using T = typename W::T;
    constexpr bool F32M = W::F32M;
    constexpr int GS = W::GS;
    __shared__ __attribute__((aligned(16))) typename W::Smem sm;
    T *dyl = sm.t.dy, *xpl = sm.t.xp;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int g = lane >> 4, r16 = lane & 15;
    const int split = blockIdx.x, c0 = blockIdx.y * W::CC, o0 = blockIdx.z * W::OC;

    f32x4 acc[OB][W::NB];
#pragma unroll
    for (int i = 0; i < OB; ++i)
#pragma unroll
        for (int j = 0; j < W::NB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // this thread's share of the bias sums: four rows, or GS channels of src[0]
    float sb[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) sb[i] = 0.f;
    const int per_img = p.tiles_x * p.tiles_y;

    for (int tile = split; tile < p.ntiles; tile += gridDim.x) {
        const int b = tile / per_img, rem = tile - b * per_img;
        const int ty0 = rem / p.tiles_x;
        const int oy0 = ty0 * W::TH, ox0 = (rem - ty0 * p.tiles_x) * W::TW;
        const int iy0 = oy0 * S - W::PAD, ix0 = ox0 * S - W::PAD;
        __syncthreads();
        // ---- output gradient [pixel][o], four rows o a thread and step
        constexpr int OG = W::OC / 4, ND = W::MT * OG / 256 > 0 ? W::MT * OG / 256 : 1;
        {
            const int og = tid % OG, o = o0 + og * 4;
            float v[ND][4];
            size_t off[ND];
            bool ok[ND];
#pragma unroll
            for (int k = 0; k < ND; ++k) {
                const int m = tid / OG + k * (256 / OG);
                const int oy = oy0 + m / W::TW, ox = ox0 + m % W::TW;
                ok[k] = m < W::MT && oy < p.Ho && ox < p.Wo && o < p.Cout;
                off[k] = ok[k] ? (((size_t)b * p.Ho + oy) * p.Wo + ox) * p.dy_pitch + o : 0;
            }
            ld_vals<4, ND>(p.dy, off, p.dy_sdt, v);
#pragma unroll
            for (int k = 0; k < ND; ++k)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (!ok[k] || o + i >= p.Cout) v[k][i] = 0.f;
#pragma unroll
            for (int k = 0; k < ND; ++k) {
                const int m = tid / OG + k * (256 / OG);
                if (m >= W::MT) continue;
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (!p.bias_src) sb[i] += v[k][i];
                if constexpr (F32M) {
                    f32x4 q;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const typename Elem<DT>::T h = Elem<DT>::make(v[k][i]);
                        q[i] = Elem<DT>::load(&h);
                    }
                    *(f32x4 *)&dyl[m * W::OP + og * 4] = q;
                } else {
                    u16x4 q;
#pragma unroll
                    for (int i = 0; i < 4; ++i) q[i] = Elem<DT>::make(v[k][i]);
                    *(u16x4 *)&dyl[m * W::OP + og * 4] = q;
                }
            }
        }
        // ---- input patch [pixel][c], zeros outside the input grid
        if constexpr (XP) {
            const ConvSrc &s = p.src[0];
            for (int pix = tid; pix < W::NPIX; pix += 256) {
                const int py = pix / W::PW, px = pix - py * W::PW;
                const int yi = iy0 + py, xi = ix0 + px;
                float v0 = 0.f, v1 = 0.f;
                if (yi >= 0 && yi < p.Hi && xi >= 0 && xi < p.Wi) {
                    const size_t o = ((size_t)b * s.hs + yi) * s.ws + xi;
                    v0 = s.scale0 * (float)((const uint8_t *)s.ptr)[o];
                    v1 = (float)s.img[o] * (1.0f / 256.0f);
                }
                const typename Elem<DT>::T h0 = Elem<DT>::make(v0), h1 = Elem<DT>::make(v1);
                xpl[2 * pix] = Elem<DT>::load(&h0);
                xpl[2 * pix + 1] = Elem<DT>::load(&h1);
            }
        } else {
            // a thread keeps one channel group: one source, one kind
            constexpr int KCG = W::KCG, PSTEP = 256 / KCG, NE = (W::NPIX + PSTEP - 1) / PSTEP;
            const int cg = tid % KCG, c = c0 + cg * GS;
            const int si = c < p.src[0].C ? 0 : 1;
            const ConvSrc &s = si ? p.src[1] : p.src[0];
            const int kind = c < p.Cin ? s.kind : (int)SRC_NONE;
            const int sdt = s.sdt ? s.sdt - 1 : DT;
            const size_t cb = (size_t)s.coff + c - (si ? p.src[0].C : 0);
            auto put = [&](int pix, const float (&v)[GS]) {
                if constexpr (F32M) {
                    *(f32x4 *)&xpl[pix * W::CP + cg * GS] = f32x4{v[0], v[1], v[2], v[3]};
                } else {
                    u16x8 q;
#pragma unroll
                    for (int i = 0; i < GS; ++i) q[i] = Elem<DT>::make(v[i]);
                    *(u16x8 *)&xpl[pix * W::CP + cg * GS] = q;
                }
            };
            // element k of this thread: its patch pixel, and whether that is in the input grid
            auto place = [&](int k, int &pix, int &py, int &px) {
                pix = tid / KCG + k * PSTEP;
                py = pix / W::PW;
                px = pix - py * W::PW;
                const int yi = iy0 + py, xi = ix0 + px;
                return pix < W::NPIX && yi >= 0 && yi < p.Hi && xi >= 0 && xi < p.Wi;
            };
            if (kind == SRC_TENSOR) {
                // elements whose loads are in flight together; 36 accumulators leave registers for half
                constexpr int U = OB * W::NB > 25 ? (NE < 3 ? NE : 3) : (NE < 6 ? NE : 6);
#pragma unroll 1
                for (int k0 = 0; k0 < NE; k0 += U) {
                    float v[U][GS];
                    size_t off[U];
                    int pix[U];
                    bool ok[U], own[U];
#pragma unroll
                    for (int k = 0; k < U; ++k) {
                        int py, px;
                        ok[k] = place(k0 + k, pix[k], py, px);
                        own[k] = ok[k] && py >= W::PAD && py < W::PAD + W::TH * S && px >= W::PAD &&
                                 px < W::PAD + W::TW * S;
                        off[k] = ok[k] ? (((size_t)b * s.hs + iy0 + py) * s.ws + ix0 + px) * s.pitch + cb : cb;
                    }
                    ld_vals<GS, U>(s.ptr, off, sdt, v);
#pragma unroll
                    for (int k = 0; k < U; ++k) {
#pragma unroll
                        for (int i = 0; i < GS; ++i)
                            if (!ok[k]) v[k][i] = 0.f;
                        if (p.bias_src && own[k]) {
#pragma unroll
                            for (int i = 0; i < GS; ++i) sb[i] += v[k][i];
                        }
                        if (pix[k] < W::NPIX) put(pix[k], v[k]);
                    }
                }
            } else if (kind == SRC_RESIZE) {
                constexpr int U = OB * W::NB > 25 || NE < 2 ? 1 : 2;
#pragma unroll 1
                for (int k0 = 0; k0 < NE; k0 += U) {
                    float v[4 * U][GS];
                    size_t off[4 * U];
                    int pix[U];
                    bool ok[U];
                    float ly[U], lx[U];
                    const size_t rb = (size_t)b * s.hs;
#pragma unroll
                    for (int k = 0; k < U; ++k) {
                        int py, px, y0, y1, x0, x1;
                        ok[k] = place(k0 + k, pix[k], py, px);
                        bilin(ok[k] ? iy0 + py : 0, s.hs, p.Hi, y0, y1, ly[k]);
                        bilin(ok[k] ? ix0 + px : 0, s.ws, p.Wi, x0, x1, lx[k]);
                        off[4 * k] = ((rb + y0) * s.ws + x0) * s.pitch + cb;
                        off[4 * k + 1] = ((rb + y0) * s.ws + x1) * s.pitch + cb;
                        off[4 * k + 2] = ((rb + y1) * s.ws + x0) * s.pitch + cb;
                        off[4 * k + 3] = ((rb + y1) * s.ws + x1) * s.pitch + cb;
                    }
                    ld_vals<GS, 4 * U>(s.ptr, off, sdt, v);
#pragma unroll
                    for (int k = 0; k < U; ++k) {
                        float r[GS];
#pragma unroll
                        for (int i = 0; i < GS; ++i) {
                            const float top = (1.f - lx[k]) * v[4 * k][i] + lx[k] * v[4 * k + 1][i];
                            const float bot = (1.f - lx[k]) * v[4 * k + 2][i] + lx[k] * v[4 * k + 3][i];
                            r[i] = ok[k] ? (1.f - ly[k]) * top + ly[k] * bot : 0.f;
                        }
                        if (pix[k] < W::NPIX) put(pix[k], r);
                    }
                }
            } else {
                constexpr int U = OB * W::NB > 25 ? 4 : 8;
#pragma unroll 1
                for (int k0 = 0; k0 < NE; k0 += U) {
                    uint32_t dv[U], iv[U];
                    int pix[U];
                    bool ok[U];
#pragma unroll
                    for (int k = 0; k < U; ++k) {
                        int py, px;
                        ok[k] = place(k0 + k, pix[k], py, px) && kind == SRC_X0;
                        const size_t o = ok[k] ? ((size_t)b * s.hs + iy0 + py) * s.ws + ix0 + px : 0;
                        dv[k] = iv[k] = 0;
                        if (kind == SRC_X0) {
                            dv[k] = ((const uint8_t *)s.ptr)[o];
                            iv[k] = s.img[o];
                        }
                    }
#pragma unroll
                    for (int k = 0; k < U; ++k) {
                        float v[GS];
#pragma unroll
                        for (int i = 0; i < GS; ++i) v[i] = 0.f;
                        if (ok[k]) {
                            v[0] = s.scale0 * (float)dv[k];
                            v[1] = (float)iv[k] * (1.0f / 256.0f);
                        }
                        if (pix[k] < W::NPIX) put(pix[k], v);
                    }
                }
            }
        }
        __syncthreads();
        // ---- accumulate
        if constexpr (F32M) {
            // column block j, this lane's column: its offset from the pixel
            int xoff[XP ? W::NB : 1];
            if constexpr (XP) {
#pragma unroll
                for (int j = 0; j < W::NB; ++j) {
                    const int col = j * 16 + r16, tap = min(col >> 1, W::TAPS - 1);
                    xoff[j] = ((tap / KS) * W::PW + tap % KS) * 2 + (col & 1);
                }
            }
#pragma unroll
            for (int r = 0; r < W::RW; ++r) {
                const int row = wave * W::RW + r;
#pragma unroll
                for (int st = 0; st < 4; ++st) {
                    const int col = 4 * st + g;
                    float a[OB];
#pragma unroll
                    for (int i = 0; i < OB; ++i) a[i] = dyl[(row * W::TW + col) * W::OP + i * 16 + r16];
                    const T *xb = xpl + ((row * S) * W::PW + col * S) * W::CP + (XP ? 0 : r16);
#pragma unroll
                    for (int j = 0; j < W::NB; ++j) {
                        float x;
                        if constexpr (XP) {
                            x = xb[xoff[j]];
                        } else {
                            const int tap = j / CB, cbk = j % CB;
                            x = xb[((tap / KS) * W::PW + tap % KS) * W::CP + cbk * 16];
                        }
#pragma unroll
                        for (int i = 0; i < OB; ++i)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], x, acc[i][j], 0, 0, 0);
                    }
                }
            }
        } else {
            using M = Mfma<DT>;
            // lane group g takes pixels 8 (g & 1) .. + 7 of row 2 wave + (g >> 1);
            // this lane's address serves pixel (r16 / 4) and columns 4 (r16 % 4) ..
            const int row = wave * W::RW + (g >> 1);
            const int col = 8 * (g & 1) + (r16 >> 2), cq = 4 * (r16 & 3);
            const uint16_t *ya = dyl + (row * W::TW + col) * W::OP + cq;
            const uint16_t *xb = xpl + ((row * S) * W::PW + col * S) * W::CP + cq;
            u16x8 a[OB];
#pragma unroll
            for (int i = 0; i < OB; ++i) a[i] = tr_frag(ya + i * 16, ya + i * 16 + 4 * W::OP);
#pragma unroll
            for (int j = 0; j < W::NB; ++j) {
                const int tap = j / CB, cbk = j % CB;
                const uint16_t *xt = xb + ((tap / KS) * W::PW + tap % KS) * W::CP + cbk * 16;
                const u16x8 x = tr_frag(xt, xt + 4 * S * W::CP);
#pragma unroll
                for (int i = 0; i < OB; ++i) acc[i][j] = M::run(a[i], x, acc[i][j]);
            }
        }
    }

    // ---- the four waves' sums, JB blocks at a time, in wave order
    constexpr int NBLK = OB * W::NB;
#pragma unroll
    for (int j0 = 0; j0 < NBLK; j0 += W::JB) {
        __syncthreads();
#pragma unroll
        for (int jj = 0; jj < W::JB; ++jj) {
            const int j = j0 + jj;
            if (j >= NBLK) continue;
            const f32x4 v = acc[j / W::NB][j % W::NB];  // row 4 g + i, column r16
#pragma unroll
            for (int i = 0; i < 4; ++i) sm.red[wave][jj * 256 + (4 * g + i) * 16 + r16] = v[i];
        }
        __syncthreads();
#pragma unroll
        for (int jj = 0; jj < W::JB; ++jj) {
            const int j = j0 + jj;
            if (j >= NBLK) continue;
            const int e = jj * 256 + tid;
            const float v = ((sm.red[0][e] + sm.red[1][e]) + sm.red[2][e]) + sm.red[3][e];
            const int o = o0 + (j / W::NB) * 16 + (tid >> 4), kb = j % W::NB, q = tid & 15;
            if constexpr (XP)
                p.part[((size_t)split * p.o_pad + o) * p.cinp + kb * 16 + q] = v;
            else
                p.part[(((size_t)split * p.o_pad + o) * W::TAPS + kb / CB) * p.cinp + c0 + (kb % CB) * 16 + q] = v;
        }
    }
    // ---- bias: rows of dy, or channels of src[0]
    constexpr int BG = W::OC / 4;                       // threads' row groups
    constexpr int SG = XP ? 1 : W::KCG;                 // threads' channel groups
    if (p.bias_src ? blockIdx.z == 0 : blockIdx.y == 0) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 8; ++i) sm.bsum[tid * 8 + i] = sb[i];
        __syncthreads();
        const int n = p.bias_src ? W::CC : W::OC, ng = p.bias_src ? SG : BG, per = p.bias_src ? GS : 4;
        if (tid < n) {
            float t = 0.f;
            for (int k = tid / per; k < 256; k += ng) t += sm.bsum[k * 8 + tid % per];
            p.part_b[(size_t)split * p.b_pad + (p.bias_src ? c0 : o0) + tid] = t;
        }
    }
}

// ---------------------------------------------------------------------------
// Sums the partials of all splits in a fixed order and writes the canonical
// gradient.  A workgroup takes 64 consecutive partial elements (so its reads
// are contiguous) and 16 runs of splits, one a wave, eight loads in flight per
// lane; the runs meet in LDS in order: 5 us a layer (91 to 330 with a thread
// walking up to 1024 splits of one element, in the canonical order, a stride of a
// whole row between neighbouring threads).
// ---------------------------------------------------------------------------
struct ReduceParams {
    const float *part, *part_b;
    int splits, o_pad, taps, cinp, b_pad;
    int rows, cols;          // valid rows and columns of the partials
    GradMap m;
    float *gw, *gb;
};

constexpr int WR_E = 64, WR_G = 16;
__global__ void __launch_bounds__(WR_E * WR_G) k_wgrad_reduce(const ReduceParams p)
{
    __shared__ float sh[WR_G][WR_E];
    const int nw = p.o_pad * p.taps * p.cinp;
    const int lane = threadIdx.x % WR_E, grp = threadIdx.x / WR_E;
    const int nblk_w = (nw + WR_E - 1) / WR_E;
    const bool bias = (int)blockIdx.x >= nblk_w;
    const int e = (bias ? (int)blockIdx.x - nblk_w : (int)blockIdx.x) * WR_E + lane;
    const int n = bias ? p.b_pad : nw;
    const float *src = bias ? p.part_b : p.part;
    const int per = (p.splits + WR_G - 1) / WR_G;
    const int s0 = grp * per, s1 = min(s0 + per, p.splits);
    float acc[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) acc[k] = 0.f;
    if (e < n)
        for (int s = s0; s < s1; s += 8) {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const bool ok = s + k < s1;
                const float v = src[(size_t)(ok ? s + k : s0) * n + e];
                acc[k] += ok ? v : 0.f;
            }
        }
    sh[grp][lane] = ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
    __syncthreads();
    if (grp != 0 || e >= n) return;
    float t = 0.f;
#pragma unroll
    for (int k = 0; k < WR_G; ++k) t += sh[k][lane];
    if (bias) {
        const int r0 = p.m.kind == GM_FE ? 32 : 1 << 30;  // FE_2's biases follow FE_2's weights
        if (e < p.m.nbias) p.gb[e < r0 ? e : e - r0 + p.m.off2] = t;
        return;
    }
    const int col = e % p.cinp, tap = (e / p.cinp) % p.taps, row = e / (p.cinp * p.taps);
    if (row >= p.rows || col >= p.cols) return;
    const int cin = p.m.cin, kk = p.m.kk;
    switch (p.m.kind) {
    case GM_OIHW: p.gw[((size_t)row * cin + col) * kk + (p.m.flip ? kk - 1 - tap : tap)] = t; break;
    case GM_SWAP: p.gw[((size_t)col * cin + row) * kk + tap] = t; break;     // row: input channel, column: output
    case GM_TAPROWS: p.gw[(size_t)col * kk + row] = t; break;                // row: tap of the one output
    case GM_Y:                                                               // columns [D 16 | FE 64 | X_0 | X_1]
        if (col < 81) p.gw[(size_t)(col < 16 ? col : (col < 80 ? col + 1 : 16)) * kk + row] = t;
        break;
    case GM_X0: p.gw[((size_t)row * 2 + (col & 1)) * kk + (col >> 1)] = t; break;
    case GM_FE:  // rows 0..31 of FE_1 read X_0 alone, rows 32..63 of FE_2 X_1
        if ((row >> 5) == (col & 1))
            p.gw[(row < 32 ? (size_t)row * kk : (size_t)(row - 32) * kk + p.m.off1) + (col >> 1)] = t;
        break;
    }
}

struct WgradPlan { int ob, cb, xp, splits, o_pad, cinp, taps, b_pad, ntiles, tx, ty, nc, no; };

// Rows and columns of a workgroup: all of the layer's when they fit, so that
// the tile is staged once; at most 36 accumulator blocks a wave (KS = 3: 32
// rows x 32 channels; KS = 5: 16 x 16), which leaves two waves a SIMD.
// Splits: 768 workgroups in all (three a CU, hiding each other's staging), at
// most one tile each.
static WgradPlan wgrad_plan(const WgradJob &j) {
    WgradPlan w{};
    const int Cin = j.s0.C + (j.s1.kind ? j.s1.C : 0);
    w.xp = j.s0.kind == SRC_X0 && !j.s1.kind && j.ks > 1;
    w.taps = w.xp ? 1 : j.ks * j.ks;
    w.ob = j.ks == 5 && !w.xp ? 1 : (j.Cout > 16 ? 2 : 1);
    w.cb = w.xp ? 1 : (j.ks == 5 ? 1 : (Cin > 16 ? 2 : 1));
    const int OC = 16 * w.ob, CC = 16 * w.cb;
    w.o_pad = cdiv(j.Cout, OC) * OC;
    w.no = w.o_pad / OC;
    if (w.xp) {
        w.cinp = cdiv(2 * j.ks * j.ks, 16) * 16;
        w.nc = 1;
    } else {
        w.nc = cdiv(Cin, CC);
        w.cinp = w.nc * CC;
    }
    w.b_pad = j.bias_src ? w.cinp : w.o_pad;
    const bool f32m = j.dtype == SV_F32 || w.xp;
    w.tx = cdiv(j.Wo, 16);
    w.ty = cdiv(j.Ho, f32m && j.stride == 2 ? 4 : 8);
    w.ntiles = j.B * w.tx * w.ty;
    w.splits = std::max(1, std::min(768 / (w.nc * w.no), w.ntiles));
    return w;
}

size_t wgrad_part_floats(const WgradJob &j) {
    const WgradPlan w = wgrad_plan(j);
    return (size_t)w.splits * ((size_t)w.o_pad * w.taps * w.cinp + w.b_pad);
}

template <int DT, int KS, int S>
static void launch_wgrad_ks(const WgradParams &p, const WgradPlan &w, hipStream_t st) {
    const dim3 grid(w.splits, w.nc, w.no);
#define SV_WG(OB, CB, XP) hipLaunchKernelGGL((k_wgrad<DT, KS, S, OB, CB, XP>), grid, dim3(256), 0, st, p)
    if constexpr (KS > 1) {
        if (w.xp) {
            if (w.ob == 2) SV_WG(2, 1, true);
            else SV_WG(1, 1, true);
            return;
        }
    }
    if constexpr (KS == 5) {
        SV_WG(1, 1, false);
    } else {
        if (w.ob == 2 && w.cb == 2) SV_WG(2, 2, false);
        else if (w.ob == 2) SV_WG(2, 1, false);
        else if (w.cb == 2) SV_WG(1, 2, false);
        else SV_WG(1, 1, false);
    }
#undef SV_WG
}

template <int DT>
static sv_status launch_wgrad_dt(int ks, int stride, const WgradParams &p, const WgradPlan &w, hipStream_t st) {
    if (ks == 1 && stride == 1) launch_wgrad_ks<DT, 1, 1>(p, w, st);
    else if (ks == 3 && stride == 1) launch_wgrad_ks<DT, 3, 1>(p, w, st);
    else if (ks == 3 && stride == 2) launch_wgrad_ks<DT, 3, 2>(p, w, st);
    else if (ks == 5 && stride == 1) launch_wgrad_ks<DT, 5, 1>(p, w, st);
    else if (ks == 5 && stride == 2) launch_wgrad_ks<DT, 5, 2>(p, w, st);
    else return SV_ERR_UNSUPPORTED;
    SV_LAUNCH_CHECK("k_wgrad");
    return SV_OK;
}

sv_status launch_wgrad(const WgradJob &j, const GradMap &m, float *part, float *gw, float *gb, hipStream_t st) {
    const WgradPlan w = wgrad_plan(j);
    WgradParams p{};
    p.src[0] = j.s0; p.src[1] = j.s1;
    p.B = j.B; p.Hi = j.Hi; p.Wi = j.Wi; p.Ho = j.Ho; p.Wo = j.Wo;
    p.Cin = j.s0.C + (j.s1.kind ? j.s1.C : 0);
    p.Cout = j.Cout;
    p.dy = j.dy; p.dy_pitch = j.dy_pitch; p.dy_sdt = j.dy_sdt;
    p.bias_src = j.bias_src;
    p.part = part;
    p.part_b = part + (size_t)w.splits * w.o_pad * w.taps * w.cinp;
    p.o_pad = w.o_pad; p.cinp = w.cinp; p.b_pad = w.b_pad;
    p.ntiles = w.ntiles; p.tiles_x = w.tx; p.tiles_y = w.ty;
    sv_status r;
    switch (j.dtype) {
    case SV_F32: r = launch_wgrad_dt<SV_F32>(j.ks, j.stride, p, w, st); break;
    case SV_BF16: r = launch_wgrad_dt<SV_BF16>(j.ks, j.stride, p, w, st); break;
    case SV_F16: r = launch_wgrad_dt<SV_F16>(j.ks, j.stride, p, w, st); break;
    default: return SV_ERR_DTYPE;
    }
    if (r != SV_OK) return r;
    ReduceParams q{};
    q.part = p.part; q.part_b = p.part_b;
    q.splits = w.splits; q.o_pad = w.o_pad; q.taps = w.taps; q.cinp = w.cinp; q.b_pad = w.b_pad;
    q.rows = j.Cout;
    q.cols = w.xp ? 2 * j.ks * j.ks : p.Cin;
    q.m = m;
    q.gw = gw; q.gb = gb;
    const int blocks = cdiv(w.o_pad * w.taps * w.cinp, WR_E) + (m.nbias ? cdiv(w.b_pad, WR_E) : 0);
    hipLaunchKernelGGL(k_wgrad_reduce, dim3(blocks), dim3(WR_E * WR_G), 0, st, q);
    SV_LAUNCH_CHECK("k_wgrad_reduce");
    return SV_OK;
}

}  // namespace sv
