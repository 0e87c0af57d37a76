// Stride-2 transposed convolutions: the stride-2 deconvolutions of the Table I
// decoder and the input gradients of the stride-2 encoder layers (5x5 there, 3x3
// in the other network).  Correlation of the zero-inserted map with the packed
// kernel, without the zeros: an output of parity (py, px) has only the taps of
// that parity, (2 ty - py, 2 tx - px) less (5 - KS) / 2, over the map's rows
// a - 1 + ty, 25 (9) products for four outputs instead of 100 (36).
//
// What bounds it: the matrix steps for FP32, latency of the few workgroups of the
// coarse levels and the patch's staging otherwise.  So a workgroup makes the 2 MB
// x 32 outputs of MB x 16 map pixels and each of its four waves the outputs of one
// parity: every weight is read by one wave only, once for MB rows, so weights go
// straight to registers and only the patch (MB + 2 rows, 18 columns, one chunk of
// channels, the next chunk's loads in flight) to LDS.  The parities have 9, 6, 6
// and 4 taps (4, 2, 2, 1 for 3x3): the workgroup's index rotates them over the
// waves, so that the SIMDs of a CU get the same work.
//
// The order of every sum is the one of the general kernel over the zero-inserted
// map: base chunks ascending, taps ascending; the results are the same bits.
//
// Measured against the general kernel (us): the Table I decoder's two layers for
// 16 BF16 images of 1242x375 110 (zero-inserted, and four parity launches) -> 30,
// for one in FP32 34 (with a split reduction) -> 23; input gradients of its
// encoder layers, 4 of 512x256 at factor 2 in FP32, 147 -> 45 and 31 -> 14; of the
// other network's, 16 of 512x256 in BF16, 20 -> 13 and 15 -> 10.
#include <type_traits>

#include "conv_impl.h"

namespace sv {

namespace {

template <int DT, int KS, int NB, int MB, bool F32SRC>
__global__ void __launch_bounds__(256) k_tconv(const ConvParams p, int tiles_x, int tiles_y, int ntn)
{
    using M = Mfma<DT>;
    using T = typename M::T;
    using vec = typename M::vec;
    constexpr int GS = M::GS, KCB = 4 * GS;
    using ST = typename std::conditional<F32SRC, float, T>::type;
    constexpr int PH = MB + 2, PW = 18, NPIX = PH * PW;
    constexpr int KCP = KCB + GS;                       // padded patch row
    constexpr int T0 = KS == 5 ? 0 : 1, NT = 3 - T0;    // the tap rows (columns) a parity may have
    constexpr int SH = (5 - KS) / 2;
    constexpr int NE = (NPIX * 4 + 255) / 256;          // patch vectors a thread
    __shared__ __attribute__((aligned(16))) T patch[2][NPIX * KCP];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int g = lane >> 4, r16 = lane & 15;
    // neighbouring tiles on one XCD
    const int nblk = (int)gridDim.x, q8 = nblk / 8, hw = (int)blockIdx.x;
    int r = hw < 8 * q8 ? (hw % 8) * q8 + hw / 8 : hw;
    const int tx = r % tiles_x; r /= tiles_x;
    const int ty = r % tiles_y; r /= tiles_y;
    const int n0 = r % ntn * NB * 16, b = r / ntn;
    const int phase = __builtin_amdgcn_readfirstlane((wave + hw) & 3), py = phase >> 1, px = phase & 1;
    const int a0 = ty * MB, b0 = tx * 16;
    const int hs = p.src[0].hs, ws = p.src[0].ws;
    const ST *src = (const ST *)p.src[0].ptr + (size_t)b * hs * ws * p.src[0].pitch + p.src[0].coff;
    const T *wpk = (const T *)p.wpk;

    // ---- staging: this thread's patch vectors, channel group tid % 4 -----------
    int off[NE];  // < 0: outside the map
#pragma unroll
    for (int j = 0; j < NE; ++j) {
        const int pix = (tid + 256 * j) >> 2;
        const int y = a0 - 1 + pix / PW, x = b0 - 1 + pix % PW;
        off[j] = pix < NPIX && y >= 0 && y < hs && x >= 0 && x < ws ? (y * ws + x) * p.src[0].pitch : -1;
    }
    const int cg = (tid & 3) * GS;
    typedef ST S4 __attribute__((ext_vector_type(4)));
    constexpr int NV = GS / 4;
    S4 pre[NE][NV];
    auto fetch = [&](int c0) {
        const bool in = c0 + cg < p.Cin;  // (channels come in whole groups)
#pragma unroll
        for (int j = 0; j < NE; ++j)
#pragma unroll
            for (int k = 0; k < NV; ++k)
                pre[j][k] = *(const S4 *)(src + (in && off[j] >= 0 ? (size_t)off[j] + c0 + cg + 4 * k : 0));
    };
    auto commit = [&](int c0, int buf) {
        const bool in = c0 + cg < p.Cin;
#pragma unroll
        for (int j = 0; j < NE; ++j) {
            const int pix = (tid + 256 * j) >> 2;
            if (pix >= NPIX) continue;
            const bool ok = in && off[j] >= 0;
            vec v;
            if constexpr (F32SRC) {
                float f[GS];
#pragma unroll
                for (int i = 0; i < GS; ++i) f[i] = ok ? pre[j][i / 4][i % 4] : 0.f;
                v = pack_vec<DT, GS>(f, 0.f);
            } else {
#pragma unroll
                for (int i = 0; i < GS; ++i) v[i] = ok ? pre[j][i / 4][i % 4] : (T)0;
            }
            *(vec *)&patch[buf][pix * KCP + cg] = v;
        }
    };

    typename M::acc acc[MB][NB];
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int n = 0; n < NB; ++n) acc[m][n] = typename M::acc{0, 0, 0, 0};
    // rows of the packed weights: past n_pad (a last tile of channels) row 0, not stored
    int nrow[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n) nrow[n] = n0 + 16 * n < p.n_pad ? n0 + 16 * n + r16 : r16;

    fetch(0);
    int buf = 0;
    for (int c0 = 0; c0 < p.Cin; c0 += KCB, buf ^= 1) {
        // this wave's weights (a tap outside the kernel reads tap 0 and is skipped)
        vec a[NT][NT][NB];
        const int wc = c0 + g * GS;
        const bool win = wc < p.cin_pad;
#pragma unroll
        for (int u = 0; u < NT; ++u)
#pragma unroll
            for (int v = 0; v < NT; ++v) {
                const int ku = 2 * (T0 + u) - py - SH, kv = 2 * (T0 + v) - px - SH;
                const int tap = ku >= 0 && ku < KS && kv >= 0 && kv < KS ? ku * KS + kv : 0;
#pragma unroll
                for (int n = 0; n < NB; ++n)
                    a[u][v][n] = *(const vec *)(wpk + ((size_t)tap * p.n_pad + nrow[n]) * p.cin_pad + (win ? wc : 0));
            }
        commit(c0, buf);
        __syncthreads();
        if (c0 + KCB < p.Cin) fetch(c0 + KCB);
        if (!win) {
#pragma unroll
            for (int u = 0; u < NT; ++u)
#pragma unroll
                for (int v = 0; v < NT; ++v)
#pragma unroll
                    for (int n = 0; n < NB; ++n)
#pragma unroll
                        for (int i = 0; i < GS; ++i) a[u][v][n][i] = (T)0;
        }
        const T *pb = patch[buf] + r16 * KCP + g * GS;
#pragma unroll
        for (int u = 0; u < NT; ++u) {
            const int ku = 2 * (T0 + u) - py - SH;
            if (ku < 0 || ku >= KS) continue;  // the whole wave's
#pragma unroll
            for (int v = 0; v < NT; ++v) {
                const int kv = 2 * (T0 + v) - px - SH;
                if (kv < 0 || kv >= KS) continue;
#pragma unroll
                for (int m = 0; m < MB; ++m) {
                    const vec x = *(const vec *)(pb + ((m + T0 + u) * PW + T0 + v) * KCP);
#pragma unroll
                    for (int n = 0; n < NB; ++n) acc[m][n] = M::run(a[u][v][n], x, acc[m][n]);
                }
            }
        }
    }
    // ---- bias, activation, backward terms and the store -------------------------
    float bias[NB][4];
#pragma unroll
    for (int n = 0; n < NB; ++n) conv_bias4<DT>(p, n0 + 16 * n + 4 * g, bias[n]);
    const int ox = 2 * (b0 + r16) + px;
    if (ox >= p.Wo) return;
#pragma unroll
    for (int m = 0; m < MB; ++m) {
        const int oy = 2 * (a0 + m) + py;
        if (oy >= p.Ho) break;
        const size_t pix = ((size_t)b * p.Ho + oy) * p.Wo + ox;
#pragma unroll
        for (int n = 0; n < NB; ++n) {
            const float v[4] = {acc[m][n][0], acc[m][n][1], acc[m][n][2], acc[m][n][3]};
            conv_epilogue<DT, true>(p, pix, n0 + 16 * n + 4 * g, v, bias[n]);
        }
    }
}

template <int DT, int KS, int NB, int MB>
sv_status launch_t(const ConvParams &p, hipStream_t st) {
    const int tx = cdiv(cdiv(p.Wo, 2), 16), ty = cdiv(cdiv(p.Ho, 2), MB), ntn = cdiv(p.Cout, NB * 16);
    const long long n = (long long)p.B * tx * ty * ntn;
    if (n >= (1ll << 31)) return SV_ERR_SHAPE;
    const bool f32src = p.src[0].sdt == 1 + SV_F32;
    if constexpr (DT != SV_F32) {
        if (f32src) {
            hipLaunchKernelGGL((k_tconv<DT, KS, NB, MB, true>), dim3((unsigned)n), dim3(256), 0, st, p, tx, ty, ntn);
            SV_LAUNCH_CHECK("k_tconv");
            return SV_OK;
        }
    }
    hipLaunchKernelGGL((k_tconv<DT, KS, NB, MB, false>), dim3((unsigned)n), dim3(256), 0, st, p, tx, ty, ntn);
    SV_LAUNCH_CHECK("k_tconv");
    return SV_OK;
}

template <int DT, int KS>
sv_status launch_k(const ConvParams &p, hipStream_t st) {
    const int nb = p.Cout <= 16 ? 1 : 2;
    // Rows a workgroup: more of them share the weights' loads and the patch's halo,
    // as long as the launch still has a workgroup for every CU (four rows: enough
    // for a CU to overlap one's loads with another's products).
    auto wgs = [&](int mb) {
        return (long long)p.B * cdiv(cdiv(p.Wo, 2), 16) * cdiv(cdiv(p.Ho, 2), mb) * cdiv(p.Cout, nb * 16);
    };
    const int mb = wgs(4) >= 400 ? 4 : wgs(2) >= 256 ? 2 : 1;
    if (nb == 1) return mb == 4 ? launch_t<DT, KS, 1, 4>(p, st) : mb == 2 ? launch_t<DT, KS, 1, 2>(p, st) : launch_t<DT, KS, 1, 1>(p, st);
    return mb == 4 ? launch_t<DT, KS, 2, 4>(p, st) : mb == 2 ? launch_t<DT, KS, 2, 2>(p, st) : launch_t<DT, KS, 2, 1>(p, st);
}

template <int DT>
sv_status launch_d(int ks, const ConvParams &p, hipStream_t st) {
    return ks == 5 ? launch_k<DT, 5>(p, st) : launch_k<DT, 3>(p, st);
}

}  // namespace

// The map is read in vectors of four elements of its own dtype, in whole channel
// groups, at 32-bit offsets from an image's first element.
bool tconv_fits(int dtype, int ks, const ConvParams &p) {
    const ConvSrc &s = p.src[0];
    return (dtype == SV_F32 || dtype == SV_BF16 || dtype == SV_F16) && (ks == 3 || ks == 5) &&
           p.src[1].kind == SRC_NONE && s.C % 8 == 0 && s.pitch % 4 == 0 && s.coff % 4 == 0 &&
           (!s.sdt || s.sdt - 1 == dtype || s.sdt - 1 == SV_F32) && p.Cin == s.C && p.Ho <= 2 * s.hs &&
           p.Wo <= 2 * s.ws && (long long)s.hs * s.ws * s.pitch < (1ll << 31);
}

sv_status launch_tconv(int dtype, int ks, const ConvParams &p, hipStream_t st) {
    if (!tconv_fits(dtype, ks, p)) return SV_ERR_UNSUPPORTED;
    switch (dtype) {
    case SV_F32: return launch_d<SV_F32>(ks, p, st);
    case SV_BF16: return launch_d<SV_BF16>(ks, p, st);
    case SV_F16: return launch_d<SV_F16>(ks, p, st);
    default: return SV_ERR_DTYPE;
    }
}

}  // namespace sv
