// Convolutions of one map read in place, or of [resize(map) | second source], a
// tile of 4 MB x 16 outputs by 16 NB channels a workgroup, each wave MB rows of it.
//
// The general kernel (conv_impl.h) stages a chunk's weights in LDS for a tile of
// four rows: for a 5x5 layer 2.5 times the bytes of its patch, and every product
// reads both operands from LDS.  Here a wave keeps the chunk's weights in
// registers, read straight from memory (the four waves' reads meet in the L1),
// for MB rows, and an input vector read from LDS serves the up to KS output rows
// it lies under.  The next chunk's patch is loaded beside the products.
//
// The order of every sum is the general kernel's: base chunks ascending, taps
// ascending; the results are the same bits.
//
// What bounds it now: the latency of a workgroup's serial steps (its loads, the
// patch through LDS, the products, the stores), with two workgroups a CU.
//
// Measured against the general kernel (us): 16 BF16 maps of the Table I network,
// 156x47: 64 -> 16 channels, stride 2, 63 -> 41, 40 -> 8 31 -> 15; the input gradients
// of 16 BF16 maps 256x128, 16 -> 16 channels of 3x3, 48 -> 20, and 128x64, 16 -> 48,
// 27 -> 17; 16 BF16 maps 256x128 of [resize 16 | x0] to 16 channels 57 -> 36; 64
// BF16 maps 156x47 of 3x3, stride 2, 32 -> 64 channels, 46 -> 29; 4 FP32 maps 128x64
// of 5x5, 40 -> 8 channels, 26 -> 18.
#include <type_traits>

#include "conv_impl.h"

namespace sv {

namespace {

// how the input is read: the map as stored, stored in FP32, or [resize(map) |
// second source] (a map as stored from a chunk's start, or x0 inside a chunk)
enum RowsMode { RM_OWN = 0, RM_F32 = 1, RM_RESIZE = 2 };

template <int DT, int KS, int S, int MB>
struct RowsTile {
    using T = typename Mfma<DT>::T;
    static constexpr int GS = Mfma<DT>::GS, KCB = 4 * GS, KCP = KCB + GS;
    static constexpr int PH = (4 * MB - 1) * S + KS, PW = 15 * S + KS, NPIX = PH * PW;
    static constexpr int LDS1 = NPIX * KCP * (int)sizeof(T);
    static constexpr int NBUF = 2 * LDS1 <= 80 * 1024 ? 2 : 1;  // two where two workgroups still fit a CU
};

template <int DT, int KS, int S, int MB, int NB, int MODE>
__global__ void __launch_bounds__(256, 2) k_conv_rows(const ConvParams p, int tiles_x, int tiles_y, int ntn)
{
    using R = RowsTile<DT, KS, S, MB>;
    using M = Mfma<DT>;
    using T = typename M::T;
    using vec = typename M::vec;
    constexpr int GS = R::GS, KCB = R::KCB, KCP = R::KCP, PW = R::PW, NPIX = R::NPIX, NBUF = R::NBUF;
    constexpr int PAD = (KS - 1) / 2;
    constexpr bool F32SRC = MODE == RM_F32, RES = MODE == RM_RESIZE;
    using ST = typename std::conditional<F32SRC, float, T>::type;
    constexpr int NE = (NPIX * 4 + 255) / 256;  // patch vectors a thread
    constexpr int NG = RES && NE > 3 ? (NE + 1) / 2 : NE;  // of them fetched ahead
    constexpr int NC = RES ? 4 : 1;                        // vectors read for each
    struct __attribute__((aligned(16))) Axis { int i0, i1; float lam; };  // i0 < 0: outside the input grid
    __shared__ __attribute__((aligned(16))) T patch[NBUF][NPIX * KCP];
    __shared__ Axis ax[RES ? R::PH + PW : 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int g = lane >> 4, r16 = lane & 15;
    // neighbouring tiles on one XCD
    const int nblk = (int)gridDim.x, q8 = nblk / 8, hw = (int)blockIdx.x;
    int r = hw < 8 * q8 ? (hw % 8) * q8 + hw / 8 : hw;
    const int tx = r % tiles_x; r /= tiles_x;
    const int ty = r % tiles_y; r /= tiles_y;
    const int n0 = r % ntn * NB * 16, b = r / ntn;
    const int oy0 = ty * 4 * MB, ox0 = tx * 16;
    const int hs = p.src[0].hs, ws = p.src[0].ws;
    const ST *src = (const ST *)p.src[0].ptr + (size_t)b * hs * ws * p.src[0].pitch + p.src[0].coff;
    const int C0 = RES ? p.src[0].C : p.Cin;
    const T *wpk = (const T *)p.wpk;

    // ---- staging: this thread's patch vectors, channel group tid % 4 -----------
    int off[NE];  // element of the map read in place (RES: the second source's pixel), < 0: outside
    const int pitch_in = RES ? 1 : p.src[0].pitch;
#pragma unroll
    for (int j = 0; j < NE; ++j) {
        const int pix = (tid + 256 * j) >> 2;
        const int y = oy0 * S - PAD + pix / PW, x = ox0 * S - PAD + pix % PW;
        off[j] = pix < NPIX && y >= 0 && y < p.Hi && x >= 0 && x < p.Wi ? (y * p.Wi + x) * pitch_in : -1;
    }
    if constexpr (RES) {
        // each patch row's and column's source pair and weight
        if (tid < R::PH + PW) {
            const bool row = tid < R::PH;
            const int o = row ? oy0 * S - PAD + tid : ox0 * S - PAD + tid - R::PH, n = row ? p.Hi : p.Wi;
            Axis q = {-1, -1, 0.f};
            if (o >= 0 && o < n) bilin(o, row ? hs : ws, n, q.i0, q.i1, q.lam);
            ax[tid] = q;
        }
        __syncthreads();
    }
    const int cg = (tid & 3) * GS;
    constexpr int VN = F32SRC || DT == SV_F32 ? 4 : RES ? 8 : 4;  // elements a load
    typedef ST SV __attribute__((ext_vector_type(VN)));
    constexpr int NV = GS / VN;
    SV pre[NG][NC][NV];
    // element j of this thread: its loads for the chunk at c0
    auto load1 = [&](int c0, int j, SV (&q)[NC][NV]) {
        const int c = c0 + cg;  // (channels come in whole groups)
        if constexpr (RES) {
            if (c0 < C0) {
                const int pix = min((tid + 256 * j) >> 2, NPIX - 1);
                const Axis ya = ax[pix / PW], xa = ax[R::PH + pix % PW];
                const int i0 = max(ya.i0, 0) * ws, i1 = max(ya.i1, 0) * ws, j0 = max(xa.i0, 0), j1 = max(xa.i1, 0);
                const int cc = c < C0 ? c : 0, pt = p.src[0].pitch;
                q[0][0] = *(const SV *)(src + (size_t)(i0 + j0) * pt + cc);
                q[1][0] = *(const SV *)(src + (size_t)(i0 + j1) * pt + cc);
                q[2][0] = *(const SV *)(src + (size_t)(i1 + j0) * pt + cc);
                q[3][0] = *(const SV *)(src + (size_t)(i1 + j1) * pt + cc);
            } else {
                const ConvSrc &s1 = p.src[1];
                const ST *sp = (const ST *)s1.ptr + (size_t)b * p.Hi * p.Wi * s1.pitch + s1.coff;
                q[0][0] = *(const SV *)(sp + (c < p.Cin && off[j] >= 0 ? (size_t)off[j] * s1.pitch + c - C0 : 0));
            }
        } else {
#pragma unroll
            for (int k = 0; k < NV; ++k)
                q[0][k] = *(const SV *)(src + (c < p.Cin && off[j] >= 0 ? (size_t)off[j] + c + VN * k : 0));
        }
    };
    auto store1 = [&](int c0, int j, const SV (&q)[NC][NV], int buf) {
        const int pix = (tid + 256 * j) >> 2, c = c0 + cg;
        if (pix >= NPIX) return;
        const bool ok = c < p.Cin && off[j] >= 0;
        vec v;
        if constexpr (RES) {
            if (c0 >= C0) {
#pragma unroll
                for (int i = 0; i < GS; ++i) v[i] = ok ? q[0][0][i] : (T)0;
            } else {
                const Axis ya = ax[pix / PW], xa = ax[R::PH + pix % PW];
                const float ly = ya.lam, lx = xa.lam, wy0 = 1.f - ly, wx0 = 1.f - lx;
                const float w00 = wy0 * wx0, w01 = wy0 * lx, w10 = ly * wx0, w11 = ly * lx;
                float f[GS];
#pragma unroll
                for (int i = 0; i < GS; ++i) {
                    const float x00 = Elem<DT>::load((const T *)&q[0][0] + i), x01 = Elem<DT>::load((const T *)&q[1][0] + i);
                    const float x10 = Elem<DT>::load((const T *)&q[2][0] + i), x11 = Elem<DT>::load((const T *)&q[3][0] + i);
                    f[i] = fmaf(w11, x11, fmaf(w10, x10, fmaf(w01, x01, w00 * x00)));
                }
                v = pack_vec<DT, GS>(f, 0.f);
                if (!ok || c >= C0) {
#pragma unroll
                    for (int i = 0; i < GS; ++i) v[i] = (T)0;
                }
                if (ok && c >= C0) {  // x0, in the group after the map's (its bytes: read here, once a call)
                    const size_t o = (size_t)b * p.Hi * p.Wi + off[j];
                    v[0] = Elem<DT>::make(p.src[1].scale0 * (float)((const uint8_t *)p.src[1].ptr)[o]);
                    v[1] = Elem<DT>::make((float)p.src[1].img[o] * (1.0f / 256.0f));
                }
            }
        } else if constexpr (F32SRC) {
            float f[GS];
#pragma unroll
            for (int i = 0; i < GS; ++i) f[i] = ok ? q[0][i / VN][i % VN] : 0.f;
            v = pack_vec<DT, GS>(f, 0.f);
        } else {
#pragma unroll
            for (int i = 0; i < GS; ++i) v[i] = ok ? q[0][i / VN][i % VN] : (T)0;
        }
        *(vec *)&patch[buf][pix * KCP + cg] = v;
    };
    auto fetch = [&](int c0) {
#pragma unroll
        for (int j = 0; j < NG; ++j) load1(c0, j, pre[j]);
    };
    auto commit = [&](int c0, int buf) {
#pragma unroll
        for (int j = 0; j < NG; ++j) store1(c0, j, pre[j], buf);
        if constexpr (NG < NE) {
#pragma unroll
            for (int j = NG; j < NE; ++j) load1(c0, j, pre[j - NG]);
#pragma unroll
            for (int j = NG; j < NE; ++j) store1(c0, j, pre[j - NG], buf);
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
    for (int c0 = 0; c0 < p.Cin; c0 += KCB) {
        vec a[KS * KS][NB];
        const int wc = c0 + g * GS;
        const bool win = wc < p.cin_pad;
#pragma unroll
        for (int t = 0; t < KS * KS; ++t)
#pragma unroll
            for (int n = 0; n < NB; ++n)
                a[t][n] = *(const vec *)(wpk + ((size_t)t * p.n_pad + nrow[n]) * p.cin_pad + (win ? wc : 0));
        if (NBUF == 1 && c0) __syncthreads();
        commit(c0, buf);
        __syncthreads();
        if (c0 + KCB < p.Cin) fetch(c0 + KCB);
        if (!win) {
#pragma unroll
            for (int t = 0; t < KS * KS; ++t)
#pragma unroll
                for (int n = 0; n < NB; ++n)
#pragma unroll
                    for (int i = 0; i < GS; ++i) a[t][n][i] = (T)0;
        }
        const T *pb = patch[buf] + (wave * MB * S * PW + r16 * S) * KCP + g * GS;
#pragma unroll
        for (int iy = 0; iy < (MB - 1) * S + KS; ++iy)
#pragma unroll
            for (int v = 0; v < KS; ++v) {
                const vec x = *(const vec *)(pb + (iy * PW + v) * KCP);
#pragma unroll
                for (int m = 0; m < MB; ++m) {
                    const int u = iy - m * S;
                    if (u < 0 || u >= KS) continue;
#pragma unroll
                    for (int n = 0; n < NB; ++n) acc[m][n] = M::run(a[u * KS + v][n], x, acc[m][n]);
                }
            }
        if (NBUF == 2) buf ^= 1;
    }
    // ---- bias, activation, backward terms and the store -------------------------
    float bias[NB][4];
#pragma unroll
    for (int n = 0; n < NB; ++n) conv_bias4<DT>(p, n0 + 16 * n + 4 * g, bias[n]);
    const int ox = ox0 + r16;
    if (ox >= p.Wo) return;
#pragma unroll
    for (int m = 0; m < MB; ++m) {
        const int oy = oy0 + wave * MB + m;
        if (oy >= p.Ho) break;
        const size_t pix = ((size_t)b * p.Ho + oy) * p.Wo + ox;
#pragma unroll
        for (int n = 0; n < NB; ++n) {
            const float v[4] = {acc[m][n][0], acc[m][n][1], acc[m][n][2], acc[m][n][3]};
            conv_epilogue<DT>(p, pix, n0 + 16 * n + 4 * g, v, bias[n]);
        }
    }
}

template <int DT, int KS, int S, int MB, int NB>
sv_status launch_r(const ConvParams &p, hipStream_t st) {
    const int tx = cdiv(p.Wo, 16), ty = cdiv(p.Ho, 4 * MB), ntn = cdiv(p.Cout, NB * 16);
    const long long n = (long long)p.B * tx * ty * ntn;
    auto run = [&](auto *fn) {
        hipLaunchKernelGGL(fn, dim3((unsigned)n), dim3(256), 0, st, p, tx, ty, ntn);
    };
    bool done = false;
    if constexpr (KS == 3 && S == 1 && NB == 1 && DT != SV_F16) {
        if (p.src[0].kind == SRC_RESIZE) {
            run(k_conv_rows<DT, KS, S, MB, NB, RM_RESIZE>);
            done = true;
        }
    }
    if constexpr (DT != SV_F32) {
        if (!done && p.src[0].sdt == 1 + SV_F32) {
            run(k_conv_rows<DT, KS, S, MB, NB, RM_F32>);
            done = true;
        }
    }
    if (!done) run(k_conv_rows<DT, KS, S, MB, NB, RM_OWN>);
    SV_LAUNCH_CHECK("k_conv_rows");
    return SV_OK;
}

int rows_nb(int ks, int cout) { return ks == 5 || cout <= 16 ? 1 : 2; }

// Rows a wave for this launch, 0: the general kernel.  More rows share a weight's
// and an input's reads, as long as the launch keeps a workgroup for nearly every
// CU (16 BF16 maps 156x47, 40 -> 8 channels of 5x5: four rows 15.3 us, two 19.7, one
// 29.5; 78x24, 80 -> 16, 240 workgroups at two rows: 12.0, one 16.2, general 12.7;
// stride 2, 64 -> 16: two rows 40.5, one 60.3).  One row pays only in FP32, where
// the matrix steps are the longer part (4 maps 64x32, 16 -> 32 channels: 7.7 us, general 13.6).
int rows_of(int dtype, int ks, int stride, const ConvParams &p) {
    const int nb = rows_nb(ks, p.Cout);
    auto wgs = [&](int mb) { return (long long)p.B * cdiv(p.Wo, 16) * cdiv(p.Ho, 4 * mb) * cdiv(p.Cout, nb * 16); };
    if (wgs(1) >= (1ll << 31)) return 0;
    if (stride == 1 && wgs(4) >= 256) return 4;
    if (wgs(2) >= 200) return 2;
    return dtype == SV_F32 && wgs(1) >= 128 ? 1 : 0;
}

template <int DT, int KS, int S, int NB>
sv_status launch_m(int mb, const ConvParams &p, hipStream_t st) {
    if constexpr (S == 1)
        if (mb == 4) return launch_r<DT, KS, S, 4, NB>(p, st);
    return mb == 2 ? launch_r<DT, KS, S, 2, NB>(p, st) : launch_r<DT, KS, S, 1, NB>(p, st);
}

template <int DT>
sv_status launch_d(int ks, int stride, int mb, const ConvParams &p, hipStream_t st) {
    if (ks == 5) return stride == 1 ? launch_m<DT, 5, 1, 1>(mb, p, st) : launch_m<DT, 5, 2, 1>(mb, p, st);
    if (stride == 1) return p.Cout <= 16 ? launch_m<DT, 3, 1, 1>(mb, p, st) : launch_m<DT, 3, 1, 2>(mb, p, st);
    return p.Cout <= 16 ? launch_m<DT, 3, 2, 1>(mb, p, st) : launch_m<DT, 3, 2, 2>(mb, p, st);
}

}  // namespace

bool conv_rows_fits(int dtype, int ks, int stride, const ConvParams &p) {
    const ConvSrc &s = p.src[0], &s1 = p.src[1];
    if (dtype == SV_I8 || (ks != 5 && ks != 3) || (stride != 1 && stride != 2) || p.tab || p.proj_out || p.ophase ||
        p.ksplit > 1 || p.amax_out)
        return false;
    // vectors of the stored elements, 32-bit offsets
    auto reads = [](const ConvSrc &q, int v) {
        return q.C % 8 == 0 && q.pitch % v == 0 && q.coff % v == 0 && (long long)q.hs * q.ws * q.pitch < (1ll << 31);
    };
    const bool own = !s.sdt || s.sdt - 1 == dtype;
    if (s.kind == SRC_TENSOR && s1.kind == SRC_NONE) {
        if (!reads(s, 4) || !(own || s.sdt - 1 == SV_F32) || p.Hi != s.hs || p.Wi != s.ws) return false;
        // a stride-2 layer's patch is staged again for each 32 channels: four times
        // (64 maps of 78x24 to 128 channels in BF16) it takes as long as the general
        // kernel's wider tiles
        if (ks == 3 && stride == 2 && p.Cout > 64) return false;
    } else if (s.kind == SRC_RESIZE && ks == 3 && stride == 1) {
        // up to 16 channels: wider layers would resize the map again for each 32
        // (64 BF16 maps of 78x24 to 64 channels 112 us against 64, of 156x47 to 32 as long)
        // (F16: the general kernel's last product and its rounding are one step)
        if (p.Cout > 16 || dtype == SV_F16) return false;
        const int kcb = dtype == SV_F32 ? 16 : 32, v = dtype == SV_F32 ? 4 : 8;
        if (!reads(s, v) || !own) return false;
        if (s1.kind == SRC_TENSOR) {
            if (s.C % kcb || !reads(s1, v) || (s1.sdt && s1.sdt - 1 != dtype) || p.Hi != s1.hs || p.Wi != s1.ws) return false;
        } else if (s1.kind != SRC_X0 || s.C % kcb == 0) {
            return false;  // (x0 in a chunk of its own: its taps are packed into that chunk, the general kernel's)
        }
        if ((long long)p.Hi * p.Wi >= (1ll << 31)) return false;
    } else {
        return false;
    }
    return rows_of(dtype, ks, stride, p) > 0;
}

sv_status launch_conv_rows(int dtype, int ks, int stride, const ConvParams &p, hipStream_t st) {
    const int mb = rows_of(dtype, ks, stride, p);
    switch (dtype) {
    case SV_F32: return launch_d<SV_F32>(ks, stride, mb, p, st);
    case SV_BF16: return launch_d<SV_BF16>(ks, stride, mb, p, st);
    case SV_F16: return launch_d<SV_F16>(ks, stride, mb, p, st);
    default: return SV_ERR_DTYPE;
    }
}

}  // namespace sv
