// Backward pass of the refinement network: the exact adjoint of the forward
// pass, for  loss = sum(dout * out) + kl_weight * KL  (Sec. III-B2 in the
// reading documented in sv.h).
//
//   * input gradients (dgrad) reuse the forward implicit-GEMM kernel with the
//     adjoint weight pack (rows = the layer's inputs, kernel flipped), those of
//     the stride-2 encoder layers the transposed convolution (tconv.hip); the
//     epilogue adds the skip-connection gradient and multiplies by the
//     leaky-ReLU derivative of the layer below;
//   * weight gradients (wgrad.hip) are an MFMA GEMM reducing over pixels: every
//     workgroup owns a fixed slice of output tiles and writes its partial sums;
//     a second kernel adds the partials in a fixed order (no float atomics), so
//     gradients are bitwise reproducible;
//   * the bilinear resizes' adjoints are gathers (each coarse pixel collects
//     from the fine pixels whose interpolation reads it), fused with the
//     leaky-ReLU derivative;
//   * the final layer's adjoint is one gather kernel producing the per-tap
//     projection gradient and, through the 9 x (c1+2) weights, the gradient of
//     G0's pre-activation;
//   * the encoder activations are recomputed from x0 (checkpointing).
#include <algorithm>

#include "net.h"
#include "prof.h"

namespace sv {

// The fine indices a coarse index i collects from along one axis (n_c coarse,
// n_f fine samples): the first one, and for k < N the weight with which fine
// index first + k reads i (0 where it does not).  Fine index Y reads i when its
// source position (Y + 1/2) n_c / n_f - 1/2 lies within one of i; positions are
// at least 1 / f apart for n_c = ceil(n_f / f), so N = 2 f + 1 covers the open
// interval of length 2 from the index at or before its start.
template <int N>
__device__ __forceinline__ int adj_axis(int i, int n_c, int n_f, float (&w)[N]) {
    const int num = (2 * i - 1) * n_f - n_c;
    const int first = num <= 0 ? 0 : num / (2 * n_c);
#pragma unroll
    for (int k = 0; k < N; ++k) {
        int i0, i1;
        float lam;
        bilin(min(first + k, n_f - 1), n_c, n_f, i0, i1, lam);
        const float v = (i0 == i ? 1.f - lam : 0.f) + (i1 == i ? lam : 0.f);
        w[k] = first + k < n_f ? v : 0.f;
    }
    return first;
}

// ---------------------------------------------------------------------------
// Bilinear resize adjoint (gather form) times the leaky-ReLU derivative of the
// coarse map:  out[b][i][j][c] = lrelu'(mask[b][i][j][c]) *
//   sum over fine (Y, X) of wy(Y -> i) wx(X -> j) in[b][Y][X][coff + c],
// for the halvings of the network (Hc = ceil(Hf / 2), Wc likewise).
// A workgroup takes one coarse row and TJ columns, TJ C / 4 = 256 where it can;
// the axis weights (an integer division each) are formed once per row and
// column, a thread then reads its 5 x 5 fine positions of four channels, the
// ones without weight as zeros.  Bound by reading the fine map (from L1 and L2
// after the first time).
// (BF16 network, 16 512x256 crops, three levels: 33 us; 77 us with the
// weights recomputed by every thread for every fine pixel of a 9 x 9 window.)
// ---------------------------------------------------------------------------
constexpr int RA_N = 5, RA_TJ = 64;

template <int DT>
__global__ void __launch_bounds__(256)
k_resize_adj(const float *__restrict__ in, int ipitch, int icoff, int Hf, int Wf,
             int Hc, int Wc, int C, int TJ, const void *__restrict__ mask,
             float *__restrict__ out)
{
    __shared__ int xs[RA_TJ];
    __shared__ float wx[RA_TJ][RA_N], wy[RA_N];
    __shared__ int ysh;
    const int i = blockIdx.y, b = blockIdx.z, j0 = blockIdx.x * TJ;
    for (int t = threadIdx.x; t <= TJ; t += 256) {
        float w[RA_N];
        if (t < TJ) {
            xs[t] = adj_axis<RA_N>(min(j0 + t, Wc - 1), Wc, Wf, w);
#pragma unroll
            for (int k = 0; k < RA_N; ++k) wx[t][k] = w[k];
        } else {
            ysh = adj_axis<RA_N>(i, Hc, Hf, w);
#pragma unroll
            for (int k = 0; k < RA_N; ++k) wy[k] = w[k];
        }
    }
    __syncthreads();
    const int cg4 = C / 4, Y0 = ysh;
    for (int e = threadIdx.x; e < TJ * cg4; e += 256) {
        const int jl = e / cg4, cg = e - jl * cg4, j = j0 + jl;
        if (j >= Wc) break;
        const int X0 = xs[jl];
        const size_t pix = ((size_t)b * Hc + i) * Wc + j;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ky = 0; ky < RA_N; ++ky) {
            const float wyk = wy[ky];
            if (wyk == 0.f) continue;  // the whole workgroup's
            const float *row = in + (((size_t)b * Hf + Y0 + ky) * Wf) * ipitch + icoff + 4 * cg;
            f32x4 v[RA_N];
#pragma unroll
            for (int kx = 0; kx < RA_N; ++kx) v[kx] = *(const f32x4 *)(row + (size_t)min(X0 + kx, Wf - 1) * ipitch);
#pragma unroll
            for (int kx = 0; kx < RA_N; ++kx) {
                const float wgt = wyk * wx[jl][kx];
#pragma unroll
                for (int q = 0; q < 4; ++q) acc[q] += wgt * (wgt != 0.f ? v[kx][q] : 0.f);
            }
        }
        const typename Elem<DT>::T *mk = (const typename Elem<DT>::T *)mask + pix * C + 4 * cg;
        f32x4 r;
#pragma unroll
        for (int q = 0; q < 4; ++q) r[q] = acc[q] * (Elem<DT>::load(mk + q) > 0.f ? 1.f : 0.1f);
        *(f32x4 *)(out + pix * C + 4 * cg) = r;
    }
}

static sv_status launch_resize_adj(int dtype, const float *in, int ipitch, int icoff, int Hf, int Wf,
                                   int Hc, int Wc, int C, const void *mask, float *out, int B,
                                   hipStream_t st) {
    const int tj = std::max(4, std::min(RA_TJ, 1024 / C));
    const dim3 grid(cdiv(Wc, tj), Hc, B);
    if (Hc > 65535 || B > 65535) return SV_ERR_SHAPE;
    switch (dtype) {
#define SV_RA(D)                                                                                  \
    case D:                                                                                       \
        hipLaunchKernelGGL(k_resize_adj<D>, grid, dim3(256), 0, st, in, ipitch, icoff, Hf, Wf, Hc, \
                           Wc, C, tj, mask, out);                                                 \
        break;
        SV_RA(SV_F32)
        SV_RA(SV_BF16)
        SV_RA(SV_F16)
#undef SV_RA
    default: return SV_ERR_DTYPE;
    }
    SV_LAUNCH_CHECK("k_resize_adj");
    return SV_OK;
}

// ---------------------------------------------------------------------------
// Final layer adjoint.  With dY = 256 * dout at full resolution, per coarse
// pixel i and tap t = (u, v):
//   dT_t(i) = sum over full-res q inside of A(q, i) * dY(q - (u-1, v-1))
// (zero where q - delta leaves the image), then
//   dpre0[c](i) = lrelu'(G0[c](i)) * sum_t W_F[c][t] dT_t(i)   for c < c1.
// dT is written with FB_DT channels (9 used, the rest 0) for the weight gradient.
//
// A workgroup owns TI x 32 coarse pixels.  A is separable, so it stages the
// tile's region of dout in LDS, sums along the rows for the three column shifts
// (each fine row once, not once per coarse row and tap), then along the columns
// for the three row shifts.  Its share of dout (the tiles' shares
// partition the image) also goes into the bias gradient's sum.
// Bound by its 116 B written a coarse pixel at c1 = 16.
// (16 512x256 crops, f = 2: 30 us; 109 us with 9 taps of every fine pixel and
// its weights per coarse pixel, and 10 us for a pass of its own for the sum.)
// ---------------------------------------------------------------------------
constexpr int FB_TJ = 32, FB_DT = 12;
static inline int fb_ti(int f) { return f <= 2 ? 8 : (f <= 4 ? 4 : 2); }
// rows (columns) of dout a tile of n coarse ones needs: the supports of the
// first and last, shifted by up to one
static inline int fb_span(int n, int f) { return (n + 1) * f + 2 * f + 4; }

template <int DT, int F>
__global__ void __launch_bounds__(256)
k_final_bwd(const float *__restrict__ dout, int H, int W, int h, int w, int TI, int srows, int scols,
            const float *__restrict__ wF, int wf_pitch, int c1,
            const typename Elem<DT>::T *__restrict__ G0, float *__restrict__ dT,
            float *__restrict__ dpre0, float *__restrict__ sum_part)
{
    constexpr int N = 2 * F + 1;  // F >= f
    extern __shared__ __attribute__((aligned(16))) float fsm[];
    float *reg = fsm;                              // [srows][scols] of dout
    float *hv = reg + srows * scols;               // [srows][3][FB_TJ]
    float *wxs = hv + srows * 3 * FB_TJ;           // [FB_TJ][N]
    float *wys = wxs + FB_TJ * N;                  // [TI][N]
    int *xs = (int *)(wys + 8 * N);                // [FB_TJ], [8]
    int *ys = xs + FB_TJ;
    float *red = (float *)(ys + 8);                // [4]
    const int tid = threadIdx.x, b = blockIdx.z;
    const int i0 = blockIdx.y * TI, j0 = blockIdx.x * FB_TJ;
    const int ni = min(TI, h - i0), nj = min(FB_TJ, w - j0);
    if (tid < ni + nj) {
        float wt[N];
        const bool row = tid < ni;
        const int k = row ? tid : tid - ni;
        const int s = adj_axis<N>(row ? i0 + k : j0 + k, row ? h : w, row ? H : W, wt);
        if (row) ys[k] = s;
        else xs[k] = s;
#pragma unroll
        for (int q = 0; q < N; ++q) (row ? wys : wxs)[k * N + q] = wt[q];
    }
    __syncthreads();
    // region of dout: one row / column before the first support to one after the last
    const int R0 = ys[0] - 1, C0 = xs[0] - 1;
    const int nr = min(srows, ys[ni - 1] + N + 1 - R0), nc = min(scols, xs[nj - 1] + N + 1 - C0);
    const float *db = dout + (size_t)b * H * W;
    // its share of the image, which its region covers: from i0 H / h to (i0 + ni) H / h
    const int oy0 = i0 * H / h, oy1 = (i0 + ni) * H / h, ox0 = j0 * W / w, ox1 = (j0 + nj) * W / w;
    float own = 0.f;
    for (int e = tid; e < nr * nc; e += 256) {
        const int r = e / nc, c = e - r * nc;
        const int y = R0 + r, x = C0 + c;
        const bool in = y >= 0 && y < H && x >= 0 && x < W;
        const float v = in ? db[(size_t)y * W + x] : 0.f;
        reg[r * scols + c] = v;
        if (in && y >= oy0 && y < oy1 && x >= ox0 && x < ox1) own += v;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) own += __shfl_xor(own, o);
    if ((tid & 63) == 0) red[tid >> 6] = own;
    __syncthreads();
    if (tid == 0)
        sum_part[((size_t)b * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
    // along the rows: hv[r][v][j] = sum_k wx[j][k] dout[r][xs[j] + k - (v - 1)]
    for (int e = tid; e < nr * FB_TJ; e += 256) {
        const int r = e / FB_TJ, j = e % FB_TJ;
        if (j >= nj) continue;
        const float *row = reg + r * scols + xs[j] - C0 - 1;
        float d[N + 2];
#pragma unroll
        for (int k = 0; k < N + 2; ++k) d[k] = row[min(k, nc - 1 - (xs[j] - C0 - 1))];
        float a[3] = {0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const float wk = wxs[j * N + k];
#pragma unroll
            for (int v = 0; v < 3; ++v) a[v] += wk != 0.f ? wk * d[k + 2 - v] : 0.f;
        }
#pragma unroll
        for (int v = 0; v < 3; ++v) hv[(r * 3 + v) * FB_TJ + j] = a[v];
    }
    __syncthreads();
    // along the columns, then the weights
    for (int e = tid; e < ni * FB_TJ; e += 256) {
        const int il = e / FB_TJ, j = e % FB_TJ;
        if (j >= nj) continue;
        float t[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) t[k] = 0.f;
        const int r0 = ys[il] - R0 - 1;
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const float wk = 256.0f * wys[il * N + k];
            if (wk == 0.f) continue;
#pragma unroll
            for (int u = 0; u < 3; ++u)
#pragma unroll
                for (int v = 0; v < 3; ++v) t[u * 3 + v] += wk * hv[((r0 + k + 2 - u) * 3 + v) * FB_TJ + j];
        }
        const size_t pix = ((size_t)b * h + i0 + il) * w + j0 + j;
        f32x4 *dt = (f32x4 *)(dT + pix * FB_DT);
        dt[0] = f32x4{t[0], t[1], t[2], t[3]};
        dt[1] = f32x4{t[4], t[5], t[6], t[7]};
        dt[2] = f32x4{t[8], 0.f, 0.f, 0.f};
        const typename Elem<DT>::T *g0 = G0 + pix * c1;
        for (int c = 0; c < c1; c += 4) {
            f32x4 r;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float sum = 0.f;
#pragma unroll
                for (int k = 0; k < 9; ++k) sum += wF[(size_t)k * wf_pitch + c + q] * t[k];
                r[q] = sum * (Elem<DT>::load(g0 + c + q) > 0.f ? 1.f : 0.1f);
            }
            *(f32x4 *)(dpre0 + pix * c1 + c) = r;
        }
    }
}

template <int DT, int F>
static void launch_final_bwd_f(const float *dout, int B, int H, int W, int h, int w, int f, const void *wF, int wf_pitch,
                               int c1, const void *G0, float *dT, float *dpre0, float *sum_part, hipStream_t st) {
    const int ti = fb_ti(f), n = 2 * F + 1;
    const int sr = fb_span(ti, f), sc = fb_span(FB_TJ, f);
    const size_t lds = sizeof(float) * ((size_t)sr * sc + sr * 3 * FB_TJ + FB_TJ * n + 8 * n + FB_TJ + 8 + 4);
    hipLaunchKernelGGL((k_final_bwd<DT, F>), dim3(cdiv(w, FB_TJ), cdiv(h, ti), B), dim3(256), lds, st, dout, H, W, h, w,
                       ti, sr, sc, (const float *)wF, wf_pitch, c1, (const typename Elem<DT>::T *)G0, dT, dpre0,
                       sum_part);
}

// tiles of k_final_bwd: its entries of sum_part
static size_t final_bwd_tiles(int B, int h, int w, int f) { return (size_t)B * cdiv(h, fb_ti(f)) * cdiv(w, FB_TJ); }

static sv_status launch_final_bwd(int dtype, const float *dout, int B, int H, int W, int h, int w, int f, const void *wF,
                                  int wf_pitch, int c1, const void *G0, float *dT, float *dpre0, float *sum_part,
                                  hipStream_t st) {
    if (cdiv(h, fb_ti(f)) > 65535 || B > 65535) return SV_ERR_SHAPE;
#define SV_FB(D)                                                                                                       \
    case D:                                                                                                            \
        if (f <= 2) launch_final_bwd_f<D, 2>(dout, B, H, W, h, w, f, wF, wf_pitch, c1, G0, dT, dpre0, sum_part, st);     \
        else if (f <= 4) launch_final_bwd_f<D, 4>(dout, B, H, W, h, w, f, wF, wf_pitch, c1, G0, dT, dpre0, sum_part, st); \
        else launch_final_bwd_f<D, 8>(dout, B, H, W, h, w, f, wF, wf_pitch, c1, G0, dT, dpre0, sum_part, st);            \
        break;
    switch (dtype) {
        SV_FB(SV_F32)
        SV_FB(SV_BF16)
        SV_FB(SV_F16)
    default: return SV_ERR_DTYPE;
    }
#undef SV_FB
    SV_LAUNCH_CHECK("k_final_bwd");
    return SV_OK;
}

// Reparameterisation and KL adjoint: from dz to d[mu | logvar].
__global__ void k_latent_bwd(const float *__restrict__ dz, const float *__restrict__ ml,
                             const float *__restrict__ eps, const float *__restrict__ extra,
                             int npix, int L, float klw, float *__restrict__ dml)
{
    const size_t n = (size_t)npix * L;
    const float inv = 1.0f / (float)n;
    for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < n;
         e += (size_t)gridDim.x * blockDim.x) {
        const size_t p = e / L;
        const int c = (int)(e - p * L);
        const float mu = ml[p * 2 * L + c], lv = ml[p * 2 * L + L + c];
        const float g = dz[e];
        float dlv = klw * 0.5f * (expf(lv) - 1.0f) * inv;
        if (eps) dlv += g * eps[e] * 0.5f * expf(0.5f * lv);
        float dmu = g + klw * mu * inv;
        if (extra) {
            dmu += extra[p * 2 * L + c];
            dlv += extra[p * 2 * L + L + c];
        }
        dml[p * 2 * L + c] = dmu;
        dml[p * 2 * L + L + c] = dlv;
    }
}

// scale * the sum of x[0..n) into *out, in a fixed order: one workgroup, each
// thread a strided run in FP64, then a tree.
__global__ void __launch_bounds__(1024) k_sum_final(const float *__restrict__ x, int n, float scale,
                                                    float *__restrict__ out)
{
    __shared__ double sh[1024];
    double t = 0.0;
    for (int i = threadIdx.x; i < n; i += 1024) t += x[i];
    sh[threadIdx.x] = t;
    __syncthreads();
    for (int k = 512; k > 0; k >>= 1) {
        if ((int)threadIdx.x < k) sh[threadIdx.x] += sh[threadIdx.x + k];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = (float)(scale * sh[0]);
}

// ---------------------------------------------------------------------------
// Workspace of the backward pass (after the forward part holding E1..E3, T).
// ---------------------------------------------------------------------------
// The weight gradient of layer li: its shape and dtype (sources and the
// output gradient are filled in by the caller; only the sources' kinds and
// channel counts matter for the workspace).  The final layer's is a 1x1
// layer with the nine taps as rows, in FP32.
static WgradJob wgrad_job(const NetShape &ns, const Levels &lv, int B, int li) {
    static const int lvl_in[NLAYERS] = {0, 1, 2, 3, 3, 2, 1, 0, 0}, lvl_out[NLAYERS] = {1, 2, 3, 3, 3, 2, 1, 0, 0};
    const LayerSpec &s = ns.ly[li];
    WgradJob j{};
    j.dtype = li == L_F ? SV_F32 : ns.dtype;
    j.ks = li == L_F ? 1 : s.k;
    j.stride = s.stride;
    j.B = B;
    j.Hi = lv.h[lvl_in[li]]; j.Wi = lv.w[lvl_in[li]];
    j.Ho = lv.h[lvl_out[li]]; j.Wo = lv.w[lvl_out[li]];
    j.Cout = li == L_F ? 9 : s.cout;
    j.s0.C = s.cin;
    j.s0.kind = li == L_E1 ? SRC_X0 : SRC_TENSOR;
    j.dy_sdt = SV_F32;
    return j;
}

struct BwdLayout {
    size_t dT, dpre0, dG1up, dpre1, dcat1, dpre2, dcat2, dpre3, dz, dML, dpreE3, dpreE2, dpreE1,
        sum, part, total;
};

static BwdLayout bwd_layout(const NetShape &ns, const Levels &lv, int B) {
    BwdLayout l;
    auto px = [&](int k) { return (size_t)B * lv.h[k] * lv.w[k]; };
    const int c1 = ns.c1, c2 = ns.c2, c3 = ns.c3, L = ns.L;
    size_t o = 0;
    auto take = [&](size_t floats) { size_t r = o; o = align256(o + floats * sizeof(float)); return r; };
    l.dT = take(px(0) * FB_DT);
    l.dpre0 = take(px(0) * c1);
    l.dG1up = take(px(0) * c1);
    l.dpre1 = take(px(1) * c1);
    l.dcat1 = take(px(1) * (c2 + c1));
    l.dpre2 = take(px(2) * c2);
    l.dcat2 = take(px(2) * (c3 + c2));
    l.dpre3 = take(px(3) * c3);
    l.dz = take(px(3) * L);
    l.dML = take(px(3) * 2 * L);
    l.dpreE3 = take(px(3) * c3);
    l.dpreE2 = take(px(2) * c2);
    l.dpreE1 = take(px(1) * c1);
    l.sum = take(final_bwd_tiles(B, lv.h[0], lv.w[0], ns.f));
    // the partial sums of the largest weight gradient (layers run one after another)
    size_t mx = 0;
    for (int li = 0; li < NLAYERS; ++li) mx = std::max(mx, wgrad_part_floats(wgrad_job(ns, lv, B, li)));
    l.part = take(mx);
    l.total = o;
    return l;
}

size_t net_bwd_workspace(const NetShape &ns, const Levels &lv, int B) {
    return bwd_layout(ns, lv, B).total;
}

static ConvSrc bsrc(const void *p, int kind, int C, int pitch, int coff, int hs, int ws, int sdt) {
    ConvSrc s{};
    s.ptr = p; s.kind = kind; s.C = C; s.pitch = pitch; s.coff = coff; s.hs = hs; s.ws = ws;
    s.sdt = sdt;
    return s;
}

#define SV_TRY(x)                       \
    do {                                \
        sv_status r_ = (x);             \
        if (r_ != SV_OK) return r_;     \
    } while (0)

// Input gradient of layer li through the forward conv kernel and the adjoint pack.
static sv_status dgrad(const NetShape &ns, const void *packed, int li, ConvSrc dy, int B, int Hi,
                       int Wi, int cout_needed, float *out, int out_pitch, const float *add,
                       int add_pitch, int add_coff, const void *mask, int mask_pitch, hipStream_t st) {
    ConvParams p{};
    p.src[0] = dy;
    p.B = B; p.Hi = Hi; p.Wi = Wi; p.Ho = Hi; p.Wo = Wi;
    p.Cin = dy.C;
    p.Cout = cout_needed;
    p.cin_pad = ns.bcin_pad[li];
    p.n_pad = ns.bn_pad[li];
    p.wpk = (const char *)packed + ns.bw_off[li];
    p.out = out; p.out_pitch = out_pitch; p.out_f32 = 1;
    p.add = add; p.add_pitch = add_pitch; p.add_coff = add_coff;
    p.mask = mask; p.mask_pitch = mask_pitch;
    p.mask_lo = 0; p.mask_hi = cout_needed;
    const int ks = ns.ly[li].k;
    if (dy.kind == SRC_ZINS && tconv_fits(ns.dtype, ks, p)) return launch_tconv(ns.dtype, ks, p, st);
    const int cfg = ks == 3 ? conv_default_tile(ns.dtype, 1, dy.C, cout_needed, B, Hi, Wi)
                            : (cout_needed <= 16 ? T4_16 : (cout_needed <= 32 ? T4_32 : T4_64));
    return launch_conv(ns.dtype, ks, 1, cfg, p, st);
}

sv_status net_backward(const NetShape &ns, const void *packed, const void *saved, int B, int H,
                       int W, const float *eps, const float *dout, const float *dml_extra,
                       float klw, float *grad, void *ws, hipStream_t st) {
    const Levels lv = net_levels(ns, H, W);
    const ActLayout a = net_act_layout(ns, lv, B);
    const BwdLayout bl = bwd_layout(ns, lv, B);
    char *w = (char *)ws;
    char *bw = w + a.ws_fwd;
    const char *sv_ = (const char *)saved;
    auto F = [&](size_t off) { return (float *)(bw + off); };
    const int c1 = ns.c1, c2 = ns.c2, c3 = ns.c3, L = ns.L, dt = ns.dtype;
    const uint8_t *disp = (const uint8_t *)(sv_ + a.disp), *img = (const uint8_t *)(sv_ + a.img);
    const float *ML = (const float *)(sv_ + a.ML);
    const void *Z = sv_ + a.Z, *G3 = sv_ + a.G3, *G2 = sv_ + a.G2, *G1 = sv_ + a.G1, *G0 = sv_ + a.G0;
    void *E1 = w + a.E1, *E2 = w + a.E2, *E3 = w + a.E3;
    const int *h = lv.h, *wd = lv.w;
    const ConvSrc none{};
    ConvSrc x0{};
    x0.ptr = disp; x0.img = img; x0.kind = SRC_X0; x0.C = 2; x0.hs = h[0]; x0.ws = wd[0];
    x0.scale0 = (float)ns.f / 256.0f;
    auto T_ = [&](const void *p, int C, int k) { return bsrc(p, SRC_TENSOR, C, C, 0, h[k], wd[k], 0); };
    auto Rz = [&](const void *p, int C, int k) { return bsrc(p, SRC_RESIZE, C, C, 0, h[k], wd[k], 0); };
    auto Gf = [&](float *p, int C, int pitch, int k) { return bsrc(p, SRC_TENSOR, C, pitch, 0, h[k], wd[k], SDT_F32); };
    float *part = F(bl.part);
    float *gl[NLAYERS];
    for (int i = 0; i < NLAYERS; ++i) gl[i] = grad + ns.p_off[i];
    // layer li's weight and bias gradient into its canonical slice
    auto wgrad = [&](int li, ConvSrc s0, ConvSrc s1, const float *dy, int dy_pitch) {
        WgradJob j = wgrad_job(ns, lv, B, li);
        j.s0 = s0; j.s1 = s1;
        j.dy = dy; j.dy_pitch = dy_pitch;
        const LayerSpec &s = ns.ly[li];
        GradMap m{};
        m.kind = li == L_F ? GM_TAPROWS : (li == L_E1 ? GM_X0 : GM_OIHW);
        m.cin = s.cin;
        m.kk = li == L_F ? 9 : s.k * s.k;
        m.nbias = li == L_F ? 0 : s.cout;
        return launch_wgrad(j, m, part, gl[li], gl[li] + (size_t)s.cout * s.cin * s.k * s.k, st);
    };

    // ---- recompute the encoder ----------------------------------------------------
    {
        auto fwd = [&](int li, ConvSrc s, int ki, int ko, void *out, int cout) {
            ConvParams p{};
            p.src[0] = s;
            p.B = B; p.Hi = h[ki]; p.Wi = wd[ki]; p.Ho = h[ko]; p.Wo = wd[ko];
            p.Cin = s.C; p.Cout = cout;
            p.cin_pad = ns.cin_pad[li]; p.n_pad = ns.n_pad[li];
            p.wpk = (const char *)packed + ns.w_off[li];
            p.bias = (const float *)((const char *)packed + ns.b_off[li]);
            p.out = out; p.out_pitch = cout; p.act = 1;
            return launch_conv(dt, 3, 2, net_default_cfg(ns, li, lv, B), p, st);
        };
        SV_TRY(launch_enc1(dt, disp, img, (float)ns.f / 256.0f, B, h[0], wd[0], h[1], wd[1], c1,
                           (const char *)packed + ns.w_off[L_E1], ns.n_pad[L_E1], ns.cin_pad[L_E1],
                           (const float *)((const char *)packed + ns.b_off[L_E1]), E1, st));
        SV_TRY(fwd(L_E2, T_(E1, c1, 1), 1, 2, E2, c2));
        SV_TRY(fwd(L_E3, T_(E2, c2, 2), 2, 3, E3, c3));
    }

    // ---- final layer -----------------------------------------------------------------
    {
        SV_TRY(launch_final_bwd(dt, dout, B, H, W, h[0], wd[0], ns.f, (const char *)packed + ns.w_off[L_F],
                                ns.cin_pad[L_F], c1, G0, F(bl.dT), F(bl.dpre0), F(bl.sum), st));
        // dW_F from X = [G0, x0] and dT (a 1x1 layer with the 9 taps as outputs), in FP32
        SV_TRY(wgrad(L_F, bsrc(G0, SRC_TENSOR, c1, c1, 0, h[0], wd[0], 1 + dt), x0, F(bl.dT), FB_DT));
        // db_F = 256 * sum(dout)
        hipLaunchKernelGGL(k_sum_final, dim3(1), dim3(1024), 0, st, F(bl.sum),
                           (int)final_bwd_tiles(B, h[0], wd[0], ns.f), 256.0f, gl[L_F] + 9 * (c1 + 2));
        SV_LAUNCH_CHECK("k_sum_final");
    }

    // ---- G0: input [resize(G1), x0] at level 0 -------------------------------------
    SV_TRY(wgrad(L_G0, Rz(G1, c1, 1), x0, F(bl.dpre0), c1));
    SV_TRY(dgrad(ns, packed, L_G0, Gf(F(bl.dpre0), c1, c1, 0), B, h[0], wd[0], c1, F(bl.dG1up), c1,
                 nullptr, 0, 0, nullptr, 0, st));
    SV_TRY(launch_resize_adj(dt, F(bl.dG1up), c1, 0, h[0], wd[0], h[1], wd[1], c1, G1, F(bl.dpre1),
                             B, st));
    // ---- G1: input [resize(G2), E1] at level 1 ---------------------------------------
    SV_TRY(wgrad(L_G1, Rz(G2, c2, 2), T_(E1, c1, 1), F(bl.dpre1), c1));
    SV_TRY(dgrad(ns, packed, L_G1, Gf(F(bl.dpre1), c1, c1, 1), B, h[1], wd[1], c2 + c1, F(bl.dcat1),
                 c2 + c1, nullptr, 0, 0, nullptr, 0, st));
    SV_TRY(launch_resize_adj(dt, F(bl.dcat1), c2 + c1, 0, h[1], wd[1], h[2], wd[2], c2, G2,
                             F(bl.dpre2), B, st));
    // ---- G2: input [resize(G3), E2] at level 2 ---------------------------------------
    SV_TRY(wgrad(L_G2, Rz(G3, c3, 3), T_(E2, c2, 2), F(bl.dpre2), c2));
    SV_TRY(dgrad(ns, packed, L_G2, Gf(F(bl.dpre2), c2, c2, 2), B, h[2], wd[2], c3 + c2, F(bl.dcat2),
                 c3 + c2, nullptr, 0, 0, nullptr, 0, st));
    SV_TRY(launch_resize_adj(dt, F(bl.dcat2), c3 + c2, 0, h[2], wd[2], h[3], wd[3], c3, G3,
                             F(bl.dpre3), B, st));
    // ---- G3 = lrelu(conv1x1(z)) -------------------------------------------------------
    const ConvSrc zsrc = eps ? T_(Z, L, 3) : bsrc(ML, SRC_TENSOR, L, 2 * L, 0, h[3], wd[3], SDT_F32);
    SV_TRY(wgrad(L_G3, zsrc, none, F(bl.dpre3), c3));
    SV_TRY(dgrad(ns, packed, L_G3, Gf(F(bl.dpre3), c3, c3, 3), B, h[3], wd[3], L, F(bl.dz), L,
                 nullptr, 0, 0, nullptr, 0, st));
    // ---- latent: reparameterisation and KL ----------------------------------------------
    {
        const int npix = B * h[3] * wd[3];
        const size_t n = (size_t)npix * L;
        const int blocks = (int)((n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096);
        hipLaunchKernelGGL(k_latent_bwd, dim3(blocks), dim3(256), 0, st, F(bl.dz), ML, eps,
                           dml_extra, npix, L, klw, F(bl.dML));
        SV_LAUNCH_CHECK("k_latent_bwd");
    }
    // ---- HEAD: [mu | logvar] = conv1x1(E3) -------------------------------------------
    SV_TRY(wgrad(L_HEAD, T_(E3, c3, 3), none, F(bl.dML), 2 * L));
    SV_TRY(dgrad(ns, packed, L_HEAD, Gf(F(bl.dML), 2 * L, 2 * L, 3), B, h[3], wd[3], c3,
                 F(bl.dpreE3), c3, nullptr, 0, 0, E3, c3, st));
    // ---- encoder (stride 2): input gradients by the transposed convolution -------------
    SV_TRY(wgrad(L_E3, T_(E2, c2, 2), none, F(bl.dpreE3), c3));
    SV_TRY(dgrad(ns, packed, L_E3, bsrc(F(bl.dpreE3), SRC_ZINS, c3, c3, 0, h[3], wd[3], SDT_F32), B, h[2],
                 wd[2], c2, F(bl.dpreE2), c2, F(bl.dcat2), c3 + c2, c3, E2, c2, st));
    SV_TRY(wgrad(L_E2, T_(E1, c1, 1), none, F(bl.dpreE2), c2));
    SV_TRY(dgrad(ns, packed, L_E2, bsrc(F(bl.dpreE2), SRC_ZINS, c2, c2, 0, h[2], wd[2], SDT_F32), B, h[1],
                 wd[1], c1, F(bl.dpreE1), c1, F(bl.dcat1), c2 + c1, c2, E1, c1, st));
    SV_TRY(wgrad(L_E1, x0, none, F(bl.dpreE1), c1));
    return SV_OK;
}

}  // namespace sv
