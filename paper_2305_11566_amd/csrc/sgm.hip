// Semi-global matching on the census cost (Sec. III-A2, Eqs. (4)-(5)), winner-
// take-all on the aggregated cost (Eq. (6)), the single matching phase
// (Sec. III-A3, Eq. (7)) and a 3 x 3 median filter: the Census + SGM member
// of the paper's matching family (S2 of Sec. IV-C), at the reduced
// resolution.
//
// The matching cost is first written as a uint8 volume.  Path costs (Eq. (4))
// run along the four axis directions: one 16-lane DPP row of a wavefront
// follows one path (four paths per wave); lane l holds the
// disparities d = l * DPL + j, j < DPL, in registers, so d - 1 and d + 1 are
// in the same lane except at the ends of its run, which come from the
// neighbouring lanes by DPP row shifts, and min_k C_r(p - r, k) is a DPP row
// rotate-and-min.  Each direction writes its path costs C_r as uint8 into a
// volume of its own, and the WTA kernel sums the four (Eq. (5)).
#include "common.h"
#include "kernels.h"

namespace sv {

constexpr int SGM_INF = 0x3fff;        // above any path cost (uint8 range)
constexpr int SGM_LANES = 16;          // lanes per path = one DPP row

template <int CTRL>
__device__ __forceinline__ int dpp(int old, int v) {
    return __builtin_amdgcn_update_dpp(old, v, CTRL, 0xf, 0xf, false);
}
// min over the 16 lanes of a DPP row, in every lane of the row
__device__ __forceinline__ int row_min(int v) {
    v = min(v, dpp<0x121>(0, v));  // row_ror:1
    v = min(v, dpp<0x122>(0, v));  // row_ror:2
    v = min(v, dpp<0x124>(0, v));  // row_ror:4
    v = min(v, dpp<0x128>(0, v));  // row_ror:8
    return v;
}

// Matching cost volume C(p, d) (the cost of Eq. (6): Hamming distance of the
// census codes, nbits + 1 where x - d < 0) as uint8 [B][h][w][Dp], Dp = D
// rounded up to a multiple of 4 (the padding is never read as a cost).  One
// workgroup = a row segment of CV_TW pixels; the right census codes it needs,
// [j0 - D + 1, j0 + CV_TW), are staged in LDS once; a thread writes four
// disparities of a pixel as one 32-bit word.
constexpr int CV_TW = 64;
__global__ void __launch_bounds__(256)
k_sgm_cost(const uint64_t *__restrict__ cl, const uint64_t *__restrict__ cr, int h, int w, int D,
           int Dp, int nbits, uint8_t *__restrict__ cost)
{
    __shared__ uint64_t seg[CV_TW + 256];
    const size_t row = ((size_t)blockIdx.z * h + blockIdx.y) * w;
    const int j0 = blockIdx.x * CV_TW;
    const int base = j0 - (D - 1);
    for (int e = threadIdx.x; e < CV_TW + D - 1; e += blockDim.x) {
        const int x = base + e;
        seg[e] = (x >= 0 && x < w) ? cr[row + x] : 0;
    }
    __syncthreads();
    const int ng = Dp / 4;
    for (int e = threadIdx.x; e < CV_TW * ng; e += blockDim.x) {
        const int px = e / ng, g = e - px * ng;
        const int j = j0 + px;
        if (j >= w) continue;
        const uint64_t lv = cl[row + j];
        uint32_t word = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int d = 4 * g + k;
            // column j - d of the right view is seg[px + D - 1 - d]
            const uint32_t c = d >= D ? 0u
                             : (j - d < 0 ? (uint32_t)(nbits + 1)
                                          : (uint32_t)__popcll(lv ^ seg[px + D - 1 - (d < D ? d : 0)]));
            word |= c << (8 * k);
        }
        *(uint32_t *)(cost + (row + j) * Dp + 4 * g) = word;
    }
}

// Path p of npath: directions 0 (left to right) and 1 (right to left) run
// along rows, 2 (top to bottom) and 3 (bottom to top) along columns;
// vol[dir][b][y][x][Dp].  The step's costs are loaded SGM_PF steps ahead into
// a ring of registers, so the dependent chain of a step is arithmetic and DPP
// only.
constexpr int SGM_PF = 16;
template <int DPL>
struct CostWords {
    static constexpr int N = DPL >= 4 ? DPL / 4 : 1;
    uint32_t v[N];
    uint32_t ok;  // bit k: word k holds costs (else it is read as zero)
};

// The costs of disparities d0 .. d0 + DPL - 1 of one pixel (p points at d0).
// The loads are unconditional (a word at or past Dp, or of a step past the
// path's end, reads `safe` instead) and the mask is applied where the costs
// are used, so nothing waits for a load until its step comes.
template <int DPL>
__device__ __forceinline__ void load_costs(const uint8_t *__restrict__ p, const uint8_t *safe, bool ok,
                                           int d0, int Dp, CostWords<DPL> &c) {
    c.ok = 0;
    if constexpr (DPL >= 4) {
#pragma unroll
        for (int k = 0; k < DPL / 4; ++k) {
            const bool okk = ok && d0 + 4 * k < Dp;
            c.v[k] = *(const uint32_t *)(okk ? p + 4 * k : safe);
            c.ok |= (uint32_t)okk << k;
        }
    } else if constexpr (DPL == 2) {
        c.v[0] = *(const uint16_t *)(ok ? p : safe);
        c.ok = ok;
    } else {
        c.v[0] = *(ok ? p : safe);
        c.ok = ok;
    }
}

template <int DPL>
__global__ void __launch_bounds__(64)
k_sgm_paths(const uint8_t *__restrict__ cost, int B, int h, int w, int D, int Dp, int P1, int P2,
            uint8_t *__restrict__ vol, uint8_t *__restrict__ sink)
{
    const int lane = threadIdx.x & (SGM_LANES - 1);
    const int path = blockIdx.x * 4 + (threadIdx.x >> 4);
    const int nrow = B * h, ncol = B * w;
    const int npath = 2 * nrow + 2 * ncol;
    if (path >= npath) return;  // whole DPP rows leave together
    int dir, line;
    if (path < 2 * nrow) { dir = path / nrow; line = path - dir * nrow; }
    else { const int q = path - 2 * nrow; dir = 2 + q / ncol; line = q - (dir - 2) * ncol; }
    int b, x0, y0, dx, dy, len;
    if (dir < 2) {
        b = line / h; y0 = line - b * h;
        dx = dir == 0 ? 1 : -1; dy = 0;
        x0 = dir == 0 ? 0 : w - 1;
        len = w;
    } else {
        b = line / w; x0 = line - b * w;
        dx = 0; dy = dir == 2 ? 1 : -1;
        y0 = dir == 2 ? 0 : h - 1;
        len = h;
    }
    const size_t plane = (size_t)h * w;
    const uint8_t *cb = cost + (size_t)b * plane * Dp;
    uint8_t *vb = vol + ((size_t)dir * B + b) * plane * Dp;
    const int d0 = lane * DPL;
    const bool lane_ok = d0 < Dp;
    // pixel offset (in pixels) of step s
    const long long step_px = (long long)dy * w + dx;
    const long long px0 = (long long)y0 * w + x0;
    // words of lanes past Dp are stored to a per-lane sink (never read), so
    // stores, like loads, need no branch
    uint8_t *my_sink = sink + (size_t)(threadIdx.x & 63) * 64;

    CostWords<DPL> ring[SGM_PF];
#pragma unroll
    for (int k = 0; k < SGM_PF; ++k)
        load_costs<DPL>(cb + (size_t)(px0 + (long long)(k < len ? k : 0) * step_px) * Dp + d0, cb,
                        lane_ok && k < len, d0, Dp, ring[k]);

    int prev[DPL];
#pragma unroll
    for (int j = 0; j < DPL; ++j) prev[j] = SGM_INF;
    int mprev = 0;
    // one step s of the path, its costs in ring slot k (refilled with step s + SGM_PF)
    auto step = [&](int k, int s) {
        int c[DPL];
#pragma unroll
        for (int j = 0; j < DPL; ++j) {
            const int q = DPL >= 4 ? j / 4 : 0;
            const uint32_t word = ((ring[k].ok >> q) & 1u) ? ring[k].v[q] : 0u;
            const int sh = DPL >= 4 ? 8 * (j % 4) : 8 * j;
            c[j] = d0 + j < D ? (int)((word >> sh) & 0xffu) : SGM_INF;
        }
        const int sn = s + SGM_PF;
        load_costs<DPL>(cb + (size_t)(px0 + (long long)(sn < len ? sn : 0) * step_px) * Dp + d0, cb,
                        lane_ok && sn < len, d0, Dp, ring[k]);
        int cur[DPL];
        if (s == 0) {
#pragma unroll
            for (int j = 0; j < DPL; ++j) cur[j] = c[j];
        } else {
            const int from_left = dpp<0x111>(SGM_INF, prev[DPL - 1]);  // row_shr:1: lane - 1
            const int from_right = dpp<0x101>(SGM_INF, prev[0]);       // row_shl:1: lane + 1
#pragma unroll
            for (int j = 0; j < DPL; ++j) {
                const int lft = j > 0 ? prev[j - 1] : from_left;
                const int rgt = j + 1 < DPL ? prev[j + 1] : from_right;
                int m = min(prev[j], min(lft, rgt) + P1);
                m = min(m, mprev + P2);
                cur[j] = c[j] >= SGM_INF ? SGM_INF : c[j] + m - mprev;
            }
        }
        int mn = cur[0];
#pragma unroll
        for (int j = 1; j < DPL; ++j) mn = min(mn, cur[j]);
        mprev = row_min(mn);
        uint8_t *o = vb + (size_t)(px0 + (long long)s * step_px) * Dp + d0;
        if constexpr (DPL >= 4) {
#pragma unroll
            for (int q = 0; q < DPL / 4; ++q) {
                uint32_t word = 0;
#pragma unroll
                for (int t = 0; t < 4; ++t) word |= (uint32_t)(cur[4 * q + t] & 0xff) << (8 * t);
                const bool okq = lane_ok && d0 + 4 * q < Dp;
                *(uint32_t *)(okq ? o + 4 * q : my_sink + 4 * q) = word;
            }
        } else if constexpr (DPL == 2) {
            *(uint16_t *)(lane_ok ? o : my_sink) = (uint16_t)((cur[0] & 0xff) | ((cur[1] & 0xff) << 8));
        } else {
            *(lane_ok ? o : my_sink) = (uint8_t)cur[0];
        }
#pragma unroll
        for (int j = 0; j < DPL; ++j) prev[j] = cur[j];
    };
    int s0 = 0;
    for (; s0 + SGM_PF <= len; s0 += SGM_PF) {
#pragma unroll
        for (int k = 0; k < SGM_PF; ++k) step(k, s0 + k);
    }
#pragma unroll
    for (int k = 0; k < SGM_PF; ++k)
        if (s0 + k < len) step(k, s0 + k);
}

// Aggregated cost (Eq. (5)) and winner-take-all (Eq. (6)), lowest d on ties;
// the four volumes are [B][h][w][Dp].
__global__ void __launch_bounds__(256)
k_sgm_wta(const uint8_t *__restrict__ vol, size_t nvox, int D, int Dp, size_t npix,
          uint8_t *__restrict__ disp)
{
    for (size_t p = blockIdx.x * (size_t)blockDim.x + threadIdx.x; p < npix;
         p += (size_t)gridDim.x * blockDim.x) {
        const uint8_t *v0 = vol + p * Dp, *v1 = v0 + nvox, *v2 = v1 + nvox, *v3 = v2 + nvox;
        int best = 0x7fffffff, bd = 0;
        for (int d = 0; d < D; d += 4) {
            const uint32_t a = *(const uint32_t *)(v0 + d), bq = *(const uint32_t *)(v1 + d);
            const uint32_t cq = *(const uint32_t *)(v2 + d), dq = *(const uint32_t *)(v3 + d);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int sh = 8 * k;
                const int s = (int)((a >> sh) & 0xff) + (int)((bq >> sh) & 0xff) +
                              (int)((cq >> sh) & 0xff) + (int)((dq >> sh) & 0xff);
                if (d + k < D && s < best) { best = s; bd = d + k; }
            }
        }
        disp[p] = (uint8_t)bd;
    }
}

// Single matching phase (Eq. (7)) with nearest-valid filling, one wave per
// row.  The target column of x is x - D(x); x is invalid when a pixel x + k,
// 0 < k < D, has the same target column (the left pixel of such a pair is
// the one hidden in the target view).  Validity is kept as one 64-bit ballot
// per 64 pixels; each invalid pixel takes the nearest valid value of its row
// (the smaller one at equal distances).  The row is staged in LDS.
constexpr int SMP_MAXW = 16384;
__global__ void __launch_bounds__(64)
k_smp(const uint8_t *__restrict__ disp, int B, int h, int w, int D, uint8_t *__restrict__ out)
{
    __shared__ uint8_t row[SMP_MAXW];
    __shared__ uint64_t valid[SMP_MAXW / 64];
    const int lane = threadIdx.x;
    const size_t base = (size_t)blockIdx.x * w;  // row blockIdx.x of B * h
    for (int x = lane; x < w; x += 64) row[x] = disp[base + x];
    __syncthreads();
    const int nch = (w + 63) / 64;
    for (int ch = 0; ch < nch; ++ch) {
        const int x = ch * 64 + lane;
        bool ok = x < w;
        if (ok) {
            const int t = x - row[x];
            for (int k = 1; k < D && x + k < w; ++k)
                if (x + k - row[x + k] == t) { ok = false; break; }
        }
        const uint64_t m = __ballot(ok);
        if (lane == 0) valid[ch] = m;
    }
    __syncthreads();
    bool any = false;
    for (int ch = 0; ch < nch; ++ch) any |= valid[ch] != 0;
    for (int x = lane; x < w; x += 64) {
        const int ch = x >> 6, bit = x & 63;
        uint8_t v = row[x];
        if (any && !((valid[ch] >> bit) & 1)) {
            // nearest valid index below x and above x (-1 / w when none)
            int lo = -1, hi = w;
            uint64_t mb = valid[ch] & ((bit ? (~0ull >> (64 - bit)) : 0ull));
            for (int c = ch; c >= 0; --c) {
                const uint64_t mm = c == ch ? mb : valid[c];
                if (mm) { lo = c * 64 + 63 - __clzll(mm); break; }
            }
            uint64_t ma = bit == 63 ? 0ull : valid[ch] & (~0ull << (bit + 1));
            for (int c = ch; c < nch; ++c) {
                const uint64_t mm = c == ch ? ma : valid[c];
                if (mm) { hi = c * 64 + __ffsll((unsigned long long)mm) - 1; break; }
            }
            const int dl = lo >= 0 ? x - lo : 0x7fffffff, dr = hi < w ? hi - x : 0x7fffffff;
            if (dl < dr) v = row[lo];
            else if (dr < dl) v = row[hi];
            else v = min(row[lo], row[hi]);
        }
        out[base + x] = v;
    }
}

// 3 x 3 median, borders replicated (median of nine by a fixed exchange network).
__device__ __forceinline__ void sort2(int &a, int &b) {
    const int t = min(a, b);
    b = max(a, b);
    a = t;
}
__global__ void __launch_bounds__(256)
k_median3(const uint8_t *__restrict__ in, int B, int h, int w, uint8_t *__restrict__ out)
{
    const size_t n = (size_t)B * h * w;
    for (size_t p = blockIdx.x * (size_t)blockDim.x + threadIdx.x; p < n;
         p += (size_t)gridDim.x * blockDim.x) {
        const int j = (int)(p % w);
        const size_t r = p / w;
        const int i = (int)(r % h);
        const uint8_t *img = in + (r - i) * w;
        const int ys[3] = {max(i - 1, 0), i, min(i + 1, h - 1)};
        const int xs[3] = {max(j - 1, 0), j, min(j + 1, w - 1)};
        int v[9];
#pragma unroll
        for (int u = 0; u < 3; ++u)
#pragma unroll
            for (int t = 0; t < 3; ++t) v[u * 3 + t] = img[(size_t)ys[u] * w + xs[t]];
        // Paeth's 19-exchange median-of-nine network
        sort2(v[1], v[2]); sort2(v[4], v[5]); sort2(v[7], v[8]);
        sort2(v[0], v[1]); sort2(v[3], v[4]); sort2(v[6], v[7]);
        sort2(v[1], v[2]); sort2(v[4], v[5]); sort2(v[7], v[8]);
        sort2(v[0], v[3]); sort2(v[5], v[8]); sort2(v[4], v[7]);
        sort2(v[3], v[6]); sort2(v[1], v[4]); sort2(v[2], v[5]);
        sort2(v[4], v[7]); sort2(v[4], v[2]); sort2(v[6], v[4]);
        sort2(v[4], v[2]);
        out[p] = (uint8_t)v[4];
    }
}

static inline int sgm_dpad(int D) { return (D + 3) & ~3; }

// the cost volume, the four path-cost volumes, and a 4 KB sink for the
// stores of lanes past the padded disparity range
constexpr size_t SGM_SINK = 4096;
size_t sgm_volume_bytes(int B, int h, int w, int D) {
    return (size_t)5 * B * h * w * sgm_dpad(D) + SGM_SINK;
}

// Path sweeps + aggregation / WTA on a uint8 cost volume already in the
// workspace (ws: cost, four path volumes, sink).
static sv_status sgm_from_cost(int B, int h, int w, int D, int P1, int P2, uint8_t *ws, uint8_t *disp,
                               hipStream_t s)
{
    const int Dp = sgm_dpad(D);
    const size_t nvox = (size_t)B * h * w * Dp;
    const uint8_t *cost = ws;
    uint8_t *vol = ws + nvox, *sink = ws + 5 * nvox;
    const int npath = 2 * B * h + 2 * B * w;
    const dim3 grid(cdiv(npath, 4));
    const int dpl = cdiv(D, SGM_LANES);
#define SV_SGM(N) \
    hipLaunchKernelGGL(k_sgm_paths<N>, grid, dim3(64), 0, s, cost, B, h, w, D, Dp, P1, P2, vol, sink)
    if (dpl <= 1) SV_SGM(1);
    else if (dpl <= 2) SV_SGM(2);
    else if (dpl <= 4) SV_SGM(4);
    else if (dpl <= 8) SV_SGM(8);
    else SV_SGM(16);
#undef SV_SGM
    SV_LAUNCH_CHECK("k_sgm_paths");
    const size_t npix = (size_t)B * h * w;
    const int blocks = (int)std::min<size_t>((npix + 255) / 256, 8192);
    hipLaunchKernelGGL(k_sgm_wta, dim3(blocks), dim3(256), 0, s, vol, nvox, D, Dp, npix, disp);
    SV_LAUNCH_CHECK("k_sgm_wta");
    return SV_OK;
}

sv_status launch_sgm(const uint64_t *cl, const uint64_t *cr, int B, int h, int w, int D, int nbits,
                     int P1, int P2, uint8_t *ws, uint8_t *disp, hipStream_t s)
{
    const int Dp = sgm_dpad(D);
    hipLaunchKernelGGL(k_sgm_cost, dim3(cdiv(w, CV_TW), h, B), dim3(256), 0, s, cl, cr, h, w, D, Dp,
                       nbits, ws);
    SV_LAUNCH_CHECK("k_sgm_cost");
    return sgm_from_cost(B, h, w, D, P1, P2, ws, disp, s);
}

// ---------------------------------------------------------------------------
// Zero-mean normalised cross-correlation cost, Eqs. (1)-(3), on the reduced
// images.  With n window pixels (clamped to the image edge) and the exact
// integer window sums SR, SRR, ST, STT, SRT of the reference and target
// values,
//   C = 1 - N / sqrt(A B),  N = n SRT - SR ST,  A = n SRR - SR^2,  B = n STT - ST^2,
// evaluated in FP64 (C = 1 for a flat window, 2 where x - d < 0), and kept as
// q = floor(32 C + 1/2) in 0..64 for the path aggregation.
//
// Bound by integer VALU work.  One workgroup = ZN_TW x ZN_TH pixels, all
// disparities.  The reference tile and the target tile (widened by the
// disparities) are kept in LDS as window columns, the 2 RY + 1 bytes above
// each other packed four to a word, with (SR, 1 / sqrt A) per pixel and
// (ST, 1 / sqrt B) per target pixel formed once.  A thread takes ZN_K adjacent
// pixels and four disparities: a column's products are one v_dot4 a word, the
// window sum SRT slides along the pixels, and lanes run along the disparities
// of a pixel, so stores are contiguous.  q is decided in FP32 from
// 32.5 - 32 N / sqrt(A B), whose error is below 2^-15; where that lies within
// 2^-14 of an integer (about one value in 8000) the thread recomputes the
// sums and decides in FP64, so every q is the FP64 one.
// (16 reduced 1242x375 pairs, D = 48, 9 x 7 windows: 41 us; 317 us with three 63-term
// sums and an FP64 square root and division a value.)
// ---------------------------------------------------------------------------
constexpr int ZN_TW = 64, ZN_TH = 4, ZN_K = 8;

// Every sum and product fits 32 bits for windows to 9 x 9: n SRR <= 81 * 81 * 255^2.
__device__ __forceinline__ int zncc_exact(int n, int SR, int SRR, int ST, int STT, int SRT) {
    const int N = n * SRT - SR * ST, A = n * SRR - SR * SR, Bv = n * STT - ST * ST;
    double C;
    if (A == 0 || Bv == 0) C = 1.0;
    else C = 1.0 - (double)N / sqrt((double)A * (double)Bv);
    return (int)floor(32.0 * C + 0.5);
}

template <int RX, int RY>
__global__ void __launch_bounds__(256)
k_zncc_cost(const uint8_t *__restrict__ ll, const uint8_t *__restrict__ lr, int h, int w, int D,
            int Dp, int words, uint8_t *__restrict__ cost)
{
    constexpr int WY = 2 * RY + 1, NW = (2 * RX + 1) * WY;
    constexpr int NQ = (WY + 3) / 4;           // words of a window column
    constexpr int NC = ZN_K + 2 * RX;          // columns of a thread's run
    constexpr int PWR = ZN_TW + 2 * RX;
    constexpr int PWT = ZN_TW + 2 * RX + 255;  // at D = 256
    struct Sum { int s; float r; };            // window sum, 1 / sqrt(n * sum of squares - sum^2) or 0
    __shared__ __attribute__((aligned(8))) uint32_t cr[ZN_TH][PWR][NQ], ct[ZN_TH][PWT][NQ];
    __shared__ Sum sr[ZN_TH][ZN_TW], st[ZN_TH][ZN_TW + 255];
    const int b = blockIdx.z;
    const int i0 = blockIdx.y * ZN_TH, j0 = blockIdx.x * ZN_TW;
    const uint8_t *L = ll + (size_t)b * h * w, *R = lr + (size_t)b * h * w;
    const int nd = (D + 3) / 4, D4 = 4 * nd;
    const int jt = j0 - (D4 - 1);              // target pixel of st[.][0]; ct[.][0] is RX before it
    const int nt = ZN_TW + D4 - 1;
    // window columns, one a thread: its WY + ZN_TH - 1 bytes, then each row's run of WY
    for (int e = threadIdx.x; e < PWR + nt + 2 * RX; e += 256) {
        const bool ref = e < PWR;
        const int c = ref ? e : e - PWR;
        const int x = min(max((ref ? j0 : jt) - RX + c, 0), w - 1);
        const uint8_t *img = (ref ? L : R) + x;
        uint32_t v[WY + ZN_TH - 1];
#pragma unroll
        for (int k = 0; k < WY + ZN_TH - 1; ++k) v[k] = img[(size_t)min(max(i0 + k - RY, 0), h - 1) * w];
#pragma unroll
        for (int y = 0; y < ZN_TH; ++y)
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                uint32_t word = 0;
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (4 * q + k < WY) word |= v[y + 4 * q + k] << (8 * k);
                if (ref) cr[y][c][q] = word;
                else ct[y][c][q] = word;
            }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < ZN_TH * (ZN_TW + nt); e += 256) {
        const int y = e / (ZN_TW + nt), c = e - y * (ZN_TW + nt);
        const bool ref = c < ZN_TW;
        uint32_t s = 0, ss = 0;
#pragma unroll
        for (int dx = 0; dx <= 2 * RX; ++dx)
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const uint32_t v = ref ? cr[y][c + dx][q] : ct[y][c - ZN_TW + dx][q];
                s = __builtin_amdgcn_udot4(v, 0x01010101u, s, false);
                ss = __builtin_amdgcn_udot4(v, v, ss, false);
            }
        const int var = NW * (int)ss - (int)s * (int)s;
        const Sum r = {(int)s, var > 0 ? __builtin_amdgcn_rsqf((float)var) : 0.f};
        if (ref) sr[y][c] = r;
        else st[y][c - ZN_TW] = r;
    }
    __syncthreads();
    constexpr int NRUN = ZN_TW / ZN_K;
    for (int item = threadIdx.x; item < ZN_TH * NRUN * nd; item += 256) {
        const int db = item % nd, pr = item / nd;
        const int y = pr / NRUN, x = (pr - y * NRUN) * ZN_K;
        const int i = i0 + y, j = j0 + x, d0 = 4 * db;
        if (i >= h || j >= w) continue;
        // column c of the run against disparity d0 + q is target column c - q + 3 of tc
        uint32_t rc[NC][NQ], tc[NC + 3][NQ];
        const int t0 = x + (D4 - 1) - d0 - 3;
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int k = 0; k < NQ; ++k) rc[c][k] = cr[y][x + c][k];
#pragma unroll
        for (int c = 0; c < NC + 3; ++c)
#pragma unroll
            for (int k = 0; k < NQ; ++k) tc[c][k] = ct[y][t0 + c][k];
        Sum a[ZN_K], t[ZN_K + 3];
#pragma unroll
        for (int k = 0; k < ZN_K; ++k) {
            a[k] = sr[y][x + k];
            a[k].r *= 32.0f;
        }
#pragma unroll
        for (int k = 0; k < ZN_K + 3; ++k) t[k] = st[y][t0 + k];
        uint32_t out[ZN_K], near = 0;
#pragma unroll
        for (int k = 0; k < ZN_K; ++k) out[k] = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int d = d0 + q;
            uint32_t P[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                P[c] = 0;
#pragma unroll
                for (int k = 0; k < NQ; ++k) P[c] = __builtin_amdgcn_udot4(rc[c][k], tc[c - q + 3][k], P[c], false);
            }
            uint32_t S = 0;
#pragma unroll
            for (int c = 0; c < 2 * RX + 1; ++c) S += P[c];
#pragma unroll
            for (int k = 0; k < ZN_K; ++k) {
                if (k) S += P[k + 2 * RX] - P[k - 1];
                const Sum tk = t[k - q + 3];
                // factors below 2^24: full-rate multiplies
                const int N = (int)__umul24(S, NW) - (int)__umul24(a[k].s, tk.s);
                const float v = fmaf(-(float)N, a[k].r * tk.r, 32.5f);
                const float fl = floorf(v);
                uint32_t qv = (uint32_t)(int)fl;
                const bool out_left = j + k < d;
                if (out_left) qv = 64;
                if (d >= D) qv = 0;
                out[k] |= qv << (8 * q);
                // v - fl in [2^-14, 1 - 2^-14]: the FP64 expression has the same floor
                if (fabsf(v - fl - 0.5f) > 0.5f - 0x1p-14f && !out_left) near |= 1u << (8 * q + k);
            }
        }
        while (near) {
            const int bit = __ffs(near) - 1;
            near &= near - 1;
            const int q = bit >> 3, k = bit & 7;
            if (d0 + q >= D) continue;
            int SRR = 0, STT = 0, SRT = 0;
            for (int dx = 0; dx <= 2 * RX; ++dx)
                for (int m = 0; m < NQ; ++m) {
                    const uint32_t rv = cr[y][x + k + dx][m], tv = ct[y][t0 + k - q + 3 + dx][m];
                    SRR = (int)__builtin_amdgcn_udot4(rv, rv, (uint32_t)SRR, false);
                    STT = (int)__builtin_amdgcn_udot4(tv, tv, (uint32_t)STT, false);
                    SRT = (int)__builtin_amdgcn_udot4(rv, tv, (uint32_t)SRT, false);
                }
            const uint32_t v = (uint32_t)zncc_exact(NW, sr[y][x + k].s, SRR, st[y][t0 + k - q + 3].s, STT, SRT);
#pragma unroll
            for (int kk = 0; kk < ZN_K; ++kk)
                if (kk == k) out[kk] = (out[kk] & ~(0xffu << (8 * q))) | (v << (8 * q));
        }
        uint8_t *o = cost + (((size_t)b * h + i) * w + j) * Dp + d0;
#pragma unroll
        for (int k = 0; k < ZN_K; ++k) {
            if (j + k >= w) break;
            if (words) {
                *(uint32_t *)(o + (size_t)k * Dp) = out[k];
            } else {
                for (int q = 0; q < 4; ++q)
                    if (d0 + q < Dp) o[(size_t)k * Dp + q] = (uint8_t)(out[k] >> (8 * q));
            }
        }
    }
}

bool zncc_window_supported(int win_w, int win_h) {
    const int rx = (win_w - 1) / 2, ry = (win_h - 1) / 2;
    if (win_w % 2 == 0 || win_h % 2 == 0) return false;
    return (rx == 1 && ry == 1) || (rx == 2 && ry == 2) || (rx == 3 && ry == 3) || (rx == 4 && ry == 3) ||
           (rx == 3 && ry == 4) || (rx == 4 && ry == 4) || (rx == 2 && ry == 1) || (rx == 1 && ry == 2);
}

sv_status launch_zncc_cost(const uint8_t *ll, const uint8_t *lr, int B, int h, int w, int D, int Dp,
                           int win_w, int win_h, uint8_t *cost, hipStream_t s)
{
    const dim3 grid(cdiv(w, ZN_TW), cdiv(h, ZN_TH), B);
    const int rx = (win_w - 1) / 2, ry = (win_h - 1) / 2;
    // four disparities as one word where every pixel's row of costs is aligned
    const int words = Dp % 4 == 0 && (uintptr_t)cost % 4 == 0;
#define SV_ZN(X, Y)                                                                                \
    if (rx == X && ry == Y) {                                                                      \
        hipLaunchKernelGGL((k_zncc_cost<X, Y>), grid, dim3(256), 0, s, ll, lr, h, w, D, Dp, words, cost); \
        SV_LAUNCH_CHECK("k_zncc_cost");                                                            \
        return SV_OK;                                                                              \
    }
    SV_ZN(1, 1) SV_ZN(2, 2) SV_ZN(3, 3) SV_ZN(4, 3) SV_ZN(3, 4) SV_ZN(4, 4) SV_ZN(2, 1) SV_ZN(1, 2)
#undef SV_ZN
    return SV_ERR_UNSUPPORTED;
}

sv_status launch_zncc_sgm(const uint8_t *ll, const uint8_t *lr, int B, int h, int w, int D, int win_w,
                          int win_h, int P1, int P2, uint8_t *ws, uint8_t *disp, hipStream_t s)
{
    sv_status r = launch_zncc_cost(ll, lr, B, h, w, D, sgm_dpad(D), win_w, win_h, ws, s);
    if (r != SV_OK) return r;
    return sgm_from_cost(B, h, w, D, P1, P2, ws, disp, s);
}

sv_status launch_smp_median(const uint8_t *disp, int B, int h, int w, int D, uint8_t *tmp,
                            uint8_t *out, hipStream_t s)
{
    if (w > SMP_MAXW) return SV_ERR_SHAPE;
    hipLaunchKernelGGL(k_smp, dim3(B * h), dim3(64), 0, s, disp, B, h, w, D, tmp);
    SV_LAUNCH_CHECK("k_smp");
    const size_t n = (size_t)B * h * w;
    const int blocks = (int)std::min<size_t>((n + 255) / 256, 8192);
    hipLaunchKernelGGL(k_median3, dim3(blocks), dim3(256), 0, s, tmp, B, h, w, out);
    SV_LAUNCH_CHECK("k_median3");
    return SV_OK;
}

}  // namespace sv
