// The decoder's last 3x3 layer at inference, G0 = conv3x3([resize(G1), x0]),
// with the final layer's projection in its epilogue, for up to 32 channels in
// 16 or 8 bits: a persistent kernel.
//
// What bounds it: the vector work around the matrix products (resizing and
// rounding the input, the epilogue) and the serial steps between a tile's
// barriers (without staging, products and stores 58 us of 114 remain).  So
//  * a workgroup walks tiles of one XCD's contiguous share (neighbouring tiles
//    read neighbouring G1 pixels through one L2) and keeps the layer's weights
//    for all of them, in registers: read from LDS they are two thirds of the
//    reads and LDS the bound (bf16, 32 channels: 134 us instead of 114).  INT8
//    operands are half as long, and its weights in LDS leave registers for one
//    more workgroup a CU: 21.9 us instead of 25.8;
//  * the input patch of a tile is made between pairs of coarse rows: a thread
//    takes one patch column and channel group, loads and unpacks the four
//    corners once and forms the two (at an edge three) patch rows they serve;
//  * the loads of the next tile's coarse rows and x0 pixels are issued before
//    the products of this one, so no tile waits for memory; its axis tables are
//    made a tile earlier still, by one wave each;
//  * a wave's rows share their input rows in registers: an operand read from
//    LDS feeds up to three output rows (18 reads instead of 36 for four rows);
//  * the projection's weights are split into their high and low parts once per
//    workgroup and kept, with the other epilogue operands, in LDS: in registers
//    they made the weights spill (154 us instead of 114).
// The order of every sum is the one of the general kernel (conv_impl.h): base
// chunks ascending, taps ascending, then x0's packed taps when x0 starts a
// chunk of its own.
//
// Measured against the general kernel with the same epilogue (us): 64 bf16 maps
// 311x94, 32 channels, 176 -> 114; 64 uneven maps in one launch 210 -> 69;
// 8 INT8 maps 32 -> 22; 8 f16 maps 128x64, 16 channels, 11.9 -> 9.7.
#include <algorithm>

#include "conv_impl.h"

namespace sv {

namespace {

template <int DT, int TH, int NB>
struct G0Tile {
    using M = Mfma<DT>;
    using T = typename M::T;
    using vec = typename M::vec;
    static constexpr int GS = M::GS;
    static constexpr int SD = Store<DT>::v;
    using ST = typename Elem<SD>::T;
    typedef ST SVec __attribute__((ext_vector_type(GS)));
    static constexpr int KCB = 32;
    static constexpr int KB = (NB * 16 + KCB - 1) / KCB;  // base chunks that hold c1 channels
    static constexpr int KCG = KB * KCB / GS;             // channel groups of a patch pixel
    static constexpr int KCP = KB * KCB + GS;             // padded patch row, in elements
    static constexpr int PH = TH + 2, PW = 18, NPIX = PH * PW;
    static constexpr int MBW = TH / 4;
    static constexpr bool WREG = DT != SV_I8 || NB == 1;
    // staging: an item is one channel group of one patch column between two
    // coarse rows; the patch's rows touch at most (PH - 1) / 2 + 2 such pairs
    // (they lie n_in / n_out apart, n_in = ceil(n_out / 2), and a run of m <=
    // n_out rows spans (m - 1) n_in / n_out < m / 2)
    static constexpr int RG = NB * 16 / GS;
    static constexpr int NI = (PH - 1) / 2 + 2;
    static constexpr int NIT = (PW * RG * NI + 255) / 256;
    static constexpr int NX = (NPIX + 255) / 256;
    static constexpr int NKX = 18, NSX = (NKX + 4 * GS - 1) / (4 * GS);
    struct Axis { int i0, i1; float lam; };               // i0 < 0: outside the input grid
    struct __attribute__((aligned(16))) Pair { int rows; float lam[3]; };  // its patch rows: first | count << 8
    typedef T XPair __attribute__((ext_vector_type(2)));
    struct Smem {
        T patch[NPIX * KCP];
        __attribute__((aligned(8))) T xp[2 * (NPIX + 1)];  // x0 pairs, a zero pair last
        float2 raw[NPIX];         // x0 itself
        T wl[WREG ? 1 : 9 * NB * 16 * KCP];
        Axis ax[3][PH + PW];
        Pair pair[2][NI];
        int first[3];               // first coarse row
        // the epilogue's operands (kept here: the weights' registers leave no room)
        typename Mfma<SD>::vec pj[2][64];  // a lane's projection operands
        f32x4 bias[NB][4], fac[NB][4], wd[4], wi[4];            // by lane group
    };
};

struct G0Geo { int Hi, Wi, hs, ws; long long sbase, obase; int oy0, ox0; };

// n / d and the remainder for 0 <= n, quotients to 2^22: a float estimate, off
// by at most one, put right by the exact remainder (a division instruction's
// sequence is three times as long and sits in a tile's serial chain).
__device__ __forceinline__ int quot(int n, int d, float rd, int &rem) {
    int q = (int)((float)n * rd);
    int r = n - q * d;
    if (r < 0) { --q; r += d; }
    else if (r >= d) { ++q; r -= d; }
    rem = r;
    return q;
}


template <int DT, int TH, int NB, bool TAB>
__global__ void __launch_bounds__(256, 2) k_g0(const ConvParams p, int total_u, int tiles_x, int tiles_y)
{
    using G = G0Tile<DT, TH, NB>;
    using M = typename G::M;
    using T = typename G::T;
    using vec = typename G::vec;
    using SVec = typename G::SVec;
    using ST = typename G::ST;
    constexpr int GS = G::GS, KB = G::KB, KCP = G::KCP, PW = G::PW, PH = G::PH, MBW = G::MBW;
    __shared__ __attribute__((aligned(16))) typename G::Smem sm;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int g = lane >> 4, r16 = lane & 15;
    const int c1 = p.Cout;
    // x0 inside the last base chunk, or in a chunk of its own
    const bool inl = c1 % G::KCB != 0;

    // this workgroup's tiles: every (grid / 8)-th of its XCD's share
    const int total = TAB ? p.tab->cum[p.stage][p.tab->n] : total_u;
    int t0, t1, dt;
    if (gridDim.x % 8 == 0) {
        const int x = blockIdx.x % 8;
        t0 = (int)((long long)total * x / 8) + blockIdx.x / 8;
        t1 = (int)((long long)total * (x + 1) / 8);
        dt = gridDim.x / 8;
    } else {
        t0 = blockIdx.x;
        t1 = total;
        dt = gridDim.x;
    }
    if (t0 >= t1) return;

    int pi = 0;  // TAB: the pair of the last tile asked for; tiles only grow
    if constexpr (TAB) pi = table_find(p.tab->cum[p.stage], p.tab->n, t0);
    const float r_img = __builtin_amdgcn_rcpf((float)(tiles_x * tiles_y)), r_tx = __builtin_amdgcn_rcpf((float)tiles_x);
    auto geo = [&](int t) {
        G0Geo q;
        if constexpr (TAB) {
            const PairTable *tab = p.tab;
            const int *cum = tab->cum[p.stage];
            while (t >= cum[pi + 1]) ++pi;
            const PairGeo &pg = tab->pair[pi];
            const int tx = cdiv_d(pg.w[0], 16);
            int c;
            const int r = quot(t - cum[pi], tx, __builtin_amdgcn_rcpf((float)tx), c);
            q.Hi = pg.h[0]; q.Wi = pg.w[0]; q.hs = pg.h[1]; q.ws = pg.w[1];
            q.sbase = pg.off[1]; q.obase = pg.off[0];
            q.oy0 = __builtin_amdgcn_readfirstlane(r * TH);
            q.ox0 = __builtin_amdgcn_readfirstlane(c * 16);
        } else {
            int r, c;
            const int b = __builtin_amdgcn_readfirstlane(quot(t, tiles_x * tiles_y, r_img, r));
            const int ty = quot(r, tiles_x, r_tx, c);
            q.Hi = p.Hi; q.Wi = p.Wi; q.hs = p.src[0].hs; q.ws = p.src[0].ws;
            q.sbase = (long long)b * q.hs * q.ws;
            q.obase = (long long)b * q.Hi * q.Wi;
            q.oy0 = __builtin_amdgcn_readfirstlane(ty * TH);
            q.ox0 = __builtin_amdgcn_readfirstlane(c * 16);
        }
        return q;
    };
    // The tables of a tile are made two tiles ahead (axes) and one ahead (pairs,
    // from axes' tables), by one wave each beside the products, so that no wave
    // waits for a division.  axes: each patch row's and column's coarse indices
    // and weight, as bilin() gives them.
    auto axes = [&](const G0Geo &q, int buf) {
        const bool row = wave == 0;
        if (wave < 2 && lane < (row ? PH : PW)) {
            const int o = (row ? q.oy0 : q.ox0) - 1 + lane;
            const int n = row ? q.Hi : q.Wi, nin = row ? q.hs : q.ws;
            typename G::Axis a = {-1, -1, 0.f};
            if (o >= 0 && o < n) {
                const int num = (2 * o + 1) * nin - n, den = 2 * n;
                a.i0 = 0;
                if (num > 0) {
                    int rem;
                    a.i0 = quot(num, den, __builtin_amdgcn_rcpf((float)den), rem);
                    a.lam = (float)rem / (float)den;
                }
                a.i1 = min(a.i0 + 1, nin - 1);
            }
            sm.ax[buf][(row ? 0 : PH) + lane] = a;
            // the first patch row inside the image (row 0 is outside for the topmost tiles)
            if (row && lane == (q.oy0 == 0 ? 1 : 0)) sm.first[buf] = a.i0;
        }
    };
    auto pairs = [&](int buf, int pbuf) {
        if (wave == 2 && lane < PH) {
            // lane = patch row: the first row of a pair writes the pair
            const typename G::Axis a = sm.ax[buf][lane];
            const int y0 = sm.first[buf], k = a.i0 - y0;
            const int up = lane ? sm.ax[buf][lane - 1].i0 : -1;
            const int d1 = lane + 1 < PH ? sm.ax[buf][lane + 1].i0 : -1, d2 = lane + 2 < PH ? sm.ax[buf][lane + 2].i0 : -1;
            const float l1 = sm.ax[buf][min(lane + 1, PH - 1)].lam, l2 = sm.ax[buf][min(lane + 2, PH - 1)].lam;
            if (a.i0 >= 0 && up != a.i0) {
                const int n = 1 + (d1 == a.i0 ? 1 + (d2 == a.i0) : 0);
                sm.pair[pbuf][k] = typename G::Pair{lane | n << 8, {a.lam, l1, l2}};
                // pairs past the last row inside
                if (lane + n >= PH || sm.ax[buf][min(lane + n, PH - 1)].i0 < 0)
                    for (int j = k + 1; j < G::NI; ++j) sm.pair[pbuf][j].rows = 0;
            }
        }
    };
    float qinv = 0.f, s_in = 0.f;
    if constexpr (DT == SV_I8) input_scale(p, qinv, s_in);
    // ---- staging ------------------------------------------------------------
    // patch groups past the map's (and past x0's) stay zero
    for (int e = tid; e < G::NPIX * G::KCG; e += 256) {
        const int c = (e % G::KCG) * GS;
        if (c >= c1) {
            vec z;
#pragma unroll
            for (int i = 0; i < GS; ++i) z[i] = 0;
            *(vec *)&sm.patch[(e / G::KCG) * KCP + c] = z;
        }
    }
    if (tid < 2) sm.xp[2 * G::NPIX + tid] = (T)0;
    const ST *src = (const ST *)p.src[0].ptr;
    const int pitch = p.src[0].pitch;
    SVec ra[G::NIT][4];
    float lxn[G::NIT];       // the fetched items' column weights, < 0: nothing to write
    float x0v[G::NX][2];
    uint32_t xd[G::NX], xi[G::NX];
    // item j of this thread
    auto item = [&](int j, int &cg, int &col, int &k) {
        const int e = tid + 256 * j;
        cg = e % G::RG;
        col = e / G::RG % PW;
        k = e / (G::RG * PW);
        return k < G::NI && cg * GS < c1;
    };
    auto x0_place = [&](const G0Geo &q, int j, int &pix, int &off) {
        pix = min(tid + j * 256, G::NPIX - 1);
        const int py = pix / PW, px = pix - py * PW;
        const int y = q.oy0 - 1 + py, x = q.ox0 - 1 + px;
        const bool ok = (y >= 0) & (y < q.Hi) & (x >= 0) & (x < q.Wi);
        off = ok ? py * q.Wi + px : q.Wi + 1;  // from the pixel above and left of the tile's first (that first one if outside)
        return ok;
    };
    // issues the loads of a tile: four corners an item, its x0 pixels
    auto fetch = [&](const G0Geo &q, int buf) {
        const int y0 = __builtin_amdgcn_readfirstlane(sm.first[buf]);
        const char *base = (const char *)(src + (size_t)(q.sbase + (long long)y0 * q.ws) * pitch);
        const uint32_t px = pitch * sizeof(ST);
#pragma unroll
        for (int j = 0; j < G::NIT; ++j) {
            int cg, col, k;
            const bool ok = item(j, cg, col, k);
            const typename G::Axis cx = sm.ax[buf][PH + col];
            lxn[j] = ok && cx.i0 >= 0 ? cx.lam : -1.f;
            const int ya = min(y0 + (ok ? k : 0), q.hs - 1) - y0, yb = min(y0 + (ok ? k : 0) + 1, q.hs - 1) - y0;
            const uint32_t c = ok ? cg * GS * sizeof(ST) : 0;
            const uint32_t xa = max(cx.i0, 0) * px + c, xb = max(cx.i1, 0) * px + c;
            const uint32_t ra0 = ya * q.ws * px, rb0 = yb * q.ws * px;
            ra[j][0] = *(const SVec *)(base + (ra0 + xa));
            ra[j][1] = *(const SVec *)(base + (ra0 + xb));
            ra[j][2] = *(const SVec *)(base + (rb0 + xa));
            ra[j][3] = *(const SVec *)(base + (rb0 + xb));
        }
        const long long o0 = q.obase + (long long)(q.oy0 - 1) * q.Wi + q.ox0 - 1;
        const uint8_t *db = (const uint8_t *)p.src[1].ptr + o0, *ib = p.src[1].img + o0;
#pragma unroll
        for (int j = 0; j < G::NX; ++j) {
            int pix, off;
            x0_place(q, j, pix, off);
            xd[j] = db[off];
            xi[j] = ib[off];
        }
    };
    // the fetched x0 bytes as values: kept apart from fetch(), since the bytes'
    // conversion waits for every load before them
    auto settle = [&](const G0Geo &q) {
#pragma unroll
        for (int j = 0; j < G::NX; ++j) {
            int pix, off;
            const bool ok = x0_place(q, j, pix, off);
            x0v[j][0] = ok ? p.src[1].scale0 * (float)xd[j] : 0.f;
            x0v[j][1] = ok ? (float)xi[j] * (1.0f / 256.0f) : 0.f;
        }
    };
    // writes the fetched tile into LDS
    auto commit = [&](const G0Geo &q, int buf, int pbuf) {
        vec z;
#pragma unroll
        for (int i = 0; i < GS; ++i) z[i] = 0;
        typename G::Pair pr[G::NIT];
#pragma unroll
        for (int j = 0; j < G::NIT; ++j) pr[j] = sm.pair[pbuf][min((tid + 256 * j) / (G::RG * PW), G::NI - 1)];
        // patch rows and columns outside the image
        if (q.oy0 == 0 || q.ox0 == 0 || q.oy0 + TH >= q.Hi || q.ox0 + 16 >= q.Wi) {
            for (int e = tid; e < G::NPIX * G::RG; e += 256) {
                const int pix = e / G::RG, py = pix / PW;
                if ((sm.ax[buf][py].i0 < 0) | (sm.ax[buf][PH + pix - py * PW].i0 < 0))
                    *(vec *)&sm.patch[pix * KCP + e % G::RG * GS] = z;
            }
        }
#pragma unroll
        for (int j = 0; j < G::NIT; ++j) {
            int cg, col, k;
            item(j, cg, col, k);
            const int r0 = pr[j].rows & 0xff, n = lxn[j] >= 0.f ? pr[j].rows >> 8 : 0;
            const float lx = lxn[j], lx0 = 1.f - lx;
            const float ly[3] = {pr[j].lam[0], pr[j].lam[1], pr[j].lam[2]};
            T *dst = sm.patch + (r0 * PW + col) * KCP + cg * GS;
            if (n == 0) continue;
            float x00[GS], x01[GS], x10[GS], x11[GS];
#pragma unroll
            for (int i = 0; i < GS; ++i) {
                x00[i] = Elem<G::SD>::load((const ST *)&ra[j][0] + i);
                x01[i] = Elem<G::SD>::load((const ST *)&ra[j][1] + i);
                x10[i] = Elem<G::SD>::load((const ST *)&ra[j][2] + i);
                x11[i] = Elem<G::SD>::load((const ST *)&ra[j][3] + i);
                if constexpr (DT == SV_I8) {
                    // INT8 codes are defined on the separable FP32 expression
                    x00[i] = lx0 * x00[i] + lx * x01[i];
                    x10[i] = lx0 * x10[i] + lx * x11[i];
                }
            }
#pragma unroll
            for (int r = 0; r < 3; ++r) {  // two rows a pair, three where the image starts or ends
                if (r >= n) continue;
                float v[GS];
                const float ly0 = 1.f - ly[r];
                if constexpr (DT == SV_I8) {
#pragma unroll
                    for (int i = 0; i < GS; ++i) v[i] = ly0 * x00[i] + ly[r] * x10[i];
                } else {
                    const float w00 = ly0 * lx0, w01 = ly0 * lx, w10 = ly[r] * lx0, w11 = ly[r] * lx;
#pragma unroll
                    for (int i = 0; i < GS; ++i) v[i] = fmaf(w11, x11[i], fmaf(w10, x10[i], fmaf(w01, x01[i], w00 * x00[i])));
                }
                *(vec *)&dst[r * PW * KCP] = pack_vec<DT, GS>(v, qinv);
            }
        }
#pragma unroll
        for (int j = 0; j < G::NX; ++j) {
            const int pix = tid + j * 256;
            if (pix >= G::NPIX) continue;
            sm.raw[pix] = make_float2(x0v[j][0], x0v[j][1]);
            float v[GS];
#pragma unroll
            for (int i = 0; i < GS; ++i) v[i] = i < 2 ? x0v[j][i < 2 ? i : 0] : 0.f;
            const vec pv = pack_vec<DT, GS>(v, qinv);
            if (inl) {
                *(vec *)&sm.patch[pix * KCP + c1] = pv;
            } else {
                *(typename G::XPair *)&sm.xp[2 * pix] = typename G::XPair{pv[0], pv[1]};
            }
        }
    };

    // the first tile's loads before the weights'
    G0Geo q = geo(t0), q1 = q;
    axes(q, 0);
    __syncthreads();
    fetch(q, 0);
    pairs(0, 0);
    if (t0 + dt < t1) {
        q1 = geo(t0 + dt);
        axes(q1, 1);
    }

    // ---- weights ------------------------------------------------------------
    const T *wpk = (const T *)p.wpk;
    vec wa[G::WREG ? KB * 9 * NB : 1];
    auto wfrag = [&](int kb, int tap, int nb) {  // rows nb 16 + r16, channels kb KCB + g GS ..
        const int c = kb * G::KCB + g * GS;
        vec v;
#pragma unroll
        for (int i = 0; i < GS; ++i) v[i] = 0;
        // columns past the resized map's: x0's two when they share the chunk
        if (c < c1 || (inl && c == c1)) {
            const vec q = *(const vec *)(wpk + ((size_t)tap * p.n_pad + nb * 16 + r16) * p.cin_pad + c);
#pragma unroll
            for (int i = 0; i < GS; ++i) v[i] = c + i < c1 + 2 ? q[i] : (T)0;
        }
        return v;
    };
    if constexpr (G::WREG) {
#pragma unroll
        for (int k = 0; k < KB; ++k)
#pragma unroll
            for (int t = 0; t < 9; ++t)
#pragma unroll
                for (int n = 0; n < NB; ++n) wa[(k * 9 + t) * NB + n] = wfrag(k, t, n);
    } else {
        // [tap][row][KCP]
        for (int e = tid; e < 9 * NB * 16 * G::KCG; e += 256) {
            const int c = (e % G::KCG) * GS, r = e / G::KCG;
            const int n = r % (NB * 16), tap = r / (NB * 16);
            vec v;
#pragma unroll
            for (int i = 0; i < GS; ++i) v[i] = 0;
            if (c < c1 || (inl && c == c1)) {
                const vec q = *(const vec *)(wpk + ((size_t)tap * p.n_pad + n) * p.cin_pad + c);
#pragma unroll
                for (int i = 0; i < GS; ++i) v[i] = c + i < c1 + 2 ? q[i] : (T)0;
            }
            *(vec *)&sm.wl[(tap * NB * 16 + n) * KCP + c] = v;
        }
    }
    // x0's packed taps: k = 2 tap + channel, lane group g k = (4 s + g) GS ..
    vec wx[G::NSX][NB];
    int xo[G::NSX][GS / 2];  // patch offset of this lane's taps from a pixel, < 0: none
#pragma unroll
    for (int s = 0; s < G::NSX; ++s)
#pragma unroll
        for (int m = 0; m < GS / 2; ++m) {
            const int tap = (s * 4 + g) * (GS / 2) + m;
            xo[s][m] = tap < 9 ? (tap / 3) * PW + tap % 3 : -1;
#pragma unroll
            for (int n = 0; n < NB; ++n)
#pragma unroll
                for (int k = 0; k < 2; ++k)
                    wx[s][n][2 * m + k] = tap < 9 && !inl
                        ? wpk[((size_t)tap * p.n_pad + n * 16 + r16) * p.cin_pad + c1 + k] : (T)0;
        }
    // the projection's operand: row = tap r16, this lane's channels n 16 + 4 g + i;
    // 16-bit types: the FP32 weight's high and low part
    using MP = Mfma<G::SD>;
    float *po = p.proj_out + 4 * g * p.proj_plane + r16;
    if (wave == 3) {
        float w8[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int n = j / 4, c = n * 16 + 4 * g + j % 4;
            w8[j] = n < NB && r16 < 9 && c < c1 ? p.proj_w[r16 * p.proj_pitch + c] : 0.f;
        }
        float hi[8], lo[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const typename Elem<G::SD>::T h = Elem<G::SD>::make(w8[j]);
            hi[j] = Elem<G::SD>::load(&h);
            lo[j] = w8[j] - hi[j];
        }
        sm.pj[0][lane] = pack_vec<G::SD, 8>(hi, 0.f);
        sm.pj[1][lane] = pack_vec<G::SD, 8>(lo, 0.f);
        if (r16 == 0) {
#pragma unroll
            for (int n = 0; n < NB; ++n) {
                float b4[4];
                conv_bias4<DT>(p, n * 16 + 4 * g, b4);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    sm.bias[n][g][i] = b4[i];
                    // INT8: the factor from an integer sum to its value
                    if constexpr (DT == SV_I8)
                        sm.fac[n][g][i] = n * 16 + 4 * g + i < c1 ? s_in * p.wscale[n * 16 + 4 * g + i] : 0.f;
                }
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int t = 4 * g + i;
                sm.wd[g][i] = t < 9 ? p.proj_w[t * p.proj_pitch + c1] : 0.f;
                sm.wi[g][i] = t < 9 ? p.proj_w[t * p.proj_pitch + c1 + 1] : 0.f;
            }
        }
    }

    settle(q);
    __syncthreads();
    int buf = 0, pbuf = 0;
    for (int t = t0; t < t1; t += dt) {
        commit(q, buf, pbuf);
        const bool more = t + dt < t1;
        const int b1 = buf == 2 ? 0 : buf + 1, b2 = b1 == 2 ? 0 : b1 + 1;
        G0Geo q2 = q1;
        __syncthreads();
        if (more) {
            fetch(q1, b1);
            pairs(b1, pbuf ^ 1);
            if (t + 2 * dt < t1) {
                q2 = geo(t + 2 * dt);
                axes(q2, b2);
            }
        }
        // ---- products -----------------------------------------------------
        typename M::acc acc[MBW][NB];
#pragma unroll
        for (int m = 0; m < MBW; ++m)
#pragma unroll
            for (int n = 0; n < NB; ++n) acc[m][n] = typename M::acc{0, 0, 0, 0};
        const int row0 = wave * MBW;
        const T *pb = sm.patch + (row0 * PW + r16) * KCP + g * GS;
        const T *wb = sm.wl + r16 * KCP + g * GS;
#pragma unroll
        for (int k = 0; k < KB; ++k)
#pragma unroll
            for (int iy = 0; iy < MBW + 2; ++iy)
#pragma unroll
                for (int v = 0; v < 3; ++v) {
                    const vec b = *(const vec *)(pb + (iy * PW + v) * KCP + k * G::KCB);
#pragma unroll
                    for (int m = 0; m < MBW; ++m) {
                        const int u = iy - m;
                        if (u < 0 || u > 2) continue;
#pragma unroll
                        for (int n = 0; n < NB; ++n) {
                            vec a;
                            if constexpr (G::WREG) a = wa[(k * 9 + u * 3 + v) * NB + n];
                            else a = *(const vec *)(wb + ((u * 3 + v) * NB + n) * 16 * KCP + k * G::KCB);
                            acc[m][n] = M::run(a, b, acc[m][n]);
                        }
                    }
                }
        if (!inl) {
#pragma unroll
            for (int m = 0; m < MBW; ++m) {
                const int base = (row0 + m) * PW + r16;
#pragma unroll
                for (int s = 0; s < G::NSX; ++s) {
                    vec b;
#pragma unroll
                    for (int j = 0; j < GS / 2; ++j) {
                        // both channels of a tap in one read
                        const int pix = xo[s][j] >= 0 ? base + xo[s][j] : G::NPIX;
                        const typename G::XPair v = *(const typename G::XPair *)&sm.xp[2 * pix];
                        b[2 * j] = v[0];
                        b[2 * j + 1] = v[1];
                    }
#pragma unroll
                    for (int n = 0; n < NB; ++n) acc[m][n] = M::run(wx[s][n], b, acc[m][n]);
                }
            }
        }
        // ---- projection: every row's product, then every row's stores --------
        f32x4 c[MBW];
        float2 x0p[MBW];
        f32x4 bias[NB], fac[NB];
#pragma unroll
        for (int n = 0; n < NB; ++n) {
            bias[n] = sm.bias[n][g];
            if constexpr (DT == SV_I8) fac[n] = sm.fac[n][g];
        }
        const typename MP::vec pj[2] = {sm.pj[0][lane], sm.pj[1][lane]};
#pragma unroll
        for (int m = 0; m < MBW; ++m) {
            x0p[m] = sm.raw[(row0 + m + 1) * PW + r16 + 1];
            // y as it would be stored, this lane's channels of pixel r16
            float y[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int n = j / 4, i = j % 4;
                y[j] = 0.f;
                if (n < NB) {
                    float v = (float)acc[m][n < NB ? n : 0][i];
                    if constexpr (DT == SV_I8) v = v * fac[n < NB ? n : 0][i];
                    v = v + bias[n < NB ? n : 0][i];
                    v = fmaxf(v, 0.1f * v);
                    y[j] = n * 16 + 4 * g < c1 ? v : 0.f;  // (c1 is a multiple of 8: all four or none)
                }
            }
            c[m] = f32x4{0.f, 0.f, 0.f, 0.f};
            const typename MP::vec yq = pack_vec<G::SD, 8>(y, 0.f);
            c[m] = MP::run(pj[0], yq, c[m]);
            c[m] = MP::run(pj[1], yq, c[m]);
        }
        // the next tile's loads are waited for here, before the stores: after them
        // the wait would be for the stores too
        if (more) settle(q1);
        const f32x4 wd = sm.wd[g], wi = sm.wi[g];
        if (g < 3 && q.ox0 + r16 < q.Wi) {
#pragma unroll
            for (int m = 0; m < MBW; ++m) {
                const int oy = q.oy0 + row0 + m;
                if (oy >= q.Hi) break;  // the whole wave's
                float *o = po + (q.obase + (long long)oy * q.Wi + q.ox0);
                *o = fmaf(wi[0], x0p[m].y, fmaf(wd[0], x0p[m].x, c[m][0]));
                if (g < 2) {
#pragma unroll
                    for (int i = 1; i < 4; ++i)
                        o[i * p.proj_plane] = fmaf(wi[i], x0p[m].y, fmaf(wd[i], x0p[m].x, c[m][i]));
                }
            }
        }
        q = q1;
        q1 = q2;
        buf = b1;
        pbuf ^= 1;
        __syncthreads();
    }
}

template <int DT, int TH, int NB>
sv_status launch_g0_t(const ConvParams &p, int grid, hipStream_t st) {
    const int tx = cdiv(p.Wo, 16), ty = cdiv(p.Ho, TH);
    const long long total = grid > 0 ? grid : (long long)p.B * tx * ty;
    const void *fn = grid > 0 ? (const void *)k_g0<DT, TH, NB, true> : (const void *)k_g0<DT, TH, NB, false>;
    // whole shares per XCD: a multiple of eight, at most what is resident
    long long n = resident_grid(fn, 0, total < 8 ? total : (total + 7) / 8 * 8);
    if (n >= 8) n -= n % 8;
    if (grid > 0) hipLaunchKernelGGL((k_g0<DT, TH, NB, true>), dim3((unsigned)n), dim3(256), 0, st, p, 0, 0, 0);
    else hipLaunchKernelGGL((k_g0<DT, TH, NB, false>), dim3((unsigned)n), dim3(256), 0, st, p, (int)total, tx, ty);
    SV_LAUNCH_CHECK("k_g0");
    return SV_OK;
}

template <int DT>
sv_status launch_g0_d(int th, const ConvParams &p, int grid, hipStream_t st) {
    const bool one = p.Cout <= 16;
    if (th == 4) return one ? launch_g0_t<DT, 4, 1>(p, grid, st) : launch_g0_t<DT, 4, 2>(p, grid, st);
    if (th == 8) return one ? launch_g0_t<DT, 8, 1>(p, grid, st) : launch_g0_t<DT, 8, 2>(p, grid, st);
    return one ? launch_g0_t<DT, 16, 1>(p, grid, st) : launch_g0_t<DT, 16, 2>(p, grid, st);
}

}  // namespace

// FP32 keeps the general kernel: one 311x94 map of 32 channels took 14.3 us
// there and 16 to 22 us in the forms of this one (twice the weights do not fit
// beside four rows' sums, and a batch of one has a tile or two a workgroup).
// Other channel counts: a group of 8 would hold both the map's and x0's, or
// the weights would not fit the registers.
bool g0_fits(int dtype, int c1) { return dtype != SV_F32 && c1 <= 32 && c1 % 8 == 0; }

// The rows a tile: a tuned layer's follow its tile (the cost of a small tile here is the
// general kernel's: its halo), any other's the number of workgroups, at least 400 of
// them (1.5 a CU) as in the tile rule, with at most a fifth more rows than four would
// compute.  Sixteen rows past 16 channels alone (8 INT8 maps of 94x311, 32 channels:
// 25.8 us against 28.7 in eight): with fewer a group's sums are too short a part of its
// time.  Over 451 sizes of 8 to 32 channels 1.02 of the best height on average, four rows
// throughout 1.08; sixteen rows at 8 and 16 channels 1.04 to 1.07.
int g0_tile_h(int cfg) {
    int th, tn;
    conv_cfg_tile(cfg, th, tn);
    return th < 8 ? 4 : th < 16 ? 8 : 16;
}

int g0_default_h(int c1, int B, int Ho, int Wo) {
    auto fits = [&](int th) {
        return (long long)B * cdiv(Ho, th) * cdiv(Wo, 16) >= 400 && 5ll * cdiv(Ho, th) * th <= 24ll * cdiv(Ho, 4);
    };
    return c1 > 16 && fits(16) ? 16 : fits(8) ? 8 : 4;
}

sv_status launch_g0(int dtype, int th, const ConvParams &p, int grid, hipStream_t st) {
    if (!p.proj_out || !g0_fits(dtype, p.Cout)) return SV_ERR_UNSUPPORTED;
    switch (dtype) {
    case SV_BF16: return launch_g0_d<SV_BF16>(th, p, grid, st);
    case SV_F16: return launch_g0_d<SV_F16>(th, p, grid, st);
    case SV_I8: return launch_g0_d<SV_I8>(th, p, grid, st);
    default: return SV_ERR_DTYPE;
    }
}

}  // namespace sv
