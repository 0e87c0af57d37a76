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

// A lane's value of another lane of its DPP row; `old` where there is none.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t old, uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)v, CTRL, 0xf, 0xf, false);
}
// min over the 16 lanes of a DPP row, in every lane of the row (a rotation has
// no lane without a source, so each step is one v_min with a DPP operand)
__device__ __forceinline__ uint32_t row_min(uint32_t v) {
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x121, 0xf, 0xf, true));  // row_ror:1
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x122, 0xf, 0xf, true));  // row_ror:2
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x124, 0xf, 0xf, true));  // row_ror:4
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x128, 0xf, 0xf, true));  // row_ror:8
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
// vol[dir][b][y][x][Dp].
//
// Bound by the dependent instructions of one wave's chain of w steps at small
// batches and by the volumes' traffic at large ones.  A lane holds its DPL path
// costs two to a register (16-bit halves, packed min and add).  With mn the
// minimum of the previous pixel, cur = min(prev, left + P1, right + P1,
// mn + P2) + (c - mn): the row minimum is needed for two of the operands only,
// and the neighbours' terms are formed beside it.  A path starts from prev =
// mn = 0, which gives cur = c.  Disparities past D get SGM_INF or'ed into
// their cost; they stay above every valid cost + P1 and never win.  Costs are
// loaded a block of SGM_PF steps ahead into one of two sets of registers, each
// used in place (a single set made the compiler copy it, and wait for the last
// store, at every block, and loads under a branch made every step of a path's
// tail wait for memory).  Pointers advance by a stride; lanes past Dp read a
// fixed cost and all write one word of the sink by a stride of 0, without a
// test (a word of the sink for each of them costs a request each: 121 us below
// instead of 44).
// (At 1/4 of 1242x375, D = 48, one pair / 16 pairs: 28 / 45 us; 58 / 122 us
// with one value a register, selects on every access and a sink word a lane.)
constexpr int SGM_PF = 16;
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

// (lo's high half, hi's low half)
__device__ __forceinline__ u16x2 mid2(u16x2 hi, u16x2 lo) {
    return __builtin_bit_cast(u16x2, __builtin_amdgcn_alignbit(__builtin_bit_cast(uint32_t, hi),
                                                               __builtin_bit_cast(uint32_t, lo), 16));
}

template <int DPL>
__global__ void __launch_bounds__(64)
k_sgm_paths(const uint8_t *__restrict__ cost, int B, int h, int w, int D, int Dp, int P1, int P2,
            uint8_t *__restrict__ vol, uint8_t *__restrict__ sink)
{
    constexpr int NR = DPL / 2;                    // registers of path costs
    constexpr int NWD = DPL >= 4 ? DPL / 4 : 1;    // words of costs (DPL = 2: a half word)
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
    const long long step = ((long long)dy * w + dx) * Dp, at0 = ((long long)y0 * w + x0) * Dp;
    // per word: where it is read and written; a word past Dp reads the first
    // costs of the image and writes the workgroup's word of the sink
    const uint8_t *lp[NWD];
    uint8_t *sp[NWD];
    long long st[NWD];
    bool ok[NWD];
    uint32_t pad[NR];  // SGM_INF in the halves whose disparity is past D
#pragma unroll
    for (int k = 0; k < NWD; ++k) {
        ok[k] = d0 + 4 * k < Dp;
        lp[k] = ok[k] ? cb + at0 + d0 + 4 * k : cb;
        sp[k] = ok[k] ? vb + at0 + d0 + 4 * k : sink + (blockIdx.x & 63) * 64;
        st[k] = ok[k] ? step : 0;
    }
#pragma unroll
    for (int r = 0; r < NR; ++r)
        pad[r] = (d0 + 2 * r < D ? 0u : (uint32_t)SGM_INF) | (d0 + 2 * r + 1 < D ? 0u : (uint32_t)SGM_INF << 16);

    // the costs of the SGM_PF steps from s on; past the path's end (guard) the
    // last step's again, so that loads are unconditional
    auto fetch = [&](uint32_t (&c)[SGM_PF][NWD], int s, bool guard) {
#pragma unroll
        for (int k = 0; k < SGM_PF; ++k) {
            const bool adv = !guard || s + k + 1 < len;
#pragma unroll
            for (int q = 0; q < NWD; ++q) {
                if constexpr (DPL == 2) c[k][q] = *(const uint16_t *)lp[q];
                else c[k][q] = *(const uint32_t *)lp[q];
                lp[q] += adv ? st[q] : 0;
            }
        }
    };
    u16x2 prev[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) prev[r] = u16x2{0, 0};
    u16x2 mn = {0, 0};  // the minimum of the previous pixel's path costs, twice
    const u16x2 p1 = {(uint16_t)P1, (uint16_t)P1}, p2 = {(uint16_t)P2, (uint16_t)P2};

    // one step with the costs cw
    auto run = [&](const uint32_t (&cw)[NWD]) {
        u16x2 c[NR];
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            // bytes 2 r and 2 r + 1 of the costs as 16-bit halves
            const uint32_t h2 = __builtin_amdgcn_perm(0u, cw[r / 2], (r & 1) ? 0x0c030c02u : 0x0c010c00u);
            c[r] = __builtin_bit_cast(u16x2, h2 | pad[r]);
        }
        // lane - 1's last and lane + 1's first register, SGM_INF at the row's ends
        const u16x2 from_l = __builtin_bit_cast(u16x2, dpp<0x111>((uint32_t)SGM_INF << 16,
                                                                  __builtin_bit_cast(uint32_t, prev[NR - 1])));
        const u16x2 from_r = __builtin_bit_cast(u16x2, dpp<0x101>((uint32_t)SGM_INF,
                                                                  __builtin_bit_cast(uint32_t, prev[0])));
        u16x2 x[NR + 1];  // x[r] = (cost 2 r - 1, cost 2 r)
        x[0] = mid2(prev[0], from_l);
#pragma unroll
        for (int r = 1; r < NR; ++r) x[r] = mid2(prev[r], prev[r - 1]);
        x[NR] = mid2(from_r, prev[NR - 1]);
        u16x2 cur[NR];
        const u16x2 q = p2 + mn;
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            u16x2 m = __builtin_elementwise_min(x[r], x[r + 1]) + p1;
            m = __builtin_elementwise_min(m, prev[r]);
            cur[r] = __builtin_elementwise_min(m, q) + (c[r] - mn);
        }
        u16x2 t = cur[0];
#pragma unroll
        for (int r = 1; r < NR; ++r) t = __builtin_elementwise_min(t, cur[r]);
        const uint32_t least = row_min(min((uint32_t)t[0], (uint32_t)t[1]));
#pragma unroll
        for (int k = 0; k < NWD; ++k) {
            if constexpr (DPL == 2) {
                *(uint16_t *)sp[k] = (uint16_t)__builtin_amdgcn_perm(0u, __builtin_bit_cast(uint32_t, cur[0]), 0x0c0c0200u);
            } else {
                *(uint32_t *)sp[k] = __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, cur[2 * k + 1]),
                                                           __builtin_bit_cast(uint32_t, cur[2 * k]), 0x06040200u);
            }
            sp[k] += st[k];
        }
        mn = u16x2{(uint16_t)least, (uint16_t)least};
#pragma unroll
        for (int r = 0; r < NR; ++r) prev[r] = cur[r];
    };
    auto full = [&](const uint32_t (&c)[SGM_PF][NWD]) {
#pragma unroll
        for (int k = 0; k < SGM_PF; ++k) run(c[k]);
    };
    auto part = [&](const uint32_t (&c)[SGM_PF][NWD], int s) {
#pragma unroll
        for (int k = 0; k < SGM_PF; ++k)
            if (s + k < len) run(c[k]);
    };
    uint32_t ra[SGM_PF][NWD], rb[SGM_PF][NWD];
    fetch(ra, 0, true);
    int s = 0;
    for (; s + 3 * SGM_PF < len; s += 2 * SGM_PF) {  // both blocks and the next are on the path
        fetch(rb, s + SGM_PF, false);
        full(ra);
        fetch(ra, s + 2 * SGM_PF, false);
        full(rb);
    }
    fetch(rb, s + SGM_PF, true);
    part(ra, s);
    fetch(ra, s + 2 * SGM_PF, true);
    part(rb, s + SGM_PF);
    part(ra, s + 2 * SGM_PF);
}

// Aggregated cost (Eq. (5)) and winner-take-all (Eq. (6)), lowest d on ties;
// the four volumes are [B][h][w][Dp].  Bound by reading the four volumes: a
// thread takes CW words (4 CW disparities) of one pixel, so a wave reads
// contiguous memory, keeps the least key (sum << 8 | d), and a pixel's nch
// threads meet in LDS.  CW = 4 (16-byte loads) where Dp is a multiple of 16.
// (16 reduced 1242x375 pairs, D = 48: 16 us; 59 us with a thread a pixel, each lane
// reading a row of its own.)
template <int CW>
__global__ void __launch_bounds__(256)
k_sgm_wta(const uint8_t *__restrict__ vol, size_t nvox, int D, int Dp, int nch, size_t npix,
          uint8_t *__restrict__ disp)
{
    typedef uint32_t words __attribute__((ext_vector_type(CW)));
    __shared__ uint32_t key[256];
    const int per = 256 / nch;  // pixels of a workgroup
    const int pl = threadIdx.x / nch, ch = threadIdx.x - pl * nch;
    for (size_t p0 = (size_t)blockIdx.x * per; p0 < npix; p0 += (size_t)gridDim.x * per) {
        uint32_t best = 0xffffffffu;
        if (pl < per && p0 + pl < npix) {
            const uint8_t *v = vol + (p0 + pl) * Dp + 4 * CW * ch;
            words q[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) q[r] = *(const words *)(v + r * nvox);
#pragma unroll
            for (int k = 0; k < CW; ++k) {
                uint32_t even = 0, odd = 0;  // sums of bytes 0, 2 and of bytes 1, 3 as 16-bit halves
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const uint32_t u = CW == 1 ? ((const uint32_t *)&q[r])[0] : q[r][k];
                    even += u & 0x00ff00ffu;
                    odd += (u >> 8) & 0x00ff00ffu;
                }
                const int d = 4 * (CW * ch + k);
                if (d < D) best = min(best, (even & 0xffffu) << 8 | (uint32_t)d);
                if (d + 1 < D) best = min(best, (odd & 0xffffu) << 8 | (uint32_t)(d + 1));
                if (d + 2 < D) best = min(best, (even >> 16) << 8 | (uint32_t)(d + 2));
                if (d + 3 < D) best = min(best, (odd >> 16) << 8 | (uint32_t)(d + 3));
            }
        }
        key[threadIdx.x] = best;
        __syncthreads();
        if ((int)threadIdx.x < per && p0 + threadIdx.x < npix) {
            uint32_t m = key[threadIdx.x * nch];
            for (int k = 1; k < nch; ++k) m = min(m, key[threadIdx.x * nch + k]);
            disp[p0 + threadIdx.x] = (uint8_t)(m & 0xffu);
        }
        __syncthreads();
    }
}

// Single matching phase (Eq. (7)) with nearest-valid filling, one workgroup
// per row.  The target column of x is x - D(x); x is invalid when a pixel
// x + k, 0 < k < D, has the same target column (the left pixel of such a pair
// is the one hidden in the target view).  Validity is kept as one 64-bit ballot
// per 64 pixels; each invalid pixel takes the nearest valid value of its row
// (the smaller one at equal distances).  The row is staged in LDS.
//
// Two pixels with one target column are apart by the difference of their
// disparities, which is below D when every disparity of the row is.  Then x is
// valid exactly when it is the last pixel with its target column, and the
// kernel finds those with one LDS maximum a pixel instead of a search over D
// pixels.  A row with a disparity of D or more, and rows too wide for the table
// in LDS (use_last = 0), are searched.
// (94 rows of 311 pixels, D = 48: 5 us; 29 us with one wave a row and the search.)
constexpr int SMP_MAXW = 16384;
constexpr int SMP_LASTW = 8192;  // widest row with the table: 43 KB of LDS
__global__ void __launch_bounds__(256)
k_smp(const uint8_t *__restrict__ disp, int w, int D, int use_last, uint8_t *__restrict__ out)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int nch = (w + 63) / 64;
    uint64_t *valid = (uint64_t *)smem;
    uint8_t *row = (uint8_t *)(valid + nch);
    int *last = (int *)(row + ((w + 3) & ~3));  // [w + 255]: last pixel with target column t - 255
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const size_t base = (size_t)blockIdx.x * w;  // row blockIdx.x of B * h
    bool big = false;
    for (int x = tid; x < w; x += 256) {
        const int d = disp[base + x];
        row[x] = (uint8_t)d;
        big |= d >= D;
    }
    if (use_last)
        for (int x = tid; x < w + 255; x += 256) last[x] = -1;
    const bool search = __syncthreads_or(big) || !use_last;
    if (!search) {
        for (int x = tid; x < w; x += 256) atomicMax(&last[x - row[x] + 255], x);
        __syncthreads();
    }
    for (int ch = wave; ch < nch; ch += 4) {
        const int x = ch * 64 + lane;
        bool ok = x < w;
        if (ok) {
            const int t = x - row[x];
            if (!search) {
                ok = last[t + 255] == x;
            } else {
                for (int k = 1; k < D && x + k < w; ++k)
                    if (x + k - row[x + k] == t) { ok = false; break; }
            }
        }
        const uint64_t m = __ballot(ok);
        if (lane == 0) valid[ch] = m;
    }
    __syncthreads();
    // (the last pixel of a row is always valid)
    for (int x = tid; x < w; x += 256) {
        const int ch = x >> 6, bit = x & 63;
        uint8_t v = row[x];
        if (!((valid[ch] >> bit) & 1)) {
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
    if (dpl <= 2) SV_SGM(2);
    else if (dpl <= 4) SV_SGM(4);
    else if (dpl <= 8) SV_SGM(8);
    else SV_SGM(16);
#undef SV_SGM
    SV_LAUNCH_CHECK("k_sgm_paths");
    const size_t npix = (size_t)B * h * w;
    const bool wide = Dp % 16 == 0 && (uintptr_t)ws % 16 == 0;
    const int nch = Dp / (wide ? 16 : 4);
    const int blocks = (int)std::min<size_t>((npix + 256 / nch - 1) / (256 / nch), 16384);
    if (wide) hipLaunchKernelGGL(k_sgm_wta<4>, dim3(blocks), dim3(256), 0, s, vol, nvox, D, Dp, nch, npix, disp);
    else hipLaunchKernelGGL(k_sgm_wta<1>, dim3(blocks), dim3(256), 0, s, vol, nvox, D, Dp, nch, npix, disp);
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
    const int use_last = w <= SMP_LASTW;
    const size_t lds = (size_t)cdiv(w, 64) * 8 + ((w + 3) & ~3) + (use_last ? (size_t)(w + 255) * 4 : 0);
    hipLaunchKernelGGL(k_smp, dim3(B * h), dim3(256), lds, s, disp, w, D, use_last, tmp);
    SV_LAUNCH_CHECK("k_smp");
    const size_t n = (size_t)B * h * w;
    const int blocks = (int)std::min<size_t>((n + 255) / 256, 8192);
    hipLaunchKernelGGL(k_median3, dim3(blocks), dim3(256), 0, s, tmp, B, h, w, out);
    SV_LAUNCH_CHECK("k_median3");
    return SV_OK;
}

}  // namespace sv
