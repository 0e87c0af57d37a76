// Weight packing of both networks: every layer's forward, adjoint and phase
// packs and biases in one launch.
#include "kernels.h"

namespace sv {

// Element e of a task's destination.  dst[tap][n][c] unless the kind says
// otherwise; entries outside the layer are zeros.
__device__ __forceinline__ float pack_value(const PackTask &t, int e) {
    const int kk = t.k * t.k;
    if (t.kind == PK_BIAS) return e < t.cout ? t.w[e] : 0.f;
    const int c = e % t.cin_pad, n = (e / t.cin_pad) % t.n_pad, tap = e / (t.cin_pad * t.n_pad);
    switch (t.kind) {
    case PK_FWD:  // rows = outputs, columns = inputs
        return n < t.cout && c < t.cin ? t.w[((size_t)n * t.cin + c) * kk + (t.aux ? kk - 1 - tap : tap)] : 0.f;
    case PK_ADJ:  // rows = inputs, columns = outputs
        return n < t.cin && c < t.cout ? t.w[((size_t)c * t.cin + n) * kk + (t.aux ? kk - 1 - tap : tap)] : 0.f;
    case PK_TAPROWS:  // the one output's taps as rows
        return n < kk && c < t.cin ? t.w[(size_t)c * kk + n] : 0.f;
    case PK_FE:  // rows 0..31: FE_1 on channel 0; rows 32..63: FE_2 on channel 1, its weights after FE_1's and biases
        return n < 64 && c == n >> 5 ? t.w[(n & 31) * kk + tap + (n >> 5) * 32 * (kk + 1)] : 0.f;
    case PK_Y: {  // taps as rows; columns [D 16 | FE 64 | X_0 | X_1] of the table's order D & X_0 & FE_1 & FE_2
        const int ci = c < 16 ? c : (c < 80 ? c + 1 : (c == 80 ? 16 : -1));
        return n < kk && ci >= 0 ? t.w[(size_t)ci * kk + n] : 0.f;
    }
    case PK_YADJ: {  // rows [D 16 | FE 64], columns = taps
        const int ci = n < 16 ? n : n + 1;
        return n < 80 && c < kk ? t.w[(size_t)ci * kk + c] : 0.f;
    }
    default: {  // PK_PHASE: parity class aux = 2 py + px of a stride-2, padding-2 5x5 deconvolution as a 3x3,
                // padding-1 correlation over the un-inserted input: output 2a + py takes input row a - 1 + t with
                // the weight row u = py + 4 - 2t (none outside 0..4), and likewise for columns
        const int u = (t.aux >> 1) + 4 - 2 * (tap / 3), v = (t.aux & 1) + 4 - 2 * (tap % 3);
        const bool ok = n < t.cout && c < t.cin && u >= 0 && u < t.k && v >= 0 && v < t.k;
        return ok ? t.w[((size_t)n * t.cin + c) * kk + u * t.k + v] : 0.f;
    }
    }
}

// Bound by launch latency: a training step packs 25 (Table I: 43) pieces of
// 100 to 40,000 values, which as kernels and copies of their own took 70
// (Table I: 169) us of a step and take 9 (12) here.  A workgroup takes PACK_WG values of
// one task.
constexpr int PACK_WG = 1024;
__global__ void __launch_bounds__(256) k_pack(const PackList list)
{
    int ti = 0;
    while (ti + 1 < list.n && (int)blockIdx.x >= list.task[ti + 1].first) ++ti;
    const PackTask &t = list.task[ti];
    const int total = pack_total(t);
    for (int e = ((int)blockIdx.x - t.first) * PACK_WG + threadIdx.x, k = 0; k < PACK_WG / 256 && e < total;
         e += 256, ++k) {
        const float v = pack_value(t, e);
        if (t.dt == SV_F32) ((float *)t.dst)[e] = v;
        else ((uint16_t *)t.dst)[e] = t.dt == SV_BF16 ? f32_to_bf16_bits(v) : f32_to_f16_bits(v);
    }
}

sv_status launch_pack(PackList &list, hipStream_t st) {
    int blocks = 0;
    for (int i = 0; i < list.n; ++i) {
        list.task[i].first = blocks;
        blocks += cdiv(pack_total(list.task[i]), PACK_WG);
    }
    if (blocks == 0) return SV_OK;
    hipLaunchKernelGGL(k_pack, dim3(blocks), dim3(256), 0, st, list);
    SV_LAUNCH_CHECK("k_pack");
    return SV_OK;
}

}  // namespace sv
