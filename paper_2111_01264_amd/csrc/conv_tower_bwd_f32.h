// Fused data-gradient chain conv3 -> conv2 in full precision: the fp32 counterpart of conv_tower_bwd.h (zero-bordered 11x11
// images of dz3 and dz2 in LDS, conv2 as four stride-1 problems) with conv_tower_f32.h's division of the work: 16x16x4 fp32
// instructions, a wavefront sums all of K for its channel tile, weights stream from L2.  Matrix-core bound: 56 k cycles a sample.
//
// The weight copies (bsh_index_w3 / bsh_index_w2<float>) hold the taps in REVERSED order, so that both the weight stream and
// the pixel addresses ascend: k = (p', q', o) with p' = KS - 1 - p reads image position (y + p', x + q').
//
// One launch per layer took 13 + 8 us at batch 32 and 41 + 30 us at batch 256; this launch takes 13 and 39 us.
#pragma once
#include "conv_tower_bwd.h"
#include "conv_tower_f32.h"

namespace dqn {

struct TowerBwdF32Args {
    const float* dz3;    // [n][49][64], already through conv3's ReLU mask
    const float* act2;   // [n][81][64]
    const float* act1;   // [n][400][32]
    const float* w3d;    // [c 64][k 576], fragment order (frag16_index)
    const float* w2d;    // four classes of [c 32][k 256], fragment order
    float* dz2;          // [n][81][64]
    float* dz1;          // [n][400][32]
    int n, per;          // samples, samples per workgroup
};

constexpr int kTbfPitch = 68;
constexpr int kTbfImg = 11 * 11 * kTbfPitch;
constexpr size_t kTowerBwdF32Smem = 2 * kTbfImg * sizeof(float);

// PARTS: whole samples, or one half / fifth of one: rows [5 part, + 5) / [2 part, + 2) of every parity class of dz1 with the rows
// of dz2 they depend on (see conv_tower_bwd_kernel).  Matrix cycles of the busiest SIMD: 56 k, 30 k, 17 k.
template <int PARTS>
__global__ __launch_bounds__(kTowerThreads) void conv_tower_bwd_f32_kernel(int n_, int per_, const float* dz3_, const float* w3d_, const float* w2d_,
                                                                           const float* act2_, const float* act1_, float* dz2_, float* dz1_)
{
    static_assert(PARTS == 1 || PARTS == 2 || PARTS == 5, "whole samples, halves or fifths");
    extern __shared__ __attribute__((aligned(16))) unsigned char tbf_smem[];
    float* sP3 = reinterpret_cast<float*>(tbf_smem);   // dz3, 7x7 at offset (2, 2) of an 11x11 image
    float* sP2 = sP3 + kTbfImg;                        // dz2, 9x9 at offset (1, 1)
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kq = lane >> 4;
    const int ct3 = wave & 3, ph = wave >> 2;          // conv3 stage: channel tile, pixel tiles ph, ph + 2, ...
    const int cls = wave & 3, ct2 = wave >> 2;         // conv2 stage: parity class (py, px) = (cls >> 1, cls & 1), channel tile
    const int part = PARTS == 1 ? 0 : static_cast<int>(blockIdx.x % PARTS);
    const int first = PARTS == 1 ? blockIdx.x * per_ : static_cast<int>(blockIdx.x / PARTS), last = PARTS == 1 ? min(n_, first + per_) : min(n_, first + 1);
    if (first >= last) return;
    // rows of this part: [y_lo, y_lo + rows) of each class; those of dz2 it depends on: [max(y_lo - 1, 0), min(y_lo + rows, 9))
    constexpr int ROWS = PARTS == 1 ? 10 : PARTS == 2 ? 5 : 2;
    const int y_lo = ROWS * part, r2_lo = max(y_lo - 1, 0), n2 = 9 * (min(y_lo + ROWS, 9) - r2_lo);
    constexpr int NC = 10 * ROWS, T2 = (NC + 15) / 16;                                  // pixels per class, tiles per wavefront of the conv2 stage
    constexpr int T3 = PARTS == 1 ? 6 : PARTS == 2 ? 3 : 2, NA = (T3 + 1) / 2, NB = T3 / 2;   // tiles of the conv3 stage; per wavefront

    // dz3 of a sample: 784 16-byte vectors, one or two per thread (the second clamped, not predicated)
    const int v1 = min(tid + 512, 783);
    auto slot = [](int v) { const int px = v >> 4; return ((px / 7 + 2) * 11 + px % 7 + 2) * kTbfPitch + (v & 15) * 4; };
    const int dst0 = slot(tid), dst1 = slot(v1);
    tf_f32x4 xv0, xv1;
    auto fetch = [&](int b) {
        const tf_f32x4* p = reinterpret_cast<const tf_f32x4*>(dz3_ + static_cast<size_t>(b) * 3136);
        xv0 = p[tid]; xv1 = p[v1];
    };
    fetch(first);
    __builtin_amdgcn_sched_barrier(0);
    for (int v = tid; v < 2 * kTbfImg / 4; v += kTowerThreads) reinterpret_cast<tf_f32x4*>(sP3)[v] = tf_f32x4{0.f, 0.f, 0.f, 0.f};   // the borders are never written again
    const float* w3 = w3d_ + ct3 * 36 * 256;
    const float* w2 = w2d_ + cls * 32 * 256 + ct2 * 16 * 256;
    auto weights = [&](int S) { return load_row(S < 36 ? w3 + S * 256 : w2 + (S - 36) * 256, lane); };
    constexpr int D3 = 12, D2 = 8;
    tf_f32x4 ring3[D3], ring2[D2], stream[kTfStream];
    __syncthreads();   // the zero fill is complete

    for (int b = first; b < last; ++b) {
        *reinterpret_cast<tf_f32x4*>(sP3 + dst0) = xv0;
        *reinterpret_cast<tf_f32x4*>(sP3 + dst1) = xv1;
        if constexpr (PARTS == 1) {
#pragma unroll
            for (int u = 0; u < D3; ++u) ring3[u] = weights(u);
        } else {
#pragma unroll
            for (int u = 0; u < kTfStream; ++u) stream[u] = weights(u);
        }
        if (b + 1 < last) fetch(b + 1);
        __syncthreads();

        // ---- conv3 data gradient ------------------------------------------------------------------------------------
        {
            const int ch = ct3 * 16 + 4 * kq;
            auto run = [&](auto nt_) {
                constexpr int NT = decltype(nt_)::value;
                const float* base[NT];
                tf_f32x4 acc[NT], mask[NT];
                const int lq = here(lane & 15);
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    const int lpx = (ph + 2 * t) * 16 + lq, pc = r2_lo * 9 + (lpx < n2 ? lpx : n2 - 1);
                    base[t] = sP3 + (pc / 9 * 11 + pc % 9) * kTbfPitch + kq * 4;
                    mask[t] = *reinterpret_cast<const tf_f32x4*>(act2_ + (static_cast<size_t>(b) * 81 + pc) * 64 + ch);   // requested now, used after the sum
                    acc[t] = tf_f32x4{0.f, 0.f, 0.f, 0.f};
                }
                if constexpr (PARTS == 1) tower_f32_rows<NT, 3, 12, 4, 11 * kTbfPitch, kTbfPitch, D3>(acc, base, w3, lane, ring3);
                else tower_f32_stream<NT, 0, 36, 12, 4, 11 * kTbfPitch, kTbfPitch, 52>(acc, base, stream, weights);
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    const int lpx = (ph + 2 * t) * 16 + lq, px = r2_lo * 9 + lpx;
                    if (lpx < n2) {
                        float v[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] = mask[t][e] > 0.f ? acc[t][e] : 0.f;
                        store4<float>(sP2 + ((px / 9 + 1) * 11 + px % 9 + 1) * kTbfPitch + ch, v[0], v[1], v[2], v[3]);
                        store4<float>(dz2_ + (static_cast<size_t>(b) * 81 + px) * 64 + ch, v[0], v[1], v[2], v[3]);
                    }
                }
            };
            if (NA == NB || ph == 0) run(std::integral_constant<int, NA>{}); else run(std::integral_constant<int, NB>{});
        }
        if constexpr (PARTS == 1) {
#pragma unroll
            for (int u = 0; u < D2; ++u) ring2[u] = weights(36 + u);
        }
        tf_f32x4 mask[T2];
        int pix[T2];
        const float* base[T2];
        const int ch = ct2 * 16 + 4 * kq, lq = here(lane & 15);
#pragma unroll
        for (int t = 0; t < T2; ++t) {
            const int lpx = t * 16 + lq, pc = y_lo * 10 + (lpx < NC ? lpx : NC - 1);
            pix[t] = (2 * (pc / 10) + (cls >> 1)) * 20 + 2 * (pc % 10) + (cls & 1);
            mask[t] = *reinterpret_cast<const tf_f32x4*>(act1_ + (static_cast<size_t>(b) * 400 + pix[t]) * 32 + ch);
            base[t] = sP2 + (pc / 10 * 11 + pc % 10) * kTbfPitch + kq * 4;
        }
        __syncthreads();

        // ---- conv2 data gradient: class cls, NC pixels -----------------------------------------------------------------
        {
            tf_f32x4 acc[T2];
#pragma unroll
            for (int t = 0; t < T2; ++t) acc[t] = tf_f32x4{0.f, 0.f, 0.f, 0.f};
            if constexpr (PARTS == 1) tower_f32_rows<T2, 2, 8, 4, 11 * kTbfPitch, kTbfPitch, D2>(acc, base, w2, lane, ring2);
            else tower_f32_stream<T2, 36, 16, 8, 4, 11 * kTbfPitch, kTbfPitch, 52>(acc, base, stream, weights);
#pragma unroll
            for (int t = 0; t < T2; ++t)
                if (t * 16 + lq < NC)
                    store4<float>(dz1_ + (static_cast<size_t>(b) * 400 + pix[t]) * 32 + ch, mask[t][0] > 0.f ? acc[t][0] : 0.f, mask[t][1] > 0.f ? acc[t][1] : 0.f,
                                  mask[t][2] > 0.f ? acc[t][2] : 0.f, mask[t][3] > 0.f ? acc[t][3] : 0.f);
        }
        if constexpr (PARTS > 1) break;
        // no barrier here: the next sample's writes to both images sit behind barriers that follow their last readers
    }
}

}  // namespace dqn
