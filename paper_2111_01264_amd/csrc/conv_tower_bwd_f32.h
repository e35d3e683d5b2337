// Fused data-gradient chain conv3 -> conv2 in full precision: the fp32 counterpart of conv_tower_bwd.h (zero-bordered 11x11
// images of dz3 and dz2 in LDS, conv2 as four stride-1 problems) on the bf16 matrix instructions with values in three exact parts, see
// conv_tower_f32.h: 56 k cycles of a compute unit per sample on the fp32 instruction, 24 k so.  conv3's stage is divided as the
// forward layers are (32 channels and a quarter of k per wavefront); conv2's stage gives a wavefront one parity class, half of its pixels
// and all of k.  Launch times (rocprofv3), fp32 instruction -> this: minibatch 32 13.6 -> 11.4 us, minibatch 256 39.6 -> 24.6 us
// (matrix cores busy for 36 %; whole samples use 245 registers, no scratch memory, and keep 160 scalars in lanes of vector registers).
//
// The weight copies (bsh_store_w3, bsh_store_w2) hold the taps in REVERSED order, so that the pixel addresses ascend with the
// weight stream: k = (p', q', o) with p' = KS - 1 - p reads image position (y + p', x + q').
//
// Every second sample is run with its gradient negated (its images in LDS hold -dz3 and -dz2; what is stored is turned back).  The bf16
// instruction rounds its sum to nearest, but aligns what it adds to the largest term and cuts the rest off DOWNWARDS: dz2 came out -8e-9 of
// its mean magnitude off on average (whole samples; up to -1.9e-8 with weights spread over three decades), which is an eighth of
// its rounding error, but the weight and bias gradients are sums over 81 B of these, the rounding errors average out there and an
// offset does not: at minibatch 256 dL/d(conv2.b) was off by 1.2e-6 where the fp32 instruction is off by 3.8e-7.  Negated, the
// cut points upwards, and the offsets of the minibatch's two halves take each other out: 3.6e-7, and every other tensor at
// minibatch 16 to 512 is as near to 64 bits as with the fp32 instruction or nearer (conv1.w 2.6 .. 6.7e-7 against 4.4 .. 16e-7).
//
// Values that have no three bf16 parts (see conv_tower_f32.h) are found by what they leave behind the masks, dz2 or dz1 that are no finite
// number; the workgroup then runs its samples again in plain fp32 (tower_bwd_f32_plain).
#pragma once
#include "conv_tower_bwd.h"
#include "conv_tower_f32.h"

namespace dqn {

// v, or -v where flip is the sign bit.
__device__ inline tf_f32x4 tf_flip(const tf_f32x4& v, uint32_t flip)
{
    return __builtin_bit_cast(tf_f32x4, __builtin_bit_cast(wg_u32x4, v) ^ flip);
}

struct TowerBwdF32Args {
    const float* dz3;    // [n][49][64], already through conv3's ReLU mask
    const float* act2;   // [n][81][64]
    const float* act1;   // [n][400][32]
    const bf16_t* w3d;   // [c 64][k 576] in three parts, third_index order
    const bf16_t* w2d;   // four classes of [c 32][k 256]
    float* dz2;          // [n][81][64]
    float* dz1;          // [n][400][32]
    const float* w3_plain;   // fp32 [o][p][q][c]: for tower_bwd_f32_plain
    const float* w2_plain;
    int n, per;          // samples, samples per workgroup
};

constexpr int kTbfPlane = 11 * 11 * 128;                 // one bf16 part of an image (bytes; layout as act2's, see tf_a2)
constexpr int kTbfXchg = 2 * 12 * 3 * 1024;              // partial sums between wavefronts: over dz3's image once that has been read
constexpr size_t kTowerBwdF32Smem = 3 * kTbfPlane + kTbfXchg + 16;
static_assert((3136 + 5184) * 4 + 16 <= kTowerBwdF32Smem, "tower_bwd_f32_plain's images");
static_assert(kTbfXchg >= 3 * kTbfPlane, "the image of dz3 and the partial sums share their place");

// One sample's rows [y, y + rows) of every parity class of dz1, and the rows of dz2 that they depend on, in plain fp32: a thread per output.
// Taps that fall outside the gradient below are products with zero, as in the zero-bordered images.  Cold.
__device__ inline void tower_bwd_f32_plain(const float* dz3, const float* w3, const float* w2, const float* act2, const float* act1, float* dz2, float* dz1,
                                           int b, int y_lo, int rows, unsigned char* smem)
{
    const int tid = threadIdx.x;
    float* s3 = reinterpret_cast<float*>(smem);   // dz3, dz2 of the sample, channels last
    float* s2 = s3 + 3136;
    __threadfence();
    __syncthreads();   // every earlier store of these gradients and every read of this LDS is done
    for (int v = tid; v < 3136; v += kTowerThreads) s3[v] = dz3[static_cast<size_t>(b) * 3136 + v];
    __syncthreads();
    const int r2_lo = max(y_lo - 1, 0), n2 = 9 * (min(y_lo + rows, 9) - r2_lo);
    for (int i = tid; i < n2 * 64; i += kTowerThreads) {
        const int c = i & 63, px = 9 * r2_lo + (i >> 6), y = px / 9, x = px % 9;
        float sum = 0.f;
#pragma unroll 16
        for (int k = 0; k < 576; ++k) {
            const int o = k & 63, p = k / 192, q = k / 64 % 3, yy = y - p, xx = x - q;
            sum = fmaf(w3[o * 576 + (p * 3 + q) * 64 + c], yy >= 0 && yy < 7 && xx >= 0 && xx < 7 ? s3[(yy * 7 + xx) * 64 + o] : 0.f, sum);
        }
        const size_t at = (static_cast<size_t>(b) * 81 + px) * 64 + c;
        const float v = act2[at] > 0.f ? sum : 0.f;
        s2[px * 64 + c] = v;
        if (px >= 9 * y_lo) dz2[at] = v;   // (the row above belongs to the part above)
    }
    __syncthreads();
    for (int i = tid; i < 2 * rows * 20 * 32; i += kTowerThreads) {
        const int c = i & 31, px = 40 * y_lo + (i >> 5), y = px / 20, x = px % 20;
        float sum = 0.f;
#pragma unroll 16
        for (int k = 0; k < 256; ++k) {
            const int o = k & 63, p2 = k >> 7, q2 = (k >> 6) & 1, yy = (y >> 1) - p2, xx = (x >> 1) - q2;
            sum = fmaf(w2[o * 512 + ((2 * p2 + (y & 1)) * 4 + 2 * q2 + (x & 1)) * 32 + c], yy >= 0 && yy < 9 && xx >= 0 && xx < 9 ? s2[(yy * 9 + xx) * 64 + o] : 0.f, sum);
        }
        const size_t at = (static_cast<size_t>(b) * 400 + px) * 32 + c;
        dz1[at] = act1[at] > 0.f ? sum : 0.f;
    }
}

// PARTS: whole samples, or one half / fifth of one: rows [5 part, + 5) / [2 part, + 2) of every parity class of dz1 with the rows
// of dz2 they depend on (see conv_tower_bwd_kernel).
template <int PARTS>
__global__ __launch_bounds__(kTowerThreads) void conv_tower_bwd_f32_kernel(int n_, int per_, const float* dz3_, const bf16_t* w3d_, const bf16_t* w2d_,
                                                                           const float* act2_, const float* act1_, float* dz2_, float* dz1_,
                                                                           const float* w3_plain, const float* w2_plain)
{
    static_assert(PARTS == 1 || PARTS == 2 || PARTS == 5, "whole samples, halves or fifths");
    extern __shared__ __attribute__((aligned(16))) unsigned char tbf_smem[];
    uint8_t* sP2 = tbf_smem;                             // dz2, 9x9 at offset (1, 1)
    uint8_t* sP3 = tbf_smem + 3 * kTbfPlane;             // dz3, 7x7 at offset (2, 2) of an 11x11 image
    float* sEx = reinterpret_cast<float*>(sP3);
    int* sPlain = reinterpret_cast<int*>(tbf_smem + kTowerBwdF32Smem - 16);   // not zero: a gradient of these samples is no finite number
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lq = lane & 15, lk = lane >> 4;
    const int cp = wave & 1, kq = wave >> 1;             // conv3 stage: 32 channels, k-quarter
    const int cls = wave & 3, ph = wave >> 2;            // conv2 stage: parity class (py, px) = (cls >> 1, cls & 1), pixel tiles ph, ph + 2, ...
    const int part = PARTS == 1 ? 0 : static_cast<int>(blockIdx.x % PARTS);
    const int first = PARTS == 1 ? blockIdx.x * per_ : static_cast<int>(blockIdx.x / PARTS), last = PARTS == 1 ? min(n_, first + per_) : min(n_, first + 1);
    if (first >= last) return;
    // rows of this part: [y_lo, y_lo + rows) of each class; those of dz2 it depends on: [max(y_lo - 1, 0), min(y_lo + rows, 9))
    constexpr int ROWS = PARTS == 1 ? 10 : PARTS == 2 ? 5 : 2;
    const int y_lo = ROWS * part, r2_lo = max(y_lo - 1, 0), n2 = 9 * (min(y_lo + ROWS, 9) - r2_lo);
    constexpr int NC = 10 * ROWS, T2 = (NC + 15) / 16, TA = (T2 + 1) / 2, TB = T2 / 2;   // pixels per class, tiles of the conv2 stage; per wavefront
    constexpr int T3 = PARTS == 1 ? 6 : PARTS == 2 ? 3 : 2, OWN = (2 * T3 + 3) / 4;      // tiles of the conv3 stage; sums a wavefront finishes

    // dz3 of a sample: 784 16-byte vectors, one or two per thread (the second clamped, not predicated)
    auto slot = [&](int v) { const int px = v >> 4; return sP3 + tf_a2((px / 7 + 2) * 11 + px % 7 + 2, (v & 15) >> 1) + 8 * (v & 1); };
    tf_f32x4 xv0, xv1;
    auto fetch = [&](int b) {
        const int t = here(tid);
        const tf_f32x4* p = reinterpret_cast<const tf_f32x4*>(dz3_ + static_cast<size_t>(b) * 3136);
        xv0 = p[t]; xv1 = p[min(t + 512, 783)];
    };
    fetch(first);
    __builtin_amdgcn_sched_barrier(0);
    // conv3's weights: k-steps [s3, s3 + 5) or + 4 of eighteen; conv2's: this class's eight; both through five slots
    const int s3 = kq < 2 ? 5 * kq : 2 + 4 * kq;
    const bf16_t* w3 = w3d_ + (2 * cp * 18 + s3) * 3 * 512;
    const bf16_t* w2 = w2d_ + cls * 3 * 32 * 256;
    bf16x8 wr[5][2][3];
    auto request3 = [&](auto s_) {   // (quarters of four steps request their last one again)
        constexpr int s = decltype(s_)::value;
        const bf16_t* p = w3 + (s < 4 || kq < 2 ? s : 3) * 3 * 512;
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int q = 0; q < 3; ++q) wr[s % 5][c][q] = load_row8(p + (c * 18 * 3 + q) * 512, lane);
    };
    auto request2 = [&](auto s_) {
        constexpr int s = decltype(s_)::value;
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int q = 0; q < 3; ++q) wr[s % 5][c][q] = load_row8(w2 + ((c * 8 + s) * 3 + q) * 512, lane);
    };
    static_for<0, 5>(request3);
    for (int v = tid; v < 6 * kTbfPlane / 16; v += kTowerThreads) reinterpret_cast<uint4*>(tbf_smem)[v] = make_uint4(0, 0, 0, 0);
    if (tid == 0) *sPlain = 0;
    __syncthreads();   // the zero fill is complete

    for (int b = first; b < last; ++b) {
        if (PARTS == 1 && b != first) {   // dz3's border again, where partial sums have been: 22 + 22 pixels above and below, 28 beside
            for (int v = here(tid); v < 3 * 72 * 8; v += kTowerThreads) {
                const int pl = v / 576, i = v % 576 >> 3, j = i - 44;
                const int px = i < 22 ? i : i < 44 ? 77 + i : (2 + (j >> 2)) * 11 + ((j & 3) < 2 ? j & 3 : 7 + (j & 3));
                *reinterpret_cast<uint4*>(sP3 + pl * kTbfPlane + px * 128 + (v & 7) * 16) = make_uint4(0, 0, 0, 0);
            }
        }
        const uint32_t flip = (b & 1) ? 0x80000000u : 0u;
        xv0 = tf_flip(xv0, flip);
        xv1 = tf_flip(xv1, flip);
        tf_store4<kTbfPlane>(slot(here(tid)), xv0[0], xv0[1], xv0[2], xv0[3]);
        tf_store4<kTbfPlane>(slot(min(here(tid) + 512, 783)), xv1[0], xv1[1], xv1[2], xv1[3]);
        __syncthreads();

        // ---- conv3 data gradient ------------------------------------------------------------------------------------
        {
            const int lk = here(lane) >> 4;
            int base[T3];
            tf_f32x4 acc[T3][2];
#pragma unroll
            for (int t = 0; t < T3; ++t) {
                const int lpx = t * 16 + here(lq), pc = r2_lo * 9 + (lpx < n2 ? lpx : n2 - 1);
                base[t] = pc / 9 * 11 + pc % 9;
                acc[t][0] = acc[t][1] = tf_f32x4{0.f, 0.f, 0.f, 0.f};
            }
            auto at = [&](auto s_, int t) {
                const int s = s3 + decltype(s_)::value, tap = s >> 1;
                return sP3 + tf_a2(base[t] + (tap / 3) * 11 + tap % 3, 4 * (s & 1) + lk);
            };
            tower_f32_tiles<T3, 5, kTbfPlane>(acc, wr, at, request2, [kq](int s, int) { return s < 4 || kq < 2; });
            // the activations that mask what this wavefront will finish: ahead of the partial sums' exchange
            tf_f32x4 mask3[OWN];
#pragma unroll
            for (int i = 0; i < OWN; ++i) {
                const int j = min(kq * OWN + i, 2 * T3 - 1), lpx = (j >> 1) * 16 + here(lq), pc = r2_lo * 9 + (lpx < n2 ? lpx : n2 - 1);
                mask3[i] = *reinterpret_cast<const tf_f32x4*>(act2_ + (static_cast<size_t>(b) * 81 + pc) * 64 + cp * 32 + (j & 1) * 16 + 4 * lk);
            }
            __syncthreads();   // dz3 has been read
            tf_f32x4 all_of = {0.f, 0.f, 0.f, 0.f};   // the sum of what this lane finishes is a finite number only if all of it is
            tower_f32_exchange<T3>(acc, sEx, cp, kq, here(lane), [&](int i, int t, int c, const tf_f32x4& sum) {
                const int lpx = t * 16 + here(lq), px = r2_lo * 9 + lpx, ch = cp * 32 + c * 16 + 4 * lk;
                if (lpx < n2) {
                    tf_f32x4 v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = mask3[i][e] > 0.f ? sum[e] : 0.f;
                    tf_store4<kTbfPlane>(sP2 + tf_a2((px / 9 + 1) * 11 + px % 9 + 1, ch >> 3) + 2 * (ch & 4), v[0], v[1], v[2], v[3]);
                    v = tf_flip(v, flip);
                    all_of += v;
                    if (px >= 9 * y_lo) store4<float>(dz2_ + (static_cast<size_t>(b) * 81 + px) * 64 + ch, v[0], v[1], v[2], v[3]);
                }
            });
            if (!__builtin_isfinite((all_of[0] + all_of[1]) + (all_of[2] + all_of[3]))) *sPlain = 1;
        }
        __syncthreads();

        // ---- conv2 data gradient: class cls, NC pixels -----------------------------------------------------------------
        {
            constexpr int NT = TA;
            const int lk = here(lane) >> 4;
            int base[NT];
            tf_f32x4 acc[NT][2], mask[NT][2];
            auto place = [&](int t) {   // this lane's pixel of tile t in dz1
                const int lpx = (ph + 2 * t) * 16 + here(lq), pc = y_lo * 10 + (lpx < NC ? lpx : NC - 1);
                return (2 * (pc / 10) + (cls >> 1)) * 20 + 2 * (pc % 10) + (cls & 1);
            };
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const int lpx = (ph + 2 * t) * 16 + here(lq), pc = y_lo * 10 + (lpx < NC ? lpx : NC - 1);
                base[t] = pc / 10 * 11 + pc % 10;
#pragma unroll
                for (int c = 0; c < 2; ++c) acc[t][c] = tf_f32x4{0.f, 0.f, 0.f, 0.f};
            }
            auto at = [&](auto s_, int t) {
                constexpr int s = decltype(s_)::value, tap = s >> 1;
                return sP2 + tf_a2(base[t] + (tap >> 1) * 11 + (tap & 1), 4 * (s & 1) + lk);
            };
            auto next = [&](auto s_) {   // the last three k-steps' weights, then (in their predecessors' registers) the masks
                constexpr int s = decltype(s_)::value;
                if constexpr (s < 3) request2(std::integral_constant<int, s + 5>{});
                if constexpr (s == 5 && PARTS == 1) {
                    if (b + 1 < last) fetch(b + 1);
                    else asm volatile("" : "=v"(xv0), "=v"(xv1));   // (or the old ones keep their registers until here)
                }
                if constexpr (s == 4)
#pragma unroll
                    for (int t = 0; t < NT; ++t)
#pragma unroll
                        for (int c = 0; c < 2; ++c)
                            mask[t][c] = *reinterpret_cast<const tf_f32x4*>(act1_ + (static_cast<size_t>(b) * 400 + place(t)) * 32 + c * 16 + 4 * lk);
            };
            tower_f32_mma<NT, 8, kTbfPlane>(acc, wr, at, next, [ph](int, int t) { return TA == TB || t < TA - 1 || ph == 0; });
            tf_f32x4 all_of = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int t = 0; t < NT; ++t)
                if ((ph + 2 * t) * 16 + lq < NC)
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        tf_f32x4 v = tf_flip(acc[t][c], flip);
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] = mask[t][c][e] > 0.f ? v[e] : 0.f;
                        store4<float>(dz1_ + (static_cast<size_t>(b) * 400 + place(t)) * 32 + c * 16 + 4 * lk, v[0], v[1], v[2], v[3]);
                        all_of += v;
                    }
            if (!__builtin_isfinite((all_of[0] + all_of[1]) + (all_of[2] + all_of[3]))) *sPlain = 1;
        }
        if constexpr (PARTS > 1) break;
        if (b + 1 < last) static_for<0, 5>(request3);
        // no barrier here: the next sample's writes to both images sit behind barriers that follow their last readers
    }
    __syncthreads();
    if (*sPlain == 0) return;
    for (int b = first; b < last; ++b) tower_bwd_f32_plain(dz3_, w3_plain, w2_plain, act2_, act1_, dz2_, dz1_, b, y_lo, ROWS, tbf_smem);
}

}  // namespace dqn
