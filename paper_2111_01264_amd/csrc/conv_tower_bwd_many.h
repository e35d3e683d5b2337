// Fused data-gradient chain conv3 -> conv2, reduced precision, for minibatches that fill the chip: the layers, operands, instructions and
// orders of addition of conv_tower_bwd.h -- every element has the same bits -- in workgroups of four wavefronts, two per
// compute unit (see conv_tower_many.h): one item each up to two samples per compute unit, above that (513 .. 1024 on 256) persistent.
//   * conv3 stage: wavefront (nt, kh) owns channel tile nt and k-quarters 2 kh, 2 kh + 1, as in conv_tower_many.h.
//   * conv2 stage: wavefront = parity class of the output pixel, both k-halves: nothing is exchanged.  Its four pixel tiles in two passes of two.
//   * The weight fragments of both stages stream through the same eighteen registers.
//   * dz1 is collected in LDS (over the exchange block, in act1's order of conv_tower_many.h) and goes to memory 16 bytes per lane, masked there
//     by act1, which is read the same way: a lane's own elements are 8 bytes at a stride of 128.
// Bound by the matrix instructions (1.6 us per sample and compute unit), the vector unit's addresses and sums, and the start until the weights
// have arrived (2 us).  Against eight wavefronts on one sample, kernel times: minibatch 512 18.9 -> 14.1 us; 256 11.4 - 12.0 -> 9.4 us and 128 10.8 -> 6.6 us as halves;
// train step at minibatch 1024 194.5 -> 169.3 us with the other changes of its kind.
#pragma once
#include "conv_tower_bwd.h"
#include "conv_tower_many.h"

namespace dqn {

constexpr size_t kTowerBwdManySmem = kManyXchgBytes + 2 * kTbImg * 2;
static_assert(2 * kTowerBwdManySmem <= 160 * 1024, "two workgroups per compute unit");
static_assert(kManyA1Bytes <= kManyXchgBytes, "dz1 is collected over the exchange block");

// PARTS = 2: an item is half a sample -- rows 5 j .. 5 j + 4 of every parity class (ten rows of dz1) with the five rows of dz2 they depend on --,
// two pixel tiles per stage instead of three and four; row 4 of dz2 is computed and stored by both halves.  One item per workgroup.
template <int PARTS>
__global__ __launch_bounds__(kManyThreads, 2) void conv_tower_bwd_many_kernel(int n_, int share_, const bf16_t* dz3_, const bf16_t* w3d_, const bf16_t* w2d_, const bf16_t* act2_,
                                                                              const bf16_t* act1_, bf16_t* dz2_, bf16_t* dz1_)
{
    typedef bf16_t T;
    typedef bf16x8 V8;
    extern __shared__ __attribute__((aligned(16))) unsigned char tbm_smem[];
    float4* sXchg = reinterpret_cast<float4*>(tbm_smem);
    unsigned char* sD1 = tbm_smem;                                 // dz1, from the end of conv3's stage to the end of the item
    T* sP3 = reinterpret_cast<T*>(tbm_smem + kManyXchgBytes);      // dz3, 7x7 at offset (2, 2) of an 11x11 image
    T* sP2 = sP3 + kTbImg;                                         // dz2, 9x9 at offset (1, 1)

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nt = wave >> 1, kh = wave & 1;     // conv3 stage
    const int py = wave >> 1, px = wave & 1;     // conv2 stage: parities of the output pixel
    auto fresh = [](int v) { asm volatile("" : "+v"(v)); return v; };   // (addresses are made again in every phase, see conv_tower_many.h)
    static_assert(PARTS == 1 || PARTS == 2, "whole samples, or halves");
    constexpr int T3 = PARTS == 1 ? 3 : 2, PASSES = PARTS == 1 ? 2 : 1;          // pixel tiles of conv3's stage; pairs of them of conv2's
    constexpr int N2 = PARTS == 1 ? 81 : 45, NC = PARTS == 1 ? 100 : 50;         // pixels of dz2, of a class of dz1
    constexpr int V2 = (N2 * 8 + kManyThreads - 1) / kManyThreads, V1 = (16 * NC + kManyThreads - 1) / kManyThreads;   // 16-byte vectors per thread of dz2, dz1
    auto sample_of = [](int it) { return PARTS == 1 ? it : it >> 1; };
    // workgroup j runs share_ >> 16 items, and one more if j < share_ & 0xFFFF
    const int base_items = share_ >> 16, more = share_ & 0xFFFF, wg = blockIdx.x;
    const int first = wg * base_items + min(wg, more), last = min(n_ * PARTS, first + base_items + (wg < more ? 1 : 0));
    if (first >= last) return;

    constexpr int kVecs3 = 49 * 8;   // dz3's 16-byte vectors: two per thread, the second one clamped
    u32x4 xv[2];
    auto fetch_dz3 = [&](int b) {
        const int t = fresh(tid);
        const unsigned char* p = reinterpret_cast<const unsigned char*>(dz3_ + static_cast<size_t>(b) * 3136);
        xv[0] = *reinterpret_cast<const u32x4*>(p + static_cast<uint32_t>(t) * 16);
        xv[1] = *reinterpret_cast<const u32x4*>(p + static_cast<uint32_t>(min(t + kManyThreads, kVecs3 - 1)) * 16);
    };
    fetch_dz3(sample_of(first));
    __builtin_amdgcn_sched_barrier(0);
    for (int v = tid; v < 2 * kTbImg / 8; v += kManyThreads) reinterpret_cast<uint4*>(sP3)[v] = make_uint4(0, 0, 0, 0);   // the borders are never written again

    V8 wf[18];   // conv3's eighteen fragments, then conv2's sixteen, then the next item's
    auto w3_of = [&]() { return w3d_ + ((nt * 36 + kh * 18) * 64 + (fresh(tid) & 63)) * 8; };
    {
        const T* p3 = w3_of();
#pragma unroll
        for (int j = 0; j < 18; ++j) wf[j] = *reinterpret_cast<const V8*>(p3 + j * 512);
    }
    // conv3 stage, k-step 18 * kh + k: tap (p, q) = (ks / 4 / 3, ks / 4 % 3), channels 16 * (ks % 4) + 8 * kg .. + 7 of
    // dz3 at (y - p, x - q): element offset relative to the pixel's own position in the padded image
    int off3[18];
#pragma unroll
    for (int k = 0; k < 18; ++k) {
        const int ks = 18 * kh + k, tap = ks >> 2, p = (tap * 11) >> 5 /* tap / 3 for tap <= 8 */, q = tap - 3 * p;
        off3[k] = -((p * 11 + q) * kTbPitch) + (ks & 3) * 16;
    }
    __syncthreads();   // the zero fill is complete

    for (int it = first; it < last; ++it) {
        const int b = sample_of(it), part = PARTS == 1 ? 0 : it & 1;
        const int y_lo = 5 * part, r2_lo = 4 * part;   // first row of each class; of dz2
        uint2 m2[T3][2];   // conv3's ReLU masks: requested now, used after the exchange
        {
            const int td = fresh(tid), lp = td & 31, kg = (td >> 5) & 1;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int v = i == 0 ? td : min(td + kManyThreads, kVecs3 - 1), p3 = v >> 3;
                *reinterpret_cast<u32x4*>(sP3 + ((p3 / 7 + 2) * 11 + p3 % 7 + 2) * kTbPitch + (v & 7) * 8) = xv[i];
            }
#pragma unroll
            for (int t = 0; t < T3; ++t)
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    m2[t][q] = *reinterpret_cast<const uint2*>(act2_ + (static_cast<size_t>(b) * 81 + r2_lo * 9 + min(t * 32 + lp, N2 - 1)) * 64 + nt * 32 + 16 * kh + 8 * q + 4 * kg);
        }
        __syncthreads();

        // ---- conv3 data gradient: 81 (45) pixels, channel tile nt, two k-quarters of 9 k-steps ------------
        {
            const int td = fresh(tid), ln = td & 63, lp = td & 31, kg = (td >> 5) & 1;
            const T* p2 = w2d_ + (wave * (32 * 256) + ln * 8);
            const T* base[T3];
#pragma unroll
            for (int t = 0; t < T3; ++t) {
                const int pc = r2_lo * 9 + min(t * 32 + lp, N2 - 1);
                base[t] = sP3 + ((pc / 9 + 2) * 11 + pc % 9 + 2) * kTbPitch + kg * 8;
            }
            constexpr int D = 6;
            auto fetch = [&](int step) { return *reinterpret_cast<const V8*>(base[step % T3] + off3[step / T3]); };   // (quarter, k-step, tile)
            V8 ring[D];
#pragma unroll
            for (int u = 0; u < D; ++u) ring[u] = fetch(u);
            f32x16 acc[2][T3];
#pragma unroll
            for (int t = 0; t < T3; ++t)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[0][t][v] = acc[1][t][v] = 0.f;
#pragma unroll
            for (int j = 0; j < 18; ++j) {
#pragma unroll
                for (int t = 0; t < T3; ++t) {
                    const int step = T3 * j + t;
                    const V8 cur = ring[step % D];
                    if (step + D < 18 * T3) ring[step % D] = fetch(step + D);
                    mma_32x32x16(acc[j / 9][t], wf[j], cur);
                }
                if (j < 16) wf[j] = *reinterpret_cast<const V8*>(p2 + j * 512);
                __builtin_amdgcn_sched_barrier(0);
            }
            float keep[T3][16];
#pragma unroll
            for (int t = 0; t < T3; ++t) many_send(sXchg + (nt * 3 + t) * (6 * 64) + ln, kh, acc[0][t], acc[1][t], keep[t]);
            __syncthreads();
#pragma unroll
            for (int t = 0; t < T3; ++t) {
                const int p2x = r2_lo * 9 + t * 32 + lp;
                T* dst = sP2 + ((p2x / 9 + 1) * 11 + p2x % 9 + 1) * kTbPitch + nt * 32 + 16 * kh + 4 * kg;
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const float4 v = many_sum(sXchg + (nt * 3 + t) * (6 * 64) + ln, kh, q, keep[t]);
                    // ReLU mask: a bf16 activation is positive iff its bit pattern is in 0x0001 .. 0x7FFF (no NaNs here)
                    const uint32_t lo = m2[t][q].x, hi = m2[t][q].y;
                    if (t * 32 + lp < N2)
                        store4<T>(dst + 8 * q, static_cast<int16_t>(lo & 0xFFFF) > 0 ? v.x : 0.f, static_cast<int16_t>(lo >> 16) > 0 ? v.y : 0.f,
                                  static_cast<int16_t>(hi & 0xFFFF) > 0 ? v.z : 0.f, static_cast<int16_t>(hi >> 16) > 0 ? v.w : 0.f);
                }
            }
        }
        __syncthreads();

        // ---- conv2 data gradient: class (py, px), 100 (50) pixels, k-step j: tap (p2, q2) = (j / 8, j / 4 % 2), channels
        // 16 * (j % 4) + 8 * kg .. + 7 of dz2 at (y2 - p2, x2 - q2)
        {
            const int td = fresh(tid), lp = td & 31, kg = (td >> 5) & 1;
            {   // dz2 to memory
                unsigned char* out = reinterpret_cast<unsigned char*>(dz2_ + static_cast<size_t>(b) * 5184);
#pragma unroll
                for (int i = 0; i < V2; ++i) {
                    const int v = r2_lo * 72 + min(td + i * kManyThreads, N2 * 8 - 1), p2x = v >> 3;
                    *reinterpret_cast<u32x4*>(out + static_cast<uint32_t>(v) * 16) = *reinterpret_cast<const u32x4*>(sP2 + ((p2x / 9 + 1) * 11 + p2x % 9 + 1) * kTbPitch + (v & 7) * 8);
                }
            }
            if (PARTS == 1) fetch_dz3(it + 1 < last ? it + 1 : it);   // the next item's: in flight while conv2's stage runs
            u32x4 m1[V1];   // conv2's ReLU masks
            const unsigned char* in1 = reinterpret_cast<const unsigned char*>(act1_ + static_cast<size_t>(b) * 12800);
#pragma unroll
            for (int i = 0; i < V1; ++i) m1[i] = *reinterpret_cast<const u32x4*>(in1 + static_cast<uint32_t>(y_lo * 160 + min(td + i * kManyThreads, 16 * NC - 1)) * 16);
            const T* p3 = w3_of();
#pragma unroll
            for (int pass = 0; pass < PASSES; ++pass) {
                const T* base[2];
                int at[2], flip[2];
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const int pc = y_lo * 10 + min((2 * pass + t) * 32 + lp, NC - 1), cy = pc / 10, cx = pc % 10;
                    base[t] = sP2 + ((cy + 1) * 11 + cx + 1) * kTbPitch + kg * 8;
                    at[t] = many_pixel(2 * cy + py, 2 * cx + px) + kg * 8;
                    flip[t] = many_flip(2 * cy + py, 2 * cx + px);
                }
                constexpr int D = 6;
                auto fetch = [&](int step) {   // (half, k-step, tile)
                    const int j = step / 2, k = j % 8;
                    return *reinterpret_cast<const V8*>(base[step % 2] - ((j / 8) * 11 + (k >> 2)) * kTbPitch + (k & 3) * 16);
                };
                V8 ring[D];
#pragma unroll
                for (int u = 0; u < D; ++u) ring[u] = fetch(u);
                f32x16 acc[2][2];
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[0][t][v] = acc[1][t][v] = 0.f;
#pragma unroll
                for (int j = 0; j < 16; ++j) {
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        const int step = 2 * j + t;
                        const V8 cur = ring[step % D];
                        if (step + D < 32) ring[step % D] = fetch(step + D);
                        mma_32x32x16(acc[j / 8][t], wf[j], cur);
                    }
                    if (PARTS == 1 && pass == PASSES - 1) {
                        wf[j] = *reinterpret_cast<const V8*>(p3 + j * 512);
                        if (j < 2) wf[16 + j] = *reinterpret_cast<const V8*>(p3 + (16 + j) * 512);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                // (lanes past the class's last pixel repeat it: the same bytes to the same place)
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        store4<T>(reinterpret_cast<T*>(sD1 + at[t] + ((q ^ flip[t]) << 4)), acc[0][t][4 * q] + acc[1][t][4 * q], acc[0][t][4 * q + 1] + acc[1][t][4 * q + 1],
                                  acc[0][t][4 * q + 2] + acc[1][t][4 * q + 2], acc[0][t][4 * q + 3] + acc[1][t][4 * q + 3]);
            }
            __syncthreads();
            unsigned char* out = reinterpret_cast<unsigned char*>(dz1_ + static_cast<size_t>(b) * 12800);
            const int te = fresh(tid);
#pragma unroll
            for (int i = 0; i < V1; ++i) {
                const int v = y_lo * 160 + min(te + i * kManyThreads, 16 * NC - 1), p1 = v >> 2, y = p1 / 20, x = p1 - 20 * y;
                // all ones where a bf16 activation is positive (0x0001 .. 0x7FFF): without its sign bit it carries into it, and the sign bit was clear
                const u32x4 act = m1[i], bit = ((((act & 0x7FFF7FFFu) + 0x7FFF7FFFu) & ~act) >> 15) & 0x00010001u, positive = (bit << 16) - bit;
                *reinterpret_cast<u32x4*>(out + static_cast<uint32_t>(v) * 16) =
                    *reinterpret_cast<const u32x4*>(sD1 + many_pixel(y, x) + (((v & 3) ^ many_flip(y, x)) << 4)) & positive;
            }
        }
        // no barrier here: the next item's writes to the images, the exchange block and over it sit behind its own barriers
    }
}

}  // namespace dqn
