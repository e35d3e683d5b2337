// Fused conv1 -> conv2 -> conv3 of the Q-network, reduced precision, for more (group, sample) items than compute units: the layers,
// operands, instructions and orders of addition of conv_tower.h -- every element has the same bits -- in persistent workgroups of four
// wavefronts, two of them per compute unit (one item each up to two items per compute unit, then as equal shares as can be).
//
// What bounds it: eight wavefronts on one sample (conv_tower.h) took 6.4 us per further sample of a compute unit, of which 1.8 us
// are matrix instructions: the two wavefronts of a SIMD stand at the same barriers.  Two workgroups on two samples fill each other's
// waits: 4 us per sample, of which the vector unit issues for 2.2 us and LDS works for 2.6 us.  512 items (two networks at minibatch 256, no
// weights to change) 19.9 -> 16.7 us, 768 items 25.6 -> 21.8 us, 1024 items 32.7 -> 27.1 us; 100 train steps at minibatch 512 12.07 -> 11.64 ms.
// 3.5 us of a launch are its start, until the first frames have arrived.
//   * Wavefront (nt, kh): channel tile nt, k-quarters 2 kh and 2 kh + 1 of conv2 and conv3, one accumulator each (a sum is
//     ((p0 + p1) + p2) + p3 whoever holds the parts).  Half as many parts are exchanged as between quarters.
//   * The weight fragments of conv2 and conv3 stream through the same eighteen registers, 136 KB per item and workgroup out of L2: kept (64 + 72
//     registers) they left too few for the rest, and a register spilled behind the next item's frames waits for the frames.
//   * LDS (two workgroups: 80 KB each): the state's buffer is the exchange block's head, and act2 lies over act1 (conv2's operands have
//     been read when its sums are finished).  act1 has 64 bytes per pixel, columns of one parity side by side (a read takes every second
//     pixel) and the chunk's number exchanged by bits of column and row.  (Orders that meet no bank twice halve the conflicts, and
//     their addresses cost what that saves: 1.00x at 1024 items, 0.99x at 768.)
//   * act1 / act2 for the backward pass go to memory from LDS, 16 bytes per lane, instead of from the accumulators, 8 bytes at a stride.
#pragma once
#include "conv_tower.h"

namespace dqn {

constexpr int kManyThreads = 256;
constexpr int kManyXchgBytes = 2 * 3 * 6 * 64 * 16;   // [nt][tile][4 + 2 quads][lane] float4
static_assert(kTowerXBytes <= kManyXchgBytes, "the state buffer overlays the exchange block");
constexpr int kManyA1Bytes = 400 * 64;
static_assert(81 * kTowerP2 * 2 <= kManyA1Bytes, "act2 lies over act1");
constexpr size_t kTowerManySmem = kManyXchgBytes + 32 * 256 * 2 + kManyA1Bytes + kManyThreads * 4;
static_assert(2 * kTowerManySmem <= 160 * 1024, "two workgroups per compute unit");
static_assert((kManyXchgBytes + 32 * 256 * 2) % 64 == 0, "act1's chunks are exchanged by flipping address bits");

// act1 in LDS: byte offset of pixel (y, x)'s 64 bytes, and what its chunk numbers (8 channels each) are exchanged by.
__device__ inline int many_pixel(int y, int x) { return (y * 20 + (x & 1) * 10 + (x >> 1)) * 64; }
__device__ inline int many_flip(int y, int x) { return ((x >> 3) ^ (y & 2)) & 3; }

// The four k-quarters of a tile, held by two wavefronts: half kh has the partial sums pa, pb of quarters 2 kh, 2 kh + 1.  Half 0 keeps the
// sum of both and sends rows 8 .. 15 of it; half 1 keeps both and sends rows 0 .. 7 of either; x: this lane's place in the tile's [6][64] float4.
// (The markers keep the compiler from folding the wavefront-uniform branches into run-time register indexing.)
__device__ inline void many_send(float4* x, int kh, const f32x16& pa, const f32x16& pb, float (&keep)[16])
{
    if (kh == 0) {
        asm volatile("; send, k-half 0");
        float s[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) s[v] = pa[v] + pb[v];
#pragma unroll
        for (int q = 0; q < 2; ++q) x[q * 64] = make_float4(s[8 + 4 * q], s[9 + 4 * q], s[10 + 4 * q], s[11 + 4 * q]);
#pragma unroll
        for (int v = 0; v < 8; ++v) { keep[v] = s[v]; keep[8 + v] = 0.f; }
        asm volatile("; sent, k-half 0" ::: "memory");
    } else {
        asm volatile("; send, k-half 1");
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            x[(2 + q) * 64] = make_float4(pa[4 * q], pa[4 * q + 1], pa[4 * q + 2], pa[4 * q + 3]);
            x[(4 + q) * 64] = make_float4(pb[4 * q], pb[4 * q + 1], pb[4 * q + 2], pb[4 * q + 3]);
        }
#pragma unroll
        for (int v = 0; v < 8; ++v) { keep[v] = pa[8 + v]; keep[8 + v] = pb[8 + v]; }
        asm volatile("; sent, k-half 1" ::: "memory");
    }
}
// Rows 8 kh + 4 q .. + 3: ((p0 + p1) + p2) + p3
__device__ inline float4 many_sum(const float4* x, int kh, int q, const float (&keep)[16])
{
    float4 r;
    if (kh == 0) {
        asm volatile("; sum, k-half 0");
        const float4 c = x[(2 + q) * 64], d = x[(4 + q) * 64];
        r = make_float4((keep[4 * q] + c.x) + d.x, (keep[4 * q + 1] + c.y) + d.y, (keep[4 * q + 2] + c.z) + d.z, (keep[4 * q + 3] + c.w) + d.w);
        asm volatile("; summed, k-half 0" ::: "memory");
    } else {
        asm volatile("; sum, k-half 1");
        const float4 s = x[q * 64];
        r = make_float4((s.x + keep[4 * q]) + keep[8 + 4 * q], (s.y + keep[4 * q + 1]) + keep[9 + 4 * q], (s.z + keep[4 * q + 2]) + keep[10 + 4 * q],
                        (s.w + keep[4 * q + 3]) + keep[11 + 4 * q]);
        asm volatile("; summed, k-half 1" ::: "memory");
    }
    return r;
}

template <bool DESC>
__global__ __launch_bounds__(kManyThreads, 2) void conv_tower_many_kernel(int n_, int groups_, int share_, int tower_blocks_, const uint8_t* x0_, const uint8_t* x1_,
                                                                          const int32_t* desc_, const uint8_t* ring_, const _Float16* w1_0_, TowerArgs a)
{
    typedef bf16_t T;
    typedef bf16x8 V8;
    extern __shared__ __attribute__((aligned(16))) unsigned char tm_smem[];
    uint8_t* sX = tm_smem;                                   // live from an item's opening barrier to the end of its conv1
    float4* sXchg = reinterpret_cast<float4*>(tm_smem);      // live from conv2's matrix work to the end of the item
    _Float16* sW1 = reinterpret_cast<_Float16*>(tm_smem + kManyXchgBytes);
    unsigned char* sA1 = tm_smem + kManyXchgBytes + 32 * 256 * 2;
    T* sA2 = reinterpret_cast<T*>(sA1);
    float* sB1 = reinterpret_cast<float*>(sA1 + kManyA1Bytes);   // biases: conv1 [32], conv2 [64], conv3 [64]
    float* sB2 = sB1 + 32;
    float* sB3 = sB2 + 64;

    if (static_cast<int>(blockIdx.x) >= tower_blocks_) {   // the append that rides along (see conv_tower_kernel)
        push_step_block(a.push, static_cast<int>(blockIdx.x) - tower_blocks_);
        return;
    }
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nt = wave >> 1, kh = wave & 1;
    // Addresses are made again in every phase (the empty asm hides that they are the same for every item): kept over the loop they take a
    // hundred registers, which are in use.
    auto fresh = [](int v) { asm volatile("" : "+v"(v)); return v; };
    // workgroup j runs share_ >> 16 items, and one more if j < share_ & 0xFFFF
    const int base_items = share_ >> 16, more = share_ & 0xFFFF, wg = blockIdx.x;
    const int first = wg * base_items + min(wg, more), last = first + base_items + (wg < more ? 1 : 0);

    // The state of an item: two 16-byte vectors per thread and frame (441 vectors; the second one clamped, not predicated).  With
    // descriptors the frames are anywhere in the replay memory; a zero frame (slot -1) is loaded from slot 0 and masked when it is stored.
    u32x4 xv[4][2];
    int slots[4] = {0, 0, 0, 0};
    uint32_t keep_x[4] = {~0u, ~0u, ~0u, ~0u};
    auto fetch_slots = [&](int g, int b) {
        if constexpr (DESC) {
            const int32_t* dp = desc_ + static_cast<size_t>(b) * kDescInts + (g > 0 ? 4 : 0);
#pragma unroll
            for (int c = 0; c < 4; ++c) slots[c] = dp[c];
        }
    };
    auto fetch_state = [&](int g, int b) {
        const int t = fresh(tid);
        const uint32_t v0 = t * 16, v1 = min(t + kManyThreads, kFrameVec16 - 1) * 16;
        const uint8_t* xg = DESC ? ring_ : (g == 0 ? x0_ : g == 1 ? x1_ : a.x[g]) + static_cast<size_t>(b) * kTowerXBytes;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int slot = DESC ? __builtin_amdgcn_readfirstlane(slots[c]) : c;
            const uint8_t* frame = xg + static_cast<size_t>(max(slot, 0)) * kFrameBytes;
            xv[c][0] = *reinterpret_cast<const u32x4*>(frame + v0);
            xv[c][1] = *reinterpret_cast<const u32x4*>(frame + v1);
            if constexpr (DESC) keep_x[c] = slot < 0 ? 0u : ~0u;
        }
    };

    int g = 0, b = first;   // item = (group, sample); no run-time division (groups <= 4)
    while (b >= n_) { b -= n_; ++g; }
    fetch_slots(g, b);
    fetch_state(g, b);   // first thing on the way: everything below it is address arithmetic

    // conv3 k-steps of this wavefront's two quarters: offsets inside a pixel's window (wavefront-uniform, plain scalar arithmetic)
    int off3[18];
#pragma unroll
    for (int k = 0; k < 18; ++k) {
        const int ks = 18 * kh + k, tap = ks >> 2, p = (tap * 11) >> 5 /* tap / 3 for tap <= 8 */, q = tap - 3 * p;
        off3[k] = (p * 9 + q) * kTowerP2 + (ks & 3) * 16;
    }

    V8 wf[18];   // conv2's sixteen fragments, then conv3's eighteen, then the next item's: a slot is requested again as soon as it has been used
    int cur_g = -1;
    for (int it = first; it < last; ++it) {
        // a new group's conv1 weights are parked in LDS
        const bool new_group = g != cur_g;
        if (new_group) {
            cur_g = g;
            const _Float16* w1g = g == 0 ? w1_0_ : a.w1[g];
            f16x8 w1v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) w1v[i] = *reinterpret_cast<const f16x8*>(w1g + (tid + i * kManyThreads) * 8);
            const int bt = tid < 160 ? tid : 159;
            const float* bp = bt < 32 ? a.b1[g] + bt : (bt < 96 ? a.b2[g] + (bt - 32) : a.b3[g] + (bt - 96));
            const float bias = *bp;
#pragma unroll
            for (int i = 0; i < 4; ++i) *reinterpret_cast<f16x8*>(sW1 + (tid + i * kManyThreads) * 8) = w1v[i];
            sB1[tid] = bias;
        }
        {
            const int t = fresh(tid);
            const int v0 = t * 16, v1 = min(t + kManyThreads, kFrameVec16 - 1) * 16;   // (clamped lanes rewrite the last vector with itself)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                *reinterpret_cast<u32x4*>(sX + c * kFrameBytes + v0) = DESC ? xv[c][0] & keep_x[c] : xv[c][0];
                *reinterpret_cast<u32x4*>(sX + c * kFrameBytes + v1) = DESC ? xv[c][1] & keep_x[c] : xv[c][1];
            }
        }
        int gn = g, bn = b + 1;   // the next item
        if (bn == n_) { bn = 0; ++gn; }
        if (it + 1 < last) fetch_slots(gn, bn);
        auto w2_of = [&](int gg) { return a.w2[gg] + ((nt * 32 + kh * 16) * 64 + fresh(lane)) * 8; };
        if (it == first) {
            const T* p2 = w2_of(g);
#pragma unroll
            for (int j = 0; j < 16; ++j) wf[j] = *reinterpret_cast<const V8*>(p2 + j * 512);
        }
        __syncthreads();

        // ---- conv1: k = (c, p, q); k-step k covers c = k / 4, p = 2 * (k % 4) + kg, q = 0..7; 13 pixel tiles over four wavefronts
        {
            auto conv1 = [&](auto nt_) {
                constexpr int NT = decltype(nt_)::value, D = 3;
                const int ln = fresh(lane), lp = ln & 31, kg = ln >> 5;
                const uint8_t* base[NT];
                f32x16 acc[NT];
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    const int px = min((wave + 4 * t) * 32 + lp, 399);
                    base[t] = sX + (4 * (px / 20) + kg) * 84 + 4 * (px % 20);
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;
                }
                auto fetch_px = [&](int t, int k) {
                    const uint32_t* wp = reinterpret_cast<const uint32_t*>(base[t] + (k / 4) * 7056 + ((k % 4) * 2) * 84);
                    return make_uint2(wp[0], wp[1]);
                };
                auto fetch_w = [&](int k) { return *reinterpret_cast<const f16x8*>(sW1 + (k * 64 + ln) * 8); };
                uint2 ring_px[NT][D];
                f16x8 ring_w[D];
#pragma unroll
                for (int u = 0; u < D; ++u) {
                    ring_w[u] = fetch_w(u);
#pragma unroll
                    for (int t = 0; t < NT; ++t) ring_px[t][u] = fetch_px(t, u);
                }
#pragma unroll
                for (int k = 0; k < 16; ++k) {
                    const f16x8 w = ring_w[k % D];
                    uint2 cur[NT];
#pragma unroll
                    for (int t = 0; t < NT; ++t) cur[t] = ring_px[t][k % D];
                    if (k + D < 16) {
                        ring_w[k % D] = fetch_w(k + D);
#pragma unroll
                        for (int t = 0; t < NT; ++t) ring_px[t][k % D] = fetch_px(t, k + D);
                    }
#pragma unroll
                    for (int t = 0; t < NT; ++t)
                        acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(w, bytes_as_f16_subnormals(cur[t].x, cur[t].y), acc[t], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                }
                // scale, bias, ReLU -> LDS; rows 8q + 4kg .. + 3 are channels of this lane's pixel
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    const int px = (wave + 4 * t) * 32 + lp;
                    if (px < 400) {
                        constexpr float kScale = 16777216.f / 255.f;
                        const int y = px / 20, x = px % 20, at = many_pixel(y, x) + kg * 8, flip = many_flip(y, x);
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const float4 bv = *reinterpret_cast<const float4*>(sB1 + 8 * q + 4 * kg);
                            const float v0 = fmaxf(acc[t][4 * q] * kScale + bv.x, 0.f), v1 = fmaxf(acc[t][4 * q + 1] * kScale + bv.y, 0.f);
                            const float v2 = fmaxf(acc[t][4 * q + 2] * kScale + bv.z, 0.f), v3 = fmaxf(acc[t][4 * q + 3] * kScale + bv.w, 0.f);
                            store4<T>(reinterpret_cast<T*>(sA1 + at + ((q ^ flip) << 4)), v0, v1, v2, v3);
                        }
                    }
                }
            };
            if (wave == 0) conv1(std::integral_constant<int, 4>{}); else conv1(std::integral_constant<int, 3>{});
        }
        __syncthreads();

        // Rows 8 kh + 4 q .. + 3 of a tile, + bias, ReLU
        auto finish = [&](int ln, int t, int q, const float (&keep)[16], const float4& bias) {
            const float4 r = many_sum(sXchg + (nt * 3 + t) * (6 * 64) + ln, kh, q, keep);
            return make_float4(fmaxf(r.x + bias.x, 0.f), fmaxf(r.y + bias.y, 0.f), fmaxf(r.z + bias.z, 0.f), fmaxf(r.w + bias.w, 0.f));
        };

        // ---- conv2: k = (p, q, c), filter row p = 2 kh + h for quarter h of this wavefront; k-step k covers q = k / 2, channels 16 * (k % 2) + 8 * kg .. + 7
        {
            const int td = fresh(tid), lp = td & 31, kg = (td >> 5) & 1;
            if (T* g1 = a.act1[g]) {   // act1 to memory, whole lines
                unsigned char* out = reinterpret_cast<unsigned char*>(g1 + static_cast<size_t>(b) * 12800);
#pragma unroll
                for (int i = 0; i < 7; ++i) {
                    const int v = min(td + i * kManyThreads, 1599), px = v >> 2, y = px / 20, x = px - 20 * y;
                    *reinterpret_cast<u32x4*>(out + static_cast<uint32_t>(v) * 16) = *reinterpret_cast<const u32x4*>(sA1 + many_pixel(y, x) + (((v & 3) ^ many_flip(y, x)) << 4));
                }
            }
            const T* p3 = a.w3[g] + ((nt * 36 + kh * 18) * 64 + (td & 63)) * 8;
            float keep[3][16];
            int base[3][2];   // [q / 2]
#pragma unroll
            for (int t = 0; t < 3; ++t) {
                const int px = min(t * 32 + lp, 80), oy = px / 9, ox = px % 9;
#pragma unroll
                for (int u = 0; u < 2; ++u) base[t][u] = many_pixel(2 * (oy + kh), 2 * (ox + u)) + ((kg ^ many_flip(2 * (oy + kh), 2 * (ox + u))) << 4);
            }
            constexpr int D = 6;
            auto fetch = [&](int step) {   // (quarter, k-step, tile)
                const int t = step % 3, k = step / 3 % 8, h = step / 24, q = k >> 1;
                return *reinterpret_cast<const V8*>(sA1 + (base[t][q >> 1] ^ ((k & 1) << 5)) + h * 1280 + (q & 1) * 640);
            };
            V8 ring[D];
#pragma unroll
            for (int u = 0; u < D; ++u) ring[u] = fetch(u);
            f32x16 acc[2][3];
#pragma unroll
            for (int t = 0; t < 3; ++t)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[0][t][v] = acc[1][t][v] = 0.f;
#pragma unroll
            for (int j = 0; j < 16; ++j) {
#pragma unroll
                for (int t = 0; t < 3; ++t) {
                    const int step = 3 * j + t;
                    const V8 cur = ring[step % D];
                    if (step + D < 48) ring[step % D] = fetch(step + D);
                    mma_32x32x16(acc[j / 8][t], wf[j], cur);
                }
                wf[j] = *reinterpret_cast<const V8*>(p3 + j * 512);
                if (j < 2) wf[16 + j] = *reinterpret_cast<const V8*>(p3 + (16 + j) * 512);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int t = 0; t < 3; ++t) many_send(sXchg + (nt * 3 + t) * (6 * 64) + (td & 63), kh, acc[0][t], acc[1][t], keep[t]);
            if (it + 1 < last) fetch_state(gn, bn);   // the next item's state: in flight while conv3 runs
            else {
#pragma unroll
                for (int c = 0; c < 4; ++c) asm volatile("" : "=v"(xv[c][0]), "=v"(xv[c][1]));   // (or the old ones keep their registers until here)
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int ch = nt * 32 + 16 * kh + 8 * q + 4 * kg;
                const float4 bv = *reinterpret_cast<const float4*>(sB2 + ch);
#pragma unroll
                for (int t = 0; t < 3; ++t) {
                    const float4 v = finish(td & 63, t, q, keep[t], bv);
                    const int px = t * 32 + lp;
                    if (px < 81) store4<T>(sA2 + px * kTowerP2 + ch, v.x, v.y, v.z, v.w);
                }
            }
        }
        __syncthreads();

        // ---- conv3: k = (p, q, c); k-step ks = 18 * kh + k covers tap ks / 4, channels 16 * (ks % 4) + 8 * kg .. + 7
        {
            const int td = fresh(tid), lp = td & 31, kg = (td >> 5) & 1;
            if (T* g2 = a.act2[g]) {
                unsigned char* out = reinterpret_cast<unsigned char*>(g2 + static_cast<size_t>(b) * 5184);
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    const int v = min(td + i * kManyThreads, 647);
                    *reinterpret_cast<u32x4*>(out + static_cast<uint32_t>(v) * 16) = *reinterpret_cast<const u32x4*>(sA2 + (v >> 3) * kTowerP2 + (v & 7) * 8);
                }
            }
            float keep[2][16];
            const T* base[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int px = min(t * 32 + lp, 48);
                base[t] = sA2 + ((px / 7) * 9 + px % 7) * kTowerP2 + kg * 8;
            }
            constexpr int D = 4;
            auto fetch = [&](int step) { return *reinterpret_cast<const V8*>(base[step % 2] + off3[step / 2]); };   // (quarter, k-step, tile)
            const T* p2 = w2_of(it + 1 < last ? gn : g);
            V8 ring[D];
#pragma unroll
            for (int u = 0; u < D; ++u) ring[u] = fetch(u);
            f32x16 acc[2][2];
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[0][t][v] = acc[1][t][v] = 0.f;
#pragma unroll
            for (int j = 0; j < 18; ++j) {
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const int step = 2 * j + t;
                    const V8 cur = ring[step % D];
                    if (step + D < 36) ring[step % D] = fetch(step + D);
                    mma_32x32x16(acc[j / 9][t], wf[j], cur);
                }
                if (j < 16) wf[j] = *reinterpret_cast<const V8*>(p2 + j * 512);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int t = 0; t < 2; ++t) many_send(sXchg + (nt * 3 + t) * (6 * 64) + (td & 63), kh, acc[0][t], acc[1][t], keep[t]);
            __syncthreads();
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int ch = nt * 32 + 16 * kh + 8 * q + 4 * kg;
                const float4 bv = *reinterpret_cast<const float4*>(sB3 + ch);
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const float4 v = finish(td & 63, t, q, keep[t], bv);
                    const int px = t * 32 + lp;
                    if (px < 49) store4<T>(a.act3[g] + (static_cast<size_t>(b) * 49 + px) * 64 + ch, v.x, v.y, v.z, v.w);
                }
            }
        }
        g = gn; b = bn;
        __syncthreads();   // the exchange block is read until here; its head is the next item's state buffer
    }
}

}  // namespace dqn
