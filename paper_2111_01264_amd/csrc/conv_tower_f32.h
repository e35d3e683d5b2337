// Fused conv1 -> conv2 -> conv3 of the Q-network in full precision: the fp32 counterpart of conv_tower.h (same workgroups of 8
// wavefronts walking (group, sample) items or bands of one, activations of conv1 and conv2 in LDS), on the bf16 matrix
// instructions.  An fp32 value from 2^-110 to the largest bf16, 3.39e38, is EXACTLY the sum of three bf16 parts (8 + 8 + 8 significand bits;
// a smaller value loses at most 2^-134, the last bit of the smallest bf16), a product of two bf16 is exact in fp32, and sums are kept in fp32:
//
//   * conv1 multiplies pixel BYTES, exact in bf16, by the weights' three parts: all products are exact.  The split is made while
//     the weights are staged.
//   * conv2 and conv3 take the six largest of the nine products of parts.  What is left out is at most 2^-24 of a product (2^-27.5 root mean
//     square: 8 million random pairs), as much as the rounding of one fp32 addition, and there are fewer additions: six instructions
//     per 32 k instead of eight of four k.  The small products are summed by themselves (see tower_f32_mma); the error against 64 bits is
//     then below that of the fp32 instruction (Q rows of 36 to 200 states 2.7 .. 4.0e-7 of the network's part against 2.9 .. 4.7e-7;
//     gradients: see conv_tower_bwd_f32.h).  Six bf16 instructions take 96 cycles of a matrix core where the fp32 ones take 256: 49 k cycles
//     of a compute unit per sample become 21 k.
//   * act1 and act2 are split when they are written to LDS, once, as three planes; conv2's and conv3's weights come split from the
//     optimiser (third_index).  A wavefront owns 32 channels and a quarter of k, so that a weight is read by one wavefront only
//     (weights stream from L2: 418 KB per item) and a pixel fragment feeds two channel tiles (LDS would otherwise be as busy as the
//     matrix cores); the quarters meet in LDS, in their order.
//   * An infinity, a NaN or a value that rounds past the largest bf16 has no such parts: its second or third one is a NaN, and so is every
//     sum that it enters.  The ReLUs of conv1 and conv2 hand a NaN on (tf_relu), every activation is in some window of the next layer,
//     so conv3's sums tell: a workgroup in which one of them is no finite number runs its items once more, at its end, in plain fp32
//     (tower_f32_plain), and what such values lead to is what fp32 arithmetic makes of them.
//
// Launch times (rocprofv3), fp32 instruction -> this: sevenths (one to twelve states) 13.6 -> 12.0 us, thirds (minibatch 32) 19.4 -> 15.0 us,
// whole samples (minibatch 256) 63 -> 45 us; act step W = 1 20.3 -> 18.5 us (18.4 before it watched for values without parts).  Of a whole
// item's cycles the matrix cores need 21 k; the rest is staging, waiting in conv1 (13 tiles on 8 wavefronts) and the exchange of the sums and
// their output; by the counters the matrix cores are busy for 39 % of the launch (minibatch 256).  The whole-sample variants use 223 (by descriptors 231)
// registers and no scratch memory; 23 (29) scalars are kept in lanes of vector registers.
#pragma once
#include "conv_tower.h"
#include "wgrad_conv.h"

namespace dqn {

typedef float tf_f32x4 __attribute__((ext_vector_type(4)));

struct TowerF32Args {
    int n, groups;
    int per;                       // items per workgroup
    int tower_blocks;              // workgroups [0, tower_blocks) run the tower, the next push.L ones the append
    const uint8_t* x[kMaxGroups];  // [n][4][84][84], 16-byte aligned (unused with a descriptor table)
    const int32_t* desc;           // the minibatch as per-sample replay slots ([n][8], see TowerArgs), or null
    const uint8_t* ring;           // with desc: the replay memory's frame array
    const float* w1[kMaxGroups];   // [32][256]
    const bf16_t* w2[kMaxGroups];  // [64][512] in three parts, third_index order
    const bf16_t* w3[kMaxGroups];  // [64][576]
    const float* b1[kMaxGroups];
    const float* b2[kMaxGroups];
    const float* b3[kMaxGroups];
    const float* w2_plain[kMaxGroups];   // fp32 [64][512], [64][576]: for tower_f32_plain
    const float* w3_plain[kMaxGroups];
    float* act1[kMaxGroups];       // [n][400][32] or null
    float* act2[kMaxGroups];       // [n][81][64] or null
    float* act3[kMaxGroups];       // [n][49][64]
    PushStepPlan push;             // optional (L = 0: none): one experience per lane into the temporary buffers
};

constexpr int kTfW1Plane = 32 * 256;                   // one bf16 part of conv1's weights, fragment order (elements)
constexpr int kTfA1Plane = 400 * 64, kTfA2Plane = 81 * 128;   // one bf16 part of act1 / act2 (bytes)
constexpr int kTfXBytes = kTowerXBytes > 3 * kTfA2Plane ? kTowerXBytes : 3 * kTfA2Plane;
constexpr size_t kTowerF32Smem = kTfXBytes + 3 * kTfW1Plane * 2 + 3 * kTfA1Plane + kTowerThreads * 4 + 16;
static_assert(kTowerF32Smem <= 160 * 1024, "one workgroup per compute unit");
constexpr size_t kTfPlainSmem = (12800 + 5184) * 4 + kTowerXBytes;
static_assert(kTfPlainSmem <= kTowerF32Smem, "tower_f32_plain's activations and state");
static_assert(kTfXBytes % 16 == 0, "16-byte vectors");

// act1 in LDS: a pixel is 64 bytes, four chunks of eight channels.  The even columns of a row come before the odd ones, so that the
// stride-2 windows of consecutive output pixels start at consecutive pixels; the chunk is turned by the pixel's place in its
// group of sixteen, so that conv1's stores (one chunk of 32 pixels) meet all banks as well as conv2's reads (all chunks of 16).
__device__ inline int tf_px1(int row, int col) { return row * 20 + (col & 1) * 10 + (col >> 1); }
__device__ inline int tf_a1(int px, int chunk) { return px * 64 + ((chunk ^ ((px >> 2) & 3)) << 4); }
// act2: a pixel is 128 bytes, eight chunks, turned by the pixel
__device__ inline int tf_a2(int px, int chunk) { return px * 128 + ((chunk ^ (px & 7)) << 4); }

// Four consecutive channels into the three planes of an activation.
template <int PLANE> __device__ inline void tf_store4(uint8_t* dst, float v0, float v1, float v2, float v3)
{
    typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
    const float v[4] = {v0, v1, v2, v3};
    bf16x4 p[3];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        float r = v[e];
#pragma unroll
        for (int q = 0; q < 3; ++q) { p[q][e] = static_cast<bf16_t>(r); r -= static_cast<float>(p[q][e]); }
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) *reinterpret_cast<bf16x4*>(dst + q * PLANE) = p[q];
}

// The value, computed no earlier than here: addresses that depend on a lane's pixel are the same for every item, and the compiler
// otherwise computes those of all stages in front of the item loop and keeps them in registers throughout.  (Whole samples, forward and
// backward, had 40 to 84 bytes per lane of them in scratch memory, and a register read back behind outstanding loads waits for those: train step at
// minibatch 256 187 -> 175 us without, 140 153 -> 145 us.  Scalars in lanes of vector registers went from 12, 24 and 148 -- forward by
// states, by descriptors, backward -- to 23, 29 and 160: no memory, a few moves per item.)
__device__ inline int here(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// Element `lane` of the 1 KB row at p (wavefront-uniform), as a scalar base plus a lane offset.  Left alone, the compiler adds the
// lane's part to the base once and keeps a 64-bit vector address for every row of an unrolled stream.
__device__ inline bf16x8 load_row8(const bf16_t* p, unsigned lane)
{
    asm volatile("" : "+s"(p));
    return reinterpret_cast<const bf16x8*>(p)[lane];
}

// acc[t][c] += (16 weight rows of channel half c) x (16 pixels of tile t) over NK k-steps of 32, every product of two fp32
// values as the six largest of the nine products of their bf16 parts.  The five small ones have sums of their own: the instruction
// rounds its result to nearest, but cuts off, downwards, what lies more than 24 bits below the largest term that it adds (accumulator
// and products alike), and with all six in one accumulator dL/d(act2) was off by 5e-7 where the fp32 instruction is off by 2e-7.  at(s, t): this lane's eight channels of tile t in k-step s, first part.  The operand of
// the next tile is requested before the matrix work of this one; done(s) when the weights of step s, w[s % 5], are used up.
// live(s, t) (uniform): false for a last k-step or tile that this wavefront does not have (two bodies, one with and one without, do not
// keep their registers in place).
template <int T, int NK, int PLANE, class At, class Done, class Live>
__device__ inline void tower_f32_mma(tf_f32x4 (&acc)[T][2], bf16x8 (&w)[5][2][3], At& at, Done& done, Live live)
{
    bf16x8 x[2][3];
    tf_f32x4 low[T][2];
#pragma unroll
    for (int t = 0; t < T; ++t) low[t][0] = low[t][1] = tf_f32x4{0.f, 0.f, 0.f, 0.f};
    auto fetch = [&](auto i_) {
        constexpr int i = decltype(i_)::value, s = i / T, t = i % T;
        const uint8_t* p = at(std::integral_constant<int, s>{}, t);
#pragma unroll
        for (int q = 0; q < 3; ++q) x[i & 1][q] = *reinterpret_cast<const bf16x8*>(p + q * PLANE);
    };
    fetch(std::integral_constant<int, 0>{});
    auto step = [&](auto i_) {
        constexpr int i = decltype(i_)::value, s = i / T, t = i % T;
        if constexpr (i + 1 < NK * T)
            if (live((i + 1) / T, (i + 1) % T)) fetch(std::integral_constant<int, i + 1>{});
        constexpr int wp[6] = {2, 0, 1, 1, 0, 0}, xp[6] = {0, 2, 1, 0, 1, 0};
        if (live(s, t))
#pragma unroll
        for (int u = 0; u < 6; ++u)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                tf_f32x4& to = u < 5 ? low[t][c] : acc[t][c];
                to = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[s % 5][c][wp[u]], x[i & 1][xp[u]], to, 0, 0, 0);
            }
        if constexpr (t == T - 1) done(std::integral_constant<int, s>{});
        __builtin_amdgcn_sched_barrier(0);
    };
    static_for<0, NK * T>(step);
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int c = 0; c < 2; ++c) acc[t][c] += low[t][c];
}
// The same for all T tiles without sums for the small products, where there are no registers for them: the small products of all k-steps
// first, then the large ones, whose operand (first parts only) is read again, five tiles ahead.
template <int T, int NK, int PLANE, class At, class Done, class Live>
__device__ inline void tower_f32_mma_passes(tf_f32x4 (&acc)[T][2], bf16x8 (&w)[5][2][3], At& at, Done& done, Live live)
{
    bf16x8 x[2][3];
    auto fetch = [&](auto i_) {
        constexpr int i = decltype(i_)::value;
        const uint8_t* p = at(std::integral_constant<int, i / T>{}, i % T);
#pragma unroll
        for (int q = 0; q < 3; ++q) x[i & 1][q] = *reinterpret_cast<const bf16x8*>(p + q * PLANE);
    };
    fetch(std::integral_constant<int, 0>{});
    auto small = [&](auto i_) {
        constexpr int i = decltype(i_)::value, s = i / T, t = i % T;
        if constexpr (i + 1 < NK * T)
            if (live((i + 1) / T, (i + 1) % T)) fetch(std::integral_constant<int, i + 1>{});
        constexpr int wp[5] = {2, 0, 1, 1, 0}, xp[5] = {0, 2, 1, 0, 1};
        if (live(s, t))
#pragma unroll
        for (int u = 0; u < 5; ++u)
#pragma unroll
            for (int c = 0; c < 2; ++c) acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[s % 5][c][wp[u]], x[i & 1][xp[u]], acc[t][c], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    static_for<0, NK * T>(small);
    auto fetch0 = [&](auto i_) {
        constexpr int i = decltype(i_)::value;
        if (live(i / T, i % T)) x[i % 6 / 3][i % 3] = *reinterpret_cast<const bf16x8*>(at(std::integral_constant<int, i / T>{}, i % T));
    };
    static_for<0, 5>(fetch0);
    auto large = [&](auto i_) {
        constexpr int i = decltype(i_)::value, s = i / T, t = i % T;
        if constexpr (i + 5 < NK * T) fetch0(std::integral_constant<int, i + 5>{});
        if (live(s, t))
#pragma unroll
        for (int c = 0; c < 2; ++c) acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[s % 5][c][0], x[i % 6 / 3][i % 3], acc[t][c], 0, 0, 0);
        if constexpr (t == T - 1) done(std::integral_constant<int, s>{});
        __builtin_amdgcn_sched_barrier(0);
    };
    static_for<0, NK * T>(large);
}
template <int T, int NK, int PLANE, class At, class Done, class Live>
__device__ inline void tower_f32_tiles(tf_f32x4 (&acc)[T][2], bf16x8 (&w)[5][2][3], At& at, Done& done, Live live)
{
    static_assert(T < 4 || (NK * T >= 5 && NK <= 5), "five requests ahead; every k-step's weights are there");
    if constexpr (T >= 4) tower_f32_mma_passes<T, NK, PLANE>(acc, w, at, done, live);
    else tower_f32_mma<T, NK, PLANE>(acc, w, at, done, live);
}

// The k-quarters of the 2 T tiles of 32 channels meet: wavefront (cp, kq) finishes tiles [kq * OWN, + OWN), adds the quarters in their order and
// hands the sums to finish(i, t, c, sum), i counting its own.  ex: 2 * 2 T * 3 KB of LDS that nobody reads any more.
template <int T, class Finish>
__device__ inline void tower_f32_exchange(const tf_f32x4 (&acc)[T][2], float* ex, int cp, int kq, int lane, Finish finish)
{
    constexpr int NS = 2 * T, OWN = (NS + 3) / 4;
    static_assert(2 * NS * 3 * 1024 <= 3 * kTfA1Plane, "the partial sums fit act1's place");
    tf_f32x4* slots = reinterpret_cast<tf_f32x4*>(ex) + cp * NS * 3 * 64 + lane;
    tf_f32x4 own[OWN];
#pragma unroll
    for (int j = 0; j < NS; ++j) {
        const int o = j / OWN;
        if (o == kq) own[j % OWN] = acc[j / 2][j % 2];
        else slots[(j * 3 + (kq < o ? kq : kq - 1)) * 64] = acc[j / 2][j % 2];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < OWN; ++i) {
        const int j = kq * OWN + i;
        if (j < NS) {
            const tf_f32x4 r0 = slots[(j * 3) * 64], r1 = slots[(j * 3 + 1) * 64], r2 = slots[(j * 3 + 2) * 64];
            const tf_f32x4 q0 = kq == 0 ? own[i] : r0, q1 = kq == 0 ? r0 : kq == 1 ? own[i] : r1, q2 = kq < 2 ? r1 : kq == 2 ? own[i] : r2, q3 = kq == 3 ? own[i] : r2;
            finish(i, j / 2, j % 2, ((q0 + q1) + q2) + q3);
        }
    }
}

// max(v, 0), but NaN stays NaN (fmaxf drops it); one instruction as well.
__device__ inline float tf_relu(float v) { return __builtin_elementwise_maximum(v, 0.f); }

// One item (its conv3 rows [r3, r3 + rows3) and what they depend on) in plain fp32: a thread per output, sums in the order of k.
// For values that have no three bf16 parts; cold, and as short as it can be.
template <bool DESC>
__device__ inline void tower_f32_plain(const TowerF32Args& a, int g, int b, int r3, int rows3, unsigned char* smem)
{
    const int tid = threadIdx.x;
    float* s1 = reinterpret_cast<float*>(smem);      // act1, act2 of the sample, channels last
    float* s2 = s1 + 12800;
    uint8_t* sx = reinterpret_cast<uint8_t*>(s2 + 5184);
    __threadfence();
    __syncthreads();   // every earlier store of these activations and every read of this LDS is done
    for (int v = tid; v < kTowerXBytes / 16; v += kTowerThreads) {
        uint4 px = make_uint4(0, 0, 0, 0);
        if (DESC) {
            const int slot = a.desc[static_cast<size_t>(b) * kDescInts + (g > 0 ? 4 : 0) + v / kFrameVec16];
            if (slot >= 0) px = reinterpret_cast<const uint4*>(a.ring)[static_cast<size_t>(slot) * kFrameVec16 + v % kFrameVec16];
        } else px = reinterpret_cast<const uint4*>(a.x[g] + static_cast<size_t>(b) * kTowerXBytes)[v];
        reinterpret_cast<uint4*>(sx)[v] = px;
    }
    __syncthreads();
    // rows of act1 and act2 that the next part has as well are stored by that part (see the kernel)
    const bool to_end = r3 + rows3 == 7;
    for (int i = tid; i < 20 * (2 * rows3 + 6) * 32; i += kTowerThreads) {
        const int o = i & 31, px = 40 * r3 + (i >> 5), y = px / 20, x = px % 20;
        float sum = 0.f;
#pragma unroll 16
        for (int k = 0; k < 256; ++k) sum = fmaf(a.w1[g][o * 256 + k], static_cast<float>(sx[(k >> 6) * 7056 + (4 * y + ((k >> 3) & 7)) * 84 + 4 * x + (k & 7)]), sum);
        const float v = fmaxf(sum * (1.f / 255.f) + a.b1[g][o], 0.f);
        s1[px * 32 + o] = v;
        if (a.act1[g] && (to_end || i < 40 * rows3 * 32)) a.act1[g][(static_cast<size_t>(b) * 400 + px) * 32 + o] = v;
    }
    __syncthreads();
    for (int i = tid; i < 9 * (rows3 + 2) * 64; i += kTowerThreads) {
        const int o = i & 63, px = 9 * r3 + (i >> 6), y = px / 9, x = px % 9;
        float sum = 0.f;
#pragma unroll 16
        for (int k = 0; k < 512; ++k) sum = fmaf(a.w2_plain[g][o * 512 + k], s1[((2 * y + (k >> 7)) * 20 + 2 * x + ((k >> 5) & 3)) * 32 + (k & 31)], sum);
        const float v = fmaxf(sum + a.b2[g][o], 0.f);
        s2[px * 64 + o] = v;
        if (a.act2[g] && (to_end || i < 9 * rows3 * 64)) a.act2[g][(static_cast<size_t>(b) * 81 + px) * 64 + o] = v;
    }
    __syncthreads();
    for (int i = tid; i < 7 * rows3 * 64; i += kTowerThreads) {
        const int o = i & 63, px = 7 * r3 + (i >> 6), y = px / 7, x = px % 7;
        float sum = 0.f;
#pragma unroll 16
        for (int k = 0; k < 576; ++k) sum = fmaf(a.w3_plain[g][o * 576 + k], s2[((y + k / 192) * 9 + x + k / 64 % 3) * 64 + (k & 63)], sum);
        a.act3[g][(static_cast<size_t>(b) * 49 + px) * 64 + o] = fmaxf(sum + a.b3[g][o], 0.f);
    }
}

// PARTS: a workgroup runs a whole sample, or one half / third / seventh of its output rows with the rows of conv2 and conv1 these
// depend on (see conv_tower_kernel; thirds and sevenths are the same bands); the host takes the smallest part for which the
// chip still holds every workgroup at once.
// DESC: the frames of a state come from the replay memory by descriptor, as in conv_tower_kernel.
template <bool DESC, int PARTS>
__global__ __launch_bounds__(kTowerThreads) void conv_tower_f32_kernel(int n_, int groups_, int per_, int tower_blocks_, const uint8_t* x0_,
                                                                       const uint8_t* x1_, const float* w1_0_, const bf16_t* w2_0_, TowerF32Args a)
{
    static_assert(!DESC || PARTS == 1, "descriptors come with minibatches that fill the chip");
    static_assert(PARTS == 1 || PARTS == 2 || PARTS == 3 || PARTS == 7, "whole samples, halves, thirds or sevenths");
    extern __shared__ __attribute__((aligned(16))) unsigned char tf_smem[];
    uint8_t* sX = tf_smem;             // the state; once conv1 has read it, act2's parts
    uint8_t* sA2 = tf_smem;
    bf16_t* sW1 = reinterpret_cast<bf16_t*>(tf_smem + kTfXBytes);
    uint8_t* sA1 = reinterpret_cast<uint8_t*>(sW1 + 3 * kTfW1Plane);   // act1's parts; once conv2 has read them, partial sums on their way between wavefronts
    float* sEx = reinterpret_cast<float*>(sA1);
    float* sB1 = reinterpret_cast<float*>(sA1 + 3 * kTfA1Plane);   // biases: conv1 [32], conv2 [64], conv3 [64]
    float* sB2 = sB1 + 32;
    float* sB3 = sB2 + 64;
    int* sPlain = reinterpret_cast<int*>(sB1 + kTowerThreads);     // not zero: a sum of these items was no finite number

    if (static_cast<int>(blockIdx.x) >= tower_blocks_) {
        push_step_block(a.push, static_cast<int>(blockIdx.x) - tower_blocks_);
        return;
    }
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int total = n_ * groups_;
    const int part = PARTS == 1 ? 0 : static_cast<int>(blockIdx.x % PARTS);
    const int first = PARTS == 1 ? blockIdx.x * per_ : static_cast<int>(blockIdx.x / PARTS), last = PARTS == 1 ? min(total, first + per_) : min(total, first + 1);
    if (first >= last) return;
    if (tid == 0) *sPlain = 0;
    // first conv3 row and pixel counts of this part (conv3 rows [r, r') need conv2 rows [r, r' + 2), those conv1 rows [2 r, 2 r' + 6))
    const int r3_lo = PARTS == 1 ? 0 : PARTS == 2 ? 4 * part : PARTS == 7 ? part : (part == 0 ? 0 : part == 1 ? 3 : 5);
    const int rows3 = PARTS == 1 ? 7 : PARTS == 2 ? 4 - part : PARTS == 7 ? 1 : (part == 0 ? 3 : 2);
    const int n3 = 7 * rows3, n2 = 9 * (rows3 + 2), n1 = 20 * (2 * rows3 + 6);
    // of act1 and act2, a part stores the rows that no later part has (both would store the same values, but for tower_f32_plain)
    const bool to_end = PARTS == 1 || r3_lo + rows3 == 7;
    const int own2 = to_end ? n2 : 9 * rows3, own1 = to_end ? n1 : 40 * rows3;
    constexpr int T2 = PARTS == 1 ? 6 : PARTS == 2 ? 4 : PARTS == 3 ? 3 : 2, T3 = PARTS == 1 ? 4 : PARTS == 7 ? 1 : 2;   // 16-pixel tiles of conv2 / conv3
    constexpr int T1 = PARTS == 1 ? 13 : PARTS == 2 ? 9 : PARTS == 3 ? 8 : 5;                                            // 32-pixel tiles of conv1

    constexpr int kXVecs = kTowerXBytes / 16;   // 1764
    auto last_of = [](int t) { return t + 1536 < kXVecs ? t + 1536 : kXVecs - 1; };
    uint4 xv0, xv1, xv2, xv3;                   // the state of the item to come, 16 bytes per lane and load (the last one clamped)
    // DESC: vector v of the state belongs to frame v / 441, so each of a thread's loads chooses between two neighbouring frames; a zero
    // frame (slot -1) is loaded from slot 0 and masked when it is stored.  The slots of an item are requested an item ahead.
    int dn[4] = {0, 0, 0, 0};
    uint32_t keep = 15u;
    auto fetch_desc = [&](int g_, int b_) {
        const int32_t* dp = a.desc + static_cast<size_t>(b_) * kDescInts + (g_ > 0 ? 4 : 0);
#pragma unroll
        for (int f = 0; f < 4; ++f) dn[f] = dp[f];
    };
    auto fetch_state = [&](int g_, int b_) {
        const int t = here(tid), last_vec = last_of(t);   // (kept over the loop, these addresses would be spilled)
        if constexpr (DESC) {
            const bool hi0 = t >= 441, hi1 = t + 512 >= 882, hi2 = t + 1024 >= 1323;
            const int s[4] = {hi0 ? dn[1] : dn[0], hi1 ? dn[2] : dn[1], hi2 ? dn[3] : dn[2], dn[3]};
            const int w[4] = {t - (hi0 ? 441 : 0), t + 512 - (hi1 ? 882 : 441), t + 1024 - (hi2 ? 1323 : 882), last_vec - 1323};
            const uint4* r = reinterpret_cast<const uint4*>(a.ring);
            auto vec = [&](int i) { return r[static_cast<size_t>(s[i] < 0 ? 0 : s[i]) * kFrameVec16 + w[i]]; };
            xv0 = vec(0); xv1 = vec(1); xv2 = vec(2); xv3 = vec(3);
            keep = (s[0] < 0 ? 0u : 1u) | (s[1] < 0 ? 0u : 2u) | (s[2] < 0 ? 0u : 4u) | (s[3] < 0 ? 0u : 8u);
        } else {
            const uint8_t* xg = g_ == 0 ? x0_ : g_ == 1 ? x1_ : a.x[g_];
            const uint4* xs = reinterpret_cast<const uint4*>(xg + static_cast<size_t>(b_) * kTowerXBytes);
            xv0 = xs[t]; xv1 = xs[t + 512]; xv2 = xs[t + 1024]; xv3 = xs[last_vec];
        }
    };
    int g = 0, b = first;
    while (b >= n_) { b -= n_; ++g; }
    if constexpr (DESC) fetch_desc(g, b);
    fetch_state(g, b);
    if (DESC && first + 1 < last) { if (b + 1 < n_) fetch_desc(g, b + 1); else fetch_desc(g + 1, 0); }

    const int lp = lane & 31, kg = lane >> 5;        // conv1: pixel / row of a 32x32 tile, k-half
    const int lq = lane & 15, lk = lane >> 4;        // conv2, conv3: pixel / row of a 16x16 tile, eight of 32 k
    const int cp = wave & 1, kq = wave >> 1;         // conv2, conv3: 32 channels, k-quarter
    for (int it = first; it < last; ++it, ++b) {
        if (b == n_) { b = 0; ++g; }
        if (PARTS > 1 || it == first || b == 0) {   // first item, or the range crosses into the next group: conv1's weights and the biases
            if (it != first) __syncthreads();   // the previous item's biases have been read
            const float* w1g = g == 0 ? w1_0_ : a.w1[g];
            const int o = tid >> 4, kc = tid & 15;   // row o, k = 16 * kc .. + 15
            tf_f32x4 w[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) w[u] = *reinterpret_cast<const tf_f32x4*>(w1g + o * 256 + kc * 16 + u * 4);
            const int bt = tid < 160 ? tid : 159;
            const float* bp = bt < 32 ? a.b1[g] + bt : (bt < 96 ? a.b2[g] + (bt - 32) : a.b3[g] + (bt - 96));
            const float bias = *bp;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                bf16x8 p[3];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    float r = w[2 * h + (e >> 2)][e & 3];
#pragma unroll
                    for (int q = 0; q < 3; ++q) { p[q][e] = static_cast<bf16_t>(r); r -= static_cast<float>(p[q][e]); }
                }
#pragma unroll
                for (int q = 0; q < 3; ++q) *reinterpret_cast<bf16x8*>(sW1 + q * kTfW1Plane + ((kc * 64) + h * 32 + o) * 8) = p[q];
            }
            sB1[tid] = bias;
        }
        {
            uint4* d = reinterpret_cast<uint4*>(sX);
            if constexpr (DESC) {
                auto mask = [&](uint4& v, int i) { const uint32_t m = (keep >> i) & 1u ? ~0u : 0u; v.x &= m; v.y &= m; v.z &= m; v.w &= m; };
                mask(xv0, 0); mask(xv1, 1); mask(xv2, 2); mask(xv3, 3);
            }
            const int t = here(tid);
            d[t] = xv0; d[t + 512] = xv1; d[t + 1024] = xv2; d[last_of(t)] = xv3;   // clamped lanes rewrite the last vector with itself
        }
        // This wavefront's weights: conv2's four k-steps, and as each is used up conv3's (steps [s3, s3 + 5) or + 4 of its eighteen).
        const bf16_t* w2p = (g == 0 ? w2_0_ : a.w2[g]) + (2 * cp * 16 + 4 * kq) * 3 * 512;
        const int s3 = kq < 2 ? 5 * kq : 2 + 4 * kq;
        const bf16_t* w3p = a.w3[g] + (2 * cp * 18 + s3) * 3 * 512;
        bf16x8 wr[5][2][3];
        auto request2 = [&](auto s_) {
            constexpr int s = decltype(s_)::value;
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int q = 0; q < 3; ++q) wr[s][c][q] = load_row8(w2p + ((c * 16 + s) * 3 + q) * 512, lane);
        };
        auto request3 = [&](auto s_) {   // (quarters of four steps request their last one again)
            constexpr int s = decltype(s_)::value;
            const bf16_t* p = w3p + (s < 4 || kq < 2 ? s : 3) * 3 * 512;
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int q = 0; q < 3; ++q) wr[s][c][q] = load_row8(p + (c * 18 * 3 + q) * 512, lane);
        };
        if constexpr (PARTS == 1) static_for<0, 4>(request2);
        __syncthreads();

        // ---- conv1: k = (c, p, q); k-step k covers c = k / 4, p = 2 * (k % 4) + kg, q = 0..7 --------------------------
        {
            float* g1 = a.act1[g];
            auto run = [&](auto nt_) {
                const int lane = here(tid) & 63, kg = lane >> 5;
                constexpr int NT = decltype(nt_)::value;   // pixel tiles of this wavefront: w (and w + 8)
                const uint8_t* base[NT];
                f32x16 acc[NT];
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    const int lpx = (wave + 8 * t) * 32 + here(lp);
                    const int pc = 2 * r3_lo * 20 + (lpx < n1 ? lpx : n1 - 1);
                    base[t] = sX + (4 * (pc / 20) + kg) * 84 + 4 * (pc % 20);
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;
                }
                auto fetch_px = [&](int t, int k) {
                    const uint32_t* wp = reinterpret_cast<const uint32_t*>(base[t] + (k / 4) * 7056 + ((k % 4) * 2) * 84);
                    return make_uint2(wp[0], wp[1]);
                };
                // Operands are requested DEPTH - 1 k-steps ahead: with one tile per wavefront and hardly a second wavefront on the SIMD, a
                // k-step's 96 matrix cycles do not cover the LDS latency (one step ahead, sevenths: 4.2 k cycles for 1.5 k of matrix work).
                constexpr int DEPTH = PARTS > 1 ? 4 : 2;
                uint2 px[DEPTH][NT];
                bf16x8 wf[DEPTH][3];
                auto fetch = [&](int buf, int k) {
#pragma unroll
                    for (int q = 0; q < 3; ++q) wf[buf][q] = *reinterpret_cast<const bf16x8*>(sW1 + q * kTfW1Plane + (k * 64 + lane) * 8);
#pragma unroll
                    for (int t = 0; t < NT; ++t) px[buf][t] = fetch_px(t, k);
                };
#pragma unroll
                for (int k = 0; k < DEPTH - 1; ++k) fetch(k, k);
                auto step = [&](auto k_) {
                    constexpr int k = decltype(k_)::value;
                    if constexpr (k + DEPTH - 1 < 16) fetch((k + DEPTH - 1) % DEPTH, k + DEPTH - 1);
                    if constexpr (PARTS > 1 && k % 4 == 0) request2(std::integral_constant<int, k / 4>{});   // (all at once they would stand in front of conv1)
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        const bf16x8 x = bf16x8_from_bytes(px[k % DEPTH][t].x, px[k % DEPTH][t].y);
#pragma unroll
                        for (int q = 2; q >= 0; --q) mma_32x32x16(acc[t], wf[k % DEPTH][q], x);   // smallest part first
                    }
                    __builtin_amdgcn_sched_barrier(0);
                };
                static_for<0, 16>(step);
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    const int lpx = (wave + 8 * t) * 32 + here(lp), px1 = 2 * r3_lo * 20 + lpx;
                    if (lpx < n1) {
                        const int at = tf_px1(px1 / 20, px1 % 20);
                        constexpr float kScale = 1.f / 255.f;
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const int ch = 8 * q + 4 * kg;
                            const float4 bv = *reinterpret_cast<const float4*>(sB1 + ch);
                            const float v0 = tf_relu(acc[t][4 * q] * kScale + bv.x), v1 = tf_relu(acc[t][4 * q + 1] * kScale + bv.y);
                            const float v2 = tf_relu(acc[t][4 * q + 2] * kScale + bv.z), v3 = tf_relu(acc[t][4 * q + 3] * kScale + bv.w);
                            tf_store4<kTfA1Plane>(sA1 + tf_a1(at, q) + 8 * kg, v0, v1, v2, v3);
                            if (g1 && lpx < own1) store4<float>(g1 + (static_cast<size_t>(b) * 400 + px1) * 32 + ch, v0, v1, v2, v3);
                        }
                    }
                }
            };
            if (T1 > 8 && wave < T1 - 8) run(std::integral_constant<int, 2>{});
            else if (T1 >= 8 || wave < T1) run(std::integral_constant<int, 1>{});
            else if constexpr (PARTS > 1) static_for<0, 4>(request2);   // no tile of conv1 for this wavefront
        }
        __syncthreads();

        // ---- conv2: k = (p, q, c); this wavefront's quarter is filter row kq, a k-step is one tap ------------------------
        {
            const int lk = here(lane) >> 4;
            int base[T2];
            tf_f32x4 acc[T2][2];
#pragma unroll
            for (int t = 0; t < T2; ++t) {
                const int lpx = t * 16 + here(lq), pc = r3_lo * 9 + (lpx < n2 ? lpx : n2 - 1);
                base[t] = (2 * (pc / 9) + kq) * 20 + pc % 9;
                acc[t][0] = acc[t][1] = tf_f32x4{0.f, 0.f, 0.f, 0.f};
            }
            auto at = [&](auto s_, int t) { constexpr int s = decltype(s_)::value; return sA1 + tf_a1(base[t] + (s & 1) * 10 + (s >> 1), lk); };
            tower_f32_tiles<T2, 4, kTfA1Plane>(acc, wr, at, request3, [](int, int) { return true; });
            request3(std::integral_constant<int, 4>{});
            __syncthreads();   // act1 has been read
            float* g2 = a.act2[g];
            tower_f32_exchange<T2>(acc, sEx, cp, kq, here(lane), [&](int, int t, int c, const tf_f32x4& sum) {
                const int lpx = t * 16 + here(lq), px = r3_lo * 9 + lpx, ch = cp * 32 + c * 16 + 4 * lk;
                const float4 bv = *reinterpret_cast<const float4*>(sB2 + ch);
                if (lpx < n2) {
                    const float v0 = tf_relu(sum[0] + bv.x), v1 = tf_relu(sum[1] + bv.y), v2 = tf_relu(sum[2] + bv.z), v3 = tf_relu(sum[3] + bv.w);
                    tf_store4<kTfA2Plane>(sA2 + tf_a2(px, ch >> 3) + 2 * (ch & 4), v0, v1, v2, v3);
                    if (g2 && lpx < own2) store4<float>(g2 + (static_cast<size_t>(b) * 81 + px) * 64 + ch, v0, v1, v2, v3);
                }
            });
        }
        // the next item's state, behind the layer whose accumulators leave no registers for it
        if (it + 1 < last) {
            if (b + 1 < n_) fetch_state(g, b + 1); else fetch_state(g + 1, 0);
            if (DESC && it + 2 < last) {
                int g2 = g, b2 = b + 2;
                while (b2 >= n_) { b2 -= n_; ++g2; }
                fetch_desc(g2, b2);
            }
        } else if constexpr (PARTS == 1) {   // (or the old state keeps its registers from its stores to here)
            auto gone = [](uint4& v) { asm volatile("" : "=v"(v.x), "=v"(v.y), "=v"(v.z), "=v"(v.w)); };
            gone(xv0); gone(xv1); gone(xv2); gone(xv3);
        }
        __syncthreads();

        // ---- conv3: k = (p, q, c), two k-steps per tap ------------------------------------------------------------------
        {
            const int lk = here(lane) >> 4;
            int base[T3];
            tf_f32x4 acc[T3][2];
#pragma unroll
            for (int t = 0; t < T3; ++t) {
                const int lpx = t * 16 + here(lq), pc = r3_lo * 7 + (lpx < n3 ? lpx : n3 - 1);
                base[t] = (pc / 7) * 9 + pc % 7;
                acc[t][0] = acc[t][1] = tf_f32x4{0.f, 0.f, 0.f, 0.f};
            }
            auto at = [&](auto s_, int t) {
                const int s = s3 + decltype(s_)::value, tap = s >> 1;
                return sA2 + tf_a2(base[t] + (tap / 3) * 9 + tap % 3, 4 * (s & 1) + lk);
            };
            auto nothing = [](auto) {};
            auto all = [](int, int) { return true; };
            if (kq < 2) tower_f32_tiles<T3, 5, kTfA2Plane>(acc, wr, at, nothing, all);
            else tower_f32_tiles<T3, 4, kTfA2Plane>(acc, wr, at, nothing, all);
            // one sum over everything that this lane has is a finite number only if all are (or may overflow: no matter).  In front of the
            // exchange's barrier: behind it every wavefront knows
            tf_f32x4 all_of = acc[0][0] + acc[0][1];
#pragma unroll
            for (int t = 1; t < T3; ++t) all_of += acc[t][0] + acc[t][1];
            if (!__builtin_isfinite((all_of[0] + all_of[1]) + (all_of[2] + all_of[3]))) *sPlain = 1;
            tower_f32_exchange<T3>(acc, sEx, cp, kq, here(lane), [&](int, int t, int c, const tf_f32x4& sum) {
                const int lpx = t * 16 + here(lq), px = r3_lo * 7 + lpx, ch = cp * 32 + c * 16 + 4 * lk;
                const float4 bv = *reinterpret_cast<const float4*>(sB3 + ch);
                if (lpx < n3)
                    store4<float>(a.act3[g] + (static_cast<size_t>(b) * 49 + px) * 64 + ch, fmaxf(sum[0] + bv.x, 0.f), fmaxf(sum[1] + bv.y, 0.f),
                                  fmaxf(sum[2] + bv.z, 0.f), fmaxf(sum[3] + bv.w, 0.f));
            });
        }
        if constexpr (PARTS > 1) break;
        // no barrier: the last exchange's lies behind every read of act2, whose place the next state takes, and the next item's
        // first barrier behind the exchange's reads, whose place its act1 takes
    }
    if (*sPlain == 0) return;
    g = 0; b = first;
    while (b >= n_) { b -= n_; ++g; }
    for (int it = first; it < last; ++it, ++b) {
        if (b == n_) { b = 0; ++g; }
        tower_f32_plain<DESC>(a, g, b, r3_lo, rows3, tf_smem);
    }
}

}  // namespace dqn
