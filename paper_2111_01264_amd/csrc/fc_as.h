// Activation-stationary GEMM for the fully connected layer fc1 (512 x 3136) and its data gradient.
//
//   out[b][n] = sum_k X[b][k] * W[n][k]        X: [M][ldx] activations (few rows), W: [N][ldw] weights
//
// With at most a few hundred rows of X the layer is bound by streaming W once, so the roles are
// the reverse of the convolution kernel: a workgroup parks a [32*TB][KC] slab of X in LDS and every
// wavefront streams 32 rows of W straight from global memory in MFMA operand layout (eight
// consecutive k per lane).  MFMA A = weights (row i = output feature), B = samples (column j = b),
// so lane l ends up with sample (l % 32) and four consecutive features per register quad.
//
// Weights arrive in MFMA fragment order (frag_index over [feature][k]): the operand of k-step ks of feature tile nt is
// the contiguous 1 KB (fp32: 2 KB) row (nt * K/16 + ks); row-major weights would be 32 separate 32-byte pieces per
// wavefront load, which is bound by the address unit (a full pass per cache line).
//
// K may be split over blockIdx.z: each slice then writes fp32 partial sums [slice][b][n], which the
// consumer kernel adds in slice order while it loads them (no separate reduction pass).
#pragma once
#include <atomic>

#include "head_kernels.h"
#include "vec4.h"

namespace dqn {

template <typename T> struct FcAsArgs {
    const T* x[kMaxGroups];      // [M][ldx]
    const T* w[kMaxGroups];      // [N][ldw]
    float* partial;              // kFcPartial: [group][slice][M][N] fp32
    T* dz;                       // kFcReluMask: [M][N]
    const T* mask;               // kFcReluMask: activation indexed like dz
    int M, N, ldx, ldw;
    uint32_t by_rows, by_cols;   // ceil(2^20 / row tiles), ceil(2^20 / feature blocks)
};

constexpr int kFcPartial = 0, kFcReluMask = 1;

// fc1 forward: 3136 in seven slices of 448, whose columns of X fit in LDS; its data gradient: 512, one slice.  Compile-time constants: the slab's
// index arithmetic (a division per vector, twice) and the stream's ends were more than half of the kernel's 690 vector instructions per wavefront, and
// it was those that bounded it (act step of 128 states 16.7 -> 15.2 us; train step at minibatch 48 52.7 -> 49.2 us, 160 71.4 -> 67.2, 256 with Double DQN
// 86.1 -> 82.7, 512 110.6 -> 104.3; fp32 at 256 195.1 -> 191.5).
template <int EPI> constexpr int kFcK = EPI == kFcPartial ? 448 : 512;

// This lane's 8 weights of k-step ks (16 k each) of the 32-feature tile nt; w is [N][K] in fragment order.
template <typename T> __device__ inline typename Vec8<T>::type fc_weights(const T* w, int nt, int ks, int K, int lane)
{
    const T* row = w + static_cast<size_t>(nt * (K >> 4) + ks) * 512;
    if constexpr (sizeof(T) == 2) return *reinterpret_cast<const typename Vec8<T>::type*>(row + lane * 8);
    else {
        typedef float f32x4 __attribute__((ext_vector_type(4)));
        const f32x4 lo = *reinterpret_cast<const f32x4*>(row + lane * 4), hi = *reinterpret_cast<const f32x4*>(row + 256 + lane * 4);
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    }
}

// SHARED: see the order of the workgroups.
template <typename T, int EPI, int TB, int WAVES, bool SHARED>
__global__ __launch_bounds__(WAVES * 64) void fc_as_kernel(FcAsArgs<T> a)
{
    typedef typename Vec8<T>::type V8;
    extern __shared__ __attribute__((aligned(32))) unsigned char as_smem[];
    T* sX = reinterpret_cast<T*>(as_smem);
    constexpr int KC = kFcK<EPI>, STEPS = KC / 16, LDK = KC + 8;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Workgroups are dealt out to the eight XCDs in turn, and each has an L2 of its own: an XCD takes a contiguous eighth of the
    // workgroups in the order (problem and slice, feature block, row tile), so that the row tiles that read the same weights share an L2.
    // (by_rows, by_cols: division by multiplication.  Moved at batch 256: 33 -> 18 MB forward, 31 -> 10 MB data gradient; 100 train steps at batch 256, Double DQN: 12.00 -> 11.54 ms; at batch 512: 12.40 -> 12.10.)
    int bx = blockIdx.x, by = blockIdx.y, bz = blockIdx.z;
    if constexpr (SHARED) {
        const uint32_t total = gridDim.x * gridDim.y * gridDim.z, l = bx + gridDim.x * (by + gridDim.y * bz);
        const uint32_t j = l < (total & ~7u) ? (l & 7) * (total >> 3) + (l >> 3) : l;
        const uint32_t col = j * a.by_rows >> 20;
        by = static_cast<int>(j - col * gridDim.y);
        bz = static_cast<int>(col * a.by_cols >> 20);
        bx = static_cast<int>(col - bz * gridDim.x);
    }
    const int g = EPI == kFcPartial ? bz / kFc1Slices : bz, slice = EPI == kFcPartial ? bz % kFc1Slices : 0;
    const int m0 = by * (TB * 32);
    const int k0 = slice * KC;
    const int lane_r = lane & 31, kg = lane >> 5;
    const int n = (bx * WAVES + wave) * 32 + lane_r;
    const bool n_ok = n < a.N;
    const int ntile = n_ok ? bx * WAVES + wave : 0, ks0 = k0 >> 4;   // N is a multiple of 32: tiles are whole

    // The weight stream: a ring of D k-steps of fragments in flight per wavefront, requested before the slab of X
    // is staged so that both latencies overlap.  Loads are never skipped (the k-step is clamped): the count of
    // loads in flight stays known to the compiler, which then waits for one slot only.
    constexpr int D = sizeof(T) == 2 ? 16 : 8;   // 16 KB per wavefront in flight: a step waits for the fragment requested D steps earlier, so the stream runs at D fragments per memory round trip
    static_assert(STEPS >= D, "the ring fills");
    const T* wg = a.w[g];
    auto wload = [&](int st) { return fc_weights<T>(wg, ntile, ks0 + st, a.ldw, lane); };
    V8 ring[D];
#pragma unroll
    for (int u = 0; u < D; ++u) ring[u] = wload(u);
    // kFcReluMask: the activations that mask this lane's outputs are requested now, not in the epilogue (there they were one
    // more dependent round trip to memory at the end of every workgroup); clamped addresses, no load is skipped
    [[maybe_unused]] float mask[TB][4][4];
    if constexpr (EPI == kFcReluMask) {
#pragma unroll
        for (int t = 0; t < TB; ++t) {
            const int b = min(m0 + t * 32 + lane_r, a.M - 1);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                load4<T>(a.mask + static_cast<size_t>(b) * a.N + min((bx * WAVES + wave) * 32 + 8 * q + 4 * kg, a.N - 4), mask[t][q]);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    {
        // the slab of X: eight 16-byte vectors in flight per thread (clamped address, masked value), then their LDS stores --
        // one vector per trip of a plain loop would be a chain of dependent memory round trips
        const T* xg = a.x[g];
        constexpr int VPR = KC / 8, VECS = TB * 32 * VPR, THREADS = WAVES * 64, N = (VECS + THREADS - 1) / THREADS;
        static_assert(VECS % THREADS == 0, "no ragged vectors");
#pragma unroll
        for (int i0 = 0; i0 < N; i0 += 8) {
            V8 val[8];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (i0 + u < N) {
                    const int v = tid + (i0 + u) * THREADS, r = v / VPR, kc8 = v % VPR;
                    const int row = m0 + r < a.M ? m0 + r : a.M - 1;
                    val[u] = vec8_keep<T>(*reinterpret_cast<const V8*>(xg + static_cast<size_t>(row) * a.ldx + k0 + kc8 * 8), m0 + r < a.M);
                }
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (i0 + u < N) {
                    const int v = tid + (i0 + u) * THREADS;
                    *reinterpret_cast<V8*>(&sX[(v / VPR) * LDK + (v % VPR) * 8]) = val[u];
                }
        }
    }
    __syncthreads();

    f32x16 acc[TB];
#pragma unroll
    for (int t = 0; t < TB; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;

    const T* xrow[TB];
#pragma unroll
    for (int t = 0; t < TB; ++t) xrow[t] = &sX[(t * 32 + lane_r) * LDK + kg * 8];
#pragma unroll
    for (int st = 0; st < STEPS; ++st) {
        const V8 w = ring[st % D];
        if (st + D < STEPS) ring[st % D] = wload(st + D);
#pragma unroll
        for (int t = 0; t < TB; ++t) mma_32x32x16(acc[t], w, *reinterpret_cast<const V8*>(xrow[t] + st * 16));
        __builtin_amdgcn_sched_barrier(0);
    }

    // lane: sample b = m0 + t*32 + lane_r; values: features 8*q + 4*kg + e of this wavefront's 32
    const int n_base = (bx * WAVES + wave) * 32;
#pragma unroll
    for (int t = 0; t < TB; ++t) {
        const int b = m0 + t * 32 + lane_r;
        if (b >= a.M) continue;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int nn = n_base + 8 * q + 4 * kg;
            if (nn >= a.N) continue;   // N is a multiple of 4
            if constexpr (EPI == kFcPartial) {
                float* dst = a.partial + ((static_cast<size_t>(g) * kFc1Slices + slice) * a.M + b) * a.N + nn;
                *reinterpret_cast<float4*>(dst) = make_float4(acc[t][4 * q], acc[t][4 * q + 1], acc[t][4 * q + 2], acc[t][4 * q + 3]);
            } else {
                const size_t idx = static_cast<size_t>(b) * a.N + nn;
                const float* m = mask[t][q];
                store4<T>(a.dz + idx, m[0] > 0.f ? acc[t][4 * q] : 0.f, m[1] > 0.f ? acc[t][4 * q + 1] : 0.f,
                          m[2] > 0.f ? acc[t][4 * q + 2] : 0.f, m[3] > 0.f ? acc[t][4 * q + 3] : 0.f);
            }
        }
    }
}

// Small-batch variant (at most 32 rows of X): one workgroup per (32 output features, K slice), its
// four wavefronts split the slice between them, both operands go straight from global memory into
// MFMA registers and the partial accumulators meet in LDS, added in wavefront order.  Streaming the
// 3.2 MB of fc1 weights within a few microseconds takes ~100 compute units pulling at once, hence
// the K slices across workgroups; like the large-batch kernel it then writes fp32 slices
// [group][slice][M][N] that the consumer adds in slice order.  (Finishing inside this kernel through
// a last-workgroup ticket was tried and is several times slower: the device-scope fence it needs
// writes back the L2 of the issuing XCD.)
template <typename T> struct FcSkArgs {
    const T* x[kMaxGroups];      // [M][ldx], M <= 32
    const T* w[kMaxGroups];      // [N][ldw]
    float* partial;              // kFcPartial: [group][slice][M][N] fp32
    T* dz;                       // kFcReluMask: [M][N]
    const T* mask;               // kFcReluMask: activation indexed like dz
    int M, N, ldx, ldw;
};

// The leading scalar parameters repeat FcSkArgs::x[0], x[1], w[0], w[1], M, N, ldx, ldw, partial: the kernel arguments'
// first 14 dwords are preloaded into scalar registers when a wavefront starts (see conv_tower_kernel).
template <typename T, int EPI, int KPW, int KSLICES>
__global__ __launch_bounds__(256) void fc_sk_kernel(const T* x0_, const T* x1_, const T* w0_, const T* w1_, int M_, int N_, int ldx_, int ldw_,
                                                    float* partial_, FcSkArgs<T> a)
{
    typedef typename Vec8<T>::type V8;
    static_assert(EPI == kFcPartial || KSLICES == 1, "only partial sums can be split over workgroups");
    __shared__ float red[4][16][64];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = blockIdx.y, n0 = blockIdx.x * 32, slice = blockIdx.z;
    const int lr = lane & 31, kg = lane >> 5;
    const int n = n0 + lr;
    const int k0 = (slice * 4 + wave) * (KPW * 16) + kg * 8;
    const int ntile = n < N_ ? blockIdx.x : 0, ks0 = (slice * 4 + wave) * KPW;   // N is a multiple of 32
    const bool x_ok = lr < M_;
    const T* xg = g == 0 ? x0_ : g == 1 ? x1_ : a.x[g];
    const T* wg = g == 0 ? w0_ : g == 1 ? w1_ : a.w[g];
    const T* xp = xg + static_cast<size_t>(x_ok ? lr : 0) * ldx_ + k0;
    V8 wf[KPW], xf[KPW];
#pragma unroll
    for (int s = 0; s < KPW; ++s) {
        wf[s] = fc_weights<T>(wg, ntile, ks0 + s, ldw_, lane);
        xf[s] = *reinterpret_cast<const V8*>(xp + s * 16);
    }
    // thread t finishes accumulator slots (v, l) = (4*(t/64) + e, t%64), e = 0..3: one quad of features of one sample.
    // kFcReluMask: the activations that mask them are requested now (clamped address), behind the operands -- in the
    // epilogue they were one more dependent round trip to memory at the end of a two-microsecond kernel
    const int q = tid >> 6, l = tid & 63;
    const int sample = l & 31;
    const int nn = n0 + 8 * q + 4 * (l >> 5);
    [[maybe_unused]] float m[4];
    if constexpr (EPI == kFcReluMask) load4<T>(a.mask + static_cast<size_t>(min(sample, M_ - 1)) * N_ + min(nn, N_ - 4), m);
    __builtin_amdgcn_sched_barrier(0);
    f32x16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
    for (int s = 0; s < KPW; ++s) mma_32x32x16(acc, wf[s], x_ok ? xf[s] : vec8_zero<T>());
#pragma unroll
    for (int v = 0; v < 16; ++v) red[wave][v][lane] = acc[v];
    __syncthreads();
    float v4[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
        v4[e] = ((red[0][4 * q + e][l] + red[1][4 * q + e][l]) + red[2][4 * q + e][l]) + red[3][4 * q + e][l];
    if (sample >= M_ || nn >= N_) return;
    if constexpr (EPI == kFcPartial) {
        float* dst = partial_ + ((static_cast<size_t>(g) * KSLICES + slice) * M_ + sample) * N_ + nn;
        *reinterpret_cast<float4*>(dst) = make_float4(v4[0], v4[1], v4[2], v4[3]);
    } else {
        const size_t idx = static_cast<size_t>(sample) * N_ + nn;
        store4<T>(a.dz + idx, m[0] > 0.f ? v4[0] : 0.f, m[1] > 0.f ? v4[1] : 0.f, m[2] > 0.f ? v4[2] : 0.f,
                  m[3] > 0.f ? v4[3] : 0.f);
    }
}

template <typename T, int EPI>
inline hipError_t launch_fc_as(hipStream_t st, FcAsArgs<T> a, int groups, hipEvent_t ev_begin = nullptr, hipEvent_t ev_end = nullptr)
{
    constexpr int WAVES = 4, slices = EPI == kFcPartial ? kFc1Slices : 1;
    const int n_blocks = (a.N + WAVES * 32 - 1) / (WAVES * 32);
    hipError_t e = hipSuccess;
    {
        // One 32-row tile of X per workgroup: with two, half as many workgroups read half as many weights and less of one's staging, streaming and
        // storing overlaps another's (train step at minibatch 160: 67 -> 70 us, 256 with Double DQN 82.6 -> 85.3, 512 104.3 -> 106.2).
        constexpr int TB = 1;
        const size_t smem = static_cast<size_t>(TB) * 32 * (kFcK<EPI> + 8) * sizeof(T);
        // Few workgroups keep the plain order: at 112 and 100 of them (128 states, minibatch 45) the other made no difference, and
        // finding it cost 0.1 us.  Plain order -> this one, whole call: 160 states (140 workgroups) 16.6 -> 16.7 us, fp32
        // 36.9 -> 36.5, 192 states (168) 16.9 -> 16.9, 256 (224) 17.6 -> 17.4, 512 24.7 -> 24.1; train step at minibatch 96 (168, forward only) 56.6 -> 55.6,
        // 128 (224) 59.2 -> 58.2, 160 (280, and 125 in the data gradient) 68.2 -> 67.2, 256 76.4 -> 73.2, 512 107.4 -> 103.7.
        const uint32_t rows = (a.M + TB * 32 - 1) / (TB * 32), cols = n_blocks, total = rows * cols * groups * slices;
        const bool shared = total >= 128 && rows > 1 && static_cast<uint64_t>(total) * rows < (1u << 20) && static_cast<uint64_t>(total) * cols < (1u << 20);
        a.by_rows = ((1u << 20) + rows - 1) / rows;
        a.by_cols = ((1u << 20) + cols - 1) / cols;
        auto kern = shared ? fc_as_kernel<T, EPI, TB, WAVES, true> : fc_as_kernel<T, EPI, TB, WAVES, false>;
        static std::atomic<size_t> attr_smem[2] = {{0}, {0}};   // launches come from the act thread and the train thread; setting the attribute twice is harmless
        if (smem > attr_smem[shared].load(std::memory_order_relaxed)) {
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, smem);
            if (e != hipSuccess) return e;
            attr_smem[shared].store(smem, std::memory_order_relaxed);
        }
        launch_timed(kern, dim3(n_blocks, rows, groups * slices), dim3(WAVES * 64), smem, st, ev_begin, ev_end, a);
    }
    e = hipGetLastError();
    return e;
}

}  // namespace dqn
