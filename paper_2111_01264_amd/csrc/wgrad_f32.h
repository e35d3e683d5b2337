// Every weight gradient of a full-precision train step in ONE launch: the fp32 counterpart of wgrad_all.h, with the same
// division of the work (conv layers sample by sample, fc1 tile by tile over the minibatch, then the small reductions).
//
// conv2, conv3 and fc1 run on the fp32 matrix instruction (32x32x2: one element per lane and operand, 64 cycles).  Both
// operands of a weight gradient are stored with the contraction index as the slow one, and this instruction wants exactly
// that: lane l holds row / column l % 32 at contraction index l / 32, so a fragment is one 4-byte LDS read per lane of 32
// consecutive elements of two rows -- no transposition, no bank conflict, and one read feeds 64 cycles of the matrix core.
// What bounds the launch is therefore the matrix core: 42 MMAC x B at 32 MAC per cycle and SIMD (conv1, which would be a third
// of that, runs on the bf16 instruction instead, see WgConv1F32).
//
// Tiled implicit GEMMs that transposed on the way into LDS (one launch per layer, at most 32 slices) took 30 + 8 + 8 + 7 + 5 us
// at batch 32 and 200 + 33 + 29 + 26 + 7 us at batch 256; this launch takes 13 us and 45 us.
#pragma once
#include "head_kernels.h"
#include "wgrad_conv.h"

namespace dqn {

typedef float wg_f32x4 __attribute__((ext_vector_type(4)));

template <int CIN_, int HIN_, int WIN_, int COUT_, int HOUT_, int WOUT_, int KS_, int S_, int CS_>
struct WgGeoF32 {
    static constexpr int CIN = CIN_, HIN = HIN_, WIN = WIN_, COUT = COUT_, HOUT = HOUT_, WOUT = WOUT_, KS = KS_, S = S_, CS = CS_;
    static constexpr int KPIX = HOUT_ * WOUT_;                    // contraction rows per sample: 81, 49
    static constexpr int KSTEPS = (KPIX + 1) / 2;                 // two pixels per matrix instruction
    static constexpr int N = KS_ * KS_ * CIN_;                    // 512, 576
    static constexpr int NT = N / 32 / CS_;                       // 32-column tiles per workgroup: 8, 6
    static constexpr int NTW = NT / 2;                            // per wavefront: wavefront w owns row tile w % 2 and column tiles w / 2, w / 2 + 2, ...
    static constexpr int IN_VECS = HIN_ * WIN_ * CIN_ / 4, DZ_VECS = KPIX * COUT_ / 4;   // 16-byte vectors per sample
    static constexpr int NVI = (IN_VECS + 255) / 256, NVD = (DZ_VECS + 255) / 256;
    static constexpr size_t SMEM = static_cast<size_t>(HIN_ * WIN_ * CIN_ + 2 * KSTEPS * COUT_) * 4;
    static_assert(COUT_ == 64 && NT % 2 == 0, "two row tiles, an even number of column tiles");
    static_assert(HIN_ * WIN_ * CIN_ * 4 < 65536, "pixel offsets fit the LDS instructions' offset field");
};
typedef WgGeoF32<32, 20, 20, 64, 9, 9, 4, 2, 2> WgConv2F32;
typedef WgGeoF32<64, 9, 9, 64, 7, 7, 3, 1, 3> WgConv3F32;

__device__ inline void mma_32x32x2(f32x16& acc, float a, float b) { acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, acc, 0, 0, 0); }

// Workgroup (slice `wg`, column block `cb`) of a channels-last layer (256 threads; smem: G::SMEM bytes, 16-byte aligned).
template <class G>
__device__ inline void wgrad_conv_f32_block(const WgConvArgs& a, int wg, int cb, unsigned char* smem)
{
    constexpr int NTW = G::NTW, NVI = G::NVI, NVD = G::NVD;
    float* sIn = reinterpret_cast<float*>(smem);
    float* sDz = sIn + G::HIN * G::WIN * G::CIN;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 31, kg = lane >> 5;
    const int first = wg * a.per, last = min(a.n, first + a.per);
    if (first >= last) return;
    if (tid < G::COUT) sDz[(2 * G::KSTEPS - 1) * G::COUT + tid] = 0.f;   // the pixel that pads an odd count (KPIX is odd)
    static_assert(G::KPIX == 2 * G::KSTEPS - 1, "one padding pixel");

    // LDS addresses of this lane's column in each of its tiles (filter element n -> offset of its input element inside a pixel's
    // window), once for a lane half at the next pixel of the same output row, once across the end of a row (the second
    // pixel of the pair is the first of the next row), once for the padding pixel (both halves at the last pixel)
    constexpr int STEP = G::S * G::CIN, WRAP = (G::S * G::WIN - (G::WOUT - 1) * G::S) * G::CIN;
    const float* col[NTW];
#pragma unroll
    for (int j = 0; j < NTW; ++j) {
        const int n = (cb * G::NT + (wave >> 1) + 2 * j) * 32 + lr;
        col[j] = sIn + ((n / (G::KS * G::CIN)) * G::WIN + (n / G::CIN) % G::KS) * G::CIN + n % G::CIN;
    }
    const int d_step = kg * STEP, d_wrap = kg * WRAP;
    const float* arow = sDz + kg * G::COUT + (wave & 1) * 32 + lr;

    f32x16 acc[NTW];
#pragma unroll
    for (int j = 0; j < NTW; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;
    double bsum[4] = {0, 0, 0, 0};   // bias gradient: column sums of dZ (a thread's vectors share their four channels; fp64: see WgGeo's Sum)
    static_assert(256 % (G::COUT / 4) == 0, "a thread's dZ vectors share their channel chunk");

    wg_f32x4 pin[NVI], pdz[NVD];
    auto fetch = [&](int b) {
        const wg_f32x4* dzp = reinterpret_cast<const wg_f32x4*>(static_cast<const float*>(a.dz) + static_cast<size_t>(b) * G::KPIX * G::COUT);
        const wg_f32x4* inp = reinterpret_cast<const wg_f32x4*>(static_cast<const float*>(a.in) + static_cast<size_t>(b) * G::HIN * G::WIN * G::CIN);
#pragma unroll
        for (int u = 0; u < NVD; ++u) pdz[u] = dzp[min(tid + u * 256, G::DZ_VECS - 1)];
#pragma unroll
        for (int u = 0; u < NVI; ++u) pin[u] = inp[min(tid + u * 256, G::IN_VECS - 1)];
    };
    auto stash = [&]() {   // surplus threads store a copy of the last vector again (same bytes, same place)
        wg_f32x4 isum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < NVD; ++u) {
            reinterpret_cast<wg_f32x4*>(sDz)[min(tid + u * 256, G::DZ_VECS - 1)] = pdz[u];
            if (cb == 0) isum += __builtin_bit_cast(wg_f32x4, __builtin_bit_cast(wg_u32x4, pdz[u]) & (G::DZ_VECS % 256 == 0 || tid + u * 256 < G::DZ_VECS ? ~0u : 0u));
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) bsum[e] += isum[e];
#pragma unroll
        for (int u = 0; u < NVI; ++u) reinterpret_cast<wg_f32x4*>(sIn)[min(tid + u * 256, G::IN_VECS - 1)] = pin[u];
    };
    // operands of step ks + 1 are requested before the matrix work of step ks
    auto contract = [&]() {
        float fa[2], fb[2][NTW];
        auto frags = [&](auto buf_, auto ks_) {
            constexpr int buf = decltype(buf_)::value, ks = decltype(ks_)::value;
            constexpr int i = 2 * ks / G::WOUT, j = 2 * ks % G::WOUT, off = (G::S * i * G::WIN + G::S * j) * G::CIN;
            const int d = 2 * ks + 1 == G::KPIX ? 0 : j + 1 == G::WOUT ? d_wrap : d_step;
            fa[buf] = arow[2 * ks * G::COUT];
#pragma unroll
            for (int t = 0; t < NTW; ++t) {
                fb[buf][t] = (col[t] + d)[off];
                if (2 * ks + 1 == G::KPIX) fb[buf][t] = kg ? 0.f : fb[buf][t];   // the padding pixel: zero on both sides, for an infinite input
            }
        };
        frags(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
        auto step = [&](auto ks_) {
            constexpr int ks = decltype(ks_)::value, buf = ks & 1;
            if constexpr (ks + 1 < G::KSTEPS) frags(std::integral_constant<int, (ks + 1) & 1>{}, std::integral_constant<int, ks + 1>{});
#pragma unroll
            for (int t = 0; t < NTW; ++t) mma_32x32x2(acc[t], fa[buf], fb[buf][t]);
            __builtin_amdgcn_sched_barrier(0);
        };
        static_for<0, G::KSTEPS>(step);
    };

    fetch(first);
    for (int b = first; b < last; ++b) {
        if (b != first) __syncthreads();   // every wavefront has finished reading the previous sample
        stash();
        if (b + 1 < last) fetch(b + 1);
        __syncthreads();
        contract();
    }

    if (cb == 0) {   // workgroup-uniform: the threads' channel sums meet in LDS (see wgrad_conv_block)
        __syncthreads();
        constexpr int LDS_E = 256 + 8, CH = G::COUT / 4, P = 256 / G::COUT, PER = 256 / CH / P;
        double* sSum = reinterpret_cast<double*>(smem);
        static_assert(4 * LDS_E * sizeof(double) <= G::SMEM, "the partial sums fit the operand buffers");
#pragma unroll
        for (int e = 0; e < 4; ++e) sSum[e * LDS_E + tid] = bsum[e];
        __syncthreads();
        const int ch = tid / P, p = tid % P;
        double sum = 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) sum += sSum[(ch & 3) * LDS_E + (ch >> 2) + CH * (p * PER + k)];
#pragma unroll
        for (int d = P / 2; d >= 1; d >>= 1) sum += __shfl_down(sum, d, P);
        if (p == 0) reinterpret_cast<double*>(a.bias_partial)[static_cast<size_t>(wg) * G::COUT + ch] = sum;
    }
    float* out = a.partial + static_cast<size_t>(wg) * G::COUT * G::N;
#pragma unroll
    for (int j = 0; j < NTW; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int m = (wave & 1) * 32 + 8 * (v >> 2) + 4 * kg + (v & 3), n = (cb * G::NT + (wave >> 1) + 2 * j) * 32 + lr;
            out[static_cast<size_t>(m) * G::N + n] = acc[j][v];
        }
}

// fc1: dW[o][f] = sum_b dZ[b][o] * act3[b][f]; a workgroup owns a 64 x 128 tile and walks the minibatch in chunks of 64 rows
// (the next chunk is requested before the current one is multiplied).
struct WgFc1F32Args {
    const float* dz;      // [B][512]
    const float* x;       // [B][3136]
    int B;
    float* grad;          // [512][3136]
};
constexpr int kWgF1fBM = 64, kWgF1fBN = 128, kWgF1fKC = 64;
constexpr size_t kWgF1fSmem = static_cast<size_t>(kWgF1fKC) * (kWgF1fBM + kWgF1fBN) * 4;
constexpr int kWgF1fCols = (3136 + kWgF1fBN - 1) / kWgF1fBN, kWgF1fRows = 512 / kWgF1fBM;   // 25 x 8 workgroups

__device__ inline void wgrad_fc1_f32_block(const WgFc1F32Args& a, int bx, int bz, unsigned char* smem)
{
    constexpr int BM = kWgF1fBM, BN = kWgF1fBN, KC = kWgF1fKC, N = 3136;
    constexpr int CVA = BM / 4, CVB = BN / 4, NA = KC * CVA / 256, NB = KC * CVB / 256;   // 16-byte vectors per row; per thread and chunk: 4 + 8
    float* sA = reinterpret_cast<float*>(smem);
    float* sB = sA + KC * BM;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 31, kg = lane >> 5;
    const int m0 = bz * BM, n0 = bx * BN, B = a.B;
    const int ka = tid / CVA, ca = (tid % CVA) * 4, kb = tid / CVB, cbv = (tid % CVB) * 4;
    const bool okb = n0 + cbv < N;                                 // the last column block is half empty
    const float* pa = a.dz + m0 + ca;
    const float* pb = a.x + (okb ? n0 + cbv : 0);
    wg_f32x4 ra[NA], rb[NB];
    auto fetch = [&](int k0) {   // rows past the minibatch repeat its last row and count as zero (cleared on both sides when they are stored)
#pragma unroll
        for (int i = 0; i < NA; ++i) ra[i] = *reinterpret_cast<const wg_f32x4*>(pa + static_cast<size_t>(min(k0 + ka + i * (256 / CVA), B - 1)) * 512);
#pragma unroll
        for (int i = 0; i < NB; ++i) rb[i] = *reinterpret_cast<const wg_f32x4*>(pb + static_cast<size_t>(min(k0 + kb + i * (256 / CVB), B - 1)) * N);
    };
    auto stash = [&](int k0) {
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int k = ka + i * (256 / CVA);
            const wg_u32x4 v = __builtin_bit_cast(wg_u32x4, ra[i]) & (k0 + k < B ? ~0u : 0u);
            *reinterpret_cast<wg_u32x4*>(sA + k * BM + ca) = v;
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int k = kb + i * (256 / CVB);
            *reinterpret_cast<wg_u32x4*>(sB + k * BN + cbv) = __builtin_bit_cast(wg_u32x4, rb[i]) & (k0 + k < B ? ~0u : 0u);
        }
    };
    f32x16 acc[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][v] = 0.f;
    const float* ap = sA + kg * BM + lr;
    const float* bp = sB + kg * BN + wave * 32 + lr;
    auto contract = [&](int rows) {   // eight minibatch rows per trip: a short last chunk costs what it holds
        for (int k = 0; k < rows; k += 8) {
            float fa[4][2], fb[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                fa[u][0] = ap[(k + 2 * u) * BM];
                fa[u][1] = ap[(k + 2 * u) * BM + 32];
                fb[u] = bp[(k + 2 * u) * BN];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int i = 0; i < 2; ++i) mma_32x32x2(acc[i], fa[u][i], fb[u]);
        }
    };
    fetch(0);
    for (int k0 = 0; k0 < B; k0 += KC) {
        if (k0 != 0) __syncthreads();   // every wavefront has finished reading the previous chunk
        stash(k0);
        if (k0 + KC < B) fetch(k0 + KC);
        __syncthreads();
        contract(min(KC, B - k0));
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int o = m0 + i * 32 + 8 * (v >> 2) + 4 * kg + (v & 3), f = n0 + wave * 32 + lr;
            if (f < N) a.grad[static_cast<size_t>(o) * N + f] = acc[i][v];
        }
}

struct WgradF32Args {
    WgConvArgs c1, c2, c3;
    WgFc1F32Args f1;
    BiasGradArgs small;
    int first[6];   // first block of: conv2, conv1, conv3, fc1, small reductions, end (the longest workgroups first)
};

constexpr size_t kWgradF32Smem = []() {
    size_t m = kSmallGradsSmem;
    if (kWgF1fSmem > m) m = kWgF1fSmem;
    if (WgConv1F32::SMEM > m) m = WgConv1F32::SMEM;
    if (WgConv2F32::SMEM > m) m = WgConv2F32::SMEM;
    if (WgConv3F32::SMEM > m) m = WgConv3F32::SMEM;
    return (m + 15) / 16 * 16;
}();
static_assert(2 * kWgradF32Smem <= 160 * 1024, "two workgroups per compute unit: one loads while the other multiplies");

__global__ __launch_bounds__(256, 2) void wgrad_f32_kernel(WgradF32Args a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char wf_smem[];
    const int blk = blockIdx.x;
    int cb;
    if (blk < a.first[1]) {
        const int slice = xcd_slice<WgConv2F32::CS>(blk, a.first[1] / WgConv2F32::CS, cb);
        wgrad_conv_f32_block<WgConv2F32>(a.c2, slice, cb, wf_smem);
    }
    else if (blk < a.first[2]) wgrad_conv_block<WgConv1F32>(a.c1, blk - a.first[1], 0, wf_smem);
    else if (blk < a.first[3]) {
        const int slice = xcd_slice<WgConv3F32::CS>(blk - a.first[2], (a.first[3] - a.first[2]) / WgConv3F32::CS, cb);
        wgrad_conv_f32_block<WgConv3F32>(a.c3, slice, cb, wf_smem);
    }
    else if (blk < a.first[4]) {
        int col, row;
        xcd_fc1_tile(blk - a.first[3], col, row);
        wgrad_fc1_f32_block(a.f1, col, row, wf_smem);
    } else small_grads_block<float>(a.small, blk - a.first[4], wf_smem);
}

}  // namespace dqn
