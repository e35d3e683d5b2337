// Matrix-core vocabulary shared by the kernels of the Q-network: operand vectors, the 32x32 matrix instruction in both
// precisions, launches with timing events.
//
// 32x32 instruction: lane l feeds row (l % 32) with k-slice 8 * (l / 32) .. + 7, and receives column (l % 32) of the 32x32
// result with rows 8 * (v / 4) + 4 * (l / 32) + (v % 4), v = 0 .. 15.  One source serves both precisions: T = __bf16 issues
// v_mfma_f32_32x32x16_bf16 (fp32 accumulate), T = float eight v_mfma_f32_32x32x2_f32 over the same 16-wide k-slice.
//
// Device-side layouts (Section 2.1; the Nature-DQN architecture of Section 5; every contraction index is contiguous where it
// is streamed):
//   input states  uint8 [n][4][84][84]          (as handed over by the caller / the replay gather)
//   conv1 out     T     [n][20][20][32]          channels-last
//   conv2 out     T     [n][9][9][64]
//   conv3 out     T     [n][7][7][64]            = fc1 input, feature index (h*7 + w)*64 + c
//   conv1 weights [32][c][p][q]  (k = c*64 + p*8 + q, eight q's = eight adjacent input bytes)
//   conv2 weights [64][p][q][c]  conv3 weights [64][p][q][c]  fc1 weights [512][(h*7+w)*64 + c]
// dqn_set_params and dqn_get_params convert from and to the public blob layout, on the device (permute_blob_kernel).
#pragma once
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dqn {

typedef __bf16 bf16_t;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

template <typename T> struct Vec8;
template <> struct Vec8<float> { typedef f32x8 type; };
template <> struct Vec8<bf16_t> { typedef bf16x8 type; };

template <typename T> __device__ inline typename Vec8<T>::type vec8_zero()
{
    typename Vec8<T>::type z;
#pragma unroll
    for (int i = 0; i < 8; ++i) z[i] = static_cast<T>(0.f);
    return z;
}

// v if keep, else all-zero bits -- as a bitwise AND, not a select: the compiler turns "select(cond, loaded
// value, 0)" back into a branch around the load, and a load that may be skipped spoils its count of loads in flight.
template <typename T> __device__ inline typename Vec8<T>::type vec8_keep(const typename Vec8<T>::type& v, bool keep)
{
    typedef uint32_t words_t __attribute__((ext_vector_type(sizeof(typename Vec8<T>::type) / 4)));
    words_t w = __builtin_bit_cast(words_t, v);
    const uint32_t m = keep ? 0xFFFFFFFFu : 0u;
#pragma unroll
    for (int i = 0; i < static_cast<int>(sizeof(w) / 4); ++i) w[i] &= m;
    return __builtin_bit_cast(typename Vec8<T>::type, w);
}

template <typename T> __device__ inline T from_float(float x) { return static_cast<T>(x); }
template <typename T> __device__ inline float to_float(T x) { return static_cast<float>(x); }

__device__ inline void mma_32x32x16(f32x16& acc, const bf16x8& a, const bf16x8& b)
{
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
}
__device__ inline void mma_32x32x16(f32x16& acc, const f32x8& a, const f32x8& b)
{
#pragma unroll
    for (int t = 0; t < 8; ++t) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[t], b[t], acc, 0, 0, 0);
}

// Launch with an optional pair of timing events bound to the kernel's OWN dispatch: the time between them is the
// kernel's begin-to-end time on the GPU, which is what a kernel trace reports.  (A pair of event records around a launch
// also spans the records themselves and the dispatch gap: about 5 us on this machine, more than many of these kernels.)
template <typename F, typename... Args>
inline void launch_timed(F kernel, dim3 grid, dim3 block, size_t smem, hipStream_t st, hipEvent_t begin, hipEvent_t end,
                         Args... args)
{
    if (begin || end) hipExtLaunchKernelGGL(kernel, grid, block, static_cast<uint32_t>(smem), st, begin, end, 0, args...);
    else hipLaunchKernelGGL(kernel, grid, block, smem, st, args...);
}

constexpr int kMaxGroups = 4;   // independent problems per launch (online/target nets, parity classes)

}  // namespace dqn
