// Four consecutive values of an operand type: store from / load into fp32 registers.
#pragma once
#include "gemm_mfma.h"

namespace dqn {

typedef float f32x4v __attribute__((ext_vector_type(4)));

template <typename T> __device__ inline void store4(T* dst, float a, float b, float c, float d);
template <> __device__ inline void store4<float>(float* dst, float a, float b, float c, float d)
{
    *reinterpret_cast<float4*>(dst) = make_float4(a, b, c, d);
}
template <> __device__ inline void store4<bf16_t>(bf16_t* dst, float a, float b, float c, float d)
{
    typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
    bf16x4 v;
    v[0] = static_cast<bf16_t>(a); v[1] = static_cast<bf16_t>(b);
    v[2] = static_cast<bf16_t>(c); v[3] = static_cast<bf16_t>(d);
    *reinterpret_cast<bf16x4*>(dst) = v;
}
template <typename T> __device__ inline void load4(const T* src, float* o);
template <> __device__ inline void load4<float>(const float* src, float* o)
{
    const float4 v = *reinterpret_cast<const float4*>(src);
    o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w;
}
template <> __device__ inline void load4<bf16_t>(const bf16_t* src, float* o)
{
    typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
    const bf16x4 v = *reinterpret_cast<const bf16x4*>(src);
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = static_cast<float>(v[i]);
}

}  // namespace dqn
