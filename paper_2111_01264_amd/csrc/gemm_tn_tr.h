// Operand fragments of a weight gradient in bf16:   C[m][n] = sum_k A(m, k) * B(n, k)   where both
// operands are stored k-major -- dY is [pixel][channel], the im2col of the layer input is
// [pixel][filter element] -- i.e. the contraction index is the *slow* one.  The MFMA wants eight
// consecutive k per lane, so earlier GPUs had to transpose on the way into LDS with 2-byte writes.
// CDNA4 has a transposing LDS read (ds_read_b64_tr_b16): the tiles are staged exactly as they come
// from memory ([k][row], 16-byte vector writes) and every lane receives four consecutive k of its
// own row per read.
//
// ds_read_b64_tr_b16 semantics used here (checked on the device): within each group of 16 lanes,
// lane i receives, for e = 0..3, element (i % 4) of the 8-byte chunk addressed by lane 4*e + i/4 of
// the group.  With lane 16*G + s addressing  tile[k0 + 8*(G/2) + 4*t + s/4][col0 + 16*(G%2) + 4*(s%4)]
// lane l ends up with tile[k0 + 8*(l/32) + 4*t + e][col0 + l%32], e = 0..3: two reads (t = 0, 1) are
// one 32x32x16 operand fragment.
#pragma once
#include "gemm_mfma.h"

namespace dqn {

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

// One operand fragment: rows k .. k+3 (first read) and k+4 .. k+7 (second read) of this lane's column.
__device__ inline bf16x8 tr_fragment(const bf16_t* p, int pitch4 /* elements between row k and row k+4 */)
{
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + pitch4));
    const bf16x4 blo = __builtin_bit_cast(bf16x4, lo), bhi = __builtin_bit_cast(bf16x4, hi);
    bf16x8 r;
#pragma unroll
    for (int e = 0; e < 4; ++e) { r[e] = blo[e]; r[4 + e] = bhi[e]; }
    return r;
}

}  // namespace dqn
