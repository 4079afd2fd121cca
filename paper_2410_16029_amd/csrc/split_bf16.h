// A float as a sum of bf16 values, shared by the fp32 products and the refresh's small orthonormalisation.
#pragma once

#include <hip/hip_runtime.h>

namespace ng {

typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

// the NP planes of two values, a in the low halves
template <int NP>
__device__ __forceinline__ void split2(float a, float b, unsigned (&p)[NP]) {
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        const f32x2_t f = {a, b};
        const bf16x2_t hv = __builtin_convertvector(f, bf16x2_t);      // v_cvt_pk_bf16_f32: nearest even
        p[i] = *reinterpret_cast<const unsigned int*>(&hv);
        a -= __uint_as_float(p[i] << 16);
        b -= __uint_as_float(p[i] & 0xffff0000u);
    }
}

}  // namespace ng
