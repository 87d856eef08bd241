// FP32 numbers as three BF16 parts of 8 bits whose sum they are (rounding to
// nearest leaves exact remainders of 2^-9 and 2^-18), for the products that
// contract FP32 operands on the BF16 matrix cores (mvm_kx.hip, mvm_fx.hip). BF16
// has FP32's exponents and its subnormal numbers go through the matrix cores as
// they are (checked on gfx950 with an in-bounds probe), so the parts hold every
// bit of a number of at least 2^-109; below, they end at 2^-133.
#pragma once

#include <hip/hip_runtime.h>

namespace ciq {
namespace bf16 {

typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int uintx4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ unsigned int pk(float a, float b) {
    return __builtin_bit_cast(unsigned int, __builtin_convertvector((floatx2{a, b}), bf16x2));
}
__device__ __forceinline__ float lo(unsigned int p) { return __builtin_bit_cast(float, p << 16); }
__device__ __forceinline__ float hi(unsigned int p) { return __builtin_bit_cast(float, p & 0xffff0000u); }

// Eight values that do not round to infinity.
__device__ __forceinline__ void split3(const float* e, bf16x8& h, bf16x8& m, bf16x8& l) {
    uintx4 hb, mb, lb;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        float x0 = e[2 * p], x1 = e[2 * p + 1];
        const unsigned int hp = pk(x0, x1);
        x0 -= lo(hp);
        x1 -= hi(hp);
        const unsigned int mp = pk(x0, x1);
        x0 -= lo(mp);
        x1 -= hi(mp);
        hb[p] = hp;
        mb[p] = mp;
        lb[p] = pk(x0, x1);
    }
    h = __builtin_bit_cast(bf16x8, hb);
    m = __builtin_bit_cast(bf16x8, mb);
    l = __builtin_bit_cast(bf16x8, lb);
}

// Infinities and NaN among them: the last part alone, so that an infinity meets
// only the first part of an entry, as the FP32 product would have multiplied it.
__device__ __forceinline__ void only_last(const float* e, bf16x8& h, bf16x8& m, bf16x8& l) {
#pragma unroll
    for (int q = 0; q < 8; ++q)
        if (!(fabsf(e[q]) < INFINITY)) {
            h[q] = m[q] = (__bf16)0.0f;
            l[q] = (__bf16)e[q];
        }
}

// One FP64 value, kept to 2^-27 of itself; infinities and NaN as above.
__device__ __forceinline__ void split3(double x, __bf16& h, __bf16& m, __bf16& l) {
    const double f = fabs(x) < INFINITY ? x : 0.0;
    h = (__bf16)(float)f;
    double r = f - (double)(float)h;
    m = (__bf16)(float)r;
    r -= (double)(float)m;
    l = (__bf16)(float)(f == x ? r : x);
}

}  // namespace bf16
}  // namespace ciq
