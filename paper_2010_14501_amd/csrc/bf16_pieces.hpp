// fp32 products on the bf16 matrix cores.
#pragma once
#include <hip/hip_runtime.h>

namespace monet {

// A float of 2^-110 and more is the sum of three bf16 numbers (8 + 8 + 8 significant bits, rounded to nearest; each remainder is
// exact in fp32): x = h + m + l.  A product keeps the six terms h*h, h*m, m*h, m*m, h*l, l*h; m*l and l*m, up to 2^-25 of it each, and l*l
// are left out.  Every term is exact
// in the matrix unit and the sums are fp32, so the result is as close to 64 bits as the fp32 matrix instruction's (fewer
// roundings: six per 16 products instead of one per product; measured side by side, normwise error of one layer).
// Six bf16 instructions take 192 cycles for what the fp32 instruction does in 512.
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
struct Pieces { unsigned h, m, l; };     // two neighbouring reduction indices: low half first

__device__ __forceinline__ unsigned pack_bf16(float a, float b) {       // to nearest
    typedef float floatx2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(unsigned, __builtin_convertvector(floatx2{a, b}, bf16x2));
}
// `lost` gathers the bits that the third piece leaves over.  For floats of 2^-110 and more there are none: the second rest has at
// most eight significant bits, so the lower half of its word is zero and bf16 holds it whole.  Below that it reaches under bf16's
// smallest number (2^-133), and pieces would give less than the fp32 product (a layer whose operand is about 2^-114: 5e-7 normwise;
// 2^-118: 9e-6; 2^-125: 1e-3).  One vector instruction per pair.
__device__ __forceinline__ Pieces split_pair(float a, float b, unsigned &lost) {
    Pieces p;
    p.h = pack_bf16(a, b);
    const float a1 = a - __uint_as_float(p.h << 16), b1 = b - __uint_as_float(p.h & 0xffff0000u);
    p.m = pack_bf16(a1, b1);
    const float a2 = a1 - __uint_as_float(p.m << 16), b2 = b1 - __uint_as_float(p.m & 0xffff0000u);
    p.l = pack_bf16(a2, b2);
    lost |= __float_as_uint(a2) | __float_as_uint(b2);
    asm volatile("" : "+v"(lost));      // here: gathered later, the rests of many pairs would stay in registers
    return p;
}
__device__ __forceinline__ bool pieces_lost(unsigned lost) { return lost & 0xffffu; }

// eight reduction indices of a lane as the three operands of v_mfma_f32_32x32x16_bf16
struct PieceRow { bf16x8 h, m, l; };
__device__ __forceinline__ PieceRow split_row(const float (&v)[8], unsigned &lost) {
    uintx4 h, m, l;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const Pieces p = split_pair(v[2 * j], v[2 * j + 1], lost);
        h[j] = p.h; m[j] = p.m; l[j] = p.l;
    }
    return {__builtin_bit_cast(bf16x8, h), __builtin_bit_cast(bf16x8, m), __builtin_bit_cast(bf16x8, l)};
}

}  // namespace monet
