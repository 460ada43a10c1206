// fp32 products on the bf16 matrix cores.
#pragma once
#include <hip/hip_runtime.h>

namespace monet {

// A float is the sum of three bf16 numbers (8 + 8 + 8 significant bits, each remainder is exact in fp32): x = h + m + l.  A
// product keeps the six terms h*h, h*m, m*h, m*m, h*l, l*h; the three left out are below 2^-25 of it.  Every term is exact
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
__device__ __forceinline__ Pieces split_pair(float a, float b) {
    Pieces p;
    p.h = pack_bf16(a, b);
    const float a1 = a - __uint_as_float(p.h << 16), b1 = b - __uint_as_float(p.h & 0xffff0000u);
    p.m = pack_bf16(a1, b1);
    p.l = pack_bf16(a1 - __uint_as_float(p.m << 16), b1 - __uint_as_float(p.m & 0xffff0000u));
    return p;
}
// The same for operands that hold infinities, NaNs or values that round to infinity in bf16 (taken only after a first pass
// has left an infinity or a NaN in the result).  All pieces are truncated, so they have the number's sign and the six terms of an
// overflowing product agree; an infinity or a NaN travels in the piece that meets only the other operand's h, and stands
// as +-1 where the other operand's infinity meets it.
__device__ __forceinline__ void split_special(float x, unsigned &h, unsigned &m, unsigned &l) {
    const unsigned u = __float_as_uint(x);
    const bool bad = (u & 0x7f800000u) == 0x7f800000u;
    const float hf = __uint_as_float(bad ? (u & 0x80000000u) | 0x3f800000u : u & 0xffff0000u);
    const float r = bad ? 0.0f : x - hf;
    const float mf = __uint_as_float(__float_as_uint(r) & 0xffff0000u);
    h = __float_as_uint(hf) >> 16;
    m = __float_as_uint(mf) >> 16;
    l = bad ? (u >> 16) | ((u & 0x007fffffu) ? 0x40u : 0u) : __float_as_uint(r - mf) >> 16;
}
__device__ __forceinline__ Pieces split_pair_special(float a, float b) {
    unsigned h0, m0, l0, h1, m1, l1;
    split_special(a, h0, m0, l0);
    split_special(b, h1, m1, l1);
    return {h0 | h1 << 16, m0 | m1 << 16, l0 | l1 << 16};
}

// eight reduction indices of a lane as the three operands of v_mfma_f32_32x32x16_bf16
struct PieceRow { bf16x8 h, m, l; };
template <bool SPECIAL>
__device__ __forceinline__ PieceRow split_row(const float (&v)[8]) {
    uintx4 h, m, l;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const Pieces p = SPECIAL ? split_pair_special(v[2 * j], v[2 * j + 1]) : split_pair(v[2 * j], v[2 * j + 1]);
        h[j] = p.h; m[j] = p.m; l[j] = p.l;
    }
    return {__builtin_bit_cast(bf16x8, h), __builtin_bit_cast(bf16x8, m), __builtin_bit_cast(bf16x8, l)};
}

}  // namespace monet
