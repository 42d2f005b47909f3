// fp32 contractions on the bf16 matrix cores (gfx950), without losing fp32's digits.
//
// An fp32 number is the sum of three bf16 numbers, x = h + m + l: h is x rounded to bf16, m what is left of it rounded to bf16, l the rest
// (8 + 8 + 8 significant bits and two signs: exact).  A product of two such sums is
//   hh' + (hm' + mh') + (mm' + hl' + lh')
// up to terms below 2^-24 of it, six matrix products with fp32 accumulation (Henry, Tang, Heinecke, "Leveraging the bfloat16 Artificial
// Intelligence Datatype For Higher-Precision Computations", ARITH 2019).  Measured against float64 over 64 to 1024 terms
// (normal, uniform and widely spread operands): 0.65 to 0.85 of the error of v_mfma_f32_16x16x4_f32, which rounds its sum more often.
// Why: the fp32 matrix instructions run at 32 multiply-adds per clock and SIMD and hold the vector unit for as long (measured: no vector
// instruction of another wave gets in); the bf16 ones run at 512, six of them at 85, and leave the vector unit free (a wave of
// reciprocals next to a wave of v_mfma_f32_32x32x16_bf16: 10.6 clocks per reciprocal against 10.1 alone).
// Small numbers: fp32 operands are multiplied by 2^24 before they are split, and the caller multiplies the sums by split_back.  A part is a
// whole multiple of 2^-149, as the number is; scaled it is zero or at least 2^-125, which bf16 holds.  (As they are, bf16 keeps multiples of
// 2^-133 of them, and operands of 1e-34, 1e-35 and 1e-36 gave errors of 2.9e-7, 2.7e-6 and 2.7e-5; scaled 1.1e-7 throughout, fp32 products
// 1.4e-7.  It costs two of thirteen instructions per pair, and 0 to 0.6 % of forward and backward over 17 shapes.)
// What it cannot do: infinities, operands past 2^104 (2e31) and sums past 2^80 (1.2e24, with a bf16 operand 2^104) are not finite; a caller that
// finds such a result redoes the work in fp32.
#pragma once
#include "common.hpp"

namespace echo {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// Loads stay where they are requested: everything else may cross this line.  (The compiler moves the loads for the next step to the end
// of this one, where fewer registers are live, and the next step then waits for a whole trip to memory.)
__device__ __forceinline__ void loads_stay() { __builtin_amdgcn_sched_barrier(0); }

// Eight consecutive operands of one lane, split: plane 0 holds the h, 1 the m, 2 the l.
struct Split8 { u32x4 p[3]; };

__device__ __forceinline__ unsigned bf16_pair(float a, float b) {           // round to nearest even, a in the low half
    return __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2){a, b}, bf16x2));
}
constexpr float kSplitScale = 0x1p24f;
// what takes the scale off a sum of products of a split operand with one of type TB
template <typename TB> __device__ constexpr float split_back = sizeof(TB) == 4 ? 0x1p-48f : 0x1p-24f;

// Two numbers into their three pairs: thirteen instructions.  (v_dot2_f32_bf16 with (-1, 0) would take a half off in one instruction instead
// of two, but it holds up the matrix instructions: 61 clocks for one of them and four v_dot2, 33 with four shifts or subtractions.)
__device__ __forceinline__ void split2(float a, float b, unsigned &h, unsigned &m, unsigned &l) {
    a *= kSplitScale;
    b *= kSplitScale;
    h = bf16_pair(a, b);
    a -= __uint_as_float(h << 16);
    b -= __uint_as_float(h & 0xffff0000u);
    m = bf16_pair(a, b);
    l = bf16_pair(a - __uint_as_float(m << 16), b - __uint_as_float(m & 0xffff0000u));
}
__device__ __forceinline__ Split8 split8(const float (&x)[8]) {
    Split8 s;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        unsigned h, m, l;
        split2(x[2 * i], x[2 * i + 1], h, m, l);
        s.p[0][i] = h;
        s.p[1][i] = m;
        s.p[2][i] = l;
    }
    return s;
}

// v_mfma_f32_32x32x16_bf16, lane l: A row l % 32, B column l % 32, both k = 8 (l / 32) .. + 7; accumulator r holds row
// 8 (r / 4) + 4 (l / 32) + r % 4 of column l % 32.
__device__ __forceinline__ f32x16 mfma32(u32x4 a, u32x4 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
__device__ __forceinline__ int mfma32_row(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }
// c += A B, the small terms first
__device__ __forceinline__ f32x16 mfma32(const Split8 &a, const Split8 &b, f32x16 c) {
    c = mfma32(a.p[1], b.p[1], c);
    c = mfma32(a.p[2], b.p[0], c);
    c = mfma32(a.p[0], b.p[2], c);
    c = mfma32(a.p[1], b.p[0], c);
    c = mfma32(a.p[0], b.p[1], c);
    return mfma32(a.p[0], b.p[0], c);
}

// the same with a B that is bf16 to begin with
__device__ __forceinline__ f32x16 mfma32(const Split8 &a, u32x4 b, f32x16 c) {
    c = mfma32(a.p[2], b, c);
    c = mfma32(a.p[1], b, c);
    return mfma32(a.p[0], b, c);
}

// c += s: the sum of a short run of products, formed from zero, on its own.  A chain of products into one accumulator rounds the whole sum six
// times per 16 terms, this once per run.
__device__ __forceinline__ void add16(f32x16 &c, const f32x16 &s) {
#pragma unroll
    for (int r = 0; r < 16; ++r) c[r] += s[r];
}
__device__ __forceinline__ f32x16 zero16() {
    f32x16 z;
#pragma unroll
    for (int r = 0; r < 16; ++r) z[r] = 0.f;
    return z;
}

}  // namespace echo
