// Three-way bf16 split of fp32 operands, shared by the kernels that multiply fp32 tensors on the bf16
// matrix instruction.
//
// An fp32 value is exactly h + m + l with h, m, l in bf16 (each the nearest bf16 to what is left of the
// value: 8 + 8 + 8 significant bits), so x*w is the sum of nine exact bf16 products.  The six largest are
// computed, every one exactly, with fp32 accumulation; the three dropped ones (m*l, l*m, l*l) come to
// about 2^-24 |x*w| at most.  v_mfma_f32_16x16x32_bf16 contracts 32 slots in 16 clocks where v_mfma_f32_16x16x4_f32
// contracts 4 in 32: six of the former do the work of eight of the latter in 96 instead of 256 clocks.
//
// bf16 ends at 2^-133 (2^-126 without denormals), where the last bits of a value below 2^-103 would be lost.
// So both operands are split at 2^24 times their value: the parts of every fp32 number, the smallest denormal
// included, are then normal bf16 numbers, and the sum is scaled back by 2^-48 with one rounding.  What overflows
// instead - factors from 2^103, sums from 2^80 on - shows as an infinity or a NaN and is computed anew
// (SplitOverflow).
#pragma once

#include "conv_common.h"

namespace gspc {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr float kSplitScale = 0x1p24f, kSplitUnscale = 0x1p-48f;

// Two (scaled) fp32 values -> the packed bf16 pairs (a in the low half) of their three parts.
__device__ __forceinline__ void split3(float a, float b, unsigned (&o)[3]) {
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        o[q] = __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{a, b}, bf16x2));
        a -= __uint_as_float(o[q] << 16);
        b -= __uint_as_float(o[q] & 0xffff0000u);
    }
}

// The products of a split operand pair, smallest first; the last one (h * h) goes to an accumulator of its
// own, so that the sum is rounded once per instruction and not six times at its full magnitude.  Error against
// fp64: over dense sums of K = 16 .. 4608 terms 0.3-0.9 x that of the fp32 instruction (with one accumulator up
// to 1.2 x); a sum of one term is off by up to 1.7 * 2^-24 of it, where the fp32 instruction rounds it correctly
// (1.0 * 2^-24).
constexpr int kSplitA[6] = {2, 0, 1, 1, 0, 0};
constexpr int kSplitB[6] = {0, 2, 1, 0, 1, 0};

// Whether a scaled sum has overflowed or met an infinity or a NaN.
struct SplitOverflow {
    unsigned most = 0u;
    __device__ __forceinline__ void see(float v) { most = max(most, __float_as_uint(v) & 0x7fffffffu); }
    __device__ __forceinline__ bool any() const { return most >= 0x7f800000u; }
};

// All of the wave's vector-memory operations are done (the compiler does not wait for loads that go into LDS).
__device__ __forceinline__ void wait_vmem0() { __builtin_amdgcn_s_waitcnt(0x0F70); }

}  // namespace gspc
