// fp32 contractions on the bf16 matrix cores.  An fp32 value is the sum of three bf16 values,
//   x = x0 + x1 + x2 (+ at most 2^-27 |x|),  x0 = bf16(x), x1 = bf16(x - x0), x2 = bf16(x - x0 - x1),
// every difference exact, and a product a*b is taken as the six terms a0b0 + a0b1 + a1b0 + a0b2 + a2b0 +
// a1b1; what is left out is below 2^-25 |a*b|, of either sign.  Products of two bf16 values are exact in
// fp32 and the matrix cores add 16 or 32 of them per instruction in fp32, so that a sum of K products is
// rounded K/16 or K/32 times instead of K/2 or K/4 times: measured against 64 bits the six-term sums are
// off by 0.6-0.9 times what v_mfma_f32_32x32x2_f32 is, for K = 64 .. 12,544 on signed and on positive
// operands.  Six bf16 MFMAs take 3/8 of the time of the fp32 MFMAs they replace (16 x the rate), and unlike
// those they leave the vector ALU free: eight v_fma_f32 behind every 32x32x16 MFMA of two wavefronts cost
// 19.2 ns per MFMA instead of 16.6 ns, where the fp32 MFMA pays their full time (27.1 -> 44.2 ns).
// What the split cannot hold: an infinity, or a value that rounds to one (above 3.39e38), leaves NaN in x1
// and so in every sum it enters; the kernels look for NaN in their sums and redo such a sum with fp32 FMAs.
// Parts below 2^-126 are flushed to zero: operands under 2^-110 keep their leading 16 bits.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ps {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));

// Two values -> their bf16 parts, packed (first value in the low half), part by part.
__device__ __forceinline__ void split2(float x, float y, uint32_t& p0, uint32_t& p1, uint32_t& p2)
{
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float floatx2 __attribute__((ext_vector_type(2)));
    auto pack = [](float a, float b) { return __builtin_bit_cast(uint32_t, __builtin_convertvector(floatx2{a, b}, bf16x2)); };
    auto low = [](uint32_t p) { return __uint_as_float(p << 16); };
    auto high = [](uint32_t p) { return __uint_as_float(p & 0xffff0000u); };
    p0 = pack(x, y);
    x -= low(p0);
    y -= high(p0);
    p1 = pack(x, y);
    p2 = pack(x - low(p1), y - high(p1));
}

// Eight consecutive k of one matrix row (or column): the operand of one lane, part by part.
struct Split8 {
    uintx4 p[3];
    __device__ __forceinline__ bf16x8 part(int i) const { return __builtin_bit_cast(bf16x8, p[i]); }
};

__device__ __forceinline__ Split8 split8(const float (&x)[8])
{
    Split8 s;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        uint32_t a, b, c;
        split2(x[2 * i], x[2 * i + 1], a, b, c);
        s.p[0][i] = a;
        s.p[1][i] = b;
        s.p[2][i] = c;
    }
    return s;
}

// The six terms in the order in which they are added up, the small ones first: part of A, part of B.
constexpr int SPLIT_TERMS = 6, TERM_A[SPLIT_TERMS] = {1, 0, 2, 0, 1, 0}, TERM_B[SPLIT_TERMS] = {1, 2, 0, 1, 0, 0};

// acc[i] += A . B[i] over one k-step for N products that share A: term by term, so that consecutive MFMAs
// belong to different sums.
template <int N>
__device__ __forceinline__ void mfma_split(const Split8& a, const Split8* const (&b)[N], floatx4* const (&acc)[N])
{
#pragma unroll
    for (int t = 0; t < SPLIT_TERMS; ++t)
#pragma unroll
        for (int i = 0; i < N; ++i)
            *acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.part(TERM_A[t]), b[i]->part(TERM_B[t]), *acc[i], 0, 0, 0);
}

// The same operand with every lane taking the value S lanes further on in its row of 16 (zero past the end).
template <int S>
__device__ __forceinline__ Split8 lanes_up(const Split8& a)
{
    Split8 r;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            r.p[i][j] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)a.p[i][j], 0x100 + S, 0xF, 0xF, true);  // row_shl:S
    return r;
}

// LDS written by some lanes of a wavefront and read by others of the same wavefront.
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace ps
