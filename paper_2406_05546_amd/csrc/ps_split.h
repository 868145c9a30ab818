// fp32 contractions on the bf16 matrix cores.  An fp32 value is the sum of three bf16 values,
//   x = x0 + x1 + x2 (+ at most 2^-27 |x|),  x0 = bf16(x), x1 = bf16(x - x0), x2 = bf16(x - x0 - x1),
// every difference exact, and a product a*b is taken as the six terms a0b0 + a0b1 + a1b0 + a0b2 + a2b0 +
// a1b1; what is left out (a1b2, a2b1, a2b2 and the tails) is at most about 2^-24 |a*b|, of either sign.
// Products of two bf16 values are exact in
// fp32, and the matrix cores add 16 or 32 of them per instruction to an fp32 accumulator, but cut off (towards
// minus infinity) what a small addend has below the large one's last bit.  So a0b0 and the five small terms
// are summed in accumulators of their own and meet at the end: measured against 64 bits such sums are off by
// 0.25-0.4 times what v_mfma_f32_32x32x2_f32 is (K = 64 .. 12,544; signed, positive and mostly zero operands;
// mean error below 2e-9 of the mean result).  With all six terms in one accumulator it is 0.6-0.9 times, 1.4 to
// 1.8 times where most operands are zero, and the mean error is -1e-8 (K = 144) to -3e-8 (K = 512), which a later
// sum over many such results does not average out.
// Six bf16 MFMAs take 3/8 of the time of the fp32 MFMAs they replace (16 x the rate), and unlike those they
// leave the vector ALU free: per 32x32x16 MFMA of two wavefronts (14.2 ns alone) four v_fma_f32 make 16.1 ns and
// eight 19.0 ns, per 16x16x32 MFMA (6.9 ns) one, two and three make 7.1, 7.8 and 9.2 ns; next to the fp32
// 32x32x2 MFMA (27.1 ns) eight take their full time (44.2 ns).
// What the split cannot hold: an infinity, or a value that rounds to one (above 3.39e38), leaves NaN in x1
// and so in every sum it enters; a0b0 can be infinite where a*b, within 2^-8 of the largest float, is not; and parts
// are multiples of 2^-133, so that operands below 2^-110 lose bits.  The kernels look for sums that are not finite, and
// for tiles whose sums are all below 2^-80 and not all zero, and form them again with fp32 matrix instructions, a
// wavefront's tile at a time, until those are NaN.  (They multiply zeros by infinities, all but conv2's weight gradient, whose
// gradients of zero take nothing out of an infinite activation: its sparse products leave most zeros out.)  What small operands take from the sums of another tile is below
// 2^-24 of its largest with up to 2^11 products and the other operands below 2^20.  Operands below 2^-134, which hold
// at most 15 bits, count as zero in a tile that has no others (no weight that is a normal number is changed by such
// gradients).  Images that are classified with margins of 60 and more have such gradients: conv2's gradient kernels
// scale them (WorkerBuffers::grad_scale), fc1's see them among others, unless a minibatch has no others.
// 256 workers of 256 images, none, 20 %, 90 % and all with a margin of 70: 4.3, 4.3, 4.5 and 7.6 ms (fp32 kernels 6.2).
// A step on weights that are all NaN takes 1.1-1.2 times as long as an ordinary one, one on a single infinite weight
// 2.6-4 times (64 workers of 128 images 0.72 -> 0.78 and 2.7 ms; with a loop of fp32 FMAs for every lost sum 55 and
// 77 ms).  Looking takes 0.3 % of conv2's gradients and nothing measurable elsewhere.
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

// The terms: five small ones, then a0b0.
constexpr int SPLIT_SMALL = 5, TERM_A[SPLIT_SMALL + 1] = {1, 0, 2, 0, 1, 0}, TERM_B[SPLIT_SMALL + 1] = {1, 2, 0, 1, 0, 0};

// A sum in its two accumulators.
template <class V>
struct SplitSum {
    V big, small;
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (unsigned i = 0; i < sizeof(V) / 4; ++i) big[i] = small[i] = 0.f;
    }
    __device__ __forceinline__ V value() const { return big + small; }
    // one term of A . B over one k-step
    __device__ __forceinline__ void add(int t, const Split8& a, const Split8& b)
    {
        V& acc = t < SPLIT_SMALL ? small : big;
        if constexpr (sizeof(V) == sizeof(floatx4))
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.part(TERM_A[t]), b.part(TERM_B[t]), acc, 0, 0, 0);
        else
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.part(TERM_A[t]), b.part(TERM_B[t]), acc, 0, 0, 0);
    }
    __device__ __forceinline__ void add(const Split8& a, const Split8& b)
    {
#pragma unroll
        for (int t = 0; t <= SPLIT_SMALL; ++t) add(t, a, b);
    }
};

// Largest magnitude of N values; NaN if one of them is.
template <int N, class V>
__device__ __forceinline__ float largest(const V& v, int first = 0)
{
    float m = fabsf(v[first]);
#pragma unroll
    for (int i = 1; i < N; ++i) m = __builtin_elementwise_maximum(m, fabsf(v[first + i]));
    return m;
}

// Which sums of a wavefront have to be formed again.  They are looked at in groups of G of every lane: those that are not
// finite; and all of a group if its largest, over all lanes, is tiny and not zero.
constexpr float SPLIT_TINY = 0x1p-80f;

template <int N, int G, class V>
__device__ __forceinline__ bool any_lost(const V& sums)
{
    bool lost = false;
#pragma unroll
    for (int i = 0; i < N; i += G) {
        const float m = largest<G>(sums, i);
        const bool finite = !__any(!(m < INFINITY));
        if (__builtin_expect(!(finite && __any(m >= SPLIT_TINY)), 0)) lost |= !finite || __any(m > 0.f);
    }
    return __builtin_expect(lost, 0);
}

// The same, a bit for each of this lane's.
template <int N, int G, class V>
__device__ __forceinline__ uint32_t lost_sums(const V& sums)
{
    uint32_t which = 0;
#pragma unroll
    for (int i = 0; i < N; i += G) {
        const float m = largest<G>(sums, i);
        const bool finite = !__any(!(m < INFINITY)), tiny = finite && !__any(m >= SPLIT_TINY) && __any(m > 0.f);
#pragma unroll
        for (int j = i; j < i + G; ++j)
            if (tiny || (!finite && !(fabsf(sums[j]) < INFINITY))) which |= 1u << j;
    }
    return which;
}

// The same value, of which the compiler knows nothing: what is worked out from it in the rare block that forms sums
// again stays there, instead of being kept in registers all through the loop around it.
__device__ __forceinline__ int rarely(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// Whether forming them again can still give any of those that were lost: NaN, once in a sum, stays.
template <int N, class V>
__device__ __forceinline__ bool worth_going_on(uint32_t which, const V& again)
{
    bool going = false;
#pragma unroll
    for (int i = 0; i < N; ++i) going |= (which >> i & 1) && again[i] == again[i];
    return __any(going);
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

// A wave-uniform value the compiler cannot prove to be one, as a scalar.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Loads through a buffer descriptor (its base must be uniform): offsets at or beyond `bytes`, negative ones
// and BUFFER_NOWHERE among them, read as zero, which is how the kernels get the zero border of a feature map.
typedef __amdgpu_buffer_rsrc_t Buffer;
constexpr uint32_t BUFFER_NOWHERE = 0x40000000u;  // stays out of range with any offset inside a map added

__device__ __forceinline__ Buffer buffer_of(const float* base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ float buffer_float(Buffer b, uint32_t offset)
{
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(b, (int)offset, 0, 0));
}
__device__ __forceinline__ floatx4 buffer_float4(Buffer b, uint32_t offset)
{
    return __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(b, (int)offset, 0, 0));
}

// 16 bytes for every lane straight to LDS, one behind the other from `lds` (uniform) on; there once vmcnt says so.
__device__ __forceinline__ void buffer_to_lds16(Buffer b, void* lds, uint32_t offset)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(b, (__attribute__((address_space(3))) void*)lds, 16, (int)offset, 0, 0, 0);
}

// LDS written by some lanes of a wavefront and read by others of the same wavefront.
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace ps
