// Shared by the float32 matrix-core kernels (slide_mfma32.hip, slide_mfma32_bwd.hip).
#pragma once
#include "slide_internal.h"
#include "slide_device.h"
#include <utility>

namespace slide {
namespace m32 {

typedef float f4 __attribute__((ext_vector_type(4)));

template <int KS> struct Dim {
    static constexpr int S = KS * KS, R = KS / 2;
    static constexpr int SM = S - 1, SB = SM / 4;           // shifts on the matrix cores, blocks of four of them
    // the weights of four channels lie in LDS as they do in memory, [channel][shift][tap]; lane l of
    // operand register j holds weight (tap, channel, shift < SM) number 64 j + l of UT taps
    static constexpr int UT = KS == 3 ? 3 : 1, UNIT = UT * 4 * SM, WV = (UNIT + 63) / 64;
    static constexpr int LASTV = (4 * S + 63) / 64;         // registers of the last shift's weights, [tap][channel]
    static constexpr int QUAD_W = 4 * S * S;
};

template <int ABID>
__device__ __forceinline__ f4 outer(float a, float b, f4 c)
{
    return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 4, ABID, 0);
}
template <typename F, int... i>
__device__ __forceinline__ void unroll_over(F&& f, std::integer_sequence<int, i...>)
{
    (f(std::integral_constant<int, i>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void unroll(F&& f) { unroll_over(f, std::make_integer_sequence<int, N>{}); }
// acc[SB] += A[block FIRST + sb] (outer) b, A in registers of 16 blocks
template <int FIRST, int SB, int NV>
__device__ __forceinline__ void outer_blocks(const float (&wv)[NV], float b, f4 (&acc)[SB])
{
    unroll<SB>([&](auto i) {
        constexpr int blk = FIRST + decltype(i)::value;
        acc[decltype(i)::value] = outer<blk % 16>(wv[blk / 16], b, acc[decltype(i)::value]);
    });
}
__device__ __forceinline__ float lane_of(float x, int lane)
{
    return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(x), lane));
}

// four neighbouring elements at any element's address (the hardware takes unaligned vector loads and stores)
template <typename T> struct Four;
template <> struct Four<float> {
    typedef f4 Any __attribute__((aligned(4)));
    static __device__ __forceinline__ f4 load(const float* p) { return *(const Any*)p; }
    static __device__ __forceinline__ void store(float* p, f4 v) { *(Any*)p = v; }
};
template <> struct Four<bf16_bits> {
    typedef uint32_t Raw __attribute__((ext_vector_type(2)));
    typedef Raw Any __attribute__((aligned(2)));
    static __device__ __forceinline__ f4 load(const bf16_bits* p)
    {
        const Raw r = *(const Any*)p;
        return f4{__uint_as_float(r[0] << 16), __uint_as_float(r[0] & 0xffff0000u),
                  __uint_as_float(r[1] << 16), __uint_as_float(r[1] & 0xffff0000u)};
    }
    static __device__ __forceinline__ void store(bf16_bits* p, f4 v)
    {
        *(Any*)p = Raw{f32_to_bf16(v[0]) | (uint32_t)f32_to_bf16(v[1]) << 16,
                       f32_to_bf16(v[2]) | (uint32_t)f32_to_bf16(v[3]) << 16};
    }
};

// what is derived from x, y and v is formed after this point (keeps the compiler from reading every
// tap and weight of a channel ahead of the first product)
template <int N>
__device__ __forceinline__ void pin(int& x, int& y, float (&v)[N])
{
    asm volatile("" : "+v"(x), "+v"(y));
#pragma unroll
    for (int i = 0; i < N; ++i) asm volatile("" : "+v"(v[i]));
}

// column strip of a plane: first column and width
__device__ __forceinline__ void strip_of(const Cut& c, int strip, int& j0, int& tw)
{
    j0 = strip * c.TW + min(strip, c.wider);
    tw = c.TW + (strip < c.wider);
}

}  // namespace m32
}  // namespace slide
