// Shared by the kernels that do float32 work on the 16-bit matrix cores by splitting (slide_split.hip, slide_split_dw.hip):
// bf16 activations, 5x5 window.
//
// A float32 weight is the sum of three bf16 values (8 significant bits each) exactly; a bf16 activation is one.  Their
// products are exact in float32, and a matrix instruction adds sixteen of them and its accumulator with little more than one
// rounding (measured, products of bf16 numbers, 16 terms and an accumulator of their size: 3.2e-8 from 64 bits, a chain of
// float32 fused multiply-adds 3.8e-8; unbiased).  So a float32 contraction over K taps is a bf16 one over 3 K slots, at sixteen
// times the float32 matrix rate per slot.  bf16 has the range of float32; numbers below 2^-110 keep fewer bits, their last terms
// being too small for it.
#pragma once
#include "slide_internal.h"
#include "slide_device.h"

namespace slide {
namespace split {

typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef float f16v __attribute__((ext_vector_type(16)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));
typedef uint32_t u2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32_any __attribute__((aligned(2)));

constexpr int KS = 5, S = 25, R = 2;

// the three terms of w, largest first; an infinite or NaN w is its own first term
__device__ __forceinline__ void split3(float w, float (&t)[3])
{
    t[0] = bf16_to_f32(f32_to_bf16(w));
    const bool fin = __builtin_fabsf(t[0]) < INFINITY;
    const float r1 = w - t[0];
    t[1] = fin ? bf16_to_f32(f32_to_bf16(r1)) : 0.0f;
    t[2] = fin ? r1 - t[1] : 0.0f;
}

// ---- operand image of the per-pixel kernels: per channel five left operands of 32 shifts (rows 25..31 zeros) by 16 slots,
// 16 bytes per lane: lane = shift + 32 * half of the slots.  The slots of one lane are four dwords of two taps each:
//   half h: d0 = row 2h, columns 0 1; d1 = row 2h, columns 2 3; d2, d3 = the same of row 2h + 1; d4 = row 4, columns 2h, 2h + 1;
//   d5 = column 4 of rows 2h and 2h + 1; x = row 4, column 4 and nothing.
// Instruction 0: d0..d3 with the third term of the weights, 1: with the second, 2: d4 d5 third, d4 d5 second, 3: d0..d3 first,
// 4: d4 d5 first, x x with the first and second terms (half 0), the third and nothing (half 1): small products first.
constexpr int PX_MM = 5;                                    // matrix instructions per channel
constexpr int PX_CH = PX_MM * 64;                           // 16-byte pieces per channel
// tap of dword d (0..6: d0..d5, x) element e of half h, -1: none
__host__ __device__ constexpr int px_tap(int h, int d, int e)
{
    return d < 4 ? (2 * h + d / 2) * KS + 2 * (d % 2) + e : d == 4 ? 4 * KS + 2 * h + e : d == 5 ? (2 * h + e) * KS + 4 : e == 0 ? S - 1 : -1;
}
// term (0..2) and dword of instruction j, dword position w, half h; term -1: nothing
__host__ __device__ constexpr int px_term(int j, int w, int h)
{
    return j == 0 ? 2 : j == 1 ? 1 : j == 2 ? (w < 2 ? 2 : 1) : j == 3 ? 0 : w < 2 ? 0 : h == 0 ? w - 2 : w == 2 ? 2 : -1;
}
__host__ __device__ constexpr int px_dword(int j, int w) { return j == 2 ? 4 + w % 2 : j == 4 ? (w < 2 ? 4 + w : 6) : w; }

// ---- key and value gradients: a (or dl) times the kernels, both as three bf16 terms.  Of their nine products the six of first with
// any, second with first and second, third with first terms are taken; the others are below 2^-26 of the whole.
// A lane of half h holds a pixel's shifts 4h..4h+3, 8+4h..8+4h+3 (A), 16+4h..16+4h+3 (B), and 24.  Left operands: [column of the tap]
// [row of the tap] of five pieces; lane = channel of 32 + 32 * half of the slots.  0, 1, 2: first, second and third terms for
// A; 3: first and second for B; 4: third for B, then of shift 24 first, first, first, second (half 0), second, third (half 1),
// for which the right operand has first, second, third, first and second, first terms.
constexpr int KV_MM = 5, KV_TAP = KV_MM * 64, KV_IMG = S * KV_TAP;     // 16-byte pieces
__host__ __device__ constexpr int kv_shift(int j, int h, int x)         // shift of slot x, -1: nothing
{
    return j < 3 ? 8 * (x / 4) + 4 * h + x % 4 : j == 3 || x < 4 ? 16 + 4 * h + x % 4 : h == 0 || x < 6 ? S - 1 : -1;
}
__host__ __device__ constexpr int kv_term(int j, int h, int x)
{
    return j < 3 ? j : j == 3 ? x / 4 : x < 4 ? 2 : h == 0 ? (x == 7 ? 1 : 0) : x == 4 ? 1 : 2;
}
// channel of row r = 16 h + i of 32 as the matrix results have it: where a pixel's q (or dO) stands for it
__host__ __device__ constexpr int kv_place(int c) { return ((c >> 2) & 1) * 16 + (c >> 3) * 4 + (c & 3); }

// the three terms of two numbers, term by term (an infinite one gives NaN)
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef float f2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void split3_pair(float x, float y, uint32_t (&t)[3])
{
    t[0] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{x, y}, bf2));
    const float x1 = x - __uint_as_float(t[0] << 16), y1 = y - __uint_as_float(t[0] & 0xffff0000u);
    t[1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{x1, y1}, bf2));
    const float x2 = x1 - __uint_as_float(t[1] << 16), y2 = y1 - __uint_as_float(t[1] & 0xffff0000u);
    t[2] = __builtin_amdgcn_perm(__float_as_uint(y2), __float_as_uint(x2), 0x07060302u);
}

__device__ __forceinline__ uint32_t lds_offset(const void* p) { return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p; }

}  // namespace split
}  // namespace slide
