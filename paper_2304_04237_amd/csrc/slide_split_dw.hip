// Kernel and bias gradients of the 5x5 window for bf16 activations, float32 sums on the half-precision matrix cores with
// split operands.
//   dwk[c,s,t] = scale * sum over items and pixels y of dl[s,y] * q[c,y] * k[c, y + off(t)]
//   dwv[c,s,t] =                                        a[s,y] * dO[c,y] * v[c, y + off(t)]
//   dbias[s]   =                                       dl[s,y]
#include "slide_split.h"

namespace slide {
namespace split {

typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef u2 u2_any __attribute__((aligned(2)));
typedef f4 f4_any __attribute__((aligned(4)));

struct DwArgs {
    const bf16_bits* y[2]; const bf16_bits* x[2];           // k, v; q, dO
    const float* p[2];                                      // dl, a: [B, heads, S, H, W]
    float* partial;                                         // [chunks][2][C][S][S]
    float* bias_partial;                                    // [chunks][heads][S], may be null
    float f[2];                                             // logit scale, 1
    int H, W, C, d, heads, ncb;
    int ntr, ntc, chunks;
    long tiles;
};

constexpr int DW_NT = 512, DW_PXS = DW_ROWS * DW_COLS;      // threads, pixels of a tile
// LDS in 16-byte pieces.  y: [channel][row][column of the tap][8 pixels], five of the four pieces of a row, so that the 25 taps of
// a read lie in different banks (a row of the taps 25 pieces on, a column five).  x: [channel][8 pixels].  p: first and second
// halves, [shift][8 pixels] and one more.
constexpr int Y_COL = DW_COLS / 8 + 1, Y_ROW = KS * Y_COL, Y_CH = (DW_ROWS + 2 * R) * Y_ROW;
constexpr int X_AT = 32 * Y_CH, X_CH = DW_PXS / 8, P_AT = X_AT + 32 * X_CH, P_S = DW_PXS / 8 + 1, F_AT = P_AT + 2 * S * P_S;
constexpr int DW_LDS = (F_AT + 32 / 4 + 32 / 4) * 16;       // then the inverse scales of the shifts and of the channels
static_assert(Y_ROW % 16 == 9 && Y_COL == 5 && DW_LDS <= (int)CU_LDS_BYTES && DW_ROWS == 4 && DW_COLS == 32, "");

// elements e0..e0+3 of a row of W, zeros outside; NARROW: rows of less than four elements.  The load and, later, the rest.
template <bool NARROW>
__device__ __forceinline__ u2 row4_load(const bf16_bits* row, int e0, int W)
{
    if (!NARROW) return *(const u2_any*)(row + row_at(e0, 4, W));
    uint32_t e[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) e[i] = e0 + i >= 0 && e0 + i < W ? row[e0 + i] : 0u;
    return u2{e[0] | e[1] << 16, e[2] | e[3] << 16};
}
template <bool NARROW>
__device__ __forceinline__ u2 row4_cut(u2 raw, int e0, int W, bool row)
{
    uint64_t v = (uint64_t)raw[1] << 32 | raw[0];
    if (!NARROW) {
        const int past = e0 - row_at(e0, 4, W);       // elements between where they belong and where they were loaded
        v = past >= 0 ? v >> (16 * min(past, 3)) : v << (16 * min(-past, 3));
        row = row && past < 4 && past > -4;
    }
    return row ? u2{(uint32_t)v, (uint32_t)(v >> 32)} : u2{0u, 0u};
}
template <bool NARROW>
__device__ __forceinline__ f4 row4_load(const float* row, int e0, int W)
{
    if (!NARROW) return *(const f4_any*)(row + row_at(e0, 4, W));
    f4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = e0 + i < W ? row[e0 + i] : 0.0f;
    return v;
}
template <bool NARROW>
__device__ __forceinline__ f4 row4_cut(f4 v, int e0, int W, bool row)
{
    if (!NARROW) {
        const int past = max(e0 - (W - 4), 0);
        if (past & 1) v = f4{v[1], v[2], v[3], 0.0f};
        if (past & 2) v = f4{v[2], v[3], 0.0f, 0.0f};
        row = row && past < 4;
    }
    return row ? v : f4{0.0f, 0.0f, 0.0f, 0.0f};
}

// (the dword by value: a bit cast of a vector's element takes the first one whatever the index)
__device__ __forceinline__ h2 as_h2(uint32_t x) { return __builtin_bit_cast(h2, x); }

// elements x-2..x+9 of a row as six dwords, zeros outside.  Rows of whole fours (4): every piece is all inside or all
// outside, and x is a multiple of eight.
template <int ROWS> struct Row12 {
    u2 v[3];
    __device__ __forceinline__ void load(const bf16_bits* row, int x, int W)
    {
#pragma unroll
        for (int j = 0; j < 3; ++j) v[j] = row4_load<ROWS == 0>(row, x - R + 4 * j, W);
    }
    __device__ __forceinline__ void get(uint32_t (&d)[6], int x, int W, bool row) const
    {
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const u2 c = row4_cut<ROWS == 0>(v[j], x - R + 4 * j, W, row);
            d[2 * j] = c[0]; d[2 * j + 1] = c[1];
        }
    }
};
template <> struct Row12<4> {
    typedef uint32_t u1_any __attribute__((aligned(2)));
    uint32_t a, z;
    u2 v[2];
    __device__ __forceinline__ void load(const bf16_bits* row, int x, int W)
    {
        auto at = [&](int i) { return row + row_at(fours_from(i, x), fours_length(i), W); };
        a = *(const u1_any*)at(0); z = *(const u1_any*)at(3);
        v[0] = *(const u2_any*)at(1); v[1] = *(const u2_any*)at(2);
    }
    __device__ __forceinline__ void get(uint32_t (&d)[6], int x, int W, bool row) const
    {
        const bool in = row && x < W, more = row && x + 4 < W;
        d[0] = row && x > 0 && x - 2 < W ? a : 0u;
        d[1] = in ? v[0][0] : 0u; d[2] = in ? v[0][1] : 0u;
        d[3] = more ? v[1][0] : 0u; d[4] = more ? v[1][1] : 0u;
        d[5] = row && x + 8 < W ? z : 0u;
    }
};

// largest of 16 neighbouring lanes, in all of them
template <typename F>
__device__ __forceinline__ uint32_t row_reduce(uint32_t x, F&& f)
{
    x = f(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x128, 0xf, 0xf, false));     // row_ror:8, 4, 2, 1
    x = f(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x124, 0xf, 0xf, false));
    x = f(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x122, 0xf, 0xf, false));
    return f(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x121, 0xf, 0xf, false));
}
typedef int16_t s2 __attribute__((ext_vector_type(2)));
// running maximum of the finite magnitudes in two bf16 elements, plus 0x80 (infinities and NaN become negative)
__device__ __forceinline__ uint32_t max_finite(uint32_t m, uint32_t two)
{
    const s2 t = __builtin_bit_cast(s2, two & 0x7fff7fffu) + s2{0x80, 0x80};
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(s2, m), t));
}
// the power of two that brings the largest of them into [2^6, 2^7), and its inverse
__device__ __forceinline__ void scale_of_max(uint32_t m, float& up, float& down)
{
    m = row_reduce(m, [](uint32_t a, uint32_t b) {
        return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(s2, a), __builtin_bit_cast(s2, b)));
    });
    const int top = max((int)(int16_t)m, (int)m >> 16) - 0x80, e = max(top >> 7, 12);       // (exponents below 12 are nothing)
    up = __uint_as_float((uint32_t)min(254 + 6 - e, 254) << 23);
    down = __uint_as_float((uint32_t)max(e - 6, 1) << 23);
}
// two scaled bf16 elements as halves
__device__ __forceinline__ uint32_t to_halves(uint32_t two, float up)
{
    const h2 v = {(_Float16)(up * __uint_as_float(two << 16)), (_Float16)(up * __uint_as_float(two & 0xffff0000u))};
    return __builtin_bit_cast(uint32_t, v);
}

// One block sums 32 channels of a head and side over its chunk of tiles of 4 rows and 32 columns.  A channel's products
// q[p] k[p + off(t)] of 16 pixels are the right operand of a matrix instruction (25 of 32 columns are its taps), dl[s,p] the
// left one (25 of 32 rows).  A product of two bf16 numbers is exactly the sum of two halves (one multiplication and one fused
// multiply-add on pairs), dl is the sum of two halves to 23 bits, and three instructions take all but the product of the
// two second terms (2^-24).  So that halves hold any value, a tile's channels and shifts are scaled by powers of two when they
// go to LDS, and the tile's sums are added to float32 totals with their inverses: short sums, which is what float32 sums
// over 10^5 pixels need anyway.  A wave has four channels, whose sums stay in its registers for the whole chunk.
// k (or v) lies in LDS once for every column of the taps, moved by it, so that eight pixels of a tap are one aligned read;
// a place whose pixel the map does not have holds zero, also where the neighbour that the tap reads is infinite.
// Bound by the vector unit (half of the time: a tile's conversions, copies and scales are as much as its products) and the
// matrix cores (a third), which take turns between a tile's two barriers.  MI355X, B=64, 28x28, C=128, 4 heads: 225 us with 4x4x1 float32
// matrix instructions, 135 like this; 127 with the second terms' products in the same sums, but then dwv is 2.09e-7 from
// 64 bits instead of 1.67e-7 (8 x 28x28; float32 instructions 1.87e-7).
// ROWS: 0 less than four columns, 1 any number, 4 whole fours
template <int ROWS>
__global__ void __launch_bounds__(DW_NT, 2)
dw_split_kernel(const DwArgs a)
{
    constexpr bool NARROW = ROWS == 0;
    extern __shared__ __align__(16) unsigned char smem[];
    u4* const lds = (u4*)smem;
    float* const fs = (float*)(lds + F_AT);                 // inverse scales: shifts, channels
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, h = lane >> 5;
    const int H = a.H, W = a.W;
    const int m = blockIdx.z, side = blockIdx.y & 1, cb = blockIdx.y >> 1, chunk = blockIdx.x;
    const long HW = (long)H * W;

    // staging: sixteen threads per channel and per shift, four rows by four pieces of eight pixels
    const int grp = tid >> 4, sr = (tid >> 2) & 3, sb = tid & 3;
    const bool ch_live = cb * 32 + grp < a.d;
    const long chan = (long)m * a.d + min(cb * 32 + grp, a.d - 1);
    const bool s_live = grp < S;
    const bool sums_bias = side == 0 && cb == 0 && a.bias_partial;
    float bsum = 0.0f;
    struct Where { long b; int y0, x0; };
    auto locate = [&](long tile) -> Where {
        const long b = tile / (a.ntr * a.ntc);
        const int r = (int)(tile - b * (a.ntr * a.ntc)), ty = r / a.ntc;
        return Where{b, ty * DW_ROWS, (r - ty * a.ntc) * DW_COLS};
    };
    Row12<ROWS> yv[2];
    u2 xv[2];
    f4 pv[2];
    auto fetch = [&](const Where& w) {
        const long base = (w.b * a.C + chan) * HW;
        const int x = w.x0 + 8 * sb;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const bf16_bits* row = a.y[side] + base + (long)min(max(w.y0 + sr + 4 * i - R, 0), H - 1) * W;
            yv[i].load(row, x, W);
        }
        const int y = min(w.y0 + sr, H - 1);
        const bf16_bits* row = a.x[side] + base + (long)y * W;
        const float* prow = a.p[side] + ((w.b * a.heads + m) * S + min(grp, S - 1)) * HW + (long)y * W;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            xv[j] = row4_load<NARROW>(row, x + 4 * j, W);
            pv[j] = row4_load<NARROW>(prow, x + 4 * j, W);
        }
    };
    auto put = [&](const Where& w) {
        const int x = w.x0 + 8 * sb;
        // pixels of the piece that the map has, as masks of the dwords
        uint32_t has[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) has[i] = x + 2 * i + 1 < W ? 0xffffffffu : x + 2 * i < W ? 0xffffu : 0u;
        uint32_t yd[2][6], top = 0u;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int y = w.y0 + sr + 4 * i - R;
            yv[i].get(yd[i], x, W, ch_live && y >= 0 && y < H);
#pragma unroll
            for (int j = 0; j < 6; ++j) top = max_finite(top, yd[i][j]);
        }
        float up, down, xup, xdown;
        scale_of_max(top, up, down);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            u4* o = lds + grp * Y_CH + (sr + 4 * i) * Y_ROW + sb;
            uint32_t v[6], odd[5];
#pragma unroll
            for (int j = 0; j < 6; ++j) v[j] = to_halves(yd[i][j], up);
#pragma unroll
            for (int j = 0; j < 5; ++j) odd[j] = __builtin_amdgcn_alignbit(v[j + 1], v[j], 16);
#pragma unroll
            for (int c = 0; c < KS; ++c) {
                u4 t;
#pragma unroll
                for (int j = 0; j < 4; ++j) t[j] = (c % 2 ? odd[c / 2 + j] : v[c / 2 + j]) & has[j];
                o[c * Y_COL] = t;
            }
        }
        const bool row = w.y0 + sr < H;
        u2 xd[2];
        top = 0u;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            if (ROWS == 4) xd[j] = ch_live && row && x + 4 * j < W ? xv[j] : u2{0u, 0u};
            else xd[j] = row4_cut<NARROW>(xv[j], x + 4 * j, W, ch_live && row);
            top = max_finite(max_finite(top, xd[j][0]), xd[j][1]);
        }
        scale_of_max(top, xup, xdown);
        lds[X_AT + grp * X_CH + (tid & 15)] = u4{to_halves(xd[0][0], xup), to_halves(xd[0][1], xup), to_halves(xd[1][0], xup), to_halves(xd[1][1], xup)};
        if ((tid & 15) == 0) fs[32 + grp] = down * xdown;
        // dl (or a)
        f4 pd[2];
        float big = 0.0f, sum = 0.0f;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            if (ROWS == 4) pd[j] = s_live && row && x + 4 * j < W ? pv[j] : f4{0.0f, 0.0f, 0.0f, 0.0f};
            else pd[j] = row4_cut<NARROW>(pv[j], x + 4 * j, W, s_live && row);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float mag = __builtin_fabsf(pd[j][e]);
                big = fmaxf(big, mag < INFINITY ? mag : 0.0f);
                sum += pd[j][e];
            }
        }
        bsum += sum;
        big = __uint_as_float(row_reduce(__float_as_uint(big), [](uint32_t p, uint32_t q) { return max(p, q); }));
        scale_for(big, up, down);
        u4 hi, lo;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            uint32_t h0, h1, l0, l1;
            split2(pd[i / 2][2 * (i % 2)] * up, h0, l0);
            split2(pd[i / 2][2 * (i % 2) + 1] * up, h1, l1);
            hi[i] = h0 | h1 << 16; lo[i] = l0 | l1 << 16;
        }
        if (s_live) {
            lds[P_AT + grp * P_S + (tid & 15)] = hi;
            lds[P_AT + (S + grp) * P_S + (tid & 15)] = lo;
            if ((tid & 15) == 0) fs[grp] = down;
        }
    };

    float total[4][13];
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < 13; ++i) total[e][i] = 0.0f;
    const int t = min(col, S - 1), tr = t / KS, tc = t - tr * KS;
    const u4* const yp = lds + wave * 4 * Y_CH + tr * Y_ROW + tc * Y_COL + h;
    const u4* const xp = lds + X_AT + wave * 4 * X_CH + h;
    const u4* const pp = lds + P_AT + t * P_S + h;
    if (tid < 7) fs[S + tid] = 0.0f;

    const long t0 = a.tiles * chunk / a.chunks, t1 = a.tiles * (chunk + 1) / a.chunks;
    Where at{}, next{};
    if (t0 < t1) { next = locate(t0); fetch(next); }
    for (long tile = t0; tile < t1; ++tile) {
        at = next;
        __syncthreads();                                    // the tile before is no longer read
        put(at);
        if (tile + 1 < t1) { next = locate(tile + 1); fetch(next); }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");      // (not for the loads in flight)
        const int th = min(DW_ROWS, H - at.y0), nks = W - at.x0 > 16 ? 2 : 1;
        // two channels at a time; the products with a second term have sums of their own, so that the others round once per 16
        // pixels (added to them as they come: three times)
#pragma unroll
        for (int e0 = 0; e0 < 4; e0 += 2) {
            f16v acc[2] = {}, small[2] = {};
#pragma unroll 1
            for (int r = 0; r < th; ++r)
#pragma unroll 1
                for (int ks = 0; ks < nks; ++ks) {
                    const u4 ph = pp[r * 4 + 2 * ks], pl = pp[S * P_S + r * 4 + 2 * ks];
                    const h8 Ph = __builtin_bit_cast(h8, ph), Pl = __builtin_bit_cast(h8, pl);
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const u4 yd = yp[(e0 + e) * Y_CH + r * Y_ROW + 2 * ks], xd = xp[(e0 + e) * X_CH + r * 4 + 2 * ks];
                        u4 g, gl;
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const h2 y2 = as_h2(yd[i]), x2 = as_h2(xd[i]);
                            const h2 hi = y2 * x2;
                            g[i] = __builtin_bit_cast(uint32_t, hi);
                            gl[i] = __builtin_bit_cast(uint32_t, __builtin_elementwise_fma(y2, x2, -hi));
                        }
                        const h8 G = __builtin_bit_cast(h8, g), L = __builtin_bit_cast(h8, gl);
                        small[e] = __builtin_amdgcn_mfma_f32_32x32x16_f16(Ph, L, small[e], 0, 0, 0);
                        small[e] = __builtin_amdgcn_mfma_f32_32x32x16_f16(Pl, G, small[e], 0, 0, 0);
                        acc[e] = __builtin_amdgcn_mfma_f32_32x32x16_f16(Ph, G, acc[e], 0, 0, 0);
                    }
                }
            const float fc0 = fs[32 + wave * 4 + e0], fc1 = fs[33 + wave * 4 + e0];
            asm volatile("" ::: "memory");                  // (the shifts' scales are read now and not kept over the loop)
#pragma unroll
            for (int i = 0; i < 13; ++i) {
                const float fr = fs[8 * (i / 4) + 4 * h + i % 4];
                total[e0][i] = fmaf(acc[0][i] + small[0][i], fr * fc0, total[e0][i]);
                total[e0 + 1][i] = fmaf(acc[1][i] + small[1][i], fr * fc1, total[e0 + 1][i]);
            }
        }
    }

    const float f = a.f[side];
    if (col < S)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int c = cb * 32 + wave * 4 + e;
            if (c >= a.d) continue;
            float* out = a.partial + (((long)chunk * 2 + side) * a.C + (long)m * a.d + c) * S * S + t;
#pragma unroll
            for (int i = 0; i < 13; ++i) {
                const int s = 8 * (i / 4) + 4 * h + i % 4;
                if (s < S) out[s * S] = f * total[e][i];
            }
        }
    if (sums_bias) {
        auto add = [](uint32_t p, uint32_t q) { return __float_as_uint(__uint_as_float(p) + __uint_as_float(q)); };
        const float b = __uint_as_float(row_reduce(__float_as_uint(bsum), add));
        if (s_live && (tid & 15) == 0) a.bias_partial[((long)chunk * a.heads + m) * S + grp] = b;
    }
}

}  // namespace split

size_t split_dw_partial_floats(const Problem& p)
{
    const split::DwSplitPlan t = split::plan_dw_split(p.B, p.H, p.W, 2 * p.heads * ((p.d() + 31) / 32));
    return (size_t)t.chunks * (2 * (size_t)p.C * p.S() * p.S() + (size_t)p.heads * p.S());
}

hipError_t launch_bwd_dw_split(const Problem& p, const void* dout, const void* q, const void* k, const void* v,
                               const float* attn_ws, const float* dl_ws, float* partial, float* dwk, float* dwv,
                               float* dbias, hipStream_t st)
{
    using namespace split;
    const int ncb = (p.d() + 31) / 32;
    const DwSplitPlan t = plan_dw_split(p.B, p.H, p.W, 2 * p.heads * ncb);
    const long side = (long)p.C * p.S() * p.S();
    DwArgs a{};
    a.y[0] = (const bf16_bits*)k; a.y[1] = (const bf16_bits*)v; a.x[0] = (const bf16_bits*)q; a.x[1] = (const bf16_bits*)dout;
    a.p[0] = dl_ws; a.p[1] = attn_ws;
    a.partial = partial;
    a.bias_partial = dbias ? partial + (size_t)t.chunks * 2 * side : nullptr;
    a.f[0] = p.logit_scale(); a.f[1] = 1.0f;
    a.H = p.H; a.W = p.W; a.C = p.C; a.d = p.d(); a.heads = p.heads; a.ncb = ncb;
    a.ntr = t.ntr; a.ntc = t.ntc; a.chunks = t.chunks; a.tiles = t.tiles;
    const auto kernel = p.W < 4 ? dw_split_kernel<0> : p.W % 4 ? dw_split_kernel<1> : dw_split_kernel<4>;
    static LdsOptIn opt_in;
    hipError_t e = opt_in.ensure({(const void*)dw_split_kernel<0>, (const void*)dw_split_kernel<1>, (const void*)dw_split_kernel<4>}, (int)CU_LDS_BYTES);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3((unsigned)t.chunks, (unsigned)(2 * ncb), (unsigned)p.heads), dim3(DW_NT), DW_LDS, st, a);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_bwd_dw_reduce(partial, dwk, dwv, side, t.chunks, a.bias_partial, dbias, p.heads * p.S(), p.accumulate, st);
}

}  // namespace slide
