// Kernel and bias gradients of the 5x5 window for bf16 activations, float32 sums on the bf16 matrix cores with split operands.
//   dwk[c,s,t] = scale * sum over items and pixels y of dl[s,y] * q[c,y] * k[c, y + off(t)]
//   dwv[c,s,t] =                                        a[s,y] * dO[c,y] * v[c, y + off(t)]
//   dbias[s]   =                                       dl[s,y]
#include "slide_split.h"

namespace slide {
namespace split {

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
// LDS in 16-byte pieces.  y: [channel][row][column of the tap][8 pixels], five of the four pieces of a row, so that neighbouring taps'
// reads lie in different banks (a column five pieces on, a row 25, a channel 205: 5, 25 and 125 modulo 16).  x: [channel][even
// pixels, odd pixels] as floats.  p: first, second and third terms, [shift][8 pixels] and one more.
constexpr int Y_COL = DW_COLS / 8 + 1, Y_ROW = KS * Y_COL, Y_CH = (DW_ROWS + 2 * R) * Y_ROW + 5;
constexpr int X_AT = 32 * Y_CH, X_CH = 2 * DW_PXS / 8 + 4, P_AT = X_AT + 32 * X_CH, P_S = DW_PXS / 8 + 1;
constexpr int DW_LDS = (P_AT + 3 * S * P_S) * 16;
static_assert(Y_ROW % 16 == 9 && Y_COL == 5 && Y_CH % 16 == S * Y_COL % 16 && DW_LDS <= (int)CU_LDS_BYTES && DW_ROWS == 4 && DW_COLS == 32, "");
// 25 taps of 32 channels are 25 tiles of 32 columns: three for each wave, one for all, which a wave has for one step of a pixel tile
constexpr int DW_TILES = S, DW_OWN = DW_TILES / (DW_NT / 64);
static_assert(DW_TILES == DW_OWN * (DW_NT / 64) + 1 && DW_PXS / 16 == DW_NT / 64, "");

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

// the upper halves of two floats: bf16 elements x, y, cut off
__device__ __forceinline__ uint32_t upper_halves(float x, float y) { return __builtin_amdgcn_perm(__float_as_uint(y), __float_as_uint(x), 0x07060302u); }

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

// sum of 16 neighbouring lanes, in all of them
__device__ __forceinline__ float row_sum(float x)
{
    auto turned = [&](auto by) { return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), decltype(by)::value, 0xf, 0xf, false)); };
    x += turned(std::integral_constant<int, 0x128>{});      // row_ror:8, 4, 2, 1
    x += turned(std::integral_constant<int, 0x124>{});
    x += turned(std::integral_constant<int, 0x122>{});
    return x + turned(std::integral_constant<int, 0x121>{});
}

// One block sums 32 channels of a head and side over its chunk of tiles of 4 rows and 32 columns.  The products
// q[p] k[p + off(t)] of 16 pixels, of 32 (channel, tap) pairs, are the right operand of a matrix instruction, dl[s,p] the left one
// (25 of 32 rows).  A product of two bf16 numbers is exactly the sum of two bf16 numbers, dl of three, and five instructions take
// all but the product of the last terms (2^-25 at most).  bf16 has the range of float32, so no number is too large or too
// small beside others.  A tile's sums are added to float32 totals: short sums, which is what float32 sums over 10^5 pixels
// need anyway.
// k (or v) lies in LDS once for every column of the taps, moved by it, so that eight pixels of a tap are one aligned read;
// a place whose pixel the map does not have holds zero, also where the neighbour that the tap reads is infinite.
// Bound by the vector unit (ten instructions for the terms of two products) and the matrix cores, which overlap badly with two
// waves per SIMD.  MI355X, B=64, 28x28, C=128, 4 heads: 225 us with 4x4x1 float32 matrix instructions, 135 like this; 130 with
// halves scaled by the largest of a tile, which lose small numbers beside large ones.  Tried: what the first terms leave by
// v_dot2_f32_bf16, two instructions less (151 us: it waits for the matrix cores); a channel's 25 taps to a matrix instruction
// instead of 32 pairs (174 with the same); reads one step earlier (139: spills).
// dwv is 1.43e-7 from 64 bits (8 x 28x28, 64 channels; float32 instructions 1.76e-7).
// ROWS: 0 less than four columns, 1 any number, 4 whole fours
template <int ROWS>
__global__ void __launch_bounds__(DW_NT, 2)
dw_split_kernel(const DwArgs a)
{
    constexpr bool NARROW = ROWS == 0;
    extern __shared__ __align__(16) unsigned char smem[];
    u4* const lds = (u4*)smem;
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
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int y = w.y0 + sr + 4 * i - R;
            uint32_t v[6], odd[5];
            yv[i].get(v, x, W, ch_live && y >= 0 && y < H);
#pragma unroll
            for (int j = 0; j < 5; ++j) odd[j] = __builtin_amdgcn_alignbit(v[j + 1], v[j], 16);
            u4* o = lds + grp * Y_CH + (sr + 4 * i) * Y_ROW + sb;
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
        f4 pd[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            if (ROWS == 4) {
                xd[j] = ch_live && row && x + 4 * j < W ? xv[j] : u2{0u, 0u};
                pd[j] = s_live && row && x + 4 * j < W ? pv[j] : f4{0.0f, 0.0f, 0.0f, 0.0f};
            } else {
                xd[j] = row4_cut<NARROW>(xv[j], x + 4 * j, W, ch_live && row);
                pd[j] = row4_cut<NARROW>(pv[j], x + 4 * j, W, s_live && row);
            }
        }
        const u4 xs = {xd[0][0], xd[0][1], xd[1][0], xd[1][1]};
        u4* const xo = lds + X_AT + grp * X_CH + (tid & 15);
        xo[0] = xs << 16;
        xo[DW_PXS / 8] = xs & 0xffff0000u;
        if (s_live) {
            u4 t[3];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float e0[3], e1[3];
                split3(pd[i / 2][2 * (i % 2)], e0);
                split3(pd[i / 2][2 * (i % 2) + 1], e1);
#pragma unroll
                for (int j = 0; j < 3; ++j) t[j][i] = upper_halves(e0[j], e1[j]);
            }
#pragma unroll
            for (int j = 0; j < 3; ++j) lds[P_AT + (j * S + grp) * P_S + (tid & 15)] = t[j];
        }
        if (sums_bias) {
#pragma unroll
            for (int j = 0; j < 2; ++j) bsum += (pd[j][0] + pd[j][1]) + (pd[j][2] + pd[j][3]);
        }
    };

    float total[DW_OWN + 1][13];
    int y_at[DW_OWN + 1], x_at[DW_OWN + 1];                 // bytes
#pragma unroll
    for (int j = 0; j <= DW_OWN; ++j) {
#pragma unroll
        for (int i = 0; i < 13; ++i) total[j][i] = 0.0f;
        const int n = 32 * (j < DW_OWN ? wave * DW_OWN + j : DW_TILES - 1) + col, c = n / S, t = n - c * S;
        y_at[j] = (c * Y_CH + t / KS * Y_ROW + t % KS * Y_COL + h) * 16;
        x_at[j] = (X_AT + c * X_CH + h) * 16;
    }
    const int p_at = (P_AT + min(col, S - 1) * P_S + h) * 16;
    const long t0 = a.tiles * chunk / a.chunks, t1 = a.tiles * (chunk + 1) / a.chunks;
    Where at{}, next{};
    if (t0 < t1) { next = locate(t0); fetch(next); }
    for (long tile = t0; tile < t1; ++tile) {
        at = next;
        __syncthreads();                                    // the tile before is no longer read
        put(at);
        if (tile + 1 < t1) { next = locate(tile + 1); fetch(next); }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");      // (not for the loads in flight)
        const int th = min(DW_ROWS, H - at.y0);
        // A step is 16 pixels of a row.  While the matrix cores multiply the products of one column tile, the vector unit forms the
        // next one's (fences for the scheduler deal them out: left alone, read, products and matrix instructions follow one
        // another).  The products with a second term have sums of their own, so that the others
        // round once per 16 pixels.
        struct Raw { u4 y, even, odd; };
        auto piece = [&](int at) { return *(const u4*)(smem + at); };
        auto read = [&](int j, int r, int ks) -> Raw {
            const int x = x_at[j] + (4 * r + 2 * ks) * 16;
            return Raw{piece(y_at[j] + (r * Y_ROW + 2 * ks) * 16), piece(x), piece(x + DW_PXS * 2)};
        };
        auto read_p = [&](int j, int r, int ks) -> bf8 { return __builtin_bit_cast(bf8, piece(p_at + (j * S * P_S + 4 * r + 2 * ks) * 16)); };
        // products of one dword's two pixels: first terms; what is left of them (`rest` holds it for the next call)
        float rest[2];
        auto form = [&](const Raw& raw, int i, u4& first, u4& second) {
            if (i == 4) { second[3] = upper_halves(rest[0], rest[1]); return; }
            const float g0 = __uint_as_float(raw.y[i] << 16) * __uint_as_float(raw.even[i]);
            const float g1 = __uint_as_float(raw.y[i] & 0xffff0000u) * __uint_as_float(raw.odd[i]);
            first[i] = upper_halves(g0, g1);
            __builtin_amdgcn_sched_barrier(0);
            if (i > 0) second[i - 1] = upper_halves(rest[0], rest[1]);
            rest[0] = g0 - __uint_as_float(__float_as_uint(g0) & 0xffff0000u); rest[1] = g1 - __uint_as_float(__float_as_uint(g1) & 0xffff0000u);
        };
        auto mul = [&](const bf8& p, const u4& g, f16v& sum) { sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p, __builtin_bit_cast(bf8, g), sum, 0, 0, 0); };
        auto fence = [] { __builtin_amdgcn_sched_barrier(0); };
        auto add = [&](int j, const f16v& sum) {
#pragma unroll
            for (int i = 0; i < 13; ++i) total[j][i] += sum[i];
        };
        auto rows = [&](auto nks) {
            constexpr int NKS = decltype(nks)::value, NB = NKS == 2 ? 2 : 3;     // (a row's products come round to the buffer they began with)
            bf8 P[3];
            u4 G[NB], L[NB];
            f16v acc[DW_OWN], small[DW_OWN];
#pragma unroll
            for (int j = 0; j < 3; ++j) P[j] = read_p(j, 0, 0);
            {
                const Raw raw = read(0, 0, 0);
#pragma unroll
                for (int i = 0; i < 5; ++i) form(raw, i, G[0], L[0]);
            }
            auto row = [&](auto at_row) {
                constexpr int r = decltype(at_row)::value;
#pragma unroll
                for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
                    for (int j = 0; j < DW_OWN; ++j) {
                        const bool first = r == 0 && ks == 0, last = j + 1 == DW_OWN;
                        const int nr = ks + 1 < NKS ? r : r + 1, nk = ks + 1 < NKS ? ks + 1 : 0;       // the next step
                        const bool more = !last || nr < DW_ROWS;
                        const int now = (ks * DW_OWN + j) % NB, then = (now + 1) % NB;
                        Raw raw;
                        if (more) raw = last ? read(0, nr, nk) : read(j + 1, r, ks);
                        auto next = [&](int i) { if (more) form(raw, i, G[then], L[then]); };
                        auto next_p = [&](int i) { if (last && more) P[i] = read_p(i, nr, nk); };
                        fence();
                        if (first) small[j] = f16v{};
                        mul(P[2], G[now], small[j]);
                        next_p(2);
                        mul(P[1], L[now], small[j]);
                        fence();
                        next(0);
                        mul(P[1], G[now], small[j]);
                        next_p(1);
                        fence();
                        next(1);
                        mul(P[0], L[now], small[j]);
                        fence();
                        next(2);
                        if (first) acc[j] = f16v{};
                        mul(P[0], G[now], acc[j]);
                        next_p(0);
                        fence();
                        next(3);
                        next(4);
                    }
            };
            row(std::integral_constant<int, 0>{});
            if (th > 1) row(std::integral_constant<int, 1>{});
            if (th > 2) row(std::integral_constant<int, 2>{});
            if (th > 3) row(std::integral_constant<int, 3>{});
#pragma unroll
            for (int j = 0; j < DW_OWN; ++j) add(j, acc[j] + small[j]);
        };
        const bool two = W - at.x0 > 16;
        if (two) rows(std::integral_constant<int, 2>{});
        else rows(std::integral_constant<int, 1>{});
        // the last column tile: each wave one step
        const int r = two ? wave >> 1 : wave, ks = two ? wave & 1 : 0;
        if (r < th) {
            const Raw raw = read(DW_OWN, r, ks);
            bf8 P[3];
            u4 G, L;
#pragma unroll
            for (int j = 0; j < 3; ++j) P[j] = read_p(j, r, ks);
#pragma unroll
            for (int i = 0; i < 5; ++i) form(raw, i, G, L);
            f16v acc = {};
            mul(P[2], G, acc);
            mul(P[1], L, acc);
            mul(P[1], G, acc);
            mul(P[0], L, acc);
            mul(P[0], G, acc);
            add(DW_OWN, acc);
        }
    }

    // the waves' sums of the last column tile: added in their order by the waves, a part of the rows each
    __syncthreads();
    float* const shared = (float*)smem;
#pragma unroll
    for (int i = 0; i < 13; ++i) shared[(wave * 13 + i) * 64 + lane] = total[DW_OWN][i];
    __syncthreads();
    const float f = a.f[side];
    auto store = [&](int tile, int i, float v) {
        const int n = 32 * tile + col, c = cb * 32 + n / S, t = n % S, s = 8 * (i / 4) + 4 * h + i % 4;
        if (c < a.d && s < S) a.partial[((((long)chunk * 2 + side) * a.C + (long)m * a.d + c) * S + s) * S + t] = f * v;
    };
#pragma unroll
    for (int j = 0; j < DW_OWN; ++j)
#pragma unroll
        for (int i = 0; i < 13; ++i) store(wave * DW_OWN + j, i, total[j][i]);
    for (int i = wave; i < 13; i += DW_NT / 64) {
        float v = 0.0f;
        for (int w = 0; w < DW_NT / 64; ++w) v += shared[(w * 13 + i) * 64 + lane];
        store(DW_TILES - 1, i, v);
    }
    if (sums_bias) {
        const float b = row_sum(bsum);
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
