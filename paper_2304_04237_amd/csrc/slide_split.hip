// Backward of bf16 activations with a 5x5 window: logits, softmax, da, dl, dq, dk and dv in float32, the learned-kernel
// contractions on the 16-bit matrix cores with their float32 operands split (slide_split.h).
#include "slide_split.h"

namespace slide {
namespace split {

constexpr int N = 13;                                       // shifts of a lane of half h: 4 h + 0..3 (+ 8, + 16), 24 (half 0)

// Operand images of both kernels.  grid = (heads * channels in 32s, 2 tensors), block = 320; zeros past the head's channels.
// d4: channels in fours.
__global__ void __launch_bounds__(PX_CH)
prep_split_kernel(const float* __restrict__ wk, const float* __restrict__ wv, u4* __restrict__ px_image, u4* __restrict__ kv_image,
                  int d, int ncb, float idw)
{
    __shared__ float w[S * S];
    const int m = blockIdx.x / (32 * ncb), c = blockIdx.x - m * (32 * ncb), heads = gridDim.x / (32 * ncb), tid = threadIdx.x;
    const int side = blockIdx.y, d4 = (d + 3) & ~3;
    const bool is = c < d;
    const float* src = (side ? wv : wk) + ((long)m * d + min(c, d - 1)) * S * S;
    for (int i = tid; i < S * S; i += PX_CH) w[i] = is ? src[i] + (i % (S + 1) == 0 ? idw : 0.0f) : 0.0f;       // shift s reads tap s
    __syncthreads();
    const int j = tid >> 6, lane = tid & 63, s = lane & 31, h = lane >> 5;
    if (c < d4) {
        u4 o = {0u, 0u, 0u, 0u};
        if (s < S)
#pragma unroll
            for (int x = 0; x < 8; ++x) {
                const int term = px_term(j, x >> 1, h), tap = px_tap(h, px_dword(j, x >> 1), x & 1);
                if (term < 0 || tap < 0) continue;
                float t[3];
                split3(w[s * S + tap], t);
                o[x >> 1] |= (uint32_t)f32_to_bf16(term == 0 ? t[0] : term == 1 ? t[1] : t[2]) << (16 * (x & 1));
            }
        px_image[((long)(side * heads + m) * d4 + c) * PX_CH + tid] = o;
    }
    u4* kv = kv_image + ((long)(side * heads + m) * ncb + c / 32) * KV_IMG + c % 32;
    for (int i = tid; i < S * KV_MM * 2; i += PX_CH) {      // (tap, piece, half)
        const int hh = i & 1, jj = (i >> 1) % KV_MM, n = (i >> 1) / KV_MM, t = (n % KS) * KS + n / KS;
        u4 o = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int x = 0; x < 8; ++x) {
            const int sh = kv_shift(jj, hh, x);
            if (sh < 0) continue;
            const int term = kv_term(jj, hh, x);
            float e[3];
            split3(w[sh * S + t], e);
            o[x >> 1] |= (uint32_t)f32_to_bf16(term == 0 ? e[0] : term == 1 ? e[1] : e[2]) << (16 * (x & 1));
        }
        kv[(n * KV_MM + jj) * 64 + 32 * hh] = o;
    }
}

struct PixelArgs {
    const bf16_bits* q; const bf16_bits* k; const bf16_bits* v; const bf16_bits* dout;
    const u4* wk; const u4* wv;                             // operand images [C][PX_CH]
    const float* bias;
    bf16_bits* out;                                         // dq
    float* a_ws; float* dl_ws;                              // [B, heads, S, H, W]
    unsigned char* xt[2];                                   // q, dO: [B, heads, H, W, channels in 32s] as kv_place has them
    int H, W, C, d;
    float scale;
    Stack cut;
};

constexpr int PG = SPLIT_PX / 64, NT = SPLIT_PX;            // a wave has 64 pixels

// One run of 256 pixels of one head, 64 per wave, in steps of four channels; the planes of all items are one tall map (Stack), so
// that every run but the last is full.  A wave's 64 pixels are two groups of 32 columns of a 32x32x16 matrix instruction,
// whose rows are the 25 shifts: five instructions form a channel's windows, which are multiplied with q (or dO) and added over
// the channels, or with dl and added over the shifts, on the vector unit.
// LDS holds a step's halo tile as [pixel][4 channels] of dwords, each the pixel and its right neighbour: the taps of a window
// row are the dwords of every other pixel, one 16-byte read for four channels, and neighbouring lanes read neighbouring
// places.  A step is fetched while the one before it is multiplied and goes to the other of two LDS buffers, the operand
// image by loads that write LDS.
// Bound by what is not overlapped: the matrix cores are busy for 37 % of the time, the vector unit for 50 %, LDS reads (36
// of 16 bytes per step and wave) for 25 %, and two waves per SIMD do not hide each other's.  MI355X, B=64, 28x28, C=128, 4
// heads: 386 us with 4x4x1 float32 matrix instructions, 155 like this, 11 of them for the compensated sums.  Tried, without
// those: a tile of 8 bytes per pixel, whose reads need no moves (137 -> 152 us: 4-byte reads at 8-byte steps meet in the
// banks), a wave per channel with its operands and eight groups' sums in registers (191 us: spills), the vector work dealt between
// the matrix instructions by hand (176 us: spills).
// ONE: planes of one element, which have no dword to load.
template <bool ONE>
__global__ void __launch_bounds__(NT, 2)
pixel_split_kernel(const PixelArgs a)
{
    constexpr int NI = SPLIT_TILE / NT;                     // places of the tile per thread

    extern __shared__ __align__(16) unsigned char smem[];
    u4* const lds = (u4*)smem;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, h = lane >> 5;
    const int H = a.H, W = a.W, d = a.d, HS = H + R;
    const int m = blockIdx.y;
    const long HW = (long)H * W, item = a.C * HW;
    const int strip = blockIdx.x / a.cut.runs, run = blockIdx.x - strip * a.cut.runs;
    const int j0 = strip * a.cut.TW + min(strip, a.cut.wider), tw = a.cut.TW + (strip < a.cut.wider);
    const long n_all = (long)a.cut.planes * H * tw, n0 = (long)run * a.cut.px;
    if (n0 >= n_all) return;
    const int npx = a.cut.npx, RP = a.cut.RP;
    const int here = (int)min((long)a.cut.px, n_all - n0);  // pixels of this run
    const int stage = 4 * PX_CH + npx;                      // 16-byte pieces of a step: operands, tile

    // item and row of the first pixel; the other ones count from there
    const long line0 = n0 / tw;
    const int x0 = (int)(n0 - line0 * tw), p0 = (int)(line0 / H), y0 = (int)(line0 - (long)p0 * H);
    const int b0 = blockIdx.z * a.cut.planes + p0;
    auto pixel = [&](int n, int& db, int& ti, int& tj) -> bool {
        const int nn = min(n, here - 1) + x0, line = nn / tw;
        tj = nn - line * tw;
        db = (y0 + line) / H; ti = y0 + line - db * H;
        return n < here;
    };
    const bool wave_live = wave * 64 < here;
    // this lane's own pixel, and its column in each group
    int db, ti, tj;
    const bool live = pixel(wave * 64 + lane, db, ti, tj);
    const uint32_t own = ((uint32_t)db * (uint32_t)item + (uint32_t)ti * W + j0 + tj) * 2u;
    const int xt_bytes = (d + 31) / 32 * 64;                // of a pixel
    const long own_px = ((long)(b0 + db) * (a.C / d) + m) * HW + (long)ti * W + j0 + tj;
    int at[2];
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        pixel(wave * 64 + 32 * g + col, db, ti, tj);
        at[g] = 4 * PX_CH + (db * HS + ti - y0) * RP + tj;  // its upper left tap
    }

    const long head = (long)b0 * item + (long)m * d * HW;
    // a tile place: where its two elements are loaded (one dword inside the plane), which of the four bytes go where
    auto place = [&](int e, uint32_t& sel) -> uint32_t {
        const int rr = e / RP, x = j0 + e - rr * RP - R, v = y0 + rr - R;
        const int db = max(v, 0) / HS, y = v - db * HS;
        const bool row = e < npx && y >= 0 && y < H && p0 + db < a.cut.planes, lo = row && x >= 0 && x < W, hi = row && x + 1 >= 0 && x + 1 < W;
        const int at = y * W + x;
        int from = 0;
        if (lo && hi) { sel = 0x03020100u; from = at; }
        else if (lo) { sel = at > 0 ? 0x0c0c0302u : 0x0c0c0100u; from = max(at - 1, 0); }
        else if (hi) { sel = at >= 0 ? 0x03020c0cu : 0x01000c0cu; from = max(at, 0); }
        else { sel = 0x0c0c0c0cu; return 0u; }
        return ((uint32_t)db * (uint32_t)item + (uint32_t)from) * 2u;
    };
    uint32_t sel[NI], off[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) off[i] = place(tid + i * NT, sel[i]);
    auto load2 = [&](const bf16_bits* base, uint32_t o) -> uint32_t {
        const char* p = (const char*)base + o;
        return ONE ? (uint32_t) * (const bf16_bits*)p : *(const u32_any*)p;
    };

    const int nq = (d + 3) >> 2, steps = 3 * nq;
    uint32_t yr[NI][4], xr[4];
    const uint32_t lds0 = lds_offset(smem);
    // step k: phase k / nq (k with q, v with dO, k again), channels 4 (k % nq) on
    auto source = [&](int k, const bf16_bits*& y, const bf16_bits*& x, const u4*& w, int& c0) {
        const int ph = k >= 2 * nq ? 2 : k >= nq;
        c0 = 4 * (k - ph * nq);
        y = (ph == 1 ? a.v : a.k) + head;
        x = (ph == 1 ? a.dout : a.q) + head;
        w = (ph == 1 ? a.wv : a.wk) + ((long)m * nq * 4 + c0) * PX_CH;
    };
    auto fetch = [&](int k) {
        const bf16_bits *y, *x; const u4* w; int c0;
        source(k, y, x, w, c0);
#pragma unroll
        for (int u = 0; u < 4 * PX_MM / PG; ++u)
            load_to_lds(w + (wave + u * PG) * 64, lane * 16u, lds0 + ((k & 1) * stage + (wave + u * PG) * 64) * 16u);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const long cb = (long)min(c0 + e, d - 1) * HW;
#pragma unroll
            for (int i = 0; i < NI; ++i) yr[i][e] = load2(y + cb, off[i]);
            xr[e] = *(const bf16_bits*)((const char*)(x + cb) + own);
        }
    };
    auto put = [&](int k) {
        u4* o = lds + (k & 1) * stage + 4 * PX_CH;
#pragma unroll
        for (int i = 0; i < NI; ++i)
            if (tid + i * NT < npx)
                o[tid + i * NT] = u4{__builtin_amdgcn_perm(0u, yr[i][0], sel[i]), __builtin_amdgcn_perm(0u, yr[i][1], sel[i]),
                                     __builtin_amdgcn_perm(0u, yr[i][2], sel[i]), __builtin_amdgcn_perm(0u, yr[i][3], sel[i])};
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");    // the operands have landed
    };

    fetch(0);
    put(0);
    // runs body(channel, channel of the step, x of both groups, windows of both groups) over one phase's channels
    auto phase = [&](int ph, auto&& body, auto&& after_quad) {
#pragma unroll 1
        for (int u = 0; u < nq; ++u) {
            const int k = ph * nq + u;
            uint32_t xq[2][2];                              // x of channels (0, 1), (2, 3), by group
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const uint32_t mine = xr[2 * i] | xr[2 * i + 1] << 16;
                const auto sw = __builtin_amdgcn_permlane32_swap(mine, mine, false, false);
                xq[0][i] = sw[0]; xq[1][i] = sw[1];
            }
            if (ph < 2 && live)
                *(u2*)(a.xt[ph] + own_px * xt_bytes + (u >> 3) * 64 + kv_place(4 * (u & 7)) * 2) = u2{xr[0] | xr[1] << 16, xr[2] | xr[3] << 16};
            __syncthreads();
            if (k + 1 < steps) fetch(k + 1);
            if (wave_live) {
                const u4* wl = lds + (k & 1) * stage + lane;
                u4 r[2][8];
#pragma unroll
                for (int g = 0; g < 2; ++g) {
                    const u4* t = lds + (k & 1) * stage + at[g];
                    const u4* th = t + 2 * h * RP;
                    r[g][0] = th[0]; r[g][1] = th[2]; r[g][2] = th[4];
                    r[g][3] = th[RP]; r[g][4] = th[RP + 2]; r[g][5] = th[RP + 4];
                    r[g][6] = t[4 * RP + 2 * h]; r[g][7] = t[4 * RP + 4];
                }
                // chain i: the five instructions of channel i / 2 and group i % 2; the vector work of the chain before follows
                bf8 A[PX_MM];
                f16v acc[2];
#pragma unroll
                for (int i = 0; i <= 8; ++i) {
                    const int e = i / 2, g = i % 2;
                    if (i < 8) {
                        if (g == 0)
#pragma unroll
                            for (int j = 0; j < PX_MM; ++j) A[j] = __builtin_bit_cast(bf8, wl[e * PX_CH + j * 64]);
                        const u4 t0 = {r[g][0][e], r[g][1][e], r[g][3][e], r[g][4][e]};
                        const uint32_t d4 = r[g][6][e], d5 = __builtin_amdgcn_perm(r[g][5][e], r[g][2][e], 0x05040100u), dx = r[g][7][e] & 0xffffu;
                        const u4 t1 = {d4, d5, d4, d5}, t2 = {d4, d5, dx, dx};
                        const bf8 B0 = __builtin_bit_cast(bf8, t0), B1 = __builtin_bit_cast(bf8, t1), B2 = __builtin_bit_cast(bf8, t2);
                        f16v c = {};
                        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[0], B0, c, 0, 0, 0);
                        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[1], B0, c, 0, 0, 0);
                        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[2], B1, c, 0, 0, 0);
                        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[3], B0, c, 0, 0, 0);
                        acc[g] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[4], B2, c, 0, 0, 0);
                    }
                    if (i > 0) {
                        const int pe = (i - 1) / 2, pg = (i - 1) % 2;
                        const uint32_t both = xq[pg][pe / 2];
                        body(4 * u + pe, pe, pg, __uint_as_float(pe % 2 ? both & 0xffff0000u : both << 16), acc[pg]);
                    }
                }
                after_quad();
            }
            if (k + 1 < steps) put(k + 1);
        }
    };
    // sum over channels of x[c] * window[c]: the channels of a step first, then the steps, with what an addition rounds away
    // carried on (dwv from 64 bits, 2 x 27x29, one head of 64: 1.72e-7 without, 1.52e-7 with it)
    auto contract = [&](int ph, float (&sum)[2][N]) {
        float four[2][N];
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int i = 0; i < N; ++i) { sum[g][i] = 0.0f; four[g][i] = 0.0f; }
        phase(ph, [&](int, int e, int g, float x, const f16v& acc) {
#pragma unroll
            for (int i = 0; i < N; ++i) four[g][i] = fmaf(x, acc[i], four[g][i]);
        }, [&]() {
#pragma unroll
            for (int g = 0; g < 2; ++g)
#pragma unroll
                for (int i = 0; i < N; ++i) {               // what the addition rounds away starts the next four
                    const float t = sum[g][i] + four[g][i];
                    four[g][i] -= t - sum[g][i];
                    sum[g][i] = t;
                }
        });
    };
    auto shift_of = [&](int i) -> int { return 8 * (i / 4) + 4 * h + i % 4; };
    auto both = [](float x, float& other) -> float {        // x of the lower half in both halves, of the upper half
        const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
        other = __uint_as_float(sw[1]);
        return __uint_as_float(sw[0]);
    };

    // where group g's column lies in a and dl (worked out anew where they are stored: kept, it would cost the sums registers)
    auto group_pixel = [&](int g, long& first) -> bool {
        int n = wave * 64 + 32 * g + col, db, ti, tj;
        asm volatile("" : "+v"(n));
        const bool there = pixel(n, db, ti, tj);
        first = ((long)(b0 + db) * (a.C / d) + m) * HW * S + (long)ti * W + j0 + tj;
        return there;
    };
    float p[2][N];
    contract(0, p);
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        long first;
        const bool there = group_pixel(g, first);
        float mx = -INFINITY, hi;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int s = shift_of(i);
            p[g][i] = s < S ? fmaf(a.scale, p[g][i], a.bias ? a.bias[m * S + min(s, S - 1)] : 0.0f) : -INFINITY;
            mx = fmaxf(mx, p[g][i]);
        }
        const float lo = both(mx, hi);
        mx = fmaxf(lo, hi);
        float den = 0.0f;
#pragma unroll
        for (int i = 0; i < N; ++i) { p[g][i] = expf(p[g][i] - mx); den += p[g][i]; }
        const float dlo = both(den, hi);
        den = dlo + hi;
        const float inv = 1.0f / den;
#pragma unroll
        for (int i = 0; i < N; ++i) {                       // p / den: the reciprocal's own rounding is taken out again
            const float e = p[g][i];
            p[g][i] = e * inv;
            p[g][i] = fmaf(fmaf(-p[g][i], den, e), inv, p[g][i]);
            if (there && shift_of(i) < S) a.a_ws[first + (long)shift_of(i) * HW] = p[g][i];
        }
    }
    float da[2][N];
    contract(1, da);
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        // (p waits in a_ws while da is summed: the sums need the registers)
        long first;
        const bool there = group_pixel(g, first);
        float dsum = 0.0f, hi;
#pragma unroll
        for (int i = 0; i < N; ++i) p[g][i] = shift_of(i) < S ? a.a_ws[first + (long)min(shift_of(i), S - 1) * HW] : 0.0f;
#pragma unroll
        for (int i = 0; i < N; ++i) dsum = fmaf(p[g][i], shift_of(i) < S ? da[g][i] : 0.0f, dsum);
        const float lo = both(dsum, hi);
        dsum = lo + hi;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            da[g][i] = shift_of(i) < S ? p[g][i] * (da[g][i] - dsum) : 0.0f;
            if (there && shift_of(i) < S) a.dl_ws[first + (long)shift_of(i) * HW] = da[g][i];
        }
    }
    bf16_bits* ob = a.out + head;
    float o[2], ov[4];
    int c0 = 0;
    phase(2, [&](int, int e, int g, float, const f16v& acc) {
        o[g] = 0.0f;
#pragma unroll
        for (int i = 0; i < N; ++i) o[g] = fmaf(da[g][i], acc[i], o[g]);
        if (g == 0) return;
        // the halves' sums: group 0 in the lower lanes, group 1 in the upper ones, each lane its own pixel
        const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(o[0]), __float_as_uint(o[1]), false, false);
        ov[e] = a.scale * (__uint_as_float(sw[0]) + __uint_as_float(sw[1]));
    }, [&]() {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (live && c0 + e < d) *(bf16_bits*)((char*)(ob + (long)(c0 + e) * HW) + own) = f32_to_bf16(ov[e]);
        c0 += 4;
    });
}

// ---- key and value gradients
//   dk[c,y] = scale * sum_t q[c, y - off(t)] * sum_s wk[c,s,t] dl[s, y - off(t)]
//   dv[c,y] =         sum_t dO[c, y - off(t)] * sum_s wv[c,s,t] a[s, y - off(t)]
struct DkdvArgs {
    const u4* image;                                        // [side][head][ncb][KV_IMG]
    const float* p[2];                                      // dl, a: [B, heads, S, H, W]
    const unsigned char* xt[2];
    bf16_bits* out[2];                                      // dk, dv
    float f[2];                                             // logit scale, 1
    int H, W, C, d, heads, ncb;
    int rows;                                               // of a band
    long columns, groups, jobs;                             // of all items; column groups of 32; groups * bands
};
constexpr int KV_WAVES = 8, KV_NT = 64 * KV_WAVES;

// A block keeps the left operands of 32 channels of one head and side in LDS (125 KB); its waves are on their own.  A wave walks
// down a band of rows of 32 columns (a column of any item to a lane: every matrix column is used whatever the map's
// width).  For each source row and column of the taps it loads the lanes' dl (or a) and q (or dO) at that column once, from
// memory or cache, and forms the sums over the shifts for the five rows of the taps, 32 channels by 32 pixels by 160 slots in
// ten instructions each, which are multiplied with q and added to the five target rows that the source row reaches.
// MI355X, B=64, 28x28, C=128, 4 heads: 330 us with 4x4x1 float32 matrix instructions, 137 like this; 87 with two halves of
// scaled numbers, five instructions, and records of them that the per-pixel kernel wrote in 10 us, which lose small numbers
// beside large ones.  The matrix cores are busy for 45 % of the time, the vector unit for 50 %, and the two hardly overlap: a wave's
// ten instructions are a chain.  Tried: splitting the next source between the matrix instructions of the last two chains
// (159 us: copies and spills), of the last chain (118 spills).
__global__ void __launch_bounds__(KV_NT, 2)
dkdv_split_kernel(const DkdvArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, h = lane >> 5;
    const int H = a.H, W = a.W, m = blockIdx.z, side = blockIdx.y & 1, cb = blockIdx.y >> 1;
    const long HW = (long)H * W;
    const u4* image = a.image + ((long)(side * a.heads + m) * a.ncb + cb) * KV_IMG;
    for (int i = wave; i < S * KV_MM; i += KV_WAVES) load_to_lds(image + i * 64, lane * 16u, lds_offset(smem) + i * 1024u);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();

    const u4* const wl = (const u4*)smem + lane;
    const int xt_px = a.ncb * 64;
    for (long job = (long)blockIdx.x * KV_WAVES + wave; job < a.jobs; job += (long)gridDim.x * KV_WAVES) {
        const long band = job / a.groups, n_ = (job - band * a.groups) * 32 + col;
        const int y0 = (int)band * a.rows, y1 = min(H, y0 + a.rows);
        const bool live = n_ < a.columns;
        const long n = live ? n_ : a.columns - 1, b = n / W;
        const int x = (int)(n - b * W);
        const long plane = b * a.heads + m;
        const float* const given = a.p[side] + (plane * S + 4 * h) * HW + x;    // of shift 4 h on
        const unsigned char* const xt = a.xt[side] + (plane * HW + x) * xt_px + cb * 64 + 32 * h;

        // dl (or a) and q (or dO) of source row y, tap column cc
        struct Source { float p[N]; u4 x0, x1; };
        auto fetch = [&](int y, int cc) -> Source {
            const int xs = x + R - cc, at = min(max(y, 0), H - 1) * W + min(max(xs, 0), W - 1) - x;
            const float* p = given + at;
            const unsigned char* t = xt + (long)at * xt_px;
            Source s;
#pragma unroll
            for (int i = 0; i < N - 1; ++i) s.p[i] = p[(8 * (i / 4) + i % 4) * HW];
            s.p[N - 1] = p[(S - 1 - 4 * h) * HW];
            s.x0 = *(const u4*)t; s.x1 = *(const u4*)(t + 16);
            return s;
        };
        float acc[KS][16];
#pragma unroll
        for (int p = 0; p < KS; ++p)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[p][i] = 0.0f;
        Source src[2];
        bf8 A[2][KV_MM];
        src[0] = fetch(y0 - R, 0);
#pragma unroll
        for (int j = 0; j < KV_MM; ++j) A[0][j] = __builtin_bit_cast(bf8, wl[j * 64]);
#pragma unroll 1
        for (int ys = y0 - R; ys < y1 + R; ++ys) {
            const int lo = ys < 0 || ys >= H ? KS : max(0, y0 - ys + R), hi = min(KS - 1, y1 - 1 - ys + R);      // rows of the taps that reach the band
#pragma unroll
            for (int cc = 0; cc < KS; ++cc) {
                src[(cc + 1) & 1] = cc + 1 < KS ? fetch(ys, cc + 1) : fetch(ys + 1, 0);
                const Source& s = src[cc & 1];
                const int xs = x + R - cc;
                const bool in = xs >= 0 && xs < W;          // columns outside the map add nothing, whatever the record says
                float xv[16];
#pragma unroll
                for (int w = 0; w < 8; ++w) {
                    const uint32_t v = in ? (w < 4 ? s.x0[w] : s.x1[w - 4]) : 0u;
                    xv[2 * w] = __uint_as_float(v << 16);
                    xv[2 * w + 1] = __uint_as_float(v & 0xffff0000u);
                }
                float v[N];
#pragma unroll
                for (int i = 0; i < N; ++i) v[i] = in ? s.p[i] : 0.0f;
                uint32_t t[(N + 1) / 2][3];
#pragma unroll
                for (int i = 0; i < N / 2; ++i) split3_pair(v[2 * i], v[2 * i + 1], t[i]);
                split3_pair(v[N - 1], v[N - 1], t[N / 2]);
                const uint32_t l12 = __builtin_amdgcn_perm(t[6][1], t[6][0], h ? 0x01000504u : 0x05040100u);    // second first, first second
                const uint32_t l31 = h ? 0u : __builtin_amdgcn_perm(t[6][2], t[6][0], 0x01000504u);             // first third
                auto quad = [&](int e0, int e1, int e) { return __builtin_bit_cast(bf8, u4{t[e0][e], t[e0 + 1][e], t[e1][e], t[e1 + 1][e]}); };
                const bf8 A1 = quad(0, 2, 0), A2 = quad(0, 2, 1), A3 = quad(0, 2, 2), B1 = quad(4, 4, 0), B2 = quad(4, 4, 1), B3 = quad(4, 4, 2);
                const bf8 B1L = __builtin_bit_cast(bf8, u4{t[4][0], t[5][0], l12, l31});
#pragma unroll
                for (int p = 0; p < KS; ++p) {
                    constexpr int LAST = S - 1;
                    const int idx = cc * KS + p, next = idx < LAST ? idx + 1 : 0;
#pragma unroll
                    for (int j = 0; j < KV_MM; ++j) A[(idx + 1) & 1][j] = __builtin_bit_cast(bf8, wl[(next * KV_MM + j) * 64]);
                    __builtin_amdgcn_sched_barrier(0);      // (the next chain's operands are on their way, and no others)
                    if (p < lo || p > hi) continue;
                    // small products first
                    const bf8 (&w)[KV_MM] = A[idx & 1];
                    f16v c = {};
                    auto mul = [&](const bf8& kernels, const bf8& given) { c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kernels, given, c, 0, 0, 0); };
                    mul(w[2], A1); mul(w[0], A3); mul(w[1], A2); mul(w[3], B3);
                    mul(w[1], A1); mul(w[0], A2); mul(w[3], B2);
                    mul(w[4], B1L); mul(w[3], B1); mul(w[0], A1);
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[p][i] = fmaf(c[i], xv[i], acc[p][i]);
                    __builtin_amdgcn_sched_barrier(0);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            src[0] = src[1];
#pragma unroll
            for (int j = 0; j < KV_MM; ++j) A[0][j] = A[1][j];
            // target row ys - 2 is complete
            if (ys >= y0 + R && live) {
                bf16_bits* o = a.out[side] + (b * a.C + (long)m * a.d + cb * 32 + 4 * h) * HW + (long)(ys - R) * W + x;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int c = 8 * (i / 4) + i % 4;
                    if (cb * 32 + 4 * h + c < a.d) o[(long)c * HW] = f32_to_bf16(acc[0][i] * a.f[side]);
                }
            }
#pragma unroll
            for (int p = 0; p < KS; ++p)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[p][i] = p + 1 < KS ? acc[p + 1][i] : 0.0f;
        }
    }
}

}  // namespace split

bool split_supported(const Problem& p) { return p.dtype == 1 && p.ksize == 5 && !p.no_split; }

// what the kernels keep in the workspace behind a, dl and the partial sums
struct SplitLayout { size_t px, kv, xt[2], bytes; int ncb; };
static SplitLayout split_layout(const Problem& p)
{
    using namespace split;
    SplitLayout l;
    l.ncb = (p.d() + 31) / 32;
    const size_t pixels = (size_t)p.B * p.heads * p.plane();
    size_t at = 0;
    auto take = [&](size_t bytes) { const size_t o = at; at += (bytes + 255) & ~(size_t)255; return o; };
    l.px = take((size_t)2 * p.heads * ((p.d() + 3) & ~3) * PX_CH * 16);
    l.kv = take((size_t)2 * p.heads * l.ncb * KV_IMG * 16);
    for (size_t& x : l.xt) x = take(pixels * l.ncb * 64);
    l.bytes = at;
    return l;
}
size_t split_workspace_bytes(const Problem& p) { return split_supported(p) ? split_layout(p).bytes : 0; }

hipError_t launch_split_prep(const Problem& p, const float* wk, const float* wv, void* ws, hipStream_t st)
{
    using namespace split;
    const SplitLayout l = split_layout(p);
    char* base = (char*)ws;
    hipLaunchKernelGGL(prep_split_kernel, dim3((unsigned)(p.heads * l.ncb * 32), 2), dim3(PX_CH), 0, st, wk, wv, (u4*)(base + l.px),
                       (u4*)(base + l.kv), p.d(), l.ncb, p.two_branch ? 1.0f : 0.0f);
    return hipGetLastError();
}

hipError_t launch_bwd_pixel_split(const Problem& p, const void* dout, const void* q, const void* k, const void* v,
                                  const float* bias, void* dq, float* a_ws, float* dl_ws, void* ws, hipStream_t st)
{
    using namespace split;
    const SplitLayout l = split_layout(p);
    unsigned char* base = (unsigned char*)ws;
    PixelArgs a{};
    a.q = (const bf16_bits*)q; a.k = (const bf16_bits*)k; a.v = (const bf16_bits*)v; a.dout = (const bf16_bits*)dout;
    a.wk = (const u4*)(base + l.px); a.wv = a.wk + (size_t)p.heads * ((p.d() + 3) & ~3) * PX_CH;
    a.bias = bias; a.out = (bf16_bits*)dq; a.a_ws = a_ws; a.dl_ws = dl_ws;
    for (int i = 0; i < 2; ++i) a.xt[i] = base + l.xt[i];
    a.H = p.H; a.W = p.W; a.C = p.C; a.d = p.d();
    a.scale = p.logit_scale();
    const int planes = stack_planes(p.B, p.H, p.W, p.C);
    a.cut = plan_stack(planes, p.H, p.W);
    const auto kernel = p.plane() == 1 ? pixel_split_kernel<true> : pixel_split_kernel<false>;
    static LdsOptIn opt_in;
    hipError_t e = opt_in.ensure({(const void*)pixel_split_kernel<true>, (const void*)pixel_split_kernel<false>}, (int)CU_LDS_BYTES);
    if (e != hipSuccess) return e;
    const size_t lds = 2 * ((size_t)a.cut.npx + 4 * PX_CH) * 16;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(a.cut.ns * a.cut.runs), (unsigned)p.heads, (unsigned)(p.B / planes)), dim3(NT), lds, st, a);
    return hipGetLastError();
}

hipError_t launch_bwd_dkdv_split(const Problem& p, const float* a_ws, const float* dl_ws, const void* ws, void* dk, void* dv, hipStream_t st)
{
    using namespace split;
    const SplitLayout l = split_layout(p);
    const unsigned char* base = (const unsigned char*)ws;
    DkdvArgs a{};
    a.image = (const u4*)(base + l.kv);
    a.p[0] = dl_ws; a.p[1] = a_ws;
    for (int i = 0; i < 2; ++i) a.xt[i] = base + l.xt[i];
    a.out[0] = (bf16_bits*)dk; a.out[1] = (bf16_bits*)dv;
    a.f[0] = p.logit_scale(); a.f[1] = 1.0f;
    a.H = p.H; a.W = p.W; a.C = p.C; a.d = p.d(); a.heads = p.heads; a.ncb = l.ncb;
    a.columns = (long)p.B * p.W;
    const Bands t = plan_bands(p.B, p.H, p.W, 2 * p.heads * l.ncb);
    a.rows = t.rows; a.groups = t.groups; a.jobs = t.jobs;
    static LdsOptIn opt_in;
    hipError_t e = opt_in.ensure({(const void*)dkdv_split_kernel}, (int)CU_LDS_BYTES);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(dkdv_split_kernel, dim3((unsigned)t.blocks, (unsigned)(2 * l.ncb), (unsigned)p.heads), dim3(KV_NT), KV_IMG * 16, st, a);
    return hipGetLastError();
}

}  // namespace slide
