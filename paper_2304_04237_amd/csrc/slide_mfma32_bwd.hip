// Float32 key, value, kernel and bias gradients on the matrix cores of gfx950, windows of 3 and 5:
// every head size, width and element type; products, sums and results in float32 like the
// general kernels of slide_generic.hip.  Both kernels are bound by the learned-kernel contraction and
// run it as outer products of four weights with 64 lanes (slide_mfma32.hip says how).
#include "slide_mfma32.h"

namespace slide {
namespace m32 {

// ---- key and value gradients
//   dk[c,y] = scale * sum_t q[c, y - off(t)] * sum_s wk[c,s,t] dl[s, y - off(t)]
//   dv[c,y] =         sum_t dO[c, y - off(t)] * sum_s wv[c,s,t] a[s, y - off(t)]
struct DkdvArgs {
    const void* x[2];           // q, dO
    const float* w[2];          // wk, wv
    const float* p[2];          // dl, a: [B, heads, S, H, W]
    void* out[2];               // dk, dv
    float f[2];                 // logit scale, 1
    int H, W, C, d;
    float idw;
    Cut cut;
};

// One run of PX = 64 * PG pixels of one head and side: waves = PG pixel groups x CG channel groups.
// A lane is a pixel y; for one tap after the other it holds the S values of a (or dl) at
// y - off(t), and the matrix cores form the sums over s for four channels at a time (rows = channels,
// K = s: no padding), which are then multiplied with the four channels of dO (or q) at y - off(t).
// LDS holds a (or dl) of the run's rows and halo as [pixel][s], NQ quads of channels of dO (or q) as
// [quad][pixel][4] and their kernels.  A tap costs S 4-byte LDS reads per lane whatever the number of
// quads, so NQ is as large as two blocks per compute unit allow.  MI355X, against one thread per
// pixel (slide_generic.hip): float32, 3x3, B=32, 56x56, C=64, 2 heads: 846 -> 53 us.
template <typename T> struct Quad;
template <> struct Quad<float> {
    typedef f4 Raw;
    static __device__ __forceinline__ Raw load(const float* b, long o, long sc, int c, int d)
    {
        Raw r;
#pragma unroll
        for (int u = 0; u < 4; ++u) r[u] = b[o + (long)min(c + u, d - 1) * sc];
        return r;
    }
    static __device__ __forceinline__ Raw pack(const float (&e)[4]) { return f4{e[0], e[1], e[2], e[3]}; }
    static __device__ __forceinline__ Raw first(Raw r, int n)          // zeros past the first n elements
    {
#pragma unroll
        for (int u = 1; u < 4; ++u) r[u] = u < n ? r[u] : 0.0f;
        return r;
    }
    static __device__ __forceinline__ f4 value(Raw r) { return r; }
    static __device__ __forceinline__ Raw zero() { return f4{0.0f, 0.0f, 0.0f, 0.0f}; }
};
template <> struct Quad<bf16_bits> {
    typedef uint32_t Raw __attribute__((ext_vector_type(2)));
    static __device__ __forceinline__ Raw load(const bf16_bits* b, long o, long sc, int c, int d)
    {
        bf16_bits e[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) e[u] = b[o + (long)min(c + u, d - 1) * sc];
        return pack(e);
    }
    static __device__ __forceinline__ Raw pack(const bf16_bits (&e)[4])
    {
        return Raw{e[0] | ((uint32_t)e[1] << 16), e[2] | ((uint32_t)e[3] << 16)};
    }
    static __device__ __forceinline__ Raw first(Raw r, int n)
    {
        return Raw{n > 1 ? r[0] : r[0] & 0xffffu, n > 3 ? r[1] : (n > 2 ? r[1] & 0xffffu : 0u)};
    }
    static __device__ __forceinline__ f4 value(Raw r)
    {
        return f4{__uint_as_float(r[0] << 16), __uint_as_float(r[0] & 0xffff0000u),
                  __uint_as_float(r[1] << 16), __uint_as_float(r[1] & 0xffff0000u)};
    }
    static __device__ __forceinline__ Raw zero() { return Raw{0u, 0u}; }
};

template <typename T, int KS, int PG, int CG, int NQ>
__global__ void __launch_bounds__(64 * PG * CG, 2)
dkdv32_kernel(const DkdvArgs a)
{
    using D = Dim<KS>;
    using Raw = typename Quad<T>::Raw;
    constexpr int S = D::S, R = D::R;
    constexpr int NT = 64 * PG * CG, PX = 64 * PG;
    constexpr int NW = NQ / CG;                             // quads per wave
    constexpr int WR = (4 * S + 63) / 64;                   // operand registers of one quad and tap
    static_assert(NQ % CG == 0, "");

    extern __shared__ __align__(16) float smem_raw[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int pg = wave % PG, cg = wave / PG;
    const int H = a.H, W = a.W, d = a.d;
    const int m = blockIdx.y, side = blockIdx.x & 1, b = blockIdx.z;
    const long HW = (long)H * W;
    const int strip = (blockIdx.x >> 1) / a.cut.runs, run = (blockIdx.x >> 1) - strip * a.cut.runs;
    int j0, tw;
    strip_of(a.cut, strip, j0, tw);
    const int n0 = run * PX;
    if (n0 >= H * tw) return;
    const int npx = a.cut.npx, RP = a.cut.RP;
    const int row0 = n0 / tw - R;
    Raw* xl = (Raw*)smem_raw;                               // [NQ][npx]
    float* pl = (float*)(xl + NQ * npx);                    // [npx][S]: S is odd, lanes read without conflicts and a tap's S values are one address
    float* wl = pl + S * npx;                               // [NQ][QUAD_W]

    const int n = n0 + pg * 64 + lane;
    const bool live = n < H * tw;
    const int nn = live ? n : H * tw - 1;
    const int ti = nn / tw, tj = nn - ti * tw;
    const long pix = (long)ti * W + j0 + tj;
    const int at = (ti - row0) * RP + tj + R;               // its own place in a tile plane
    const long item = ((long)b * a.C + (long)m * d) * HW;
    const T* xb = (const T*)a.x[side] + item;
    const float* pb = a.p[side] + ((long)b * (a.C / d) + m) * S * HW;
    const float* wb = a.w[side] + (long)m * d * S * S;
    T* ob = (T*)a.out[side] + item + pix;
    const float f = a.f[side];

    auto tile_pixel = [&](int e, bool& in) -> long {
        const int rr = e / RP, xx = e - rr * RP;
        const int y = row0 + rr, x = j0 + xx - R;
        in = y >= 0 && y < H && x >= 0 && x < W;
        return in ? (long)y * W + x : 0;
    };
    int woff[WR];                                           // lane l: channel l & 3, shift l >> 2
#pragma unroll
    for (int j = 0; j < WR; ++j) {
        const int l = min(j * 64 + lane, 4 * S - 1);
        woff[j] = (l & 3) * (S * S) + (l >> 2) * S;
    }
    const bool wave_live = n0 + pg * 64 < H * tw;           // (the last run's waves past the strip only stage)

    // the quads and kernels of a step, fetched while the step before is multiplied
    constexpr int NI = 2;                                   // pixels per thread fetched ahead
    constexpr int NWT = (NQ * D::QUAD_W + NT - 1) / NT;     // weights per thread
    constexpr bool AHEAD_W = NWT <= 24;
    bool in[NI]; long off[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        off[i] = tile_pixel(min(tid + i * NT, npx - 1), in[i]);
    }
    Raw xr[NI][NQ];
    float wr[AHEAD_W ? NWT : 1];
    auto fetch = [&](int c0) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int u = 0; u < NQ; ++u) xr[i][u] = Quad<T>::load(xb, off[i], HW, c0 + 4 * u, d);
        if (AHEAD_W)
#pragma unroll
            for (int u = 0; u < NWT; ++u) {
                const int idx = tid + u * NT;
                wr[u] = (idx < NQ * D::QUAD_W && c0 * S * S + idx < d * S * S) ? wb[(long)c0 * S * S + idx] : 0.0f;
            }
    };
    fetch(0);
    for (int e = tid; e < npx; e += NT) {
        bool ok;
        const long o = tile_pixel(e, ok);
        float v[S];
#pragma unroll
        for (int s = 0; s < S; ++s) v[s] = pb[(long)s * HW + o];
#pragma unroll
        for (int s = 0; s < S; ++s) pl[e * S + s] = ok ? v[s] : 0.0f;
    }

    for (int c0 = 0; c0 < d; c0 += 4 * NQ) {
        if (c0 > 0) __syncthreads();                        // the step before is no longer read
#pragma unroll
        for (int i = 0; i < NI; ++i)
            if (tid + i * NT < npx)
#pragma unroll
                for (int u = 0; u < NQ; ++u) xl[u * npx + tid + i * NT] = in[i] ? xr[i][u] : Quad<T>::zero();
        for (int e = tid + NI * NT; e < npx; e += NT) {     // (maps of a few columns, wide windows)
            bool ok;
            const long o = tile_pixel(e, ok);
#pragma unroll
            for (int u = 0; u < NQ; ++u) xl[u * npx + e] = ok ? Quad<T>::load(xb, o, HW, c0 + 4 * u, d) : Quad<T>::zero();
        }
        if (AHEAD_W) {
#pragma unroll
            for (int u = 0; u < NWT; ++u)
                if (tid + u * NT < NQ * D::QUAD_W) wl[tid + u * NT] = wr[u];
        } else {
#pragma unroll 4
            for (int idx = tid; idx < NQ * D::QUAD_W; idx += NT)
                wl[idx] = c0 * S * S + idx < d * S * S ? wb[(long)c0 * S * S + idx] : 0.0f;
        }
        if (a.idw != 0.0f) {                                // the fixed shift path of the two-branch form: shift t reads tap t
            __syncthreads();
            for (int i = tid; i < min(NQ * 4, d - c0) * S; i += NT) wl[(i / S) * (S * S) + (i % S) * (S + 1)] += a.idw;
        }
        __syncthreads();
        if (c0 + 4 * NQ < d) fetch(c0 + 4 * NQ);
        if (!wave_live) continue;

        f4 acc[NW];
#pragma unroll
        for (int u = 0; u < NW; ++u) acc[u] = f4{0.0f, 0.0f, 0.0f, 0.0f};
        float p[S], pn[S];
        int src = at + R * RP + R;                          // y - off(0)
#pragma unroll
        for (int s = 0; s < S; ++s) p[s] = pl[src * S + s];
#pragma unroll 1
        for (int t = 0; t < S; ++t) {
            const int next = t + 1 < S ? (((t + 1) % KS) ? src - 1 : src - RP + (KS - 1)) : src;
#pragma unroll
            for (int s = 0; s < S; ++s) pn[s] = pl[next * S + s];
#pragma unroll
            for (int u = 0; u < NW; ++u) {
                const int qd = cg + u * CG;
                float wv[WR];
#pragma unroll
                for (int j = 0; j < WR; ++j) wv[j] = wl[qd * D::QUAD_W + woff[j] + t];
                const f4 x = Quad<T>::value(xl[qd * npx + src]);
                f4 ck = {0.0f, 0.0f, 0.0f, 0.0f};
                unroll<S>([&](auto sc) {
                    constexpr int s = decltype(sc)::value;
                    ck = outer<s % 16>(wv[s / 16], p[s], ck);
                });
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[u][e] = fmaf(ck[e], x[e], acc[u][e]);
            }
            src = next;
#pragma unroll
            for (int s = 0; s < S; ++s) p[s] = pn[s];
        }
        if (live) {
#pragma unroll
            for (int u = 0; u < NW; ++u)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int c = c0 + 4 * (cg + u * CG) + e;
                    if (c < d) Elem<T>::store(ob + (long)c * HW, f * acc[u][e]);
                }
        }
    }
}

template <typename T, int KS, bool FEW>
static hipError_t launch_dkdv(const Problem& p, DkdvArgs& a, hipStream_t st)
{
    constexpr Block b = dkdv_block(KS, sizeof(T), FEW);
    constexpr auto kernel = dkdv32_kernel<T, KS, b.PG, b.CG, b.NQ>;
    a.cut = plan_cut(p.H, p.W, KS, b);
    static LdsOptIn opt_in;
    hipError_t e = opt_in.ensure({(const void*)kernel}, (int)CU_LDS_BYTES);
    if (e != hipSuccess) return e;
    const dim3 grid((unsigned)(2 * a.cut.ns * a.cut.runs), (unsigned)p.heads, (unsigned)p.B);
    hipLaunchKernelGGL(kernel, grid, dim3(64 * b.PG * b.CG), dkdv_lds(a.cut, KS, sizeof(T), b), st, a);
    return hipGetLastError();
}
template <typename T, int KS>
static hipError_t launch_dkdv_t(const Problem& p, DkdvArgs& a, hipStream_t st)
{
    if (dkdv_few(p.B, p.heads, p.H, p.W, KS, sizeof(T))) return launch_dkdv<T, KS, true>(p, a, st);
    return launch_dkdv<T, KS, false>(p, a, st);
}

// ---- kernel and bias gradients
//   dwk[c,s,t] = scale * sum over items and pixels y of dl[s,y] * q[c,y] * k[c, y + off(t)]
//   dwv[c,s,t] =                                        a[s,y] * dO[c,y] * v[c, y + off(t)]
//   dbias[s]   =                                       dl[s,y]
struct DwArgs {
    const void* y[2]; const void* x[2];     // k, v; q, dO
    const float* p[2];                      // dl, a: [B, heads, S, H, W]
    float* partial;                         // [chunks][2][C][S][S]
    float* bias_partial;                    // [chunks][heads][S]
    float f[2];
    int H, W, C, d, heads;
    int TR, TC, ntr, ntc;                   // tiles of TR rows and TC columns
    long items;                             // batch
    long tiles;                             // all of them, over the batch
    int chunks;
    int KST, QST;                           // floats per channel of the y and x tiles in LDS
    int group;                              // quads of a walker between two additions to its totals
};

// pixels x..x+3 of row y, zeros outside the map and where !ok, by one load from wherever the row
// starts (the hardware takes any element's address); VEC: W % 4 == 0, a quad is whole.  Otherwise the last
// quad of a row reads into the next one, except within four elements of the tensor's end (`left`:
// elements from base to there), where its elements are loaded one by one; cut() clears what is past
// the row, apart from the load so that nothing waits for it before it is needed (training step, bf16, 3x3,
// 1 x 200x333, C=96: 183 us with an element per load, 201 with the cut at the load, 178).
template <typename T, bool VEC> struct Row4 {
    using Raw = typename Quad<T>::Raw;
    typedef Raw RawAny __attribute__((aligned(sizeof(T))));
    static __device__ __forceinline__ Raw load(const T* base, int y, int x, int W, bool ok, long left)
    {
        if (!ok) return Quad<T>::zero();
        const T* p = base + (long)y * W + x;
        if (VEC) return *(const RawAny*)p;
        if ((long)y * W + x + 4 <= left) return *(const RawAny*)p;
        T e[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) e[u] = x + u < W ? p[u] : T(0);
        return Quad<T>::pack(e);
    }
    static __device__ __forceinline__ f4 cut(Raw r, int x, int W) { return Quad<T>::value(VEC ? r : Quad<T>::first(r, W - x)); }
};

// One block sums 32 channels of a head and one side over its chunk of tiles.  A lane is a channel, its
// half of the wave one of two walkers over the tile's quads of four pixels; per pixel the products
// x * y of the taps are formed once and the matrix cores multiply them with S - 1 shifts' dl (or a),
// four rows at a time, broadcast inside a half (cbsz = 3); the last shift is a vector
// multiply-add.  The S^2 sums of a channel stay in registers: all 81 of a 3x3 window in each of four waves,
// which share the pixels; with a 5x5 window a wave holds three taps and eight waves see the same pixels (tap
// 24 is dealt out by blocks of four shifts).
// A running sum over a whole chunk would round with every pixel, so a walker's sums start at zero every few quads
// (a.group; the first products need no accumulator, so that is free) and are added to totals, two values to a
// register: the halves of the wave are summed on the way, the lower lanes keep one value, the upper ones the
// next.  The totals take the registers that tiles of eight rows and, at 5x5, six taps per wave had.  A vector
// instruction costs 5.6 cycles between the matrix instructions (by the counters), which is why the quad's
// addresses are 24-bit arithmetic and only the waves that sum dbias do so.  MI355X, against one block per channel and shift
// (slide_generic.hip) and a launch of its own for dbias: float32, 3x3, B=32, 56x56, C=64, 2 heads: 598 -> 61 us; bf16, 3x3,
// B=128, 28x28, C=128, 4 heads: 1854 -> 94 us.  With running sums over the chunk they took 62 and 88 us.  Error of dwv against 64 bits (2-norm, two-branch; those kernels,
// the running sums, these): 3x3 float32 as above 1.91, 2.47, 1.61e-7; 5x5 as above in float32 2.56, 4.11, 2.26e-7.
template <typename T, int KS, bool VEC>
__global__ void __launch_bounds__(dw_threads(KS), 2)
dw32_kernel(const DwArgs a)
{
    using D = Dim<KS>;
    constexpr int S = D::S, SM = D::SM, SB = D::SB, R = D::R;
    constexpr int NT = dw_threads(KS), WAVES = NT / 64;
    constexpr int ROLES = KS == 3 ? 1 : 8, NTAP = KS == 3 ? 9 : 3;
    constexpr bool EXTRA = KS == 5;                         // tap 24: a block of shifts in each of waves 0..5, the last shift in wave 6
    constexpr int WALK = 2 * WAVES / ROLES;
    constexpr int AR = 4 * SM / 32;                         // registers of the four pixels' shifts
    constexpr int AQ = 4 * SM + 1;                          // floats per quad in LDS (odd: the quads' writes spread over the banks)
    constexpr int NV = NTAP * S + (EXTRA ? 5 : 0), NP = (NV + 1) / 2;   // a lane's sums, totals

    extern __shared__ __align__(16) float smem_raw[];
    float* const smem = smem_raw;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int role = wave % ROLES, half = lane >> 5, ch = lane & 31;
    const int walker = (wave / ROLES) * 2 + half;
    const int H = a.H, W = a.W, d = a.d, TR = a.TR, TC = a.TC;
    // blocks of one chunk are neighbours: they read the same a (or dl)
    const int m = blockIdx.y, side = blockIdx.x & 1;
    const int ncb = (d + DW_CH - 1) / DW_CH;
    const int chunk = (blockIdx.x >> 1) / ncb, cb = (blockIdx.x >> 1) - chunk * ncb;
    const long HW = (long)H * W;
    const int RS = TC + 2 * R;
    float* yl = smem;                                       // [32][KST]: [TR + 2R][RS]
    float* xl = yl + DW_CH * a.KST;                         // [32][QST]: [TR][TC]
    float* ll = xl + DW_CH * a.QST;                         // last shift [quad][4]; 32 * (KST + QST) is a multiple of 4
    float* zl = ll + TR * TC;                               // [DW_ZEROS] zeros
    float* al = zl + DW_ZEROS;                              // [quad][AQ]: pixel x shift
    const T* yb = (const T*)a.y[side];
    const T* xb = (const T*)a.x[side];
    const float* pb = a.p[side];

    // sums of a group: value v < NTAP * S is shift v % S of tap v / S of this wave, the others are tap 24's
    f4 acc[NTAP][SB], xacc;
    float last[NTAP], xlast = 0.0f;
    float bsum[AR] = {}, blast = 0.0f;
    float total[NP], btotal[AR], bltotal = 0.0f;
#pragma unroll
    for (int j = 0; j < NP; ++j) total[j] = 0.0f;
#pragma unroll
    for (int j = 0; j < AR; ++j) btotal[j] = 0.0f;
    const bool sums_bias = side == 0 && cb == 0 && role == 0 && a.bias_partial;
    const int y_at = ch * a.KST, x_at = DW_CH * a.KST + ch * a.QST, l_at = (int)(ll - smem), zero_at = (int)(zl - smem), a_at = (int)(al - smem);
    int toff[NTAP];
#pragma unroll
    for (int i = 0; i < NTAP; ++i) {
        const int t = role * NTAP + i;
        toff[i] = (t / KS) * RS + t % KS;
    }
    auto add_group = [&]() {
        unroll<NP>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            auto value = [&](auto vc) -> float {
                constexpr int v = decltype(vc)::value;
                if constexpr (v < NTAP * S) {
                    if constexpr (v % S < SM) return acc[v / S][v % S / 4][v % S % 4];
                    else return last[v / S];
                } else if constexpr (v < NTAP * S + 4 && v < NV) return xacc[v - NTAP * S];
                else if constexpr (v < NV) return xlast;
                else return 0.0f;
            };
            const auto swapped = __builtin_amdgcn_permlane32_swap(__float_as_uint(value(std::integral_constant<int, 2 * j>{})),
                                                                  __float_as_uint(value(std::integral_constant<int, 2 * j + 1>{})), false, false);
            total[j] += __uint_as_float(swapped[0]) + __uint_as_float(swapped[1]);
        });
        if (sums_bias) {
#pragma unroll
            for (int j = 0; j < AR; ++j) btotal[j] += bsum[j];
            bltotal += blast;
        }
    };

    if (tid < DW_ZEROS) zl[tid] = 0.0f;
    // staging: LN lanes per channel, of which 2^w.lg (>= the tile's quads per row) take a row
    constexpr int LN = NT / DW_CH;
    const int sch = tid / LN, sl = tid % LN;
    const bool sc_live = cb * DW_CH + sch < d;
    const long chan = (long)m * d + min(cb * DW_CH + sch, d - 1);

    // a tile's elements on their way from memory to LDS: fetched while the tile before is multiplied
    constexpr DwLoads LOADS = dw_loads(KS, sizeof(T), VEC);
    constexpr int HL = 2 * R, RPI = LN / HL, HR = (DW_MAX_ROWS + 2 * R + RPI - 1) / RPI;    // halo columns; rows of them per step, steps
    using Raw = typename Quad<T>::Raw;
    Raw yv[LOADS.y], xv[LOADS.x];
    T hv[HR];
    f4 pv[LOADS.p];
    struct Where { long b; int y0, x0, th, tw, qpr, lg; };
    auto locate = [&](long tile) -> Where {
        Where w;
        w.b = tile / (a.ntr * a.ntc);
        const int r = (int)(tile - w.b * (a.ntr * a.ntc));
        const int ty = r / a.ntc, tx = r - ty * a.ntc;
        w.y0 = ty * TR; w.x0 = tx * TC;
        w.th = min(TR, H - w.y0); w.tw = min(TC, W - w.x0);
        w.qpr = (w.tw + 3) >> 2;
        w.lg = dw_row_lanes_log2(w.qpr);
        return w;
    };
    // n / by for n < 1024, by <= 8 (24-bit multiplications: a vector instruction costs 5-6 cycles between the matrix
    // instructions, a 32-bit product four times that)
    auto inverse = [](int by) -> unsigned { return (65536u + by - 1) / by; };
    auto divided = [](int n, unsigned inv) -> int { return (int)(__umul24((unsigned)n, inv) >> 16); };
    auto fetch = [&](const Where& w) {
        const T* yc = yb + (w.b * a.C + chan) * HW;
        const T* xc = xb + (w.b * a.C + chan) * HW;
        const long left = (a.items * a.C - (w.b * a.C + chan)) * HW;
        const int r0 = sl >> w.lg, step = LN >> w.lg, q = sl & ((1 << w.lg) - 1), x = w.x0 + 4 * q;
        const bool col = sc_live && q < w.qpr;
#pragma unroll
        for (int i = 0; i < LOADS.y; ++i) {
            const int rr = r0 + i * step, y = w.y0 + rr - R;
            yv[i] = Row4<T, VEC>::load(yc, y, x, W, col && rr < w.th + 2 * R && y >= 0 && y < H, left);
        }
        // the R columns on each side of the tile's 4 * qpr
#pragma unroll
        for (int i = 0; i < HR; ++i) {
            const int rr = sl / HL + i * RPI, h = sl % HL;
            const int y = w.y0 + rr - R, xx = w.x0 + (h < R ? h - R : 4 * w.qpr + h - R);
            const bool in = sc_live && rr < w.th + 2 * R && y >= 0 && y < H && xx >= 0 && xx < W;
            hv[i] = in ? yc[(long)y * W + xx] : T(0);
        }
#pragma unroll
        for (int i = 0; i < LOADS.x; ++i) xv[i] = Row4<T, VEC>::load(xc, w.y0 + r0 + i * step, x, W, col && r0 + i * step < w.th, left);
        const unsigned ir = inverse(w.th);
#pragma unroll
        for (int i = 0; i < LOADS.p; ++i) {
            const int r = (tid >> w.lg) + i * (NT >> w.lg), sh = divided(r, ir), rr = r - sh * w.th;
            const long plane = (w.b * a.heads + m) * S + min(sh, SM);
            pv[i] = Row4<float, VEC>::load(pb + plane * HW, w.y0 + rr, x, W, sh < S && q < w.qpr, (a.items * a.heads * S - plane) * HW);
        }
    };
    auto put = [&](const Where& w) {
        const int r0 = sl >> w.lg, step = LN >> w.lg, q = sl & ((1 << w.lg) - 1), x = w.x0 + 4 * q;
#pragma unroll
        for (int i = 0; i < HR; ++i) {
            const int rr = sl / HL + i * RPI, h = sl % HL;
            if (rr < w.th + 2 * R) yl[sch * a.KST + rr * RS + (h < R ? h : 4 * w.qpr + h)] = Elem<T>::load(&hv[i]);
        }
        if (q >= w.qpr) return;
#pragma unroll
        for (int i = 0; i < LOADS.y; ++i) {
            const int rr = r0 + i * step;
            if (rr < w.th + 2 * R) {
                float* o = yl + sch * a.KST + rr * RS + R + 4 * q;
                const f4 v = Row4<T, VEC>::cut(yv[i], x, W);
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = v[e];
            }
        }
#pragma unroll
        for (int i = 0; i < LOADS.x; ++i) {
            const int rr = r0 + i * step;
            if (rr < w.th) {
                float* o = xl + sch * a.QST + rr * TC + 4 * q;
                const f4 v = Row4<T, VEC>::cut(xv[i], x, W);
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = v[e];
            }
        }
        const unsigned ir = inverse(w.th);
#pragma unroll
        for (int i = 0; i < LOADS.p; ++i) {
            const int r = (tid >> w.lg) + i * (NT >> w.lg), sh = divided(r, ir), rr = r - sh * w.th;
            if (sh < S) {
                const int qi = rr * w.qpr + q;
                const f4 v = Row4<float, VEC>::cut(pv[i], x, W);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (sh < SM) al[qi * AQ + e * SM + sh] = v[e];
                    else ll[qi * 4 + e] = v[e];
                }
            }
        }
    };

    const long t0 = a.tiles * chunk / a.chunks, t1 = a.tiles * (chunk + 1) / a.chunks;
    Where at{}, next{};
    if (t0 < t1) { next = locate(t0); fetch(next); }
    for (long tile = t0; tile < t1; ++tile) {
        at = next;
        __syncthreads();                                    // the tile before is no longer read
        put(at);
        if (tile + 1 < t1) { next = locate(tile + 1); fetch(next); }
        __syncthreads();
        const int tw = at.tw, qpr = at.qpr, nq = at.th * at.qpr;

        const unsigned iq = inverse(qpr);
        // one quad of each walker; FIRST of a group: the sums start with its products
        auto round = [&](auto first, int q0) {
            constexpr bool FIRST = decltype(first)::value;
            const int qi = min(q0 + walker, nq - 1);
            const bool mine = q0 + walker < nq;
            const int row = divided(qi, iq);
            const int live = VEC ? 4 : mine ? min(4, tw - 4 * (qi - __mul24(row, qpr))) : 0;   // pixels of the quad
            // (products of pixels that are none must be zeros also where a neighbour is infinite: rows that
            // are no whole quads are masked, a walker past the last quad reads zeros, of dl and a too)
            const float* yq = smem + (VEC && !mine ? zero_at : y_at + 4 * qi + __mul24(row, RS - 4 * qpr));
            const float* xq = smem + (VEC && !mine ? zero_at : x_at + 4 * qi + __mul24(row, TC - 4 * qpr));
            const float* aq = smem + (mine ? a_at + __mul24(qi, AQ) : zero_at);
            float A[AR];
#pragma unroll
            for (int j = 0; j < AR; ++j) A[j] = aq[j * 32 + ch];
            const f4 L = *(const f4*)(smem + (mine ? l_at + 4 * qi : zero_at));
            float A2 = 0.0f;                                // lanes 4e..4e+3: pixel e, this wave's four shifts of tap 24
            if (EXTRA) A2 = aq[((ch >> 2) & 3) * SM + min(role * 4, SM - 4) + (ch & 3)];
            if (sums_bias) {
#pragma unroll
                for (int j = 0; j < AR; ++j) bsum[j] = FIRST ? A[j] : bsum[j] + A[j];
                const float l = ch < 4 ? L[ch & 3] : 0.0f;
                blast = FIRST ? l : blast + l;
            }
            float x[4], y[NTAP][4], ye[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = xq[e];
            if (KS == 3) {
                float w[3][6];
#pragma unroll
                for (int r = 0; r < 3; ++r)
#pragma unroll
                    for (int c = 0; c < 6; ++c) w[r][c] = yq[r * RS + c];
#pragma unroll
                for (int i = 0; i < NTAP; ++i)
#pragma unroll
                    for (int e = 0; e < 4; ++e) y[i][e] = w[(i / 3) % 3][i % 3 + e];
            } else {
#pragma unroll
                for (int i = 0; i < NTAP; ++i)
#pragma unroll
                    for (int e = 0; e < 4; ++e) y[i][e] = yq[toff[i] + e];
#pragma unroll
                for (int e = 0; e < 4; ++e) ye[e] = yq[4 * RS + 4 + e];
            }
            // (a vector instruction between two matrix instructions costs the issue of about one more, measured:
            // a pixel's vector work comes first, then its matrix instructions back to back)
            unroll<4>([&](auto ec) {
                constexpr int e = decltype(ec)::value;
                constexpr bool NEW = FIRST && e == 0;
                const f4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
                float g[NTAP], ge = 0.0f;
#pragma unroll
                for (int i = 0; i < NTAP; ++i) {
                    g[i] = x[e] * y[i][e];
                    if (!VEC) g[i] = e < live ? g[i] : 0.0f;
                    last[i] = NEW ? L[e] * g[i] : fmaf(L[e], g[i], last[i]);
                }
                if (EXTRA) {
                    ge = x[e] * ye[e];
                    if (!VEC) ge = e < live ? ge : 0.0f;
                    xlast = NEW ? L[e] * ge : fmaf(L[e], ge, xlast);
                }
                __builtin_amdgcn_sched_barrier(0);
                unroll<NTAP>([&](auto ic) {
                    constexpr int i = decltype(ic)::value;
                    unroll<SB>([&](auto sc) {
                        constexpr int sb = decltype(sc)::value, blk = e * SB + sb;
                        acc[i][sb] = __builtin_amdgcn_mfma_f32_4x4x1f32(A[blk / 8], g[i], NEW ? zero : acc[i][sb], 3, blk % 8, 0);
                    });
                });
                if (EXTRA) xacc = __builtin_amdgcn_mfma_f32_4x4x1f32(A2, ge, NEW ? zero : xacc, 3, e, 0);
                __builtin_amdgcn_sched_barrier(0);
            });
        };
        for (int q0 = 0; q0 < nq;) {
            const int end = min(nq, q0 + a.group * WALK);
            round(std::true_type{}, q0);
            for (q0 += WALK; q0 < end; q0 += WALK) round(std::false_type{}, q0);
            add_group();
        }
    }

    // the waves' totals through LDS [wave][channel][s][t] (5x5: one such array, a wave writes its taps)
    constexpr int NRED = KS == 3 ? WAVES : 1;
    float* red = smem + (KS == 3 ? wave : 0) * DW_CH * S * S + ch * (S * S);
    const float f = a.f[side];
    __syncthreads();
    unroll<NP>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        int at_[2]; bool ok[2];
        for (int h = 0; h < 2; ++h) {
            const int v = 2 * j + h, x = v - NTAP * S;
            if (x < 0) { at_[h] = (v % S) * S + role * NTAP + v / S; ok[h] = true; }
            else if (x < 4) { at_[h] = (role * 4 + x) * S + 24; ok[h] = EXTRA && role < 6; }
            else { at_[h] = SM * S + 24; ok[h] = EXTRA && x == 4 && role == 6; }
        }
        if (half ? ok[1] : ok[0]) red[half ? at_[1] : at_[0]] = total[j];
    });
    __syncthreads();
    const int nch = min(DW_CH, d - cb * DW_CH);
    float* out = a.partial + (((long)chunk * 2 + side) * a.C + (long)m * d + cb * DW_CH) * S * S;
    for (int i = tid; i < nch * S * S; i += NT) {
        float sum[NRED];
#pragma unroll
        for (int w = 0; w < NRED; ++w) sum[w] = smem[w * DW_CH * S * S + i];
#pragma unroll
        for (int w = 1; w < NRED; w *= 2)
#pragma unroll
            for (int c = 0; c + w < NRED; c += 2 * w) sum[c] += sum[c + w];
        out[i] = f * sum[0];
    }

    if (side == 0 && cb == 0 && a.bias_partial) {
        __syncthreads();
        // [wave][half][pixel x shift], then the last shift's four pixels
        constexpr int BW = 4 * SM + 4;
        float* bl = smem + (wave * 2 + half) * BW;
        if (role == 0) {
#pragma unroll
            for (int j = 0; j < AR; ++j) bl[j * 32 + ch] = btotal[j];
            if (ch < 4) bl[4 * SM + ch] = bltotal;
        }
        __syncthreads();
        if (tid < S) {
            float sum = 0.0f;
            for (int w = 0; w < WALK; ++w) {                // (5x5: the waves saw the same pixels)
                float four = 0.0f;
                for (int e = 0; e < 4; ++e) four += smem[w * BW + (tid < SM ? e * SM + tid : 4 * SM + e)];
                sum += four;
            }
            a.bias_partial[((long)chunk * a.heads + m) * S + tid] = sum;
        }
    }
}

template <typename T, int KS, bool VEC>
static hipError_t launch_dw(const Problem& p, const DwArgs& a, const DwPlan& t, hipStream_t st)
{
    static LdsOptIn opt_in;
    hipError_t e = opt_in.ensure({(const void*)dw32_kernel<T, KS, VEC>}, (int)CU_LDS_BYTES);
    if (e != hipSuccess) return e;
    const dim3 grid((unsigned)(2 * t.chunks * ((p.d() + DW_CH - 1) / DW_CH)), (unsigned)p.heads);
    hipLaunchKernelGGL((dw32_kernel<T, KS, VEC>), grid, dim3(dw_threads(KS)), t.lds, st, a);
    return hipGetLastError();
}

}  // namespace m32

size_t bwd_dw_m32_partial_floats(const Problem& p)
{
    if (!m32_supported(p)) return 0;
    const m32::DwPlan t = m32::plan_dw(p.B, p.H, p.W, p.C, p.heads, p.ksize, p.dtype == 0 ? 4 : 2);
    return (size_t)t.chunks * (2 * (size_t)p.C * p.S() * p.S() + (size_t)p.heads * p.S());
}

hipError_t launch_bwd_dkdv_m32(const Problem& p, const void* dout, const void* q, const float* wk, const float* wv,
                               const float* attn_ws, const float* dl_ws, void* dk, void* dv, hipStream_t st)
{
    m32::DkdvArgs a{};
    a.x[0] = q; a.x[1] = dout; a.w[0] = wk; a.w[1] = wv; a.p[0] = dl_ws; a.p[1] = attn_ws;
    a.out[0] = dk; a.out[1] = dv; a.f[0] = p.logit_scale(); a.f[1] = 1.0f;
    a.H = p.H; a.W = p.W; a.C = p.C; a.d = p.d();
    a.idw = p.two_branch ? 1.0f : 0.0f;
    if (p.dtype == 0)
        return p.ksize == 3 ? m32::launch_dkdv_t<float, 3>(p, a, st) : m32::launch_dkdv_t<float, 5>(p, a, st);
    return p.ksize == 3 ? m32::launch_dkdv_t<bf16_bits, 3>(p, a, st) : m32::launch_dkdv_t<bf16_bits, 5>(p, a, st);
}

hipError_t launch_bwd_dw_m32(const Problem& p, const void* dout, const void* q, const void* k, const void* v,
                             const float* attn_ws, const float* dl_ws, float* partial, float* dwk, float* dwv,
                             float* dbias, hipStream_t st)
{
    const m32::DwPlan t = m32::plan_dw(p.B, p.H, p.W, p.C, p.heads, p.ksize, p.dtype == 0 ? 4 : 2);
    const long side = (long)p.C * p.S() * p.S();
    m32::DwArgs a{};
    a.y[0] = k; a.y[1] = v; a.x[0] = q; a.x[1] = dout; a.p[0] = dl_ws; a.p[1] = attn_ws;
    a.partial = partial;
    a.bias_partial = dbias ? partial + (size_t)t.chunks * 2 * side : nullptr;
    a.f[0] = p.logit_scale(); a.f[1] = 1.0f;
    a.H = p.H; a.W = p.W; a.C = p.C; a.d = p.d(); a.heads = p.heads;
    a.TR = t.TR; a.TC = t.TC; a.ntr = t.ntr; a.ntc = t.ntc; a.items = p.B; a.tiles = t.tiles; a.chunks = t.chunks;
    a.KST = t.KST; a.QST = t.QST; a.group = t.group;
    const bool vec = p.W % 4 == 0;
    hipError_t e;
#define SLIDE_DW(T, KS) (vec ? m32::launch_dw<T, KS, true>(p, a, t, st) : m32::launch_dw<T, KS, false>(p, a, t, st))
    if (p.dtype == 0) e = p.ksize == 3 ? SLIDE_DW(float, 3) : SLIDE_DW(float, 5);
    else              e = p.ksize == 3 ? SLIDE_DW(bf16_bits, 3) : SLIDE_DW(bf16_bits, 5);
#undef SLIDE_DW
    if (e != hipSuccess) return e;
    return launch_bwd_dw_reduce(partial, dwk, dwv, side, t.chunks, a.bias_partial, dbias, p.heads * p.S(), p.accumulate, st);
}

}  // namespace slide
