// Float32 Slide Attention on the matrix cores of gfx950, windows of 3 and 5: every head size,
// width, layout and element type; products, sums and results in float32 like the general kernels
// of slide_generic.hip, which state the same operator one multiply-add at a time.
//
// What bounds these kernels is the learned-kernel contraction, k^2 shifts by k^2 taps per channel
// and pixel.  v_mfma_f32_4x4x1_16b_f32 with a broadcast left operand (cbsz = 4) is an outer product of
// four weights with 64 lanes: D[r][lane] += A[4 * abid + r] * B[lane], 256 float32 multiply-adds in
// 8 cycles (9.3 issued back to back, measured; by the counters the matrix cores are busy for 8, and a
// vector instruction beside them takes 5 to 6 more).  It multiplies and adds with one rounding, to nearest, and keeps
// denormals (checked against fmaf on a million products).  A lane is a pixel, a register of A
// holds 64 weights, so the weights come as one coalesced LDS read per 64 of them instead of one
// scalar load per multiply-add, which is what held the general kernels at 4.6 TFLOP/s.  Of the k^2
// shifts of a channel k^2 - 1 (8 or 24, a multiple of four) go through the matrix cores and the
// last one is a vector multiply-add, so no matrix row is padding.
#include "slide_mfma32.h"

namespace slide {
namespace m32 {

struct PixelArgs {
    const void* q; const void* k; const void* v; const void* dout;
    const float* wk; const float* wv; const float* bias;
    void* out;                  // forward: out; backward: dq
    float* lse;                 // forward, may be null
    float* a_ws; float* dl_ws;  // backward: [B, heads, S, H, W]
    int H, W, C, d;
    long sc, sp;                // element (b, c, pixel) at b*C*H*W + c*sc + pixel*sp
    float idw, scale;
    Cut cut;
};

// One run of PX = 64 * PG pixels of one head: waves = PG pixel groups x CG channel groups.
// CQ quads of channels are staged per step (CG waves take CQ / CG of them each); their halo tile
// lies in LDS as [quad][pixel][4 channels], so a tap is one 16-byte read for four channels (the
// LDS moves 190 B per cycle and CU that way, 82 in 4-byte reads, measured).  The next step's
// elements are fetched into registers while the current one is multiplied.  MI355X, against one
// thread per pixel (slide_generic.hip): float32, 3x3, B=32, 56x56, C=64, 2 heads: forward 335 -> 56
// us, backward 503 -> 89 us; one
// 14x14 map of 2 heads, forward: 18.9 -> 10 us.
// FOUR: a quad's channels are neighbours in memory (channels last, whole quads): one load, one store instead of
// four (bf16, 3x3, B=64, 27x27, C=128, 4 heads: 84 -> 58 us per call; float32, B=32, 56x56, C=64: 123 -> 76).
template <typename T, int KS, int PG, int CG, int CQ, bool BWD, bool FOUR>
__global__ void __launch_bounds__(64 * PG * CG, CG > 1 ? 2 : (KS == 3 ? 4 : 2))
pixel32_kernel(const PixelArgs a)
{
    using D = Dim<KS>;
    constexpr int S = D::S, SM = D::SM, SB = D::SB, R = D::R;
    constexpr int NT = 64 * PG * CG, PX = 64 * PG;
    constexpr int EW = 256, TG = NT / EW, QPT = CQ / TG;    // staging: EW pixels wide, TG quad groups, QPT quads per thread
    constexpr int NI = KS == 5 && CG > 1 ? 1 : 2;           // pixels per thread fetched ahead (5x5, shared channels: two would spill registers)
    constexpr int NW = (CQ * 4 * S * S + NT - 1) / NT;      // weights per thread
    constexpr bool AHEAD_W = NW <= 24;
    static_assert(NT % EW == 0 && CQ % TG == 0 && CQ % CG == 0, "");

    extern __shared__ __align__(16) float smem_raw[];
    float* const smem = smem_raw;                           // (through a pointer: 16-byte accesses keep their alignment)
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int pg = wave % PG, cg = wave / PG;
    const int H = a.H, W = a.W, d = a.d;
    const int m = blockIdx.y, b = blockIdx.z;
    const long HW = (long)H * W;
    const int strip = blockIdx.x / a.cut.runs, run = blockIdx.x - strip * a.cut.runs;
    int j0, tw;
    strip_of(a.cut, strip, j0, tw);
    const int n0 = run * PX;
    if (n0 >= H * tw) return;
    const int npx = a.cut.npx, RP = a.cut.RP;
    const int row0 = n0 / tw - R;                           // first staged row of the map (may be negative)
    float* tile = smem;                                     // [CQ][npx][4]
    float* wl = smem + CQ * npx * 4;                        // [CQ][QUAD_W]
    float* xl = wl + CQ * D::QUAD_W;                        // [CQ][PX][4]

    const bool wave_live = n0 + pg * 64 < H * tw;           // (the last run's waves past the strip only stage)
    // this lane's pixel
    const int n = n0 + pg * 64 + lane;
    const bool live = n < H * tw;
    const int nn = live ? n : H * tw - 1;
    const int ti = nn / tw, tj = nn - ti * tw;
    const long pix = (long)ti * W + j0 + tj;
    const int at = ((ti - row0 - R) * RP + tj) * 4;         // its upper left tap in a tile plane

    const long item = (long)b * a.C * HW + (long)m * d * a.sc;
    // staging: pixels e = (tid % EW) + i * EW of the tile
    const int e0 = tid % EW, tg = tid / EW;
    auto tile_pixel = [&](int e, bool& in) -> long {
        const int rr = e / RP, xx = e - rr * RP;
        const int y = row0 + rr, x = j0 + xx - R;
        in = e < npx && y >= 0 && y < H && x >= 0 && x < W;
        return in ? ((long)y * W + x) * a.sp : 0;
    };
    bool in[NI]; long off[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) off[i] = tile_pixel(e0 + i * EW, in[i]);
    const int pe = tid % PX, peg = tid / PX;                // staging of x: pixel pe, quads peg, peg + CG, ...
    long xoff;
    {
        const int nx = min(n0 + pe, H * tw - 1);
        const int xi = nx / tw;
        xoff = ((long)xi * W + j0 + nx - xi * tw) * a.sp;
    }

    // channels c..c+3 of the head (past d: the last one again, their weights are zeros)
    auto load4 = [&](const T* base, long o, int c) -> f4 {
        f4 r;
        if (FOUR) return Four<T>::load(base + o + min(c, d - 4));
#pragma unroll
        for (int u = 0; u < 4; ++u) r[u] = Elem<T>::load(base + o + (long)min(c + u, d - 1) * a.sc);
        return r;
    };
    // this lane's weights (float offsets from a quad's weights, for the operand registers above)
    int woff[D::WV], loff[D::LASTV];
#pragma unroll
    for (int j = 0; j < D::WV; ++j) {
        const int f = min(j * 64 + lane, D::UNIT - 1);
        const int tt = f / (4 * SM), r = f - tt * (4 * SM), e = r / SM;
        woff[j] = e * (S * S) + (r - e * SM) * S + tt;
    }
#pragma unroll
    for (int j = 0; j < D::LASTV; ++j) {
        const int f = min(j * 64 + lane, 4 * S - 1);
        loff[j] = (f & 3) * (S * S) + SM * S + (f >> 2);
    }

    // what a step stages, on its way from memory: of a tensor y, of x (q or dO; null: none) and of the kernels w
    struct Fetched { f4 y[NI][QPT], x[CQ / CG]; float w[AHEAD_W ? NW : 1]; };
    Fetched shared_set;
    struct Source { const T* y; const T* x; const float* w; };
    auto source = [&](const void* yp, const void* xp, const float* w) {
        return Source{(const T*)yp + item, xp ? (const T*)xp + item : nullptr, w + (long)m * d * S * S};
    };
    auto fetch = [&](const Source& src, int c0, Fetched& to) {
        auto &yr = to.y; auto &xr = to.x; auto &wr = to.w;
        const T *yb = src.y, *xb = src.x;
        const float* wb = src.w;
        // (a step stages the quads that the head still has: the eight of the shared form are 32 channels.  The forward's large
        // blocks stage two quads whatever the head: leaving one out cost them registers, 54 -> 56 us at stage 1)
        auto fetch_quads = [&](int c0, auto all) {
            constexpr bool ALL = decltype(all)::value;
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int u = 0; u < QPT; ++u)
                    if (ALL || c0 + 4 * (tg + u * TG) < d) yr[i][u] = load4(yb, off[i], c0 + 4 * (tg + u * TG));
            if (xb)
#pragma unroll
                for (int u = 0; u < CQ / CG; ++u)
                    if (ALL || c0 + 4 * (peg + u * CG) < d) xr[u] = load4(xb, xoff, c0 + 4 * (peg + u * CG));
        };
        if (CQ == 1 || (CG == 1 && !BWD) || c0 + 4 * CQ <= d) fetch_quads(c0, std::true_type{});
        else fetch_quads(c0, std::false_type{});
        if (AHEAD_W)
#pragma unroll
            for (int u = 0; u < NW; ++u) {
                const int idx = tid + u * NT;
                wr[u] = (idx < CQ * 4 * S * S && c0 * S * S + idx < d * S * S) ? wb[c0 * S * S + idx] : 0.0f;
            }
    };
    // runs `body(quad, offset of the quad's tile, of its weights, x of this lane)` over this wave's quads
    auto phase = [&](const Source& src, auto&& body) {
        const T *yb = src.y, *xb = src.x;
        const float* wb = src.w;
        // The 3x3 backward spills seven registers with a set per phase, two with one set for all (float32, B=32, 56x56, C=64: 91 -> 86
        // us); the 5x5 kernels spill none and take 1 to 2 % longer with one set (45x45, 13 planes: 111.7 -> 113.6 us).
        Fetched own_set;
        Fetched& to = KS == 5 ? own_set : shared_set;
        auto &yr = to.y; auto &xr = to.x; auto &wr = to.w;
        fetch(src, 0, to);
        for (int c0 = 0; c0 < d; c0 += 4 * CQ) {
            __syncthreads();                                // the step before is no longer read
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int u = 0; u < QPT; ++u)
                    if (e0 + i * EW < npx) *(f4*)(tile + ((tg + u * TG) * npx + e0 + i * EW) * 4) = in[i] ? yr[i][u] : f4{0.0f, 0.0f, 0.0f, 0.0f};
            for (int e = e0 + NI * EW; e < npx; e += EW) {   // (maps of a few columns, wide windows)
                bool ok;
                const long o = tile_pixel(e, ok);
#pragma unroll
                for (int u = 0; u < QPT; ++u)
                    *(f4*)(tile + ((tg + u * TG) * npx + e) * 4) = ok ? load4(yb, o, c0 + 4 * (tg + u * TG)) : f4{0.0f, 0.0f, 0.0f, 0.0f};
            }
            if (xb)
#pragma unroll
                for (int u = 0; u < CQ / CG; ++u) *(f4*)(xl + ((peg + u * CG) * PX + pe) * 4) = xr[u];
            if (AHEAD_W) {
#pragma unroll
                for (int u = 0; u < NW; ++u)
                    if (tid + u * NT < CQ * 4 * S * S) wl[tid + u * NT] = wr[u];
            } else {
#pragma unroll 4
                for (int idx = tid; idx < CQ * 4 * S * S; idx += NT)
                    wl[idx] = c0 * S * S + idx < d * S * S ? wb[c0 * S * S + idx] : 0.0f;
            }
            // the fixed shift path of the two-branch form: 1 + w, rounded to 24 bits as slide_reparam rounds it.  That is one
            // rounding where adding the shifted value on its own takes one more per tap: out 1.31e-7 from 64 bits here,
            // 1.42e-7 on the general kernels (float32, 3x3, 56x56)
            if (a.idw != 0.0f) {
                __syncthreads();
                for (int i = tid; i < min(CQ * 4, d - c0) * S; i += NT) wl[(i / S) * (S * S) + (i % S) * (S + 1)] += a.idw;
            }
            __syncthreads();
            if (c0 + 4 * CQ < d) fetch(src, c0 + 4 * CQ, to);
#pragma unroll 1
            for (int u = cg; u < CQ && wave_live; u += CG) {
                if (c0 + 4 * u >= d) break;
                body(c0 + 4 * u, u * npx * 4 + at, CQ * npx * 4 + u * D::QUAD_W, xl + (u * PX + pg * 64 + lane) * 4);
            }
        }
    };

    // win[e][s] = sum over taps of W[c+e,s,t] y[c+e,t] of a quad's four channels: the sums over shifts s < SM in
    // acc[e], the last shift's in last[e]
    auto window_sums = [&](int yo, int wo, f4 (&acc)[4][SB], float (&last)[4]) {
        float wv[D::WV], wlast[D::LASTV];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            last[e] = 0.0f;
#pragma unroll
            for (int i = 0; i < SB; ++i) acc[e][i] = f4{0.0f, 0.0f, 0.0f, 0.0f};
        }
#pragma unroll
        for (int j = 0; j < D::LASTV; ++j) wlast[j] = smem[wo + loff[j]];
        unroll<S>([&](auto tc) {
            constexpr int t = decltype(tc)::value;
            if (t % KS == 0) pin(yo, wo, wlast);            // (one window row in registers at a time)
            if (t % D::UT == 0)
#pragma unroll
                for (int j = 0; j < D::WV; ++j) wv[j] = smem[wo + woff[j] + t];
            const f4 yt = *(const f4*)(smem + yo + ((t / KS) * RP + t % KS) * 4);
            // (vector work first, then the matrix instructions back to back: between two of them a
            // vector instruction costs the issue of about one more, measured)
            unroll<4>([&](auto ec) {
                constexpr int e = decltype(ec)::value;
                last[e] = fmaf(lane_of(wlast[(4 * t + e) / 64], (4 * t + e) % 64), yt[e], last[e]);
            });
            asm volatile("" : "+v"(last[0]), "+v"(last[1]), "+v"(last[2]), "+v"(last[3]));
            __builtin_amdgcn_sched_barrier(0);
            unroll<4>([&](auto ec) {
                constexpr int e = decltype(ec)::value;
                outer_blocks<((t % D::UT) * 4 + e) * SB>(wv, yt[e], acc[e]);
            });
            __builtin_amdgcn_sched_barrier(0);
        });
    };

    // sums over shifts: sum[s] += sum over channels of x[c] * (sum over taps of W[c,s,t] y[c,t])
    auto contract = [&](const Source& src, float (&sum)[S]) {
        // A channel's window is summed before x multiplies it, as in the general kernels, and the channels are added
        // in fours, the fours in fours: their sum is what rounds most.  Error of out against 64 bits (2-norm), float32,
        // merged kernels, 32 channels per head: 1.26e-7 (3x3, 56x56), 1.94e-7 (5x5, 28x28), the general kernels 1.26e-7 and
        // 1.94e-7; with x multiplied in first and the rows of all quads added one by one 1.47e-7 and 2.36e-7, at the same time.
        // (CG > 1: a wave has few quads, and the shares are added as a tree)
        float part[S];
        int left = 4;                                       // quads until part is added to the total, which lies in LDS
        float* const total = xl + CQ * PX * 4 + pg * 64 + lane;     // [S][PX], CG == 1
#pragma unroll
        for (int s = 0; s < S; ++s) part[s] = 0.0f;
        if (CG == 1)
#pragma unroll
            for (int s = 0; s < S; ++s) total[s * PX] = 0.0f;
        phase(src, [&](int, int yo, int wo, const float* xq) {
            f4 acc[4][SB];
            float last[4];
            window_sums(yo, wo, acc, last);
            const f4 x = *(const f4*)xq;
#pragma unroll
            for (int s = 0; s < S; ++s) {
                float four = x[0] * (s < SM ? acc[0][s / 4 % SB][s % 4] : last[0]);
#pragma unroll
                for (int e = 1; e < 4; ++e) four = fmaf(x[e], s < SM ? acc[e][s / 4 % SB][s % 4] : last[e], four);
                part[s] += four;
            }
            if (CG == 1 && --left == 0) {
                left = 4;
#pragma unroll
                for (int s = 0; s < S; ++s) { total[s * PX] += part[s]; part[s] = 0.0f; }
            }
        });
#pragma unroll
        for (int s = 0; s < S; ++s) sum[s] = CG == 1 ? total[s * PX] + part[s] : part[s];
        if (CG > 1) {                                       // the channel groups' shares, added in a fixed order
            float* red = smem;                              // [CG][S][PX]
            __syncthreads();
#pragma unroll
            for (int s = 0; s < S; ++s) red[(cg * S + s) * PX + pg * 64 + lane] = sum[s];
            __syncthreads();
#pragma unroll
            for (int s = 0; s < S; ++s) {
                float r[CG];
#pragma unroll
                for (int c = 0; c < CG; ++c) r[c] = red[(c * S + s) * PX + pg * 64 + lane];
#pragma unroll
                for (int w = 1; w < CG; w *= 2)
#pragma unroll
                    for (int c = 0; c + w < CG; c += 2 * w) r[c] += r[c + w];
                sum[s] = r[0];
                asm volatile("" : "+v"(sum[s]) :: "memory");
            }
            // (the next phase starts with a barrier before it writes LDS)
        }
    };
    // out[c] = f * sum over shifts of p[s] * (sum over taps of W[c,s,t] y[c,t])
    auto expand = [&](const Source& src, const float (&p)[S], float f) {
        T* ob = (T*)a.out + item + pix * a.sp;
        phase(src, [&](int c, int yo, int wo, const float*) {
            f4 acc[4][SB];
            float last[4];
            window_sums(yo, wo, acc, last);
            f4 ov;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float o = p[SM] * last[e];
#pragma unroll
                for (int s = 0; s < SM; ++s) o = fmaf(p[s], acc[e][s / 4][s % 4], o);
                ov[e] = f * o;
            }
            if (FOUR) {
                if (live) Four<T>::store(ob + c, ov);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (live && c + e < d) Elem<T>::store(ob + (long)(c + e) * a.sc, ov[e]);
            }
        });
    };

    float p[S];
    contract(source(a.k, a.q, a.wk), p);
    float mx = -INFINITY;
#pragma unroll
    for (int s = 0; s < S; ++s) {
        p[s] = fmaf(a.scale, p[s], a.bias ? a.bias[m * S + s] : 0.0f);
        mx = fmaxf(mx, p[s]);
    }
    float den = 0.0f;
#pragma unroll
    for (int s = 0; s < S; ++s) { p[s] = expf(p[s] - mx); den += p[s]; }
    const float inv = 1.0f / den;
#pragma unroll
    for (int s = 0; s < S; ++s) {                           // p / den: the reciprocal's own rounding is taken out again
        const float e = p[s];
        p[s] = e * inv;
        p[s] = fmaf(fmaf(-p[s], den, e), inv, p[s]);
    }
    if (!BWD) {
        if (a.lse && live && cg == 0) a.lse[((long)b * (a.C / d) + m) * HW + pix] = mx + logf(den);
        expand(source(a.v, nullptr, a.wv), p, 1.0f);
    } else {
        // (p waits in a_ws while da is summed: the sums need the registers.  The barriers of `contract` order the
        // stores before the other channel groups' loads)
        float* const a_px = a.a_ws + ((long)b * (a.C / d) + m) * S * HW + pix;
        float* const dl_px = a.dl_ws + ((long)b * (a.C / d) + m) * S * HW + pix;
        if (live && cg == 0)
#pragma unroll
            for (int s = 0; s < S; ++s) a_px[(long)s * HW] = p[s];
        float da[S];
        contract(source(a.v, a.dout, a.wv), da);
#pragma unroll
        for (int s = 0; s < S; ++s) p[s] = a_px[(long)s * HW];
        float dsum = 0.0f;
#pragma unroll
        for (int s = 0; s < S; ++s) dsum = fmaf(p[s], da[s], dsum);
#pragma unroll
        for (int s = 0; s < S; ++s) {
            da[s] = p[s] * (da[s] - dsum);
            if (live && cg == 0) dl_px[(long)s * HW] = da[s];
        }
        expand(source(a.k, nullptr, a.wk), da, a.scale);
    }
}

template <typename T, int KS, bool FEW, bool BWD, bool FOUR>
static hipError_t launch_pixel(const Problem& p, PixelArgs& a, hipStream_t st)
{
    constexpr Block b = pixel_block(KS, FEW);
    constexpr auto kernel = pixel32_kernel<T, KS, b.PG, b.CG, b.NQ, BWD, FOUR>;
    a.cut = plan_cut(p.H, p.W, KS, b);
    static LdsOptIn opt_in;
    hipError_t e = opt_in.ensure({(const void*)kernel}, (int)CU_LDS_BYTES);
    if (e != hipSuccess) return e;
    const dim3 grid((unsigned)(a.cut.ns * a.cut.runs), (unsigned)p.heads, (unsigned)p.B);
    hipLaunchKernelGGL(kernel, grid, dim3(64 * b.PG * b.CG), pixel_lds(a.cut, KS, b), st, a);
    return hipGetLastError();
}

template <typename T, int KS, bool BWD, bool FOUR = false>
static hipError_t launch_pixel_t(const Problem& p, PixelArgs& a, hipStream_t st)
{
    if constexpr (!BWD && !FOUR)
        if (p.nhwc && p.d() % 4 == 0) return launch_pixel_t<T, KS, false, true>(p, a, st);
    if (pixel_few(p.B, p.heads, p.H, p.W, p.d(), KS)) return launch_pixel<T, KS, true, BWD, FOUR>(p, a, st);
    return launch_pixel<T, KS, false, BWD, FOUR>(p, a, st);
}

static PixelArgs pixel_args(const Problem& p, const void* q, const void* k, const void* v, const float* wk,
                            const float* wv, const float* bias, void* out)
{
    PixelArgs a{};
    a.q = q; a.k = k; a.v = v; a.wk = wk; a.wv = wv; a.bias = bias; a.out = out;
    a.H = p.H; a.W = p.W; a.C = p.C; a.d = p.d();
    a.sc = p.nhwc ? 1 : p.plane(); a.sp = p.nhwc ? p.C : 1;
    a.idw = p.two_branch ? 1.0f : 0.0f;
    a.scale = 1.0f / sqrtf((float)p.d());
    return a;
}

}  // namespace m32

bool m32_supported(const Problem& p) { return p.ksize == 3 || p.ksize == 5; }

hipError_t launch_fwd_m32(const Problem& p, const void* q, const void* k, const void* v, const float* wk,
                          const float* wv, const float* bias, void* out, float* lse, hipStream_t st)
{
    m32::PixelArgs a = m32::pixel_args(p, q, k, v, wk, wv, bias, out);
    a.lse = lse;
    if (p.dtype == 0)
        return p.ksize == 3 ? m32::launch_pixel_t<float, 3, false>(p, a, st) : m32::launch_pixel_t<float, 5, false>(p, a, st);
    return p.ksize == 3 ? m32::launch_pixel_t<bf16_bits, 3, false>(p, a, st) : m32::launch_pixel_t<bf16_bits, 5, false>(p, a, st);
}

hipError_t launch_bwd_pixel_m32(const Problem& p, const void* dout, const void* q, const void* k, const void* v,
                                const float* wk, const float* wv, const float* bias, void* dq, float* a_ws,
                                float* dl_ws, hipStream_t st)
{
    m32::PixelArgs a = m32::pixel_args(p, q, k, v, wk, wv, bias, dq);
    a.dout = dout; a.a_ws = a_ws; a.dl_ws = dl_ws;
    if (p.dtype == 0)
        return p.ksize == 3 ? m32::launch_pixel_t<float, 3, true>(p, a, st) : m32::launch_pixel_t<float, 5, true>(p, a, st);
    return p.ksize == 3 ? m32::launch_pixel_t<bf16_bits, 3, true>(p, a, st) : m32::launch_pixel_t<bf16_bits, 5, true>(p, a, st);
}

}  // namespace slide
