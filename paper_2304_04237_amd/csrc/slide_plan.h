// Host-side planning that needs nothing but the sizes: no HIP header, so that a plan can be checked for
// every size on a machine without a GPU.
#pragma once
#include <stddef.h>
#include <initializer_list>

namespace slide {

// the most compute units that anything is planned for
constexpr int MAX_CU_PLANNED = 256;
constexpr size_t CU_LDS_BYTES = 160 * 1024;                    // of a compute unit

// ---- half-precision tile kernels: a (batch, head) plane is cut into tiles of th x tw pixels
namespace t16 {

struct TilePlan {
    int th, tw, n_tc, nA, nB, hb, TA, TB;
    int v_off, buf_bytes;    // the two halo tensors of a tile occupy buf_bytes of LDS
    int halo_px;             // halo pixels of a full tile: (th + 2r) * (tw + 2r)
};

// makespan of dealing big-first: TA tiles of cost cA first, then TB tiles of cost cB, G blocks
inline double queue_makespan(long TA, double cA, long TB, double cB, int G)
{
    const long qa = TA / G, ra = TA % G;
    const double lo = qa * cA, hi = (ra ? qa + 1 : qa) * cA;
    if (TB == 0) return hi;
    // smallest M with sum_b floor((M - L_b) / cB) >= TB, tried on the grid lo + j*cB, hi + j*cB
    double best = 1e300;
    for (long j = 0; j <= TB / G + 2; ++j) {
        for (int w = 0; w < 2; ++w) {
            const double M = (w ? hi : lo) + j * cB;
            if (M < hi) continue;
            const long cap = (G - ra) * (long)((M - lo) / cB + 1e-9) + ra * (long)((M - hi) / cB + 1e-9);
            if (cap >= TB && M < best) best = M;
        }
    }
    return best;
}

// Tile heights for a kernel that may spend lds_budget bytes on one tile buffer holding two
// halo tensors of px_bytes per halo pixel each (64 for a staged activation tensor).
// px_bytes_extra: further LDS bytes per halo pixel that the kernel places after the buffer.
// pass_waves > 0: the kernel deals the 16-pixel passes of a tile to that many waves and does
// not overlap the staging of a tile with its passes; a tile then costs the rounds of passes
// its busiest wave runs plus a staging share, instead of its rows.
inline TilePlan plan_tiles(int B, int H, int W, int heads, int ksize, int n_cu, int lds_budget, int px_bytes_a, int px_bytes_b,
                           int px_bytes_extra, int pass_waves)
{
    const int r2 = 2 * (ksize / 2);
    TilePlan t;
    t.tw = W <= 64 ? W : 64;
    t.n_tc = (W + t.tw - 1) / t.tw;
    if (t.n_tc > 1 && W % 8 != 0) t.tw = ((W + t.n_tc - 1) / t.n_tc + 7) & ~7;  // even shares, in whole staging chunks
    const int px_bytes = px_bytes_a + px_bytes_b + px_bytes_extra;
    int th_max = (lds_budget - 256) / (px_bytes * (t.tw + r2)) - r2;
    if (th_max < 1) th_max = 1;
    if (th_max > H) th_max = H;
    const long planes = (long)B * heads * t.n_tc;
    // choose the tile heights that minimise the makespan of dealing the tiles to one block
    // per compute unit slot (cost of a tile: its rows plus a fixed share for the halo rows
    // and the per-tile overhead)
    double best = 1e300;
    t.th = th_max; t.nA = H / th_max; t.nB = (H % th_max) ? 1 : 0; t.hb = H % th_max;
    int tallest = th_max, lowest = th_max / 2 < 1 ? 1 : th_max / 2;
    if (planes * ((H + th_max - 1) / th_max) < n_cu) {
        // such tiles leave compute units without one, so lower ones are tried too, from the height on at which
        // every tile has a unit of its own (a taller one takes longer and leaves more units idle)
        // (bf16, 3x3, 2 heads, 24x24: forward 10.9 -> 8.6 us; trying every height took 5 us of host time there, 17 at 64x9)
        const int per_plane = (int)(n_cu / planes);
        tallest = (H + per_plane - 1) / per_plane;
        lowest = 1;
        if (tallest > th_max) tallest = th_max;
    }
    for (int th = tallest; th >= lowest; --th) {
        for (int drop = 0; drop < 2; ++drop) {
            const int nA = H / th - drop;
            if (nA < 0) continue;
            const int rem = H - nA * th;
            for (int nB = (rem + th - 1) / th; nB <= (rem + th - 1) / th + 2; ++nB) {
                if ((rem == 0) != (nB == 0)) continue;
                const int hb = nB ? (rem + nB - 1) / nB : 0;
                if (nB && (hb < 1 || (long)hb * (nB - 1) >= rem)) continue;
                auto cost = [&](int rows) {
                    if (pass_waves <= 0) return rows + 1.5;
                    const int passes = (rows * t.tw + 15) / 16;
                    return (double)((passes + pass_waves - 1) / pass_waves) + 0.35 + 0.035 * (rows + r2);
                };
                const double ms = queue_makespan(planes * nA, cost(th), planes * nB, cost(hb), n_cu);
                if (ms < best - 1e-9) { best = ms; t.th = th; t.nA = nA; t.nB = nB; t.hb = hb; }
            }
        }
    }
    t.TA = (int)(planes * t.nA);
    t.TB = (int)(planes * t.nB);
    const int halo_px = (t.th + r2) * (t.tw + r2);
    t.halo_px = halo_px;
    t.v_off = halo_px * px_bytes_a;
    if ((t.v_off & 127) == 0) t.v_off += 64;             // the two tensors start 64 B apart mod 128
    t.buf_bytes = (t.v_off + halo_px * px_bytes_b + 127) & ~127;
    return t;
}

}  // namespace t16

namespace m32 {

// ---- float32 matrix-core kernels (slide_mfma32.hip, slide_mfma32_bwd.hip)
// A block: PG groups of 64 pixels, CG groups of channels, NQ quads of channels per step.
struct Block { int PG, CG, NQ; };
// per-pixel kernels and dk/dv kernel, for many pixels and for few of them
constexpr Block pixel_block(int ks, bool few) { return few ? Block{1, 8, 8} : Block{4, 1, ks == 3 ? 2 : 1}; }
constexpr Block dkdv_block(int ks, int element_bytes, bool few)
{
    return few ? Block{1, 4, ks == 3 ? 8 : 4} : Block{4, 1, (ks == 3 ? 4 : 1) * (element_bytes == 2 ? 2 : 1)};
}

// How a plane is cut: ns column strips of TW or TW + 1 columns (the first `wider` of them), each flattened row by
// row and cut into runs of PX pixels, so that nearly every lane has a pixel whatever the map's width.  A
// run touches NR - 2R rows; LDS holds those rows and the halo, RP pixels each.  The strips are even because the
// narrowest sets the rows and the widest their length: strips of one width with a remainder of a few columns asked
// for more LDS than there is (5x5 from 2715 columns on, 3x3 from 3539).
struct Cut { int TW, wider, ns, runs, NR, RP, npx; };

inline Cut plan_cut(int H, int W, int PX, int R, int max_tw)
{
    Cut c;
    c.ns = (W + max_tw - 1) / max_tw;
    c.TW = W / c.ns;
    c.wider = W - c.ns * c.TW;
    const int widest = c.TW + (c.wider > 0);
    c.runs = (int)(((long)H * widest + PX - 1) / PX);
    int rows = (PX - 2) / c.TW + 2;
    if (rows > H) rows = H;
    c.NR = rows + 2 * R;
    c.RP = widest + 2 * R;
    c.npx = c.NR * c.RP;
    return c;
}
inline Cut plan_cut(int H, int W, int ks, const Block& b) { return plan_cut(H, W, 64 * b.PG, ks / 2, 64 - 2 * (ks / 2)); }

// LDS bytes of a block: tile, kernels and x of a step, the pixels' sums over channels (where channel groups share a
// pixel: those of every group, in the place of the step) ...
inline size_t pixel_lds(const Cut& c, int ks, const Block& b)
{
    const size_t S = (size_t)ks * ks, PX = 64 * (size_t)b.PG;
    const size_t step = (size_t)b.NQ * ((size_t)c.npx * 4 + 4 * S * S + PX * 4), sums = (size_t)b.CG * S * PX;
    return (b.CG == 1 ? step + sums : step > sums ? step : sums) * sizeof(float);
}
// ... tile and kernels of a step, a (or dl) of the tile
inline size_t dkdv_lds(const Cut& c, int ks, int element_bytes, const Block& b)
{
    const size_t S = (size_t)ks * ks;
    return (size_t)c.npx * ((size_t)b.NQ * 4 * element_bytes + S * sizeof(float)) + (size_t)b.NQ * 4 * S * S * sizeof(float);
}

// Blocks of 256 pixels, or of 64 whose channels eight waves share.  The large ones take 2.5 (3x3) or 8.7 us (5x5) per
// quad of channels up to two to a compute unit; of the small ones a unit holds one, and each set of 256 of them
// takes 7.6 us, or 16 and 2.2 for every quad, per eight quads (MI355X, float32 forward, 1..24 channels per head, maps of
// 15x15 to 93x93 with 8 heads; three compute units' worth of 5x5 blocks slow each other down by 1.6).  Choosing by
// the number of blocks alone (small ones below 512 large) took 38 us instead of 9 for 93x93 and heads of 4 channels.
inline bool pixel_few(int B, int heads, int H, int W, int d, int ks)
{
    const long large = ((long)H * W + 255) / 256 * heads * B;
    if (large >= 512) return false;
    const long sets = (((long)H * W + 63) / 64 * heads * B + MAX_CU_PLANNED - 1) / MAX_CU_PLANNED;
    const int quads = (d + 3) / 4, eights = (quads + 7) / 8;
    if (ks == 3) return sets * (5.3 + 2.3 * eights) < 3.5 + 2.5 * quads;
    return sets * eights * (16 + 2.2 * (quads < 8 ? quads : 8)) < (3.5 + 8.7 * quads) * (large > MAX_CU_PLANNED ? 1.6 : 1.0);
}
// dk/dv kernel: blocks of 256 pixels where those give every compute unit two and two fit its LDS (maps of a few columns
// have tall runs with much halo), else 64 pixels whose channels four waves share.  5x5, float32, B=32,
// 2 heads, large and small form: 28x28 125 and 220 us, 40x40 224 and 398.  From 41 columns on a second large block does not fit
// (bf16 has twice the quads of half the size, the same bytes), and the small form runs although one large block per compute
// unit is the faster one there too: 45x45 239 and 492, 56x56 388 and 730.  Maps of a few columns have not been compared.
inline bool dkdv_few(int B, int heads, int H, int W, int ks, int element_bytes)
{
    if (((long)H * W + 255) / 256 * heads * 2 * B < 512) return true;
    const Block b = dkdv_block(ks, element_bytes, false);
    return dkdv_lds(plan_cut(H, W, ks, b), ks, element_bytes, b) > CU_LDS_BYTES / 2;
}

// ---- kernel and bias gradients: chunks of tiles of TR rows and TC columns
constexpr int DW_CH = 32;                                   // channels per block
constexpr int DW_ZEROS = 160;                               // as many as the taps of a quad span: 4 * 36 + 8
constexpr int dw_threads(int ks) { return ks == 3 ? 256 : 512; }
// quads of four pixels that a thread fetches of y, x and a (or dl) for one tile: what the registers beside the sums
// hold.  whole: W % 4 == 0, rows are whole quads (else a quad costs some registers for its bounds)
struct DwLoads { int y, x, p; };
constexpr DwLoads dw_loads(int ks, int element_bytes, bool whole)
{
    return ks == 5 ? DwLoads{6, 4, 3} : element_bytes == 4 ? DwLoads{6, 4, 2} : whole ? DwLoads{10, 8, 3} : DwLoads{8, 6, 2};
}
// lanes that stage a row of so many quads
constexpr int dw_row_lanes_log2(int quads) { return quads > 4 ? 3 : quads > 2 ? 2 : quads > 1 ? 1 : 0; }
constexpr int DW_MAX_ROWS = 8;                              // rows of a tile
struct DwPlan { int TR, TC, ntr, ntc, KST, QST, chunks, group; long tiles; size_t lds; };

inline DwPlan plan_dw(int B, int H, int W, int C, int heads, int ks, int element_bytes)
{
    const int S = ks * ks, R = ks / 2, d = C / heads;
    DwPlan t;
    auto lds = [&](int TR, int TC) {
        t.KST = ((TR + 2 * R) * (TC + 2 * R)) | 1;          // odd: 32 channels, 32 banks
        t.QST = (TR * TC) | 1;
        const size_t tile = (size_t)DW_CH * (t.KST + t.QST) + (size_t)TR * TC + DW_ZEROS + (size_t)TR * (TC / 4) * (4 * (S - 1) + 1);
        const size_t red = (size_t)DW_CH * S * S * (ks == 3 ? dw_threads(ks) / 64 : 1);
        return (tile > red ? tile : red) * sizeof(float);
    };
    // blocks: eight waves on every compute unit.  Tiles: those that cost the fewest rounds of one quad per walker.  Where that
    // gives far fewer tiles than chunks wanted, lower ones, down to 8 pixels of each walker: more blocks, and
    // their sums are as short as those of the general kernel's threads
    const int per_cu = 512 / dw_threads(ks), walkers = ks == 3 ? 8 : 2;
    const long jobs = 2L * heads * ((d + DW_CH - 1) / DW_CH);
    long n = per_cu * MAX_CU_PLANNED / jobs;                // (a few blocks more would run after all others)
    if (n < 1) n = 1;
    auto rounds = [&](int th, int tw) { return (th * ((tw + 3) / 4) + walkers - 1) / walkers; };
    const int strips = (W + 31) / 32, even = ((W + strips - 1) / strips + 3) & ~3;
    double best = 0;
    const DwLoads most = dw_loads(ks, element_bytes, W % 4 == 0);
    const int lanes = dw_threads(ks) / DW_CH;               // that stage a channel
    for (int TR = DW_MAX_ROWS < H ? DW_MAX_ROWS : H; TR >= 1; --TR)
        for (int TC : {even, 32}) {
            const int quads = 1 << dw_row_lanes_log2(TC / 4);
            if (lds(TR, TC) > CU_LDS_BYTES / per_cu || (TR + 2 * R) * quads > lanes * most.y || TR * quads > lanes * most.x ||
                S * TR * quads > dw_threads(ks) * most.p) continue;
            const int ntr = (H + TR - 1) / TR, ntc = (W + TC - 1) / TC, lr = H - (ntr - 1) * TR, lc = W - (ntc - 1) * TC;
            // a tile costs its rounds, the rows it stages and its barriers; a chunk has whole tiles, so the block with the most of
            // them has up to one more than the average (bf16, 5x5, 30 x 54x40, 3 heads: 395 us with tiles of the fewest rounds and
            // two blocks more than there is room for, 223 like this, and the same plan for float32; 3x3, 1 x 200x333, 3 heads 73 and 66)
            auto tile = [&](int th, int tw) { return rounds(th, tw) + 1.5 + 0.1 * (th + 2 * R); };
            const double plane = (ntr - 1.0) * ((ntc - 1.0) * tile(TR, TC) + tile(TR, lc)) + (ntc - 1.0) * tile(lr, TC) + tile(lr, lc);
            const long tiles = (long)B * ntr * ntc, chunks = n < tiles ? n : tiles;
            const double cost = B * plane / chunks + tile(TR, TC) * ((tiles + chunks - 1) / chunks - (double)tiles / chunks) + 0.02 * chunks;
            if (best == 0 || cost < best) { best = cost; t.TR = TR; t.TC = TC; }
        }
    t.ntc = (W + t.TC - 1) / t.TC;
    while (t.TR > 1 && 4L * B * ((H + t.TR - 1) / t.TR) * t.ntc < 3 * n && t.TR * t.TC > 8 * walkers) --t.TR;
    t.ntr = (H + t.TR - 1) / t.TR;
    t.lds = lds(t.TR, t.TC);
    t.tiles = (long)B * t.ntr * t.ntc;
    if (n > t.tiles) n = t.tiles;
    t.chunks = (int)n;
    // quads of a walker between two additions to its totals: 3x3 32 pixels, 12 where its whole share is not much more (the
    // additions cost nothing there).  5x5: a share of n quads in groups of g rounds like 2 g + n / 2 g roundings, least at
    // g = sqrt(n) / 2, which is what is taken up to 64 quads; beyond, longer groups for time (32 pixels cost 6 % more than 64).
    // Merged kernels, float32, C=64, 2 heads, dwv against 64 bits (mean of 10 inputs), dw kernel, MI355X: 4 x 28x28 (7 quads)
    // groups of 3 1.791e-7, 19.6 us, of 2 1.771e-7, 20.2 us (general kernels 1.762e-7); 4 x 56x56 (28) of 3 1.869e-7, 46.7 us,
    // of 2 1.868e-7, 49.6 us; 32 x 28x28 (50) of 8 2.024e-7, 66.6 us, of 4 1.955e-7, 71.1 us (general kernels 1.996e-7)
    const long share = t.tiles / n * rounds(t.TR, t.TC);
    t.group = ks == 3 ? (share <= 16 ? 3 : 8) : share <= 16 ? 2 : share <= 32 ? 3 : share <= 64 ? 4 : share <= 128 ? 8 : 16;
    return t;
}

}  // namespace m32
namespace split {

// ---- 5x5 window, float32 work on the bf16 matrix cores (slide_split.hip)
constexpr int SPLIT_PX = 256;                               // pixels of a block
constexpr int SPLIT_TILE = 768;                             // places of its halo tile, three per thread

// The planes of several items as one tall map: R empty rows between two of them are the lower halo of one and the upper halo
// of the next.  It is cut into even column strips (Cut says why), a strip flattened row by row (without the empty rows) and cut
// into runs of px pixels, of which only the last is not full.  A run's halo tile is NR rows of RP pixels.
struct Stack { int planes, TW, wider, ns, px, runs, NR, RP, npx; };

inline Stack plan_stack(int planes, int H, int W)
{
    constexpr int R = 2, MAX_TW = 64 - 2 * R;
    Stack c;
    c.planes = planes;
    c.ns = (W + MAX_TW - 1) / MAX_TW;
    c.TW = W / c.ns;
    c.wider = W - c.ns * c.TW;
    const int widest = c.TW + (c.wider > 0);
    c.RP = widest + 2 * R;
    for (c.px = SPLIT_PX;; c.px -= 32) {                    // (less than 256 on maps of a few columns or rows)
        long rows = (c.px - 2) / c.TW + 2, gaps;            // that a run touches, and the empty ones between them
        if (rows > (long)planes * H) rows = (long)planes * H;
        gaps = (rows - 1 + H - 1) / H;
        if (gaps > planes - 1) gaps = planes - 1;
        c.NR = (int)(rows + R * gaps) + 2 * R;
        c.npx = c.NR * c.RP;
        if (c.npx <= SPLIT_TILE || c.px <= 32) break;
    }
    c.runs = (int)(((long)planes * H * widest + c.px - 1) / c.px);
    return c;
}
// how many planes are stacked: all, unless a run's tile may reach further from its first plane than 32-bit offsets do
inline int stack_planes(int B, int H, int W, int C)
{
    const long reach = plan_stack(B, H, W).NR / (H + 2) + 2;
    return 2L * C * H * W * reach < (1L << 32) ? B : 1;
}

// key and value gradients: jobs of 32 columns (of all items) by a band of rows, dealt to the waves of at most one block per
// compute unit for `sets` sets of operands.  A row of a band costs 25 chains, a band about as much as two rows besides.
struct Bands { int rows, blocks; long groups, jobs; };
inline Bands plan_bands(int B, int H, int W, int sets)
{
    Bands t;
    t.groups = ((long)B * W + 31) / 32;
    const long most = MAX_CU_PLANNED / sets > 1 ? MAX_CU_PLANNED / sets : 1;
    double best = 0;
    for (int rows = 1, bands; rows <= H && rows <= 512; rows = bands > 1 ? (H - 1) / (bands - 1) + 1 : H + 1) {     // (the lowest of each number of bands)
        bands = (H + rows - 1) / rows;
        const long jobs = t.groups * bands, blocks = (jobs + 7) / 8 < most ? (jobs + 7) / 8 : most;
        const double cost = ((jobs + 8 * blocks - 1) / (8 * blocks)) * (rows + 1.5) * (blocks * sets > MAX_CU_PLANNED ? (double)(blocks * sets) / MAX_CU_PLANNED : 1.0);
        if (best == 0 || cost < best) { best = cost; t.rows = rows; t.blocks = (int)blocks; t.jobs = jobs; }
    }
    return t;
}

// kernel gradients: tiles of 4 rows and 32 columns, dealt in chunks to one block per compute unit for `sets` sets of 32 channels
constexpr int DW_ROWS = 4, DW_COLS = 32;
struct DwSplitPlan { int ntr, ntc, chunks; long tiles; };
inline DwSplitPlan plan_dw_split(int B, int H, int W, int sets)
{
    DwSplitPlan t;
    t.ntr = (H + DW_ROWS - 1) / DW_ROWS;
    t.ntc = (W + DW_COLS - 1) / DW_COLS;
    t.tiles = (long)B * t.ntr * t.ntc;
    const long n = MAX_CU_PLANNED / sets > 1 ? MAX_CU_PLANNED / sets : 1;
    t.chunks = (int)(n < t.tiles ? n : t.tiles);
    return t;
}
// where the vector of n elements that belongs at element e of a row of W (at least n) is read: inside the row, whatever e is
constexpr int row_at(int e, int n, int W) { return e < 0 ? 0 : e < W - n ? e : W - n; }
// the four vectors that hold elements x-2..x+9 of a row of whole fours: first element and length of vector i
constexpr int fours_from(int i, int x) { return i == 0 ? x - 2 : x + 4 * (i - 1); }
constexpr int fours_length(int i) { return i == 0 || i == 3 ? 2 : 4; }

}  // namespace split
}  // namespace slide
