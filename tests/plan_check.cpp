// Checks of the host-side plans (slide_plan.h) over all sizes; prints what is wrong and returns 1.
#include "slide_plan.h"
#include <cmath>
#include <algorithm>
#include <chrono>
#include <cstdio>
#include <vector>

using namespace slide;
static int wrong = 0;
#define CHECK(cond, ...) do { if (!(cond)) { if (++wrong <= 20) { printf(__VA_ARGS__); printf("\n"); } } } while (0)

// strips cover the map, a run's rows fit the tile, blocks fit the LDS
static void cuts(int H, int W, bool brute)
{
    for (int ks : {3, 5})
        for (int esz : {2, 4})
            for (int which = 0; which < 4; ++which) {
                const bool few = which & 1;
                const m32::Block b = which < 2 ? m32::pixel_block(ks, few) : m32::dkdv_block(ks, esz, few);
                const m32::Cut c = m32::plan_cut(H, W, ks, b);
                const int R = ks / 2, PX = 64 * b.PG, widest = c.TW + (c.wider > 0);
                CHECK(c.TW >= 1 && c.wider >= 0 && c.wider < c.ns && (long)c.ns * c.TW + c.wider == W, "strips do not cover %dx%d", H, W);
                CHECK(c.RP == widest + 2 * R && c.npx == c.NR * c.RP && (long)c.runs * PX >= (long)H * widest, "sizes of %dx%d", H, W);
                if (brute)
                    for (int tw = c.TW; tw <= widest; ++tw)
                        for (long n0 = 0; n0 < (long)H * tw; n0 += PX) {
                            const long last = std::min((long)H * tw, n0 + PX) - 1;
                            CHECK(last / tw - n0 / tw + 1 + 2 * R <= c.NR, "a run of %dx%d touches more rows than are staged", H, W);
                        }
                // the form for few pixels runs wherever the other is refused
                if (which == 2 && m32::dkdv_few(1 << 16, 1 << 16, H, W, ks, esz)) continue;
                const size_t lds = which < 2 ? m32::pixel_lds(c, ks, b) : m32::dkdv_lds(c, ks, esz, b);
                CHECK(lds <= CU_LDS_BYTES, "%s, window %d, %d-byte elements, %dx%d: %zu bytes of LDS", which < 2 ? "per-pixel" : "dk/dv", ks, esz, H, W, lds);
            }
}

// tiles cover the map, what is staged of one fits the threads' loads and the LDS, chunks are not empty
static void gradients(int B, int H, int W, int C, int heads)
{
    for (int ks : {3, 5})
        for (int esz : {2, 4}) {
            const m32::DwPlan t = m32::plan_dw(B, H, W, C, heads, ks, esz);
            const m32::DwLoads most = m32::dw_loads(ks, esz, W % 4 == 0);
            // (bf16 5x5 calls that bring the float32 kernels' workspace bring what those need for bf16)
            CHECK(ks == 3 || t.chunks == m32::plan_dw(B, H, W, C, heads, ks, 4).chunks, "chunks of %dx%dx%d differ by type", B, H, W);
            const int R = ks / 2, S = ks * ks, NT = m32::dw_threads(ks), lanes = NT / m32::DW_CH;
            CHECK(t.TR >= 1 && t.TR <= m32::DW_MAX_ROWS && t.TC >= 4 && t.TC <= 32 && t.TC % 4 == 0 && (long)t.ntr * t.TR >= H && (t.ntr - 1) * t.TR < H &&
                  (long)t.ntc * t.TC >= W && (t.ntc - 1) * t.TC < W, "tiles of %dx%d, window %d", H, W, ks);
            CHECK(t.tiles == (long)B * t.ntr * t.ntc && t.chunks >= 1 && t.chunks <= t.tiles && t.group >= 1, "chunks of %dx%dx%d", B, H, W);
            // a walker's share of n quads in groups of g: a group is a sum of 4 g terms, the totals one of n / g, and a running sum of
            // m terms rounds like m / 2 roundings of its result: 2 g + n / 2 g, 2 sqrt(n) at best; short shares of
            // the 5x5 window stay within what whole groups allow
            if (const double n = (double)(t.tiles / t.chunks * ((t.TR * (t.TC / 4) + 1) / 2)); ks == 5 && n <= 64) {
                const double group = t.group < n ? t.group : n;
                CHECK(2 * group + n / (2 * group) <= 2 * std::sqrt(n) + 1.7, "sums of %dx%dx%d, %d channels, %d heads: %g quads in groups of %d", B, H, W, C, heads, n, t.group);
            }
            for (int cols : {t.TC, W - (t.ntc - 1) * t.TC}) {
                const int row = 1 << m32::dw_row_lanes_log2((cols + 3) / 4);
                CHECK((cols + 3) / 4 <= row && row <= lanes, "quads of %dx%d", H, W);
                CHECK(t.TR + 2 * R <= lanes / row * most.y && t.TR <= lanes / row * most.x && S * t.TR <= NT / row * most.p, "loads of %dx%d, window %d, %d-byte elements", H, W, ks, esz);
            }
            CHECK(t.KST % 2 && t.QST % 2 && t.KST >= (t.TR + 2 * R) * (t.TC + 2 * R) && t.QST >= t.TR * t.TC, "rows of %dx%d", H, W);
            const size_t floats = (size_t)m32::DW_CH * (t.KST + t.QST) + t.TR * t.TC + m32::DW_ZEROS + (size_t)t.TR * (t.TC / 4) * (4 * (S - 1) + 1);
            CHECK(t.lds >= floats * 4 && t.lds >= (size_t)m32::DW_CH * S * S * (ks == 3 ? 4 : 1) * 4 && t.lds <= CU_LDS_BYTES / (512 / NT), "LDS of %dx%d, window %d: %zu", H, W, ks, t.lds);
            CHECK((ks - 1) * (t.TC + 2 * R) + ks + 3 <= m32::DW_ZEROS, "zeros of %dx%d", H, W);
        }
}

// the split kernels: strips cover the map, a run's rows and the empty ones between planes fit the tile, offsets fit 32 bits; bands
static void stacks(int B, int H, int W, int C)
{
    const int planes = split::stack_planes(B, H, W, C), R = 2;
    CHECK(planes == B || planes == 1, "planes of %dx%dx%d", B, H, W);
    const split::Stack c = split::plan_stack(planes, H, W);
    const int widest = c.TW + (c.wider > 0);
    CHECK(c.TW >= 1 && c.wider >= 0 && c.wider < c.ns && (long)c.ns * c.TW + c.wider == W && c.RP == widest + 2 * R, "strips of %dx%d", H, W);
    CHECK(c.px >= 32 && c.px % 32 == 0 && c.px <= split::SPLIT_PX && c.npx == c.NR * c.RP && c.npx <= split::SPLIT_TILE, "tile of %dx%dx%d: %d", B, H, W, c.npx);
    CHECK((long)c.runs * c.px >= (long)planes * H * widest, "runs of %dx%dx%d", B, H, W);
    for (int tw = c.TW; tw <= widest; ++tw)
        for (long n0 = 0; n0 < (long)planes * H * tw && n0 < 40L * c.px; n0 += c.px) {
            const long l0 = n0 / tw, l1 = (std::min((long)planes * H * tw, n0 + c.px) - 1) / tw;
            CHECK(l1 - l0 + R * (l1 / H - l0 / H) + 1 + 2 * R <= c.NR, "a run of %dx%dx%d touches more rows than are staged", B, H, W);
        }
    // (a tile starts at most R rows above its first pixel's plane row and is NR rows tall)
    CHECK(planes == 1 || 2L * C * H * W * (c.NR / (H + R) + 2) < (1L << 32), "reach of %dx%dx%d, %d channels", B, H, W, C);
    for (int sets : {2, 8, 66, 600}) {
        const split::Bands t = split::plan_bands(B, H, W, sets);
        const long bands = (H + t.rows - 1) / t.rows;
        const split::DwSplitPlan w = split::plan_dw_split(B, H, W, sets);
        CHECK(w.ntr * 4L >= H && (w.ntr - 1) * 4L < H && w.ntc * 32L >= W && (w.ntc - 1) * 32L < W && w.tiles == (long)B * w.ntr * w.ntc &&
              w.chunks >= 1 && w.chunks <= w.tiles, "kernel gradients of %dx%dx%d", B, H, W);
        CHECK(t.rows >= 1 && t.blocks >= 1 && t.groups * 32 >= (long)B * W && (t.groups - 1) * 32 < (long)B * W && t.jobs == t.groups * bands, "bands of %dx%dx%d", B, H, W);
    }
}

// the split kernel gradients' loads of a row lie inside it, for every column tile and every thread's piece of it, and hold
// every element of the row that the piece wants
static void rows(int W)
{
    for (int x0 = 0; x0 < W; x0 += split::DW_COLS)
        for (int x = x0; x < x0 + split::DW_COLS; x += 8) {
            if (W % 4 == 0)
                for (int i = 0; i < 4; ++i) {
                    const int e = split::fours_from(i, x), n = split::fours_length(i), at = split::row_at(e, n, W);
                    CHECK(at >= 0 && at + n <= W, "vector %d of piece %d reads elements %d..%d of %d", i, x, at, at + n - 1, W);
                    CHECK(at == e || e < 0 || e >= W, "vector %d of piece %d of %d is moved inside the row", i, x, W);
                    CHECK(e == (i == 0 ? x - 2 : split::fours_from(i - 1, x) + split::fours_length(i - 1)), "vectors of piece %d", x);
                }
            if (W >= 4)
                for (int e = x - 2; e < x + 10; e += 4) {
                    const int at = split::row_at(e, 4, W);
                    CHECK(at >= 0 && at + 4 <= W && (at == e || e < 0 || e > W - 4), "four elements at %d of %d read at %d", e, W, at);
                }
        }
}

// the half-precision tile kernels' heights: as good as those found by trying every height down to one row where the tallest
// tiles leave compute units without one, down to half the tallest elsewhere
static double tile_makespan(int H, long planes, int th, int nA, int nB, int hb, int tw, int r2, int waves)
{
    auto cost = [&](int rows) {
        if (waves <= 0) return rows + 1.5;
        const int passes = (rows * tw + 15) / 16;
        return (double)((passes + waves - 1) / waves) + 0.35 + 0.035 * (rows + r2);
    };
    return t16::queue_makespan(planes * nA, cost(th), planes * nB, cost(hb), MAX_CU_PLANNED);
}
static void tiles(int B, int H, int W, int heads, int ks, int budget, int waves)
{
    const t16::TilePlan t = t16::plan_tiles(B, H, W, heads, ks, MAX_CU_PLANNED, budget, 64, 64, 0, waves);
    const int r2 = 2 * (ks / 2);
    const long planes = (long)B * heads * t.n_tc;
    CHECK((long)t.n_tc * t.tw >= W && (t.n_tc - 1) * t.tw < W && t.nA * t.th + t.nB * t.hb >= H && (t.nB ? t.nA * t.th + (t.nB - 1) * t.hb < H : t.nA * t.th == H) &&
          t.TA == planes * t.nA && t.TB == planes * t.nB && t.hb <= t.th && (t.th == 1 || t.buf_bytes <= budget), "tiles of %dx%dx%d", B, H, W);
    int th_max = std::min(H, std::max(1, (budget - 256) / (128 * (t.tw + r2)) - r2));
    const bool few = planes * ((H + th_max - 1) / th_max) < MAX_CU_PLANNED;
    double best = 1e300;
    for (int th = th_max; th >= (few ? 1 : std::max(1, th_max / 2)); --th)
        for (int nA = H / th; nA >= 0 && nA >= H / th - 1; --nA) {
            const int rem = H - nA * th;
            for (int nB = (rem + th - 1) / th; nB <= (rem + th - 1) / th + 2; ++nB) {
                if ((rem == 0) != (nB == 0)) continue;
                const int hb = nB ? (rem + nB - 1) / nB : 0;
                if (nB && (hb < 1 || hb * (nB - 1) >= rem)) continue;
                best = std::min(best, tile_makespan(H, planes, th, nA, nB, hb, t.tw, r2, waves));
            }
        }
    const double now = tile_makespan(H, planes, t.th, t.nA, t.nB, t.hb, t.tw, r2, waves);
    CHECK(now <= best + 1e-6, "tiles of %dx%dx%d, %d heads: %g, there are some of %g", B, H, W, heads, now, best);
}

// bands: those that trying every height finds
static void every_band(int B, int H, int W, int sets)
{
    const split::Bands t = split::plan_bands(B, H, W, sets);
    const long most = std::max(MAX_CU_PLANNED / sets, 1);
    double best = 0;
    int low = 0;
    for (int rows = 1; rows <= H && rows <= 512; ++rows) {
        const long jobs = t.groups * ((H + rows - 1) / rows), blocks = std::min((jobs + 7) / 8, most);
        const double cost = ((jobs + 8 * blocks - 1) / (8 * blocks)) * (rows + 1.5) * (blocks * sets > MAX_CU_PLANNED ? (double)(blocks * sets) / MAX_CU_PLANNED : 1.0);
        if (best == 0 || cost < best) { best = cost; low = rows; }
    }
    CHECK(t.rows == low, "bands of %dx%dx%d, %d sets: %d rows, %d are best", B, H, W, sets, t.rows, low);
}

// microseconds of one call, at its fastest of several rounds
template <typename F> static double microseconds(F&& plan)
{
    double best = 1e300;
    for (int round = 0; round < 5; ++round) {
        const auto t0 = std::chrono::steady_clock::now();
        for (int i = 0; i < 20000; ++i) plan(i);
        best = std::min(best, std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count() * 1e6 / 20000);
    }
    return best;
}

int main()
{
    const long plane = 0x7fffffffL / 64;                    // the largest map the library accepts
    std::vector<int> heights = {1, 2, 3, 4, 5, 7, 8, 16, 31, 32, 64, 65, 128, 200, 256, 300, 1000, 4096};
    for (int H : heights)
        for (int W = 1; W <= 12000 && (long)H * W <= plane; ++W) cuts(H, W, H <= 300 && W <= 200);
    for (int H = 1; H <= 300; ++H) cuts(H, (int)(plane / H), false);
    for (int W = 1; W <= 300; ++W) cuts((int)(plane / W), W, false);
    for (int H : {1, 2, 3, 5, 7, 8, 13, 14, 16, 28, 31, 41, 56, 64, 200, 224, 1000})
        for (int W = 1; W <= 700; ++W)
            for (int B : {1, 3, 64, 1000})
                for (int heads : {1, 4, 33}) gradients(B, H, W, heads * (W % 3 == 0 ? 8 : W % 3 == 1 ? 32 : 65), heads);
    for (int H : {1, 2, 3, 5, 9, 14, 16, 28, 41, 56, 64, 150, 200, 300, 1000})
        for (int W = 1; W <= 350; W += W < 70 ? 1 : 7)
            for (int B : {1, 2, 8, 64})
                for (int heads : {1, 2, 8}) {
                    tiles(B, H, W, heads, 3, 77000, 0);
                    tiles(B, H, W, heads, 3, 81920, 0);
                    tiles(B, H, W, heads, 5, 60000, 8);
                }
    for (int H : {1, 2, 3, 5, 7, 14, 28, 41, 57, 200, 1000})
        for (int W = 1; W <= 700; W += W < 140 ? 1 : 9)
            for (int B : {1, 2, 3, 64, 1000})
                for (int C : {1, 96, 4096}) stacks(B, H, W, C);
    stacks(1, 1, (int)plane, 1); stacks(2, (int)plane, 1, 64); stacks(2, 5000, 6000, 512);
    for (int W = 1; W <= 4096; ++W) rows(W);
    // planning is part of every call: it must stay a fraction of a microsecond
    const auto t0 = std::chrono::steady_clock::now();
    long sum = 0;
    for (int i = 0; i < 100000; ++i) sum += t16::plan_tiles(1, 64, 9 + (i & 1), 2, 3, MAX_CU_PLANNED, 77000, 64, 64, 0, 0).th;
    const double us = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count() * 10;
    CHECK(us < 4, "planning 64x9 takes %.2f us (%ld)", us, sum);
    for (int H : {1, 2, 3, 5, 14, 28, 56, 97, 200, 513, 600, 1000})
        for (int W : {1, 14, 28, 333})
            for (int B : {1, 3, 64})
                for (int sets : {2, 8, 66, 600}) every_band(B, H, W, sets);
    for (int H : {28, 200, 600}) {
        const double split_us = microseconds([&](int i) {
            sum += split::plan_bands(64, H, 28 + (i & 1), 8).rows + split::plan_stack(64, H, 28 + (i & 1)).npx + split::plan_dw_split(64, H, 28 + (i & 1), 8).chunks;
        });
        CHECK(split_us < 1, "planning the split kernels for %d rows takes %.2f us (%ld)", H, split_us, sum);
    }
    printf("%d wrong\n", wrong);
    return wrong != 0;
}
