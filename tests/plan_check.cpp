// Checks of the host-side plans (slide_plan.h) over all sizes; prints what is wrong and returns 1.
#include "slide_plan.h"
#include <algorithm>
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

int main()
{
    const long plane = 0x7fffffffL / 64;                    // the largest map the library accepts
    std::vector<int> heights = {1, 2, 3, 4, 5, 7, 8, 16, 31, 32, 64, 65, 128, 200, 256, 300, 1000, 4096};
    for (int H : heights)
        for (int W = 1; W <= 12000 && (long)H * W <= plane; ++W) cuts(H, W, H <= 300 && W <= 200);
    for (int H = 1; H <= 300; ++H) cuts(H, (int)(plane / H), false);
    for (int W = 1; W <= 300; ++W) cuts((int)(plane / W), W, false);
    printf("%d wrong\n", wrong);
    return wrong != 0;
}
