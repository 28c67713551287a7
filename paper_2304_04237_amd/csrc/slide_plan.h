// Host-side planning that needs nothing but the sizes: no HIP header, so that a plan can be checked for
// every size on a machine without a GPU.
#pragma once
#include <stddef.h>

namespace slide {

constexpr size_t CU_LDS_BYTES = 160 * 1024;                    // of a compute unit

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

// blocks of 256 pixels where those give every compute unit two; the dk/dv kernel: and two fit its LDS (maps of a
// few columns have tall runs with much halo).  Else 64 pixels whose channels eight (dk/dv: four) waves share
inline bool pixel_few(int B, int heads, int H, int W) { return ((long)H * W + 255) / 256 * heads * B < 512; }
inline bool dkdv_few(int B, int heads, int H, int W, int ks, int element_bytes)
{
    if (((long)H * W + 255) / 256 * heads * 2 * B < 512) return true;
    const Block b = dkdv_block(ks, element_bytes, false);
    return dkdv_lds(plan_cut(H, W, ks, b), ks, element_bytes, b) > CU_LDS_BYTES / 2;
}

}  // namespace m32
}  // namespace slide
