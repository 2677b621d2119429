// Geometry of conv3_kernel's operators (host code): which convolutions it takes and how a launch is tiled.
#pragma once
#include "device_util.h"
#include "kernels.h"

namespace gacer {

// Output positions per tile: 256 or 128.  Input pixels (LDS rows) staged for them per channel block:
constexpr int conv3_rows(int bm) { return bm == 256 ? 384 : 256; }
static constexpr int CONV3_STRIP = 56;         // most columns of a strip

// Whether bm consecutive positions of a strip and their one-pixel halo fit: the last of them lies at most `down` image rows
// below the first, each of which adds two pixels of padding, and the taps reach two padded rows and two pixels further.
constexpr bool conv3_fits(int tw, int bm)
{
    const int down = (tw + bm - 2) / tw;
    return bm + 2 + 2 * down + 2 * (tw + 2) <= conv3_rows(bm);
}
constexpr bool conv3_fits_all(int tw_lo, int tw_hi, int bm)
{
    for (int tw = tw_lo; tw <= tw_hi; ++tw)
        if (!conv3_fits(tw, bm)) return false;
    return true;
}
static constexpr int CONV3_STRIP_MIN = 5;      // images under 5 pixels wide have too many rows in a tile of 256
static_assert(conv3_fits_all(CONV3_STRIP_MIN, CONV3_STRIP, 256) && conv3_fits_all(CONV3_STRIP_MIN, CONV3_STRIP, 128), "LDS rows");

struct Conv3Geom {
    int tw, strips;            // the image is cut into `strips` column strips of `tw` (the last one may be narrower)
    int rows, row_lo;          // image rows (images x H) of the launch, and the first of them in the tensor
    int tiles_strip;           // tiles of bm positions per strip, positions counted row by row through all images
    int tiles_m, tiles_n, n_major;
    unsigned div_tw[2], div_tw2[2], div_h[2], div_strip[2], div_tiles_m[2], div_tiles_n[2];
};

// Columns per strip
inline int conv3_strip(int W) { const int n = (W + CONV3_STRIP - 1) / CONV3_STRIP; return (W + n - 1) / n; }

// Workgroup tiles 128 channels wide unless 64 leave less of the last tile empty.
inline int conv3_bn(int N) { return (N + 127) / 128 * 128 <= (N + 63) / 64 * 64 ? 128 : 64; }

// Workgroups of a launch with tiles of bm positions x bn channels
inline int64_t conv3_wgs(const GemmArgs &a, int bm, int bn)
{
    const int tw = conv3_strip(a.W);
    const int64_t positions = (int64_t)((a.m_hi - a.m_lo) / a.W) * tw, strips = (a.W + tw - 1) / tw;
    return strips * ((positions + bm - 1) / bm) * ((a.n_hi - a.n_lo + bn - 1) / bn);
}

// Whether the operator (its UNSPLIT shape, so that every chunk of it adds in the same order) runs on conv3_kernel: from about
// three tiles of 256 positions on four compute units.  One launch in a chain, microseconds on the tiled kernels / here, by the number of
// such tiles: 196 (16 images 28x28 512->512) 75.6 / 57.4, (8 images 56x56 128->256) 25.7 / 20.6, (4 images 112x112 64->128) 18.5 / 14.5,
// (16 images 56x56 64->64) 12.6 / 10.5.  The limit is where it was before the epilogue of both became shorter; today the crossing lies at
// about 100: 147 (12 images 56x56 64->64) 10.8 / 9.9, 100 (8 images 28x28 512->512) 38.3 / 37.7, 98 (4 images 56x56 256->256)
// 23.0 / 22.3, (8 images 56x56 64->64) 8.7 / 7.6, 68 (3 images 75x75 128->128) 12.9 / 13.6, 52 (4 images 28x28 512->512) 27.2 / 28.6,
// 50 (2 images 56x56 256->256) 16.0 / 17.0.  Chunks of the operators taken (measured with longer epilogues): half of the images or of the
// channels 42.2 / 36.2 (8 images 28x28 512->512), a quarter 28.1 / 27.0 (4 images) and 28.4 / 32.4 (128 channels), an eighth
// 20.4 / 22.8 (2 images); 2 images 56x56 256->256 16.4 / 15.1.
inline bool conv3_takes(const GemmArgs &a)
{
    if (a.dtype != DT_BF16 || a.kh != 3 || a.kw != 3 || a.stride != 1 || a.pad != 1 || a.Cin % 64 || a.b_trans || a.pre_scale) return false;
    if (a.Ho != a.H || a.Wo != a.W || a.zb * a.zh != 1 || a.z_lo || a.x_pix % 8 || a.x_img != (int64_t)a.H * a.W * a.x_pix) return false;
    if (((uintptr_t)a.x | (uintptr_t)a.w) & 15) return false;
    if (conv3_strip(a.W) < CONV3_STRIP_MIN) return false;
    const int N = a.n_hi - a.n_lo;
    return N > 32 && conv3_wgs(a, 256, conv3_bn(N)) >= 180;
}

// Tile of one launch, chunks of a decomposed operator included (the tile never changes an element's order of additions).
// 256 x 128 moves the fewest bytes per MFMA once there are well over one such tile per compute unit; 256 x 64 while those reach
// half of the units; 128 x 64 below.  One launch alone, microseconds of 256x128 / 256x64 / 128x64, by the number of 256x128 tiles:
// 50 (2 images 56x56 256->256) 33.4 / 19.1 / 15.1, 100 (8 images 28x28 512->512) 59.7 / 36.2 / 37.1, 196 (16 of those) 66.3 / 57.0 /
// 71.6, 358 (16 images 75x75 128->128) 35.9 / 32.5 / 38.3, 392 (16 images 56x56 256->256) 59.7 / 62.7 / 74.4, 784 (32 of those)
// 114.6 / 109.8 / 134.4, 1568 (32 images 112x112 64->128) 77.2 / 78.3 / 93.7.  By the number of 256x64 tiles at 64 channels: 98 (8
// images 56x56) 10.4 / 7.9, 196 (16) 12.2 / 9.8, 264 (3 images 150x150) 14.1 / 15.3, 392 (32 images 56x56) 16.0 / 18.1.
// Alone, 128 x 64 gains up to 256 tiles, but other tenants use the units that a launch leaves: the round of VGG-16, 8 images, halved
// along the batch, ResNet-50, 16 images, halved along the channels, and MobileNetV3, 32 images, takes 1760 us with 128 x 64 below 256
// tiles, 1730 below 128 and 1717 with 256 x 128 throughout (which alone costs that VGG 864 instead of 775, in quarters 1436
// instead of 1183).
struct Conv3Tile { int bm, bn; };
inline Conv3Tile conv3_tile(const GemmArgs &a)
{
    if (conv3_bn(a.n_hi - a.n_lo) == 128 && conv3_wgs(a, 256, 128) > 360) return {256, 128};
    return {conv3_wgs(a, 256, 64) >= 128 ? 256 : 128, 64};
}

}  // namespace gacer
