// Geometry of conv3_kernel's operators (host code): which convolutions it takes and how a launch is tiled.
#pragma once
#include "device_util.h"
#include "kernels.h"

namespace gacer {

// Output positions per tile: 256, 128 or 64.  Input pixels (LDS rows) staged for them per channel block:
constexpr int conv3_rows(int bm) { return bm == 256 ? 384 : bm == 128 ? 256 : 192; }
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
static_assert(conv3_fits_all(CONV3_STRIP_MIN, CONV3_STRIP, 256) && conv3_fits_all(CONV3_STRIP_MIN, CONV3_STRIP, 128) &&
              conv3_fits_all(CONV3_STRIP_MIN, CONV3_STRIP, 64), "LDS rows");

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

// Whether the operator (its UNSPLIT shape, so that every chunk of it adds in the same order) runs on conv3_kernel: from about three tiles
// of 128 positions x 64 channels on four compute units.  One launch in a chain, microseconds on the tiled kernels / here, by the
// number of such tiles: 392 (16 images 28x28 128->256) 20.4 / 16.3, (32 images 28x28 128->128) 14.6 / 12.2, 392 (4 images 56x56 256->256) 22.3 / 19.0, 344
// (7 images 28x28 512->512) 36.2 / 35.3, 296 (6 images) 37.2 / 33.4, 248 (5 images) 28.0 / 24.8, 200 (16 images 14x14 512->512) 25.5 / 20.7, 196 (32 images 14x14
// 256->256) 15.5 / 12.8, (16 images 28x28 128->128) 10.0 / 8.6, (8 images 56x56 64->64) 7.2 / 6.8, 108 (3 images 37x41 192->192) 9.9 / 10.1, 104 (8 images 14x14
// 512->512) 18.5 / 19.5, 100 (16 images 14x14 256->256) 11.4 / 12.1, 98 (8 images 28x28 128->128) 7.5 / 8.2.
inline bool conv3_takes(const GemmArgs &a)
{
    if (a.dtype != DT_BF16 || a.kh != 3 || a.kw != 3 || a.stride != 1 || a.pad != 1 || a.Cin % 64 || a.b_trans || a.pre_scale) return false;
    if (a.Ho != a.H || a.Wo != a.W || a.zb * a.zh != 1 || a.z_lo || a.x_pix % 8 || a.x_img != (int64_t)a.H * a.W * a.x_pix) return false;
    if (((uintptr_t)a.x | (uintptr_t)a.w) & 15) return false;
    if (conv3_strip(a.W) < CONV3_STRIP_MIN) return false;
    const int N = a.n_hi - a.n_lo;
    return N > 32 && conv3_wgs(a, 128, 64) >= 180;
}

// Tile of one launch, chunks of a decomposed operator included (the tile never changes an element's order of additions).
// 256 x 128 moves the fewest bytes per MFMA once there are well over one such tile per compute unit; 256 x 64 if 128 x 64 would leave some units
// a second tile and K is long, or if there is more than one per unit; 128 x 64 below, and 64 x 64 where those leave half of the units empty (only chunks come
// there).  One launch alone,
// microseconds of 256x128 / 256x64 / 128x64, by the number of 256x64 tiles: 98 (16
// images 28x28 128->128) 19.8 / 12.1 / 8.6, 104 (16 images 14x14 512->512) 55.7 / 29.0 / 20.7, 196 (32 images 28x28 128->128) 20.4 / 12.9 / 12.2, (64 images
// 14x14 256->256) 32.5 / 19.0 / 19.9, 200 (8 images 28x28 512->512) 57 / 32.3 / 35.7, 392 (8 images 56x56 256->256) 33.9 / 31.3 / 38.4, 784 (16 images 28x28
// 512->512) 59.3 / 57.5 / 73.2;
// at 64 channels 196 (16 images 56x56) 14.5 / 9.8 / 9.1, 392 (32 images 56x56) - / 16.0 / 18.1.  Between those, 256x64 / 128x64: K of 256 or 512 channels
// 128 (20 images 14x14 512->512, 248 tiles of 128x64) 29.5 / 24.3, 132 (42 images 14x14 256->256, 260) 18.8 / 18.7, 136 (21 images 14x14 512->512, 264) 29.8 / 32.0, 152 (24
// images) 30.2 / 33.0, 148 (48 images 14x14 256->256) 19.3 / 19.5, 176 (7 images 28x28 512->512) 31.7 / 34.6; 64 or 128 channels 148 (24 images 28x28 128->128)
// 12.7 / 12.2, 172 (14 images 56x56 64->64) 10.0 / 9.2, 222 (36 images 28x28 128->128) 13.9 / 13.9, 245 (20 images 56x56 64->64) 10.7 / 10.1, 258 (21 images) 12.5 /
// 13.6, 258 (42 images 28x28 128->128) 18.0 / 19.9.
// Operators in two or four chunks, microseconds on the tiled kernels (they would add in another
// order) / on 128x64 / on 64x64, by the 128x64 tiles of a chunk: 52 (four of 32 images 14x14 256->256) 40.0 / 46.3 / 32.8, 50 (four of 512 channels, 16 images 14x14)
// 66.6 / 77.1 / 58.3, 98 (halves of 16 images 28x28 128->128) 14.6 / 16.1 / 12.8, (8 images 56x56 64->64) 11.1 / 12.5 / 10.3, 104 (16 images 14x14 512->512)
// 33.6 / 39.0 / 31.4, 124 (20 images) 34.7 / 39.1 / 36.1, 124 (40 images 14x14 256->256) 21.3 / 24.1 / 20.9, 136 (44 images) - / 24.0 / 27.4, 148 (24 images
// 14x14 512->512) 47.6 / 39.8 / 47.9, 172 (28 images 28x28 128->128) 18.1 / 16.6 / 18.2.
// In rounds other tenants use the units that a launch leaves, so alone is not all: VGG-16, 8 images, halved along the batch, ResNet-50, 16
// images, halved along the channels, and MobileNetV3, 32 images, took 1760 us with 128 x 64 below 256 tiles, 1730 below 128 (both with two
// weight stages).
struct Conv3Tile { int bm, bn; };
inline Conv3Tile conv3_tile(const GemmArgs &a)
{
    if (conv3_bn(a.n_hi - a.n_lo) == 128 && conv3_wgs(a, 256, 128) > 360) return {256, 128};
    if (conv3_wgs(a, 128, 64) <= 128) return {64, 64};
    return {(a.Cin >= 256 ? conv3_wgs(a, 128, 64) : conv3_wgs(a, 256, 64)) > 256 ? 256 : 128, 64};
}

}  // namespace gacer
