// Geometry of conv3_kernel's operators (host code): which convolutions it takes and how their positions are tiled.
#pragma once
#include "device_util.h"
#include "kernels.h"

namespace gacer {

static constexpr int CONV3_BM = 256;           // output positions per tile
static constexpr int CONV3_ROWS = 384;         // input pixels (LDS rows) staged per tile and channel block

struct Conv3Geom {
    int tw, strips;            // the image is cut into `strips` column strips of `tw` (the last one may be narrower)
    int rows, row_lo;          // image rows (images x H) of the launch, and the first of them in the tensor
    int tiles_strip;           // tiles of CONV3_BM positions per strip, positions counted row by row through all images
    int tiles_m, tiles_n, n_major;
    unsigned div_tw[2], div_tw2[2], div_h[2], div_strip[2], div_tiles_m[2], div_tiles_n[2];
};

// Columns per strip: at most 56, so that 256 consecutive positions and their halo are at most CONV3_ROWS pixels.
inline int conv3_strip(int W) { const int n = (W + 55) / 56; return (W + n - 1) / n; }

// Workgroup tiles 128 channels wide unless 64 leave less of the last tile empty.
inline int conv3_bn(int N) { return (N + 127) / 128 * 128 <= (N + 63) / 64 * 64 ? 128 : 64; }

// Whether the operator (its UNSPLIT shape, so that every chunk of it adds in the same order) runs on conv3_kernel: from about
// three workgroups on four compute units; below, smaller tiles fill the chip better.  At 196 workgroups, microseconds on the
// tiled kernels / here: 16 images 28x28 512->512 84.1 / 71.4, 8 images 56x56 128->256 29.9 / 27.3, 16 images 56x56 64->64
// 14.4 / 11.4.
inline bool conv3_takes(const GemmArgs &a)
{
    if (a.dtype != DT_BF16 || a.kh != 3 || a.kw != 3 || a.stride != 1 || a.pad != 1 || a.Cin % 64 || a.b_trans || a.pre_scale) return false;
    if (a.Ho != a.H || a.Wo != a.W || a.zb * a.zh != 1 || a.z_lo || a.x_pix % 8 || a.x_img != (int64_t)a.H * a.W * a.x_pix) return false;
    if (((uintptr_t)a.x | (uintptr_t)a.w) & 15) return false;
    const int tw = conv3_strip(a.W), down = (tw + CONV3_BM - 2) / tw;           // rows that 256 positions reach down at most
    if (CONV3_BM + 2 + 2 * down + 2 * (tw + 2) > CONV3_ROWS) return false;      // images under 5 pixels wide
    const int N = a.n_hi - a.n_lo, bn = conv3_bn(N);
    const int64_t positions = (int64_t)((a.m_hi - a.m_lo) / a.W) * tw, strips = (a.W + tw - 1) / tw;
    return N > 32 && strips * ((positions + CONV3_BM - 1) / CONV3_BM) * ((N + bn - 1) / bn) >= 180;
}

}  // namespace gacer
