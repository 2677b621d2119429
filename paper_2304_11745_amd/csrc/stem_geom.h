// Geometry of stem_kernel's operators (host code): which convolutions it takes and how their data lies in LDS and at the ends of its tensor.
#pragma once
#include <hip/hip_runtime.h>
#include "kernels.h"

namespace gacer {

static constexpr int STEM_BM = 128;            // output positions per workgroup and tile

struct StemGeom {
    int pairs;                 // k groups (two 16-byte chunks) per tap row: ceil(kw * Cin / (2 VEC))
    int rowb;                  // LDS bytes per weight row
    int rs, lead;              // LDS bytes per strip row; element of a strip row that holds the image row's element 0
    int shift;                 // elements by which strip chunks are displaced against the image row (bf16: makes reads even)
    int cpr;                   // chunks per strip row that hold image data
    int strip_bytes;
    int tiles_img, tiles;      // tiles per image and in the launch
};

// Fills *out for workgroups of 32 * tn channels; false when the kernel does not take the operator: input positions with gaps, or
// weights and input strip too large for half the LDS of a compute unit (with one workgroup per unit the generic gather loader
// is as fast: 64x11x11x3 fp32, 8 images, 41.8 us here, 39.4 there).
inline bool stem_geometry(const GemmArgs &a, int tn, StemGeom *out)
{
    const int VEC = a.dtype == DT_BF16 ? 8 : 4, ESZ = 16 / VEC;
    StemGeom g;
    if (a.x_pix != a.Cin || a.x_img != (int64_t)a.H * a.W * a.Cin || a.b_trans || a.zb * a.zh != 1 || a.z_lo) return false;
    const int run = a.kw * a.Cin;
    g.pairs = (run + 2 * VEC - 1) / (2 * VEC);
    g.rowb = a.kh * g.pairs * 32 + 16;                 // an odd number of 16-byte units: fragment reads of 16 rows hit all banks once
    g.lead = (a.pad * a.Cin + VEC - 1) / VEC * VEC;
    g.shift = a.dtype == DT_BF16 ? (g.lead - a.pad * a.Cin) & 1 : 0;
    g.lead += g.shift;
    const int64_t WC = (int64_t)a.W * a.Cin;
    const int64_t cpr = (WC + g.shift + VEC - 1) / VEC;
    const int64_t reach = (int64_t)((a.Wo - 1) * a.stride - a.pad + a.kw) * a.Cin;     // elements right of the image row's start that are read,
    const int64_t last = (reach > WC ? reach : WC) + 3 * VEC;                          // plus the last group's padding and the funnel's dword
    const int64_t rs = (((g.lead - g.shift) + (last > cpr * VEC ? last : cpr * VEC)) * ESZ + 31) / 16 * 16;
    const int64_t n_oh = (STEM_BM - 1 + a.Wo - 1) / a.Wo + 1, rows = ((n_oh < a.Ho ? n_oh : a.Ho) - 1) * a.stride + a.kh;
    const int64_t strip = rs * rows > 4 * 32 * 144 ? rs * rows : 4 * 32 * 144;         // also holds the epilogue patches of four waves
    if (strip + (int64_t)32 * tn * (g.rowb + 4) > 80 * 1024) return false;         // two workgroups per compute unit at least
    g.cpr = (int)cpr;
    g.rs = (int)rs;
    g.strip_bytes = (int)strip;
    g.tiles_img = (a.Ho * a.Wo + STEM_BM - 1) / STEM_BM;
    g.tiles = ((a.m_hi - a.m_lo) / (a.Ho * a.Wo)) * g.tiles_img;
    *out = g;
    return true;
}

// Whether a strip, read in chunks of 20 bytes, may reach over an end of the tensor: it holds the tensor's first row, or its last
// rows (`rows` image rows from the tensor's start) end within three chunks of the tensor's end.  Counted in elements: in bytes
// the sum does not fit an int for tensors just below the 2 GiB that a tensor may have.
__host__ __device__ inline bool stem_edge(bool first_row, int rows, int WC, int elements, int VEC)
{
    return first_row || rows * WC > elements - 3 * VEC;
}

}  // namespace gacer
