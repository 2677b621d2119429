// Geometry of expand_dw_kernel's launches (host code): how an image is cut into bands, what a workgroup keeps in LDS.
#pragma once
#include "kernels.h"

namespace gacer {

struct ExpandGeom {
    static constexpr int TW = 2;                   // depthwise outputs of a row that a thread forms together
    static constexpr int LDS_MAX = 53 * 1024;      // three workgroups on a unit
    static constexpr int PROW = 32 * 2 + 16;       // LDS bytes of a position's 32 channels
    int rowb, k_blocks;                            // bytes of a K block per row, blocks
    int rows, bands, blocks, tiles;                // output rows per band, bands, blocks of 32 channels, tiles of 32 positions per band
    int mid_at, lds, workgroups;                   // LDS offset of the pointwise result, LDS bytes
};

// A band of `rows` output rows and its LDS
inline void expand_band(ExpandGeom &e, const StreamArgs &d, int rows)
{
    const int in_rows = (rows - 1) * d.stride + d.k, held = in_rows < d.H ? in_rows : d.H;
    e.rows = rows;
    e.bands = (d.Ho + rows - 1) / rows;
    e.tiles = (held * d.W + 31) / 32;
    e.mid_at = e.k_blocks * (e.tiles * 32 + 32) * e.rowb;
    // the second output of a thread's pair may lie beyond the row: its window is read (and not used) up to stride columns further
    e.lds = e.mid_at + (in_rows * (d.W + 2 * (d.k / 2)) + d.stride) * ExpandGeom::PROW;
}

// Bands are halved while LDS does not hold them, and while there are few workgroups: with fewer than two per unit down to a tile per
// wave, with fewer than one on half of the units further (one image 14x14 64->384, 7 / 4 rows: 4.87 / 4.28 us, 28x28 32->192 5.23 / 4.19).
inline ExpandGeom expand_geometry(const GemmArgs &g, const StreamArgs &d)
{
    ExpandGeom e;
    const int k_bytes = g.K * 2;
    e.rowb = (k_bytes + 63) / 64 * 64 < (k_bytes + 127) / 128 * 128 ? 64 : 128;
    e.k_blocks = (k_bytes + e.rowb - 1) / e.rowb;
    e.blocks = (d.C + 31) / 32;
    expand_band(e, d, d.Ho);
    auto wgs = [&]() { return (int64_t)(d.n_hi - d.n_lo) * e.bands * e.blocks; };
    while (e.rows > 1 && (e.lds > ExpandGeom::LDS_MAX || (e.rows > 2 && ((wgs() < 512 && e.tiles > 4) || (wgs() < 128 && e.tiles > 3))))) expand_band(e, d, (e.rows + 1) / 2);
    e.workgroups = (int)wgs();
    return e;
}

// Whether the pair (whole operators; the executor has checked their kinds, strides and alignment) runs as one launch.  Measured as above
// the kernel, two launches / one: images up to 28 pixels wide gain while the wide tensor times the bytes of K stays under about 5e8 (32
// images 7x7 160->960 9.48 / 8.04, 14x14 80->480 11.0 / 11.1, 96->576 11.6 / 12.3), 5x5 windows under 2.5e8 (8 images 14x14 112->672
// 9.67 / 7.24, 32 images 16.7 / 17.8); wider ones only where a launch leaves units idle (one image 112x112 16->96 6.50 / 5.92, 8 images
// 13.9 / 14.4, 32 images 34.7 / 39.3), with 5x5 windows not at all (one image 56x56 24->72 5.86 / 6.28).
inline bool expand_dw_takes(const GemmArgs &g, const StreamArgs &d)
{
    if (g.dtype != DT_BF16) return false;
    const ExpandGeom e = expand_geometry(g, d);
    if (e.lds > ExpandGeom::LDS_MAX || (int64_t)(d.n_hi - d.n_lo) * e.bands * e.blocks > 1 << 24) return false;
    const int64_t work = (int64_t)(d.n_hi - d.n_lo) * d.H * d.W * d.C * g.K * 2;
    if (d.W > 28) return d.k == 3 && e.workgroups <= 256;
    return work <= (d.k == 3 ? 500000000 : 250000000);
}

}  // namespace gacer
