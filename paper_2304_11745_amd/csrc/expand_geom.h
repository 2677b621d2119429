// Geometry of expand_dw_kernel's launches (host code): how an image is cut into bands, what a workgroup keeps in LDS.
#pragma once
#include <algorithm>
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

// Whether the pair (whole operators; the executor has checked their kinds, strides and alignment) runs as one launch: while what it forms,
// counted as products (the halo and the rest of the last tiles included) times how often a position is formed, stays below a bound, since that
// grows faster than what two launches take.  Us two launches / one, by that count in 1e9: 3x3 one image 28x28 40->240 (0.13) 5.6 / 4.3, 8 images 28x28
// 40->240 (1.1) 7.9 / 6.6, 14x14 96->576 (0.3) 6.7 / 5.9, 32 images 7x7 160->960 (0.8) 9.5 / 8.1; 16 images 28x28 40->240 (1.2, more
// workgroups than fit at once) 10.0 / 11.0, 32 images (2.4) 16.5 / 18.4, 4 images 28x28 160->480 (2.6) 9.3 / 12.7, 8 images 14x14 192->768 (2.8) 9.2 / 10.5.
// 5x5 one image 14x14 112->672 (0.4) 5.9 / 5.0, 8 images (1.8, bands of four rows) 9.7 / 7.1, 8 images 28x28 40->120 (1.2) 7.8 / 7.0; 16 images
// (2.4) 9.6 / 10.3, 8 images 28x28 80->160 (4.2, bands of one row) 8.9 / 12.9, 32 images 7x7 256->256 (17, likewise) 8.0 / 16.4.  Of 4290 pairs of 1 to 64
// images the rule takes 3949, 56 of which are more than 3 % slower as one launch (by 17 % at most); a bound on the operators' own products had taken 250
// of those, up to twice as slow.  Images wider than 28 pixels only where a launch leaves units idle (one image 112x112 16->96 6.50 / 5.92, 8 images 13.9 / 14.4,
// 32 images 34.7 / 39.3), with 5x5 windows not at all (one image 56x56 24->72 5.86 / 6.28).
inline bool expand_dw_takes(const GemmArgs &g, const StreamArgs &d)
{
    if (g.dtype != DT_BF16) return false;
    const ExpandGeom e = expand_geometry(g, d);
    if (e.lds > ExpandGeom::LDS_MAX || (int64_t)(d.n_hi - d.n_lo) * e.bands * e.blocks > 1 << 24) return false;
    const double formed = (double)e.workgroups * e.tiles * 32 * 32 * (e.k_blocks * e.rowb), again = (double)e.bands * e.tiles * 32 / ((double)d.H * d.W);
    const double count = formed * again;
    if (d.k == 3) return count <= 1.5e9 && e.workgroups <= 256 * (d.W > 28 ? 1 : std::min(8, 160 * 1024 / e.lds));
    if (d.W > 28 || count <= 1e8) return d.W <= 28;
    return e.rows >= 2 && d.W > 4 && count <= (d.W <= 16 && e.rows >= 4 ? 2e9 : d.stride == 1 ? 1.3e9 : d.W <= 16 ? 5e8 : 3e8);
}

}  // namespace gacer
