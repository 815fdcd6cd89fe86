// What a block of conv_mfma16u works on and which bytes its lanes read.  Host and device, without a header of HIP: a test walks
// whole launches with the host's compiler and checks every offset against its buffer.
#pragma once

#include "divide.h"

namespace gspc {

// What the kernel reads, in one piece: the scalar loads of its arguments are the first link of the chain, and a second
// round of them another (so nothing is asked of the launch, such as the grid's size, that is not in here, and there is no
// hole: with a number for the host among them the loads were cut in five and 32 -> 64 on 32x32 at stride 2, g = 2, N = 64 took
// 7.00 us for 6.91).
struct TileUnit {
    const float *x, *w;
    float *y;
    const float *res;
    unsigned x_bytes, w_bytes;
    int blocks, parts;               // channel blocks: four channels, 1x1: sixteen; waves that share one (3x3)
    int mtiles, CPG, KPG, Cin, Cout; // mtiles: filter tiles per group
    int H, W, Wout;
    unsigned HWo, npix;              // Hout * Wout, N * HWo
    unsigned per_xcd, more, px_tiles;    // tiles of an XCD's blocks; XCDs that have one more; pixel tiles
    unsigned m_HWo, m_Wout, m_px, m_mt;  // reciprocals (div_magic)
    int relu;
    unsigned tiles;                      // of the launch (for the host)
};

// The geometry of a layer and its launch: K x K filters at stride S, channel blocks and filter tiles as packed.
inline void unit_layer(TileUnit &t, int N, int Cin, int H, int W, int Cout, int groups, int K, int Hout, int Wout, int mtiles) {
    t.CPG = Cin / groups;
    t.KPG = Cout / groups;
    t.blocks = K == 3 ? (t.CPG + 3) / 4 : (t.CPG + 15) / 16;
    t.mtiles = mtiles;
    t.Cin = Cin;
    t.Cout = Cout;
    t.H = H;
    t.W = W;
    t.Wout = Wout;
    t.HWo = Hout * Wout;
    t.npix = (unsigned)N * t.HWo;
    t.m_HWo = div_magic(t.HWo);
    t.m_Wout = div_magic(Wout);
    t.px_tiles = (t.npix + 15) / 16;
    t.m_px = div_magic(t.px_tiles);
    t.m_mt = div_magic(mtiles);
    t.tiles = t.px_tiles * mtiles * groups;
    t.per_xcd = t.tiles / 8;
    t.more = t.tiles % 8;
    t.x_bytes = (unsigned)N * Cin * H * W * 4;
}

// Tiles are numbered pixel tile innermost, and the blocks of one XCD (block % 8) take consecutive ones, so that few
// of the eight level-2 caches fetch a filter tile.  A launch has as many blocks as tiles: with the same number for every XCD,
// up to seven blocks had no tile, and their filters lay up to seven groups behind the buffer.
inline unsigned unit_blocks(const TileUnit &t) { return t.tiles; }
struct UnitTileAt {
    unsigned px, mt, j;              // pixel tile, filter tile of the group, group
};
GSPC_HD UnitTileAt unit_tile(const TileUnit &t, unsigned block) {
    const unsigned xcd = block & 7, id = xcd * t.per_xcd + (xcd < t.more ? xcd : t.more) + (block >> 3);
    const unsigned ft = fast_div(id, t.m_px), px = id - ft * t.px_tiles, j = fast_div(ft, t.m_mt);
    return {px, ft - j * t.mtiles, j};
}

// A wave's channel blocks are first, first + waves ..; where there are twice as many waves as blocks (3x3, t.parts) two or three
// waves share one, kernel row by kernel row (bits of rows).
struct UnitWave {
    int first, rows;
};
GSPC_HD UnitWave unit_share(const TileUnit &t, int wave) {
    const int part = wave >= 2 * t.blocks ? 2 : wave >= t.blocks ? 1 : 0;
    return {part < t.parts ? wave - part * t.blocks : t.blocks, t.parts == 3 ? 1 << part : part ? 4 : 3};
}

// Weights: [g][channel block][filter tile]([kernel row])[64 lanes][3 or 4], KR kernel rows of WLANE bytes per lane.  Scalar offset
// of the tile's first channel block, and from there to the next one; then the lane's offset in a kernel row that its wave multiplies.
template <int KR, unsigned WLANE>
GSPC_HD unsigned unit_w_base(const TileUnit &t, const UnitTileAt &a) {
    return (a.j * t.blocks * t.mtiles + a.mt) * (KR * 64 * WLANE);
}
template <int KR, unsigned WLANE>
GSPC_HD unsigned unit_w_step(const TileUnit &t) {
    return t.mtiles * (KR * 64 * WLANE);
}
template <unsigned WLANE>
GSPC_HD unsigned unit_w_lane(const TileUnit &t, int u, bool on, unsigned lane) {
    return ((u < t.blocks) & on) ? lane * WLANE : kOob;
}

// Pixel li of a tile: image, place in the output plane, first row and column of its window in the input plane, and the column
// that is loaded first.  3x3 (padding 1): the three columns are loaded from inside the row; at its left (right) end they move one
// place up (down) and a zero takes the place of the column outside.
struct UnitPixel {
    unsigned n, rem;
    int ih0, iw0, start;
    bool live;
};
template <int KH, int S>
GSPC_HD UnitPixel unit_pixel(const TileUnit &t, const UnitTileAt &a, unsigned li) {
    // (the tile's first pixel in scalar registers; a tile spans images where planes are small)
    unsigned n0 = fast_div(a.px * 16, t.m_HWo), r0 = a.px * 16 - n0 * t.HWo;
    const bool low = r0 >= t.HWo;
    n0 += low ? 1 : 0;
    r0 -= low ? t.HWo : 0;
    const unsigned dn = fast_div(r0 + li, t.m_HWo), rem = r0 + li - dn * t.HWo;
    const unsigned oh = fast_div(rem, t.m_Wout), ow = rem - oh * t.Wout;
    const int ih0 = (int)oh * S - KH / 2, iw0 = (int)ow * S - KH / 2;
    const int inside = iw0 < 0 ? 0 : iw0, last = t.W - 3;
    return {n0 + dn, rem, ih0, iw0, KH == 3 && inside > last ? last : inside, a.px * 16 + li < t.npix};
}

// Inputs: the lane's offset in row k of the window, in the group's channel lg, or kOob; and with the first channel of a load, c channels
// further by a scalar offset.  A lane's channels of a block are lg, 1x1: lg, lg + 4, lg + 8 and lg + 12; past the group's they have
// zero weights and must be zeros too (0 * inf).
template <int KH>
GSPC_HD unsigned unit_x_row(const TileUnit &t, const UnitTileAt &a, const UnitPixel &p, unsigned lg, int k, bool on) {
    const unsigned at = ((p.n * t.Cin + a.j * t.CPG + lg) * (unsigned)(t.H * t.W) + p.ih0 * t.W + p.start) * 4u + k * t.W * 4;
    return (p.live & on & ((KH == 1) | ((unsigned)(p.ih0 + k) < (unsigned)t.H))) ? at : kOob;   // (&: a choice, not branches)
}
GSPC_HD unsigned unit_x_lane(const TileUnit &t, unsigned row, unsigned lg, int c) { return c < t.CPG - (int)lg ? row : kOob; }

}  // namespace gspc
