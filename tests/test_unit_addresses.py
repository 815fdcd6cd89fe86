"""Every byte that a launch of the kernel without staging asks for, walked on the host through the index arithmetic that the
kernel itself is compiled from (csrc/unit_index.h): inside its buffer, or an offset that the hardware drops."""
import subprocess

import pytest

from paper_2006_09791_amd import build
from paper_2006_09791_amd import workloads as wl

S = wl.ConvShape
SHAPES = [
    # N Cin H W Cout KH KW stride pad groups
    S(1, 64, 32, 32, 64, 3, 3, 1, 1, 4),
    S(1, 1024, 4, 4, 16, 1, 1, 1, 0, 1),      # one tile, 64 KB of filters
    S(1, 16, 1, 3, 16, 3, 3, 1, 1, 1),
    S(3, 70, 9, 5, 33, 3, 3, 1, 1, 1),        # padded channels and filters
    S(5, 60, 29, 37, 84, 3, 3, 1, 1, 3),
    S(2, 50, 9, 7, 24, 1, 1, 2, 0, 1),
    S(1, 4, 9, 7, 16, 3, 3, 1, 1, 1),         # waves that share the only channel block
    S(1, 23, 10, 9, 17, 3, 3, 2, 1, 1),
    S(71, 8, 3, 3, 12, 3, 3, 1, 1, 1),        # tiles that span images
    S(45, 48, 1, 3, 40, 1, 1, 1, 0, 1),
    S(3, 24, 6, 5, 24, 3, 3, 2, 1, 2),
]

PROGRAM = r"""
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "unit_index.h"
using namespace gspc;

static long bad;
// An access of size bytes at the lane's offset vo and the scalar offset so.
static bool inside(unsigned vo, unsigned so, unsigned size, unsigned bytes) { return (unsigned long long)vo + so + size <= bytes; }
// (and no word of a dropped access may lie past 2^32, where its offset would be small again)
static bool dropped(unsigned vo, unsigned size, unsigned bytes) { return vo >= bytes && (unsigned long long)vo + size <= 1ull << 32; }

template <int K, int S> void walk(const TileUnit &t, int nw) {
    constexpr int KR = K == 3 ? 3 : 1, UB = K == 3 ? 2 : 4;
    constexpr unsigned WLANE = K == 3 ? 12 : 16, XSIZE = K == 3 ? 12 : 4;
    std::vector<char> seen(t.tiles);                              // every tile is some block's, once
    for (unsigned block = 0; block < unit_blocks(t); ++block) {
        const UnitTileAt a = unit_tile(t, block);
        const unsigned id = (a.j * t.mtiles + a.mt) * t.px_tiles + a.px;
        bad += a.px >= t.px_tiles || a.mt >= (unsigned)t.mtiles || id >= t.tiles || seen[id]++;
    }
    for (unsigned block = 0; block < unit_blocks(t); ++block)
        for (int wave = 0; wave < nw; ++wave) {
            const UnitTileAt tile = unit_tile(t, block);
            const UnitWave w = t.parts > 1 ? unit_share(t, wave) : UnitWave{wave, 7};
            const unsigned base = unit_w_base<KR, WLANE>(t, tile), step = unit_w_step<KR, WLANE>(t);
            for (int n = 0, u = w.first; n < UB || u < t.blocks; ++n, u += nw)
                for (int k = 0; k < KR; ++k)
                    for (unsigned lane = 0; lane < 64; ++lane) {
                        const bool on = w.rows >> k & 1;
                        const unsigned vo = unit_w_lane<WLANE>(t, u, on, lane), so = base + u * step + k * 64 * WLANE;
                        bad += u < t.blocks && on ? !inside(vo, so, WLANE, t.w_bytes) : !dropped(vo, WLANE, t.w_bytes);
                    }
            for (unsigned lane = 0; lane < 64; ++lane) {
                const unsigned lg = lane / 16, q = tile.px * 16 + lane % 16;
                const UnitPixel pix = unit_pixel<K, S>(t, tile, lane % 16);
                const int n = q / t.HWo, oh = q % t.HWo / t.Wout, ow = q % t.Wout;   // what the definition reads
                for (int r = 0, u = w.first; r < UB || u < t.blocks; ++r, u += nw)
                    for (int e = 0; e < (K == 3 ? 3 : 4); ++e) {
                        const int k = K == 3 ? e : 0, c = K == 3 ? u * 4 : u * 16 + 4 * e;
                        const bool on = w.rows >> k & 1;
                        const unsigned row = unit_x_row<K>(t, tile, pix, lg, k, on), vo = unit_x_lane(t, row, lg, c), so = c * t.H * t.W * 4;
                        const int ih = oh * S - K / 2 + k, ch = c + (int)lg, col = K == 3 ? std::min(std::max(ow * S - 1, 0), t.W - 3) : ow * S;
                        if (q < t.npix && on && ch < t.CPG && ih >= 0 && ih < t.H) {
                            const unsigned want = (((n * t.Cin + tile.j * t.CPG + ch) * t.H + ih) * t.W + col) * 4;
                            bad += !inside(vo, so, XSIZE, t.x_bytes) || vo + so != want;
                        } else {
                            bad += !dropped(vo, XSIZE, t.x_bytes);
                        }
                    }
            }
        }
}

int main(int, char **a) {
    int v[10];
    for (int i = 0; i < 10; ++i) v[i] = std::atoi(a[1 + i]);
    const int K = v[5], S = v[7], pad = v[8], groups = v[9], Ho = (v[2] + 2 * pad - K) / S + 1, Wo = (v[3] + 2 * pad - K) / S + 1;
    TileUnit t{};
    unit_layer(t, v[0], v[1], v[2], v[3], v[4], groups, K, Ho, Wo, (v[4] / groups + 15) / 16);
    t.w_bytes = (unsigned)(groups * t.blocks * t.mtiles) * (K == 3 ? 2304 : 1024);
    for (int nw = 2; nw <= 16; nw *= 2)
        for (t.parts = 1; t.parts <= (K == 3 && nw >= 2 * t.blocks ? std::min(nw / t.blocks, 3) : 1); ++t.parts)
            K == 3 ? S == 1 ? walk<3, 1>(t, nw) : walk<3, 2>(t, nw) : S == 1 ? walk<1, 1>(t, nw) : walk<1, 2>(t, nw);
    std::printf("%ld\n", bad);
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("unit")
    (d / "walk.cpp").write_text(PROGRAM)
    exe = str(d / "walk")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", build.CSRC, str(d / "walk.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("s", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_every_address_is_inside_or_dropped(program, s):
    out = subprocess.run([program] + [str(v) for v in s], check=True, capture_output=True, text=True).stdout
    assert int(out) == 0
