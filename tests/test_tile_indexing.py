"""The index arithmetic of the LDS-tile forms (dd_tile_shape.h), compiled as it is by the host compiler and walked
brick by brick: every site of the field is in exactly one brick, every brick has a slot of its own, and what a site
reads as its x, y and z neighbours is a staged entry (a site of the brick or one of the halo entries that the
workgroup loads) holding that neighbour.

Stencil (whole rows) for L = 2..64, half hop (rows of one parity, both parities) for even L = 2..128, with one
slice, few and many.  The workgroups' staging is restated here: site entries i < 128 (256 in the half hop), halo
entries up to 256 behind them.
"""
import ctypes
import os
import subprocess

import pytest

from conftest import ROOT

CSRC = os.path.join(ROOT, "paper_1612_06424_amd", "csrc")
SRC = r"""
#include <vector>
#include "dd_tile_shape.h"
using namespace dd;
// 0, or a number that names the check that failed; slip plants a mistake in what is staged
extern "C" int walk(int L, int nt, int half, int slip) {
    const int len = half ? L / 2 : L, NS = half ? kTileSites : kDslSites, NH = half ? kTileSites : kDslHalo;
    const EoTile ts = half ? eo_tile_shape(L, nt) : dslash_tile_shape(L, nt);
    if (!tile_fits(ts)) return 1;
    const int nblk = eo_tile_blocks(ts), nsite = nt * L * L * len;
    std::vector<int> seen(nsite, 0), slot(nblk, 0), staged;
    for (int lin = 0; lin < nblk; lin++) {
        const Brick b = tile_brick(ts, lin, L, nt);
        if (b.blk < 0 || b.blk >= nblk || slot[b.blk]++) return 2;
        const int n = b.RT * b.RZ * b.RY * len, nhalo = halo_rows(b, L) * b.RT * len;
        if (b.RT < 1 || b.RZ < 1 || b.RY < 1 || n > NS || nhalo > NH) return 3;
        staged.assign(NS + NH, -1);
        for (int i = 0; i < n; i++) {
            const BrickSite s = brick_site(b, len, i);
            const int t = b.t0 + s.rt, z = b.z0 + s.rz, y = b.y0 + s.ry;
            if (t >= nt || z >= L || y >= L || s.x >= len) return 4;
            staged[i] = ((t * L + z) * L + y) * len + s.x;
            if (seen[staged[i]]++) return 5;
        }
        for (int k = 0; k < NH; k++) {
            const HaloSite h = halo_site(b, L, len, k);
            if (h.t < 0 || h.t >= nt || h.z < 0 || h.z >= L || h.y < 0 || h.y >= L || h.x < 0 || h.x >= len) return 6;
            if (k < nhalo) staged[NS + k] = ((h.t * L + h.z) * L + h.y) * len + h.x;
        }
        if (slip == 1 && nhalo > 1) staged[NS + nhalo - 1] = staged[NS];
        if (slip == 2 && n > 1) staged[0] = staged[1];
        for (int i = 0; i < n; i++) {
            const BrickSite s = brick_site(b, len, i);
            const int t = b.t0 + s.rt, z = b.z0 + s.rz, y = b.y0 + s.ry;
            auto at = [&](int zz, int yy, int xx) { return ((t * L + (zz + L) % L) * L + (yy + L) % L) * len + xx; };
            const BrickYZ yz = brick_yz(b, s, L, len, NS, i);
            for (int e : {yz.ym, yz.yp, yz.zm, yz.zp})
                if (e < 0 || e >= NS + NH) return 7;
            if (staged[yz.ym] != at(z, y - 1, s.x) || staged[yz.yp] != at(z, y + 1, s.x)) return 8;
            if (staged[yz.zm] != at(z - 1, y, s.x) || staged[yz.zp] != at(z + 1, y, s.x)) return 9;
            for (int bo = 0; bo < (half ? 2 : 1); bo++) {
                const BrickX xx = half ? brick_x_half(s, len, bo) : brick_x(s, len);
                if (xx.xm < 0 || xx.xm >= n || xx.xp < 0 || xx.xp >= n) return 10;
                // half rows: the site is at x = 2 s.x + bo, entry x' of the other parity at 2 x' + 1 - bo
                const int x = half ? 2 * s.x + bo : s.x, xm = (x + L - 1) % L, xp = (x + 1) % L;
                if (staged[xx.xm] != at(z, y, half ? xm / 2 : xm) || staged[xx.xp] != at(z, y, half ? xp / 2 : xp))
                    return 11;
            }
        }
    }
    for (int s : seen)
        if (s != 1) return 12;
    return 0;
}
"""


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    d = tmp_path_factory.mktemp("walk")
    (d / "s.cpp").write_text(SRC)
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-shared", "-fPIC", "-I", CSRC, str(d / "s.cpp"),
                           "-o", str(d / "s.so")])
    return ctypes.CDLL(str(d / "s.so")).walk


def test_stencil_bricks(walk):
    for L in range(2, 65):
        for nt in (1, 2, 5, 11) if L <= 32 else (1, 3):
            assert walk(L, nt, 0, 0) == 0, (L, nt)


def test_half_hop_bricks(walk):
    for L in range(2, 129, 2):
        for nt in (1, 2, 5, 11) if L <= 32 else (1, 3):
            assert walk(L, nt, 1, 0) == 0, (L, nt)


@pytest.mark.parametrize("half", [0, 1])
def test_many_slices(walk, half):
    for L, nt in ((2, 64), (4, 64), (6, 33), (8, 37), (16, 40)):
        assert walk(L, nt, half, 0) == 0, (L, nt)


def test_rows_too_long_for_a_brick(walk):
    assert walk(65, 2, 0, 0) == 1 and walk(130, 2, 1, 0) == 1


@pytest.mark.parametrize("half", [0, 1])
@pytest.mark.parametrize("slip", [1, 2])
def test_a_wrong_entry_is_caught(walk, half, slip):
    assert walk(16, 3, half, slip) != 0 and walk(32, 2, half, slip) != 0
