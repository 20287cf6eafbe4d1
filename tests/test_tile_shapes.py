"""The brick shapes of the LDS-tile forms (dd_tile_shape.h), compiled as they are by the host compiler, over
every L that a lattice may have (T L^3 144 < 2^31 allows L up to 195 at T = 2): an accepted shape covers the
field, and its sites and halo rows fit what a workgroup stages.  Where no brick fits the form is refused, so
that the launch keeps to the time sweep.
"""
import ctypes
import os
import subprocess

import pytest

from conftest import ROOT

CSRC = os.path.join(ROOT, "paper_1612_06424_amd", "csrc")
NTS = (1, 2, 3, 5, 7, 16, 64)
SRC = """
#include "dd_tile_shape.h"
extern "C" {
void eo_shape(int L, int nt, int* s) { dd::EoTile t = dd::eo_tile_shape(L, nt);
    int v[7] = {t.rt, t.ry, t.rz, t.ntt, t.nty, t.ntz, t.tb}; for (int k = 0; k < 7; k++) s[k] = v[k]; }
void dslash_shape(int L, int nt, int* s) { dd::EoTile t = dd::dslash_tile_shape(L, nt);
    int v[7] = {t.rt, t.ry, t.rz, t.ntt, t.nty, t.ntz, t.tb}; for (int k = 0; k < 7; k++) s[k] = v[k]; }
int eo_ok(int L, int nt) { return dd::eo_tile_ok(L, nt); }
int dslash_ok(int L, int nt, int bytes) { return dd::dslash_tile_ok(L, nt, (size_t)bytes); }
int dslash_form(int L, int nt, int ncol, int bytes, int timed, int sums) {
    return dd::dslash_tile_form(L, nt, ncol, (size_t)bytes, timed != 0, sums != 0); }
int eo_form(int L, int nt, int ncol, int bytes) { return dd::eo_tile_form(L, nt, ncol, (size_t)bytes); }
int eo_cols(int L, int nt, int ncol) { return dd::eo_tile_cols(L, nt, ncol); }
void limits(int* s) { s[0] = dd::kTileSites; s[1] = dd::kDslSites; s[2] = dd::kDslHalo; }
}
"""


@pytest.fixture(scope="module")
def shapes(tmp_path_factory):
    d = tmp_path_factory.mktemp("tile")
    (d / "s.cpp").write_text(SRC)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-shared", "-fPIC", "-I", CSRC, str(d / "s.cpp"),
                           "-o", str(d / "s.so")])
    return ctypes.CDLL(str(d / "s.so"))


def _shape(fn, L, nt):
    s = (ctypes.c_int * 7)()
    fn(L, nt, s)
    return list(s)


def _check(shape, L, length, nt, sites, halo):
    rt, ry, rz, ntt, nty, ntz, tb = shape
    assert min(rt, ry, rz, tb) >= 1 and max(ry, rz) <= L and rt <= nt
    assert rt * ry * rz * length <= sites, "more sites than threads"
    rows = (2 * rz if ry < L else 0) + (2 * ry if rz < L else 0)
    assert rt * rows * length <= halo, "halo sites that are not staged"
    for n, r, ext in ((ntt, rt, nt), (nty, ry, L), (ntz, rz, L)):
        assert (n - 1) * r < ext <= n * r, "the bricks cover the extent, each with a row of it"


def test_accepted_shapes_fit_and_the_others_are_refused(shapes):
    lim = (ctypes.c_int * 3)()
    shapes.limits(lim)
    sites_eo, sites, halo = lim
    for L in range(2, 196):
        for nt in NTS:
            if nt * L ** 3 * 144 >= 2 ** 31:
                continue
            if L % 2 == 0:
                ok = bool(shapes.eo_ok(L, nt))
                assert ok == (L <= 128), (L, nt)  # one row has four halo rows of L / 2 sites, 256 are staged
                if ok:
                    _check(_shape(shapes.eo_shape, L, nt), L, L // 2, nt, sites_eo, sites_eo)
                else:
                    assert _shape(shapes.eo_shape, L, nt) == [0] * 7
            for nbytes in (4, 8):
                ok = bool(shapes.dslash_ok(L, nt, nbytes))
                assert ok == (L <= 64 and 24 * nbytes * nt * L ** 3 < 2 ** 31), (L, nt)
            s = _shape(shapes.dslash_shape, L, nt)
            if L <= 64:
                _check(s, L, L, nt, sites, halo)
            else:
                assert s == [0] * 7


def test_the_stencil_takes_the_form_only_where_it_fits(shapes):
    """The rule that picks the form (by sizes alone) over every L, on both sides of the timing's threshold."""
    taken = 0
    for L in range(2, 196):
        for nt in NTS:
            if nt * L ** 3 * 144 >= 2 ** 31:
                continue
            for nbytes in (4, 8):
                for ncol in (1, 2, 4, 6, 12, 48):
                    timed = nt * L ** 3 * ncol >= 2 ** 18
                    for sums in (0, 1):
                        if shapes.dslash_form(L, nt, ncol, nbytes, int(timed), sums):
                            assert shapes.dslash_ok(L, nt, nbytes), (L, nt, ncol, nbytes)
                            taken += 1
                    # launches with sums never take it where those without do not
                    assert (shapes.dslash_form(L, nt, ncol, nbytes, int(timed), 1)
                            <= shapes.dslash_form(L, nt, ncol, nbytes, int(timed), 0))
    assert taken > 0


def test_the_untimed_half_hop_takes_the_form_only_where_it_fits(shapes):
    """FP32: in one round of at most 256 workgroups; FP64: in 256 bricks or more."""
    taken = {4: 0, 8: 0}
    for L in range(2, 196, 2):
        for nt in NTS:
            if nt * L ** 3 * 144 >= 2 ** 31:
                continue
            for ncol in (1, 2, 3, 5, 12):
                for nbytes in (4, 8):
                    if not shapes.eo_form(L, nt, ncol, nbytes):
                        continue
                    taken[nbytes] += 1
                    assert shapes.eo_ok(L, nt)
                    s, kc = _shape(shapes.eo_shape, L, nt), shapes.eo_cols(L, nt, ncol)
                    bricks = s[3] * s[4] * s[5]
                    assert 1 <= kc <= ncol
                    if nbytes == 4:
                        assert bricks * -(-ncol // kc) <= 256
                        assert kc == 1 or bricks * -(-ncol // (kc - 1)) > 256, "as many workgroups as fit"
                    else:
                        assert bricks >= 256 and ncol >= 4 and kc == ncol
    assert min(taken.values()) > 0
