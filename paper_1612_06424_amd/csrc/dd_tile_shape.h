// dd_tile_shape.h -- what the LDS-tile forms of the half hop (dd_eo_tile.h) and of the stencil (dd_dslash_tile.h)
// share: the brick shapes, the fields that the two forms take, and the indices of a brick's sites, halo and
// neighbours.  Integer arithmetic only, so that the host tests compile it as it is, without HIP.
#pragma once

#include <cstddef>

#ifdef __HIPCC__
#define DD_TILE_FN __host__ __device__ __forceinline__
#else
#define DD_TILE_FN inline
#endif

namespace dd {

constexpr int kTileSites = 256;            // half hop: output sites of a workgroup at most, and halo sites
constexpr int kDslSites = 128;             // stencil: sites of a workgroup at most
constexpr int kDslHalo = 2 * kDslSites;    // and halo sites

// Brick of rt x rz x ry whole x rows (time, z, y) and the numbers of bricks per extent; all zero where no
// brick fits.
struct EoTile {
    int rt, ry, rz;
    int ntt, nty, ntz;
    int tb;  // bricks of a time block (consecutive workgroups)
};

// The bricks of a field of L^3 x nt whose x rows have `len` staged sites: of the shapes whose sites
// and halo sites fit one workgroup, the one with the least workgroups and halo together (bricks at the end of an
// extent that they do not divide are cut short).  Rows too long for any (one row has four halo rows) give
// none.  A time block of 4 bricks keeps the slices that neighbouring workgroups read in one L2.
inline EoTile tile_shape(int L, int len, int nt, int sites, int halo) {
    EoTile best{0, 0, 0, 0, 0, 0, 0};
    double score = 1e30;
    for (int ry = 1; ry <= L && ry * len <= sites; ry++)
        for (int rz = 1; rz <= L && ry * rz * len <= sites; rz++) {
            const int sl = ry * rz * len, hr = ((ry < L ? 2 * rz : 0) + (rz < L ? 2 * ry : 0)) * len;
            if (hr > halo) continue;
            int rt = sites / sl;
            if (hr > 0 && halo / hr < rt) rt = halo / hr;
            if (rt > nt) rt = nt;
            const int nty = (L + ry - 1) / ry, ntz = (L + rz - 1) / rz, ntt = (nt + rt - 1) / rt;
            const double sc = (double)nty * ntz * ntt * (sites + 0.5 * hr * rt);
            if (sc < score) {
                score = sc;
                best = EoTile{rt, ry, rz, ntt, nty, ntz, 1};
            }
        }
    best.tb = best.ntt < 4 ? best.ntt : 4;
    return best;
}
inline bool tile_fits(const EoTile& t) { return t.rt > 0; }
inline int eo_tile_blocks(const EoTile& t) { return t.ntt * t.nty * t.ntz; }

// A workgroup's brick: its first slice and rows, how many there are (cut short at the ends), its slot.
struct Brick {
    int t0, y0, z0, RT, RY, RZ, blk;
};

// Workgroup -> brick: time fastest within a time block, then groups of 4 x 2 bricks in (y, z), whose halos lie
// mostly inside the group (both FP64 half hops on 16 x 32^3: 951 us row by row, 922 so; FP32 the same either way).
DD_TILE_FN Brick tile_brick(const EoTile& ts, int lin, int L, int nt) {
    const int ntile = ts.nty * ts.ntz;
    const int tbk = lin / (ts.tb * ntile);
    const int inb = lin - tbk * ts.tb * ntile;
    const int left = ts.ntt - tbk * ts.tb, tbs = ts.tb < left ? ts.tb : left;
    int tile = inb / tbs;
    const int bt = tbk * ts.tb + (inb - tile * tbs);
    if (ts.nty % 4 == 0 && ts.ntz % 2 == 0) {
        const int grp = tile >> 3, in8 = tile & 7, ng = ts.nty >> 2;
        tile = ((grp / ng) * 2 + (in8 >> 2)) * ts.nty + (grp % ng) * 4 + (in8 & 3);
    }
    Brick b;
    b.t0 = bt * ts.rt;
    b.y0 = (tile % ts.nty) * ts.ry;
    b.z0 = (tile / ts.nty) * ts.rz;
    b.RT = ts.rt < nt - b.t0 ? ts.rt : nt - b.t0;
    b.RY = ts.ry < L - b.y0 ? ts.ry : L - b.y0;
    b.RZ = ts.rz < L - b.z0 ? ts.rz : L - b.z0;
    b.blk = bt * ntile + tile;
    return b;
}

// Site i of a brick whose rows have len sites: its row in the brick (time slowest, then z, then y) and place in the row.
struct BrickSite {
    int row, x, rt, rz, ry;
};
DD_TILE_FN BrickSite brick_site(const Brick& b, int len, int i) {
    BrickSite s;
    s.row = i / len;
    s.x = i - s.row * len;
    const int rr = s.row / b.RY;
    s.ry = s.row - rr * b.RY;
    s.rt = rr / b.RZ;
    s.rz = rr - s.rt * b.RZ;
    return s;
}

// Halo rows of a slice of the brick: y0 - 1 and y0 + RY (RZ rows each), then z0 - 1 and z0 + RZ (RY rows each);
// none in a direction that the brick spans.
DD_TILE_FN int halo_rows_y(const Brick& b, int L) { return b.RY < L ? 2 * b.RZ : 0; }
DD_TILE_FN int halo_rows(const Brick& b, int L) { return halo_rows_y(b, L) + (b.RZ < L ? 2 * b.RY : 0); }

// Where halo entry k of a brick lies: slice, row and place in the row; past the last entry any site of the field.
struct HaloSite {
    int t, z, y, x;
};
DD_TILE_FN HaloSite halo_site(const Brick& b, int L, int len, int k) {
    const int hy = halo_rows_y(b, L), hrow = halo_rows(b, L);
    HaloSite h;
    int hr = k / len;
    h.x = k - hr * len;
    if (hr >= hrow * b.RT) hr = 0;
    const int ht = hrow > 0 ? hr / hrow : 0;
    h.t = b.t0 + ht;
    hr -= ht * hrow;
    if (hr < hy) {
        h.y = hr < b.RZ ? b.y0 - 1 : b.y0 + b.RY;
        h.z = b.z0 + (hr < b.RZ ? hr : hr - b.RZ);
    } else {
        const int q = hr - hy;
        h.z = q < b.RY ? b.z0 - 1 : b.z0 + b.RZ;
        h.y = b.y0 + (q < b.RY ? q : q - b.RY);
    }
    h.y = h.y < 0 ? h.y + L : (h.y >= L ? h.y - L : h.y);
    h.z = h.z < 0 ? h.z + L : (h.z >= L ? h.z - L : h.z);
    return h;
}

// Staged entries (sites first, halo from NS on) of the y and z neighbours of site i.
struct BrickYZ {
    int ym, yp, zm, zp;
};
DD_TILE_FN BrickYZ brick_yz(const Brick& b, const BrickSite& s, int L, int len, int NS, int i) {
    const int hy = halo_rows_y(b, L), h0 = NS + s.rt * halo_rows(b, L) * len + s.x;  // this slice's halo rows
    BrickYZ n;
    n.ym = s.ry > 0 ? i - len : (b.RY < L ? h0 + s.rz * len : i + (b.RY - 1) * len);
    n.yp = s.ry < b.RY - 1 ? i + len : (b.RY < L ? h0 + (b.RZ + s.rz) * len : i - (b.RY - 1) * len);
    n.zm = s.rz > 0 ? i - len * b.RY : (b.RZ < L ? h0 + (hy + s.ry) * len : i + (b.RZ - 1) * b.RY * len);
    n.zp = s.rz < b.RZ - 1 ? i + len * b.RY : (b.RZ < L ? h0 + (hy + b.RY + s.ry) * len : i - (b.RZ - 1) * b.RY * len);
    return n;
}

// Staged entries of the x neighbours: of a whole row, and of a half row, whose other-parity sites lie at 2 x + 1 - bo
// where the site itself is at 2 x + bo.
struct BrickX {
    int xm, xp;
};
DD_TILE_FN BrickX brick_x(const BrickSite& s, int len) {
    return BrickX{s.row * len + (s.x == 0 ? len - 1 : s.x - 1), s.row * len + (s.x == len - 1 ? 0 : s.x + 1)};
}
DD_TILE_FN BrickX brick_x_half(const BrickSite& s, int len, int bo) {
    return BrickX{s.row * len + (bo ? s.x : (s.x == 0 ? len - 1 : s.x - 1)),
                  s.row * len + (bo ? (s.x + 1 == len ? 0 : s.x + 1) : s.x)};
}

// Half fields: rows of L / 2 sites.  A brick fits up to L = 128.
inline EoTile eo_tile_shape(int L, int nt) { return tile_shape(L, L / 2, nt, kTileSites, kTileSites); }
inline bool eo_tile_ok(int L, int nt) { return tile_fits(eo_tile_shape(L, nt)); }
// Columns per workgroup that put all columns of a field into one round of workgroups, one to each of the 256
// CUs (a workgroup fills a CU's register file), or all columns of a brick into one where the bricks alone are more.
inline int eo_tile_cols(int L, int nt, int ncol) {
    const int bricks = eo_tile_blocks(eo_tile_shape(L, nt));
    const int groups = bricks > 0 && bricks <= 256 ? 256 / bricks : 1;
    return groups < ncol ? (ncol + groups - 1) / groups : 1;
}

// Whether an untimed launch takes the form.  FP32: where one round of workgroups holds it, with a column each or, in
// full bricks, several one after the other; a second round costs more than the sweep's shorter workgroups.
// Mixed solves, ms, form and sweep of one slice per chunk: one column of 32 x 16^3 (256 bricks) 3.46 and 3.56, of 8 x 24^3
// (240) 3.21 and 3.26, of 6 x 28^3 (294) 4.43 and 3.96, of 6 x 32^3 (384) 5.15 and 4.52; 12 columns of 16 x 4^3 2.47 and
// 2.60; 9 of 16 x 12^3 (64) 4.48 and 4.95; 3 of 4 x 26^3 (180, three quarters full) 3.76 and 3.52; on the wrong side 5 of
// 8 x 18^3 (96 bricks, three columns one after the other) 4.61 and 4.27, 6 of 20 x 10^3 3.41 and 3.13.
// FP64: where a whole workgroup per CU has columns to loop over and the bricks are full (us a half hop, 12 columns:
// 16 x 32^3, 1024 bricks, 418 against the sweep's 579; 32 x 16^3, 256 bricks, 86 against 140; 8 x 16^3, 64 bricks, 36
// against 31; solves, ms: 4 columns of 16 x 20^3 14.3 and 16.6, 12 of 4 x 40^3, 0.64 full, 85 and 74, 4 of 2 x 96^3,
// 0.19 full, 302 and 142).
inline bool eo_tile_form(int L, int nt, int ncol, size_t real_bytes) {
    const int bricks = eo_tile_blocks(eo_tile_shape(L, nt));
    if (bricks == 0) return false;
    const double fill = 0.5 * nt * L * L * L / ((double)kTileSites * bricks);
    if (real_bytes == 8) return ncol >= 4 && bricks >= 256 && fill >= 0.8;
    return bricks <= 256 && ((long long)bricks * ncol <= 256 || fill >= 0.8);
}

// Whether an FP32 launch of the form may read two rows of a link and rebuild the third in FP32 (SU(3) links
// only): fields whose launch is timed, with an even number of columns or the rows of L = 16 and 32.  The
// rebuilt row is less exact than a stored one (rounding, and what the links are off SU(3)), so launches
// that have always read nine entries go on doing so: small fields, and odd column counts at other L.  Two rows
// in those too are faster (ms, two and nine: the one-column force on 32 x 16^3 19.6 and 21.5, the factorised
// propagator on 16 x 4^3 8.3 and 8.9, a solve of three columns of 16 x 24^3 10.2 and 10.9).
inline bool eo_two_rows(int L, int nt, int ncol) {
    return (size_t)nt * L * L * L * ncol >= ((size_t)1 << 18) && (ncol % 2 == 0 || L == 16 || L == 32);
}

// Whole fields, in time blocks of 8.  A brick fits up to L = 64.
inline EoTile dslash_tile_shape(int L, int nt) {
    EoTile t = tile_shape(L, L, nt, kDslSites, kDslHalo);
    t.tb = t.ntt < 8 ? t.ntt : 8;
    return t;
}
// A dropped time hop is read from 2 GiB past the column's start, which has to lie outside the column.
inline bool dslash_tile_ok(int L, int nt, size_t real_bytes) {
    return (size_t)24 * nt * L * L * L * real_bytes < ((size_t)1 << 31) && tile_fits(dslash_tile_shape(L, nt));
}


// Whether a launch on a field takes the form: by sizes alone, not by a timing, since the form adds the hops of a
// site in another order than the sweep and a result must not depend on how two launches happened to be
// timed (the launch shapes within a form give the same bits).  `timed`: the shape is timed, the best of each form
// compared below (us, sweep and form); else the untimed shapes (default_sched).  `sums`: the launch forms sums
// (inside solves).
// Untimed: bricks that give every CU two workgroups and are nearly full.
// Links past the 256 MB Infinity Cache are read from HBM, which the sweep does best where its x hops need no loads (L
// divides 64) and its columns go by ones or twos: us FP64, 64 x 32^3 1 column 444 and 482, 2 669 and 754, 3 1121 and
// 1012, 4 of 48 x 32^3 936 and 959, 6 1557 and 1339; 128 x 16^3 116 and 141, 175 and 222, 265 and 279, 305 and 363, 477
// and 498; FP32 64 x 32^3 2 columns 407 and 428.  (12 x 32^3, links of 227 MB, 91 and 85, 138 and 135.)
// FP64: bricks three quarters full win with one column too (32 x 24^3 113 and 104; 12 columns of 6 x 16^3, 192
// bricks, 51.9 and 44.3; but 4 of 32 x 14^3 58 and 61); down to 0.6 with columns to share the links (8 x 40^3, 2 columns
// 209 and 223, 6 columns 590 and 551); below that never (8 x 48^3, 12 columns 2068 and 2518).
// The sums cost the form 24 registers that it has to spill, the sweep few: full bricks still win (ms a
// solve of the full operator, 12 columns: 30 x 15^3, 0.82 full, 77.8 and 75.0; 8 x 21^3 52.7 and 49.5; 8 x 32^3 173
// and 162), others do not (16 x 24^3, 0.75 full, 160 and 162, 4 columns 52.8 and 56.9; 16 x 17^3, 0.71, 55.9 and 61.2).
// FP32 moves half the bytes past the same instructions, so one column never pays (64 x 32^3 1.18 of the
// sweep's time); from two on full bricks do (8 x 32^3 46.7 and 42.3), others with several columns and bricks
// enough (4 columns of 32 x 24^3 188 and 174, of 48 x 12^3, 768 bricks, 1.05, of 16 x 19^3, 1120, a solve 14.9 and
// 15.8 ms) or with all twelve (16 x 18^3 0.89); sums spill nothing there.
inline bool dslash_tile_form(int L, int nt, int ncol, size_t real_bytes, bool timed, bool sums) {
    if (!dslash_tile_ok(L, nt, real_bytes)) return false;
    const int bricks = eo_tile_blocks(dslash_tile_shape(L, nt));
    const double fill = (double)nt * L * L * L / ((double)kDslSites * bricks);
    if (!timed) return bricks >= 512 && fill >= 0.9;
    if (bricks < 192) return false;
    const bool lanes = L >= 4 && 64 % L == 0;
    if (lanes && (size_t)72 * real_bytes * nt * L * L * L > ((size_t)256 << 20) && (ncol <= 2 || ncol == 4)) return false;
    if (real_bytes == 8 && sums) return fill >= 0.8;
    if (real_bytes == 8) return fill >= 0.75 || (fill >= 0.6 && ncol >= 6);
    return ncol >= 2 && (fill >= 0.87 || (ncol >= 4 && fill >= 0.75 && bricks >= 1536) || (ncol >= 12 && fill >= 0.8));
}

}  // namespace dd
