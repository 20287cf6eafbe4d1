// dd_dslash_tile.h -- the Wilson-Dirac stencil with its input staged in LDS.
//
// The operator of dd_dslash.h, organised as the even-odd half hop of dd_eo_tile.h is: a workgroup owns a
// brick of whole x rows (rt slices x rz x ry rows, at most 128 sites) and loops over a group of
// columns; two threads share a site, part A with the links of its time and x hops in registers, part
// B with those of its y and z hops; per column the spinors of the brick and of the one-row halo around
// each of its slices in y and z are staged in LDS.  A link is read once per launch, a spinor about
// twice (on a 16 x 32^3 slab, 12 columns, FP64: 2.6 GB read where 1.5 are needed; the sweep reads each
// link once per column pair and, with its neighbours in other L2 lines by then, a spinor three times).
// What bounds it: the phases of a column (copy in, hops, copy out) wait for each other at barriers,
// so two workgroups share a CU and fill each other's waits: with 256 sites and one workgroup of 512
// threads per CU D on 64 x 32^3, 12 columns, took 3472 us in FP64 and 1924 in FP32, this form 3146 and
// 1870, the sweep 4160 and 2208; on 32 x 16^3 185 and 99 us against 266 and 137.  Time blocks of 8
// bricks (FP64 on 64 x 32^3: 4 bricks 3444 us, 8 3146, 16 3688).  Clearing the links of dropped hops, which
// may hold anything, costs FP64 2 % of that (3163 -> 3230 us through the library).  A site's hops are added
// as (time and x) + (y and z), not one after the other as in the sweep, so the two forms agree to rounding;
// which one a launch takes depends on its sizes only (dslash_tile_form).
#pragma once

#include "dd_eo_tile.h"

namespace dd {

constexpr int kDslNT = 2 * kDslSites;      // two threads per site

template <typename R>
struct TileArgs {
    const cpx<R>* U;    // [4][9][vlink]
    const cpx<R>* in;   // column 0 of the field
    cpx<R>* out;
    const cpx<R>* aux;
    R mass, f;          // 1/(2 kappa) (EPI_HOP: kappa); f = +1 for D^+, -1 for D
    const ColState* st; // of column 0; nullable
    double* partial;    // slot of (column 0, block 0)
    int nblk;           // slots per column
};

// Columns [col_lo, col_hi) of brick blk_lin.  A stopped column is passed over.
template <typename R, int EPI>
__device__ __forceinline__ void dslash_lds_body(const Geo& g, const EoTile& ts, const TileArgs<R>& A, int blk_lin,
                                                int col_lo, int col_hi) {
    constexpr int NU = tile_units<R>(), NS = kDslSites, ST = kDslSites + kDslHalo, NWAVE = kDslNT / kWave;
    constexpr uint32_t CB = sizeof(cpx<R>);
    constexpr bool SUM = EPI != EPI_STORE && EPI != EPI_HOP;
    constexpr bool AUX = EPI == EPI_RESID || EPI == EPI_DOT_AUX;
    constexpr bool PRE = sizeof(R) == 4;  // the next column's staging sites are loaded ahead
    __shared__ f32x4v s_tile[NU * ST];
    // the halves of the sums: a region of their own in FP32; in FP64 they take the tile's place
    // once it has been read (74 KB a workgroup against 98)
    __shared__ f32x4v s_own[PRE ? NU * NS : 1];
    __shared__ double s_red[SUM ? 2 : 1][NWAVE][3];
    f32x4v* s_acc = PRE ? s_own : s_tile;

    auto next_live = [&](int c) {
        while (c < col_hi && A.st != nullptr && !A.st[c].active) c++;
        return c;
    };
    int col = next_live(col_lo);
    if (col >= col_hi) return;  // uniform over the workgroup

    const int L = g.L, L2 = g.L2, L3 = g.L3, nt = g.nt, nsite = g.nsite;
    const uint32_t cs = (uint32_t)nsite * CB, fs = 12u * cs, ls = (uint32_t)g.vlink * CB;
    const Brick bk = tile_brick(ts, blk_lin, L, nt);
    const int blk = bk.blk;

    const int tid = (int)threadIdx.x;
    const bool partB = __builtin_amdgcn_readfirstlane(tid / NS) != 0;
    const int i = tid % NS;
    const int nsit = bk.RT * bk.RZ * bk.RY * L;
    const bool act = i < nsit;
    const int ic = min(i, nsit - 1);
    const BrickSite bs = brick_site(bk, L, ic);
    const int x = bs.x, y = bk.y0 + bs.ry, z = bk.z0 + bs.rz, tl = bk.t0 + bs.rt;
    const int sp = (z * L + y) * L + x;
    const int s = tl * L3 + sp;
    auto tglob = [&](int t) {
        const int tg = g.t0 + t;
        return tg >= g.T ? tg - g.T : tg;
    };
    const int sl = tglob(tl) * L3 + sp;  // this site's links
    const size_t cst = (size_t)12 * (size_t)nsite;
    auto frsrc = [&](int c) { return make_rsrc(A.in + (size_t)c * cst, fs); };
    auto load = [&](rsrc_t f, uint32_t vo, cpx<R> (&p)[12]) {
#pragma unroll
        for (int c = 0; c < 12; c++) p[c] = bload<R>(f, vo, (uint32_t)c * cs);
    };
    auto put = [&](int idx, const cpx<R> (&p)[12]) { tile_put<R, ST>(s_tile, idx, p); };
    auto link = [&](int mu, int site, cpx<R> (&w)[9]) {
        bload_link<R>(make_rsrc(A.U + (size_t)(9 * mu) * g.vlink, 9u * ls), ls, site, w);
    };

    int it = 0, prev = 0;
    auto write_sum = [&]() {
        if (SUM && tid < 3) {
            double v = 0;
            const int td = loop_index<R>(tid);
#pragma unroll
            for (int w = 0; w < NWAVE; w++) v += s_red[(it - 1) & 1][w][td];
            A.partial[((size_t)prev * A.nblk + blk) * 3 + td] = v;
        }
    };
    auto give = [&](const cpx<R> (&a)[12], auto PB) {
        constexpr int O = 1 - decltype(PB)::value;
        const int ia = loop_index<R>(i);
        if constexpr (sizeof(R) == 4) {
#pragma unroll
            for (int k = 0; k < 3; k++)
                s_acc[(3 * O + k) * NS + ia] = f32x4v{a[6 * O + 2 * k].re, a[6 * O + 2 * k].im, a[6 * O + 2 * k + 1].re,
                                                     a[6 * O + 2 * k + 1].im};
        } else {
#pragma unroll
            for (int k = 0; k < 6; k++) s_acc[(6 * O + k) * NS + ia] = __builtin_bit_cast(f32x4v, a[6 * O + k]);
        }
    };
    // six components of half B of a site at s
    auto six = [&](const f32x4v* s, int stride, int idx, cpx<R> (&v)[6], auto PB) {
        constexpr int B = decltype(PB)::value;
        if constexpr (sizeof(R) == 4) {
#pragma unroll
            for (int k = 0; k < 3; k++) {
                const f32x4v u = s[(3 * B + k) * stride + idx];
                v[2 * k] = cpx<R>{u.x, u.y};
                v[2 * k + 1] = cpx<R>{u.z, u.w};
            }
        } else {
#pragma unroll
            for (int k = 0; k < 6; k++) v[k] = __builtin_bit_cast(cpx<double>, s[(6 * B + k) * stride + idx]);
        }
    };
    auto load_half = [&](const cpx<R>* f, int c, cpx<R> (&v)[6], auto PB) {
        constexpr int B = decltype(PB)::value;
        const rsrc_t r = make_rsrc(f + (size_t)c * cst, fs);
#pragma unroll
        for (int k = 0; k < 6; k++) v[k] = bload<R>(r, (uint32_t)s * CB, (uint32_t)(6 * B + k) * cs);
    };
    auto finish = [&](int c, const cpx<R> (&a)[12], const cpx<R> (&pv)[6], const cpx<R> (&xv)[6], auto PB) {
        constexpr int B = decltype(PB)::value;
        const rsrc_t ro = make_rsrc(A.out + (size_t)c * cst, act ? fs : 0u);
        double d0 = 0, d1 = 0, d2 = 0;
        const int ia = loop_index<R>(i);
        const R half = R(0.5);
        cpx<R> b[6];
        six(s_acc, NS, ia, b, PB);
#pragma unroll
        for (int k = 0; k < 6; k++) {
            const cpx<R> v = a[6 * B + k] + b[k];
            const cpx<R> pc = pv[k], qv = xv[k];
            cpx<R> o = EPI == EPI_HOP ? mk<R>(A.mass * v.re, A.mass * v.im)
                                      : mk<R>(A.mass * pc.re - half * v.re, A.mass * pc.im - half * v.im);
            if (EPI == EPI_RESID) o = qv - o;
            if (EPI == EPI_DOT_AUX) {
                d0 += (double)qv.re * o.re + (double)qv.im * o.im;
                d1 += (double)qv.re * o.im - (double)qv.im * o.re;
            } else if (EPI == EPI_TS) {
                d0 += (double)o.re * pc.re + (double)o.im * pc.im;
                d1 += (double)o.re * pc.im - (double)o.im * pc.re;
                d2 += (double)o.re * o.re + (double)o.im * o.im;
            } else if (EPI == EPI_RESID || EPI == EPI_NORM) {
                d0 += (double)o.re * o.re + (double)o.im * o.im;
            }
            // past the caches, which the input halos need: D+D with sums, 12 columns, FP64 30 x 15^3 269 -> 241 us, 16 x
            // 24^3 519 -> 506, FP32 8 x 27^3 230 -> 207, 32 x 16^3 121 -> 116
            bstore_nt<R>(ro, (uint32_t)s * CB, (uint32_t)(6 * B + k) * cs, o);
        }
        if constexpr (SUM) {
            const int w = tid / kWave;
            const double v0 = wave_sum(act ? d0 : 0.0);
            const double v1 = EPI == EPI_DOT_AUX || EPI == EPI_TS ? wave_sum(act ? d1 : 0.0) : 0.0;
            const double v2 = EPI == EPI_TS ? wave_sum(act ? d2 : 0.0) : 0.0;
            if (tid % kWave == 0) {
                s_red[it & 1][w][0] = v0;
                s_red[it & 1][w][1] = v1;
                s_red[it & 1][w][2] = v2;
            }
        }
    };

    const R f = A.f;
    cpx<R> w0[9], w1[9], w2[9], w3[9];
    if (!partB) {
        using PB = std::integral_constant<int, 0>;
        const int tg = tglob(tl);
        const R phb = (tl > 0 || g.whole) ? (tg == 0 ? R(g.bc) : R(1)) : R(0);
        const R phf = (tl < nt - 1 || g.whole) ? (tg == g.T - 1 ? R(g.bc) : R(1)) : R(0);
        const int tb = tl > 0 ? tl - 1 : nt - 1, tf = tl < nt - 1 ? tl + 1 : 0;
        // a dropped hop reads past the field's resource, which gives zeros (a column is below 2 GiB)
        const uint32_t vf = phf != R(0) ? (uint32_t)(tf * L3 + sp) * CB : 0x80000000u;
        const uint32_t vb = phb != R(0) ? (uint32_t)(tb * L3 + sp) * CB : 0x80000000u;
        const uint32_t v0 = (uint32_t)s * CB;
        cpx<R> q[12];
        if (PRE) load(frsrc(col), v0, q);
        link(0, sl, w0);
        link(0, tglob(tb) * L3 + sp, w1);
        link(1, sl, w2);
        link(1, sl + ((x == 0) ? (L - 1) : -1), w3);
#pragma unroll
        for (int k = 0; k < 9; k++) {
            w0[k] = phf != R(0) ? phf * w0[k] : mk<R>(0, 0);  // the link of a dropped hop may hold anything
            w1[k] = phb != R(0) ? phb * w1[k] : mk<R>(0, 0);
        }
        const BrickX nx = brick_x(bs, L);
        for (;;) {
            const int nxt = next_live(col + 1);
            cpx<R> pf[12], pb[12], a[12], hh[6];
            if (!PRE) load(frsrc(col), v0, q);
            load(frsrc(col), vf, pf);
            if (PRE) load(frsrc(col), vb, pb);
            hop_fence<R>();
            put(loop_index<R>(i), q);
            hop_fence<R>();
#pragma unroll
            for (int k = 0; k < 12; k++) a[k] = mk<R>(0, 0);
            if (!PRE) {
                project_f<R, 0>(pf, hh, f);
                hop_fence<R>();
                load(frsrc(col), vb, pb);
                hop_f<R, 0, false>(a, w0, hh, f);
                hop_fence<R>();
                project_f<R, 0>(pb, hh, -f);
                hop_f<R, 0, true>(a, w1, hh, -f);
                hop_fence<R>();
            }
            __syncthreads();
            if (it > 0) write_sum();
            if (PRE && nxt < col_hi) load(frsrc(nxt), v0, q);
            hop_fence<R>();
            tile_project<R, ST, 1>(s_tile, loop_index<R>(nx.xp), hh, f);
            hop_f<R, 1, false>(a, w2, hh, f);
            hop_fence<R>();
            tile_project<R, ST, 1>(s_tile, loop_index<R>(nx.xm), hh, -f);
            hop_f<R, 1, true>(a, w3, hh, -f);
            hop_fence<R>();
            if (PRE) {
                project_f<R, 0>(pf, hh, f);
                hop_f<R, 0, false>(a, w0, hh, f);
                project_f<R, 0>(pb, hh, -f);
                hop_f<R, 0, true>(a, w1, hh, -f);
            }
            cpx<R> pv[6], xv[6];
            six(s_tile, ST, loop_index<R>(ic), pv, PB{});  // this site's own spinor
            if (!PRE) __syncthreads();  // the tile has been read
            give(a, PB{});
            hop_fence<R>();
            if (AUX) load_half(A.aux, col, xv, PB{});
            hop_fence<R>();
            __syncthreads();
            finish(col, a, pv, xv, PB{});
            hop_fence<R>();
            if (!PRE) __syncthreads();  // the next column's staging takes the sums' place
            it++;
            prev = col;
            col = nxt;
            if (col >= col_hi) break;
        }
    } else {
        using PB = std::integral_constant<int, 1>;
        auto halo_off = [&](int k) {
            const HaloSite hs = halo_site(bk, L, L, k);
            return (uint32_t)(hs.t * L3 + (hs.z * L + hs.y) * L + hs.x) * CB;
        };
        const uint32_t v0 = halo_off(i), v1 = halo_off(NS + i);
        cpx<R> q[12], q2[12];
        auto issue = [&](int c) {
            load(frsrc(c), v0, q);
            load(frsrc(c), v1, q2);
        };
        if (PRE) issue(col);
        link(2, sl, w0);
        link(2, sl + ((y == 0) ? (L - 1) * L : -L), w1);
        link(3, sl, w2);
        link(3, sl + ((z == 0) ? (L - 1) * L2 : -L2), w3);
        const BrickYZ nb = brick_yz(bk, bs, L, L, NS, ic);
        for (;;) {
            const int nxt = next_live(col + 1);
            cpx<R> a[12], hh[6];
            if (!PRE) {
                load(frsrc(col), v0, q);
                hop_fence<R>();
                put(loop_index<R>(NS + i), q);
                hop_fence<R>();
                load(frsrc(col), v1, q);
                put(loop_index<R>(2 * NS + i), q);
            } else {
                put(NS + i, q);
                put(2 * NS + i, q2);
            }
            hop_fence<R>();
            __syncthreads();
            if (PRE && nxt < col_hi) issue(nxt);
            hop_fence<R>();
#pragma unroll
            for (int k = 0; k < 12; k++) a[k] = mk<R>(0, 0);
            tile_project<R, ST, 2>(s_tile, loop_index<R>(nb.yp), hh, f);
            hop_f<R, 2, false>(a, w0, hh, f);
            hop_fence<R>();
            tile_project<R, ST, 2>(s_tile, loop_index<R>(nb.ym), hh, -f);
            hop_f<R, 2, true>(a, w1, hh, -f);
            hop_fence<R>();
            tile_project<R, ST, 3>(s_tile, loop_index<R>(nb.zp), hh, f);
            hop_f<R, 3, false>(a, w2, hh, f);
            hop_fence<R>();
            tile_project<R, ST, 3>(s_tile, loop_index<R>(nb.zm), hh, -f);
            hop_f<R, 3, true>(a, w3, hh, -f);
            hop_fence<R>();
            cpx<R> pv[6], xv[6];
            six(s_tile, ST, loop_index<R>(ic), pv, PB{});  // this site's own spinor
            if (!PRE) __syncthreads();
            give(a, PB{});
            hop_fence<R>();
            if (AUX) load_half(A.aux, col, xv, PB{});
            hop_fence<R>();
            __syncthreads();
            finish(col, a, pv, xv, PB{});
            hop_fence<R>();
            if (!PRE) __syncthreads();
            it++;
            prev = col;
            col = nxt;
            if (col >= col_hi) break;
        }
    }
    if (SUM) {
        __syncthreads();
        write_sum();
    }
}

}  // namespace dd
