// dd_eo_tile.h -- the even-odd half hop with its input staged in LDS.
//
// The same operator as the time-sweep kernels of dd_eo.h,
//     out = a_self * self + c_hop * (H in)_site     (in: the other parity),
// organised so that a spinor is read from memory about twice per launch and a link once:
//   * a workgroup owns a brick of whole x rows (rt slices x rz x ry rows, at most 256 output
//     sites) and loops over a group of columns;
//   * two threads share an output site: part A holds the links of its time and x hops, part B
//     those of its y and z hops, four links each, in registers for every column (eight links of a
//     site would take 288 registers in FP64);
//   * per column part A stages the input spinors of the brick's rows in LDS and part B those of
//     the one-row halo around each slice in y and z; the spatial hops read LDS, the two time hops
//     read the thread's own site on the slices either side; the halves of the sum are exchanged
//     through LDS and each part finishes six of the twelve components.
// What bounds it: the bytes that miss L2 (a plain copy reaches 4.75 TB/s here, reads from the
// Infinity Cache no more than 7.2 TB/s).  The sweeps fetch the y and z neighbours of a tile and
// the links of a column pair again and again: 1.07 GB read per launch of the first FP32 half hop on a
// 16 x 32^3 slab with 12 columns (0.40 GB needed), this form 0.63 GB.  Measured there (us, 12
// columns, sweep -> this form): FP32 first half 249 -> 195, second 304 -> 240; FP64 first 579 -> 418,
// second 669 -> 526; on 32 x 16^3 FP32 58 -> 46 and 68 -> 50, FP64 140 -> 86 and 161 -> 128.  The
// FP32 kernel loads the next column's staging sites while it computes (195 to 216 registers);
// the FP64 one has no registers left for that (256) and keeps the scheduler to one hop at a time,
// without which it spills more than a hundred and runs slower than the sweep.  Copies straight to
// LDS in place of the staging registers were slower (240 us), since the wait for them also waits
// for the stores issued behind them.  With few workgroups the loop over columns runs serially on
// part of the chip, and the one-slice sweep is the faster one (eo_default_sched).
#pragma once

#include <type_traits>

#include "dd_eo.h"
#include "dd_tile_shape.h"

namespace dd {

constexpr int kTileNT = 2 * kTileSites;       // two threads per output site

// project / accum of dd_wilson.h with the sign as a factor f = +1 or -1 (the products are exact, so
// the values are the same, and D and D^+ share one kernel).
template <typename R, int MU>
__device__ __forceinline__ void project_f(const cpx<R> (&p)[12], cpx<R> (&h)[6], R f) {
#pragma unroll
    for (int c = 0; c < 3; c++) {
        const cpx<R> p0 = p[c], p1 = p[3 + c], p2 = p[6 + c], p3 = p[9 + c];
        if (MU == 0) {
            h[c] = p0 - f * p2;
            h[3 + c] = p1 - f * p3;
        } else if (MU == 1) {
            h[c] = p0 - f * imul(p3);
            h[3 + c] = p1 - f * imul(p2);
        } else if (MU == 2) {
            h[c] = p0 - f * p3;
            h[3 + c] = p1 + f * p2;
        } else {
            h[c] = p0 - f * imul(p2);
            h[3 + c] = p1 + f * imul(p3);
        }
    }
}
template <typename R, int MU>
__device__ __forceinline__ void accum_f(cpx<R> (&a)[12], const cpx<R> (&u)[6], R f) {
#pragma unroll
    for (int c = 0; c < 3; c++) {
        const cpx<R> u0 = u[c], u1 = u[3 + c];
        a[c] = a[c] + u0;
        a[3 + c] = a[3 + c] + u1;
        if (MU == 0) {
            a[6 + c] = a[6 + c] - f * u0;
            a[9 + c] = a[9 + c] - f * u1;
        } else if (MU == 1) {
            a[6 + c] = a[6 + c] + f * imul(u1);
            a[9 + c] = a[9 + c] + f * imul(u0);
        } else if (MU == 2) {
            a[6 + c] = a[6 + c] + f * u1;
            a[9 + c] = a[9 + c] - f * u0;
        } else {
            a[6 + c] = a[6 + c] + f * imul(u0);
            a[9 + c] = a[9 + c] - f * imul(u1);
        }
    }
}
// a += (1 + f gamma_MU)-reconstruction of W h, W = U or (BWD) U^+.
template <typename R, int MU, bool BWD>
__device__ __forceinline__ void hop_f(cpx<R> (&a)[12], const cpx<R> (&w)[9], const cpx<R> (&h)[6], R f) {
    cpx<R> t[6];
    transport<R, BWD>(w, h, R(1), t);
    accum_f<R, MU>(a, t, f);
}

// LDS units are 16 bytes: two components of a site in FP32, one in FP64.
template <typename R>
constexpr int tile_units() { return sizeof(R) == 8 ? 12 : 6; }
// FP64: keeps the compiler from holding the LDS addresses derived from idx across the column loop
template <typename R>
__device__ __forceinline__ int loop_index(int idx) {
    if constexpr (sizeof(R) == 8) asm volatile("" : "+v"(idx));
    return idx;
}
template <typename R, int ST>
__device__ __forceinline__ void tile_put(f32x4v* __restrict__ s, int idx, const cpx<R> (&p)[12]) {
    if constexpr (sizeof(R) == 4) {
#pragma unroll
        for (int q = 0; q < 6; q++) s[q * ST + idx] = f32x4v{p[2 * q].re, p[2 * q].im, p[2 * q + 1].re, p[2 * q + 1].im};
    } else {
#pragma unroll
        for (int q = 0; q < 12; q++) s[q * ST + idx] = __builtin_bit_cast(f32x4v, p[q]);
    }
}
template <typename R, int ST>
__device__ __forceinline__ void tile_get(const f32x4v* __restrict__ s, int idx, cpx<R> (&p)[12]) {
    if constexpr (sizeof(R) == 4) {
#pragma unroll
        for (int q = 0; q < 6; q++) {
            const f32x4v v = s[q * ST + idx];
            p[2 * q] = cpx<R>{v.x, v.y};
            p[2 * q + 1] = cpx<R>{v.z, v.w};
        }
    } else {
#pragma unroll
        for (int q = 0; q < 12; q++) p[q] = __builtin_bit_cast(cpx<double>, s[q * ST + idx]);
    }
}
// One colour of project_f.
template <typename R, int MU>
__device__ __forceinline__ void project_colour(cpx<R> p0, cpx<R> p1, cpx<R> p2, cpx<R> p3, cpx<R>& h0, cpx<R>& h1, R f) {
    if (MU == 0) {
        h0 = p0 - f * p2;
        h1 = p1 - f * p3;
    } else if (MU == 1) {
        h0 = p0 - f * imul(p3);
        h1 = p1 - f * imul(p2);
    } else if (MU == 2) {
        h0 = p0 - f * p3;
        h1 = p1 + f * p2;
    } else {
        h0 = p0 - f * imul(p2);
        h1 = p1 + f * imul(p3);
    }
}
template <typename R, int ST, int MU>
__device__ __forceinline__ void tile_project(const f32x4v* __restrict__ s, int idx, cpx<R> (&h)[6], R f) {
    if constexpr (sizeof(R) == 8) {
#pragma unroll
        for (int c = 0; c < 3; c++) {
            cpx<R> p[4];
#pragma unroll
            for (int k = 0; k < 4; k++) p[k] = __builtin_bit_cast(cpx<double>, s[(3 * k + c) * ST + idx]);
            project_colour<R, MU>(p[0], p[1], p[2], p[3], h[c], h[3 + c], f);
        }
    } else {
        cpx<R> p[12];
        tile_get<R, ST>(s, idx, p);
        project_f<R, MU>(p, h, f);
    }
}

// The spinor at byte offset vo (16 bytes per half site) of a half-field column.
template <typename R>
__device__ __forceinline__ void hload_at(rsrc_t f, uint32_t cs, uint32_t vo, cpx<R> (&p)[12]) {
    if constexpr (sizeof(R) == 8) {
#pragma unroll
        for (int c = 0; c < 12; c++) p[c] = bload<R>(f, vo, (uint32_t)c * cs);
    } else {
#pragma unroll
        for (int q = 0; q < 6; q++) {
            const f32x4v v = __builtin_bit_cast(f32x4v, __builtin_amdgcn_raw_buffer_load_b128(f, (int)vo, (int)((uint32_t)q * 2u * cs), 0));
            p[2 * q] = cpx<R>{v.x, v.y};
            p[2 * q + 1] = cpx<R>{v.z, v.w};
        }
    }
}

// FP64 holds the scheduler to one hop at a time (256 registers); FP32 lets it run ahead.
template <typename R>
__device__ __forceinline__ void hop_fence() {
    if constexpr (sizeof(R) == 8) __builtin_amdgcn_sched_barrier(0);
}

template <typename R>
struct EoTileArgs {
    const cpx<R>* U;      // REC: two rows per link
    const cpx<R>* in;     // column 0 of the field
    const cpx<R>* self;
    cpx<R>* out;
    const cpx<R>* aux;
    R a_self, c_hop, f;   // f = +1 for D^+, -1 for D: forward hops project with 1 + f gamma
    int p_out;
    const ColState* st;   // of column 0; nullable
    double* partial;      // slot of (column 0, block 0)
    int nblk;             // slots per column
};

// The columns of [lo, hi) (at most 64) that are not stopped, as bits..
__device__ __forceinline__ uint64_t live_columns(const ColState* st, int lo, int hi) {
    const int k = (int)threadIdx.x % kWave;
    bool on = k < hi - lo;
    if (st != nullptr && on) on = st[lo + k].active != 0;
    return __ballot(on);
}

// Columns [col_lo, col_hi) of brick blk_lin.  A stopped column (ColState inactive) is passed over:
// its output and partial slots keep their values.  NTS: non-temporal output stores.
template <typename R, int EPI, bool SELF, bool REC, bool NTS>
__device__ __forceinline__ void eo_tile_body(const Geo& g, const EoTile& ts, const EoTileArgs<R>& A, int blk_lin,
                                             int col_lo, int col_hi) {
    constexpr int NU = tile_units<R>(), ST = kTileNT, NS = kTileSites, NWAVE = kTileNT / kWave;
    constexpr uint32_t CB = sizeof(cpx<R>);
    constexpr bool SUM = EPI != EPI_STORE;
    constexpr bool AUX = EPI == EPI_RESID || EPI == EPI_DOT_AUX;
    __shared__ f32x4v s_tile[NU * ST];
    __shared__ f32x4v s_acc[NU * NS];
    __shared__ double s_red[SUM ? 2 : 1][NWAVE][3];

    // FP32 learns which columns run in one load, while its link loads are in flight; FP64 asks column by
    // column (12 columns, 16 x 32^3 mixed, 495 -> 486 ms a solve; 32 x 16^3 FP64 90.5 -> 92.2)
    uint64_t live = sizeof(R) == 4 ? live_columns(A.st, col_lo, col_hi) : 0;
    auto next_col = [&](int c) {
        if constexpr (sizeof(R) == 4) {
            c = live ? col_lo + __builtin_ctzll(live) : col_hi;
            live &= live - 1;
        } else {
            while (c < col_hi && A.st != nullptr && !A.st[c].active) c++;
        }
        return c;
    };
    int col = 0;
    if (sizeof(R) == 8) {
        col = next_col(col_lo);
        if (col >= col_hi) return;  // uniform over the workgroup
    }

    const int L = g.L, L2 = g.L2, L3 = g.L3, LH = L >> 1, nt = g.nt, nh = g.nsite >> 1;
    const uint32_t cs = (uint32_t)nh * CB, fs = 12u * cs, ls = 2u * (uint32_t)nh * CB;
    const Brick bk = tile_brick(ts, blk_lin, L, nt);
    const int blk = bk.blk;

    const int tid = (int)threadIdx.x;
    const bool partB = __builtin_amdgcn_readfirstlane(tid / NS) != 0;
    const int i = tid % NS;
    const int nsit = bk.RT * bk.RZ * bk.RY * LH;
    const bool act = i < nsit;
    const int ic = min(i, nsit - 1);
    const BrickSite bs = brick_site(bk, LH, ic);
    const int y = bk.y0 + bs.ry, z = bk.z0 + bs.rz, tl = bk.t0 + bs.rt;
    const int bo = (A.p_out + tl + y + z) & 1;
    const int x = 2 * bs.x + bo;
    const int sp = (z * L + y) * L + x;
    const int s = tl * L3 + sp, h = s >> 1;
    int sh0;  // the half site this thread stages
    if (!partB) {
        sh0 = (tl * L3 + (z * L + y) * L) / 2 + bs.x;
    } else {
        const HaloSite hs = halo_site(bk, L, LH, i);
        sh0 = (hs.t * L3 + (hs.z * L + hs.y) * L) / 2 + hs.x;
    }
    constexpr bool PAIRED_LINKS = REC && sizeof(R) == 4;
    const uint32_t ubytes = PAIRED_LINKS ? 5u * (uint32_t)nh * 16u : 17u * (uint32_t)nh * CB;
    auto lrsrc = [&](int mu, int par) {
        return make_rsrc(A.U + (PAIRED_LINKS ? rec_link_base(mu, par, nh) : (size_t)(mu * 18 + par) * nh), ubytes);
    };
    const size_t cst = (size_t)12 * (size_t)nh;
    auto frsrc = [&](int c) { return make_rsrc(A.in + (size_t)c * cst, fs); };
    cpx<R> q[12];  // the staging site of the next column
    auto issue = [&](int c) { hload_spinor<R>(frsrc(c), cs, 0u, sh0, q); };

    int it = 0, prev = 0;  // columns done; the last of them
    auto write_sum = [&]() {
        if (SUM && tid < 3) {
            double v = 0;
            const int td = loop_index<R>(tid);
#pragma unroll
            for (int w = 0; w < NWAVE; w++) v += s_red[(it - 1) & 1][w][td];
            A.partial[((size_t)prev * A.nblk + blk) * 3 + td] = v;
        }
    };
    // the two threads of a site exchange halves of their sums; thread part B finishes components 6..11
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
    auto load_half = [&](const cpx<R>* f, int c, cpx<R> (&v)[6], auto PB) {
        constexpr int B = decltype(PB)::value;
        const rsrc_t r = make_rsrc(f + (size_t)c * cst, fs);
#pragma unroll
        for (int k = 0; k < 3; k++) hload_pair<R>(r, cs, 0u, h, 3 * B + k, v[2 * k], v[2 * k + 1]);
    };
    auto finish = [&](int c, const cpx<R> (&a)[12], const cpx<R> (&sv)[6], const cpx<R> (&xv)[6], auto PB) {
        constexpr int B = decltype(PB)::value;
        const rsrc_t ro = make_rsrc(A.out + (size_t)c * cst, act ? fs : 0u);
        double d0 = 0, d1 = 0, d2 = 0;
        const int ia = loop_index<R>(i);
#pragma unroll
        for (int k = 0; k < 3; k++) {
            cpx<R> b[2], r[2];
            if constexpr (sizeof(R) == 4) {
                const f32x4v v = s_acc[(3 * B + k) * NS + ia];
                b[0] = cpx<R>{v.x, v.y};
                b[1] = cpx<R>{v.z, v.w};
            } else {
                b[0] = __builtin_bit_cast(cpx<double>, s_acc[(6 * B + 2 * k) * NS + ia]);
                b[1] = __builtin_bit_cast(cpx<double>, s_acc[(6 * B + 2 * k + 1) * NS + ia]);
            }
#pragma unroll
            for (int e = 0; e < 2; e++) {
                const cpx<R> v = a[6 * B + 2 * k + e] + b[e];
                const cpx<R> pc = sv[2 * k + e], qv = xv[2 * k + e];
                cpx<R> o = SELF ? mk<R>(A.a_self * pc.re + A.c_hop * v.re, A.a_self * pc.im + A.c_hop * v.im)
                                : mk<R>(A.c_hop * v.re, A.c_hop * v.im);
                if (EPI == EPI_RESID) o = qv - o;
                r[e] = o;
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
            }
            hstore_pair<R, NTS>(ro, cs, 0u, h, 3 * B + k, r[0], r[1]);
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
        const int tg = g.t0 + tl >= g.T ? g.t0 + tl - g.T : g.t0 + tl;
        // time hops: dropped at a slab's ends, across the time edge of a whole lattice with time_bc
        const R phb = (tl > 0 || g.whole) ? (tg == 0 ? R(g.bc) : R(1)) : R(0);
        const R phf = (tl < nt - 1 || g.whole) ? (tg == g.T - 1 ? R(g.bc) : R(1)) : R(0);
        const int hb = ((tl > 0 ? tl - 1 : nt - 1) * L3 + sp) >> 1, hf = ((tl < nt - 1 ? tl + 1 : 0) * L3 + sp) >> 1;
        // a dropped hop reads past the field's resource, which gives zeros
        const uint32_t vf = phf != R(0) ? (uint32_t)hf * 16u : 0x80000000u, vb = phb != R(0) ? (uint32_t)hb * 16u : 0x80000000u;
        const int xm1 = (x == 0) ? (L - 1) : -1;
        bload_link_r<R, REC>(lrsrc(0, A.p_out), ls, h, w0);
        bload_link_r<R, REC>(lrsrc(0, 1 - A.p_out), ls, hb, w1);
        bload_link_r<R, REC>(lrsrc(1, A.p_out), ls, h, w2);
        bload_link_r<R, REC>(lrsrc(1, 1 - A.p_out), ls, (s + xm1) >> 1, w3);
        if (sizeof(R) == 4) {
            col = next_col(col_lo);
            if (col >= col_hi) return;  // uniform over the workgroup
            issue(col);
        }
        // the factor of the time edge goes into the link
#pragma unroll
        for (int k = 0; k < 9; k++) {
            w0[k] = phf != R(0) ? phf * w0[k] : mk<R>(0, 0);  // the link of a dropped hop may hold anything
            w1[k] = phb != R(0) ? phb * w1[k] : mk<R>(0, 0);
        }
        const BrickX nx = brick_x_half(bs, LH, bo);
        for (;;) {
            const int nxt = next_col(col + 1);
            cpx<R> pf[12], pb[12], a[12], hh[6];
            if (sizeof(R) == 8) issue(col);
            hload_at<R>(frsrc(col), cs, vf, pf);
            if (sizeof(R) == 4) hload_at<R>(frsrc(col), cs, vb, pb);
            hop_fence<R>();
            tile_put<R, ST>(s_tile, loop_index<R>(tid), q);
            hop_fence<R>();
#pragma unroll
            for (int k = 0; k < 12; k++) a[k] = mk<R>(0, 0);
            if (sizeof(R) == 8) {
                project_f<R, 0>(pf, hh, f);
                hop_fence<R>();
                hload_at<R>(frsrc(col), cs, vb, pb);
                hop_f<R, 0, false>(a, w0, hh, f);
                hop_fence<R>();
                project_f<R, 0>(pb, hh, -f);
                hop_f<R, 0, true>(a, w1, hh, -f);
                hop_fence<R>();
            }
            __syncthreads();
            if (it > 0) write_sum();
            if (sizeof(R) == 4 && nxt < col_hi) issue(nxt);
            hop_fence<R>();
            tile_project<R, ST, 1>(s_tile, loop_index<R>(nx.xp), hh, f);
            hop_f<R, 1, false>(a, w2, hh, f);
            hop_fence<R>();
            tile_project<R, ST, 1>(s_tile, loop_index<R>(nx.xm), hh, -f);
            hop_f<R, 1, true>(a, w3, hh, -f);
            hop_fence<R>();
            if (sizeof(R) == 4) {
                project_f<R, 0>(pf, hh, f);
                hop_f<R, 0, false>(a, w0, hh, f);
                project_f<R, 0>(pb, hh, -f);
                hop_f<R, 0, true>(a, w1, hh, -f);
            }
            cpx<R> sv[6], xv[6];
            give(a, PB{});
            hop_fence<R>();
            if (SELF || EPI == EPI_TS) load_half(A.self, col, sv, PB{});
            if (AUX) load_half(A.aux, col, xv, PB{});
            hop_fence<R>();
            __syncthreads();
            finish(col, a, sv, xv, PB{});
            hop_fence<R>();
            it++;
            prev = col;
            col = nxt;
            if (col >= col_hi) break;
        }
    } else {
        using PB = std::integral_constant<int, 1>;
        const int ym1 = (y == 0) ? (L - 1) * L : -L, zm1 = (z == 0) ? (L - 1) * L2 : -L2;
        bload_link_r<R, REC>(lrsrc(2, A.p_out), ls, h, w0);
        bload_link_r<R, REC>(lrsrc(2, 1 - A.p_out), ls, (s + ym1) >> 1, w1);
        bload_link_r<R, REC>(lrsrc(3, A.p_out), ls, h, w2);
        bload_link_r<R, REC>(lrsrc(3, 1 - A.p_out), ls, (s + zm1) >> 1, w3);
        if (sizeof(R) == 4) {
            col = next_col(col_lo);
            if (col >= col_hi) return;
            issue(col);
        }
        const BrickYZ nb = brick_yz(bk, bs, L, LH, NS, ic);
        for (;;) {
            const int nxt = next_col(col + 1);
            cpx<R> a[12], hh[6];
            if (sizeof(R) == 8) issue(col);
            hop_fence<R>();
            tile_put<R, ST>(s_tile, loop_index<R>(tid), q);
            hop_fence<R>();
            __syncthreads();
            if (sizeof(R) == 4 && nxt < col_hi) issue(nxt);
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
            cpx<R> sv[6], xv[6];
            give(a, PB{});
            hop_fence<R>();
            if (SELF || EPI == EPI_TS) load_half(A.self, col, sv, PB{});
            if (AUX) load_half(A.aux, col, xv, PB{});
            hop_fence<R>();
            __syncthreads();
            finish(col, a, sv, xv, PB{});
            hop_fence<R>();
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
