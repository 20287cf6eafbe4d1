// dirac_tile.hip -- launches of the Wilson-Dirac stencil's LDS-tile form on one lattice or slab
// (the arithmetic lives in dd_dslash_tile.h).
#include "dd_dslash_tile.h"

namespace dd {

namespace {

// workgroup -> brick, then group of cpw columns
template <typename R, int EPI>
__global__ __launch_bounds__(kDslNT, 2) void k_dslash_lds(Geo g, EoTile ts, TileArgs<R> a, int ncol, int cpw,
                                                         int remap) {
    const int lb = remap ? xcd_remap(blockIdx.x, gridDim.x) : (int)blockIdx.x;
    const int grp = lb / a.nblk;
    dslash_lds_body<R, EPI>(g, ts, a, lb - grp * a.nblk, grp * cpw, min(ncol, grp * cpw + cpw));
}

}  // namespace

bool dslash_lds_ok(const Geo& g, size_t real_bytes) { return dslash_tile_ok(g.L, g.nt, real_bytes); }

bool dslash_lds_form(const Geo& g, size_t real_bytes, int ncol, bool sums) {
    return dslash_tile_form(g.L, g.nt, ncol, real_bytes, stencil_timed(g, ncol), sums);
}

int dslash_lds_blocks(const Geo& g) { return eo_tile_blocks(dslash_tile_shape(g.L, g.nt)); }

template <typename R>
void launch_dslash_lds(dd_ctx* c, const Geo& g, const StencilSched& sc, const cpx<R>* U, R mass, int dag, int epi,
                       const cpx<R>* in, cpx<R>* out, const cpx<R>* aux, int ncol, double* partial,
                       const ColState* st) {
    const EoTile ts = dslash_tile_shape(g.L, g.nt);
    TileArgs<R> a;
    a.U = U;
    a.in = in;
    a.out = out;
    a.aux = aux;
    a.mass = mass;
    a.f = R(dag ? 1 : -1);
    a.st = st;
    a.partial = partial;
    a.nblk = eo_tile_blocks(ts);
    const int cpw = sc.kc < 1 ? 1 : (sc.kc < ncol ? sc.kc : ncol);
    const dim3 grid((unsigned)(a.nblk * ((ncol + cpw - 1) / cpw))), block(kDslNT);
#define DD_LDS_CASE(E) \
    hipLaunchKernelGGL((k_dslash_lds<R, E>), grid, block, 0, c->stream, g, ts, a, ncol, cpw, sc.remap)
    switch (epi) {
        case EPI_STORE: DD_LDS_CASE(EPI_STORE); break;
        case EPI_DOT_AUX: DD_LDS_CASE(EPI_DOT_AUX); break;
        case EPI_TS: DD_LDS_CASE(EPI_TS); break;
        case EPI_RESID: DD_LDS_CASE(EPI_RESID); break;
        case EPI_HOP: DD_LDS_CASE(EPI_HOP); break;
        default: DD_LDS_CASE(EPI_NORM); break;
    }
#undef DD_LDS_CASE
}

template void launch_dslash_lds<double>(dd_ctx*, const Geo&, const StencilSched&, const cpx<double>*, double, int, int,
                                        const cpx<double>*, cpx<double>*, const cpx<double>*, int, double*,
                                        const ColState*);
template void launch_dslash_lds<float>(dd_ctx*, const Geo&, const StencilSched&, const cpx<float>*, float, int, int,
                                       const cpx<float>*, cpx<float>*, const cpx<float>*, int, double*,
                                       const ColState*);

}  // namespace dd
