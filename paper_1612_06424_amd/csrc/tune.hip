// tune.hip -- per-context autotuner of the stencil launch shape.
//
// The best (workgroup size, time-chunk length, XCD remap, columns per thread,
// tile shape and order) depends on the precision, the number of columns and the
// lattice geometry (how many
// workgroups are resident per XCD against how much of the 4 MB L2 one time
// slice of them touches).  The first launch for a new key times every
// candidate of its form on scratch buffers of the same size (best of three timings)
// and keeps the fastest; later launches reuse it.  Small problems use the default
// shape untimed.  Which form a launch takes (the sweep or the LDS tile) depends on its
// sizes only (dslash_tile_form), and the shapes of a form differ in nothing but
// speed, so a timing never decides a bit of D's result.
//
// With the environment variable DD_TUNE_CACHE naming a file, a new context
// loads the choices stored there and every new choice is appended to it, so
// that separate processes (for instance the passes of a profiler) launch the
// same shapes.
#include <algorithm>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <fstream>
#include <sstream>
#include <string>

#include "dd_internal.h"

namespace dd {

namespace {

std::string key_of(const Geo& g, int kind, int ncol) {
    return std::to_string(kind) + ":" + std::to_string(ncol) + ":" + std::to_string(g.L) + ":" +
           std::to_string(g.T) + ":" + std::to_string(g.nt) + ":" + std::to_string(g.whole);
}

template <typename R>
StencilSched tune(dd_ctx* c, const Geo& g, int ncol, bool sums) {  // sums: timed with |D in|^2
    StencilSched best = default_sched(g, sizeof(R) == 8 ? 0 : 1, ncol, sums);
    const size_t nf = (size_t)ncol * 12 * g.nsite, nl = (size_t)36 * g.vlink;
    // slots of the shapes below: tiles of 128 sites and chunks of one slice, or bricks
    const size_t slots = std::max((size_t)((g.L3 + 127) / 128) * g.nt, (size_t)dslash_lds_blocks(g)) * ncol;
    cpx<R>*in = nullptr, *out = nullptr, *U = nullptr;
    double* partial = nullptr;
    if (hipMalloc(&in, nf * sizeof(cpx<R>)) != hipSuccess || hipMalloc(&out, nf * sizeof(cpx<R>)) != hipSuccess ||
        hipMalloc(&U, nl * sizeof(cpx<R>)) != hipSuccess ||
        (sums && hipMalloc((void**)&partial, slots * 3 * sizeof(double)) != hipSuccess)) {
        (void)hipGetLastError();
        if (in) (void)hipFree(in);
        if (out) (void)hipFree(out);
        if (U) (void)hipFree(U);
        return best;
    }
    (void)hipMemsetAsync(in, 0, nf * sizeof(cpx<R>), c->stream);
    (void)hipMemsetAsync(U, 0, nl * sizeof(cpx<R>), c->stream);
    hipEvent_t e0, e1;
    (void)hipEventCreate(&e0);
    (void)hipEventCreate(&e1);
    const int saved_timing = c->timing;
    c->timing = 0;
    float best_ms = 1e30f;
    auto time_shape = [&](const StencilSched& sc) {
        auto time = [&](int n) {
            (void)hipEventRecord(e0, c->stream);
            for (int r = 0; r < n; r++)
                launch_dslash_sched<R>(c, g, sc, U, 0.125, 0, sums ? EPI_NORM : EPI_STORE, in, out, nullptr, ncol,
                                        partial, nullptr);
            (void)hipEventRecord(e1, c->stream);
            (void)hipEventSynchronize(e1);
            float t = 0;
            (void)hipEventElapsedTime(&t, e0, e1);
            return t;
        };
        // after a first launch, the best of three timings of three launches each (one timing picked
        // shapes by noise); a shape whose first timing is far behind is not timed again
        (void)time(1);
        float ms = 1e30f;
        for (int rep = 0; rep < 3; rep++) {
            const float t = time(3);
            ms = t < ms ? t : ms;
            if (ms > 1.3f * best_ms) return;
        }
        if (ms < best_ms) {
            best_ms = ms;
            best = sc;
        }
    };
    // the LDS-tile form, the columns in 1 to 3 groups
    const bool tile = (best.blocked & 8) != 0;
    for (int parts = 1; tile && parts <= 3 && parts <= ncol; parts++) {
        StencilSched sc = best;
        sc.kc = (ncol + parts - 1) / parts;
        time_shape(sc);
    }
    const int tcs[] = {1, 2, 4, 8, 16, 1 << 20};
    const bool large = (size_t)g.nsite * ncol > (size_t)1 << 21;  // short chunks only fill the chip on smaller fields
    for (int kc = 1; !tile && kc <= 4; kc++)
    for (int nt : {128, 256})
        for (int tcv : tcs)
            for (int remap : {0, 1})
            for (int bl = 0; bl < 4; bl++) {
                StencilSched sc;
                sc.nt = nt;
                sc.tc = tcv > g.nt ? g.nt : tcv;
                sc.remap = remap;
                sc.kc = kc;
                sc.blocked = bl;
                if (large && tcv < 4) continue;
                if (tcv != sc.tc && tcv != (1 << 20)) continue;  // same as a shorter candidate
                if (sched_kc(sc, ncol, sizeof(R), (size_t)12 * g.nsite * sizeof(cpx<R>)) != kc) continue;
                if ((bl & 1) && brick_rows(g, nt) == 0) continue;          // bricks do not fit
                if ((bl & 2) && (g.nt + sc.tc - 1) / sc.tc < 2) continue;  // one chunk: the same order
                time_shape(sc);
            }
    c->timing = saved_timing;
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    (void)hipStreamSynchronize(c->stream);
    (void)hipFree(in);
    (void)hipFree(out);
    (void)hipFree(U);
    if (partial) (void)hipFree(partial);
    (void)hipGetLastError();
    return best;
}

}  // namespace

void tune_cache_load(dd_ctx* c) {
    const char* path = std::getenv("DD_TUNE_CACHE");
    if (path == nullptr || *path == 0) return;
    std::ifstream f(path);
    std::string line;
    while (std::getline(f, line)) {
        // key nt tc remap [kc [blocked]]
        std::istringstream in(line);
        std::string key;
        StencilSched sc;
        if (!(in >> key >> sc.nt >> sc.tc >> sc.remap)) continue;
        if (!(in >> sc.kc)) sc.kc = 1;
        if (!(in >> sc.blocked)) sc.blocked = 0;
        c->sched[key] = sc;
    }
}

void tune_cache_store(dd_ctx* c, const std::string& key, const StencilSched& sc) {
    c->sched[key] = sc;
    const char* path = std::getenv("DD_TUNE_CACHE");
    if (path == nullptr || *path == 0) return;
    std::ofstream f(path, std::ios::app);
    f << key << " " << sc.nt << " " << sc.tc << " " << sc.remap << " " << sc.kc << " " << sc.blocked << "\n";
}

StencilSched stencil_sched(dd_ctx* c, const Geo& g, int kind, int ncol, bool sums) {
    // launches with sums have a shape of their own where they take the other form, and in solves of the full operator,
    // which launch hardly anything else: the FP32 sweep with sums pays for two columns per thread what the one
    // without does not (16 x 17^3, 4 columns: 51 us a launch in D's shape, 39 in its own)
    const size_t rb = kind == 0 ? 8 : 4;
    const bool own = sums && stencil_timed(g, ncol) &&
                     (c->full_solve || dslash_lds_form(g, rb, ncol, true) != dslash_lds_form(g, rb, ncol, false));
    const std::string k = (own ? "s" : "") + key_of(g, kind, ncol);
    auto it = c->sched.find(k);
    if (it != c->sched.end()) {
        StencilSched hit = it->second;  // (a stored shape may name a form that does not fit the field)
        if ((hit.blocked & 8) && !dslash_lds_ok(g, rb)) hit.blocked = 0;
        return hit;
    }
    StencilSched sc = default_sched(g, kind, ncol, sums);
    if (c->autotune && stencil_timed(g, ncol))
        sc = kind == 0 ? tune<double>(c, g, ncol, sums) : tune<float>(c, g, ncol, sums);
    tune_cache_store(c, k, sc);
    return sc;
}

int stencil_slots(dd_ctx* c, const Geo& g, int kind, int ncol) {
    return stencil_blocks(g, stencil_sched(c, g, kind, ncol, true));
}

}  // namespace dd
