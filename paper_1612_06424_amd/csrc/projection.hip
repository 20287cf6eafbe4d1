// projection.hip -- quark-line projection (Sec. 3.3, Eqs. 16-17).
//
// The factorised propagator crosses a frontier through the field on one time
// slice (the slice the frontier hop reads).  Projecting that field on N_m
// orthonormal vectors phi_i, P_L = sum_i phi_i phi_i^+, cuts the quark line.
// The vectors come from inverse iteration of the Dirac operator of a slab Pi
// around the frontier, V <- orthonormalize(D_Pi^-1 V), restricted to the slice,
// spin-projected with the projector (1 +- gamma_0)/2 that the hop applies, and
// orthonormalised again.
//
// Orthonormalisation is Cholesky QR applied twice: G = V^+ V (N_m x N_m), G =
// R^+ R, V <- V R^-1.  Vectors are [N_m][n] complex128 (n = 12 x sites of the
// field, components outermost as in every field of the library).  The Gram
// matrix is summed from fixed per-workgroup partials in a fixed order, so the
// result is reproducible run to run.  Gram matrix and combination run on the FP64 matrix cores.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>

#include "dd_internal.h"
#include "dd_wilson.h"

namespace dd {

namespace {

typedef double dbl4 __attribute__((ext_vector_type(4)));

constexpr int kGT = 32;          // Gram tile: kGT x kGT outputs (2 x 2 matrix-core blocks) per workgroup
constexpr int kGThreads = 512;   // eight wavefronts, each 16 of every 128 rows
constexpr int kGBlocks = 512;    // workgroups aimed at: two per CU
constexpr int kCB = 32;          // output columns per workgroup of the combine kernel
constexpr int kCP = 64;          // rows of the small matrix staged in LDS at a time
constexpr int kCR = 2;           // blocks of 16 rows per wavefront of the combine kernel
constexpr int kCholLds = 64;     // largest matrix factorised in LDS

__device__ inline cpx<double> cj(cpx<double> a) { return {a.re, -a.im}; }

// v_mfma_f64_16x16x4f64: a 16 x 4 block (lane l holds A[l % 16][l / 16]) times a 4 x 16 block (lane l
// holds B[l / 16][l % 16]) into a 16 x 16 accumulator (lane l holds rows l / 16 + 4 e, e = 0..3, of
// column l % 16).
__device__ __forceinline__ dbl4 mfma(double a, double b, dbl4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// One workgroup's tile of a Gram partial: TA x TB blocks of 16 x 16 over the rows [r0, r1).  DIAG: A
// and B are the same vectors (TA = TB, the block below the diagonal left out).  A wavefront takes 16 rows
// per step: lane l holds rows base + l / 16 + 4 j (j = 0..3) of vector l % 16 of each block, so a load is
// 64 contiguous bytes of each of 16 vectors, and the four MFMAs of a row quartet contract them.  Vectors
// past the end repeat the last one (their outputs are not stored); rows past r1 count as zero.
template <bool DIAG, int TA, int TB>
__device__ __forceinline__ void xgram_tile(int a0, int b0, int na, int nb, long long n, long long r0, long long r1,
                                           const cpx<double>* __restrict__ A, const cpx<double>* __restrict__ B,
                                           cpx<double>* __restrict__ Gp, double (*sh)[512]) {
    const int tid = (int)threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const cpx<double>*pa[TA], *pb[TB];
#pragma unroll
    for (int t = 0; t < TA; t++) pa[t] = A + (size_t)min(a0 + t * 16 + (lane & 15), na - 1) * n;
#pragma unroll
    for (int t = 0; t < TB; t++) pb[t] = B + (size_t)min(b0 + t * 16 + (lane & 15), nb - 1) * n;
    dbl4 re[TA][TB], im[TA][TB];
#pragma unroll
    for (int t = 0; t < TA; t++)
#pragma unroll
        for (int u = 0; u < TB; u++) re[t][u] = im[t][u] = dbl4{0.0, 0.0, 0.0, 0.0};
    constexpr int kStep = 16 * (kGThreads / 64);
    for (long long base = r0 + wv * 16; base < r1; base += kStep) {
        cpx<double> va[TA][4], vb[TB][4];
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const long long i = base + (lane >> 4) + 4 * j;
            const bool ok = i < r1;
            const long long ic = ok ? i : r0;
#pragma unroll
            for (int t = 0; t < TA; t++) {
                va[t][j] = pa[t][ic];
                if (!ok) va[t][j] = cpx<double>{0.0, 0.0};
            }
            if constexpr (!DIAG) {
#pragma unroll
                for (int t = 0; t < TB; t++) {
                    vb[t][j] = pb[t][ic];
                    if (!ok) vb[t][j] = cpx<double>{0.0, 0.0};
                }
            }
        }
#pragma unroll
        for (int j = 0; j < 4; j++)
#pragma unroll
            for (int t = 0; t < TA; t++)
#pragma unroll
                for (int u = 0; u < TB; u++) {
                    if (DIAG && u < t) continue;
                    const cpx<double> x = va[t][j], y = DIAG ? va[u][j] : vb[u][j];
                    re[t][u] = mfma(x.re, y.re, re[t][u]);
                    im[t][u] = mfma(x.re, y.im, im[t][u]);
                    re[t][u] = mfma(x.im, y.im, re[t][u]);
                    im[t][u] = mfma(-x.im, y.re, im[t][u]);
                }
    }
    // the eight wavefronts' sums, in wavefront order
#pragma unroll
    for (int t = 0; t < TA; t++)
#pragma unroll
        for (int u = 0; u < TB; u++) {
            if (DIAG && u < t) continue;
#pragma unroll
            for (int e = 0; e < 4; e++) {
                sh[wv][((e * 4 + (lane >> 4)) * 16 + (lane & 15)) * 2] = re[t][u][e];
                sh[wv][((e * 4 + (lane >> 4)) * 16 + (lane & 15)) * 2 + 1] = im[t][u][e];
            }
            __syncthreads();
            double s = 0;
#pragma unroll
            for (int w = 0; w < kGThreads / 64; w++) s += sh[w][tid];
            const int a = a0 + t * 16 + tid / 32, b = b0 + u * 16 + (tid / 2) % 16;
            if (a < na && b < nb) reinterpret_cast<double*>(Gp + (size_t)a * nb + b)[tid & 1] = s;
            __syncthreads();
        }
}

// Gp[chunk][a][b] = sum over the chunk's `rows` rows i of conj(A[a][i]) B[b][i] (tile (ta, tb) of
// kGT x kGT; with sym, A = B, only the tiles ta <= tb).  The vectors are read once per tile, which bounds
// the time up to 32 vectors (one tile); the products take 15 us on the FP64 matrix cores.  24
// vectors, four calls of 8 x 16^3 and six of one slice: 36 us on average; products of scalars from LDS, a
// 16 x 16 tile and 8192 rows per workgroup, took 490.
__global__ __launch_bounds__(kGThreads, 2) void k_xgram_partial(int na, int nb, long long n, long long rows,
                                                                const cpx<double>* __restrict__ A,
                                                                const cpx<double>* __restrict__ B, int sym,
                                                                cpx<double>* __restrict__ Gp) {
    const int ta = blockIdx.x, tb = blockIdx.y, chunk = blockIdx.z;
    if (sym && ta > tb) return;  // uniform over the workgroup
    const long long r0 = (long long)chunk * rows, r1 = std::min(n, r0 + rows);
    __shared__ double sh[kGThreads / 64][512];
    const int a0 = ta * kGT, b0 = tb * kGT;
    Gp += (size_t)chunk * na * nb;
    const bool a1 = na - a0 <= 16, b1 = nb - b0 <= 16;  // one block of vectors is enough
    if (sym && ta == tb) {
        if (a1)
            xgram_tile<true, 1, 1>(a0, b0, na, nb, n, r0, r1, A, B, Gp, sh);
        else
            xgram_tile<true, 2, 2>(a0, b0, na, nb, n, r0, r1, A, B, Gp, sh);
    } else if (b1) {
        if (a1)
            xgram_tile<false, 1, 1>(a0, b0, na, nb, n, r0, r1, A, B, Gp, sh);
        else
            xgram_tile<false, 2, 1>(a0, b0, na, nb, n, r0, r1, A, B, Gp, sh);
    } else {
        xgram_tile<false, 2, 2>(a0, b0, na, nb, n, r0, r1, A, B, Gp, sh);
    }
}

// G[a][b] = sum of the partials (chunks k, k + 16, .. by thread k of 16, then those in order); with sym
// the lower triangle is the conjugate of the upper one.  16 entries per workgroup.
__global__ __launch_bounds__(256) void k_xgram_reduce(int na, int nb, int nchunk, int sym,
                                                      const cpx<double>* __restrict__ Gp, cpx<double>* __restrict__ G) {
    __shared__ cpx<double> sh[16][17];
    const int le = threadIdx.x & 15, lc = threadIdx.x >> 4;
    const int e = blockIdx.x * 16 + le;
    const bool ok = e < na * nb;
    const int a = ok ? e / nb : 0, b = ok ? e % nb : 0;
    const int ua = sym && a > b ? b : a, ub = sym && a > b ? a : b;
    cpx<double> s = {0.0, 0.0};
#pragma unroll 8
    for (int c = lc; c < nchunk; c += 16) s = s + Gp[((size_t)c * na + ua) * nb + ub];
    sh[lc][le] = s;
    __syncthreads();
    if (lc != 0 || !ok) return;
    for (int k = 1; k < 16; k++) s = s + sh[k][le];
    G[e] = (sym && a > b) ? cj(s) : s;
}

// One workgroup: G = R^+ R (R upper triangular, positive real diagonal), then Rinv = R^-1 (upper
// triangular, zeros below the diagonal).  flag = 1 if a pivot is not positive and finite (the vectors are
// linearly dependent in FP64).  Row elimination of [G | 1] in place: after step k, row k holds
// L^-1 = (R^-1)^+ up to column k and R behind it, and the rows below are updated by all threads at
// once, so the serial chain is n steps of two barriers (24 vectors: 15 us; pivots and rows computed from
// global memory one after the other, 255).  M is in LDS up to kCholLds vectors, in global memory above.
__device__ __forceinline__ void chol_inv(int n, cpx<double>* M, const cpx<double>* __restrict__ G,
                                         cpx<double>* __restrict__ Rinv, int* __restrict__ flag) {
    const int tid = (int)threadIdx.x, nth = (int)blockDim.x;
    bool bad = false;  // the same in every thread
    for (int e = tid; e < n * n; e += nth) M[e] = G[e];
    __syncthreads();
    for (int k = 0; k < n; k++) {
        double d = M[(size_t)k * n + k].re;
        if (!(d > 0.0) || !std::isfinite(d)) {
            bad = true;
            d = 1.0;
        }
        const double inv = 1.0 / sqrt(d);
        __syncthreads();  // the pivot has been read
        for (int c = tid; c < n; c += nth) {
            const cpx<double> v = M[(size_t)k * n + c];
            M[(size_t)k * n + c] = c == k ? cpx<double>{inv, 0.0} : cpx<double>{v.re * inv, v.im * inv};
        }
        __syncthreads();
        for (int e = tid; e < (n - k - 1) * n; e += nth) {
            const int i = k + 1 + e / n, c = e % n;
            if (c > k && c < i) continue;  // below the diagonal of what is left of G: never read
            const cpx<double> f = cj(M[(size_t)k * n + i]);  // R[k][i]^*
            const cpx<double> v = c == k ? cpx<double>{0.0, 0.0} : M[(size_t)i * n + c];
            M[(size_t)i * n + c] = v - f * M[(size_t)k * n + c];
        }
        __syncthreads();
    }
    for (int e = tid; e < n * n; e += nth) {
        const int i = e / n, j = e % n;  // R^-1[i][j] = (L^-1[j][i])^*
        Rinv[e] = i <= j ? cj(M[(size_t)j * n + i]) : cpx<double>{0.0, 0.0};
    }
    if (tid == 0 && bad) flag[0] = 1;
}
__global__ __launch_bounds__(512) void k_chol_inv(int n, const cpx<double>* __restrict__ G,
                                                  cpx<double>* __restrict__ Rinv, int* __restrict__ flag) {
    __shared__ cpx<double> M[kCholLds * kCholLds];
    chol_inv(n, M, G, Rinv, flag);
}
__global__ __launch_bounds__(1024) void k_chol_inv_global(int n, const cpx<double>* __restrict__ G, cpx<double>* M,
                                                          cpx<double>* __restrict__ Rinv, int* __restrict__ flag) {
    chol_inv(n, M, G, Rinv, flag);
}

// out[b][i] = sum_a A[a][i] M[a][b] for the kCB columns b of this workgroup (with tri, M is upper
// triangular).  M (na x nb) goes through LDS kCP rows at a time; a wavefront owns kCR blocks of 16 rows i
// and both blocks of 16 columns, so up to 32 columns A is read once, and a load or store is 256 contiguous
// bytes.  Bound by its two passes over the vectors: 24 vectors, four calls of 8 x 16^3 and six of one slice, 41 us
// on average (products of scalars, 16 columns per workgroup: 68).
__global__ __launch_bounds__(256) void k_combine(int na, int nb, long long n, const cpx<double>* __restrict__ A,
                                                 const cpx<double>* __restrict__ M, int tri,
                                                 cpx<double>* __restrict__ out) {
    __shared__ cpx<double> sm[kCP][kCB + 1];
    const int lane = (int)threadIdx.x & 63, wv = (int)threadIdx.x >> 6;
    const int b0 = blockIdx.y * kCB;
    const bool two = nb - b0 > 16;  // uniform over the workgroup
    const long long i0 = ((long long)blockIdx.x * 4 + wv) * (16 * kCR) + (lane & 15);
    long long ic[kCR];
#pragma unroll
    for (int r = 0; r < kCR; r++) ic[r] = std::min(i0 + 16 * r, n - 1);
    dbl4 re[2][kCR], im[2][kCR];
#pragma unroll
    for (int t = 0; t < 2; t++)
#pragma unroll
        for (int r = 0; r < kCR; r++) re[t][r] = im[t][r] = dbl4{0.0, 0.0, 0.0, 0.0};
    const int ka = tri ? std::min(na, b0 + kCB) : na;
    for (int p0 = 0; p0 < ka; p0 += kCP) {
        const int np = std::min(kCP, ka - p0), np4 = (np + 3) & ~3;
        if (p0) __syncthreads();  // the panel before has been used
        for (int e = threadIdx.x; e < np4 * kCB; e += 256) {
            const int a = e / kCB, j = e % kCB;
            sm[a][j] = (a < np && b0 + j < nb) ? M[(size_t)(p0 + a) * nb + b0 + j] : cpx<double>{0.0, 0.0};
        }
        __syncthreads();
#pragma unroll 4
        for (int a = 0; a < np4; a += 4) {
            const int al = a + (lane >> 4);
            const bool ok = al < np;
            const cpx<double>* row = A + (size_t)(p0 + (ok ? al : 0)) * n;
            cpx<double> v[kCR];
#pragma unroll
            for (int r = 0; r < kCR; r++) {
                v[r] = row[ic[r]];
                if (!ok) v[r] = cpx<double>{0.0, 0.0};  // (an infinity of another vector must not meet a zero of M)
            }
#pragma unroll
            for (int t = 0; t < 2; t++) {
                if (t == 1 && !two) break;
                const cpx<double> m = sm[al][t * 16 + (lane & 15)];
#pragma unroll
                for (int r = 0; r < kCR; r++) {
                    re[t][r] = mfma(m.re, v[r].re, re[t][r]);
                    im[t][r] = mfma(m.re, v[r].im, im[t][r]);
                    re[t][r] = mfma(-m.im, v[r].im, re[t][r]);
                    im[t][r] = mfma(m.im, v[r].re, im[t][r]);
                }
            }
        }
    }
#pragma unroll
    for (int t = 0; t < 2; t++)
#pragma unroll
        for (int r = 0; r < kCR; r++)
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const int b = b0 + t * 16 + (lane >> 4) + 4 * e;
                const long long i = i0 + 16 * r;
                if (b < nb && i < n) out[(size_t)b * n + i] = cpx<double>{re[t][r][e], im[t][r][e]};
            }
}

// W[a][c][s] = ((1 + SGN gamma_0)/2 V[a] on slice k of the slab)_c(s)
template <int SGN>
__global__ __launch_bounds__(256) void k_slice_project(int nvec, int L3, int nsite, int k,
                                                       const cpx<double>* __restrict__ V, cpx<double>* __restrict__ W) {
    const int s = blockIdx.x * 256 + threadIdx.x;
    const int a = blockIdx.y;
    if (s >= L3 || a >= nvec) return;
    cpx<double> p[12], h[6], o[12];
#pragma unroll
    for (int c = 0; c < 12; c++) {
        p[c] = V[((size_t)a * 12 + c) * nsite + (size_t)k * L3 + s];
        o[c] = cpx<double>{0.0, 0.0};
    }
    project<double, 0, SGN>(p, h);
    accum<double, 0, SGN>(o, h);
#pragma unroll
    for (int c = 0; c < 12; c++) W[((size_t)a * 12 + c) * L3 + s] = cpx<double>{0.5 * o[c].re, 0.5 * o[c].im};
}

// Partials of a Gram matrix: as many as fill kGBlocks workgroups, each of at least one step of rows.
int gram_max_chunks(int na, int nb) {
    return std::max(1, kGBlocks / (((na + kGT - 1) / kGT) * ((nb + kGT - 1) / kGT)));
}

// G = A^+ B (na x nb); Gp: gram_max_chunks x na x nb scratch
void launch_xgram(dd_ctx* c, int na, int nb, long long n, const cpx<double>* A, const cpx<double>* B, bool sym,
                  cpx<double>* Gp, cpx<double>* G) {
    const long long step = 16 * (kGThreads / 64), want = gram_max_chunks(na, nb);
    const long long rows = ((n + want - 1) / want + step - 1) / step * step;
    const int nchunk = (int)((n + rows - 1) / rows);
    const dim3 grid((unsigned)((na + kGT - 1) / kGT), (unsigned)((nb + kGT - 1) / kGT), (unsigned)nchunk);
    hipLaunchKernelGGL(k_xgram_partial, grid, dim3(kGThreads), 0, c->stream, na, nb, n, rows, A, B,
                       sym ? 1 : 0, Gp);
    hipLaunchKernelGGL(k_xgram_reduce, dim3((unsigned)((na * nb + 15) / 16)), dim3(256), 0, c->stream, na, nb,
                       nchunk, sym ? 1 : 0, Gp, G);
}

void launch_combine(dd_ctx* c, int na, int nb, long long n, const cpx<double>* A, const cpx<double>* M, bool tri,
                    cpx<double>* out) {
    const long long per = 4 * 16 * kCR;
    const dim3 grid((unsigned)((n + per - 1) / per), (unsigned)((nb + kCB - 1) / kCB));
    hipLaunchKernelGGL(k_combine, grid, dim3(256), 0, c->stream, na, nb, n, A, M, tri ? 1 : 0, out);
}

struct OrthoWork {
    cpx<double>* Gp;
    cpx<double>* G;
    cpx<double>* R;
    cpx<double>* Rinv;
    int* flag;
};

// scratch of Gram matrices na x nb
dd_status ortho_work(dd_ctx* c, int na, int nb, OrthoWork* w) {
    dd_status e = DD_OK;
    const size_t nn = (size_t)na * nb;
    w->Gp = (cpx<double>*)workspace(c, W_PROJ_G, (size_t)gram_max_chunks(na, nb) * nn * sizeof(cpx<double>), &e);
    if (e != DD_OK) return e;
    cpx<double>* m = (cpx<double>*)workspace(c, W_PROJ_R, (3 * nn + 1) * sizeof(cpx<double>), &e);
    if (e != DD_OK) return e;
    w->G = m;
    w->R = m + nn;
    w->Rinv = m + 2 * nn;
    w->flag = (int*)(m + 3 * nn);
    return DD_OK;
}

// out = V R^-1 twice (Cholesky QR 2); V and tmp are overwritten
void orthonormalize(dd_ctx* c, int nvec, long long n, cpx<double>* V, cpx<double>* tmp, const OrthoWork& w) {
    for (int pass = 0; pass < 2; pass++) {
        cpx<double>* src = pass == 0 ? V : tmp;
        cpx<double>* dst = pass == 0 ? tmp : V;
        launch_xgram(c, nvec, nvec, n, src, src, true, w.Gp, w.G);
        if (nvec <= kCholLds)
            hipLaunchKernelGGL(k_chol_inv, dim3(1), dim3(512), 0, c->stream, nvec, w.G, w.Rinv, w.flag);
        else
            hipLaunchKernelGGL(k_chol_inv_global, dim3(1), dim3(1024), 0, c->stream, nvec, w.G, w.R, w.Rinv, w.flag);
        launch_combine(c, nvec, nvec, n, src, w.Rinv, true, dst);
    }
}

}  // namespace

// Quark-line projection vectors of the frontier hop that leaves slice k of the
// slab g (the region Pi around the frontier) forward (sign = +1) or backward
// (-1): inverse iteration from v0 ([nvec][12][|Pi|]), n_iter solves of 12
// columns at a time, Cholesky QR 2 after each, then restriction to slice k,
// spin projection and Cholesky QR 2 into phi ([nvec][12][L^3]).
dd_status projection_basis(dd_ctx* c, const cpx<double>* U, double kappa, const Geo& g, int k, int sign, int nvec,
                           int n_iter, const cpx<double>* v0, cpx<double>* phi, const dd_solver_params& p,
                           dd_solve_stats* stats) {
    const auto t_start = std::chrono::steady_clock::now();
    dd_status e = DD_OK;
    const int L3 = g.L3, npi = g.nsite;
    const long long n = 12LL * npi, ns = 12LL * L3;
    cpx<double>* V = (cpx<double>*)workspace(c, W_PROJ_V, 2 * (size_t)nvec * n * sizeof(cpx<double>), &e);
    if (e != DD_OK) return e;
    cpx<double>* Vt = V + (size_t)nvec * n;
    OrthoWork w;
    if ((e = ortho_work(c, nvec, nvec, &w)) != DD_OK) return e;
    DD_HIP(c, hipMemsetAsync(w.flag, 0, sizeof(int), c->stream));
    DD_HIP(c, hipMemcpyAsync(V, v0, (size_t)nvec * n * sizeof(cpx<double>), hipMemcpyDeviceToDevice, c->stream));
    orthonormalize(c, nvec, n, V, Vt, w);
    DD_HIP(c, hipGetLastError());
    int flag = 0;
    DD_HIP(c, hipMemcpyAsync(&flag, w.flag, sizeof(int), hipMemcpyDeviceToHost, c->stream));
    DD_HIP(c, hipStreamSynchronize(c->stream));
    if (flag) return fail(c, DD_ERR_BREAKDOWN, "start vectors linearly dependent in FP64");
    dd_solve_stats tot;
    std::memset(&tot, 0, sizeof(tot));
    tot.nrhs = nvec;
    dd_status worst = DD_OK;
    for (int it = 0; it < n_iter; it++) {
        // V <- D_Pi^-1 V, DD_MAX_RHS columns per solve
        for (int a0 = 0; a0 < nvec; a0 += DD_MAX_RHS) {
            const int nc = std::min(DD_MAX_RHS, nvec - a0);
            dd_solve_stats st;
            e = solve(c, U, kappa, g, nc, V + (size_t)a0 * n, Vt + (size_t)a0 * n, p, &st, 0);
            if (e != DD_OK && e != DD_ERR_NOCONV) return e;
            if (e == DD_ERR_NOCONV) worst = e;
            tot.iters += st.iters;
            tot.updates += st.updates;
            tot.restarts += st.restarts;
            for (int j = 0; j < nc; j++) tot.true_rel_resid[0] = std::max(tot.true_rel_resid[0], st.true_rel_resid[j]);
        }
        std::swap(V, Vt);
        orthonormalize(c, nvec, n, V, Vt, w);
        DD_HIP(c, hipGetLastError());
    }
    const dim3 sg((unsigned)((L3 + 255) / 256), (unsigned)nvec);
    if (sign > 0)
        hipLaunchKernelGGL(k_slice_project<1>, sg, dim3(256), 0, c->stream, nvec, L3, npi, k, V, phi);
    else
        hipLaunchKernelGGL(k_slice_project<-1>, sg, dim3(256), 0, c->stream, nvec, L3, npi, k, V, phi);
    orthonormalize(c, nvec, ns, phi, Vt, w);
    DD_HIP(c, hipGetLastError());
    DD_HIP(c, hipMemcpyAsync(&flag, w.flag, sizeof(int), hipMemcpyDeviceToHost, c->stream));
    DD_HIP(c, hipStreamSynchronize(c->stream));
    tot.ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t_start).count();
    if (stats) *stats = tot;
    if (flag) return fail(c, DD_ERR_BREAKDOWN, "projection vectors linearly dependent in FP64");
    if (worst != DD_OK) return fail(c, worst, "an inverse-iteration solve did not converge: " + c->err);
    return DD_OK;
}

// field (ncol columns of a slab of nt slices, [ncol][12][nt L3]): slice k replaced by
// P_L of it, P_L = sum_i phi_i phi_i^+ with phi [nvec][12][L3] orthonormal
dd_status project_slice(dd_ctx* c, int L3, int nt, int k, int ncol, cpx<double>* field, int nvec,
                        const cpx<double>* phi) {
    dd_status e = DD_OK;
    const long long ns = 12LL * L3;
    cpx<double>* buf = (cpx<double>*)workspace(c, W_PROJ_V, 2 * (size_t)ncol * ns * sizeof(cpx<double>), &e);
    if (e != DD_OK) return e;
    cpx<double>* out = buf + (size_t)ncol * ns;
    OrthoWork w;
    if ((e = ortho_work(c, nvec, ncol, &w)) != DD_OK) return e;
    launch_slab_embed(c, L3, nt, k, 1, ncol, buf, field, 1);        // the slice, [ncol][12][L3]
    launch_xgram(c, nvec, ncol, ns, phi, buf, false, w.Gp, w.G);    // C = phi^+ field (nvec x ncol)
    launch_combine(c, nvec, ncol, ns, phi, w.G, false, out);                // phi C
    launch_slab_embed(c, L3, nt, k, 1, ncol, out, field, 0);
    DD_HIP(c, hipGetLastError());
    return DD_OK;
}

}  // namespace dd
