// dd_gemm_plan.h -- tile width and k splits of the baryon-block product (nucleon.hip).  Host arithmetic only,
// without HIP, so that the host tests compile it as it is.
#pragma once

#include <algorithm>
#include <cstddef>

namespace dd {

constexpr int kGM = 64, kGK = 16;  // rows of a workgroup's tile (complex entries) and k step

// The product's launch: blocks of 16 columns per wavefront (tile width 32 nj) and splits of the k range for a matrix
// M x N and nkt steps of k.  Both are those of the least estimated time of the product and of writing and adding the
// partial results, with at most about 16 workgroups per CU in all.  A step of a wavefront is 32 nj MFMAs of 64
// cycles; w workgroups on a CU share its matrix cores, and a step has 1.1 us of latency that only the others
// hide; `fit` workgroups run per CU, the last round with as many as are left, and a tenth of a round is lost to
// uneven ends.  The factors: one block has twice the LDS reads per MFMA that two have (16^3, 96 vectors, nothing
// padded: 6305 us and 6092), three leave two wavefronts per SIMD (6190).  So 480 columns (120 vectors) are
// taken by threes on 16^3 (11.82 ms; twos pad to 512 and take 12.19), but on 12^3, with fewer steps to split,
// by twos (5.36 and 5.53).  Blocks on one 16^3 slice, two blocks and 16 workgroups per CU throughout and
// so, ms: 4 vectors 0.23 and 0.075, 24 0.27 and 0.15, 48 0.61 and 0.54, 80 1.92 and 1.87; two 4^3 slices, 24
// vectors: 0.046 and 0.042; two 8^3 slices, 192: 6.45 and 6.36.
struct GemmPlan {
    int nj, ns;
};
inline GemmPlan zgemm_plan(size_t M, int N, int nkt) {
    GemmPlan best{1, 1};
    double best_us = 1e300;
    for (int nj = 1; nj <= 3; nj++) {
        const int ntile = (int)(((M + kGM - 1) / kGM) * ((N + 32 * nj - 1) / (32 * nj)));
        const int fit = nj == 3 ? 2 : nj == 2 ? 3 : 5, lim = std::max(1, std::min(nkt, (16 * 256 + ntile - 1) / ntile));
        const double mfma = 2048.0 * nj / 2.35e3;  // us of a step per workgroup on the CU
        const double factor = nj == 1 ? 1.08 : nj == 2 ? 1.0 : 1.03;
        const auto step = [&](long long w) { return w ? std::max((double)w * mfma, mfma + 1.1) : 0.0; };
        for (int ns = 1; ns <= lim;) {  // the least ns of each count of steps per split
            const int kps = (nkt + ns - 1) / ns;
            const long long wgs = (long long)ntile * ns, full = wgs / (256 * fit), rem = wgs % (256 * fit);
            const double us = factor * (kps * ((double)full * step(fit) + step((rem + 255) / 256) + 0.1 * step(fit)) +
                                        ns * (0.15 + (double)(M * N) * 2 * 16 / 5e6));
            if (us < best_us) {
                best_us = us;
                best = GemmPlan{nj, ns};
            }
            if (kps == 1) break;
            ns = (nkt + kps - 2) / (kps - 1);
        }
    }
    return best;
}

}  // namespace dd
