"""The baryon-block product's launch plan (dd_gemm_plan.h, compiled as it is by the host compiler) over every
vector count and a range of chunk sizes, and a host emulation of the product's index arithmetic at the three
tile widths it is launched with (32, 64 and 96 columns: 1, 2 and 3 blocks of 16 per wavefront).

The emulation restates the kernel's panel staging (thread t: A entries (t % 64, t / 64 + 4 r), B entries
(t % 16, t / 16 + 16 r), r < 2 blocks), its split of a tile over four wavefronts (32 rows x 16 blocks columns each) and
the lane layout of v_mfma_f64_16x16x4f64 (lane l holds A[l % 16][l / 16], B[l / 16][l % 16] and rows l / 16 + 4 e of
column l % 16 of the result).
"""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from conftest import ROOT

CSRC = os.path.join(ROOT, "paper_1612_06424_amd", "csrc")
SRC = """
#include "dd_gemm_plan.h"
extern "C" void plan(long long M, int N, int nkt, int* s) {
    dd::GemmPlan p = dd::zgemm_plan((size_t)M, N, nkt); s[0] = p.nj; s[1] = p.ns; }
"""
GM, GK = 64, 16


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("gemm")
    (d / "s.cpp").write_text(SRC)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-shared", "-fPIC", "-I", CSRC, str(d / "s.cpp"),
                           "-o", str(d / "s.so")])
    lib = ctypes.CDLL(str(d / "s.so"))

    def call(M, N, nkt):
        s = (ctypes.c_int * 2)()
        lib.plan(ctypes.c_longlong(M), N, nkt, s)
        return s[0], s[1]
    return call


def test_plans_are_launchable(plan):
    seen = set()
    for n in range(1, 257):
        M, N = n * (n + 1) // 2, 4 * n
        for sites in (1, 5, 27, 64, 200, 512, 1728, 4096, 32768):
            if M * 3 * sites * 16 >= 2 ** 31:
                continue
            nkt = -(-3 * sites // GK)
            nj, ns = plan(M, N, nkt)
            seen.add(nj)
            assert 1 <= nj <= 3 and 1 <= ns <= nkt
            kps = -(-nkt // ns)
            assert (ns - 1) * kps < nkt <= ns * kps, "every split has a step, all steps are in one"
            tiles = -(-M // GM) * -(-N // (32 * nj))
            assert ns == 1 or tiles * (ns - 1) < 16 * 256, "about 16 workgroups per CU at most"
            # a shorter last chunk, run with the same plan, has no more splits
            for last in {1, nkt // 2 or 1, nkt}:
                k = -(-last // ns)
                assert -(-last // k) <= ns
    assert seen == {1, 2, 3}


def mfma(a, b, c):
    A = np.zeros((16, 4))
    B = np.zeros((4, 16))
    lanes = np.arange(64)
    A[lanes % 16, lanes // 16] = a
    B[lanes // 16, lanes % 16] = b
    D = A @ B
    out = c.copy()
    for e in range(4):
        out[:, e] += D[lanes // 16 + 4 * e, lanes % 16]
    return out


def emulate(A, B, nj, ns, slip=False):
    """Sum of the splits' C, and how often each entry of each split was written; slip: a wavefront's columns start
    at 32 instead of 16 nj (the planted mistake)."""
    M, K = A.shape
    N = B.shape[1]
    gn = 32 * nj
    tm, tn, nkt = -(-M // GM), -(-N // gn), -(-K // GK)
    kps = -(-nkt // ns)
    nsplit = -(-nkt // kps)
    C = np.zeros((nsplit, M, N), complex)
    written = np.zeros((nsplit, M, N), int)
    lanes = np.arange(64)
    t = np.arange(256)
    for w in range(tm * tn * nsplit):
        nt, mt, sp = w % tn, (w // tn) % tm, w // (tn * tm)
        m0, n0 = mt * GM, nt * gn
        acc = np.zeros((4, 2, nj, 2, 64, 4))
        for kt in range(sp * kps, min(nkt, sp * kps + kps)):
            k0 = kt * GK
            As = np.full((GK, GM), np.nan, complex)
            Bs = np.full((GK, gn), np.nan, complex)
            for r in range(4):
                m, k = m0 + (t & 63), k0 + (t >> 6) + 4 * r
                ok = (m < M) & (k < K)
                As[(t >> 6) + 4 * r, t & 63] = np.where(ok, A[np.minimum(m, M - 1), np.minimum(k, K - 1)], 0)
            for r in range(2 * nj):
                k, n = k0 + (t & 15), n0 + (t >> 4) + 16 * r
                ok = (k < K) & (n < N)
                Bs[t & 15, (t >> 4) + 16 * r] = np.where(ok, B[np.minimum(k, K - 1), np.minimum(n, N - 1)], 0)
            assert not np.isnan(As).any() and not np.isnan(Bs).any(), "the panels are staged in full"
            for wv in range(4):
                wm, wn = wv & 1, wv >> 1
                for ks in range(GK // 4):
                    kk = 4 * ks + (lanes >> 4)
                    for i in range(2):
                        a = As[kk, wm * 32 + i * 16 + (lanes & 15)]
                        for j in range(nj):
                            b = Bs[kk, (wn * (32 if slip else 16 * nj) + j * 16 + (lanes & 15)) % gn]
                            re, im = acc[wv, i, j]
                            re = mfma(a.imag, -b.imag, mfma(a.real, b.real, re))
                            im = mfma(a.imag, b.real, mfma(a.real, b.imag, im))
                            acc[wv, i, j] = re, im
        for wv in range(4):
            wm, wn = wv & 1, wv >> 1
            for i in range(2):
                for j in range(nj):
                    for e in range(4):
                        row = m0 + wm * 32 + i * 16 + (lanes >> 4) + 4 * e
                        col = n0 + wn * 16 * nj + j * 16 + (lanes & 15)
                        ok = (row < M) & (col < N)
                        C[sp, row[ok], col[ok]] = acc[wv, i, j, 0][ok, e] + 1j * acc[wv, i, j, 1][ok, e]
                        np.add.at(written, (sp, row[ok], col[ok]), 1)
    return C.sum(0), written


def _matrices(M, N, K):
    rng = np.random.default_rng(M + N + K)
    return (rng.standard_normal((M, K)) + 1j * rng.standard_normal((M, K)),
            rng.standard_normal((K, N)) + 1j * rng.standard_normal((K, N)))


@pytest.mark.parametrize("nj", [1, 2, 3])
@pytest.mark.parametrize("M,N,K,ns", [(1, 4, 48, 3), (70, 96, 33, 2), (65, 100, 20, 1), (15, 33, 50, 4)])
def test_every_entry_once_and_the_product(M, N, K, ns, nj):
    A, B = _matrices(M, N, K)
    C, written = emulate(A, B, nj, ns)
    assert (written == 1).all()
    ref = A @ B
    assert np.abs(C - ref).max() < 1e-12 * np.abs(ref).max()


@pytest.mark.parametrize("nj", [1, 3])
def test_a_wrong_column_origin_is_caught(nj):
    A, B = _matrices(15, 60, 30)
    C, _ = emulate(A, B, nj, 1, slip=True)
    assert np.abs(C - A @ B).max() > 1e-3
