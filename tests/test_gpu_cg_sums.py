"""GPU check of CGNR's sums: rows of partial slots added up by the vector kernels themselves (one slot,
several, nearly as many as that allows) and by a launch of their own, with columns that stop at different
iterations and one that never starts.

The residual is recomputed by the oracle in FP64: |b - D x| <= 1.1 tol |b| at tol = 1e-10 (the oracle's
rounding is 1e-13).
"""
import numpy as np
import pytest
import torch

import oracle as O
from helpers import gaussian_field, lib, random_links, step

pytestmark = pytest.mark.gpu

KAPPA, TOL = 0.12, 1e-10


@pytest.mark.parametrize("T,L,precond", [(4, 4, "eo"), (5, 5, "none"), (16, 8, "eo"), (12, 30, "eo"), (16, 32, "eo")])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_cgnr_residuals(T, L, precond, prec):
    dd = lib()
    step(f"CGNR sums T={T} L={L} {precond} {prec}")
    U = random_links(T, L, 0.3, 9100)
    ncol = 3 if L < 20 else 2
    b = gaussian_field(T * L ** 3, ncol, 9101)
    b[-1] = 0
    if ncol > 2:
        b[1] = 0
        b[1, 3, 2] = 1.0  # a point source stops at another iteration; the last column is zero
    p = dd.solver_params(tol=TOL, solver=dd.DD_CGNR, prec=dd.DD_FP64 if prec == "fp64" else dd.DD_MIXED,
                         precond=dd.DD_PRECOND_EO if precond == "eo" else dd.DD_PRECOND_NONE)
    ctx = dd.Context(T, L, -1)
    x, st = dd.block_solve(ctx, dd.pack_links(U), KAPPA, dd.pack_field(b), None, p)
    x = dd.unpack_field(x)
    r = b - O.apply_dirac(U, KAPPA, T, L, -1, x)
    for j in range(ncol - 1):
        assert np.linalg.norm(r[j]) <= 1.1 * TOL * np.linalg.norm(b[j])
    assert np.abs(x[-1]).max() == 0
    assert 0 < st["iters"] < 200
