"""GPU parity of the projection vectors at the edges of the Gram, factorisation and combine tiles:
one vector, 16 and 32 per block and one more, the largest matrix factorised in LDS and the next one,
with row counts that are no multiple of a wavefront's 16 rows.

Bars as for the projection: vectors orthonormal to 1e-12, the projector within 1e-10 of the oracle's.
"""
import numpy as np
import pytest
import torch

import oracle as O
from helpers import gaussian_field, lib, random_links, relerr, step

pytestmark = pytest.mark.gpu

CASES = [  # vectors, T, L, pi
    (1, 8, 3, (2, 3)),
    (16, 8, 3, (6, 4)),
    (17, 8, 3, (2, 3)),
    (32, 8, 4, (2, 3)),
    (33, 8, 3, (2, 3)),
    (64, 8, 3, (6, 4)),
    (65, 8, 3, (2, 3)),
]


@pytest.mark.parametrize("nvec,T,L,pi", CASES)
def test_projection_tiles_vs_oracle(nvec, T, L, pi):
    dd = lib()
    step(f"projection tiles nvec={nvec} L={L} pi={pi}")
    U = random_links(T, L, 0.3, 8300)
    v0 = gaussian_field(pi[1] * L ** 3, nvec, 8301 + nvec)
    t = (pi[0] + 1) % T
    ref = O.projection_basis(U, 0.12, T, L, -1, pi, t, 1, v0, 1, tol=1e-13)[0]
    p = dd.solver_params(tol=1e-13, max_iter=20000, prec=dd.DD_FP64)
    phi, _ = dd.projection_basis(dd.Context(T, L, -1), dd.pack_links(U), 0.12, pi, t, 1, dd.pack_field(v0), 1, p)
    got = phi.cpu().permute(0, 2, 1).contiguous().numpy().reshape(nvec, -1)
    want = ref.reshape(nvec, -1)
    assert np.abs(got.conj() @ got.T - np.eye(nvec)).max() < 1e-12
    assert relerr(got.T @ got.conj(), want.T @ want.conj()) < 1e-10
