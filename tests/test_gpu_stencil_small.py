"""GPU parity of the stencil's untuned shapes: chunks of 1, 2, 4 and 8 slices, at and just past the
wavefront counts where the rule changes, fields shorter than a chunk, and slabs across the time edge.

Bars: element-wise within 1e-13 (FP64) / 2e-6 (FP32) of the largest element.
"""
import numpy as np
import pytest
import torch

import oracle as O
from helpers import gaussian_field, lib, random_links, step

pytestmark = pytest.mark.gpu

CASES = [  # T, L, dom, ncol, dtype
    (16, 16, None, 1, torch.complex128),     # 1024 wavefronts: one slice
    (17, 16, None, 1, torch.complex128),     # past it: two slices, the last chunk short
    (9, 16, (5, 7), 5, torch.complex128),    # four slices across the time edge, last chunk of three
    (16, 16, None, 5, torch.complex128),     # eight slices
    (3, 16, None, 12, torch.complex128),     # fewer slices than the chunk
    (2, 4, None, 2, torch.complex128),
    (16, 16, None, 4, torch.complex64),      # 4096 wavefronts: one slice
    (11, 15, (7, 9), 10, torch.complex64),   # two slices, odd L, ragged tiles
]


@pytest.mark.parametrize("T,L,dom,ncol,dtype", CASES)
def test_untuned_stencil_vs_oracle(T, L, dom, ncol, dtype, monkeypatch):
    dd = lib()
    step(f"untuned stencil T={T} L={L} dom={dom} ncol={ncol} {dtype}")
    monkeypatch.delenv("DD_TUNE_CACHE", raising=False)
    U = random_links(T, L, 0.4, 7000 + T)
    psi = gaussian_field((T if dom is None else dom[1]) * L ** 3, ncol, 7001)
    ref = O.apply_dirac(U, 0.1287, T, L, -1, psi, dom)
    ctx = dd.Context(T, L, -1)
    out = dd.apply_dirac(ctx, dd.pack_links(U, dtype), 0.1287, dd.pack_field(psi, dtype), dom)
    tol = 1e-13 if dtype == torch.complex128 else 2e-6
    assert np.abs(dd.unpack_field(out) - ref).max() / np.abs(ref).max() < tol
