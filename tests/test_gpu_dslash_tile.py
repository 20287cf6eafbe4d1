"""GPU parity of the stencil's LDS-tile form (dd_dslash_tile.h): bricks that do not divide the
field, several slices per brick, whole planes inside one, odd L, column groups that do not divide the
columns, slabs across the time edge, dropped time hops, and every epilogue with columns that stop at
different iterations.

The form is forced through the launch-shape cache (tile flag bit 3, kc columns per workgroup).  Bars:
D element-wise within 1e-13 (FP64) / 2e-6 (FP32) of the largest element, as for the sweep; the solves
of the full operator to 1e-12 within 1e-10 of the oracle's (condition number below 1e2 at kappa = 0.12).
"""
import numpy as np
import pytest
import torch

import oracle as O
from helpers import gaussian_field, lib, random_links, relerr, step

pytestmark = pytest.mark.gpu

CASES = [  # T, L, bc, dom, ncol, columns per workgroup
    (7, 3, -1, None, 5, 2),       # several slices of whole planes per brick, the last brick short
    (6, 4, 0, None, 3, 3),        # Dirichlet time walls: both time hops dropped at the ends
    (9, 5, 1, (6, 5), 12, 5),     # odd L, across the time edge
    (5, 15, -1, (1, 2), 2, 1),
    (4, 16, -1, None, 4, 4),
    (4, 22, -1, (3, 2), 1, 1),    # bricks that do not divide L
]


def _cache(tmp_path, monkeypatch, T, L, dom, ncol, cpw, remap):
    nt, whole = (T, 1) if dom is None else (dom[1], 0)
    path = tmp_path / "s.txt"
    path.write_text("".join(f"{k}:{ncol}:{L}:{T}:{nt}:{whole} 256 1 {remap} {cpw} 8\n" for k in (0, 1)))
    monkeypatch.setenv("DD_TUNE_CACHE", str(path))


@pytest.mark.parametrize("T,L,bc,dom,ncol,cpw", CASES)
def test_tile_stencil_vs_oracle(T, L, bc, dom, ncol, cpw, tmp_path, monkeypatch):
    dd = lib()
    U = random_links(T, L, 0.4, 6100 + L)
    psi = gaussian_field((T if dom is None else dom[1]) * L ** 3, ncol, 6101)
    ref = O.apply_dirac(U, 0.1287, T, L, bc, psi, dom)
    for dtype, tol, name in ((torch.complex128, 1e-13, "double"), (torch.complex64, 2e-6, "float")):
        step(f"tile stencil {name} T={T} L={L} bc={bc} dom={dom} ncol={ncol} cpw={cpw}")
        _cache(tmp_path, monkeypatch, T, L, dom, ncol, cpw, remap=L % 2)
        ctx = dd.Context(T, L, bc)
        dd.set_kernel_timing(ctx, True)
        out = dd.apply_dirac(ctx, dd.pack_links(U, dtype), 0.1287, dd.pack_field(psi, dtype), dom)
        torch.cuda.synchronize()
        assert list(dd.kernel_timing(ctx)) == [f"k_dslash_lds<{name}, 0>"]
        assert np.abs(dd.unpack_field(out) - ref).max() / np.abs(ref).max() < tol


@pytest.mark.parametrize("solver", [0, 1])
def test_tile_stencil_solves_vs_oracle(solver, tmp_path, monkeypatch):
    """Unpreconditioned solves: D and D^+ with the norm, <r^, v> and <t, s> epilogues and the residual."""
    dd = lib()
    T, L, bc, dom, ncol = 6, 5, -1, (4, 4), 5
    U = random_links(T, L, 0.3, 6200)
    b = gaussian_field(dom[1] * L ** 3, ncol, 6201)
    b[-1] = 0
    b[-1, 7, 3] = 1.0  # a point source stops at another iteration than the volume sources
    ref, _, _, ost = O.solve(U, 0.12, T, L, bc, b, dom=dom, tol=1e-13, method=1)
    assert ost == 0
    for prec, tol, bar in ((dd.DD_FP64, 1e-12, 1e-10), (dd.DD_MIXED, 1e-10, 1e-7)):
        step(f"tile stencil solve solver={solver} prec={prec}")
        _cache(tmp_path, monkeypatch, T, L, dom, ncol, 3, remap=1)
        ctx = dd.Context(T, L, bc)
        dd.set_kernel_timing(ctx, True)
        p = dd.solver_params(tol=tol, prec=prec, solver=solver, precond=dd.DD_PRECOND_NONE)
        x, st = dd.block_solve(ctx, dd.pack_links(U), 0.12, dd.pack_field(b), dom, p)
        assert all(n.startswith("k_dslash_lds<") for n in dd.kernel_timing(ctx))
        assert max(st["true_rel_resid"][:ncol]) <= tol
        assert relerr(dd.unpack_field(x), ref) < bar
