"""GPU parity of the LDS-tile half hop (dd_eo_tile.h) where its bricks do not divide the field:
several slices per brick (small L), bricks cut short in y, z and time, whole rows and
planes inside one brick, and columns in groups that do not divide their number.

The form is forced through the launch-shape cache (tile flag bit 3, kc columns per
workgroup) in FP64 and FP32; links of the FP32 recursion are read as two rows (SU(3)) or nine
entries (scaled links).  Bars: the solves run to 1e-12 (FP64) or 1e-10 (mixed) on operators
with a condition number below 1e2 (kappa = 0.12), so an answer lies within 1e-10 of the oracle's in FP64
and 1e-7 in mixed precision; the reported residual is the full operator's.
"""
import pytest
import torch

import oracle as O
from helpers import gaussian_field, lib, random_links, relerr, step

pytestmark = pytest.mark.gpu

CASES = [  # T, L, bc, dom, ncol, columns per workgroup
    (9, 4, 0, None, 5, 2),        # 8 slices of 4 x 4 rows per brick, the last brick 1 slice
    (7, 6, -1, (5, 5), 3, 3),     # 2 slices of 6 x 6 rows, across the time edge
    (4, 10, 1, None, 2, 1),       # 5 x 10 rows: whole y or z extents
    (5, 14, -1, (1, 3), 4, 3),
    (4, 22, -1, (2, 2), 2, 2),    # bricks that do not divide L
]


def _run(dd, T, L, bc, dom, ncol, cpw, prec, solver, scale, path, monkeypatch):
    nt, whole = (T, 1) if dom is None else (dom[1], 0)
    path.write_text("".join(f"eo:{k}:{ncol}:{L}:{T}:{nt}:{whole} 256 1 1 {cpw} 8\n" for k in (0, 1)))
    monkeypatch.setenv("DD_TUNE_CACHE", str(path))
    U = random_links(T, L, 0.3, 5100 + L) * scale
    b = gaussian_field(nt * L ** 3, ncol, 5101)
    b[-1] = 0
    b[-1, 7, 3] = 1.0  # a point source stops at another iteration than the volume sources
    ctx = dd.Context(T, L, bc)
    dd.set_kernel_timing(ctx, True)
    p = dd.solver_params(tol=1e-12 if prec == dd.DD_FP64 else 1e-10, prec=prec, solver=solver)
    x, st = dd.block_solve(ctx, dd.pack_links(U), 0.12, dd.pack_field(b), dom, p)
    names = list(dd.kernel_timing(ctx))
    want = "k_eo_lds<double" if prec == dd.DD_FP64 else "k_eo_lds<float"
    assert any(n.startswith(want) for n in names), names
    assert max(st["true_rel_resid"][:ncol]) <= p.tol
    ref, _, _, ost = O.solve(U, 0.12, T, L, bc, b, dom=dom, tol=1e-13, method=1)
    assert ost == 0
    return relerr(dd.unpack_field(x), ref)


@pytest.mark.parametrize("T,L,bc,dom,ncol,cpw", CASES)
def test_tile_bricks_vs_oracle(T, L, bc, dom, ncol, cpw, tmp_path, monkeypatch):
    dd = lib()
    for prec, solver, scale in ((dd.DD_FP64, 1, 1.0), (dd.DD_FP64, 0, 1.0), (dd.DD_MIXED, 1, 1.0), (dd.DD_MIXED, 1, 0.97)):
        step(f"tile half hop T={T} L={L} bc={bc} dom={dom} ncol={ncol} prec={prec} solver={solver} scale={scale}")
        err = _run(dd, T, L, bc, dom, ncol, cpw, prec, solver, scale, tmp_path / "s.txt", monkeypatch)
        assert err < (1e-10 if prec == dd.DD_FP64 else 1e-7)


@pytest.mark.parametrize("solver", [0, 1])
def test_batched_tile_vs_oracle(solver, tmp_path, monkeypatch):
    """The batched launch of the same form: domains whose brick shapes and column counts differ."""
    dd = lib()
    step(f"batched tile half hop solver={solver}")
    batch = [(8, 4, 0, 0.12, 3), (4, 6, 0, 0.125, 12), (9, 4, 0, 0.12, 5), (4, 10, -1, 0.12, 1)]
    items, refs = [], []
    for i, (T, L, bc, kappa, ncol) in enumerate(batch):
        U = random_links(T, L, 0.3, 5200 + i)
        b = gaussian_field(T * L ** 3, ncol, 5300 + i)
        items.append(dict(T=T, L=L, time_bc=bc, U=dd.pack_links(U), kappa=kappa, b=dd.pack_field(b),
                          x=torch.empty((ncol, 12, T * L ** 3), dtype=torch.complex128, device="cuda")))
        refs.append((U, b))
    sig = "".join(f":{T}x{L}x{ncol}b{bc}" for (T, L, bc, _, ncol) in batch)
    path = tmp_path / "s.txt"
    path.write_text(f"beo:0{sig} 256 1 1 4 8\nbeo:1{sig} 256 1 0 5 8\n")
    monkeypatch.setenv("DD_TUNE_CACHE", str(path))
    ctx = dd.Context(8, 4, 0)
    dd.set_kernel_timing(ctx, True)
    for prec, tol, bar in ((dd.DD_FP64, 1e-12, 1e-10), (dd.DD_MIXED, 1e-10, 1e-7)):
        stats = dd.block_solve_batched(ctx, items, dd.solver_params(tol=tol, prec=prec, solver=solver))
        for it, (U, b), st, (T, L, bc, kappa, ncol) in zip(items, refs, stats, batch):
            assert max(st["true_rel_resid"][:ncol]) <= tol
            ref, _, _, ost = O.solve(U, kappa, T, L, bc, b, tol=1e-13, method=1)
            assert ost == 0
            assert relerr(dd.unpack_field(it["x"]), ref) < bar
    names = list(dd.kernel_timing(ctx))
    assert any(n.startswith("k_beo_lds<double") for n in names), names  # the eager launches (the FP32 ones replay a graph)
