"""GPU parity of the stencil and of the even-odd solves on lattices whose x rows are as long as, or longer than,
the LDS-tile forms can stage (64 sites in the stencil, 128 in the half hop, dd_tile_shape.h): at the limit
the form runs, above it every launch is a time sweep, whether the shape is timed, chosen untimed or named in
the stored shapes.

The oracle solves a lattice of L / n sites a side; links and sources repeated n times in x, y and z then
give the same answer repeated.  Bars: D element-wise within 1e-13 (FP64) / 2e-6 (FP32) of the largest
element; solves at kappa = 0.12 (condition number below 1e2) to 1e-12 (FP64) within 1e-10, to 1e-10 (mixed) within
1e-7 of the oracle's.
"""
import numpy as np
import pytest
import torch

import oracle as O
from helpers import gaussian_field, lib, random_links, step

pytestmark = pytest.mark.gpu


def _repeat(a, nt, l, n):
    """[..., nt l^3] on a lattice of l^3 repeated to (n l)^3."""
    lead = a.shape[:-1]
    return a.reshape(*lead, nt, l, l, l).repeat(*[1] * len(lead), 1, n, n, n).reshape(*lead, -1).contiguous()


def _maxrel(a, b):
    return ((a - b).abs().max() / b.abs().max()).item()


def _cache(tmp_path, monkeypatch, lines):
    path = tmp_path / "s.txt"
    path.write_text("".join(lines))
    monkeypatch.setenv("DD_TUNE_CACHE", str(path))


@pytest.mark.parametrize("L,n,stored", [(64, 4, True), (66, 2, False), (66, 2, True), (130, 5, False), (130, 5, True)])
@pytest.mark.parametrize("name,dtype,tol", [("double", torch.complex128, 1e-13), ("float", torch.complex64, 2e-6)])
def test_stencil_vs_oracle(L, n, stored, name, dtype, tol, tmp_path, monkeypatch):
    dd = lib()
    T, bc, dom, ncol, kappa, l = 3, -1, (2, 2), 2, 0.1287, L // n
    step(f"stencil of long rows L={L} {name} stored={stored}")
    kind = 0 if name == "double" else 1
    _cache(tmp_path, monkeypatch, [f"{kind}:{ncol}:{L}:{T}:{dom[1]}:0 256 1 1 {ncol} 8\n"] if stored else [])
    U = random_links(T, l, 0.4, 8100 + L)
    psi = gaussian_field(dom[1] * l ** 3, ncol, 8101)
    ref = O.apply_dirac(U, kappa, T, l, bc, psi, dom)
    ctx = dd.Context(T, L, bc)
    dd.set_kernel_timing(ctx, True)
    out = dd.apply_dirac(ctx, _repeat(dd.pack_links(U, dtype), T, l, n), kappa,
                         _repeat(dd.pack_field(psi, dtype), dom[1], l, n), dom)
    torch.cuda.synchronize()
    names = list(dd.kernel_timing(ctx))
    assert len(names) == 1 and names[0].startswith("k_dslash_lds<" if L <= 64 else "k_dslash<"), names
    assert _maxrel(out, _repeat(dd.pack_field(ref, dtype), dom[1], l, n)) < tol


@pytest.mark.parametrize("L,n,stored", [(128, 8, True), (130, 5, False), (130, 5, True)])
def test_even_odd_solves_vs_oracle(L, n, stored, tmp_path, monkeypatch):
    dd = lib()
    T, bc, ncol, kappa, l = 2, -1, 4, 0.12, L // n
    U = random_links(T, l, 0.3, 8200 + L)
    b = gaussian_field(T * l ** 3, ncol, 8201)
    ref, _, _, ost = O.solve(U, kappa, T, l, bc, b, tol=1e-13, method=1)
    assert ost == 0
    _cache(tmp_path, monkeypatch, [f"eo:{k}:{ncol}:{L}:{T}:{T}:1 256 1 1 {ncol} 8\n" for k in (0, 1)] if stored else [])
    ctx = dd.Context(T, L, bc)
    dd.set_kernel_timing(ctx, True)
    Ud, bd, xd = (_repeat(f, T, l, n) for f in (dd.pack_links(U), dd.pack_field(b), dd.pack_field(ref)))
    for prec, tol, bar in ((dd.DD_FP64, 1e-12, 1e-10), (dd.DD_MIXED, 1e-10, 1e-7)):
        step(f"even-odd solve of long rows L={L} prec={prec} stored={stored}")
        x, st = dd.block_solve(ctx, Ud, kappa, bd, None, dd.solver_params(tol=tol, prec=prec))
        assert max(st["true_rel_resid"][:ncol]) <= tol
        assert (torch.linalg.norm(x - xd) / torch.linalg.norm(xd)).item() < bar
    names = list(dd.kernel_timing(ctx))
    form = "k_eo_lds<" if L <= 128 else "k_eo_hop"
    for real in ("double", "float"):
        assert any(k.startswith(form) and f"<{real}" in k for k in names), names
    if L > 128:
        assert not any("_lds<" in k for k in names), names


@pytest.mark.parametrize("stored", [False, True])
def test_batch_with_one_long_domain_vs_oracle(stored, tmp_path, monkeypatch):
    """One domain whose rows are too long keeps the whole batched launch in the sweep."""
    dd = lib()
    batch = [(2, 130, 5, 0, 2), (4, 6, 1, 0, 4)]  # T, L, repeats, bc, columns
    items, refs = [], []
    for i, (T, L, n, bc, ncol) in enumerate(batch):
        l = L // n
        U = random_links(T, l, 0.3, 8300 + i)
        b = gaussian_field(T * l ** 3, ncol, 8310 + i)
        ref, _, _, ost = O.solve(U, 0.12, T, l, bc, b, tol=1e-13, method=1)
        assert ost == 0
        items.append(dict(T=T, L=L, time_bc=bc, U=_repeat(dd.pack_links(U), T, l, n), kappa=0.12,
                          b=_repeat(dd.pack_field(b), T, l, n),
                          x=torch.empty((ncol, 12, T * L ** 3), dtype=torch.complex128, device="cuda")))
        refs.append(_repeat(dd.pack_field(ref), T, l, n))
    sig = "".join(f":{T}x{L}x{ncol}b{bc}" for (T, L, _, bc, ncol) in batch)
    _cache(tmp_path, monkeypatch, [f"beo:{k}{sig} 256 1 1 2 8\n" for k in (0, 1)] if stored else [])
    ctx = dd.Context(8, 4, 0)
    dd.set_kernel_timing(ctx, True)
    for prec, tol, bar in ((dd.DD_FP64, 1e-12, 1e-10), (dd.DD_MIXED, 1e-10, 1e-7)):
        step(f"batch with one long domain prec={prec} stored={stored}")
        stats = dd.block_solve_batched(ctx, items, dd.solver_params(tol=tol, prec=prec))
        for it, ref, st in zip(items, refs, stats):
            assert max(st["true_rel_resid"][:ref.shape[0]]) <= tol
            assert (torch.linalg.norm(it["x"] - ref) / torch.linalg.norm(ref)).item() < bar
    names = list(dd.kernel_timing(ctx))
    assert any(k.startswith("k_beo_hop<double") for k in names) and not any("_lds<" in k for k in names), names
