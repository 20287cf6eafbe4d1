"""Time hops that a Dirichlet wall or a slab's end drops: their links are not part of the operator,
so NaN there must not reach any result, in the untuned launch forms and in the LDS-tile forms.

Stencil: the same values as with ordinary links there (bitwise).  Solves: tolerance 1e-10 on both
sides, so their solutions agree to 1e-8 (the links then fail the two-row check, which changes rounding).
"""
import pytest
import torch

from helpers import gaussian_field, lib, random_links, relerr, step

pytestmark = pytest.mark.gpu

T, L, NCOL = 6, 4, 3


def _setup(dd, dom):
    """packed links, the same with NaN on dropped time links, boundary condition"""
    U = dd.pack_links(random_links(T, L, 0.3, 9300))
    bad = U.clone()
    last = T - 1 if dom is None else (dom[0] + dom[1] - 1) % T
    bad[0].view(9, T, L ** 3)[:, last] = complex("nan")
    if dom is not None:
        bad[0].view(9, T, L ** 3)[:, (dom[0] - 1) % T] = complex("nan")
    return U, bad, (0 if dom is None else -1)


def _force(tmp_path, monkeypatch, dom, tile):
    monkeypatch.delenv("DD_TUNE_CACHE", raising=False)
    if tile:
        nt, whole = (T, 1) if dom is None else (dom[1], 0)
        key = f"{NCOL}:{L}:{T}:{nt}:{whole} 256 1 1 2 8\n"
        path = tmp_path / "s.txt"
        path.write_text("".join(f"{pre}{k}:{key}" for pre in ("", "eo:") for k in (0, 1)))
        monkeypatch.setenv("DD_TUNE_CACHE", str(path))


@pytest.mark.parametrize("tile", [False, True])
@pytest.mark.parametrize("dom", [None, (4, 4), (1, 3)])
def test_dropped_links_are_not_read(dom, tile, tmp_path, monkeypatch):
    dd = lib()
    step(f"dropped hops dom={dom} tile={tile}")
    U, bad, bc = _setup(dd, dom)
    n = (T if dom is None else dom[1]) * L ** 3
    psi = dd.pack_field(gaussian_field(n, NCOL, 9301))
    _force(tmp_path, monkeypatch, dom, tile)
    for dtype in (torch.complex128, torch.complex64):
        ctx = dd.Context(T, L, bc)
        want = dd.apply_dirac(ctx, U.to(dtype), 0.12, psi.to(dtype), dom)
        got = dd.apply_dirac(ctx, bad.to(dtype), 0.12, psi.to(dtype), dom)
        assert torch.equal(want, got)
    for prec in (dd.DD_FP64, dd.DD_MIXED):
        ctx = dd.Context(T, L, bc)
        p = dd.solver_params(tol=1e-10, prec=prec)
        want, _ = dd.block_solve(ctx, U, 0.12, psi, dom, p)
        got, _ = dd.block_solve(ctx, bad, 0.12, psi, dom, p)
        assert relerr(dd.unpack_field(got), dd.unpack_field(want)) < 1e-8
