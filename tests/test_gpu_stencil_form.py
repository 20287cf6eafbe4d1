"""Which form of the stencil a launch takes, the time sweep or the LDS tile, on both sides of every line of the
rule (dslash_tile_form, by sizes alone) for untimed (below 2^18 site-columns) and timed launches; the
untimed sweep's chunks of 1, 2 and 4 slices; and, of a timed launch, that its result is bitwise that of other
shapes of the same form, so that a timing decides nothing but speed.

The kernel names tell the form.  Bars: element-wise within 1e-13 (FP64) / 2e-6 (FP32) of the largest element of
the oracle's.
"""
import numpy as np
import pytest
import torch

import oracle as O
from helpers import gaussian_field, lib, random_links, step

pytestmark = pytest.mark.gpu

C128, C64 = torch.complex128, torch.complex64
SUMS = [  # T, L, ncol, D in solves by the LDS tile: FP64 fields of bricks four fifths full
    (16, 24, 2, False),                  # 0.75 full (dd_apply_dirac takes the tile there)
    (10, 15, 8, True),                   # 320 bricks, 0.82 full
    (8, 19, 5, False),                   # 0.77 full
]
UNTIMED = [  # T, L, dom, ncol, dtype, LDS tile
    (16, 16, None, 1, C128, True),       # 512 full bricks
    (15, 16, None, 1, C128, False),      # 480; one slice
    (15, 16, None, 3, C64, False),
    (8, 31, None, 1, C128, True),        # 2048 bricks, 0.91 full
    (12, 20, None, 1, C128, False),      # 840 bricks, 0.89 full; two slices
    (11, 20, (7, 9), 3, C128, False),    # four slices across the time edge, the last chunk of one
    (8, 30, None, 1, C64, True),
    (11, 15, (7, 9), 8, C64, False),     # odd L, ragged tiles
    (3, 4, None, 2, C64, False),
]
TIMED = [  # T, L, ncol, dtype, LDS tile
    (6, 16, 11, C128, True),             # 192 full bricks
    (5, 16, 13, C128, False),            # 160
    (16, 24, 2, C128, True),             # 0.75 full
    (16, 22, 2, C128, False),            # 0.69 full
    (16, 22, 6, C128, True),
    (4, 36, 6, C128, False),             # 0.56 full
    (16, 32, 2, C128, False),            # links past 256 MB, L divides 64
    (13, 32, 2, C128, True),             # 245 MB
    (10, 30, 1, C64, False),
    (10, 30, 2, C64, True),              # 0.94 full
    (11, 24, 4, C64, True),              # 1584 bricks, 0.75 full
    (11, 24, 3, C64, False),
    (10, 24, 4, C64, False),             # 1440 bricks
    (8, 18, 12, C64, True),              # 432 bricks, 0.84 full
    (8, 18, 11, C64, False),
]


def _apply(dd, T, L, dom, U, psi, kappa):
    ctx = dd.Context(T, L, -1)
    dd.set_kernel_timing(ctx, True)
    out = dd.apply_dirac(ctx, U, kappa, psi, dom)
    torch.cuda.synchronize()
    names = list(dd.kernel_timing(ctx))
    assert len(names) == 1
    return out, names[0]


def _maxrel(a, b):
    return np.abs(a - b).max() / np.abs(b).max()


@pytest.mark.parametrize("T,L,dom,ncol,dtype,tile", UNTIMED)
def test_untimed_form_vs_oracle(T, L, dom, ncol, dtype, tile, monkeypatch):
    dd = lib()
    step(f"untimed form T={T} L={L} dom={dom} ncol={ncol} {dtype}")
    monkeypatch.delenv("DD_TUNE_CACHE", raising=False)
    nsite = (T if dom is None else dom[1]) * L ** 3
    assert nsite * ncol < 2 ** 18
    U = random_links(T, L, 0.4, 7100 + L)
    psi = gaussian_field(nsite, ncol, 7101)
    out, name = _apply(dd, T, L, dom, dd.pack_links(U, dtype), dd.pack_field(psi, dtype), 0.1287)
    assert name.startswith("k_dslash_lds<" if tile else "k_dslash<"), name
    ref = O.apply_dirac(U, 0.1287, T, L, -1, psi, dom)
    assert _maxrel(dd.unpack_field(out), ref) < (1e-13 if dtype == C128 else 2e-6)


@pytest.mark.parametrize("T,L,ncol,dtype,tile", TIMED)
def test_timed_form_and_bits(T, L, ncol, dtype, tile, monkeypatch, tmp_path):
    dd = lib()
    step(f"timed form T={T} L={L} ncol={ncol} {dtype}")
    monkeypatch.delenv("DD_TUNE_CACHE", raising=False)
    assert T * L ** 3 * ncol >= 2 ** 18
    U = random_links(T, L, 0.4, 7200 + L)
    psi = gaussian_field(T * L ** 3, ncol, 7201)
    Ud, pd = dd.pack_links(U, dtype), dd.pack_field(psi, dtype)
    out, name = _apply(dd, T, L, None, Ud, pd, 0.1287)
    assert name.startswith("k_dslash_lds<" if tile else "k_dslash<"), name
    ref = O.apply_dirac(U, 0.1287, T, L, -1, psi, None)
    assert _maxrel(dd.unpack_field(out), ref) < (1e-13 if dtype == C128 else 2e-6)
    kind = 0 if dtype == C128 else 1
    for k, shape in enumerate(("256 1 1 1 8", "256 1 0 5 8") if tile else ("128 1 0 1 0", "256 4 1 2 2")):
        path = tmp_path / f"s{k}.txt"
        path.write_text(f"{kind}:{ncol}:{L}:{T}:{T}:1 {shape}\n")
        monkeypatch.setenv("DD_TUNE_CACHE", str(path))
        other, oname = _apply(dd, T, L, None, Ud, pd, 0.1287)
        assert oname.split("<")[0] == name.split("<")[0]
        assert torch.equal(other, out), (name, shape)


@pytest.mark.parametrize("T,L,ncol,tile", SUMS)
def test_form_inside_solves(T, L, ncol, tile, monkeypatch):
    """Unpreconditioned FP64 solves: every launch (with sums) takes one form; dd_apply_dirac, without, its own."""
    dd = lib()
    step(f"form inside solves T={T} L={L} ncol={ncol}")
    monkeypatch.delenv("DD_TUNE_CACHE", raising=False)
    assert T * L ** 3 * ncol >= 2 ** 18
    U = random_links(T, L, 0.3, 7300 + L)
    b = gaussian_field(T * L ** 3, ncol, 7301)
    ctx = dd.Context(T, L, -1)
    dd.set_kernel_timing(ctx, True)
    Ud, bd = dd.pack_links(U), dd.pack_field(b)
    for solver in (0, 1):
        x, st = dd.block_solve(ctx, Ud, 0.11, bd, None, dd.solver_params(tol=1e-10, solver=solver, precond=1))
        assert max(st["true_rel_resid"][:ncol]) <= 1e-10
        r = bd - dd.apply_dirac(ctx, Ud, 0.11, x)
        assert (torch.linalg.norm(r) / torch.linalg.norm(bd)).item() <= 2e-10
    names = [n for n in dd.kernel_timing(ctx) if not n.endswith("double, 0>") and ", 0, 0, " not in n]
    assert names and all(n.startswith("k_dslash_lds<" if tile else "k_dslash<") for n in names), names
