"""Which form of the even-odd half hop an untimed launch takes (eo_tile_form), on both sides of its lines, by
kernel name: the FP32 hops of mixed solves below 2^18 site-columns, and the FP64 hops that prepare the
source and reconstruct the odd sites (untimed at any size).  Each solve meets 1e-10 on the full
FP64 residual.
"""
import pytest

from helpers import gaussian_field, lib, random_links, step

pytestmark = pytest.mark.gpu

FP32 = [  # T, L, ncol, LDS tile
    (16, 4, 12, True),
    (32, 16, 1, True),    # 256 bricks: one round of workgroups
    (6, 32, 1, False),    # 384
    (4, 22, 1, True),     # 120 bricks, 0.69 full, a column each
    (4, 22, 2, True),
    (4, 22, 3, False),
    (8, 18, 5, True),     # 96 bricks, 0.95 full: two groups of columns
    (4, 34, 1, False),    # 432 bricks
]
FP64 = [
    (16, 20, 4, True),    # 256 bricks, 0.98 full
    (16, 20, 3, False),
    (4, 40, 4, False),    # 0.64 full
]


def _names(dd, T, L, ncol, monkeypatch):
    monkeypatch.delenv("DD_TUNE_CACHE", raising=False)
    ctx = dd.Context(T, L, -1)
    dd.set_kernel_timing(ctx, True)
    U = random_links(T, L, 0.3, 9300 + L)
    b = gaussian_field(T * L ** 3, ncol, 9301)
    _, st = dd.block_solve(ctx, dd.pack_links(U), 0.12, dd.pack_field(b), None,
                           dd.solver_params(tol=1e-10, prec=dd.DD_MIXED))
    assert max(st["true_rel_resid"][:ncol]) <= 1e-10
    return list(dd.kernel_timing(ctx))


@pytest.mark.parametrize("T,L,ncol,tile", FP32)
def test_fp32_form(T, L, ncol, tile, monkeypatch):
    dd = lib()
    step(f"untimed FP32 half hop T={T} L={L} ncol={ncol}")
    assert T * L ** 3 * ncol < 2 ** 18
    names = [n for n in _names(dd, T, L, ncol, monkeypatch) if "<float" in n]
    assert names and all(n.startswith("k_eo_lds<" if tile else "k_eo_hop<") for n in names), names


@pytest.mark.parametrize("T,L,ncol,tile", FP64)
def test_fp64_form(T, L, ncol, tile, monkeypatch):
    dd = lib()
    step(f"untimed FP64 half hop T={T} L={L} ncol={ncol}")
    names = _names(dd, T, L, ncol, monkeypatch)
    # source preparation and reconstruction: stored (epilogue 0), with a self field
    want = "k_eo_lds<double, 0, true, " if tile else "k_eo_hop<double, 0, 0, 256, true, "
    other = "k_eo_hop<double, 0, 0, 256, true, " if tile else "k_eo_lds<double, 0, true, "
    assert any(n.startswith(want) for n in names) and not any(n.startswith(other) for n in names), names
