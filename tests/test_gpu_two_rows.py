"""Which FP32 half hops read two rows of an SU(3) link and rebuild the third (a less exact link): in the
LDS-tile form only timed fields (2^18 site-columns and more) with an even number of columns, or of L = 16
and 32; batches whose column counts are all even.  Everything else reads the nine entries.  The
kernel names tell (the last but one parameter of k_eo_lds, the last of k_beo_lds); each solve meets 1e-10 on
the full FP64 residual.
"""
import pytest
import torch

from helpers import gaussian_field, lib, random_links, step

pytestmark = pytest.mark.gpu

CASES = [  # T, L, ncol, two rows
    (16, 4, 12, False),   # untimed, even column count
    (32, 16, 1, False),   # untimed, one column
    (4, 16, 3, False),
    (16, 16, 3, False),   # the largest untimed one of L = 16
    (16, 16, 4, True),    # 2^18 site-columns
    (16, 16, 5, True),
    (8, 20, 5, False),    # timed, odd column count, another L
    (8, 20, 6, True),
]


def _solve(dd, T, L, ncol, monkeypatch, tmp_path):
    # the form is named for both precisions, whatever the timing would pick
    path = tmp_path / "s.txt"
    path.write_text("".join(f"eo:{k}:{ncol}:{L}:{T}:{T}:1 256 1 1 {ncol} 8\n" for k in (0, 1)))
    monkeypatch.setenv("DD_TUNE_CACHE", str(path))
    ctx = dd.Context(T, L, -1)
    dd.set_kernel_timing(ctx, True)
    U = random_links(T, L, 0.3, 9000 + L)
    b = gaussian_field(T * L ** 3, ncol, 9001)
    _, st = dd.block_solve(ctx, dd.pack_links(U), 0.12, dd.pack_field(b), None,
                           dd.solver_params(tol=1e-10, prec=dd.DD_MIXED))
    assert max(st["true_rel_resid"][:ncol]) <= 1e-10
    return [n for n in dd.kernel_timing(ctx) if n.startswith("k_eo_lds<float")]


@pytest.mark.parametrize("T,L,ncol,two", CASES)
def test_two_row_links(T, L, ncol, two, monkeypatch, tmp_path):
    dd = lib()
    step(f"two-row links T={T} L={L} ncol={ncol}")
    names = _solve(dd, T, L, ncol, monkeypatch, tmp_path)
    assert names and all(n.split(", ")[3] == ("true" if two else "false") for n in names), names


@pytest.mark.parametrize("odd", [False, True])
def test_two_row_links_batched(odd, monkeypatch, tmp_path):
    dd = lib()
    step(f"two-row links of a batch, odd={odd}")
    batch = [(8, 4, 4), (4, 6, 3 if odd else 2)]
    items = []
    for i, (T, L, ncol) in enumerate(batch):
        items.append(dict(T=T, L=L, time_bc=0, U=dd.pack_links(random_links(T, L, 0.3, 9100 + i)), kappa=0.12,
                          b=dd.pack_field(gaussian_field(T * L ** 3, ncol, 9110 + i)),
                          x=torch.empty((ncol, 12, T * L ** 3), dtype=torch.complex128, device="cuda")))
    sig = "".join(f":{T}x{L}x{ncol}b0" for T, L, ncol in batch)
    path = tmp_path / "s.txt"
    path.write_text("".join(f"beo:{k}{sig} 256 1 1 2 8\n" for k in (0, 1)))
    monkeypatch.setenv("DD_TUNE_CACHE", str(path))
    ctx = dd.Context(8, 4, 0)
    dd.set_kernel_timing(ctx, True)
    stats = dd.block_solve_batched(ctx, items, dd.solver_params(tol=1e-10, prec=dd.DD_MIXED))
    for st, (_, _, ncol) in zip(stats, batch):
        assert max(st["true_rel_resid"][:ncol]) <= 1e-10
    names = [n for n in dd.kernel_timing(ctx) if n.startswith("k_beo_lds<float")]
    assert names and all(n.rstrip(">").split(", ")[3] == ("false" if odd else "true") for n in names), names
