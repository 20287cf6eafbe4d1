"""GPU parity of the baryon-block product at its tile widths (32, 64 and 96 columns, exact and ragged),
split counts of one and many, and a last chunk shorter than the others.

Bar as for the other block tests: within 1e-12 of the largest entry.
"""
import os

import numpy as np
import pytest
import torch

import oracle as O
from helpers import gaussian_field, lib, step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nt,L,chunk", [
    (4, 1, 8, None),    # 16 columns: one block, many splits
    (8, 1, 3, None),    # 32 columns: one block, full
    (16, 2, 4, None),   # 64: two blocks, full
    (17, 1, 4, 24),     # 68 of 96, chunks of 24, 24 and 16 sites
    (24, 1, 4, None),   # 96: three blocks, full
    (25, 1, 3, 5),      # 100 of 128, a chunk of 15 rows: one step of k, one split
    (40, 1, 3, None),   # 160 of 192: two tiles of three blocks, 820 rows
])
def test_block_tiles_vs_oracle(n, nt, L, chunk, monkeypatch):
    dd = lib()
    step(f"baryon block tiles n={n} nt={nt} L={L} chunk={chunk}")
    monkeypatch.delenv("DD_BLOCK_CHUNK", raising=False)
    if chunk:
        monkeypatch.setenv("DD_BLOCK_CHUNK", str(chunk))
    s = gaussian_field(nt * L ** 3, n, 4700 + n)
    ref = O.baryon_blocks(L, s)
    B = dd.baryon_blocks(dd.Context(8, L, -1), dd.pack_field(s))
    torch.cuda.synchronize()
    got = B.detach().cpu().numpy().transpose(0, 3, 4, 1, 2)
    assert np.abs(got - ref).max() < 1e-12 * np.abs(ref).max()
