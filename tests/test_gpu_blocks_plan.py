"""GPU parity of the baryon-block product at sizes whose plan (zgemm_plan) takes each tile width, with one and several
splits and a last chunk shorter than the others (tests/test_gemm_plan.py holds the plan itself).

The oracle forms the blocks of seven of the vectors, the first and the last among them, whose entries the full
blocks hold too.  Bar as for the other block tests: within 1e-12 of the largest entry.
"""
import numpy as np
import pytest
import torch

import oracle as O
from helpers import gaussian_field, lib, step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,L,chunk", [
    (24, 4, None),   # 32 columns wide, many splits
    (64, 4, None),   # 64 wide, 3 splits
    (57, 5, 70),     # chunks of 70 and 55 sites
    (65, 8, None),   # 96 wide (260 columns of 288), 5 splits
    (113, 3, None),  # 96 wide, one split
])
def test_block_plans_vs_oracle(n, L, chunk, monkeypatch):
    dd = lib()
    step(f"baryon block plan n={n} L={L} chunk={chunk}")
    monkeypatch.delenv("DD_BLOCK_CHUNK", raising=False)
    if chunk:
        monkeypatch.setenv("DD_BLOCK_CHUNK", str(chunk))
    s = gaussian_field(L ** 3, n, 4800 + n)
    sub = sorted({0, 1, n // 3, n // 2, n - 9, n - 2, n - 1})
    ref = O.baryon_blocks(L, s[sub])
    B = dd.baryon_blocks(dd.Context(8, L, -1), dd.pack_field(s))
    torch.cuda.synchronize()
    got = B.detach().cpu().numpy().transpose(0, 3, 4, 1, 2)[0]
    got = got[np.ix_(sub, sub, sub)][None]
    assert np.isfinite(got).all() and got.shape == ref.shape
    assert np.abs(got - ref).max() < 1e-12 * np.abs(ref).max()
