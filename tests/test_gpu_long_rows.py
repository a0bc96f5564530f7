"""Rows longer than the sliced operator takes, all their columns within its 16 bits: one of 2^25 entries beside the
diagonal, whose 64-fold no int holds, and whole slices of 65,536 and 65,537, which fill their slots.

The matrix is 4 I + N with N^2 = 0 (couplings of even rows to the next), so the solution is known row by row, and
TFQMR reaches it in two steps.  A long row is n copies of 1/n, so that only the order of its sum rounds: by lanes of
64, at most n / 64 u of the coupling's term (6e-11), a quarter of which reaches x.
"""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hz():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    import paper_2112_06465_amd as hz

    return hz


@pytest.mark.parametrize("long,rows", [(2**25, [100]), (2**16, range(0, 64)), (2**16 + 1, range(64, 128))])
def test_long_rows(hz, monkeypatch, long, rows):
    monkeypatch.setenv("HZ_SPMV_LANES", "64")
    n = 500
    lens = np.where(np.arange(n) % 2 == 0, 2, 1).astype(np.int64)
    lens[list(rows)] = 1 + long
    i = torch.arange(n, device="cuda:0")
    rp = torch.zeros(n + 1, dtype=torch.int32, device="cuda:0")
    rp[1:] = torch.from_numpy(lens.cumsum()).to("cuda:0")
    row = torch.repeat_interleave(i, torch.from_numpy(lens).to("cuda:0"))
    first = torch.zeros(row.numel(), dtype=torch.bool, device="cuda:0")
    first[rp[:-1].long()] = True
    to = torch.where(i % 2 == 0, i + 1, i)  # odd rows that are long repeat their diagonal with zeros
    ci = torch.where(first, row, to[row]).to(torch.int32)
    share = torch.from_numpy(np.where(np.arange(n) % 2 == 0, 1.0 / (lens - (lens > 1)), 0.0)).to("cuda:0")
    vals = torch.where(first, 4.0, share[row]).to(torch.complex128)
    last = rp[1:].long() - 1  # the diagonal that counts is the last one of the row
    odd = (i % 2 == 1)
    vals[rp[:-1].long()[odd]] = 0.0
    vals[last[odd]] = 4.0
    b = torch.randn(n, dtype=torch.complex128, generator=torch.Generator("cuda:0").manual_seed(1), device="cuda:0")
    want = b / 4.0
    want[0::2] = (b[0::2] - want[1::2]) / 4.0
    x, info = hz.ztfqmr_solve(rp, ci, vals, b, rtol=1e-9, flags=hz.PRECOND_JACOBI | hz.X0_ZERO | hz.NO_REORDER)
    err = ((x - want).norm() / want.norm()).item()
    print(f"{long}: {info['iterations']} iterations, error {err:.2e}")
    assert info["status"] == hz.OK and err <= 1e-9 * 1.1
