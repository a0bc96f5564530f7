"""The BiCGStab iteration at the edges of its launch map: fewer than 8 blocks (one group of rows), groups of 16-row
multiples whose last ones are short or empty, rows that fill a block's steps exactly or by one more, and the sizes on
both sides of the line between the fused and the split iteration.

The systems are diagonally dominant, so that under Jacobi their iterates barely amplify rounding: a relative
perturbation of 1e-16 of b moves the oracle's iterate by 3e-16 after 5 iterations at every size here, while the GPU
and the oracle add the dot products of n terms in different orders (n u < 2e-11 relative at worst, about
sqrt(n) u = 1e-13 for rounding of random sign at the largest n).  1e-12 is the bound that the sub-block products of
the same family are held to.  Without Jacobi the diagonal's random phases leave the same perturbation 3e-14 after
one iteration and 1e-10 to 1 after five, so one iteration is compared.
"""

import numpy as np
import pytest
import torch

import oracle as O
from workloads.csr import CSR

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hz():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    import paper_2112_06465_amd as hz

    return hz


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def dominant(n, seed, most=13):
    """0 .. most-1 off-diagonal entries per row within 200 columns, and a diagonal of modulus 2 + their absolute sum."""
    rng = np.random.default_rng(seed)
    rows = np.repeat(np.arange(n, dtype=np.int64), rng.integers(0, most, n))
    cols = np.clip(rows + rng.integers(1, 201, rows.size) * rng.choice([-1, 1], rows.size), 0, n - 1)
    keep = cols != rows
    key = np.unique(rows[keep] * n + cols[keep])
    rows, cols = key // n, key % n
    vals = rng.standard_normal(rows.size) + 1j * rng.standard_normal(rows.size)
    absum = np.bincount(rows, weights=np.abs(vals), minlength=n)
    r, c = np.concatenate([rows, np.arange(n)]), np.concatenate([cols, np.arange(n)])
    v = np.concatenate([vals, (2.0 + absum) * np.exp(1j * rng.uniform(0, 2 * np.pi, n))])
    o = np.lexsort((c, r))
    rp = np.zeros(n + 1, np.int32)
    np.cumsum(np.bincount(r, minlength=n), out=rp[1:])
    return CSR(rp, c[o].astype(np.int32), v[o])


@pytest.mark.parametrize("fused", ["0", "1", None])
@pytest.mark.parametrize("n", [1, 3, 129, 1023, 1041, 2049, 16 * 1024 + 1, 57344, 57345, 140001])
def test_iterates_follow_the_oracle(hz, monkeypatch, n, fused):
    if fused is not None:
        monkeypatch.setenv("HZ_FUSED", fused)
    A = dominant(n, seed=n)
    rng = np.random.default_rng(5)
    b = rng.standard_normal(n) + 1j * rng.standard_normal(n)
    for jacobi in (False, True):
        flags = (hz.PRECOND_JACOBI if jacobi else hz.PRECOND_NONE) | hz.X0_ZERO | hz.NO_REORDER
        for iters in (1, 5) if jacobi else (1,):
            x, info = hz.zbicgstab_solve(dev(A.row_ptr), dev(A.col_idx), dev(A.vals), dev(b), rtol=1e-9 if n < 8 else 0.0,
                                         maxiter=iters, flags=flags)
            xo, io = O.zbicgstab(A, b, tol=1e-9 if n < 8 else 0.0, maxiter=iters, jacobi=jacobi)
            assert info["iterations"] == io["iterations"] and info["status"] == io["status"]
            err = np.linalg.norm(x.cpu().numpy() - xo) / np.linalg.norm(xo)
            print(f"n={n} jacobi={jacobi} after {iters}: {err:.2e}")
            assert err <= 1e-12
            if n >= 8:
                assert abs(info["relres_recursive"] - io["relres_recursive"]) <= 1e-9 * io["relres_recursive"]
