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


def regular(n, k, seed, far=0):
    """About k off-diagonal entries in every row, at k common offsets within 150 rows (2 % of them missing at random),
    dominated by the diagonal; far > 0 adds one entry that many rows from the diagonal."""
    rng = np.random.default_rng(seed)
    offsets = rng.choice(np.concatenate([np.arange(-150, 0), np.arange(1, 151)]), k, replace=False) if k else np.zeros(0, int)
    r = np.repeat(np.arange(n, dtype=np.int64), k)
    c = (np.arange(n, dtype=np.int64)[:, None] + offsets[None, :]).ravel()
    keep = (c >= 0) & (c < n) & (rng.random(r.size) > 0.02)
    r, c = r[keep], c[keep]
    if far:
        r, c = np.append(r, 7), np.append(c, 7 + far)
    vals = rng.standard_normal(r.size) + 1j * rng.standard_normal(r.size)
    absum = np.bincount(r, weights=np.abs(vals), minlength=n)
    r, c = np.concatenate([r, np.arange(n)]), np.concatenate([c, np.arange(n)])
    v = np.concatenate([vals, (2.0 + absum) * np.exp(1j * rng.uniform(0, 2 * np.pi, n))])
    o = np.lexsort((c, r))
    rp = np.zeros(n + 1, np.int32)
    np.cumsum(np.bincount(r, minlength=n), out=rp[1:])
    return CSR(rp, c[o].astype(np.int32), v[o])


# Off-diagonal entries a row on both sides of the batches of 4 to 7 slots, and rows past and short of a slice's end;
# sizes on both sides of the fused form's line for the sliced operator; an entry at the 16-bit columns' limit (from
# row 7, in the slice of row 0: 32,767 rows away at most) and one past it, which leaves the matrix in CSR.
SLICED = [(12544, k, 0) for k in (0, 1, 3, 4, 7, 8, 13, 14)] + [
    (12545, 6, 0), (12607, 13, 0), (40000, 13, 32760), (40000, 13, 32761), (163840, 6, 0), (163841, 6, 0)]


@pytest.mark.parametrize("n,k,far", SLICED)
def test_sliced_operator_follows_the_oracle(hz, n, k, far):
    """The iterates of a Jacobi solve on the sliced operator (or, where it cannot hold the matrix, in CSR) against the
    oracle's, with the bound above; the asynchronous solve, which leaves the choice to the device, bit for bit the
    same; and one complex64 correction, whose operator is sliced at any size."""
    A = regular(n, k, seed=n + k, far=far)
    rng = np.random.default_rng(8)
    b = rng.standard_normal(n) + 1j * rng.standard_normal(n)
    rp, ci, v, bd = dev(A.row_ptr), dev(A.col_idx), dev(A.vals), dev(b)
    iters = 1 if k == 0 else 5  # a diagonal matrix is solved by the first step
    flags = hz.PRECOND_JACOBI | hz.X0_ZERO | hz.NO_REORDER
    tol = 1e-9 if k == 0 else 0.0
    x, info = hz.zbicgstab_solve(rp, ci, v, bd, rtol=tol, maxiter=iters, flags=flags)
    xo, io = O.zbicgstab(A, b, tol=tol, maxiter=iters, jacobi=True)
    assert info["iterations"] == io["iterations"] and info["status"] == io["status"]
    err = np.linalg.norm(x.cpu().numpy() - xo) / np.linalg.norm(xo)
    print(f"n={n} k={k} far={far}: {err:.2e}")
    assert err <= 1e-12
    xa, ia = hz.zbicgstab_solve_async(rp, ci, v, bd, rtol=tol, maxiter=iters, flags=hz.PRECOND_JACOBI | hz.X0_ZERO)
    assert torch.equal(torch.view_as_real(x), torch.view_as_real(xa))
    assert hz.read_info(ia)["iterations"] == info["iterations"]
    for more in (0, hz.RELIABLE):
        xm, im = hz.zbicgstab_solve_mixed(rp, ci, v, bd, rtol=1e-10, flags=flags | more)
        assert im["status"] == hz.OK
        assert np.linalg.norm(b - O.zspmv(A, xm.cpu().numpy())) <= 1e-10 * (1 + 1e-3) * np.linalg.norm(b)


def test_row_without_diagonal_is_invalid(hz):
    """A missing diagonal under Jacobi: refused by the synchronous solve, reported by the asynchronous one."""
    A = regular(12544, 6, seed=3)
    rows = A.row_of_entry()
    keep = ~((rows == 5000) & (A.col_idx == 5000))
    rp = np.zeros(A.n + 1, np.int32)
    np.cumsum(np.bincount(rows[keep], minlength=A.n), out=rp[1:])
    rp, ci, v = dev(rp), dev(A.col_idx[keep]), dev(A.vals[keep])
    b = dev(np.ones(A.n, complex))
    with pytest.raises(hz.HelmzError) as e:
        hz.zbicgstab_solve(rp, ci, v, b, flags=hz.PRECOND_JACOBI | hz.X0_ZERO)
    assert e.value.code == -1
    _, info = hz.zbicgstab_solve_async(rp, ci, v, b, maxiter=2, flags=hz.PRECOND_JACOBI | hz.X0_ZERO)
    assert hz.read_info(info)["status"] == -1
