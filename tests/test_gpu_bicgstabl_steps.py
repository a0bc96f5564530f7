"""BiCGstab(l) where its deferred updates can go wrong: a breakdown inside a cycle, whose iterate holds the complete
steps; every l; sizes at the edges of the blocks of the Gram and update kernels; the sliced operator and CSR.

* Breakdowns: integer systems whose scalars are dyadic, so that every operation is exact and x is known in closed
  form (rational arithmetic of the same steps).  x is compared bit for bit.
* Every l: one cycle from zero on the coarse cylinder within 1e-7, the bound that one cycle of l = 8 is held to
  elsewhere; the basis is the worse conditioned the larger l is.
* Sizes: one cycle with l = 2 on diagonally dominant systems.  The basis [r_1 r_2] has a
  condition below 10 there, so that the normal equations lose at most its square, 100 times n-term rounding (1e-13
  for errors of random sign at the largest n), and a relative perturbation of 1e-16 of b moves the oracle's iterate
  by 5e-14: together 1e-11; 1e-10 leaves one digit.
"""

import numpy as np
import pytest
import torch

import oracle as O
import workloads as W
from oracle.bicgstabl import bicgstab_l
from workloads.csr import CSR

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hz():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    import paper_2112_06465_amd as hz

    return hz


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def solve(hz, A, b, **kw):
    x, info = hz.zbicgstabl_solve(dev(A.row_ptr), dev(A.col_idx), dev(A.vals), dev(b), **kw)
    return x.cpu().numpy(), info


def dense(rows):
    n = len(rows)
    return CSR(np.arange(0, n * n + 1, n, dtype=np.int32), np.tile(np.arange(n, dtype=np.int32), n),
               np.array(rows, dtype=complex).ravel())


# rows, b, x after the complete steps of the cycle in which <r~, A u_j> or rho vanishes
BREAKDOWNS = [
    ([[-3, 0], [3, 0]], [1, 1], [0, 0]),  # step 0, <r~, A u>
    ([[2, -1], [0, 0]], [-2, -2], [-4, -4]),  # step 1, <r~, A u>
    ([[-1, 2], [3, -2]], [2, -2], [-0.5, 0.5]),  # step 1, rho
    ([[2, -3, -2, -3], [-2, -2, -2, -3], [-2, 1, -1, 1], [3, -2, 1, -2]], [0, 0, 2, 0], [-1, -1, -0.5, 0.5]),  # 2, <r~, A u>
    ([[3, 2, -1], [0, -1, 0], [1, -1, 1]], [2, -1, -2], [2, 1, 1.5]),  # step 2, rho
    ([[3, 1, 2, -3], [2, -1, 3, 1], [1, 2, -1, 2], [0, -1, 1, 1]], [2, -2, 0, 2], [18.75, -66.75, 5.25, -18]),  # 3, <r~, A u>
    ([[-1, 3, 2, 2], [-1, 0, 2, -3], [1, -1, 0, 0], [-1, -1, -3, -1]], [0, -2, -1, 1], [10.5, 11.5, -5.5, -6.5]),  # 4, rho
]


@pytest.mark.parametrize("rows,b,x", BREAKDOWNS)
def test_breakdown_keeps_the_complete_steps(hz, rows, b, x):
    A = dense(rows)
    got, info = solve(hz, A, np.array(b, complex), ell=8, rtol=0.0, maxcycles=3, flags=hz.X0_ZERO | hz.NO_REORDER)
    xo, io = bicgstab_l(A, np.array(b, complex), ell=8, tol=0.0, maxcycles=3)
    assert info["status"] == hz.BREAKDOWN == io["status"] and info["iterations"] == 0 == io["iterations"]
    assert np.array_equal(got, np.array(x, complex))
    assert np.array_equal(xo, np.array(x, complex))


@pytest.mark.parametrize("jacobi", [False, True])
@pytest.mark.parametrize("ell", [1, 2, 3, 4, 5, 6, 7, 8])
def test_one_cycle_of_every_l(hz, ell, jacobi):
    A, b, _ = W.config_cylinder(h=0.1)
    flags = (hz.PRECOND_JACOBI if jacobi else hz.PRECOND_NONE) | hz.X0_ZERO | hz.NO_REORDER
    x, info = solve(hz, A, b, ell=ell, rtol=1e-30, maxcycles=1, flags=flags)
    xo, io = bicgstab_l(A, b, ell=ell, tol=1e-30, maxcycles=1, jacobi=jacobi)
    assert info["iterations"] == 1 == io["iterations"] and info["status"] == hz.NOT_CONVERGED
    err = np.linalg.norm(x - xo) / np.linalg.norm(xo)
    print(f"l={ell} jacobi={jacobi}: {err:.2e}")
    assert err <= 1e-7


def dominant(n, far=0):
    rng = np.random.default_rng(n + far)
    r = np.repeat(np.arange(n, dtype=np.int64), 6)
    c = (np.arange(n, dtype=np.int64)[:, None] + np.array([-9, -5, -1, 2, 5, 7])[None, :]).ravel()
    keep = (c >= 0) & (c < n)
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
    return CSR(rp, c[o].astype(np.int32), v[o]), rng.standard_normal(n) + 1j * rng.standard_normal(n)


@pytest.mark.parametrize("n,far", [(5, 0), (63, 0), (255, 0), (257, 0), (511, 0), (513, 0), (131072, 0), (131073, 0),
                                   (262144, 0), (262145, 0), (40000, 32761)])
def test_sizes_at_the_edges_of_the_blocks(hz, n, far):
    A, b = dominant(n, far)
    flags = hz.PRECOND_JACOBI | hz.X0_ZERO | hz.NO_REORDER
    x, info = solve(hz, A, b, ell=2, rtol=0.0, maxcycles=1, flags=flags)
    xo, io = bicgstab_l(A, b, ell=2, tol=0.0, maxcycles=1, jacobi=True)
    assert info["iterations"] == 1 == io["iterations"]
    err = np.linalg.norm(x - xo) / np.linalg.norm(xo)
    print(f"n={n} far={far}: {err:.2e}")
    assert err <= 1e-10
    assert abs(info["relres_recursive"] - io["relres_recursive"]) <= 1e-8 * io["relres_recursive"]
