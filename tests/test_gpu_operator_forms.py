"""Which operator a Jacobi solve ran on, and the sliced one's streaming loads.

* A stored zero at the end of a row changes no sum of a product in CSR, whose order is that of the row.  One far from
  the diagonal keeps the matrix out of slices, so: two such matrices give the same bits (both CSR), and the matrix
  without the zero other bits, since slices sum in another order.  The iterates agree to 1e-12, the bound that every
  form is held to against the oracle.
* Above 128 MiB of slots (7,456,540 entries) the products' loads are streamed: the same bounds against the oracles, by
  the derivations of the forms' own tests (sums of n terms in another order, sqrt(n) u = 1e-13 here).
"""

import numpy as np
import pytest
import torch

import oracle as O
from oracle.bicgstabl import bicgstab_l
from oracle.tfqmr import tfqmr
from test_gpu_initial_guess import sliced
from test_gpu_iteration import regular
from workloads.csr import CSR

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hz():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    import paper_2112_06465_amd as hz

    return hz


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def with_zeros(A, at):
    """A with a stored zero appended to each of the rows `at`, in the last column."""
    ends = A.row_ptr[np.asarray(at) + 1]
    rp = A.row_ptr + np.searchsorted(np.asarray(at), np.arange(A.n + 1), side="left").astype(np.int32)
    return CSR(rp, np.insert(A.col_idx, ends, A.n - 1).astype(np.int32), np.insert(A.vals, ends, 0.0))


def solve(hz, name, A, b):
    args = dev(A.row_ptr), dev(A.col_idx), dev(A.vals), dev(b)
    flags = hz.PRECOND_JACOBI | hz.X0_ZERO | hz.NO_REORDER
    if name == "bicgstab":
        return hz.zbicgstab_solve(*args, rtol=0.0, maxiter=5, flags=flags)[0].cpu().numpy()
    if name == "async":
        return hz.zbicgstab_solve_async(*args, rtol=0.0, maxiter=5, flags=flags & ~hz.NO_REORDER)[0].cpu().numpy()
    if name == "bicgstabl":
        return hz.zbicgstabl_solve(*args, ell=2, rtol=0.0, maxcycles=1, flags=flags)[0].cpu().numpy()
    return hz.ztfqmr_solve(*args, rtol=1e-30, maxiter=3, flags=flags)[0].cpu().numpy()


@pytest.mark.parametrize("name,bound", [("bicgstab", 1e-12), ("async", 1e-12), ("bicgstabl", 1e-10), ("tfqmr", 1e-12)])
def test_each_operator_has_its_own_bits(hz, name, bound):
    A = regular(40000, 13, seed=21)
    rng = np.random.default_rng(4)
    b = rng.standard_normal(A.n) + 1j * rng.standard_normal(A.n)
    one, two = with_zeros(A, [7]), with_zeros(A, [7, 100])
    assert sliced(A) and not sliced(one) and not sliced(two)
    xs, x1, x2 = (solve(hz, name, m, b) for m in (A, one, two))
    assert np.array_equal(x1.view(np.float64), x2.view(np.float64))
    assert not np.array_equal(xs.view(np.float64), x1.view(np.float64))
    assert np.linalg.norm(xs - x1) <= bound * np.linalg.norm(x1)


@pytest.fixture(scope="module")
def large():
    A = regular(560000, 13, seed=22)
    assert sliced(A) and 18 * A.nnz > 128 << 20
    rng = np.random.default_rng(5)
    return A, rng.standard_normal(A.n) + 1j * rng.standard_normal(A.n)


@pytest.mark.parametrize("name", ["bicgstab", "async", "bicgstabl", "tfqmr"])
def test_streamed_slices_follow_the_oracle(hz, large, name):
    A, b = large
    if name == "bicgstabl":
        want, bound = bicgstab_l(A, b, ell=2, tol=0.0, maxcycles=1, jacobi=True)[0], 1e-10
    elif name == "tfqmr":
        want, bound = tfqmr(A, b, tol=1e-30, maxiter=3, jacobi=True)[0], 1e-12
    else:
        want, bound = O.zbicgstab(A, b, tol=0.0, maxiter=5, jacobi=True)[0], 1e-12
    x = solve(hz, name, A, b)
    err = np.linalg.norm(x - want) / np.linalg.norm(want)
    print(f"{name}: {err:.2e}")
    assert err <= bound
