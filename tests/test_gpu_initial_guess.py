"""Every solver that takes x, from a guess under Jacobi: on a matrix that is sliced, on one that is kept in CSR by a
single far column, and on a renumbered one.

The recursive residual before the first step is compared with the host's ||b - A x0|| / ||b||: both are sums of n
rounded terms, in another order, so they agree to n u (4e-12 at the largest n) at worst.  The systems are diagonally dominant, so that
the true residual of the solution follows the recursive one: it is held to the tolerance and a hundredth.
"""

import numpy as np
import pytest
import torch

import oracle as O
from test_gpu_iteration import regular
from workloads.csr import permute_symmetric

pytestmark = pytest.mark.gpu

TOL = 1e-10


@pytest.fixture(scope="module")
def hz():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    import paper_2112_06465_amd as hz

    return hz


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def sliced(A):
    """Whether the matrix fits the sliced operator: 16-bit columns from the slice's first row, and no more slots (64
    times a slice's longest row, the diagonal left out) than entries."""
    base = A.row_of_entry() // 64 * 64
    far = A.col_idx - base
    lens = np.zeros((A.n + 63) // 64 * 64, np.int64)
    lens[: A.n] = np.diff(A.row_ptr) - 1
    return far.min() >= -32768 and far.max() <= 32767 and 64 * lens.reshape(-1, 64).max(1).sum() <= A.nnz


def matrix(kind):
    A = regular(40000, 13, seed=3, far=32761 if kind == "far" else 0)
    if kind == "renumbered":
        A = permute_symmetric(A, np.random.default_rng(4).permutation(A.n))
    assert sliced(A) == (kind == "sliced")
    return A


def solver(hz, name):
    if name == "async":
        def run(*args, flags, **kw):
            x, info = hz.zbicgstab_solve_async(*args, flags=flags & ~hz.NO_REORDER, **kw)
            return x, hz.read_info(info)

        return run
    return {"bicgstab": hz.zbicgstab_solve, "bicgstabl": hz.zbicgstabl_solve, "tfqmr": hz.ztfqmr_solve,
            "mixed": hz.zbicgstab_solve_mixed}[name]


@pytest.mark.parametrize("name,kind", [(name, kind) for name in ("bicgstab", "async", "bicgstabl", "tfqmr", "mixed")
                                       for kind in ("sliced", "far", "renumbered")
                                       if (name, kind) != ("async", "renumbered")])  # which does not renumber
def test_guess_under_jacobi(hz, name, kind):
    A = matrix(kind)
    rng = np.random.default_rng(6)
    b, near = (rng.standard_normal(A.n) + 1j * rng.standard_normal(A.n) for _ in range(2))
    args = dev(A.row_ptr), dev(A.col_idx), dev(A.vals), dev(b)
    order = hz.REORDER if kind == "renumbered" else hz.NO_REORDER
    x, info = solver(hz, name)(*args, rtol=TOL, flags=hz.PRECOND_JACOBI | hz.X0_ZERO | order)
    assert info["status"] == hz.OK
    x0 = 0.5 * x.cpu().numpy() + 1e-3 * near / np.abs(A.vals).max()
    x, info = solver(hz, name)(*args, x=dev(x0), rtol=TOL, flags=hz.PRECOND_JACOBI | order)
    res = np.linalg.norm(b - O.zspmv(A, x.cpu().numpy())) / np.linalg.norm(b)
    print(f"{name} {kind}: true residual {res:.2e}")
    assert info["status"] == hz.OK and res <= TOL * 1.01
    if name != "mixed":
        limit = {"maxcycles": 0} if name == "bicgstabl" else {"maxiter": 0}
        x, info = solver(hz, name)(*args, x=dev(x0), rtol=TOL, flags=hz.PRECOND_JACOBI | order, **limit)
        r0 = np.linalg.norm(b - O.zspmv(A, x0)) / np.linalg.norm(b)
        assert info["status"] == hz.NOT_CONVERGED and info["iterations"] == 0
        assert abs(info["relres_recursive"] - r0) <= 1e-11 * r0
        assert np.abs(x.cpu().numpy() - x0).max() <= 1e-14 * np.abs(x0).max()  # scaled by D and back
