"""A diagonal entry without a usable reciprocal, in a row and column of its own (an eliminated node): NaN, infinite, or
of a modulus whose square leaves the range of a double.  No solve may report success: D^-1 holds a NaN, an infinity
or a zero there, so the first product is not finite, or the system is singular.
"""

import numpy as np
import pytest
import torch

from test_gpu_initial_guess import sliced, solver
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


def with_lone_row(A, i, d):
    """A with row and column i cleared but for the diagonal d."""
    rows = A.row_of_entry()
    keep = ((rows != i) & (A.col_idx != i)) | ((rows == i) & (A.col_idx == i))
    rp = np.zeros(A.n + 1, np.int32)
    np.cumsum(np.bincount(rows[keep], minlength=A.n), out=rp[1:])
    vals = A.vals[keep]
    vals[rp[i]] = d
    return CSR(rp, A.col_idx[keep], vals)


@pytest.mark.parametrize("d", [complex(np.nan, 0), complex(0, np.inf), 1e-200, 1e200 + 1e200j], ids=str)
@pytest.mark.parametrize("name", ["bicgstab", "async", "bicgstabl", "tfqmr", "adjoint"])
def test_no_success_without_a_reciprocal(hz, name, d):
    A = with_lone_row(regular(12544, 6, seed=11), 7000, d)
    assert sliced(A)
    rng = np.random.default_rng(2)
    b = dev(rng.standard_normal(A.n) + 1j * rng.standard_normal(A.n))
    args = dev(A.row_ptr), dev(A.col_idx), dev(A.vals)
    flags = hz.PRECOND_JACOBI | hz.NO_REORDER
    if name == "adjoint":
        _, _, info = hz.zbicgstab_adjoint(*args, b, b, rtol=1e-10, maxiter=200, flags=flags, want_grad_vals=False)
    else:
        limit = {"maxcycles": 30} if name == "bicgstabl" else {"maxiter": 200}
        _, info = solver(hz, name)(*args, b, rtol=1e-10, flags=flags | hz.X0_ZERO, **limit)
    print(name, d, info)
    if abs(d) == 2**0.5 * 1e200:
        assert info["status"] in (hz.NOT_CONVERGED, hz.BREAKDOWN, hz.NONFINITE)
    else:
        assert info["status"] == hz.NONFINITE


@pytest.mark.parametrize("d", [1e-150, 1e150j])
@pytest.mark.parametrize("name", ["bicgstab", "async", "bicgstabl", "tfqmr", "adjoint"])
def test_extreme_reciprocals_are_used(hz, name, d):
    """Moduli at the ends of the range that has one: the lone unknown is b / d to a few roundings."""
    i = 7000
    A = with_lone_row(regular(12544, 6, seed=11), i, d)
    rng = np.random.default_rng(2)
    b = rng.standard_normal(A.n) + 1j * rng.standard_normal(A.n)
    args = dev(A.row_ptr), dev(A.col_idx), dev(A.vals)
    flags = hz.PRECOND_JACOBI | hz.NO_REORDER
    if name == "adjoint":
        x, _, info = hz.zbicgstab_adjoint(*args, dev(b), dev(b), rtol=1e-10, flags=flags, want_grad_vals=False)
        d = np.conj(d)
    else:
        x, info = solver(hz, name)(*args, dev(b), rtol=1e-10, flags=flags | hz.X0_ZERO)
    assert info["status"] == hz.OK
    assert abs(x[i].item() * d - b[i]) <= 1e-10 * np.linalg.norm(b)
