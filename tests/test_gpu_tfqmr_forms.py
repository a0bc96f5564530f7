"""TFQMR's iteration in its forms: two launches (u' and u formed per gathered column) and four, on the CSR operator and
on the sliced one, at sizes on both sides of a slice, a block and the lines between the forms, and every way to end.

The systems are diagonally dominant; the iterates of three iterations are held to 1e-12 of the oracle's, the bound of
three iterations on the coarse cylinder, which amplifies more.  The two forms do the same arithmetic per element and
add the same partial sums, so their results are the same bit for bit.
"""

import numpy as np
import pytest
import torch

from oracle.tfqmr import tfqmr
from test_gpu_bicgstabl_steps import dominant
from workloads.csr import CSR

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hz():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    import paper_2112_06465_amd as hz

    return hz


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def both(hz, monkeypatch, A, b, **kw):
    """The result of the default form, after checking that the two forms agree bit for bit."""
    args = dev(A.row_ptr), dev(A.col_idx), dev(A.vals), dev(b)
    out = []
    for fused in ("0", "1", None):
        if fused is None:
            monkeypatch.delenv("HZ_FUSED")
        else:
            monkeypatch.setenv("HZ_FUSED", fused)
        out.append(hz.ztfqmr_solve(*args, **kw))
    for x, info in out[:2]:
        assert torch.equal(torch.view_as_real(x), torch.view_as_real(out[2][0])) and info == out[2][1]
    return out[2][0].cpu().numpy(), out[2][1]


@pytest.mark.parametrize("n,far,jacobi", [
    (3, 0, True), (63, 0, True), (65, 0, True), (1023, 0, False), (1025, 0, True), (8192, 0, True), (8193, 0, False),
    (57344, 0, False), (57345, 0, False), (163840, 0, True), (163841, 0, True), (40000, 32761, True)])
def test_iterates_follow_the_oracle(hz, monkeypatch, n, far, jacobi):
    A, b = dominant(n, far)
    flags = (hz.PRECOND_JACOBI if jacobi else hz.PRECOND_NONE) | hz.X0_ZERO | hz.NO_REORDER
    iters = 1 if n < 8 else 3
    x, info = both(hz, monkeypatch, A, b, rtol=1e-30, maxiter=iters, flags=flags)
    xo, io = tfqmr(A, b, tol=1e-30, maxiter=iters, jacobi=jacobi)
    assert info["status"] == hz.NOT_CONVERGED and info["iterations"] == iters == io["iterations"]
    err = np.linalg.norm(x - xo) / np.linalg.norm(xo)
    print(f"n={n} far={far} jacobi={jacobi}: {err:.2e}")
    assert err <= 1e-12
    assert abs(info["relres_recursive"] - io["relres_recursive"]) <= 1e-8 * io["relres_recursive"]


@pytest.mark.parametrize("jacobi", [False, True])
@pytest.mark.parametrize("tol", [1e-1, 1e-2, 1e-3, 1e-4, 1e-7, 1e-10])
def test_exits_in_either_half_step(hz, monkeypatch, tol, jacobi):
    """Tolerances that end the solve after a first or a second half step.  Without Jacobi on the matrix scaled by its
    diagonal, which converges alike: a relative perturbation of 1e-16 of b moves the solution by 4e-16."""
    A, b = dominant(5000)
    if not jacobi:
        diag = A.vals[A.col_idx == A.row_of_entry()]
        A = CSR(A.row_ptr, A.col_idx, A.vals / diag[A.col_idx])
    flags = (hz.PRECOND_JACOBI if jacobi else hz.PRECOND_NONE) | hz.X0_ZERO | hz.NO_REORDER
    x, info = both(hz, monkeypatch, A, b, rtol=tol, flags=flags)
    xo, io = tfqmr(A, b, tol=tol, jacobi=jacobi)
    assert info["status"] == hz.OK and info["iterations"] == io["iterations"]
    assert np.linalg.norm(x - xo) <= 1e-9 * np.linalg.norm(xo)
    assert abs(info["relres_recursive"] - io["relres_recursive"]) <= 1e-6 * io["relres_recursive"]


def test_identity_ends_at_once(hz, monkeypatch):
    n = 2000
    A = CSR(np.arange(n + 1, dtype=np.int32), np.arange(n, dtype=np.int32), np.full(n, 2.0 - 0.5j))
    b = np.random.default_rng(1).standard_normal(n) + 0j
    for flags in (hz.PRECOND_JACOBI, hz.PRECOND_NONE):
        x, info = both(hz, monkeypatch, A, b, rtol=1e-14, flags=flags | hz.X0_ZERO | hz.NO_REORDER)
        assert info["status"] == hz.OK and info["iterations"] == 1
        assert np.linalg.norm(x - b / (2.0 - 0.5j)) <= 1e-14 * np.linalg.norm(b / (2.0 - 0.5j))
