"""The batched iteration at the edges of its launch map: a block's one tile of rows and its second (64, 16 or 4 rows a
tile by the number of systems, 256 blocks), rows that fill a batch of gathers or exceed it by one, and idle lanes.

The systems are those of the one-system iteration's tests, whose iterates barely amplify rounding: under Jacobi five
iterations, without it one, are held to 1e-12 of the oracle's (rounding of n-term sums in another order at the
largest n).
"""

import numpy as np
import pytest
import torch

import oracle as O
from test_gpu_iteration import dominant

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hz():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    import paper_2112_06465_amd as hz

    return hz


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def cn(rng, *shape):
    return rng.standard_normal(shape) + 1j * rng.standard_normal(shape)


def check(hz, A, vals, rhs, run):
    for jacobi in (True, False):
        flags = (hz.PRECOND_JACOBI if jacobi else hz.PRECOND_NONE) | hz.X0_ZERO
        iters = 5 if jacobi else 1
        x, infos = run(flags, iters)
        x = x.cpu().numpy()
        for j, v in enumerate(vals):
            xo, io = O.zbicgstab(A.with_vals(v), rhs[j], tol=0.0, maxiter=iters, jacobi=jacobi)
            assert infos[j]["iterations"] == iters == io["iterations"] and infos[j]["status"] == hz.NOT_CONVERGED
            err = np.linalg.norm(x[:, j] - xo) / np.linalg.norm(xo)
            assert err <= 1e-12, (jacobi, j, err)
            assert abs(infos[j]["relres_recursive"] - io["relres_recursive"]) <= 1e-9 * io["relres_recursive"]


@pytest.mark.parametrize("n,B", [(63, 3), (65, 16), (1000, 1), (16384, 2), (16385, 3), (16449, 16), (40000, 5)])
def test_explicit_values_follow_the_oracle(hz, n, B):
    A = dominant(n, seed=n)
    rng = np.random.default_rng(B)
    vals = [A.vals * np.exp(0.3j * j) * (1.0 + 0.1 * j) for j in range(B)]
    rhs = cn(rng, B, n)
    args = dev(A.row_ptr), dev(A.col_idx), dev(np.stack(vals, 1)), dev(rhs.T)
    check(hz, A, vals, rhs, lambda flags, it: hz.zbicgstab_solve_batched(*args, rtol=0.0, maxiter=it, flags=flags))


@pytest.mark.parametrize("n,B", [(65, 3), (16384, 16), (16385, 2), (40000, 3)])
def test_sweep_follows_the_oracle(hz, n, B):
    A = dominant(n, seed=n + 1)
    rng = np.random.default_rng(B)
    diag = A.col_idx == A.row_of_entry()
    K, M, Bm = A.vals.real.copy(), 0.01 * A.vals.imag, 0.02 * np.abs(A.vals)
    K[diag] = 1.5 * np.abs(A.vals[diag])  # the diagonal exceeds the row's other moduli
    M[diag] = 0.0
    ks = np.linspace(0.5, 2.0, B)
    vals = [K - k * k * M + 1j * k * Bm for k in ks]
    rhs = cn(rng, B, n)
    args = dev(A.row_ptr), dev(A.col_idx), dev(K), dev(M), dev(Bm), ks, dev(rhs.T)
    check(hz, A, vals, rhs, lambda flags, it: hz.zbicgstab_solve_sweep(*args, rtol=0.0, maxiter=it, flags=flags))


@pytest.mark.parametrize("n,B", [(4096, 17), (4097, 17), (1024, 65), (1025, 65), (3000, 128)])
def test_wide_lanes_solve_the_adjoint(hz, n, B):
    """More than 16 systems in one launch (64 and 256 lanes), through the batched adjoint."""
    A = dominant(n, seed=n)
    vals = [A.vals * np.exp(0.1j * j) for j in range(B)]
    G = cn(np.random.default_rng(B), n, B)
    lam, _, infos = hz.zbicgstab_adjoint_batched(dev(A.row_ptr), dev(A.col_idx), dev(np.stack(vals, 1)), None, dev(G),
                                                 rtol=1e-10, flags=hz.PRECOND_JACOBI, want_grad_vals=False)
    lam = lam.cpu().numpy()
    dense = np.zeros(A.n, complex)
    for j in (0, 1, B // 2, B - 1):
        assert infos[j]["status"] == hz.OK
        rows = A.row_of_entry()
        y = dense.copy()
        np.add.at(y, A.col_idx, np.conj(vals[j]) * lam[rows, j])
        assert np.linalg.norm(y - G[:, j]) <= 1e-10 * (1 + 1e-3) * np.linalg.norm(G[:, j])
