"""The batched sweep's D^-1 = 1 / (K_ii - k^2 M_ii + i k B_ii), which its kernels rebuild for every element, with all
three terms different from zero: iterates against the oracle on the assembled systems, with the bound of the other
batched tests (5 iterations of diagonally dominant systems, 1e-12).
"""

import numpy as np
import pytest
import torch

from test_gpu_iteration import dominant
from test_gpu_multi_iteration import check, cn, dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hz():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    import paper_2112_06465_amd as hz

    return hz


@pytest.mark.parametrize("n,B", [(65, 3), (16385, 2), (2000, 16)])
def test_every_term_of_the_diagonal(hz, n, B):
    A = dominant(n, seed=n + 2)
    rng = np.random.default_rng(B)
    diag = A.col_idx == A.row_of_entry()
    size = np.abs(A.vals[diag])
    K, M, Bm = A.vals.real.copy(), 0.01 * A.vals.imag, 0.02 * np.abs(A.vals)
    M[diag] = 0.3 * size * rng.uniform(0.5, 1.0, n)
    K[diag] = (1.5 + 4 * 0.3) * size  # exceeds the row's other moduli by what k^2 M takes at most (k <= 2)
    Bm[diag] = 0.4 * size
    ks = np.linspace(0.5, 2.0, B)
    vals = [K - k * k * M + 1j * k * Bm for k in ks]
    rhs = cn(rng, B, n)
    args = dev(A.row_ptr), dev(A.col_idx), dev(K), dev(M), dev(Bm), ks, dev(rhs.T)
    check(hz, A, vals, rhs, lambda flags, it: hz.zbicgstab_solve_sweep(*args, rtol=0.0, maxiter=it, flags=flags))
