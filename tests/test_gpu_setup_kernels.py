"""The set-up kernels' edges, exactly: rows of every length around the row sort's lanes (16 a row, four entries each) and
past them, with repeated columns, whose order must be kept; and transposes whose row pointers end inside, at and past a
round of the scan (16,384 elements) and of a thread's 16.
"""

import numpy as np
import pytest
import torch

from workloads.csr import CSR

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hz():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    import paper_2112_06465_amd as hz

    return hz


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


@pytest.mark.parametrize("lengths", [[0, 1, 2], [15, 16, 17, 0, 1], [47, 48, 49, 63, 64], [65, 1, 200, 64, 0], [3] * 40])
def test_rows_are_sorted_stably(hz, lengths):
    rng = np.random.default_rng(len(lengths))
    n = 7 * len(lengths)
    lens = np.tile(lengths, 7)
    rp = np.zeros(n + 1, np.int32)
    np.cumsum(lens, out=rp[1:])
    ci = rng.integers(0, n, rp[-1]).astype(np.int32)  # repeated columns among them
    v = rng.standard_normal(ci.size) + 1j * np.arange(ci.size)
    perm = rng.permutation(n).astype(np.int32)
    inv = np.empty(n, np.int32)
    inv[perm] = np.arange(n, dtype=np.int32)
    rp2, ci2, v2 = (t.cpu().numpy() for t in hz.csr_zpermute(dev(rp), dev(ci), dev(v), dev(perm), dev(inv)))
    want_c, want_v = [], []
    for o in perm:
        c, w = inv[ci[rp[o]:rp[o + 1]]], v[rp[o]:rp[o + 1]]
        order = np.argsort(c, kind="stable")
        want_c.append(c[order])
        want_v.append(w[order])
    assert np.array_equal(np.diff(rp2), lens[perm])
    assert np.array_equal(ci2, np.concatenate(want_c)) and np.array_equal(v2, np.concatenate(want_v))


@pytest.mark.parametrize("n", [1, 14, 15, 16, 17, 1023, 16382, 16383, 16384, 16385, 40001])
def test_transpose_of_every_length(hz, n):
    """lambda of a non-symmetric, diagonally dominant system; A^H lambda is formed here and compared to 1e-12."""
    rng = np.random.default_rng(n)
    r = np.concatenate([np.arange(n), np.arange(n), np.arange(n)])
    c = np.concatenate([np.arange(n), (np.arange(n) * 7 + 3) % n, np.minimum(np.arange(n) + 1, n - 1)])
    key = np.unique(r.astype(np.int64) * n + c)
    r, c = (key // n).astype(np.int64), (key % n).astype(np.int32)
    v = rng.standard_normal(r.size) + 1j * rng.standard_normal(r.size)
    v[r == c] = 20.0 + 3.0j
    rp = np.zeros(n + 1, np.int32)
    np.cumsum(np.bincount(r, minlength=n), out=rp[1:])
    A = CSR(rp, c, v)
    g = rng.standard_normal(n) + 1j * rng.standard_normal(n)
    lam, _, info = hz.zbicgstab_adjoint(dev(A.row_ptr), dev(A.col_idx), dev(A.vals), dev(g), dev(g), rtol=1e-13,
                                        flags=hz.PRECOND_JACOBI | hz.NO_REORDER)
    y = np.zeros(n, complex)
    np.add.at(y, A.col_idx, np.conj(A.vals) * lam.cpu().numpy()[r])
    assert info["status"] == hz.OK
    assert np.linalg.norm(y - g) <= 1e-12 * np.linalg.norm(g)
