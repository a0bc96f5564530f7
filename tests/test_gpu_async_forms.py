"""The asynchronous solve, whose products choose the operator's form on the device, against the synchronous one, bit for
bit: on both sides of the lines between the fused and the split iteration (57,344, 131,072 and 163,840 rows), for
matrices that are sliced and one far column away from it, with vector rows and with tiles, with and without Jacobi,
stopped by the limit and converged with launches to spare.
"""

import numpy as np
import pytest
import torch

from test_gpu_initial_guess import sliced
from test_gpu_iteration import regular

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hz():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    import paper_2112_06465_amd as hz

    return hz


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


@pytest.mark.parametrize("lanes", [None, "1"])
@pytest.mark.parametrize("n,far", [(12544, 0), (40000, 32761), (57345, 0), (57345, 32761), (131072, 32761), (131073, 0),
                                   (131073, 32761), (163840, 0), (163840, 32761), (163841, 0), (163841, 32761)])
def test_same_bits_as_synchronous(hz, monkeypatch, n, far, lanes):
    if lanes is not None:
        monkeypatch.setenv("HZ_SPMV_LANES", lanes)
    A = regular(n, 6, seed=n, far=far)
    assert sliced(A) == (far == 0)
    rng = np.random.default_rng(9)
    args = dev(A.row_ptr), dev(A.col_idx), dev(A.vals), dev(rng.standard_normal(n) + 1j * rng.standard_normal(n))
    for precond, kw in ((hz.PRECOND_JACOBI, dict(rtol=0.0, maxiter=5)), (hz.PRECOND_JACOBI, dict(rtol=1e-9, maxiter=70)),
                        (hz.PRECOND_NONE, dict(rtol=0.0, maxiter=2))):
        xs, want = hz.zbicgstab_solve(*args, flags=precond | hz.X0_ZERO | hz.NO_REORDER, **kw)
        calls = [hz.zbicgstab_solve_async]
        if hz.zbicgstab_workspace_bytes(n, A.nnz, precond) <= hz.zbicgstab_noalloc_max_bytes():
            calls.append(hz.zbicgstab_solve_noalloc)
        for call in calls:
            x, info = call(*args, flags=precond | hz.X0_ZERO, **kw)
            assert hz.read_info(info) == want
            assert torch.equal(torch.view_as_real(x), torch.view_as_real(xs))
        assert want["status"] == (hz.OK if kw["rtol"] > 0 else hz.NOT_CONVERGED)
