"""The set-up kernels with 16 lanes a row (the row sort) or a node (the ordering keys) past the rows of one launch,
2^24, and past the 2^28 whose threads one launch cannot hold.  Exact.
"""

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hz():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    import paper_2112_06465_amd as hz

    return hz


@pytest.mark.parametrize("n", [2**24 + 5, 2**28 + 17])
def test_rows_past_one_launch_are_sorted(hz, n):
    """Rows reversed; every 16th has three entries, whose columns the reversal puts in falling order, the others one."""
    i = torch.arange(n, dtype=torch.int32, device="cuda:0")
    many = i % 16 == 3
    rp = torch.zeros(n + 1, dtype=torch.int32, device="cuda:0")
    torch.cumsum(torch.where(many, 3, 1), 0, dtype=torch.int32, out=rp[1:])
    ci = torch.empty(int(rp[-1]), dtype=torch.int32, device="cuda:0")
    ci[rp[:-1].long()] = torch.where(many, i - 3, i)
    at = rp[:-1][many].long()
    ci[at + 1], ci[at + 2] = i[many], i[many] - 1
    vals = torch.empty(ci.numel(), dtype=torch.complex128, device="cuda:0")
    torch.view_as_real(vals)[:, 0] = ci
    torch.view_as_real(vals)[:, 1] = 1.0
    perm = n - 1 - i
    rp2, ci2, v2 = hz.csr_zpermute(rp, ci, vals, perm, perm)
    assert torch.equal(rp2[1:] - rp2[:-1], (rp[1:] - rp[:-1]).flip(0))
    first = rp2[:-1].long()
    assert torch.equal(ci2[first[~many[perm.long()]]], i[~many[perm.long()]])
    at = first[many[perm.long()]]
    k = i[many[perm.long()]]
    for e, c in enumerate((k, k + 1, k + 3)):
        assert torch.equal(ci2[at + e], c)
    assert torch.equal(torch.view_as_real(v2)[:, 0], (n - 1 - ci2).double())


def test_level_past_one_launch_is_ordered(hz):
    """4,096 nodes with 4,100 leaves each, numbered in turn, so that the last level has more than 2^24 nodes: they must
    follow their parents' order, and their own numbers below one parent."""
    mids, per = 4096, 4100
    leaves = mids * per
    n = 1 + mids + leaves
    d = "cuda:0"
    leaf = torch.arange(leaves, device=d)
    parent = 1 + leaf % mids
    # rows: the root -> every inner node, an inner node -> its leaves, a leaf -> its parent (the first leaf -> the root too)
    lens = torch.ones(n, dtype=torch.int64, device=d)
    lens[0], lens[1:1 + mids], lens[1 + mids] = mids, per, 2
    rp = torch.zeros(n + 1, dtype=torch.int32, device=d)
    rp[1:] = lens.cumsum(0)
    inner = (1 + mids + torch.arange(mids, device=d)[:, None] + mids * torch.arange(per, device=d)[None, :]).reshape(-1)
    ci = torch.cat([1 + torch.arange(mids, device=d), inner, torch.zeros(1, dtype=torch.int64, device=d), parent]).to(torch.int32)
    perm, inv, level = hz.csr_level_order(rp, ci)
    # from the first leaf: its parent and the root, then that parent's leaves and the other inner nodes, then the rest
    last = level == 3
    assert int(level.max()) == 3 and int(last.sum()) == leaves - per > 2**24
    tail = perm[n - (leaves - per):].long()
    assert bool(last[tail].all()) and torch.equal(torch.sort(tail).values, torch.nonzero(last).reshape(-1))
    key = inv[parent[tail - 1 - mids]].long() * n + tail
    assert bool((key[1:] > key[:-1]).all())
    assert torch.equal(inv[perm.long()], torch.arange(n, dtype=torch.int32, device=d))
