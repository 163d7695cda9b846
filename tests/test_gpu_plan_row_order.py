"""Plans on both sides of the bound up to which work lists stay in row order and are filled before their sizes are read back (rows plus chunks of the larger side,
16,384): square and lopsided blocks, hubs in either direction, no edges.  Sums of small integers are exact: both directions equal torch's bit for
bit, and the sizes that the plan reports add up."""
import numpy as np
import pytest
import torch

from gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_dst,n_src,E,hub", [(1, 1, 0, False), (300, 1900, 1700, True), (5, 9000, 8000, False), (16000, 3, 20000, False), (16254, 16254, 8192, True), (16255, 16255, 8192, True),
                                               (16256, 100, 8192, True), (100, 16256, 8192, True), (16383, 16383, 0, False), (16384, 16384, 63, False), (2000, 13000, 18000, True)])
def test_row_order(n_dst, n_src, E, hub):
    from paper_2305_17469_amd import binding as B
    rng = np.random.default_rng(n_dst + E)
    dst, src = rng.integers(0, n_dst, E), rng.integers(0, n_src, E)
    if hub:                                   # rows of several chunks in both directions
        dst[: E // 4], src[E // 4: E // 2] = n_dst // 2, n_src // 3
    dst = np.sort(dst)
    rowptr = torch.from_numpy(np.concatenate([[0], np.cumsum(np.bincount(dst, minlength=n_dst))]).astype(np.int32)).cuda()
    announce("row order", n_dst, n_src, E, hub)
    g = B.Graph(rowptr, torch.from_numpy(src.astype(np.int32)).cuda(), n_src)
    d, s = torch.from_numpy(dst).cuda(), torch.from_numpy(src).cuda()
    F = 20
    X = torch.from_numpy(rng.integers(-4, 5, (n_src, F)).astype(np.float32)).cuda()
    G = torch.from_numpy(rng.integers(-4, 5, (n_dst, F)).astype(np.float32)).cuda()
    assert torch.equal(B.gt_aggregate_fwd(g, "sum", X), torch.zeros((n_dst, F), device="cuda:0").index_add_(0, d, X[s]))
    assert torch.equal(B.gt_aggregate_bwd(g, "sum", G), torch.zeros((n_src, F), device="cuda:0").index_add_(0, s, G[d]))
    i = g.info()
    chunk = 512
    while chunk > 64 and E / chunk < 4096:
        chunk //= 2
    for side, count in (("fwd", np.bincount(dst, minlength=n_dst)), ("bwd", np.bincount(src, minlength=n_src))):
        split = count > chunk + chunk // 2
        assert i[side + "_split_rows"] == split.sum()
        assert i[side + "_items"] == (~split).sum() + ((count[split] + chunk - 1) // chunk).sum()
