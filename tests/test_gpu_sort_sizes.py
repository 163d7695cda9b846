"""Plan and renumbering at the sizes where the sort and scan change form (one launch up to 16,384 pairs; tiles of 1,024 up
to 131,072, of 4,096 up to 524,288, of 4,096 or 8,192 with scanned counts beyond), with long runs of empty rows and of
vertices without out-edges.  Integer results: equal to numpy's stable sort, element by element."""
import numpy as np
import pytest
import torch

from gpu_util import announce, up_i32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E", [1, 63, 2047, 2049, 16384, 16385, 131072, 131073, 524288, 524289, 1048577])
@pytest.mark.parametrize("n", [3, 300, 70001])
def test_plan_structure(n, E):
    from paper_2305_17469_amd import binding as B
    rng = np.random.default_rng(E + n)
    # destinations and sources from three narrow bands, so that most rows are empty in long runs
    band = np.array([0, n // 2, n - 1])
    dst = np.sort(np.minimum(band[rng.integers(0, 3, E)] + rng.integers(0, max(1, n // 50), E), n - 1))
    src = np.minimum(band[rng.integers(0, 3, E)] + rng.integers(0, max(1, n // 50), E), n - 1)
    rp = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(np.bincount(dst, minlength=n), out=rp[1:])
    announce("plan sizes", "n", n, "E", E)
    g = B.Graph(up_i32(rp), up_i32(src), n)
    got = [t.cpu().numpy() for t in g.outputs()]
    perm = np.argsort(src, kind="stable")
    rpt = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(np.bincount(src, minlength=n), out=rpt[1:])
    for name, a, b in zip(("in_deg", "out_deg", "rowptr_t", "colidx_t", "perm"), got,
                          (np.diff(rp), np.diff(rpt), rpt, dst[perm], perm)):
        assert np.array_equal(a, b), name
    # the per-entry coefficients of both orders, through aggregations of ones and of the vertex ids
    deg = np.diff(rp)
    inv = np.where(deg > 0, 1.0 / np.sqrt(np.maximum(deg, 1)), 0.0)
    X = torch.arange(n, device="cuda:0", dtype=torch.float32).reshape(n, 1).repeat(1, 4) / n
    x = np.arange(n) / n
    for what, f, ref in (("fwd", lambda: B.gt_aggregate_fwd(g, "symnorm", X), np.bincount(dst, inv[src] * inv[dst] * x[src], n)),
                         ("bwd", lambda: B.gt_aggregate_bwd(g, "symnorm", X), np.bincount(src, inv[src] * inv[dst] * x[dst], n)),
                         ("mean", lambda: B.gt_aggregate_bwd(g, "mean", X), np.bincount(src, x[dst] / deg[dst], n))):
        y = f().cpu().numpy().astype(np.float64)
        # positive terms: the relative error of an fp32 sum of k terms is at most k 2^-24, and 4 more roundings per term
        assert (np.abs(y - ref[:, None]) <= (max(deg.max(), np.diff(rpt).max()) + 4) * 2.0 ** -24 * ref[:, None] + 1e-30).all(), what


@pytest.mark.parametrize("n_picked", [5, 16300, 16500, 131000, 140000, 530000])
def test_reindex_first_met_order(n_picked):
    from paper_2305_17469_amd import binding as B
    rng = np.random.default_rng(n_picked)
    n_vertices = 300007
    dst = rng.choice(n_vertices, 100, replace=False).astype(np.int32)
    picked = rng.integers(0, max(200, n_picked // 3), n_picked).astype(np.int32)
    announce("reindex sizes", n_picked)
    src, local = B.gt_reindex(up_i32(dst), up_i32(picked), n_vertices)
    seen = np.concatenate([dst, picked])
    ids, first = np.unique(seen, return_index=True)
    order = np.argsort(first, kind="stable")
    new = np.empty(ids.size, dtype=np.int64)
    new[order] = np.arange(ids.size)
    assert np.array_equal(src.cpu().numpy(), ids[order])
    assert np.array_equal(local.cpu().numpy(), new[np.searchsorted(ids, picked)])
