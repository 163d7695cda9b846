"""Rows without 16-byte alignment (contiguous tensors of odd widths, base addresses off by one element) against the
same call on padded, aligned rows: every output element is the same sum of the same terms in the same order, so the
two results are equal bit for bit (the aligned path is compared with the oracle elsewhere).  Widths sit at the
edges of a vector (4 / 8 elements), of a lane group and of a column tile.  Guard elements around the outputs
must stay untouched.
"""
import numpy as np
import pytest
import torch

from gt_inputs import graphs
from gpu_util import announce, pad_to, up_i32

pytestmark = pytest.mark.gpu
GUARD = 1.25


def _graph():
    rp, ci = graphs.rmat_csr(10, 8, seed=41, self_loops=False)
    n = rp.size - 1
    dst = np.repeat(np.arange(n), np.diff(rp))
    rng = np.random.default_rng(3)
    rp, ci = graphs.csr_from_pairs(np.concatenate([ci, rng.choice(n, 400, replace=False)]),
                                   np.concatenate([dst, np.full(400, 11)]), n, n)   # one split row
    return rp, ci, n


def _rows(vals, dtype, aligned, off):
    """`vals` [n, F] as padded rows, or contiguous rows that start `off` elements into their buffer."""
    n, F = vals.shape
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    ld = pad_to(F, dtype) if aligned else F
    off = 0 if aligned else off
    buf = torch.full((off + n * ld + 16,), GUARD, dtype=tdt, device="cuda:0")
    t = buf.as_strided((n, F), (ld, 1), off)
    t.copy_(vals)
    return buf, t


def _guards_ok(buf, t, aligned, off):
    n, F = t.shape
    flat = buf.float()
    lo, hi = (0, buf.numel() - 16) if aligned else (off, off + n * F)
    return bool((flat[:lo] == GUARD).all()) and bool((flat[hi:] == GUARD).all())


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("F", [1, 3, 4, 5, 7, 8, 9, 15, 17, 31, 33, 47, 63, 65, 127, 129, 257, 513, 1025, 2049])
def test_unaligned_rows_match_padded_rows(F, dtype):
    from paper_2305_17469_amd import binding as B
    rp, ci, n = _graph()
    g = B.Graph(up_i32(rp), up_i32(ci), n)
    gen = torch.Generator(device="cuda:0").manual_seed(F)
    src = [torch.randn((n, F), device="cuda:0", generator=gen) for _ in range(2)]
    ew = torch.randn((g.n_edges, F), device="cuda:0", generator=gen)
    sw = torch.randn((g.n_edges,), device="cuda:0", generator=gen)
    for off in (0, 1, 3):
        announce("unaligned rows", dtype, "F", F, "offset", off)
        got = []
        for aligned in (True, False):
            _, X = _rows(src[0], dtype, aligned, off)
            _, D = _rows(src[1], dtype, aligned, off)
            _, W = _rows(ew, dtype, aligned, off)
            outs = {}

            def out(name, rows):
                buf, t = _rows(torch.full((rows, F), 7.0, device="cuda:0"), dtype, aligned, off)
                outs[name] = (buf, t)
                return t
            for reduce in ("mean", "symnorm"):
                B.gt_aggregate_fwd(g, reduce, X, out=out("fwd " + reduce, n))
                B.gt_aggregate_bwd(g, reduce, D, out=out("bwd " + reduce, n))
            B.gt_neighbor_apply_fwd(g, "mul", X, D, out=out("edge mul", g.n_edges))
            dot = B.gt_neighbor_apply_fwd(g, "dot", X, D)
            B.gt_neighbor_apply_bwd(g, "mul", W, X, D, out_dXs=out("mul dXs", n), out_dXd=out("mul dXd", n))
            B.gt_pull_fwd(g, "mean", "add", X, W, out=out("pull add", n))
            B.gt_pull_fwd(g, "sum", "scale", X, sw, out=out("pull scale", n))
            B.gt_pull_bwd(g, "mean", "mul", D, X, W, out_dXs=out("pull mul dXs", n), out_dW=out("pull mul dW", g.n_edges))
            torch.cuda.synchronize()
            for name, (buf, t) in outs.items():
                assert _guards_ok(buf, t, aligned, off), (name, F, off, "guard overwritten")
            got.append(({k: t.clone() for k, (_, t) in outs.items()}, dot))
        for k in got[0][0]:
            assert torch.equal(got[0][0][k], got[1][0][k]), (k, F, dtype, off)
        # the dot product's columns are spread over the lanes alike, apart from the last vector's: sums of at most F
        # fp32 products in another order, |difference| <= 2 F 2^-24 sum |x d|
        xs, ds = (t.to(torch.bfloat16).double() if dtype == "bf16" else t.double() for t in src)
        rows = torch.repeat_interleave(torch.arange(n, device="cuda:0"), up_i32(np.diff(rp)).long())
        mag = (xs[up_i32(ci).long()].abs() * ds[rows].abs()).sum(1)
        assert bool(((got[0][1].double() - got[1][1].double()).abs() <= 2 * F * 2.0 ** -24 * mag + 1e-30).all()), ("dot", F)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_unaligned_rows_keep_infinities_and_nan_apart(dtype):
    """An infinity or NaN in one vertex's row reaches exactly the outputs that gather that row, in its columns."""
    from paper_2305_17469_amd import binding as B
    rp, ci, n = _graph()
    g = B.Graph(up_i32(rp), up_i32(ci), n)
    F = 13
    X = torch.ones((n, F), device="cuda:0")
    hub = int(np.bincount(ci, minlength=n).argmax())
    X[hub, F - 1] = float("inf")
    X[n - 1, 0] = float("nan")
    announce("unaligned rows inf/nan", dtype)
    Y = B.gt_aggregate_fwd(g, "sum", X.to(torch.bfloat16) if dtype == "bf16" else X).float().cpu().numpy()
    has = np.zeros((2, n), dtype=bool)
    dst = np.repeat(np.arange(n), np.diff(rp))
    has[0, dst[ci == hub]] = True
    has[1, dst[ci == n - 1]] = True
    assert (np.isinf(Y[:, F - 1]) == has[0]).all() and (np.isnan(Y[:, 0]) == has[1]).all()
    assert np.isfinite(Y[:, 1:F - 1]).all()


@pytest.mark.parametrize("hub", [63, 64, 96, 97, 128, 700, 5000])
@pytest.mark.parametrize("F,dtype", [(3, "f32"), (16, "f32"), (41, "f32"), (100, "bf16"), (200, "f32")])
def test_long_rows_summed_by_many_groups(F, dtype, hub):
    """Long items are sliced over the groups of a wavefront or workgroup, and partial rows over the groups of a wavefront:
    rows around the lengths where an item becomes long or split, on a list of few items (row order) and one of many
    (sorted), against sums in 64 bits.  Bound: a term passes through at most hub fp32 additions, |error| <=
    hub 2^-24 sum |x| (bf16: plus the rounding of the result)."""
    from paper_2305_17469_amd import binding as B
    for n in (6000, 40000):
        rng = np.random.default_rng(hub + n)
        dst = np.concatenate([np.repeat(np.arange(0, n, 37), 3), np.full(hub, 5), np.full(max(hub - 1, 1), 17)])
        src = np.concatenate([rng.integers(0, n, dst.size - hub - max(hub - 1, 1)), rng.choice(n, hub, replace=False),
                              rng.choice(n, max(hub - 1, 1), replace=False)])
        rp, ci = graphs.csr_from_pairs(src, dst, n, n)
        g = B.Graph(up_i32(rp), up_i32(ci), n)
        announce("long rows", dtype, "F", F, "hub", hub, "n", n)
        X = torch.randn((n, F), device="cuda:0", generator=torch.Generator(device="cuda:0").manual_seed(hub))
        if dtype == "bf16":
            X = X.to(torch.bfloat16)
        Y = B.gt_aggregate_fwd(g, "sum", X)
        rows = torch.repeat_interleave(torch.arange(n, device="cuda:0"), up_i32(np.diff(rp)).long())
        t = X.double()[up_i32(ci).long()]
        ref = torch.zeros((n, F), dtype=torch.float64, device="cuda:0").index_add_(0, rows, t)
        mag = torch.zeros((n, F), dtype=torch.float64, device="cuda:0").index_add_(0, rows, t.abs())
        bound = hub * 2.0 ** -24 * mag + (2.0 ** -8 * ref.abs() if dtype == "bf16" else 0)
        assert bool(((Y.double() - ref).abs() <= bound).all())
        assert torch.equal(Y, B.gt_aggregate_fwd(g, "sum", X))


@pytest.mark.parametrize("n,F,dtype", [(530000, 64, "bf16"), (60000, 200, "f32"), (530000, 17, "f32"), (90000, 256, "bf16")])
def test_long_rows_of_large_tables(n, F, dtype):
    """The same where the table is past 32 MiB (two rows in flight): mean of rows of 63 to 5,000 entries, bound as above."""
    from paper_2305_17469_amd import binding as B
    hubs = [63, 64, 65, 96, 127, 129, 700, 5000]
    rng = np.random.default_rng(n)
    dst = np.concatenate([np.repeat(np.arange(0, n, 4), 2)] + [np.full(h, 11 * (i + 1)) for i, h in enumerate(hubs)])
    src = np.concatenate([rng.integers(0, n, dst.size - sum(hubs))] + [rng.choice(n, h, replace=False) for h in hubs])
    rp, ci = graphs.csr_from_pairs(src, dst, n, n)
    g = B.Graph(up_i32(rp), up_i32(ci), n)
    announce("long rows, large table", dtype, "F", F, "n", n)
    v = 8 if dtype == "bf16" else 4
    X = torch.randn((n, (F + v - 1) // v * v), device="cuda:0", generator=torch.Generator(device="cuda:0").manual_seed(n))
    X = (X.to(torch.bfloat16) if dtype == "bf16" else X)[:, :F]
    Y = B.gt_aggregate_fwd(g, "mean", X)
    deg = up_i32(np.diff(rp)).long()
    rows = torch.repeat_interleave(torch.arange(n, device="cuda:0"), deg)
    t = X.double()[up_i32(ci).long()]
    zero = torch.zeros((n, F), dtype=torch.float64, device="cuda:0")
    ref, mag = zero.index_add(0, rows, t) / deg.clamp(min=1)[:, None], zero.index_add(0, rows, t.abs()) / deg.clamp(min=1)[:, None]
    bound = (deg[:, None] + 1) * 2.0 ** -24 * mag + (2.0 ** -8 * ref.abs() if dtype == "bf16" else 0)
    assert bool(((Y.double() - ref).abs() <= bound).all())
    assert torch.equal(Y, B.gt_aggregate_fwd(g, "mean", X))
