"""The aggregation on graphs at both sides of its rules for long rows: every row long, too few of them to fill the chip and
more than enough; a few hub rows among short ones (split rows, shared-out items); short rows only, with and without the
launches that hold several ids per lane.  Widths for every lane-group size, both types, padded and contiguous rows, both
directions, against 64 bits: |error| <= (n + 2) 2^-24 sum |x| for a row of n entries (any order of fp32 additions), one bf16
rounding more for bf16 results."""
import numpy as np
import pytest
import torch

from gpu_util import announce

pytestmark = pytest.mark.gpu


def _fixed(n, d, rng):
    return np.arange(0, n * d + 1, d), rng.integers(0, n, (n, d))


def _graph(name):
    rng = np.random.default_rng(len(name))
    if name.startswith("long"):
        n, d = {"long130": (600, 130), "long600": (900, 600), "long130many": (9000, 130)}[name]
        rowptr, col = _fixed(n, d, rng)
        return n, rowptr, np.sort(col, axis=1).reshape(-1)
    if name == "hubs":
        deg = rng.integers(0, 20, 30000)
        deg[rng.choice(30000, 12, replace=False)] = rng.integers(300, 6000, 12)
    elif name == "hubswide":   # (a table past 32 MiB at the widest rows, whose hubs are shared out with two rows in flight)
        deg = rng.integers(2, 10, 70000)
        deg[rng.choice(70000, 20, replace=False)] = rng.integers(300, 6000, 20)
    elif name == "hubsmid":    # (hubs that a workgroup each sums whole, in a launch of column tiles)
        deg = rng.integers(8, 21, 90000)
        deg[rng.choice(90000, 30, replace=False)] = rng.integers(500, 1000, 30)
    elif name == "skewed":     # (three long items to ten)
        deg = np.where(rng.random(8000) < 0.3, rng.integers(32, 130, 8000), rng.integers(0, 20, 8000))
    else:
        deg = rng.integers(8, 25, {"short": 20000, "shortmany": 140000}[name])
    rowptr = np.concatenate([[0], np.cumsum(deg)])
    return len(deg), rowptr, rng.integers(0, len(deg), rowptr[-1])


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
@pytest.mark.parametrize("name", ["long130", "long600", "long130many", "hubs", "hubswide", "skewed", "short", "shortmany"])
def test_long_and_short_rows(name, dtype):
    from paper_2305_17469_amd import binding as B
    n, rowptr, col = _graph(name)
    g = B.Graph(torch.from_numpy(rowptr.astype(np.int32)).cuda(), torch.from_numpy(col.astype(np.int32)).cuda(), n)
    deg = torch.from_numpy(np.diff(rowptr)).cuda()
    dst, src = torch.repeat_interleave(torch.arange(n, device="cuda:0"), deg), torch.from_numpy(col).long().cuda()
    gen = torch.Generator(device="cuda:0").manual_seed(n)
    v = 4 if dtype == torch.float32 else 8
    for F in (3 * v, 5 * v + 3, 9 * v, 17 * v + 1, 33 * v):      # groups of 4, 8, 16, 32, 64 lanes
        for padded in (True, False):
            ld = (F + v - 1) // v * v if padded else F
            X = torch.randn((n, ld), device="cuda:0", generator=gen).to(dtype)[:, :F]
            for fn, a, b in ((B.gt_aggregate_fwd, src, dst), (B.gt_aggregate_bwd, dst, src)):
                announce("long rows", name, dtype, F, "padded", padded, fn.__name__)
                got = fn(g, "sum", X).double()
                ref = torch.zeros((n, F), dtype=torch.float64, device="cuda:0").index_add_(0, b, X.double()[a])
                mag = torch.zeros((n, F), dtype=torch.float64, device="cuda:0").index_add_(0, b, X.double().abs()[a])
                cnt = torch.bincount(b, minlength=n).double()[:, None]
                bound = (cnt + 2) * 2.0 ** -24 * mag + (2.0 ** -8 * ref.abs() if dtype == torch.bfloat16 else 0)
                assert bool(((got - ref).abs() <= bound).all()), (name, F, padded, fn.__name__)
                assert torch.equal(got, fn(g, "sum", X).double())


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
@pytest.mark.parametrize("name", ["long130", "long600", "hubsmid"])
def test_column_tiles_of_long_rows(name, dtype):
    """Rows of whole lines in two and three column tiles (pairs share out the XCDs) whose long items are shared out and whose split rows are
    summed whole: plain in both directions, and in a layer that transforms first (by the unit matrix) with bias and ReLU in the epilogue."""
    from paper_2305_17469_amd import binding as B
    n, rowptr, col = _graph(name)
    g = B.Graph(torch.from_numpy(rowptr.astype(np.int32)).cuda(), torch.from_numpy(col.astype(np.int32)).cuda(), n)
    deg = torch.from_numpy(np.diff(rowptr)).cuda()
    dst, src = torch.repeat_interleave(torch.arange(n, device="cuda:0"), deg), torch.from_numpy(col).long().cuda()
    gen = torch.Generator(device="cuda:0").manual_seed(n)
    v, half = (4, 0.0) if dtype == torch.float32 else (8, 2.0 ** -8)

    def sums(X, a, b):
        ref, mag = (torch.zeros_like(X, dtype=torch.float64) for _ in range(2))
        for c in range(0, X.shape[1], 64):
            x = X[:, c:c + 64].double()[a]
            ref[:, c:c + 64].index_add_(0, b, x)
            mag[:, c:c + 64].index_add_(0, b, x.abs())
        return ref, mag, torch.bincount(b, minlength=n).double()[:, None]

    for F in (32 * v, 48 * v):
        X = torch.randn((n, F), device="cuda:0", generator=gen).to(dtype)
        for fn, a, b in ((B.gt_aggregate_fwd, src, dst), (B.gt_aggregate_bwd, dst, src)):
            announce("tiles of long rows", name, dtype, F, fn.__name__)
            ref, mag, cnt = sums(X, a, b)
            got = fn(g, "sum", X)
            assert bool(((got.double() - ref).abs() <= (cnt + 2) * 2.0 ** -24 * mag + half * ref.abs()).all()), (name, F, fn.__name__)
            assert torch.equal(got, fn(g, "sum", X))
        d = B.make_desc("sum", "f32" if dtype == torch.float32 else "bf16", True, F, F)
        bias = torch.randn(F, device="cuda:0", generator=gen)
        announce("tiles of long rows, layer", name, dtype, F)
        Y, used = B.gt_layer_fwd(g, d, X, torch.eye(F, device="cuda:0", dtype=dtype), bias, B.LayerBuffers(g, d), "comb_first")
        assert used == "comb_first"
        ref, mag, cnt = sums(X, src, dst)
        ref = ref + bias.double()
        bound = (cnt + 3) * 2.0 ** -24 * (mag + bias.double().abs()) + half * ref.abs()
        assert bool(((Y.double() - ref.clamp(min=0)).abs() <= bound).all()), (name, F)
