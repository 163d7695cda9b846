"""Gathers whose coefficients are found through the permutation (source-side derivatives of dot scores and of the scaled aggregation) ask for the places
a batch ahead: rows that end just before, at and after one, two and three batches of every lane-group size, hubs cut into chunks or shared out, a graph without edges.
Against 64 bits: |error| <= (n + 4) 2^-24 sum |terms| over the n terms of a sum, one bf16 rounding."""
import pytest
import torch

from gpu_util import announce

pytestmark = pytest.mark.gpu

DEGREES = [0, 1, 3, 4, 5, 8, 9, 12, 13, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 127, 128, 129, 191, 192, 193]


def _graph(kind):
    """Sources with out-degrees around multiples of the batch sizes; "hubs": a few of thousands besides; "many": enough of them to fill the chip."""
    gen = torch.Generator(device="cuda:0").manual_seed(9)
    out = DEGREES * (400 if kind == "many" else 3) + ([700, 9000] if kind == "hubs" else [])
    n = len(out)
    src = torch.repeat_interleave(torch.arange(n, device="cuda:0"), torch.tensor(out, device="cuda:0"))
    src = src[torch.randperm(src.numel(), device="cuda:0", generator=gen)]
    dst = torch.sort(torch.randint(0, n, (src.numel(),), device="cuda:0", generator=gen)).values
    return n, src, dst


def _rowptr(dst, n):
    p = torch.zeros(n + 1, dtype=torch.int64, device="cuda:0")
    p[1:] = torch.cumsum(torch.bincount(dst, minlength=n), 0)
    return p.int()


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
@pytest.mark.parametrize("kind,F", [(k, F) for k in ("even", "hubs") for F in (3, 8, 13, 16, 23, 41, 64, 130, 300, 1030)] + [("many", F) for F in (13, 64)])
def test_source_side(kind, F, dtype):
    from paper_2305_17469_amd import binding as B
    n, src, dst = _graph(kind)
    g = B.Graph(_rowptr(dst, n), src.int(), n)
    gen = torch.Generator(device="cuda:0").manual_seed(F)
    W = torch.randn(src.numel(), device="cuda:0", generator=gen)
    v = 4 if dtype == torch.float32 else 8
    terms = torch.bincount(src, minlength=n).double()[:, None]
    indeg = torch.bincount(dst, minlength=n).double()
    for ld in (F, (F + v - 1) // v * v + v):
        announce("score lookup", kind, F, dtype, ld)

        def rows():
            t = torch.full((n, ld), float("nan"), device="cuda:0", dtype=dtype)
            t[:, :F] = torch.randn((n, F), device="cuda:0", generator=gen).to(dtype)
            return t[:, :F]

        Xs, Xd = rows(), rows()
        got = dict(dot=B.gt_neighbor_apply_bwd(g, "dot", W, Xs, Xd)[0], sum=B.gt_pull_bwd(g, "sum", "scale", Xd, Xs, W)[0],
                   mean=B.gt_pull_bwd(g, "mean", "scale", Xd, Xs, W)[0])
        for name, y in got.items():
            f = W.double() / (indeg[dst] if name == "mean" else 1.0)
            ref = torch.zeros((n, F), dtype=torch.float64, device="cuda:0")
            mag = torch.zeros_like(ref)
            for i in range(0, src.numel(), 100_000):
                t = Xd.double()[dst[i:i + 100_000]] * f[i:i + 100_000, None]
                ref.index_add_(0, src[i:i + 100_000], t)
                mag.index_add_(0, src[i:i + 100_000], t.abs())
            bound = (terms + 4) * 2.0 ** -24 * mag + (2.0 ** -8 * ref.abs() if dtype == torch.bfloat16 else 0)
            assert bool(((y.double() - ref).abs() <= bound + 1e-30).all()), name


def test_no_edges():
    from paper_2305_17469_amd import binding as B
    g = B.Graph(torch.zeros(8, dtype=torch.int32, device="cuda:0"), torch.empty(0, dtype=torch.int32, device="cuda:0"), 7)
    X, W = torch.ones((7, 12), device="cuda:0"), torch.empty(0, device="cuda:0")
    for y in (*B.gt_neighbor_apply_bwd(g, "dot", W, X, X), B.gt_pull_bwd(g, "sum", "scale", X, X, W)[0], B.gt_pull_bwd(g, "mean", "scale", X, X, W)[0]):
        assert y.shape == (7, 12) and not bool(y.any())
