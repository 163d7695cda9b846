"""Both derivatives of the scaled aggregation from one gather over the transposed structure: every lane-group size, sources with no, few and thousands of
out-edges (whole rows, chunks, long items shared out), uniform graphs, padded rows (NaN in the padding) and contiguous ones of every width class, sum and mean, and the
sizes on both sides of the rule.  Against 64 bits: |error| <= (n + 2) 2^-24 sum |terms| over the n terms of a sum, one bf16 rounding of dXs; dW overwriting W
gives the same bits."""
import numpy as np
import pytest
import torch

from gpu_util import announce

pytestmark = pytest.mark.gpu


def _graph(kind):
    rng = np.random.default_rng(5)
    if kind == "hubs":      # few sources hold most edges: chunks and partial rows in the transposed schedule
        n, E = 6000, 90_000
        p = 1.0 / (np.arange(n) + 1.0)
        src = rng.choice(n, E, p=p / p.sum())
    elif kind == "large":   # enough edges that long items are not shared out
        n, E = 60_000, 5_000_000
        p = 1.0 / (np.arange(n) + 30.0)
        src = rng.choice(n, E, p=p / p.sum())
    elif kind == "many":    # uniform, more edges than the L2s hold scores of
        n, E = 60_000, 1_700_000
        src = rng.integers(0, n, E)
    else:
        n, E = 5003, 60_000
        src = rng.integers(0, n, E)
    dst = np.sort(rng.integers(0, n - 3, E))
    return n, torch.from_numpy(src).cuda(), torch.from_numpy(dst).cuda()


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
@pytest.mark.parametrize("kind,F", [("hubs", F) for F in (3, 16, 17, 31, 64, 65, 101, 128, 160, 256, 257, 512)] + [("even", F) for F in (8, 23, 47, 64, 100, 140, 250, 300)] +
                         [("large", F) for F in (8, 32, 33, 64, 100)] + [("many", F) for F in (8, 20, 47, 64)])
def test_derivatives(kind, F, dtype):
    from paper_2305_17469_amd import binding as B
    n, src, dst = _graph(kind)
    deg = torch.bincount(dst, minlength=n)
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda:0")
    rowptr[1:] = torch.cumsum(deg, 0)
    g = B.Graph(rowptr.int(), src.int(), n)
    gen = torch.Generator(device="cuda:0").manual_seed(F)
    W = torch.randn(src.numel(), device="cuda:0", generator=gen)
    v = 4 if dtype == torch.float32 else 8
    for reduce in ("sum", "mean"):
        for ld in (F, (F + v - 1) // v * v + v):
            announce("scale derivatives", kind, F, dtype, reduce, ld)

            def rows():
                t = torch.full((n, ld), float("nan"), device="cuda:0", dtype=dtype)
                t[:, :F] = torch.randn((n, F), device="cuda:0", generator=gen).to(dtype)
                return t[:, :F]

            dY, Xs = rows(), rows()
            out = torch.full((n, ld), 3.0, device="cuda:0", dtype=dtype)
            W2 = W.clone()
            dXs, dW = B.gt_pull_bwd(g, reduce, "scale", dY, Xs, W, out_dXs=out[:, :F])
            assert bool((out[:, F:] == 3).all())
            _, same = B.gt_pull_bwd(g, reduce, "scale", dY, Xs, W2, out_dW=W2)
            assert torch.equal(same, dW)
            f = (1.0 / deg.double()[dst] if reduce == "mean" else torch.ones_like(W, dtype=torch.float64))[:, None]
            ref = torch.zeros((n, F), dtype=torch.float64, device="cuda:0")
            mag = torch.zeros_like(ref)
            for i in range(0, src.numel(), 500_000):
                s, d, c = src[i:i + 500_000], dst[i:i + 500_000], f[i:i + 500_000]
                t = dY.double()[d] * c
                p = t * Xs.double()[s]
                assert bool(((dW[i:i + 500_000].double() - p.sum(1)).abs() <= (F + 4) * 2.0 ** -24 * p.abs().sum(1)).all())
                t = t * W.double()[i:i + 500_000, None]
                ref.index_add_(0, s, t)
                mag.index_add_(0, s, t.abs())
            terms = torch.bincount(src, minlength=n).double()[:, None]
            bound = (terms + 4) * 2.0 ** -24 * mag + (2.0 ** -8 * ref.abs() if dtype == torch.bfloat16 else 0)
            assert bool(((dXs.double() - ref).abs() <= bound + 1e-30).all())
