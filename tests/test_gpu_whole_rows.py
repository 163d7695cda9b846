"""Split rows of small graphs, summed by a workgroup each or in chunks: longest rows on both sides of the limit of 64 entries per lane group, for every
group size, alone and among short rows, with mean, symmetric norm and plain sums, both directions, padded and contiguous rows, against
64 bits: |error| <= (n + 4) 2^-24 sum |terms| for a row of n entries, one bf16 rounding more for bf16 results."""
import numpy as np
import pytest
import torch

from gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
@pytest.mark.parametrize("longest", [97, 255, 256, 257, 512, 513, 1024, 1025, 2048, 2049, 4096, 4097])
def test_split_rows(longest, dtype):
    from paper_2305_17469_amd import binding as B
    rng = np.random.default_rng(longest)
    n = 5000
    deg = rng.integers(0, 9, n)
    deg[rng.choice(n, 7, replace=False)] = [longest, longest, 97, 98, 130, max(97, longest - 1), max(97, longest // 2)]
    rowptr = np.concatenate([[0], np.cumsum(deg)])
    dst = torch.repeat_interleave(torch.arange(n, device="cuda:0"), torch.from_numpy(deg).cuda())
    src = torch.from_numpy(rng.integers(0, n, rowptr[-1])).cuda()
    rp, ci = torch.from_numpy(rowptr.astype(np.int32)).cuda(), src.int()
    rt = torch.zeros(n + 1, dtype=torch.int64, device="cuda:0")
    rt[1:] = torch.cumsum(torch.bincount(src, minlength=n), 0)
    order = torch.sort(src, stable=True).indices
    gen = torch.Generator(device="cuda:0").manual_seed(longest)
    v = 4 if dtype == torch.float32 else 8
    din = torch.from_numpy(deg).cuda().double()
    inv = torch.where(din > 0, din.clamp(min=1).rsqrt(), torch.zeros_like(din))
    # the graph and its transpose: long rows in either direction
    for g, to, frm, d_in in ((B.Graph(rp, ci, n), dst, src, din), (B.Graph(rt.int(), dst[order].int(), n), src, dst, None)):
        for F in (3 * v, 8 * v, 12 * v, 16 * v - 3, 30 * v, 50 * v):
            for padded in (True, False):
                ld = (F + v - 1) // v * v if padded else F
                X = torch.randn((n, ld), device="cuda:0", generator=gen).to(dtype)[:, :F]
                for reduce in ("sum", "mean", "symnorm") if d_in is not None and padded else ("sum",):
                    announce("whole rows", longest, dtype, F, padded, reduce)
                    for fn, a, b in ((B.gt_aggregate_fwd, frm, to), (B.gt_aggregate_bwd, to, frm)):
                        c = 1.0 if reduce == "sum" else (1.0 / d_in.clamp(min=1))[to][:, None] if reduce == "mean" else (inv[to] * inv[frm])[:, None]
                        got, t = fn(g, reduce, X).double(), X.double()[a] * c
                        ref, mag = (torch.zeros((n, F), dtype=torch.float64, device="cuda:0").index_add_(0, b, x) for x in (t, t.abs()))
                        cnt = torch.bincount(b, minlength=n).double()[:, None]
                        bound = (cnt + 4) * 2.0 ** -24 * mag + (2.0 ** -8 * ref.abs() if dtype == torch.bfloat16 else 0)
                        assert bool(((got - ref).abs() <= bound).all()), (longest, F, padded, reduce, fn.__name__)
                        assert torch.equal(got, fn(g, reduce, X).double())
