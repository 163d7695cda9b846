"""Edge products of long items, which are cut into parts: rows of lengths around the parts', the batches' and the chunks' ends in a graph
whose other rows are short, for every lane-group size and a width past one column tile; operands whose row padding holds NaN, which no
result may show.  Against 64 bits: |error| <= (F + 2) 2^-24 sum |terms| (any order of fp32 additions), products one rounding."""
import numpy as np
import pytest
import torch

from gpu_util import announce

pytestmark = pytest.mark.gpu
LENGTHS = [32, 33, 63, 64, 65, 95, 96, 97, 127, 128, 129, 191, 192, 193, 255, 256, 257, 511, 512, 513, 767, 768, 769, 1025]


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
@pytest.mark.parametrize("F", [3, 14, 23, 60, 101, 250, 1100])
def test_parts(F, dtype):
    from paper_2305_17469_amd import binding as B
    rng = np.random.default_rng(F)
    deg = rng.integers(0, 6, 6000)
    deg[rng.choice(6000, len(LENGTHS), replace=False)] = LENGTHS
    rowptr = np.concatenate([[0], np.cumsum(deg)])
    n = len(deg)
    src = torch.from_numpy(rng.integers(0, n, rowptr[-1])).cuda()
    g = B.Graph(torch.from_numpy(rowptr.astype(np.int32)).cuda(), src.int(), n)
    dst = torch.repeat_interleave(torch.arange(n, device="cuda:0"), torch.from_numpy(deg).cuda())
    gen = torch.Generator(device="cuda:0").manual_seed(F)
    v = 4 if dtype == torch.float32 else 8
    ld = (F + v - 1) // v * v + v

    def rows():
        t = torch.full((n, ld), float("nan"), device="cuda:0", dtype=dtype)
        t[:, :F] = torch.randn((n, F), device="cuda:0", generator=gen).to(dtype)
        return t[:, :F]

    Xs, Xd = rows(), rows()
    p = Xs.double()[src] * Xd.double()[dst]
    announce("edge parts", F, dtype)
    w = B.gt_neighbor_apply_fwd(g, "dot", Xs, Xd)
    assert bool(((w.double() - p.sum(1)).abs() <= (F + 2) * 2.0 ** -24 * p.abs().sum(1)).all())
    m = B.gt_neighbor_apply_fwd(g, "mul", Xs, Xd)
    assert bool(((m.double() - p).abs() <= (2.0 ** -8 if dtype == torch.bfloat16 else 2.0 ** -23) * p.abs() + 1e-38).all())
    _, dw = B.gt_pull_bwd(g, "sum", "scale", Xd, Xs, w)
    assert torch.equal(dw, w)   # the same products in the same order
    _, dw = B.gt_pull_bwd(g, "sum", "add", Xd, Xs, m)
    assert torch.equal(dw, Xd[dst])


@pytest.mark.parametrize("dtype,F,mib", [(torch.float32, 64, 96), (torch.float32, 64, 224), (torch.float32, 60, 224), (torch.float32, 116, 320),
                                         (torch.bfloat16, 128, 96), (torch.bfloat16, 128, 224), (torch.bfloat16, 72, 224), (torch.bfloat16, 520, 320)], ids=str)
def test_streamed_edge_tensor(dtype, F, mib):
    """Edge tensors just below and above a line of the rule for streaming: rows of whole lines are read past the caches from 96 MiB on and
    written past them from 224, others from 224 and, if long, 320.  The same edges give the same results bit for bit, and all are within (n + 2) 2^-24 sum |terms| and one bf16 rounding of 64 bits."""
    from paper_2305_17469_amd import binding as B
    es = 4 if dtype == torch.float32 else 2
    n, E = 5000, (mib << 20) // (F * es) + 1000
    rng = np.random.default_rng(F)
    dst = torch.from_numpy(np.sort(rng.integers(0, n, E))).cuda()
    src = torch.from_numpy(rng.integers(0, n, E)).cuda()
    gen = torch.Generator(device="cuda:0").manual_seed(F)
    Xs, Xd, dY = (torch.randn((n, F), device="cuda:0", generator=gen).to(dtype) for _ in range(3))

    def graph(m):
        rowptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda:0")
        rowptr[1:] = torch.cumsum(torch.bincount(dst[:m], minlength=n), 0)
        return B.Graph(rowptr.int(), src[:m].int(), n)

    big, less = graph(E), graph(E - 2000)
    announce("streamed", dtype, F, mib, E)
    r = 2.0 ** -8 if dtype == torch.bfloat16 else 0.0
    m = B.gt_neighbor_apply_fwd(big, "mul", Xs, Xd)
    p = Xs.double()[src] * Xd.double()[dst]
    assert bool(((m.double() - p).abs() <= (r or 2.0 ** -23) * p.abs() + 1e-38).all())
    assert torch.equal(m[:E - 2000], B.gt_neighbor_apply_fwd(less, "mul", Xs, Xd))
    cnt = torch.bincount(dst, minlength=n).double()[:, None]
    kept = dst[E - 2000]   # rows before this one are the same in both graphs
    for h in ("add", "mul"):
        y = B.gt_pull_fwd(big, "sum", h, Xs, m)
        t = Xs.double()[src] + m.double() if h == "add" else Xs.double()[src] * m.double()
        ref, mag = (torch.zeros((n, F), dtype=torch.float64, device="cuda:0").index_add_(0, dst, x) for x in (t, t.abs()))
        assert bool(((y.double() - ref).abs() <= (cnt + 2) * 2.0 ** -23 * mag + r * ref.abs()).all()), h
        assert torch.equal(y[:kept], B.gt_pull_fwd(less, "sum", h, Xs, m[:E - 2000].contiguous())[:kept])
    _, dw = B.gt_pull_bwd(big, "sum", "add", dY, Xs, m)
    assert torch.equal(dw, dY[dst])
