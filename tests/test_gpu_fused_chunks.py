"""The fused layer on power-law graphs whose table is past the line from which the chunks of its long rows are shared out by their own bytes, and just below it:
against 64 bits, |error| <= 2e-2 (bf16: A X and the result rounded) or 1e-5 (fp32) of sum |terms|, all rows, twice the same bits."""
import numpy as np
import pytest
import torch

from gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,fi,fo,dt", [(300_001, 128, 64, "bf16"), (290_000, 128, 64, "bf16"), (600_007, 57, 20, "bf16"), (300_003, 64, 70, "f32"), (300_003, 66, 33, "f32")])
def test_chunks(n, fi, fo, dt):
    from paper_2305_17469_amd import binding as B
    rng = np.random.default_rng(n)
    long = rng.choice(n, 300, replace=False)
    deg = rng.integers(0, 8, n)
    deg[long] = rng.integers(500, 6000, 300)      # chunks of 512 and their remainders
    rowptr = torch.from_numpy(np.concatenate([[0], np.cumsum(deg)])).cuda()
    src = torch.from_numpy(rng.integers(0, n, int(rowptr[-1]))).cuda()
    dst = torch.repeat_interleave(torch.arange(n, device="cuda:0"), rowptr[1:] - rowptr[:-1])
    g = B.Graph(rowptr.int(), src.int(), n)
    gen = torch.Generator(device="cuda:0").manual_seed(n)
    dtype = torch.bfloat16 if dt == "bf16" else torch.float32
    v = 16 // (2 if dt == "bf16" else 4)
    X = torch.randn((n, (fi + v - 1) // v * v), device="cuda:0", generator=gen).to(dtype)[:, :fi]
    W = (torch.randn((fi, fo), device="cuda:0", generator=gen) * fi ** -0.5).to(dtype)
    announce("fused chunks", n, fi, fo, dt)
    Y = B.gt_aggregate_combine_fwd(g, "mean", X, W)
    assert torch.equal(Y, B.gt_aggregate_combine_fwd(g, "mean", X, W))
    M, mag = (torch.zeros((n, fi), dtype=torch.float64, device="cuda:0") for _ in range(2))
    for i in range(0, src.numel(), 1_000_000):
        t = X.double()[src[i:i + 1_000_000]]
        M.index_add_(0, dst[i:i + 1_000_000], t)
        mag.index_add_(0, dst[i:i + 1_000_000], t.abs())
    inv = 1.0 / torch.from_numpy(deg).cuda().clamp(min=1).double()[:, None]
    bound = (2e-2 if dt == "bf16" else 1e-5) * (mag * inv) @ W.double().abs()
    assert bool(((Y.double() - (M * inv) @ W.double()).abs() <= bound + 1e-30).all())
