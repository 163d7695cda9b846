"""The aggregation of rows cut into column tiles, on both sides of the rules for it: uniform and skewed graphs, one table small enough for tiles
to share out the XCDs and one beyond, launches below and above the sizes at which items are shared out; full and ragged last tiles,
one, two, three and ten tiles, rows that begin at lines and rows that do not.  Both types and directions, against 64 bits:
|error| <= (n + 2) 2^-24 sum |x| for a row of n entries (any order of fp32 additions), one bf16 rounding more for bf16 results."""
import numpy as np
import pytest
import torch

from gpu_util import announce

pytestmark = pytest.mark.gpu


def _degrees(name):
    rng = np.random.default_rng(len(name))
    n, lo, hi, hubs, most = {"uniform": (3001, 0, 17, 0, 0), "uniformlarge": (70001, 5, 17, 0, 0), "skewed": (60001, 5, 20, 30, 12000),
                             "skewedlong": (150001, 16, 35, 110, 40000), "skewedtable": (1250003, 2, 5, 40, 12000)}[name]
    deg = rng.integers(lo, hi, n)
    if hubs:
        deg[rng.choice(n, hubs, replace=False)] = rng.integers(most // 2, most, hubs)
    return deg, rng


# fp32 columns and row stride (bf16: twice as many); the stride is a multiple of a line's 32 floats except in the last rows
SHAPES = {"uniform": [(128, 128), (120, 128), (192, 192), (602, 608), (150, 152)], "uniformlarge": [(128, 128), (250, 256)],
          "skewed": [(128, 128), (113, 128), (160, 160), (250, 256), (602, 608), (602, 604)], "skewedlong": [(128, 128)],
          "skewedtable": [(128, 128), (260, 260)]}


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
@pytest.mark.parametrize("name", list(SHAPES))
def test_column_tiles(name, dtype):
    from paper_2305_17469_amd import binding as B
    deg, rng = _degrees(name)
    n, E = len(deg), int(deg.sum())
    col = torch.from_numpy(rng.integers(0, n, E)).cuda()
    rowptr = torch.from_numpy(np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)).cuda()
    g = B.Graph(rowptr, col.int(), n)
    dst = torch.repeat_interleave(torch.arange(n, device="cuda:0"), torch.from_numpy(deg).cuda())
    gen = torch.Generator(device="cuda:0").manual_seed(n)
    k = 1 if dtype == torch.float32 else 2
    for F, ld in SHAPES[name]:
        if F > 300 and k == 2:
            continue
        F, ld = F * k - (k - 1) * (F % 2), ld * k
        X = torch.randn((n, ld), device="cuda:0", generator=gen).to(dtype)[:, :F]
        out = torch.full((n, ld), 7.0, device="cuda:0", dtype=dtype)[:, :F]
        for fn, a, b in ((B.gt_aggregate_fwd, col, dst), (B.gt_aggregate_bwd, dst, col)):
            announce("column tiles", name, dtype, F, ld, fn.__name__)
            got = fn(g, "sum", X, out)
            cnt = torch.bincount(b, minlength=n).double()[:, None]
            for c in range(0, F, 64):   # (64 columns at a time: a term of every edge is held in 64 bits)
                x = X[:, c:c + 64].double()[a]
                ref = torch.zeros((n, x.shape[1]), dtype=torch.float64, device="cuda:0").index_add_(0, b, x)
                mag = torch.zeros_like(ref).index_add_(0, b, x.abs_())
                bound = (cnt + 2) * 2.0 ** -24 * mag + (2.0 ** -8 * ref.abs() if dtype == torch.bfloat16 else 0)
                assert bool(((got[:, c:c + 64].double() - ref).abs() <= bound).all()), (name, F, ld, c, fn.__name__)
            again = got.clone()
            assert torch.equal(again, fn(g, "sum", X, out))
            assert bool((out.as_strided((n, ld), (ld, 1))[:, F:] == 7).all())
