"""Which instance of the aggregation kernel a shape takes (lanes per row, vectors per lane, rows in flight), on both sides of the rules for rows in flight
and column tiles; the results against 64 bits: |error| <= (n + 2) 2^-24 sum |x| for a row of n entries (any order of fp32 additions), one bf16
rounding more for bf16 results."""
import numpy as np
import pytest
import torch

from gpu_util import announce

pytestmark = pytest.mark.gpu

# rows, entries per row, hub rows, their entries: graphs without hubs are uniform, those with hubs skewed
GRAPHS = {"even20k": (20000, 25, 0, 0), "sparse66k": (66000, 4, 0, 0), "even66k": (66000, 16, 0, 0), "even131k": (131072, 25, 0, 0),
          "sparse131k": (131072, 4, 0, 0), "even30k130": (30000, 130, 0, 0), "even1m": (1000003, 8, 0, 0), "few6k600": (6000, 600, 0, 0), "hubs20k": (20000, 22, 40, 1500),
          "hubs33k": (33000, 26, 40, 2500), "hubs262k": (262144, 8, 60, 8000), "hubs2m": (2097152, 11, 300, 9000)}
# columns, stride, type, (lanes, vectors per lane, rows in flight); strides of whole lines of 128 bytes may be cut into tiles of 16 lanes
CASES = [("even131k", 4, 4, "f32", (4, 1, 8)),        # the table fits the L2s
         ("even131k", 16, 16, "f32", (4, 1, 1)),      # past them, several ids per lane
         ("even131k", 32, 32, "f32", (8, 1, 1)),
         ("even131k", 64, 64, "f32", (16, 1, 2)),
         ("even131k", 47, 47, "bf16", (8, 1, 1)),
         ("even20k", 64, 64, "f32", (16, 1, 8)),      # fits the L2s
         ("sparse66k", 64, 64, "f32", (16, 1, 8)),    # few entries per row
         ("hubs262k", 13, 13, "f32", (4, 1, 8)),      # skewed
         ("hubs2m", 13, 16, "f32", (4, 1, 1)),        # past the last-level cache, shared out
         ("even66k", 200, 200, "f32", (64, 1, 1)),    # uniform rows of a wavefront
         ("even66k", 130, 132, "f32", (64, 1, 2)),    # ... little more than half of which they cover
         ("even1m", 200, 200, "f32", (64, 1, 2)),     # ... of a table far beyond the caches
         ("even30k130", 300, 300, "f32", (64, 2, 1)),
         ("even30k130", 602, 602, "bf16", (64, 2, 1)),
         ("sparse66k", 300, 300, "f32", (64, 2, 2)),
         ("sparse66k", 1030, 1032, "f32", (64, 4, 1)),
         ("even66k", 256, 256, "f32", (16, 1, 2)),    # tiles
         ("even131k", 256, 256, "f32", (16, 1, 1)),   # ... of longer rows
         ("few6k600", 301, 301, "f32", (64, 2, 2)),   # few long rows
         ("sparse131k", 256, 256, "f32", (64, 1, 2)),   # few entries per row
         ("sparse131k", 160, 160, "f32", (16, 1, 2)),
         ("hubs20k", 256, 256, "f32", (64, 1, 8)),    # skewed: whole rows with eight in flight
         ("hubs20k", 512, 512, "f32", (16, 1, 2)),    # no chains
         ("hubs33k", 200, 224, "f32", (64, 1, 8)),
         ("hubs262k", 320, 320, "f32", (16, 1, 8)),
         ("hubs262k", 300, 300, "f32", (32, 1, 2)),   # no whole lines, past the last-level cache
         ("hubs262k", 200, 200, "f32", (64, 1, 2))]


def _graph(name):
    n, d, hubs, most = GRAPHS[name]
    rng = np.random.default_rng(n + d)
    deg = np.full(n, d)
    if hubs:
        deg[rng.choice(n, hubs, replace=False)] = rng.integers(most // 2, most, hubs)
    return torch.from_numpy(deg).cuda(), torch.from_numpy(rng.integers(0, n, int(deg.sum()))).cuda()


@pytest.mark.parametrize("name", list(GRAPHS))
def test_instances(name):
    from paper_2305_17469_amd import binding as B
    deg, col = _graph(name)
    n = deg.numel()
    rowptr = torch.zeros(n + 1, dtype=torch.int32, device="cuda:0")
    rowptr[1:] = torch.cumsum(deg, 0)
    g = B.Graph(rowptr, col.int(), n)
    # every 97th row and the longest ones
    rows = torch.unique(torch.cat([torch.arange(0, n, 97, device="cuda:0"), torch.topk(deg, 64).indices]))
    d = deg[rows]
    to = torch.repeat_interleave(torch.arange(rows.numel(), device="cuda:0"), d)
    at = torch.arange(int(d.sum()), device="cuda:0") - torch.repeat_interleave(torch.cumsum(d, 0) - d, d)
    frm = col[torch.repeat_interleave(rowptr[rows].long(), d) + at]
    gen = torch.Generator(device="cuda:0").manual_seed(n)
    for _, F, ld, dt, want in (c for c in CASES if c[0] == name):
        dtype = torch.float32 if dt == "f32" else torch.bfloat16
        X = torch.randn((n, ld), device="cuda:0", generator=gen).to(dtype)[:, :F]
        out = torch.empty((n, ld), device="cuda:0", dtype=dtype)[:, :F]
        announce("instances", name, F, ld, dt)
        B.gt_trace_reset()
        B.gt_trace_enable(True)
        got = B.gt_aggregate_fwd(g, "sum", X, out)
        torch.cuda.synchronize()
        B.gt_trace_enable(False)
        took = [v[1:4] for v in B.gt_trace_variants()]
        B.gt_trace_reset()
        assert took == [want], (name, F, ld, dt, took)
        for c in range(0, F, 64):
            x = X[:, c:c + 64].double()[frm]
            ref, mag = (torch.zeros((rows.numel(), x.shape[1]), dtype=torch.float64, device="cuda:0").index_add_(0, to, t) for t in (x, x.abs()))
            bound = (d[:, None] + 2) * 2.0 ** -24 * mag + (2.0 ** -8 * ref.abs() if dt == "bf16" else 0)
            assert bool(((got[rows][:, c:c + 64].double() - ref).abs() <= bound).all()), (name, F, ld, dt, c)
