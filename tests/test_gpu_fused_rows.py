"""gt_aggregate_combine_fwd where its work on rows changes: rows around the lengths that one group, a whole wavefront or (split)
several chunks sum, entry counts around a 32-row block and on both sides of the counts from which a workgroup has 8 and 16
wavefronts.  Against sums and products in 64 bits: a term passes through at most hub + K + 4 fp32 operations, so
|error| <= (hub + K + 4) 2^-24 (|A| |X| |W| + |b|); bf16: the aggregated row (2^-8 |A X| |W|) and the result (2^-8) rounded too."""
import numpy as np
import pytest
import torch

from gt_inputs import graphs
from gpu_util import announce, up_i32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,hub", [(1, 1), (33, 31), (700, 63), (700, 64), (5000, 65), (5000, 128), (5000, 129), (20000, 3000),
                                   (65535, 127), (65600, 64), (131071, 700), (131200, 200)])
@pytest.mark.parametrize("dtype,fi,fo", [("f32", 16, 64), ("f32", 37, 20), ("bf16", 256, 64), ("bf16", 64, 47), ("bf16", 8, 128)])
def test_rows_at_the_edges(n, hub, dtype, fi, fo):
    from paper_2305_17469_amd import binding as B
    rng = np.random.default_rng(n + hub)
    rows = np.arange(0, n, 3)
    dst = np.concatenate([np.repeat(rows, 5), np.full(hub, n // 2), np.full(hub, n - 1)])
    src = np.concatenate([rng.integers(0, n, 5 * rows.size), rng.choice(n, hub, replace=False), rng.choice(n, hub, replace=False)])
    rp, ci = graphs.csr_from_pairs(src, dst, n, n)
    g = B.Graph(up_i32(rp), up_i32(ci), n)
    gen = torch.Generator(device="cuda:0").manual_seed(n)
    tdt, v = (torch.bfloat16, 8) if dtype == "bf16" else (torch.float32, 4)
    X = torch.randn((n, (fi + v - 1) // v * v), device="cuda:0", generator=gen).to(tdt)[:, :fi]
    W = torch.randn((fi, fo), device="cuda:0", generator=gen).to(tdt)
    b = torch.randn(fo, device="cuda:0", generator=gen)
    deg = up_i32(np.diff(rp)).long()
    at = torch.repeat_interleave(torch.arange(n, device="cuda:0"), deg)
    t = X.double()[up_i32(ci).long()]
    zero = torch.zeros((n, fi), dtype=torch.float64, device="cuda:0")
    AX, mag = zero.index_add(0, at, t), zero.index_add(0, at, t.abs())
    for reduce in ("sum", "mean"):
        announce("fused rows", dtype, fi, fo, "n", n, "hub", hub, reduce)
        d = deg.clamp(min=1)[:, None].double() if reduce == "mean" else 1.0
        ref = (AX / d) @ W.double() + b.double()
        bound = (int(deg.max()) + fi + 4) * 2.0 ** -24 * ((mag / d) @ W.double().abs() + b.double().abs())
        if dtype == "bf16":
            bound += 2.0 ** -8 * ((AX / d).abs() @ W.double().abs() + ref.abs())
        out = torch.full((n, fo), float("nan"), device="cuda:0", dtype=tdt)
        B.gt_aggregate_combine_fwd(g, reduce, X, W, b, False, out=out)
        assert bool(((out.double() - ref).abs() <= bound).all())
        again = torch.empty_like(out)
        B.gt_aggregate_combine_fwd(g, reduce, X, W, b, False, out=again)
        assert torch.equal(out, again)


@pytest.mark.parametrize("hubs", [0, 512, 513, 2000])
def test_inference_layer_on_both_sides_of_the_rule(hubs):
    """Forward-only aggregation-first layer on a 32 MiB table of 64-byte rows: one kernel up to one long row in 1,024, two
    beyond.  Bound as above."""
    from paper_2305_17469_amd import binding as B
    n, fi, fo = 524288, 16, 24
    rng = np.random.default_rng(hubs)
    dst = np.concatenate([np.repeat(np.arange(0, n, 2), 2), np.repeat(np.arange(hubs) * 200 + 1, 90)])
    rp, ci = graphs.csr_from_pairs(rng.integers(0, n, dst.size), dst, n, n)
    g = B.Graph(up_i32(rp), up_i32(ci), n)
    gen = torch.Generator(device="cuda:0").manual_seed(hubs)
    X, W = torch.randn((n, fi), device="cuda:0", generator=gen), torch.randn((fi, fo), device="cuda:0", generator=gen)
    b = torch.randn(fo, device="cuda:0", generator=gen)
    d = B.make_desc("mean", "f32", False, fi, fo, need_dx=False, dy_is_dz=True)
    announce("inference layer, hubs", hubs)
    Y, used = B.gt_layer_fwd(g, d, X, W, b, B.LayerBuffers(g, d), "agg_first", inference=True)
    deg = up_i32(np.diff(rp)).long()
    at = torch.repeat_interleave(torch.arange(n, device="cuda:0"), deg)
    t = X.double()[up_i32(ci).long()]
    zero = torch.zeros((n, fi), dtype=torch.float64, device="cuda:0")
    div = deg.clamp(min=1)[:, None].double()
    ref = zero.index_add(0, at, t) / div @ W.double() + b.double()
    mag = zero.index_add(0, at, t.abs()) / div @ W.double().abs() + b.double().abs()
    assert used == "agg_first" and bool(((Y.double() - ref).abs() <= (int(deg.max()) + fi + 4) * 2.0 ** -24 * mag).all())
