"""Tables of narrow rows that a uniform graph gathers from a copy at whole-line strides (64 or 128 bytes), where the workspace has room for it: widths at
both ends of each stride, contiguous, padded and offset rows, aligned and unaligned results, both directions.  Bit for bit what the same call gives
without that room (every row is summed in the order of its entries), and against 64 bits: |error| <= (deg + 2) 2^-24 sum |terms| + 2^-8 |result| in bf16.  Memory
around the result and the workspace's last bytes stay.  Layers whose own tables have such strides, both orders."""
import ctypes

import pytest
import torch

from gpu_util import announce

pytestmark = pytest.mark.gpu
N = 450_001


@pytest.fixture(scope="module")
def graph():
    from paper_2305_17469_amd import binding as B
    gen = torch.Generator(device="cuda:0").manual_seed(3)
    deg = torch.randint(10, 40, (N,), device="cuda:0", generator=gen)
    deg[::97] = 0
    rowptr = torch.zeros(N + 1, dtype=torch.int64, device="cuda:0")
    rowptr[1:] = torch.cumsum(deg, 0)
    col = torch.randint(0, N, (int(rowptr[-1]),), device="cuda:0", generator=gen)
    rows = torch.repeat_interleave(torch.arange(N, device="cuda:0"), deg)
    return B.Graph(rowptr.int(), col.int(), N), rows, col, deg


def _table(F, dtype, ld, off, gen):
    buf = torch.full((off + N * ld + 8,), float("nan"), dtype=dtype, device="cuda:0")
    t = buf[off:off + N * ld].view(N, ld)[:, :F]
    return t.copy_(torch.randn((N, F), device="cuda:0", generator=gen))


@pytest.mark.parametrize("F,dt,ld,off", [(33, "bf16", 33, 0), (47, "bf16", 47, 0), (47, "bf16", 48, 0), (47, "bf16", 47, 5), (63, "bf16", 63, 0), (64, "bf16", 64, 8), (64, "bf16", 65, 1),
                                         (31, "bf16", 31, 0), (32, "bf16", 33, 0), (17, "f32", 17, 0), (31, "f32", 31, 3), (32, "f32", 36, 0), (15, "f32", 15, 0), (21, "f32", 24, 0)])
@pytest.mark.parametrize("reduce", ["mean", "symnorm"])
def test_same_as_in_place(graph, F, dt, ld, off, reduce):
    from paper_2305_17469_amd import binding as B
    g, rows, col, deg = graph
    dtype = torch.bfloat16 if dt == "bf16" else torch.float32
    gen = torch.Generator(device="cuda:0").manual_seed(F)
    X = _table(F, dtype, ld, off, gen)
    need = ctypes.c_size_t()
    assert B.lib.gt_aggregate_ws_size(g.handle, F, ctypes.byref(need)) == 0
    assert need.value >= N * 64          # room for the copy (this graph splits no row)
    for transposed in (False, True):
        for ldy in (F, (F + 7) // 8 * 8):
            outs = []
            for room in (need.value, 256):
                announce("repacked rows", F, dt, ld, off, reduce, transposed, ldy, room)
                ws = torch.full((need.value + 64,), 7, dtype=torch.uint8, device="cuda:0")
                buf = torch.full((N * ldy + 8,), 3.0, dtype=dtype, device="cuda:0")
                Y = buf[:N * ldy].view(N, ldy)
                call = B.lib.gt_aggregate_bwd if transposed else B.lib.gt_aggregate_fwd
                assert call(g.handle, B.REDUCE[reduce], 1 if dt == "bf16" else 0, F, X.data_ptr(), ld, Y.data_ptr(), ldy, ws.data_ptr(), room, None) == 0
                torch.cuda.synchronize()
                assert bool((Y[:, F:] == 3).all()) and bool((buf[N * ldy:] == 3).all()) and bool((ws[room:] == 7).all())
                outs.append(Y[:, :F].clone())
            assert torch.equal(outs[0], outs[1])
    if off == 0:
        inv = torch.where(deg > 0, deg.double().rsqrt(), torch.zeros_like(deg, dtype=torch.float64))
        cf = (inv[rows] * inv[col] if reduce == "symnorm" else 1.0 / deg.double()[rows])[:, None]   # of the backward direction, run last
        ref = torch.zeros((N, F), dtype=torch.float64, device="cuda:0")
        mag = torch.zeros_like(ref)
        for i in range(0, rows.numel(), 2_000_000):
            t = X[rows[i:i + 2_000_000]].double() * cf[i:i + 2_000_000]
            ref.index_add_(0, col[i:i + 2_000_000], t)
            mag.index_add_(0, col[i:i + 2_000_000], t.abs())
        n_in = torch.bincount(col, minlength=N).double()[:, None]
        bound = (n_in + 4) * 2.0 ** -24 * mag + (2.0 ** -8 * ref.abs() if dt == "bf16" else 0)
        assert bool(((outs[0].double() - ref).abs() <= bound + 1e-30).all())


@pytest.mark.parametrize("dt,fi,fo", [("bf16", 60, 47), ("f32", 70, 41), ("bf16", 101, 130)])
def test_layers(graph, dt, fi, fo):
    from paper_2305_17469_amd import binding as B
    g = graph[0]
    dtype = torch.bfloat16 if dt == "bf16" else torch.float32
    gen = torch.Generator(device="cuda:0").manual_seed(fi)
    X, dY = torch.randn((N, fi), device="cuda:0", generator=gen).to(dtype), torch.randn((N, fo), device="cuda:0", generator=gen).to(dtype)
    W = (torch.randn((fi, fo), device="cuda:0", generator=gen) * fi ** -0.5).to(dtype)
    b = torch.randn(fo, device="cuda:0", generator=gen)
    desc = B.make_desc("mean", dt, True, fi, fo)
    got = {}
    for order in ("agg_first", "comb_first"):
        announce("repacked rows, layer", dt, fi, fo, order)
        bufs = B.LayerBuffers(g, desc)
        Y, used = B.gt_layer_fwd(g, desc, X, W, b, bufs, order)
        r = B.gt_layer_bwd(g, desc, used, dY, X, W, Y, bufs, order)
        got[order] = (Y, r["dX"], r["dW"], r["db"])
    # the two orders round in different places: compared with one another in the 2-norm
    for x, y in zip(got["agg_first"], got["comb_first"]):
        x, y = x.double(), y.double()
        assert float((x - y).norm()) <= (2e-2 if dt == "bf16" else 2e-5) * float(y.norm())
