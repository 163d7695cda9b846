"""Tables of narrow rows that a uniform graph gathers from a copy at whole-line strides (64 or 128 bytes), where the workspace has room for it: widths at
both ends of each stride, contiguous, padded and offset rows, aligned and unaligned results, both directions; and tables that are not copied: of one line per
row, of more than 128 bytes, of at most 32.  The copy is in the workspace afterwards, or the workspace as it was.  Bit for bit what the same call gives
without that room (every row is summed in the order of its entries), and against 64 bits: |error| <= (deg + 2) 2^-24 sum |terms| + 2^-8 |result| in bf16.  Memory
around the result and the workspace's last bytes stay.  Layers whose own tables have such strides, both orders, against 64 bits."""
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


@pytest.mark.parametrize("F,dt,ld,off", [(33, "bf16", 33, 0), (47, "bf16", 47, 0), (47, "bf16", 48, 0), (47, "bf16", 47, 5), (63, "bf16", 63, 0), (64, "bf16", 64, 8), (64, "bf16", 65, 1), (47, "bf16", 64, 20),
                                         (31, "bf16", 31, 0), (32, "bf16", 33, 0), (17, "f32", 17, 0), (31, "f32", 31, 3), (32, "f32", 36, 0), (15, "f32", 15, 0), (21, "f32", 24, 0),
                                         (47, "bf16", 64, 0), (33, "f32", 33, 0), (16, "bf16", 19, 3)])
@pytest.mark.parametrize("reduce", ["mean", "symnorm"])
def test_same_as_in_place(graph, F, dt, ld, off, reduce):
    from paper_2305_17469_amd import binding as B
    g, rows, col, deg = graph
    dtype = torch.bfloat16 if dt == "bf16" else torch.float32
    gen = torch.Generator(device="cuda:0").manual_seed(F)
    X = _table(F, dtype, ld, off, gen)
    rb, need = F * X.element_size(), ctypes.c_size_t()
    stride = 0 if rb <= 32 or rb > 128 or (ld, off) == (64, 0) else 64 if rb <= 64 else 128
    for transposed in (False, True):
        assert B.lib.gt_aggregate_best_ws_size(g.handle, int(transposed), B._dtype(X), F, X.data_ptr(), ld, ctypes.byref(need)) == 0
        assert need.value == N * stride          # (this graph splits no row)
        for ldy in (F, (F + 7) // 8 * 8):
            outs = []
            for room in (max(need.value, 256), 256):
                announce("repacked rows", F, dt, ld, off, reduce, transposed, ldy, room)
                ws = torch.full((max(need.value, 256) + 64,), 7, dtype=torch.uint8, device="cuda:0")
                buf = torch.full((N * ldy + 8,), 3.0, dtype=dtype, device="cuda:0")
                Y = buf[:N * ldy].view(N, ldy)
                call = B.lib.gt_aggregate_bwd if transposed else B.lib.gt_aggregate_fwd
                assert call(g.handle, B.REDUCE[reduce], 1 if dt == "bf16" else 0, F, X.data_ptr(), ld, Y.data_ptr(), ldy, ws.data_ptr(), room, None) == 0
                torch.cuda.synchronize()
                assert bool((Y[:, F:] == 3).all()) and bool((buf[N * ldy:] == 3).all()) and bool((ws[room:] == 7).all())
                if stride and room > 256:
                    assert torch.equal(ws[:N * stride].view(N, stride)[:, :rb], X.contiguous().view(torch.uint8))
                else:
                    assert bool((ws == 7).all())
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
    _, rows, col, deg = graph
    coef = 1.0 / deg.clamp(min=1).double()[:, None]

    def gather(T, to, at, scale):
        out = torch.zeros((N, T.shape[1]), dtype=torch.float64, device="cuda:0")
        for i in range(0, rows.numel(), 1_000_000):
            out.index_add_(0, to[i:i + 1_000_000], T[at[i:i + 1_000_000]] * (scale[i:i + 1_000_000] if scale is not None else 1.0))
        return out

    M = gather(X.double(), rows, col, None) * coef
    Z = M @ W.double() + b.double()
    # Every path rounds twice to the working type (an intermediate table and the result, 2^-9 of each value in bf16), so the 2-norm is off by less
    # than 2^-8; fp32: sums of up to 40 x 101 terms, and of 450,001 in splits of a few thousand for dW and db.
    tol = 2.0 ** -8 if dt == "bf16" else 1e-5
    for order in ("agg_first", "comb_first"):
        announce("repacked rows, layer", dt, fi, fo, order)
        bufs = B.LayerBuffers(g, desc)
        Y, used = B.gt_layer_fwd(g, desc, X, W, b, bufs, order)
        r = B.gt_layer_bwd(g, desc, used, dY, X, W, Y, bufs, order)
        dZ = dY.double() * (Y > 0)          # (the activation as it was taken)
        dX = gather(dZ @ W.double().T, col, rows, coef[rows])
        for name, got, ref in (("Y", Y, Z.clamp(min=0)), ("dX", r["dX"], dX), ("dW", r["dW"], M.T @ dZ), ("db", r["db"], dZ.sum(0))):
            err = float((got.double() - ref).norm() / ref.norm())
            assert err <= tol, (order, name, err)


@pytest.mark.parametrize("transposed", [False, True])
def test_layer_has_room_for_rows_across_two_lines(transposed):
    """Rows of 94 bytes at a stride of 128 that all lie in two lines: at 9 entries per row the copy pays for these, not for rows at every offset (1.73 lines).  The
    layer's scratch, sized without the stride, has the room: the copy's first rows are found there."""
    from paper_2305_17469_amd import binding as B
    n, deg, fi, fo = 300_000, 9, (120, 47)[not transposed], (47, 120)[not transposed]
    gen = torch.Generator(device="cuda:0").manual_seed(5)
    g = B.Graph((torch.arange(n + 1, device="cuda:0") * deg).int(), torch.randint(0, n, (n * deg,), device="cuda:0", generator=gen).int(), n)

    def rows(F, across):
        buf = torch.zeros(n * 128 + 64, dtype=torch.bfloat16, device="cuda:0")
        t = buf[20:20 + n * 64].view(n, 64)[:, :F] if across else buf[:n * 120].view(n, 120)[:, :F]
        return t.copy_(torch.randn((n, F), device="cuda:0", generator=gen))
    X, dY = rows(fi, not transposed), rows(fo, transposed)
    W = torch.randn((fi, fo), device="cuda:0", generator=gen).bfloat16()
    desc = B.make_desc("sum", "bf16", False, fi, fo)
    bufs = B.LayerBuffers(g, desc)
    announce("room in a layer's scratch", transposed)
    order = "comb_first" if transposed else "agg_first"
    Y, used = B.gt_layer_fwd(g, desc, X, W, None, bufs, order)
    bufs.scratch.fill_(7)
    if transposed:
        B.gt_layer_bwd(g, desc, used, dY, X, W, Y, bufs, order)
        table = dY
    else:
        B.gt_layer_fwd(g, desc, X, W, None, bufs, order)
        table = X
    torch.cuda.synchronize()
    lines = bufs.scratch[:bufs.scratch.numel() // 128 * 128].view(-1, 128)[:, :94]
    first = table[:3].contiguous().view(torch.uint8)
    at = (lines == first[0]).all(1).nonzero().flatten().tolist()
    assert any(torch.equal(lines[i:i + 3], first) for i in at)
