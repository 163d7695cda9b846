"""The scratch of the aggregation's entry points: each call has its own, so one Graph serves several streams at a time, and a captured graph keeps to
its own memory whatever is called afterwards.  Tables are of a uniform graph whose narrow rows are copied into the scratch and gathered from there; every
result is bit for bit that of the same call without room for the copy."""
import ctypes

import pytest
import torch

from gpu_util import announce

pytestmark = pytest.mark.gpu
N = 450_001


@pytest.fixture(scope="module")
def graph():
    from paper_2305_17469_amd import binding as B
    gen = torch.Generator(device="cuda:0").manual_seed(7)
    deg = torch.randint(12, 40, (N,), device="cuda:0", generator=gen)
    rowptr = torch.zeros(N + 1, dtype=torch.int64, device="cuda:0")
    rowptr[1:] = torch.cumsum(deg, 0)
    col = torch.randint(0, N, (int(rowptr[-1]),), device="cuda:0", generator=gen)
    return B.Graph(rowptr.int(), col.int(), N)


def _table(F, seed):
    return torch.randn((N, F), device="cuda:0", generator=torch.Generator(device="cuda:0").manual_seed(seed)).bfloat16()


def _in_place(g, X, transposed=False):
    """The call with the least workspace: the table is gathered where it is."""
    from paper_2305_17469_amd import binding as B
    Y, ws = torch.empty_like(X), torch.empty(256, dtype=torch.uint8, device="cuda:0")
    call = B.lib.gt_aggregate_bwd if transposed else B.lib.gt_aggregate_fwd
    assert call(g.handle, B.REDUCE["mean"], 1, X.shape[1], X.data_ptr(), X.stride(0), Y.data_ptr(), Y.stride(0), ws.data_ptr(), 256, None) == 0
    torch.cuda.synchronize()
    return Y


def test_blocks_of_two_calls_are_apart(graph):
    X = _table(47, 1)
    a, b = graph.aggregate_ws(47, X), graph.aggregate_ws(47, X)
    assert a.data_ptr() + a.numel() <= b.data_ptr() or b.data_ptr() + b.numel() <= a.data_ptr()


def test_two_streams(graph):
    from paper_2305_17469_amd import binding as B
    tables = [_table(47, 1), _table(47, 2)]
    want = [(_in_place(graph, X), _in_place(graph, X, True)) for X in tables]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    got = [[], []]
    announce("aggregation, two streams")
    for _ in range(6):
        for i, st in enumerate(streams):
            with torch.cuda.stream(st):
                got[i].append((B.gt_aggregate_fwd(graph, "mean", tables[i]), B.gt_aggregate_bwd(graph, "mean", tables[i])))
    torch.cuda.synchronize()
    for i in range(2):
        for Y, dX in got[i]:
            assert torch.equal(Y, want[i][0]) and torch.equal(dX, want[i][1])


def test_handle_of_the_current_stream():
    from paper_2305_17469_amd import binding as B
    st = torch.cuda.Stream()
    assert B._stream() == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(st):
        assert B._stream() == st.cuda_stream != torch.cuda.default_stream().cuda_stream
    assert B._stream() == torch.cuda.current_stream().cuda_stream


def test_captured_call_keeps_to_its_memory(graph):
    from paper_2305_17469_amd import binding as B
    X, wide = _table(28, 3), _table(47, 4)
    Y = torch.empty_like(X)
    want, want_wide = _in_place(graph, X), _in_place(graph, wide)
    st = torch.cuda.Stream()
    st.wait_stream(torch.cuda.current_stream())
    announce("aggregation, captured")
    with torch.cuda.stream(st):
        B.gt_aggregate_fwd(graph, "mean", X, out=Y)
    torch.cuda.synchronize()
    captured = torch.cuda.CUDAGraph()
    with torch.cuda.graph(captured, stream=st):
        B.gt_aggregate_fwd(graph, "mean", X, out=Y)
    held = []
    for k in range(3):
        assert torch.equal(B.gt_aggregate_fwd(graph, "mean", wide), want_wide)     # a larger need than the captured call's
        held += [torch.full((N, 64), 3 + k, dtype=torch.uint8, device="cuda:0") for _ in range(4)]
        Y.zero_()
        captured.replay()
        torch.cuda.synchronize()
        assert torch.equal(Y, want)
    assert all(bool((t == 3 + i // 4).all()) for i, t in enumerate(held))


def test_sizes(graph):
    """What a call needs is what it refuses to go without; the room for a copy comes on top, for the table at hand alone."""
    from paper_2305_17469_amd import binding as B
    least, best = ctypes.c_size_t(), ctypes.c_size_t()
    assert graph.info()["fwd_split_rows"] == 0 and graph.info()["bwd_split_rows"] == 0

    def sizes(g, X, F, dtype, ld, transposed=0):
        assert B.lib.gt_aggregate_ws_size(g.handle, F, ctypes.byref(least)) == 0
        assert B.lib.gt_aggregate_best_ws_size(g.handle, transposed, dtype, F, X, ld, ctypes.byref(best)) == 0
        return least.value, best.value
    for transposed in (0, 1):
        assert sizes(graph, 4096, 47, 1, 47, transposed) == (0, N * 128)
        assert sizes(graph, 4096, 28, 1, 28, transposed) == (0, N * 64)
        assert sizes(graph, 4096, 47, 1, 64, transposed) == (0, 0)             # one line per row as it is
        assert sizes(graph, 4096 + 64, 47, 1, 64, transposed) == (0, N * 128)  # two
        assert sizes(graph, 4096, 47, 0, 47, transposed) == (0, 0)             # rows past 128 bytes
        assert sizes(graph, 4096, 12, 1, 12, transposed) == (0, 0)             # and of up to 32
    assert B.lib.gt_aggregate_best_ws_size(graph.handle, 0, 7, 47, 4096, 47, ctypes.byref(best)) == 1
    assert B.lib.gt_aggregate_best_ws_size(graph.handle, 0, 1, 47, 4096, 47, None) == 1
    assert B.lib.gt_aggregate_best_ws_size(None, 0, 1, 47, 4096, 47, ctypes.byref(best)) == 1
    # a graph with split rows: partial rows are needed, its tables are not copied
    rowptr = torch.arange(3, device="cuda:0", dtype=torch.int32) * 4000
    skewed = B.Graph(rowptr, torch.randint(0, N, (8000,), device="cuda:0", dtype=torch.int32), N)
    need, most = sizes(skewed, 4096, 47, 1, 47)
    assert 0 < need <= most
    X, Y = _table(47, 5), torch.zeros((2, 47), dtype=torch.bfloat16, device="cuda:0")
    ws = torch.empty(need, dtype=torch.uint8, device="cuda:0")
    announce("aggregation, least scratch")
    call = B.lib.gt_aggregate_fwd
    assert call(skewed.handle, 0, 1, 47, X.data_ptr(), 47, Y.data_ptr(), 47, ws.data_ptr(), need, None) == 0
    assert call(skewed.handle, 0, 1, 47, X.data_ptr(), 47, Y.data_ptr(), 47, ws.data_ptr(), need - 1, None) == 3
    # the entry point without scratch takes every graph whose partial rows fit, and gathers in place
    out = torch.empty_like(X)
    B.gt_aggregate_fwd_static(graph, "mean", X, out)
    assert torch.equal(out, _in_place(graph, X))


def test_calls_take_what_they_need(graph):
    """Sizes are asked for once per width, or per table where its stride and alignment count; a call that needs nothing allocates nothing."""
    buf = torch.empty(20 + N * 64, dtype=torch.bfloat16, device="cuda:0")
    lines, across = buf[:N * 64].view(N, 64)[:, :47], buf[20:20 + N * 64].view(N, 64)[:, :47]
    packed, wide = buf[:N * 47].view(N, 47), torch.empty((N, 80), dtype=torch.bfloat16, device="cuda:0")
    for _ in range(2):
        assert graph._scratch(47) == (None, None, 0)
        for table, want in ((lines, 0), (across, N * 128), (packed, N * 128), (lines, 0), (packed[:, :28], N * 64), (wide, 0), (wide.float(), 0)):
            for transposed in (False, True):
                ws, ptr, n = graph._scratch(table.shape[1], table, transposed)
                assert n == want and ((ws, ptr) == (None, None) if want == 0 else ws.numel() == n and ptr == ws.data_ptr() and ptr % 256 == 0)


def test_timing_record_has_the_copy_in_it():
    """The record of a gather from a copy spans both kernels.  Degree 12, where the copy is some 12 % of the call: the record has to reach 95 % of what events
    around the call measure (launch overhead is 1 %)."""
    from paper_2305_17469_amd import binding as B
    n, deg = 2_000_000, 12
    gen = torch.Generator(device="cuda:0").manual_seed(9)
    g = B.Graph((torch.arange(n + 1, device="cuda:0") * deg).int(), torch.randint(0, n, (n * deg,), device="cuda:0", generator=gen).int(), n)
    X = torch.randn((n, 47), device="cuda:0", generator=gen).bfloat16()
    assert g.aggregate_ws(47, X).numel() == n * 128
    Y, shares = torch.empty_like(X), []
    announce("aggregation, timing record")
    for _ in range(3):
        B.gt_aggregate_fwd(g, "sum", X, out=Y)
    for _ in range(9):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        B.gt_trace_reset()
        B.gt_trace_enable(True)
        try:
            a.record()
            B.gt_aggregate_fwd(g, "sum", X, out=Y)
            b.record()
            recs = B.gt_trace_records()
        finally:
            B.gt_trace_enable(False)
            B.gt_trace_reset()
        b.synchronize()
        assert len(recs) == 1 and recs[0][0] == 0
        shares.append(recs[0][4] / a.elapsed_time(b))
    assert 0.95 <= sorted(shares)[4] <= 1.001, shares
