"""The scratch of the aggregation's entry points: each call has its own, so one Graph serves several streams at a time, and a captured graph keeps to
its own memory whatever is called afterwards.  Tables are of a uniform graph whose narrow rows are copied into the scratch and gathered from there; every
result is bit for bit that of the same call without room for the copy."""
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
    a, b = graph.aggregate_ws(47), graph.aggregate_ws(47)
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
