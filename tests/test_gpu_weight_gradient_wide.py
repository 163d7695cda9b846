"""bf16 weight gradients on both sides of the rules for the tiles of 320 x 256, 256 x 320 and 640 x 128: outputs around the ends of tiles, reductions
around steps of 32 and at the thresholds, operands padded (NaN in the padding) or contiguous from any element of a buffer, the element past the end NaN.  Against 64 bits with the
bound of the weight-gradient tests, twice the same bits; the column sums that ride along through a layer's bias gradient."""
import pytest
import torch

from gpu_util import announce

pytestmark = pytest.mark.gpu


def _rows(n, F, padded, off, gen):
    ld = (F + 7) // 8 * 8 if padded else F
    buf = torch.full((off + n * ld + 1,), float("nan"), device="cuda:0", dtype=torch.bfloat16)
    t = buf[off:off + n * ld].view(n, ld)[:, :F]
    return t.copy_(torch.randn((n, F), device="cuda:0", generator=gen))


@pytest.mark.parametrize("padded", [True, False], ids=["padded", "contiguous"])
@pytest.mark.parametrize("M,N,K", [(320, 256, 98304), (321, 250, 98335), (602, 255, 98336), (256, 320, 98305), (255, 321, 98311), (640, 128, 98304), (639, 127, 98367),
                                   (641, 66, 98305), (65, 257, 98309), (1024, 320, 16384), (1023, 319, 16385), (700, 600, 16400), (300, 99, 49152), (129, 300, 49183), (129, 200, 98304),
                                   (257, 256, 98303)])
def test_wide_tiles(M, N, K, padded):
    from paper_2305_17469_amd import binding as B
    gen = torch.Generator(device="cuda:0").manual_seed(M + N + K)
    for offa, offg in ((0, 0), (5, 2)):
        if padded and offa:
            continue
        A, G = _rows(K, M, padded, offa, gen), _rows(K, N, padded, offg, gen)
        announce("wide weight gradient", M, N, K, padded, offa)
        dW = B.gt_combine(A, G, transA=True, out_dtype=torch.float32)
        a, g = A.double().t(), G.double()
        assert bool(((dW.double() - a @ g).abs() <= 1e-5 * (a.abs() @ g.abs())).all())
        assert torch.equal(dW, B.gt_combine(A, G, transA=True, out_dtype=torch.float32))


@pytest.mark.parametrize("n,fi,fo,padded", [(98311, 300, 130, True), (49157, 131, 300, False), (98305, 600, 100, True)])
def test_bias_gradient(n, fi, fo, padded):
    from paper_2305_17469_amd import binding as B
    gen = torch.Generator(device="cuda:0").manual_seed(n)
    g = B.Graph(torch.arange(n + 1, dtype=torch.int32, device="cuda:0"), torch.randperm(n, device="cuda:0", generator=gen).int(), n)
    X, dY = _rows(n, fi, padded, 0, gen), _rows(n, fo, padded, 0, gen)
    W = torch.randn((fi, fo), device="cuda:0", generator=gen).bfloat16()
    desc = B.make_desc("sum", "bf16", False, fi, fo, need_dx=False, dy_is_dz=True)
    bufs = B.LayerBuffers(g, desc)
    announce("wide weight gradient, bias", n, fi, fo, padded)
    Y, used = B.gt_layer_fwd(g, desc, X, W, torch.zeros(fo, device="cuda:0"), bufs, "agg_first")
    r = B.gt_layer_bwd(g, desc, used, dY, X, W, Y, bufs, "agg_first")
    d = dY.double()
    assert bool(((r["db"].double() - d.sum(0)).abs() <= 1e-5 * d.abs().sum(0)).all())


@pytest.mark.parametrize("padded", [True, False], ids=["padded", "contiguous"])
@pytest.mark.parametrize("M,N,K", [(640, 128, 131072), (639, 127, 131075), (602, 100, 131073), (300, 99, 73728), (641, 66, 73731), (1024, 320, 20480), (1023, 319, 20481), (700, 600, 20490)])
def test_wide_tiles_at_lines(M, N, K, padded):
    test_wide_tiles(M, N, K, padded)
