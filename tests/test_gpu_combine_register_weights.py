"""bf16 products whose weights stay in registers (blocks of 32 rows, 16 to 128 columns per wavefront, at most two column slices) on
both sides of the rules that choose them: every instance at its last and one of its first terms, rows around a block and fewer
blocks than workgroups, columns around 8, 16 and a slice; both orders of the weights, rows of C aligned, padded and contiguous, bias
and ReLU, NaN in the operands' row padding.  Against 64 bits: |error| <= (K + 2) 2^-24 sum |terms| + 2^-8 |result|.
Masked input gradients (combination first) against the same call without the mask, bit for bit."""
import numpy as np
import pytest
import torch

from gpu_util import announce
from test_gpu_combine_rows import _check

pytestmark = pytest.mark.gpu


# (rows, columns, terms); the first that one slice holds: N <= 128, 256, 384, 512, 640, 1024
@pytest.mark.parametrize("transB", [False, True], ids=["NN", "NT"])
@pytest.mark.parametrize("M,N,K", [(2000, 65, 257), (2017, 128, 512), (8223, 127, 640), (2001, 121, 832), (2031, 66, 1024), (4097, 129, 384), (12288, 256, 511),
                                   (2049, 255, 640), (65567, 250, 640 - 31), (98305, 199, 638), (49152, 257, 256), (49153, 384, 225), (32801, 384, 320), (2048, 300, 416),
                                   (49183, 512, 250), (49155, 385, 319), (98309, 602, 64), (49157, 640, 128), (49154, 602, 256), (131073, 641, 65), (131087, 1024, 128),
                                   (49159, 1001, 256), (49161, 700, 300), (49163, 513, 512), (1024, 129, 641), (1055, 256, 1024), (16384, 200, 700)])
def test_register_weights(M, N, K, transB):
    v8 = (N + 7) // 8 * 8
    for bias, relu, ldc in ((True, True, N), (False, False, v8), (True, False, v8 + 8), (False, True, N + 1)):
        _check(M, N, K, torch.bfloat16, transB, bias, relu, ldc)


# contiguous operands of any width, at any element of a buffer; the element past the end of each is NaN
@pytest.mark.parametrize("transB", [False, True], ids=["NN", "NT"])
@pytest.mark.parametrize("M,N,K", [(2000, 65, 257), (1024, 130, 511), (2031, 127, 1023), (2001, 300, 66), (1025, 255, 602), (2051, 601, 129), (32801, 601, 130), (65541, 270, 65),
                                   (32769, 1001, 250), (1033, 700, 300), (1030, 200, 702)])
def test_contiguous(M, N, K, transB):
    from paper_2305_17469_amd import binding as B
    gen = torch.Generator(device="cuda:0").manual_seed(M + N + K)

    def packed(n, F, off):
        t = torch.full((off + n * F + 1,), float("nan"), device="cuda:0", dtype=torch.bfloat16)
        t = t[off:off + n * F].view(n, F)
        return t.copy_(torch.randn((n, F), device="cuda:0", generator=gen))

    for offa, offw in ((0, 0), (3, 0), (0, 1), (2, 6)):
        A, W = packed(M, K, offa), packed(N, K, offw) if transB else packed(K, N, offw)
        announce("register weights, contiguous", M, N, K, "NT" if transB else "NN", offa, offw)
        out = torch.full((M * N + 9,), 7.0, device="cuda:0", dtype=torch.bfloat16)
        got = B.gt_combine(A, W, transB=transB, out=out[1:1 + M * N].view(M, N))
        w = (W.t() if transB else W).double().contiguous()
        ref, mag = A.double() @ w, A.double().abs() @ w.abs()
        assert bool(((got.double() - ref).abs() <= (K + 2) * 2.0 ** -24 * mag + 2.0 ** -8 * ref.abs()).all())
        assert bool((out[0] == 7) and (out[1 + M * N:] == 7).all())


@pytest.mark.parametrize("pad_writable", [False, True])
@pytest.mark.parametrize("n,fi,fo", [(49155, 301, 200), (49153, 602, 104), (20011, 100, 304), (16385, 127, 520), (16400, 128, 512)])
def test_masked(n, fi, fo, pad_writable):
    from paper_2305_17469_amd import binding as B
    rng = np.random.default_rng(n)
    rowptr = torch.arange(n + 1, dtype=torch.int32, device="cuda:0")
    g = B.Graph(rowptr, torch.from_numpy(rng.permutation(n).astype(np.int32)).cuda(), n)
    gen = torch.Generator(device="cuda:0").manual_seed(n)

    def rows(F, fill=0.0):
        t = torch.full((n, (F + 7) // 8 * 8), fill, device="cuda:0", dtype=torch.bfloat16)
        t[:, :F] = torch.randn((n, F), device="cuda:0", generator=gen)
        return t

    X, dY, W = rows(fi, 5.0), rows(fo), torch.randn((fi, fo), device="cuda:0", generator=gen).bfloat16()
    got = []
    for in_relu in (False, True):
        announce("register weights, mask", n, fi, fo, pad_writable, in_relu)
        desc = B.make_desc("sum", "bf16", False, fi, fo, need_dx=True, in_relu=in_relu, dy_is_dz=True, pad_writable=pad_writable)
        out = rows(fi, 3.0)
        B.gt_layer_bwd(g, desc, "comb_first", dY[:, :fo], X[:, :fi], W, None, B.LayerBuffers(g, desc), "comb_first", out_dX=out[:, :fi])
        assert bool((out[:, fi:] == (0 if pad_writable else 3)).all())
        got.append(out[:, :fi])
    assert torch.equal(got[1], torch.where(X[:, :fi] > 0, got[0], torch.zeros_like(got[0])))


# the same at the lines where the row tiles come to full rounds, and where few terms keep little of A in flight
@pytest.mark.parametrize("transB", [False, True], ids=["NN", "NT"])
@pytest.mark.parametrize("M,N,K", [(4095, 129, 384), (4095, 256, 511), (8191, 255, 640), (98305, 129, 513), (65537, 130, 300), (32769, 300, 416), (65537, 512, 250), (65539, 385, 319), (524291, 300, 65),
                                   (524288, 511, 128), (393217, 602, 64), (393221, 750, 100), (196611, 1001, 128), (196609, 1100, 66), (131072, 641, 250), (49153, 640, 256),
                                   (98304, 100, 300), (262145, 70, 260), (18432, 128, 300), (18433, 70, 600), (32769, 128, 512), (8191, 200, 700), (16384, 150, 900)])
def test_register_weights_at_lines(M, N, K, transB):
    test_register_weights(M, N, K, transB)


@pytest.mark.parametrize("transB", [False, True], ids=["NN", "NT"])
@pytest.mark.parametrize("M,N,K", [(2000, 257, 70), (18432, 300, 127), (32769, 257, 70), (33001, 500, 100), (393217, 333, 75), (2001, 601, 100), (24577, 601, 100), (32771, 700, 90), (32773, 1001, 66),
                                   (8193, 601, 129), (18433, 401, 300), (2003, 401, 200)])
def test_contiguous_at_lines(M, N, K, transB):
    test_contiguous(M, N, K, transB)


@pytest.mark.parametrize("n,fi,fo", [(65539, 130, 300), (98311, 100, 304), (393217, 602, 104), (131075, 700, 200)])
def test_masked_at_lines(n, fi, fo):
    for pad_writable in (False, True):
        test_masked(n, fi, fo, pad_writable)
