"""bf16 products on both sides of the rules for the row-tiled kernel (128 x 256 tiles, k-tiles of 64): rows, columns and terms around the
ends of its tiles, both orders of the weights, rows of C aligned, padded and contiguous, bias and ReLU; operands whose row padding
holds NaN and rows past which there is nothing.  The weights of the weight-stationary kernels in [k][n] order with every ragged patch.
Against 64 bits: |error| <= (K + 2) 2^-24 sum |terms| + 2^-8 |result|."""
import pytest
import torch

from gpu_util import announce

pytestmark = pytest.mark.gpu


def _rows(n, F, dtype, gen, pad=8):
    ld = (F + pad - 1) // pad * pad
    t = torch.full((n, ld), float("nan"), device="cuda:0", dtype=dtype)
    t[:, :F] = torch.randn((n, F), device="cuda:0", generator=gen).to(dtype)
    return t[:, :F]


def _check(M, N, K, dtype, transB, bias, relu, ldc):
    from paper_2305_17469_amd import binding as B
    gen = torch.Generator(device="cuda:0").manual_seed(M + N + K)
    A, W = _rows(M, K, dtype, gen), _rows(N, K, dtype, gen) if transB else _rows(K, N, dtype, gen)
    b = torch.randn(N, device="cuda:0", generator=gen) if bias else None
    out = torch.full((M, ldc), 7.0, device="cuda:0", dtype=dtype)
    announce("rows", M, N, K, dtype, "NT" if transB else "NN", bias, relu, ldc)
    got = B.gt_combine(A, W, b, relu=relu, transB=transB, out=out[:, :N])
    w = (W.t() if transB else W).double().contiguous()
    ref, mag = A.double() @ w, A.double().abs() @ w.abs()
    if bias:
        ref, mag = ref + b.double(), mag + b.double().abs()
    ref = ref.clamp(min=0) if relu else ref
    bound = (K + 2) * 2.0 ** -24 * mag + (2.0 ** -8 * ref.abs() if dtype == torch.bfloat16 else 0)
    assert bool(((got.double() - ref).abs() <= bound).all())
    assert bool((out[:, N:] == 7).all())


@pytest.mark.parametrize("transB", [False, True], ids=["NN", "NT"])
@pytest.mark.parametrize("M,N,K", [(1024, 129, 64), (1030, 602, 64), (1500, 279, 100), (1500, 281, 100), (2000, 129, 64), (1025, 256, 257), (1151, 257, 319),
                                   (4095, 65, 65), (4096, 65, 65), (4223, 130, 256), (8191, 200, 127), (8192, 300, 129), (8193, 513, 255),
                                   (16001, 602, 200), (20001, 72, 602), (50001, 128, 602), (65537, 257, 200), (9001, 512, 1000), (320001, 602, 66),
                                   (350001, 602, 66), (440001, 602, 66), (350001, 602, 130)])
def test_row_tiles(M, N, K, transB):
    v8 = (N + 7) // 8 * 8
    for bias, relu, ldc in ((True, True, N), (False, False, v8), (True, False, v8 + 8), (False, True, N + 1)):
        _check(M, N, K, torch.bfloat16, transB, bias, relu, ldc)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
@pytest.mark.parametrize("N,K", [(3, 5), (33, 17), (41, 128), (65, 64), (130, 100), (255, 33), (256, 256), (300, 40), (602, 63)])
def test_stationary_weights(N, K, dtype):
    _check(8200, N, K, dtype, False, True, False, N)
    _check(33003, N, K, dtype, False, False, True, (N + 7) // 8 * 8)
