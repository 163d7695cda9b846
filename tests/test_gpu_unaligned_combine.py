"""gt_combine on rows without 16-byte alignment (contiguous operands and outputs of odd widths, bases off by one element)
at the sizes where the kernels and their tails change: rows at the weight-stationary kernels' threshold and around the
row blocks, widths around a 16-byte chunk, a 128-byte slice and the 64- / 128- / 256-column slices, several 256 x 256 tiles
of the weight gradient.  Against products in 64 bits; fp32: |error| <= 1e-5 sum |a b| (as in test_gpu_combine), bf16 results
one rounding more.  Guard elements around C must stay untouched."""
import pytest
import torch

from gpu_util import announce

pytestmark = pytest.mark.gpu
GUARD = 3.5

SHAPES = [(8192, 1, 1), (8193, 3, 5), (8200, 47, 100), (8223, 65, 9), (9001, 602, 33), (8255, 130, 127), (8192, 259, 255),
          (8196, 7, 130), (9000, 31, 301), (8300, 600, 127), (20000, 5, 1000), (300, 41, 602), (4099, 100, 603)]


def _mat(r, c, dtype, off, gen):
    buf = torch.randn(off + r * c + 9, device="cuda:0", generator=gen).to(dtype)
    return buf[off:off + r * c].view(r, c)


def _check(got, A, B, bias, relu, what):
    ref, mag = A.double() @ B.double(), A.double().abs() @ B.double().abs()
    if bias is not None:
        ref, mag = ref + bias.double(), mag + bias.double().abs()
    if relu:
        ref = ref.clamp(min=0)
    bound = 1e-5 * mag + 1e-30 + (2.0 ** -8 * ref.abs() if got.dtype == torch.bfloat16 else 0)
    assert bool(((got.double() - ref).abs() <= bound).all()), what


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_rows_without_alignment(shape, dtype):
    from paper_2305_17469_amd import binding as B
    M, N, K = shape
    gen = torch.Generator(device="cuda:0").manual_seed(M + N + K)
    bias = torch.randn(N, device="cuda:0", generator=gen)
    for off in (0, 1):
        A, W, Wt = _mat(M, K, dtype, off, gen), _mat(K, N, dtype, off, gen), _mat(N, K, dtype, off, gen)
        for name, kw, b in (("nn", dict(bias=bias, relu=True), W), ("nt", dict(transB=True), Wt)):
            announce("unaligned combine", dtype, shape, name, "offset", off)
            buf = torch.full((off + M * N + 16,), GUARD, device="cuda:0", dtype=dtype)
            C = buf[off:off + M * N].view(M, N)
            B.gt_combine(A, b, out=C, **kw)
            _check(C, A, b.t() if name == "nt" else b, kw.get("bias"), kw.get("relu"), (name, shape, off))
            assert bool((buf[:off] == GUARD).all()) and bool((buf[off + M * N:] == GUARD).all()), (name, "guard")
        G = _mat(M, N, dtype, off, gen)
        dW = B.gt_combine(A, G, transA=True, out_dtype=torch.float32)
        _check(dW, A.t(), G, None, False, ("tn", shape, off))


@pytest.mark.parametrize("shape", [(257, 70, 16500), (602, 256, 24600), (300, 520, 50000), (1024, 512, 66000)],
                         ids=lambda s: "x".join(map(str, s)))
def test_bf16_weight_gradient_over_several_tiles(shape):
    from paper_2305_17469_amd import binding as B
    M, N, K = shape
    gen = torch.Generator(device="cuda:0").manual_seed(K)
    pad = lambda c: (c + 7) // 8 * 8   # noqa: E731
    A = torch.randn((K, pad(M)), device="cuda:0", generator=gen).bfloat16()[:, :M]
    G = torch.randn((K, pad(N)), device="cuda:0", generator=gen).bfloat16()[:, :N]
    announce("bf16 weight gradient tiles", shape)
    dW = B.gt_combine(A, G, transA=True, out_dtype=torch.float32)
    _check(dW, A.t(), G, None, False, shape)
    assert torch.equal(dW, B.gt_combine(A, G, transA=True, out_dtype=torch.float32))
