"""More work than one launch can hold (2^32 threads) on the GPU: the forward, the input gradient and the encoder
block's attention go on in a further launch, the patch gather and its adjoint stride on, with the same results.

One channel and one group element keep the tensors small (2 GiB each).  The layer is then y = w x + b, two roundings
of fp16 (the spectrum of the weight is the weight); bound 2 u of the result, here on the first rows, on those around
the end of the first launch and on the last ones.
"""
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

U = 2.0 ** -11


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("plan", [None, "1,8,1,0"])
def test_rows_of_several_launches(monkeypatch, plan):
    from paper_2607_21271_amd import ops
    if plan is not None:
        monkeypatch.setenv("EQL_XS_PLAN", plan)  # the most threads a row: the first launch ends at 2^27 rows
    N = (1 << 30) + 77 if plan is None else (1 << 27) + 77
    say("many rows", N, plan)
    part = torch.randn(1 << 20, device="cuda", dtype=torch.float16)
    x = part.repeat(N // part.numel() + 1)[:N].view(N, 1, 1)
    x[-77:] += 1.0
    w = torch.full((1, 1, 1), 0.75, dtype=torch.float16, device="cuda")
    b = torch.full((1,), 0.5, dtype=torch.float16, device="cuda")
    spec = ops.weight_spectrum(w)
    y = ops.forward(x, spec, b, 1, 1, 1)
    for a, z in ((0, 1 << 20), ((1 << 27) - 4096, (1 << 27) + 77), (N - (1 << 20), N)):
        ref = x[a:z].double() * 0.75 + 0.5
        assert float((y[a:z].double() - ref).abs().max()) <= 2 * U * float(ref.abs().max())
    del y
    dx = ops.backward_input(x, spec, 1, 1, 1)
    for a, z in ((0, 1 << 20), ((1 << 27) - 4096, (1 << 27) + 77), (N - (1 << 20), N)):
        ref = x[a:z].double() * 0.75
        assert float((dx[a:z].double() - ref).abs().max()) <= 2 * U * float(ref.abs().max())


def test_attention_of_several_launches():
    """2^24 and more (image, head) pairs of one token: softmax over one key, so the output is v."""
    from paper_2607_21271_amd.blocks import EQViTBlock
    B, H, D, T = (1 << 15) + 5, 512, 32, 4
    say("attention pairs", B * H)
    C = H * D // T
    blk = EQViTBlock(T, C, H, linear="standard", device="cuda", dtype=torch.float16)
    part = torch.randn(1 << 10, 1, 3 * C, T, device="cuda", dtype=torch.float16)
    qkv = part.repeat(B // part.shape[0] + 1, 1, 1, 1)[:B]
    with torch.no_grad():
        o = blk.attention(qkv)
    assert torch.equal(o, qkv[:, :, 2 * C:])


def test_patches_of_many_pixels():
    """2^26 pixels, one wave each (a grid of 2^32 threads wraps to none): at k = 1 the patch is the pixel, gathered and
    scattered back."""
    from paper_2607_21271_amd import gconv
    H, W = 8192, 8192
    say("pixels", H * W)
    f = torch.randn(1, H, W, 1, 1, device="cuda").to(torch.float16)
    X = gconv.gather(f, 1, 1)
    assert torch.equal(X.flatten(), f.flatten())
    assert torch.equal(gconv.scatter(X, 1, H, W, 1, 1, 1), f)
