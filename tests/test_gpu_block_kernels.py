"""Layer-norm and attention kernels of the encoder block against the same sums in float64.

Sizes sit at the edges: tokens around the 16-query tiles and 32-key steps, one token, the longest sequence, few and
many (image, head) pairs; norm rows of one vector up to 16 KB, odd group orders.  Bounds: 16-bit outputs carry one
rounding (unit roundoff u) and, in attention, the rounded probabilities (another u, weights summing to one), so 4 u of
the largest value; fp32 norms 1e-5.
"""
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

DT = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
TOL = {"f32": 1e-5, "f16": 4 * 2.0 ** -11, "bf16": 4 * 2.0 ** -8}


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _err(a, b):
    return float((a.double() - b).abs().max() / b.abs().max())


@pytest.mark.parametrize("T,C,rows", [(1, 8, 1), (3, 8, 5), (4, 192, 1001), (8, 96, 197), (5, 72, 70), (2, 1024, 9),
                                      (4, 257 * 2, 33), (16, 128, 8200), (4, 1024, 515), (8, 512, 7)])
@pytest.mark.parametrize("dt", ["f32", "f16", "bf16"])
def test_group_norm(T, C, rows, dt):
    from paper_2607_21271_amd.blocks import GroupLayerNorm
    say("group norm", T, C, rows, dt)
    torch.manual_seed(T * C)
    m = GroupLayerNorm(C, device="cuda", dtype=DT[dt])
    x = (torch.randn(rows, C, T, device="cuda") * 3 + 2).to(DT[dt])
    with torch.no_grad():
        m.weight.add_(torch.randn(C, device="cuda").to(DT[dt]))
        m.bias.add_(torch.randn(C, device="cuda").to(DT[dt]))
        y = m(x)
        xd = x.double()
        mu = xd.mean((-2, -1), keepdim=True)
        var = (xd - mu).square().mean((-2, -1), keepdim=True)
        ref = (xd - mu) / (var + m.eps).sqrt() * m.weight.double()[:, None] + m.bias.double()[:, None]
    assert y.dtype == x.dtype and _err(y, ref) <= TOL[dt]
    # a call that wants gradients takes torch's operations
    assert m(x.clone().requires_grad_(True)).requires_grad


@pytest.mark.parametrize("shape", [(1,), (192, 1), (1, 192)])
def test_group_norm_affine_of_another_shape(shape):
    """A weight or bias that is not one value a channel keeps torch's broadcasting (the kernel reads C values of each):
    a shared bias, and shapes that torch widens or refuses."""
    from paper_2607_21271_amd.blocks import GroupLayerNorm
    say("group norm affine", shape)
    torch.manual_seed(5)
    x = torch.randn(7, 192, 4, device="cuda")
    for name in ("weight", "bias"):
        m = GroupLayerNorm(192, device="cuda")
        setattr(m, name, torch.nn.Parameter(torch.randn(shape, device="cuda"), requires_grad=False))
        xd = x.double()
        mu = xd.mean((-2, -1), keepdim=True)
        n = (xd - mu) / ((xd - mu).square().mean((-2, -1), keepdim=True) + m.eps).sqrt()
        with torch.no_grad():
            try:
                ref = n * m.weight.double()[:, None] + m.bias.double()[:, None]
            except RuntimeError:
                with pytest.raises(RuntimeError):
                    m(x)
                continue
            y = m(x)
        assert y.shape == ref.shape and _err(y, ref) <= TOL["f32"]


@pytest.mark.parametrize("B,L,heads,D", [(1, 1, 1, 64), (2, 16, 3, 64), (1, 17, 2, 32), (3, 32, 1, 128), (2, 33, 5, 64),
                                         (1, 50, 12, 64), (2, 65, 3, 32), (1, 128, 2, 128), (1, 129, 2, 64),
                                         (5, 145, 6, 64), (50, 197, 12, 64), (1, 224, 3, 128), (2, 225, 2, 32),
                                         (1, 256, 3, 64), (1, 256, 1, 128)])
@pytest.mark.parametrize("dt", ["f16", "bf16"])
def test_attention(B, L, heads, D, dt):
    from paper_2607_21271_amd.blocks import EQViTBlock
    say("attention", B, L, heads, D, dt)
    torch.manual_seed(L)
    T = 4
    C = heads * D // T
    blk = EQViTBlock(T, C, heads, linear="standard", device="cuda", dtype=DT[dt])
    qkv = torch.randn(B, L, 3 * C, T, device="cuda").to(DT[dt])
    qkv[:, :, :C] *= 3  # peaked rows among flat ones
    with torch.no_grad():
        o = blk.attention(qkv)
        q, k, v = qkv.double().view(B, L, 3, heads, D).permute(2, 0, 3, 1, 4).contiguous()
        a = torch.softmax(q @ k.transpose(-1, -2).contiguous() * D ** -0.5, -1)
        ref = (a @ v).permute(0, 2, 1, 3).reshape(B, L, C, T)
    assert o.shape == ref.shape and _err(o, ref) <= TOL[dt]


def test_attention_infinities():
    """A query whose scores hold an infinity or a NaN gives NaN, its neighbours are untouched."""
    from paper_2607_21271_amd.blocks import EQViTBlock
    say("attention infinities")
    blk = EQViTBlock(4, 32, 2, linear="standard", device="cuda", dtype=torch.float16)
    torch.manual_seed(0)
    qkv = torch.randn(1, 21, 96, 4, device="cuda").to(torch.float16)
    with torch.no_grad():
        ref = blk.attention(qkv)
        bad = qkv.clone()
        bad[0, 5, 0, 0] = float("nan")   # head 0 of query 5
        bad[0, 9, 16, 0] = float("inf")  # head 1 of query 9
        o = blk.attention(bad)
    hit = torch.zeros(1, 21, 32, 4, dtype=torch.bool, device="cuda")
    hit[0, 5, :16] = True
    hit[0, 9, 16:] = True
    assert bool(o[hit].isnan().all()) and torch.equal(o[~hit], ref[~hit])
