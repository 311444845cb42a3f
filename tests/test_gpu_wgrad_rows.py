"""Weight gradient over rows that start at half a word (16-bit types, odd group
orders), against the fp64 oracle.

The kernels read such a row as the aligned words around it.  What can go wrong:
the alignment of a row by the parity of its element offset (odd and even channel
counts of x and dy), the last word of a tensor with an odd number of elements,
and the rows past the end that fill up the last chunk, whose first word would
hold what follows the tensor.  So the tensors here are cut from longer buffers
whose rest is NaN.  Each kernel is forced in turn (EQL_WGRAD_KIND: 0 staged, 1
register-direct; EQL_BWD_FUSED=1: single pass, fp16).  Bar as for the layer.
"""
import pytest

import synth
from gpu_util import TOL, rel_err, say, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _cut(a, dt):
    """a on the device, followed by NaN."""
    t = to_dev(a, dt)
    buf = torch.full((t.numel() + 64,), float("nan"), dtype=t.dtype, device="cuda")
    buf[:t.numel()] = t.flatten()
    return buf[:t.numel()].view(t.shape)


CASES = [(T, *c) for T in (1, 3, 5, 7, 9, 11, 13, 15) for c in ((5, 3, 1), (17, 33, 31), (16, 9, 65), (21, 40, 259))]


@pytest.mark.parametrize("dt", ["f16", "bf16"])
@pytest.mark.parametrize("T,Cin,Cout,N", CASES, ids=["T%d-%dx%d-N%d" % c for c in CASES])
def test_half_word_rows(orc, monkeypatch, T, Cin, Cout, N, dt):
    from paper_2607_21271_amd import ops
    inp = synth.draw(T, Cin, Cout, N, True, 8800 + 31 * T + Cin + Cout).rounded(dt)
    x, dy = _cut(inp.x, dt), _cut(inp.dy, dt)
    dw_ref, db_ref = orc.backward_weight(inp.x, inp.dy)
    for kind in ("0", "1"):
        say("half-word rows", T, Cin, Cout, N, dt, "kind", kind)
        monkeypatch.setenv("EQL_WGRAD_KIND", kind)
        dw, db = ops.backward_weight(x, dy, T, Cin, Cout, with_bias=True)
        errs = {"dw": rel_err(dw.float().cpu().numpy(), dw_ref), "db": rel_err(db.float().cpu().numpy(), db_ref)}
        for k, v in errs.items():
            assert v <= TOL[dt], (kind, k, v)
    monkeypatch.delenv("EQL_WGRAD_KIND")
    if dt == "f16":
        say("  single pass")
        monkeypatch.setenv("EQL_BWD_FUSED", "1")
        wspec = ops.weight_spectrum(to_dev(inp.w, dt))
        dx, dw, db = ops.backward(x, dy, wspec, T, Cin, Cout, with_bias=True)
        assert rel_err(dx.float().cpu().numpy(), orc.backward_input(inp.dy, inp.w)) <= TOL[dt]
        assert rel_err(dw.float().cpu().numpy(), dw_ref) <= TOL[dt]
        assert rel_err(db.float().cpu().numpy(), db_ref) <= TOL[dt]
