"""GPU parity of the forward / input-gradient kernel (csrc/eql_xs.h) against the
fp64 oracle in every form of its plan: one, two and four row tiles, all steps
staged at once or in chunks (the last one odd), outputs split over workgroups,
fewer and more waves than output tiles, channel counts off every tile and
rows that start at half a word (16-bit types, odd T and odd channel counts).

EQL_XS_PLAN=RT,NW,osplit,kc forces a plan; one that the layer cannot run fails the
launch, so a pass that returns ran the named plan.  A plan belongs to one direction:
each case runs the forward of Ci -> Co and the input gradient of the mirrored layer.
Bar as for the layer: max|gpu - oracle| / max|oracle| <= 1e-5 (fp32), 5e-3 (fp16),
4e-2 (bf16).
"""
import pytest

import synth
from gpu_util import TOL, rel_err, run_gpu, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# (T, Ci, Co, N, bias, plan)
CASES = [(1, 33, 17, 130, True, "4,2,1,0"), (1, 160, 40, 67, False, "4,3,1,2"), (2, 70, 100, 65, True, "4,4,2,2"),
         (3, 37, 53, 77, True, "4,2,1,0"), (3, 131, 35, 49, True, "2,4,1,2"), (4, 24, 96, 200, True, "4,2,1,0"),
         (4, 135, 66, 70, True, "4,8,1,2"), (4, 200, 72, 33, False, "1,3,2,4"), (5, 37, 21, 100, True, "2,4,1,0"),
         (5, 101, 50, 40, False, "2,4,1,2"), (6, 130, 40, 45, True, "2,3,1,2"), (7, 39, 53, 95, True, "2,3,2,0"),
         (7, 161, 18, 31, True, "1,2,1,4"), (8, 96, 200, 50, True, "2,4,3,0"), (8, 170, 60, 47, False, "2,4,1,2"),
         (9, 65, 33, 45, True, "1,4,1,2"), (12, 64, 50, 34, True, "1,8,1,0"), (13, 19, 35, 33, True, "1,1,1,0"),
         (15, 97, 40, 18, True, "1,3,1,2"), (16, 48, 70, 17, True, "1,4,5,2"), (16, 64, 16, 1, True, "1,4,1,0")]


def _inputs(T, Ci, Co, N, bias, kind, dt, seed):
    """Inputs of the layer whose pass `kind` contracts Ci channels into Co."""
    Cin, Cout = (Ci, Co) if kind == "y" else (Co, Ci)
    return synth.draw(T, Cin, Cout, N, bias, seed).rounded(dt)


def _oracle(orc, inp, kind):
    return orc.forward(inp.x, inp.w, inp.b) if kind == "y" else orc.backward_input(inp.dy, inp.w)


@pytest.mark.parametrize("dt", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("kind", ["y", "dx"])
@pytest.mark.parametrize("T,Ci,Co,N,bias,plan", CASES, ids=["T%d-%dx%d-N%d-%s-%s" % c for c in CASES])
def test_forced_plans_match_oracle(orc, monkeypatch, T, Ci, Co, N, bias, plan, kind, dt):
    say("xs plan", T, Ci, Co, N, bias, plan, kind, dt)
    monkeypatch.setenv("EQL_XS_PLAN", plan)
    inp = _inputs(T, Ci, Co, N, bias, kind, dt, 9950 + 17 * T + Ci + Co)
    err = rel_err(run_gpu(inp, dt, want=(kind,))[kind], _oracle(orc, inp, kind))
    say("  ", "%.2e" % err)
    assert err <= TOL[dt], err


@pytest.mark.parametrize("kind", ["y", "dx"])
@pytest.mark.parametrize("plan", ["2,4,1,0", "1,3,2,2", "4,4,1,4", "4,4,1,0"])
def test_plans_agree_bitwise(monkeypatch, plan, kind):
    """A plan only deals the work out: every one sums each output in the same
    order, so the bits do not depend on it."""
    inp = _inputs(4, 140, 50, 333, True, kind, "f16", 9990)
    monkeypatch.setenv("EQL_XS_PLAN", "1,8,1,0")
    ref = run_gpu(inp, "f16", want=(kind,))[kind]
    monkeypatch.setenv("EQL_XS_PLAN", plan)
    assert (run_gpu(inp, "f16", want=(kind,))[kind] == ref).all()


@pytest.mark.parametrize("plan", ["4,2,1,4", "8,4,1,0", "1,4,1,3", "4,8,0,1", "1,9,1,0", "nonsense"])
def test_a_plan_the_layer_cannot_run_is_refused(monkeypatch, plan):
    """Four tiles for two waves in chunks, a row tile count without a kernel, an odd chunk, the pipelined form at T = 4,
    nine waves, no plan at all."""
    from paper_2607_21271_amd import _lib
    inp = _inputs(4, 140, 50, 33, True, "y", "f16", 9991)
    monkeypatch.setenv("EQL_XS_PLAN", plan)
    with pytest.raises(_lib.EqlError) as e:
        run_gpu(inp, "f16", want=("y",))
    assert e.value.status == _lib.EQL_ERR_LAUNCH


# The pipelined form: one turn and several a workgroup (16,384 rows are one turn of 256 CUs), a last chunk past the
# channels, ragged rows and widths, one to five staging waves, chunks of one and two steps.
PIPE_CASES = [(384, 96, 130, "4,8,0,1"), (70, 77, 64, "4,7,0,1"), (170, 90, 1, "4,8,0,1"), (33, 65, 16500, "4,8,0,1"),
              (100, 96, 40007, "4,8,0,1"), (131, 50, 201, "4,8,0,2"), (96, 16, 99, "4,6,0,2"), (64, 80, 33000, "4,8,0,1")]


@pytest.mark.parametrize("dt", ["f16", "bf16"])
@pytest.mark.parametrize("kind", ["y", "dx"])
@pytest.mark.parametrize("Ci,Co,N,plan", PIPE_CASES, ids=["%dx%d-N%d-%s" % c for c in PIPE_CASES])
def test_pipelined_form(orc, monkeypatch, Ci, Co, N, plan, kind, dt):
    """Same bits as a plan of one row tile that stages everything at once (every plan sums in the same order); the
    oracle on the smaller ones."""
    say("pipelined", Ci, Co, N, plan, kind, dt)
    T = 8
    inp = _inputs(T, Ci, Co, N, True, kind, dt, 9900 + Ci + Co)
    monkeypatch.setenv("EQL_XS_PLAN", "1,4,1,0")
    ref = run_gpu(inp, dt, want=(kind,))[kind]
    monkeypatch.setenv("EQL_XS_PLAN", plan)
    got = run_gpu(inp, dt, want=(kind,))[kind]
    assert (got == ref).all()
    if N <= 1000:
        err = rel_err(got, _oracle(orc, inp, kind))
        assert err <= TOL[dt], err
