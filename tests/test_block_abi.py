"""Argument checks of the encoder block's C entry points, which come before any HIP call (CPU)."""
import pytest

from paper_2607_21271_amd import _lib as L

P, Q, R = 1 << 20, 1 << 30, 1 << 40  # never dereferenced


def norm(x=P, w=Q, b=Q + 4096, y=R, rows=3, T=4, C=8, dt=L.EQL_F16):
    return L.eqlinear_group_norm(x, w, b, y, rows, T, C, 1e-6, dt, None)


def attn(qkv=P, o=R, B=1, L_=5, heads=2, D=64, scale=0.125, dt=L.EQL_F16):
    return L.eqlinear_attention(qkv, o, B, L_, heads, D, scale, dt, None)


@pytest.mark.parametrize("kw,status", [
    (dict(dt=3), L.EQL_ERR_INVALID_ARG), (dict(T=0), L.EQL_ERR_INVALID_ARG), (dict(rows=-1), L.EQL_ERR_INVALID_ARG),
    (dict(w=None), L.EQL_ERR_INVALID_ARG), (dict(x=None), L.EQL_ERR_INVALID_ARG), (dict(y=P + 64), L.EQL_ERR_INVALID_ARG),
    (dict(T=17), L.EQL_ERR_UNSUPPORTED), (dict(T=3, C=5), L.EQL_ERR_UNSUPPORTED),
    (dict(C=2049), L.EQL_ERR_UNSUPPORTED), (dict(C=1025, T=8), L.EQL_ERR_UNSUPPORTED),
    (dict(C=1028, dt=L.EQL_F32), L.EQL_ERR_UNSUPPORTED),
    (dict(x=P + 8), L.EQL_ERR_ALIGNMENT), (dict(b=Q + 4097), L.EQL_ERR_ALIGNMENT)])
def test_group_norm_arguments(kw, status):
    assert norm(**kw) == status


@pytest.mark.parametrize("kw,status", [
    (dict(dt=-1), L.EQL_ERR_INVALID_ARG), (dict(L_=0), L.EQL_ERR_INVALID_ARG), (dict(B=-1), L.EQL_ERR_INVALID_ARG),
    (dict(scale=0.0), L.EQL_ERR_INVALID_ARG), (dict(scale=float("nan")), L.EQL_ERR_INVALID_ARG),
    (dict(o=None), L.EQL_ERR_INVALID_ARG), (dict(o=P + 16), L.EQL_ERR_INVALID_ARG),
    (dict(dt=L.EQL_F32), L.EQL_ERR_UNSUPPORTED), (dict(L_=257), L.EQL_ERR_UNSUPPORTED),
    (dict(D=48), L.EQL_ERR_UNSUPPORTED), (dict(qkv=P + 2), L.EQL_ERR_ALIGNMENT)])
def test_attention_arguments(kw, status):
    assert attn(**kw) == status
