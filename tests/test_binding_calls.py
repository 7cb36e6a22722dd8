"""What the binding refuses before anything reaches the library, and that a refused call keeps nothing (host only)."""
import sys

import pytest
import torch

from paper_2506_06266_amd import binding as cb

Q, K = torch.zeros(2, 8, 4, 64), torch.zeros(2, 8, 2, 64)
Z, CU = torch.zeros(2, 3, 64), torch.zeros(3, dtype=torch.int32)
X, IDX = torch.zeros(4, 64), torch.zeros(4, 2, dtype=torch.int32)

CALLS = {
    "attn_fwd": lambda q=Q, **kw: cb.cart_attn_fwd(q, K, K, Z, Z, **kw),
    "attn_bwd": lambda q=Q, **kw: cb.cart_attn_bwd(q, K, K, Z, Z, Q, X, Q, **kw),
    "kl": lambda q=X, **kw: cb.cart_distill_kl_fwd_bwd(q, IDX, None, 1.0, **kw),
    "topk": lambda q=X, **kw: cb.cart_teacher_topk(q, 2, **kw),
    "decode": lambda q=Q[0], **kw: cb.cart_decode(q, Z, Z, K[0], K[0], CU, 4, **kw),
    "composed": lambda q=Q[0], **kw: cb.cart_decode_composed(q, [], None, None, None, K[0], K[0], CU, 4, **kw),
}


@pytest.mark.parametrize("name", CALLS)
def test_refused_tensors(name):
    call = CALLS[name]
    q = call.__defaults__[0]
    with pytest.raises(ValueError, match="contiguous device tensors"):
        call()                              # host memory
    with pytest.raises(TypeError, match="unsupported dtype"):
        call(q.half())
    with pytest.raises(ValueError):
        call(q[0])                          # a dimension short
    with pytest.raises((TypeError, AttributeError)):
        call(None)
    with pytest.raises((TypeError, AttributeError)):
        call(q.numpy())


@pytest.mark.parametrize("kw", [dict(scale="1"), dict(scale=torch.ones(())), dict(impl=1.0)])
def test_refused_numbers(kw):
    for name in ("attn_fwd", "attn_bwd", "decode"):
        with pytest.raises(TypeError):
            CALLS[name](**kw)
    with pytest.raises(TypeError):
        cb.cart_decode(Q[0], Z, Z, K[0], K[0], CU, 2.5)


def test_refused_segments():
    with pytest.raises(ValueError, match="contiguous device tensors"):
        cb.cart_decode_composed(Q[0], [(Z, Z)], None, None, None, K[0], K[0], CU, 4)
    for shared in (None, [Z], [(Z,)], [(None, Z)]):
        with pytest.raises((TypeError, ValueError, AttributeError)):
            cb.cart_decode_composed(Q[0], shared, None, None, None, K[0], K[0], CU, 4)


def test_accumulating_needs_the_gradients():
    with pytest.raises(ValueError, match="d_z_k"):
        CALLS["attn_bwd"](dz_accumulate=True)


def test_refused_calls_keep_no_references():
    held = [Q, K, Z, X, IDX, CU]
    before = [sys.getrefcount(t) for t in held]
    for _ in range(50):
        for call in CALLS.values():
            with pytest.raises(ValueError):
                call()
    assert [sys.getrefcount(t) for t in held] == before
