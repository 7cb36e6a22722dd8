"""What the binding takes and what it refuses before anything reaches the library, and that a refused call keeps nothing (host only)."""
import sys
from fractions import Fraction

import numpy as np
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


@pytest.mark.parametrize("kw", [dict(scale="1"), dict(scale=1j), dict(scale=torch.ones(2)), dict(impl=1.0), dict(impl=torch.ones(()))])
def test_refused_numbers(kw):
    for name in ("attn_fwd", "attn_bwd", "decode"):
        with pytest.raises((TypeError, ValueError), match="^(?!tensors handed)"):
            CALLS[name](**kw)
    with pytest.raises(TypeError):
        cb.cart_decode(Q[0], Z, Z, K[0], K[0], CU, 2.5)
    for accumulate in (None, [], "x"):
        with pytest.raises((TypeError, ValueError), match="int"):
            CALLS["attn_bwd"](dz_accumulate=accumulate)


# A number of any kind that a ctypes field takes gets as far as the check of the tensors, here too
INTEGERS = [4, True, np.int64(4), np.uint8(4), torch.tensor(4), torch.tensor([4]), np.array(4)]
REALS = [1, 0.5, np.float32(0.5), np.float64(0.5), np.int64(1), torch.tensor(0.5), torch.tensor([0.5]), Fraction(1, 2)]


@pytest.mark.parametrize("n", INTEGERS, ids=repr)
def test_accepted_integers(n):
    for call in (lambda: CALLS["attn_fwd"](impl=n), lambda: CALLS["attn_bwd"](n_frozen=n), lambda: CALLS["attn_bwd"](impl=n),
                 lambda: CALLS["kl"](mode=n), lambda: cb.cart_teacher_topk(X, n, teacher_idx=IDX, teacher_logp=X),
                 lambda: cb.cart_decode(Q[0], Z, Z, K[0], K[0], CU, n),
                 lambda: cb.cart_decode_composed(Q[0], [], None, None, None, K[0], K[0], CU, n),
                 lambda: cb.cart_decode_static(Q[0], Z, Z, K[0], K[0], CU, n)):
        with pytest.raises(ValueError, match="contiguous device tensors"):
            call()


@pytest.mark.parametrize("x", REALS, ids=repr)
def test_accepted_reals(x):
    for name in ("attn_fwd", "attn_bwd", "decode", "composed"):
        with pytest.raises(ValueError, match="contiguous device tensors"):
            CALLS[name](scale=x)
    with pytest.raises(ValueError, match="contiguous device tensors"):
        cb.cart_distill_kl_fwd_bwd(X, IDX, None, x)


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
