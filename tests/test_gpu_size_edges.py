"""Every kernel variant at the sizes where its split can go wrong -- tile edges, remainders, the
smallest and largest of its range, both sides of each dispatch rule -- against the fp64 oracle."""
import numpy as np
import pytest
import torch

from oracle import cartridge_oracle as orc
from paper_2506_06266_amd import binding as cb

pytestmark = pytest.mark.gpu

DEV = "cuda"
# Largest difference over the tensor's largest value.  fp32: sums of up to a few thousand terms in
# another order, far below sqrt(n) 2^-24 x 10.  bf16: the output's rounding (2^-9) plus the bf16
# rounding of P and dS (2^-9 each, relative to the largest term): observed at most 5e-3.
TOL = {torch.float32: 2e-5, torch.bfloat16: 2e-2}


def f64(t):
    return t.detach().to("cpu", torch.float64).numpy()


def rel_err(x, ref):
    x = f64(x)
    assert x.shape == ref.shape and np.isfinite(x).all()
    return float(np.abs(x - ref).max() / max(np.abs(ref).max(), 1e-300))


def attn_case(rows, Hq, Hkv, D, P, dtype, seed):
    g = torch.Generator().manual_seed(seed)
    rn = lambda *sz, std=1.0: (std * torch.randn(*sz, generator=g)).to(dtype)
    return [rn(*rows, Hq, D, std=0.5), rn(*rows, Hkv, D, std=0.5), rn(*rows, Hkv, D), rn(Hkv, P, D, std=0.5),
            rn(Hkv, P, D), rn(*rows, Hq, D)]


def check_attn(q, k, v, zk, zv, do, impl=cb.IMPL_AUTO, n_frozen=0):
    P = zk.shape[1]
    n = [f64(t) for t in (q, k, v, zk, zv, do)]
    ref = list(orc.attn_fwd(*n[:5])) + [x.copy() for x in orc.attn_bwd(*n)]
    for x in ref[5:]:
        x[:, :n_frozen] = 0
    a = [t.to(DEV) for t in (q, k, v, zk, zv)]
    if P == 0:
        a[3:] = [None, None]
    o, lse = cb.cart_attn_fwd(*a, impl=impl)
    out = [o, lse] + list(cb.cart_attn_bwd(*a, o, lse, do.to(DEV), impl=impl, n_frozen=n_frozen))
    torch.cuda.synchronize()
    for nm, x, r in list(zip(["o", "lse", "d_q", "d_k", "d_v", "d_zk", "d_zv"], out, ref))[: 5 if P == 0 else 7]:
        if np.abs(r).max() < 1e-12:     # a softmax over one key: the exact gradient is 0
            assert np.abs(f64(x)).max() < 1e-2, nm
            continue
        e = rel_err(x, r)
        assert e <= TOL[q.dtype], (nm, e)


# The forward and dQ workgroups hold four (64 tokens, query head) units of one KV head: groupings
# that divide four, that straddle two token blocks, that exceed four, with sequences ending inside,
# at and just past a block of 64 tokens.
@pytest.mark.parametrize("B,S,Hq,Hkv,P", [(2, 65, 3, 1, 70), (1, 129, 6, 2, 0), (1, 64, 5, 1, 64), (2, 63, 7, 1, 33),
                                          (1, 193, 12, 2, 130), (1, 320, 1, 1, 5), (3, 1, 4, 1, 3)])
def test_attention_query_blocks(B, S, Hq, Hkv, P):
    check_attn(*attn_case((B, S), Hq, Hkv, 128, P, torch.bfloat16, 31 * S + Hq), impl=cb.IMPL_MFMA)
