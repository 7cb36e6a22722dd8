"""Every kernel variant at the sizes where its split can go wrong -- tile edges, remainders, the
smallest and largest of its range, both sides of each dispatch rule -- against the fp64 oracle."""
import numpy as np
import pytest
import torch

from oracle import cartridge_oracle as orc
from paper_2506_06266_amd import binding as cb
from paper_2506_06266_amd import synth
from test_backward_plan import plan

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


def best_us(call, runs=5):
    call()
    best = float("inf")
    for _ in range(runs):
        t = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        t[0].record()
        call()
        t[1].record()
        t[1].synchronize()
        best = min(best, 1e3 * t[0].elapsed_time(t[1]))
    return best


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



# Sequences of one or two units (64 tokens of one query head of the group), enough of them that blocks run whole:
# one wavefront's rows or two's, a unit of one row, and just past two units.
@pytest.mark.parametrize("B,S,Hq,Hkv,P", [(300, 64, 1, 1, 3), (270, 65, 1, 1, 64), (260, 128, 2, 2, 5), (260, 33, 2, 1, 70), (280, 1, 2, 1, 1),
                                          (260, 129, 1, 1, 3), (260, 64, 3, 1, 3), (130, 40, 4, 2, 0)])
def test_attention_of_many_short_sequences(B, S, Hq, Hkv, P):
    check_attn(*attn_case((B, S), Hq, Hkv, 128, P, torch.bfloat16, 13 * S + P), impl=cb.IMPL_MFMA)


# Small launches: query blocks split along their key tiles (forward, dQ), the key-stationary kernel cut
# into chunks of token rows and parts of the heads.  Many short parts, parts with a ragged prefix tile
# or nothing but masked tiles, blocks of one part among split ones, no prefix, one token block, a
# split last round after a whole one (the last shape: 36 blocks of one KV head's 32).
@pytest.mark.parametrize("B,S,Hq,Hkv,P", [(1, 300, 4, 1, 700), (1, 700, 8, 2, 0), (2, 500, 3, 1, 129), (1, 64, 2, 2, 2000),
                                          (1, 65, 1, 1, 63), (1, 1000, 4, 1, 5), (1, 129, 8, 1, 1024), (9, 250, 32, 8, 321)])
def test_attention_small_launches(B, S, Hq, Hkv, P):
    check_attn(*attn_case((B, S), Hq, Hkv, 128, P, torch.bfloat16, 7 * S + P), impl=cb.IMPL_MFMA, n_frozen=min(P, 3))


# Backward in one launch: own-key blocks all ahead of dQ's blocks, all behind them, some of either (one sequence of 2100
# tokens), dQ whole and split beside chunks of the token rows and parts of the heads; and in two (more blocks than the CUs of
# a KV head take in four rounds; above, the smaller launches no longer come there).
@pytest.mark.parametrize("B,S,Hq,Hkv,P", [(4, 200, 8, 2, 300), (3, 130, 8, 1, 900), (1, 300, 24, 8, 0), (1, 2100, 2, 1, 200), (140, 24, 4, 4, 3),
                                          (130, 40, 32, 8, 70)])
def test_attention_backward_launches(B, S, Hq, Hkv, P):
    check_attn(*attn_case((B, S), Hq, Hkv, 128, P, torch.bfloat16, 5 * S + P), impl=cb.IMPL_MFMA, n_frozen=min(P, 1))


# Scores that overflow the forward's fixed softmax reference (one key 200 nats above the first ones): rows
# computed again by the wavefront itself where blocks run whole (whole rounds of 32 blocks per KV head; rows of
# 1 .. 127 keys, around the eight taken at a time) and by the finishing kernel where they are split.
@pytest.mark.parametrize("B,S,Hq,Hkv,P,hot", [(32, 40, 8, 8, 87, 7), (32, 70, 16, 8, 41, 33), (32, 9, 8, 8, 32, 0), (1, 300, 8, 1, 600, 100)])
def test_attention_forward_recomputes_overflowing_rows(B, S, Hq, Hkv, P, hot):
    g = torch.Generator().manual_seed(S)
    u = torch.randn(128, generator=g)
    u *= (200.0 * 128 ** 0.5) ** 0.5 / u.norm()
    rn = lambda *sz, std=1.0: std * torch.randn(*sz, generator=g)
    q, k = u + rn(B, S, Hq, 128, std=0.05), rn(B, S, Hkv, 128, std=0.05)
    k[:, hot] += u
    t = [x.to(torch.bfloat16) for x in (q, k, rn(B, S, Hkv, 128), rn(Hkv, P, 128, std=0.05), rn(Hkv, P, 128))]
    o_ref, lse_ref = orc.attn_fwd(*[f64(x) for x in t])
    o, lse = cb.cart_attn_fwd(*[x.to(DEV) for x in t], impl=cb.IMPL_MFMA)
    torch.cuda.synchronize()
    assert rel_err(o, o_ref) <= TOL[torch.bfloat16] and rel_err(lse, lse_ref) <= TOL[torch.bfloat16]


# (the last: backward in two launches)
@pytest.mark.parametrize("lens,Hq,Hkv,P", [([700, 1, 90], 4, 1, 300), ([64, 64, 64], 2, 2, 1000), ([5, 3, 400, 131], 4, 2, 0),
                                           ([29] * 295, 32, 8, 20)])
def test_packed_small_launches(lens, Hq, Hkv, P):
    q, k, v, zk, zv, do = attn_case((sum(lens),), Hq, Hkv, 128, P, torch.bfloat16, sum(lens) + P)
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32)
    n = [f64(t) for t in (q, k, v, zk, zv, do)]
    ref = list(orc.attn_varlen_fwd(*n[:5], cu.numpy())) + list(orc.attn_varlen_bwd(*n, cu.numpy()))
    a = [t.to(DEV) for t in (q, k, v, zk, zv, cu)]
    if P == 0:
        a[3] = a[4] = None
    o, lse = cb.cart_attn_varlen_fwd(*a, max(lens))
    out = [o, lse] + list(cb.cart_attn_varlen_bwd(*a, max(lens), o, lse, do.to(DEV)))
    torch.cuda.synchronize()
    for x, r in list(zip(out, ref))[: 5 if P == 0 else 7]:
        assert rel_err(x, r) <= TOL[torch.bfloat16]



# A packed launch of more than one round of blocks: 35 blocks of a KV head's 32 CUs, the 32 with the last rows run whole and
# the first 192 rows are split along the prefix (its last tile ragged).  HOT: one key 200 nats above the first ones,
# in the last sequence, whose rows lie in whole blocks, and in the first one, whose rows are split.
MIXED_LENS, MIXED_P = [64, 300, 500, 1, 70, 640, 200, 465], 1501


def mixed_case(hot):
    T, Hq, Hkv = sum(MIXED_LENS), 32, 8
    q, k, v, zk, zv, do = attn_case((T,), Hq, Hkv, 128, MIXED_P, torch.bfloat16, 77)
    if hot:
        g = torch.Generator().manual_seed(3)
        u = torch.randn(128, generator=g)
        u *= (200.0 * 128 ** 0.5) ** 0.5 / u.norm()
        q = (u + 0.05 * torch.randn(T, Hq, 128, generator=g)).to(torch.bfloat16)
        zk = (0.05 * torch.randn(Hkv, MIXED_P, 128, generator=g)).to(torch.bfloat16)
        k = 0.05 * torch.randn(T, Hkv, 128, generator=g)
        k[[9, T - 400]] += u
        k = k.to(torch.bfloat16)
    cu = torch.tensor(np.concatenate([[0], np.cumsum(MIXED_LENS)]), dtype=torch.int32)
    return [q, k, v, zk, zv, cu], do


def test_packed_whole_and_split_blocks():
    a, do = mixed_case(False)
    n = [f64(t) for t in a[:5]]
    ref = [*orc.attn_varlen_fwd(*n, a[5].numpy()), *orc.attn_varlen_bwd(*n, f64(do), a[5].numpy())]
    d = [t.to(DEV) for t in a]
    o, lse = cb.cart_attn_varlen_fwd(*d, max(MIXED_LENS))
    out = [o, lse, *cb.cart_attn_varlen_bwd(*d, max(MIXED_LENS), o, lse, do.to(DEV))]
    torch.cuda.synchronize()
    for x, r in zip(out, ref):
        assert rel_err(x, r) <= TOL[torch.bfloat16]


def test_packed_whole_and_split_blocks_overflowing():
    a, _ = mixed_case(True)
    o_ref, lse_ref = orc.attn_varlen_fwd(*[f64(t) for t in a[:5]], a[5].numpy())
    o, lse = cb.cart_attn_varlen_fwd(*[t.to(DEV) for t in a], max(MIXED_LENS))
    torch.cuda.synchronize()
    T = sum(MIXED_LENS)
    assert lse_ref[:, T - 300].min() > 150 and lse_ref[:, 20].min() > 150 and lse_ref[:, 100].max() < 20
    assert rel_err(o, o_ref) <= TOL[torch.bfloat16] and rel_err(lse, lse_ref) <= TOL[torch.bfloat16]


# The fp32 kernels (any head_dim up to 256; bf16 inputs widened): head sizes around the operand blocks
# of 16 and the three register layouts, tokens and slots around the blocks of 16, one token, no prefix.
VECTOR_CASES = [(torch.float32, 2, 17, 2, 1, 5, 33), (torch.float32, 1, 16, 4, 2, 16, 16), (torch.float32, 3, 1, 2, 2, 64, 1),
                (torch.float32, 2, 130, 4, 1, 64, 0), (torch.float32, 1, 65, 3, 1, 66, 15), (torch.float32, 2, 31, 2, 1, 128, 140),
                (torch.float32, 1, 33, 2, 1, 132, 20), (torch.float32, 1, 20, 2, 1, 256, 17), (torch.bfloat16, 2, 40, 4, 2, 64, 50),
                (torch.bfloat16, 1, 18, 2, 1, 37, 9), (torch.bfloat16, 1, 70, 2, 2, 128, 0),
                # a wavefront's blocks of token rows in dK / dV: many and not all wavefronts the same, head_dim below its registers'
                (torch.float32, 3, 50, 4, 1, 100, 33), (torch.float32, 3, 45, 4, 1, 40, 20), (torch.bfloat16, 5, 19, 3, 1, 72, 40),
                # ... and the prefix blocks' split into parts, of different lengths
                (torch.float32, 5, 40, 6, 2, 64, 35), (torch.float32, 3, 70, 4, 1, 128, 20), (torch.bfloat16, 7, 33, 4, 2, 200, 17),
                (torch.float32, 9, 20, 8, 1, 33, 3),
                # (two launches below head_dim 129: many blocks; one query head a KV head.  The last two just below each line)
                (torch.float32, 5, 130, 16, 16, 33, 0), (torch.bfloat16, 6, 121, 16, 16, 64, 9), (torch.float32, 4, 61, 16, 16, 128, 0),
                (torch.float32, 3, 76, 16, 16, 65, 0), (torch.float32, 4, 140, 16, 16, 64, 0), (torch.float32, 2, 81, 16, 16, 112, 0)]


@pytest.mark.parametrize("dtype,B,S,Hq,Hkv,D,P", VECTOR_CASES, ids=lambda v: str(v).replace("torch.", ""))
def test_attention_vector(dtype, B, S, Hq, Hkv, D, P):
    check_attn(*attn_case((B, S), Hq, Hkv, D, P, dtype, S + D), impl=cb.IMPL_VECTOR, n_frozen=min(P, 2))


def test_attention_vector_split_prefix_accumulates():
    t = attn_case((4, 40), 8, 2, 64, 20, torch.float32, 1)
    ref = orc.attn_bwd(*[f64(x) for x in t])[3:]
    q, k, v, zk, zv, do = (x.to(DEV) for x in t)
    o, lse = cb.cart_attn_fwd(q, k, v, zk, zv)
    gk, gv = (torch.ones(2, 20, 64, device=DEV) for _ in range(2))
    cb.cart_attn_bwd(q, k, v, zk, zv, o, lse, do, d_z_k=gk, d_z_v=gv, dz_accumulate=True, n_frozen=3)
    torch.cuda.synchronize()
    for g, r in zip((gk, gv), ref):
        assert (g[:, :3] == 1).all() and rel_err(g[:, 3:] - 1, r[:, 3:]) <= 5 * TOL[torch.float32]    # (and the sum with 1: 2^-24 of it)


# A NaN or an infinity reaches exactly the results whose sums hold it: tokens 11 .. leave the rows before
# them alone (padding behind a sequence's end), tokens .. 4 the gradients of the keys behind them.
@pytest.mark.parametrize("D", [64, 128, 256])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_attention_vector_hidden_nonfinite(D, bad):
    t = attn_case((2, 21), 2, 1, D, 5, torch.float32, D)
    n = [f64(x) for x in t]
    o_ref, lse_ref = orc.attn_fwd(*n[:5])
    g_ref = orc.attn_bwd(*n)
    q, k, v, zk, zv, do = (x.to(DEV) for x in t)
    o0, lse0 = cb.cart_attn_fwd(q, k, v, zk, zv, impl=cb.IMPL_VECTOR)
    kb, vb = k.clone(), v.clone()
    kb[:, 11:] = bad
    vb[:, 11:] = bad
    o, lse = cb.cart_attn_fwd(q, kb, vb, zk, zv, impl=cb.IMPL_VECTOR)
    dq = cb.cart_attn_bwd(q, kb, vb, zk, zv, o0, lse0, do, impl=cb.IMPL_VECTOR)[0]
    qb, db = q.clone(), do.clone()
    qb[:, :5] = bad
    db[:, :5] = bad
    _, dk, dv, _, _ = cb.cart_attn_bwd(qb, k, v, zk, zv, o0, lse0, db, impl=cb.IMPL_VECTOR)
    torch.cuda.synchronize()
    tol = TOL[torch.float32]
    assert rel_err(o[:, :11], o_ref[:, :11]) <= tol and rel_err(lse[:, :, :11], lse_ref[:, :, :11]) <= tol
    assert rel_err(dq[:, :11], g_ref[0][:, :11]) <= tol
    assert rel_err(dk[:, 5:], g_ref[1][:, 5:]) <= tol and rel_err(dv[:, 5:], g_ref[2][:, 5:]) <= tol
    assert not torch.isfinite(o[:, 11:]).any() and not torch.isfinite(dk[:, :5]).any()
    if bad != bad:
        assert torch.isnan(o[:, 11:]).all() and torch.isnan(dq[:, 11:]).all() and torch.isnan(dv[:, :5]).all()


# Loss: every width of the row kernel at its last size and just past it, rows that start at every
# offset from a 16-byte boundary and a 128-byte line (odd vocabularies), more records than threads, more rows than the
# launch has workgroups.  (data type, rows, vocabulary, records)
LOSS_CASES = [
    (torch.bfloat16, 9, 5, 3), (torch.bfloat16, 5, 4096, 20), (torch.bfloat16, 9, 4107, 200), (torch.bfloat16, 3, 8199, 20),
    (torch.bfloat16, 3, 32768, 20), (torch.bfloat16, 9, 32777, 300), (torch.bfloat16, 5, 65543, 20),
    (torch.bfloat16, 2, 131079, 20), (torch.bfloat16, 3, 140003, 20), (torch.bfloat16, 4100, 131, 4),
    (torch.float32, 7, 3, 2), (torch.float32, 5, 2048, 140), (torch.float32, 5, 2055, 20), (torch.float32, 5, 4099, 20),
    (torch.float32, 3, 16385, 20), (torch.float32, 3, 32771, 20), (torch.float32, 2, 65536, 20), (torch.float32, 5, 65541, 1024),
    (torch.float32, 300, 65541, 5), (torch.float32, 3, 98307, 20), (torch.float32, 3, 120001, 20), (torch.float32, 2050, 2060, 4),
    # (slots counted from a 128-byte line, up to seven more than vectors: the fullest rows of each width)
    (torch.bfloat16, 9, 4047, 20), (torch.bfloat16, 9, 4049, 20), (torch.bfloat16, 9, 32719, 20), (torch.bfloat16, 9, 65487, 20),
    (torch.bfloat16, 9, 131023, 20), (torch.float32, 33, 2023, 20), (torch.float32, 33, 16359, 20), (torch.float32, 9, 98279, 20),
    # what is not resident: one turn, just more, more turns than are requested ahead, several rows a workgroup
    (torch.float32, 3, 102400, 20), (torch.float32, 3, 102407, 20), (torch.float32, 65, 102407, 5), (torch.float32, 3, 131072, 20),
    (torch.float32, 300, 114697, 5), (torch.float32, 2, 135165, 20),
    (torch.bfloat16, 3, 163851, 20), (torch.bfloat16, 270, 172032, 5),
    # a turn at a time or ahead: rows on half of the CUs from three turns on, on fewer from as many as make 512 with the rows, or thirteen
    (torch.float32, 128, 106496, 5), (torch.float32, 128, 106499, 5), (torch.float32, 127, 106499, 5), (torch.float32, 3, 147459, 20),
    (torch.bfloat16, 128, 147463, 5), (torch.bfloat16, 2, 229376, 20), (torch.bfloat16, 2, 229385, 20),
    (torch.float32, 128, 106500, 5), (torch.float32, 127, 106500, 5), (torch.float32, 64, 128256, 5), (torch.float32, 63, 128256, 5),
    (torch.float32, 3, 147460, 20), (torch.bfloat16, 128, 147464, 5), (torch.bfloat16, 43, 229376, 5), (torch.bfloat16, 42, 229376, 5),
]


@pytest.mark.parametrize("dtype,N,V,K", LOSS_CASES, ids=lambda v: str(v).replace("torch.", ""))
def test_loss_rows(dtype, N, V, K):
    g = torch.Generator().manual_seed(V + K)
    x = (3.0 * torch.randn(N, V, generator=g)).to(dtype)
    if V > 1000:
        x[0, V // 2:] = float("-inf")              # a masked tail
        x[-1] = x[-1] + 60.0                        # far from 0
    idx = torch.stack([torch.randperm(V // 2 if n == 0 and V > 1000 else V, generator=g)[:K] for n in range(N)]).to(torch.int32)
    lp = torch.log_softmax(2.0 * torch.randn(N, K, generator=g), 1) - 0.1
    idx[-1, 0] = -1
    scale = 1.0 / N
    xs, fin = f64(x), torch.isfinite(x).numpy()
    for mode, ref in ((cb.KL_TOPK, orc.distill_kl), (cb.KL_REST, orc.distill_kl_rest_bucket)):
        loss_ref, dl_ref, kl_ref = ref(np.where(fin, xs, -1e4), idx.numpy(), f64(lp), scale)
        d = x.to(DEV)
        row = torch.empty(N, device=DEV)
        loss, dl = cb.cart_distill_kl_fwd_bwd(d, idx.to(DEV), lp.to(DEV), scale, mode=mode, row_kl=row)
        loss2, dl2 = cb.cart_distill_kl_fwd_bwd(d, idx.to(DEV), lp.to(DEV), scale, mode=mode, d_logits=d)   # in place
        torch.cuda.synchronize()
        assert torch.equal(dl, dl2) and torch.equal(loss, loss2)
        # rest bucket: the student's mass off the records is 1 - S in fp32, an error of a few 2^-24
        # in a difference of order min(1 - S) (small only where nearly every token is recorded)
        p = np.exp(xs - xs.max(1, keepdims=True))
        rec = idx.numpy() >= 0
        off = 1.0 - (np.take_along_axis(p, np.maximum(idx.numpy(), 0), 1) * rec).sum(1) / p.sum(1)
        ill = 2.0 ** -22 / off.min() if mode == cb.KL_REST else 0.0
        assert rel_err(dl, dl_ref) <= TOL[dtype] + ill
        assert abs(loss.item() - loss_ref) <= (1e-4 + ill) * max(abs(loss_ref), 1e-3)
        assert rel_err(row, kl_ref) <= 1e-4 + ill


# The records of a row are passed by all of its threads: a thousand of them may cost a few times the row, not more
# (3.4 and 2.4 times the 20 records' time; 8.2 and 7.3 with one record after the other).
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "f32"])
def test_loss_time_of_many_records(dtype):
    N, V = 4096, 32000
    x = torch.randn(N, V, device=DEV).to(dtype)
    d = torch.empty_like(x)
    us = []
    for K in (20, 1000):
        idx = torch.arange(K, dtype=torch.int32, device=DEV).expand(N, K).contiguous()
        lp = torch.full((N, K), -8.0, device=DEV)
        us.append(best_us(lambda: cb.cart_distill_kl_fwd_bwd(x, idx, lp, 1.0, d_logits=d)))
    assert us[1] < 5.0 * us[0], us


# Rows of more than 2 GB (bf16; the second starts inside a 128-byte line) and more than 4 GB (fp32): past what
# a 31-bit and a 32-bit offset reach.
@pytest.mark.parametrize("dtype,N,V", [(torch.bfloat16, 2, 2 ** 30 + 9), (torch.float32, 1, 2 ** 30 + 5)], ids=["bf16", "f32"])
def test_loss_rows_past_two_and_four_gigabytes(dtype, N, V):
    chunk = 2 ** 26
    x = torch.empty(N, V, dtype=dtype, device=DEV)
    g = torch.Generator(device=DEV).manual_seed(V)
    for n in range(N):
        for c in x[n].split(chunk):
            c.copy_(torch.randn(c.numel(), generator=g, device=DEV))
    idx = torch.tensor([[3, V // 2 + 1, V - 2]] * N, dtype=torch.int32, device=DEV)
    lp = torch.log(torch.tensor([[0.5, 0.3, 0.1]] * N, device=DEV))
    scale = float(2 ** 30)
    row = torch.empty(N, device=DEV)
    loss, dl = cb.cart_distill_kl_fwd_bwd(x, idx, lp, scale, row_kl=row)
    t, M = lp.double().exp(), lp.double().exp().sum(1)
    for n in range(N):
        lse = torch.logsumexp(torch.stack([torch.logsumexp(c.double(), 0) for c in x[n].split(chunk)]), 0)
        kl = (t[n] * (lp[n].double() - x[n, idx[n].long()].double() + lse)).sum()
        assert abs(row[n].item() - kl.item()) <= 1e-4 * abs(kl.item())
        for c0 in range(0, V, chunk):
            ref = scale * M[n] * torch.exp(x[n, c0:c0 + chunk].double() - lse)
            for j in range(3):
                i = int(idx[n, j]) - c0
                if 0 <= i < ref.numel():
                    ref[i] -= scale * t[n, j]
            got = dl[n, c0:c0 + chunk].double()
            # (every element on its own: one rounding of the result, and the exponent's rounding, 2^-24 of |x log2 e - lse2| < 64)
            assert ((got - ref).abs() <= (2.0 ** -8 if dtype == torch.bfloat16 else 2e-5) * ref.abs()).all(), (n, c0)


# Teacher records: the three widths of the row kernel at and past their last size, rows starting at
# every offset, K at the edges of the widths and beyond the finite logits of a row, rows made of ties.
TOPK_CASES = [
    (torch.bfloat16, 9, 33, 20), (torch.bfloat16, 9, 4099, 128), (torch.bfloat16, 5, 32771, 129), (torch.bfloat16, 3, 32775, 20),
    (torch.bfloat16, 3, 98311, 256), (torch.bfloat16, 3, 98320, 64), (torch.bfloat16, 9, 131, 131), (torch.bfloat16, 3, 20003, 512),
    (torch.float32, 9, 7, 7), (torch.float32, 5, 16387, 128), (torch.float32, 5, 16389, 20), (torch.float32, 3, 49155, 257),
    (torch.float32, 3, 49161, 20), (torch.float32, 2, 130001, 64),
    # more records than vectors, all of a row, as many as threads
    (torch.bfloat16, 5, 1024, 1024), (torch.bfloat16, 5, 4096, 600), (torch.bfloat16, 3, 32000, 1000), (torch.bfloat16, 3, 8195, 1023),
    (torch.float32, 5, 1025, 1024), (torch.float32, 5, 2003, 1000), (torch.float32, 3, 5000, 1024), (torch.float32, 9, 3, 1), (torch.float32, 9, 30, 29),
]


@pytest.mark.parametrize("dtype,N,V,K", TOPK_CASES, ids=lambda v: str(v).replace("torch.", ""))
def test_topk_rows(dtype, N, V, K):
    g = torch.Generator().manual_seed(V + K)
    x = 3.0 * torch.randn(N, V, generator=g)
    x[1] = torch.round(x[1])                                   # thousands of ties at every level
    if V > 100:
        x[-1] = -1.0e4                                         # few logits above the rest, at both ends of the row
        x[-1, :3], x[-1, -3:] = 1.0, 1.0
    x = x.to(dtype)
    idx_ref, lp_ref = orc.teacher_topk(f64(x), K)
    idx, lp = cb.cart_teacher_topk(x.to(DEV), K)
    torch.cuda.synchronize()
    assert np.array_equal(idx.cpu().numpy().astype(np.int64), idx_ref)
    assert np.abs(f64(lp) - lp_ref).max() <= 2e-6 * max(1.0, np.abs(lp_ref).max())


# As many records as logits: the time may be some tens of times that of 20 of them, not hundreds (22; 1275 with a pass
# over the row for every record).
def test_topk_time_of_all_records():
    x = torch.randn(4096, 1024, device=DEV).to(torch.bfloat16)
    us = [best_us(lambda: cb.cart_teacher_topk(x, K)) for K in (20, 1024)]
    assert us[1] < 100.0 * us[0], us


# fp32 rows of many records: a tenth more of them must not list the row's better half (47 and 68; 63 and 323 with a bound that K + K / 4 + 8 maxima reach)
def test_topk_time_of_many_fp32_records():
    x = torch.randn(128, 16384, device=DEV)
    us = [best_us(lambda: cb.cart_teacher_topk(x, K)) for K in (700, 800)]
    assert us[1] < 2.5 * us[0], us


# Rows with fewer finite logits than records (the lowest indices of the rest follow), of one value, of two with the
# border inside the records; signed zeros are one value.
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "f32"])
@pytest.mark.parametrize("V,K", [(700, 300), (9001, 40), (20000, 700)])
def test_topk_rows_of_few_values(dtype, V, K):
    x = torch.zeros(6, V)
    x[0] = float("-inf")
    x[0, torch.randperm(V, generator=torch.Generator().manual_seed(V))[:K // 2]] = torch.randn(K // 2)
    x[1] = -3.5
    x[2] = 12.0
    x[3, 1::2] = -0.0
    x[4, V - K // 2:] = 1.0
    x[5] = -1.0
    x[5, ::7] = -0.5
    x = x.to(dtype)
    idx, lp = cb.cart_teacher_topk(x.to(DEV), K)
    xs = np.where(x.float().numpy() == 0, 0.0, f64(x))
    ref = np.argsort(-xs, axis=1, kind="stable")[:, :K]
    assert np.array_equal(idx.cpu().numpy(), ref)
    with np.errstate(divide="ignore"):
        top = xs.max(1, keepdims=True)
        want = np.take_along_axis(xs, ref, 1) - top - np.log(np.exp(xs - top).sum(1, keepdims=True))
    got, fin = f64(lp), np.isfinite(want)
    # (fp32: the log-sum-exp's rounding, 2^-23 of at most 24, and its sum's, a few 2^-24)
    assert (got[~fin] == want[~fin]).all() and np.abs(got[fin] - want[fin]).max() <= 5e-6


# Decode: streamed ranges that cross from own rows into private cartridges and from one cartridge to
# the next, requests without one in between, cartridges shorter than a step and longer than a range,
# the merge with four wavefronts a row (few rows) and with one, a request cut into the most ranges.
DECODE_CASES = [
    # B, Hq, Hkv, shared slots, pool slots, longest own
    (3, 4, 1, 0, 1, 40), (5, 8, 2, 33, 31, 70), (6, 8, 2, 700, 64, 1), (4, 6, 3, 100, 777, 65), (40, 8, 1, 64, 40, 3),
    (70, 32, 8, 65, 33, 20), (2, 2, 1, 10, 3000, 5000), (1, 7, 1, 1, 0, 4161), (64, 32, 2, 0, 0, 90),
    # ranges of about one short request: of 8 rows, one row each, more requests than ranges
    (31, 32, 8, 100, 0, 12), (130, 4, 2, 40, 0, 1), (500, 8, 8, 33, 0, 30), (300, 16, 16, 0, 0, 100),
    # own rows and private cartridges cut at different lengths: short requests beside long cartridges, cartridges of a
    # slot or two, one long request among them
    (200, 16, 8, 47, 786, 20), (223, 8, 8, 100, 1, 9), (60, 8, 1, 0, 7, 2), (30, 4, 2, 10, 3, 2000), (5, 8, 8, 0, 33, 300),
    # ranges of one step: few requests, the longest one that has them and one just past it, ranges that straddle requests
    (4, 32, 8, 2048, 0, 150), (3, 8, 2, 200, 0, 512), (3, 8, 2, 200, 0, 513), (9, 8, 2, 0, 0, 33), (20, 6, 2, 70, 0, 100),
]


@pytest.mark.parametrize("B,Hq,Hkv,P,pool_p,most", DECODE_CASES)
def test_decode_ranges(B, Hq, Hkv, P, pool_p, most):
    g = torch.Generator().manual_seed(B + P + pool_p)
    rn = lambda *sz, std=1.0: (std * torch.randn(*sz, generator=g)).to(torch.bfloat16)
    lens = torch.randint(1, most + 1, (B,), generator=g)
    lens[-1] = most
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lens.numpy())]), dtype=torch.int32)
    q, k, v = rn(B, Hq, 128, std=0.6), rn(int(cu[-1]), Hkv, 128, std=0.6), rn(int(cu[-1]), Hkv, 128)
    shared = [(rn(Hkv, P, 128, std=0.6), rn(Hkv, P, 128))] if P else []
    pk = pv = cid = None
    if pool_p:
        pk, pv = rn(3, Hkv, pool_p, 128, std=0.6), rn(3, Hkv, pool_p, 128)
        cid = torch.tensor([(2 * b) % 4 - 1 if b % 5 else -1 for b in range(B)], dtype=torch.int32)   # some without, some shared
    dv = lambda t: None if t is None else t.to(DEV)
    o, lse = cb.cart_decode_composed(dv(q), [(dv(a), dv(b)) for a, b in shared], dv(pk), dv(pv), dv(cid), dv(k), dv(v), dv(cu), most)
    torch.cuda.synchronize()
    z = lambda t: None if t is None else f64(t)
    o_ref, lse_ref = orc.decode_composed(f64(q), [(f64(a), f64(b)) for a, b in shared], z(pk), z(pv),
                                         None if cid is None else cid.numpy(), f64(k), f64(v), cu.numpy())
    assert rel_err(o, o_ref) <= TOL[torch.bfloat16] and rel_err(lse, lse_ref) <= TOL[torch.bfloat16]


# The row maximum of bf16 logits comes from their bits: rows without a positive logit, of zeros of both signs, with one positive at either end,
# masked ones; full, short and odd rows of every width of the workgroup
@pytest.mark.parametrize("V", [5, 64, 1000, 4104, 9001, 20000, 32768, 50257, 65537, 131073])
def test_loss_row_maxima(V):
    g = torch.Generator().manual_seed(V)
    x = -4.0 - 3.0 * torch.rand(8, V, generator=g)
    x[1] = torch.where(torch.rand(V, generator=g) < 0.5, 0.0, -0.0)
    x[2, 0], x[3, -1] = 2.5, 2.5
    x[4, V // 2] = -0.0
    x[5, : V // 2] = float("-inf")
    x[6] = -300.0                        # (at 30000 the log-sum-exp's rounding in 32 bits, 2^-10, is more than the bound below)
    x[7] = 3.0 * torch.randn(V, generator=g)
    x = x.to(torch.bfloat16)
    K = min(3, V)
    idx = torch.stack([torch.randperm(V, generator=g)[:K] for _ in range(8)]).to(torch.int32)
    idx[5] = V - 1 - torch.arange(K, dtype=torch.int32)        # (a recorded token of probability 0 has no finite divergence)
    logp = torch.log_softmax(torch.randn(8, K, generator=g), 1) + float(np.log(0.9))
    row = torch.empty(8, dtype=torch.float32, device=DEV)
    loss, dl = cb.cart_distill_kl_fwd_bwd(x.to(DEV), idx.to(DEV), logp.to(DEV), 1.0 / 8, row_kl=row)
    torch.cuda.synchronize()
    l_ref, dl_ref, row_ref = orc.distill_kl(f64(x), idx.numpy(), f64(logp), 1.0 / 8)
    assert np.abs(f64(row) - row_ref).max() <= 1e-4 * np.abs(row_ref).max() and abs(loss.item() - l_ref) <= 1e-4 * abs(l_ref)
    for n in range(8):
        assert rel_err(dl[n], dl_ref[n]) <= TOL[torch.bfloat16], n


# A wrong maximum of a thread's logits shows only where one of them lies further above the rest than an exponential of 32 bits reaches: single
# logits 250 above the others, at every element of a vector, in the first, the middle and the last ones, and in one of 32 vectors anywhere
@pytest.mark.parametrize("base,top", [(-200.0, 50.0), (-300.0, -50.0)])
@pytest.mark.parametrize("dtype,V", [(torch.bfloat16, v) for v in (64, 1000, 4104, 9001, 20000, 32768, 50257, 65537, 131073)] + [(torch.float32, v) for v in (1000, 50257, 100003)])
def test_loss_maxima_far_above_the_rest(dtype, V, base, top):
    e = 8 if dtype == torch.bfloat16 else 4
    g = torch.Generator().manual_seed(V)
    at = [[v * e + i] for v in (0, V // e // 2, V // e - 1) for i in range(e)] + [[V - 1]]
    for _ in range(16):
        v = torch.randperm(V // e, generator=g)[:max(1, V // e // 32)]
        at.append((v * e + torch.randint(0, e, v.shape, generator=g)).tolist())
    N, K = len(at), 3
    x = base + 8.0 * torch.rand(N, V, generator=g)
    for n, p in enumerate(at):
        x[n, p] = top + torch.rand(len(p), generator=g)
    x = x.to(dtype)
    idx = torch.stack([torch.randperm(V, generator=g)[:K] for _ in range(N)]).to(torch.int32)
    idx[::2, 0] = torch.tensor([p[0] for p in at[::2]], dtype=torch.int32)
    idx[::2, 1:] = (idx[::2, :1] + torch.tensor([[V // 3, V // 2]], dtype=torch.int32)) % V
    logp = torch.log_softmax(torch.randn(N, K, generator=g), 1) + float(np.log(0.9))
    row = torch.empty(N, dtype=torch.float32, device=DEV)
    loss, dl = cb.cart_distill_kl_fwd_bwd(x.to(DEV), idx.to(DEV), logp.to(DEV), 1.0 / N, row_kl=row)
    torch.cuda.synchronize()
    l_ref, dl_ref, row_ref = orc.distill_kl(f64(x), idx.numpy(), f64(logp), 1.0 / N)
    assert rel_err(row, row_ref) <= 1e-4 and abs(loss.item() - l_ref) <= 1e-4 * abs(l_ref)
    for n in range(N):
        assert rel_err(dl[n], dl_ref[n]) <= TOL[dtype], n


# Token rows of one chunk: the key side stores dZ itself, frozen rows as zeros (up to 128 tokens are never cut)
@pytest.mark.parametrize("P,n_frozen", [(200, 0), (200, 1), (200, 32), (200, 63), (200, 64), (200, 65), (200, 130), (200, 200), (1, 1), (128, 96)])
def test_dz_of_one_chunk(P, n_frozen):
    q, k, v, zk, zv, do = attn_case((1, 100), 8, 2, 128, P, torch.bfloat16, 3 * P + n_frozen)
    check_attn(q, k, v, zk, zv, do, impl=cb.IMPL_MFMA, n_frozen=n_frozen)
    a = [t.to(DEV) for t in (q, k, v, zk, zv)]
    o, lse = cb.cart_attn_fwd(*a)
    dz = [torch.full((2, P, 128), float("nan"), device=DEV) for _ in range(2)]
    first = [t.clone() for t in cb.cart_attn_bwd(*a, o, lse, do.to(DEV), n_frozen=n_frozen, d_z_k=dz[0], d_z_v=dz[1])[3:]]
    assert all((t[:, :n_frozen] == 0).all() and torch.isfinite(t).all() for t in first)
    # added to what is there: the sums' own kernel
    cb.cart_attn_bwd(*a, o, lse, do.to(DEV), n_frozen=n_frozen, d_z_k=dz[0], d_z_v=dz[1], dz_accumulate=True)
    assert all(torch.equal(t, 2 * f) for t, f in zip(dz, first))


# ... of several sequences, batched and packed, by one launch of all gradients and by two, beside split query blocks (the last)
@pytest.mark.parametrize("lens,packed,Hq,Hkv,P,one_launch", [([60] * 2, False, 8, 2, 200, True), ([40] * 3, False, 4, 1, 130, True), ([1] * 32, False, 8, 8, 130, False),
                                                             ([24] * 32, False, 16, 8, 1500, False), ([5, 40, 1, 64], True, 8, 2, 200, True),
                                                             ([10] * 148 + [9] * 147, True, 16, 16, 64, False), ([300, 299], True, 16, 16, 1500, False)])
@pytest.mark.parametrize("n_frozen", [0, 1, 33])
def test_dz_of_one_chunk_of_several_sequences(lens, packed, Hq, Hkv, P, one_launch, n_frozen):
    p = plan(len(lens), max(lens), Hq, Hkv, P, sum(lens) if packed else 0)
    assert p.n_part == 1 and p.one_launch == one_launch
    rows = (sum(lens),) if packed else (len(lens), lens[0])
    q, k, v, zk, zv, do = attn_case(rows, Hq, Hkv, 128, P, torch.bfloat16, P + Hq + n_frozen)
    n = [f64(t) for t in (q, k, v, zk, zv, do)]
    a = [t.to(DEV) for t in (q, k, v, zk, zv)]
    dz = [torch.full((Hkv, P, 128), float("nan"), device=DEV) for _ in range(2)]
    if packed:
        cu = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32)
        ref = [x.copy() for x in orc.attn_varlen_bwd(*n, cu.numpy())]
        fwd = a + [cu.to(DEV), max(lens)]
        bwd = lambda **kw: cb.cart_attn_varlen_bwd(*fwd, *cb.cart_attn_varlen_fwd(*fwd), do.to(DEV), n_frozen=n_frozen, d_z_k=dz[0], d_z_v=dz[1], **kw)
    else:
        ref = [x.copy() for x in orc.attn_bwd(*n)]
        bwd = lambda **kw: cb.cart_attn_bwd(*a, *cb.cart_attn_fwd(*a), do.to(DEV), n_frozen=n_frozen, d_z_k=dz[0], d_z_v=dz[1], **kw)
    for x in ref[3:]:
        x[:, :n_frozen] = 0
    out = [x.clone() for x in bwd()]
    torch.cuda.synchronize()
    for x, r in zip(out, ref):
        if np.abs(r).max() < 1e-12:
            assert np.abs(f64(x)).max() < 1e-2
        else:
            assert rel_err(x, r) <= TOL[torch.bfloat16]
    assert all((t[:, :n_frozen] == 0).all() for t in out[3:])
    bwd(dz_accumulate=True)
    assert all(torch.equal(t, 2 * f) for t, f in zip(dz, out[3:]))


# fp32 rows: the bound of the candidates is settled before the last bits: rows whose values differ in those only, in steps of each
# power of two, of either sign, with -inf
# (records up to and from a quarter of the 256, 512 and 1024 threads on)
@pytest.mark.parametrize("V,K", [(4096, 1), (4096, 7), (9001, 20), (50257, 19), (70001, 64), (16384, 64), (16384, 65), (30000, 128), (30000, 129),
                                 (50257, 256), (50257, 257), (16384, 513), (50257, 815), (16384, 900), (70001, 1000)])
def test_topk_bound_of_fp32_rows(V, K):
    g = torch.Generator().manual_seed(V + K)
    r = lambda: torch.randint(0, 4 * K + 40, (V,), generator=g, dtype=torch.int32)
    one = torch.tensor([1.0]).view(torch.int32)
    x = torch.empty(8, V)
    x[0] = (one + r()).view(torch.float32)
    x[1] = -(one + r()).view(torch.float32)
    x[2] = 2.0 ** (r() % 200 - 100).float()
    x[3] = -(2.0 ** (r() % 200 - 100).float())
    x[4] = torch.where(r() > 2 * K, float("-inf"), 0.0) + torch.randn(V, generator=g)
    x[5] = torch.where(torch.arange(V) % (V // (K + 1)) == 0, 5.0, -5.0)
    x[6] = (r() * 2 ** 12 + one).view(torch.float32)
    x[7] = torch.randn(V, generator=g).abs() * 1.0e-38
    idx, lp = cb.cart_teacher_topk(x.to(DEV), K)
    ref = torch.sort(x, dim=1, descending=True, stable=True)[1][:, :K]
    assert torch.equal(idx.cpu().long(), ref)
    want = x.double().gather(1, ref) - torch.logsumexp(x.double(), 1, keepdim=True)
    # (values up to 2^99: relative to the row's largest)
    scale = x.double().abs().where(torch.isfinite(x), torch.zeros(1, dtype=torch.float64)).amax(1, keepdim=True).clamp(min=24.0)
    assert ((lp.cpu().double() - want).abs() <= 5e-7 * scale).all()


# More rows than workgroups of 1024 threads: the first half of a workgroup's next row is requested ahead (rows that begin anywhere in a
# line; one, two and three rows a workgroup; in place)
@pytest.mark.parametrize("N,V", [(257, 65543), (515, 66000), (520, 131066)])
def test_loss_rows_requested_ahead(N, V):
    K = 7
    g = torch.Generator(device=DEV).manual_seed(V)
    x = (3.0 * torch.randn(N, V, generator=g, device=DEV)).to(torch.bfloat16)
    idx = torch.randint(0, V // K, (N, K), generator=g, device=DEV) + torch.arange(K, device=DEV) * (V // K)
    logp = torch.log_softmax(torch.randn(N, K, generator=g, device=DEV), 1) + float(np.log(0.9))
    idx = idx.to(torch.int32)
    row = torch.empty(N, dtype=torch.float32, device=DEV)
    loss, dl = cb.cart_distill_kl_fwd_bwd(x, idx, logp, 1.0 / N, row_kl=row)
    for c in torch.arange(N, device=DEV).split(64):
        lp = torch.log_softmax(x[c].double(), 1)
        t = logp[c].double().exp()
        want = (t * (logp[c].double() - lp.gather(1, idx[c].long()))).sum(1)
        assert ((row[c].double() - want).abs() <= 1e-4 * want.abs().max()).all()
        d = t.sum(1, keepdim=True) * lp.exp()
        d.scatter_add_(1, idx[c].long(), -t)
        e = (dl[c].double() - d / N).abs().amax(1) / (d / N).abs().amax(1)
        assert e.max().item() <= TOL[torch.bfloat16]
    loss2, dl2 = cb.cart_distill_kl_fwd_bwd(x, idx, logp, 1.0 / N, d_logits=x)
    assert torch.equal(dl2, dl) and loss2.item() == loss.item()


# The offsets of up to 128 requests are held a lane each, those of more looked up in memory (requests of one row among them)
@pytest.mark.parametrize("B", [1, 2, 62, 63, 64, 65, 126, 127, 128, 129])
def test_decode_finds_the_request_of_a_range(B):
    g = torch.Generator().manual_seed(B)
    rn = lambda *sz, std=0.6: (std * torch.randn(*sz, generator=g)).to(torch.bfloat16)
    lens = torch.randint(1, 90, (B,), generator=g)
    lens[::3] = 1
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lens.numpy())]), dtype=torch.int32)
    q, k, v, zk, zv = rn(B, 8, 128), rn(int(cu[-1]), 2, 128), rn(int(cu[-1]), 2, 128), rn(2, 50, 128), rn(2, 50, 128)
    o, lse = cb.cart_decode(*(t.to(DEV) for t in (q, zk, zv, k, v, cu)), int(lens.max()))
    torch.cuda.synchronize()
    o_ref, lse_ref = orc.decode(*(f64(t) for t in (q, zk, zv, k, v)), cu.numpy())
    assert rel_err(o, o_ref) <= TOL[torch.bfloat16] and rel_err(lse, lse_ref) <= TOL[torch.bfloat16]


# Several shared segments: each in parts of one length (segments of a part, of somewhat more, of one slot, beside much longer ones)
@pytest.mark.parametrize("B,segs", [(40, (2048, 2048, 2048, 2048)), (7, (700, 1, 33)), (3, (4000, 32, 64, 5)), (90, (1700, 1300, 1)), (1, (31, 3000)),
                                    (20, (1, 1, 1, 1, 1, 1, 1, 1)), (12, (0, 900, 0, 420))])
def test_decode_segments_in_equal_parts(B, segs):
    g = torch.Generator().manual_seed(B + sum(segs))
    rn = lambda *sz, std=0.6: (std * torch.randn(*sz, generator=g)).to(torch.bfloat16)
    lens = torch.randint(1, 60, (B,), generator=g)
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lens.numpy())]), dtype=torch.int32)
    q, k, v = rn(B, 8, 128), rn(int(cu[-1]), 2, 128), rn(int(cu[-1]), 2, 128)
    shared = [(rn(2, p, 128), rn(2, p, 128)) for p in segs]
    dv = lambda t: t.to(DEV)
    o, lse = cb.cart_decode_composed(dv(q), [(dv(a), dv(b)) for a, b in shared], None, None, None, dv(k), dv(v), dv(cu), int(lens.max()))
    torch.cuda.synchronize()
    o_ref, lse_ref = orc.decode_composed(f64(q), [(f64(a), f64(b)) for a, b in shared], None, None, None, f64(k), f64(v), cu.numpy())
    assert rel_err(o, o_ref) <= TOL[torch.bfloat16] and rel_err(lse, lse_ref) <= TOL[torch.bfloat16]


# The merge reads slots that no part of the launch writes: what the workspace holds there does not matter (few output rows, four wavefronts a row, and many;
# requests that reach into fewer ranges than the longest, with and without a cartridge)
@pytest.mark.parametrize("B,Hq,Hkv,P,pool_p,most", [(4, 32, 8, 2048, 0, 150), (1, 8, 2, 0, 0, 9000), (9, 16, 8, 300, 700, 2500), (64, 32, 8, 100, 260, 700), (65, 32, 8, 100, 260, 700),
                                                    (200, 16, 4, 4000, 0, 600)])
def test_decode_in_a_workspace_of_nan(B, Hq, Hkv, P, pool_p, most):
    g = torch.Generator().manual_seed(B + P)
    rn = lambda *sz, std=0.6: (std * torch.randn(*sz, generator=g)).to(torch.bfloat16)
    lens = torch.randint(1, max(2, most // 8), (B,), generator=g)
    lens[0] = most
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lens.numpy())]), dtype=torch.int32)
    T = int(cu[-1])
    q, k, v, shared = rn(B, Hq, 128), rn(T, Hkv, 128), rn(T, Hkv, 128), [(rn(Hkv, P, 128), rn(Hkv, P, 128))] if P else []
    pk = pv = cid = None
    if pool_p:
        pk, pv, cid = rn(3, Hkv, pool_p, 128), rn(3, Hkv, pool_p, 128), (torch.arange(B) % 4 - 1).to(torch.int32)
    dv = lambda t: None if t is None else t.to(DEV)
    a = (dv(q), [(dv(x), dv(y)) for x, y in shared], dv(pk), dv(pv), dv(cid), dv(k), dv(v), dv(cu), most)
    ws = [torch.full((1 << 26,), b, dtype=torch.uint8, device=DEV) for b in (0xff, 0)]
    o, lse = cb.cart_decode_composed(*a, workspace=ws[0])
    o2, lse2 = cb.cart_decode_composed(*a, workspace=ws[1])
    torch.cuda.synchronize()
    assert torch.equal(o, o2) and torch.equal(lse, lse2)
    z = lambda t: None if t is None else f64(t)
    o_ref, lse_ref = orc.decode_composed(f64(q), [(f64(x), f64(y)) for x, y in shared], z(pk), z(pv), None if cid is None else cid.numpy(), f64(k), f64(v), cu.numpy())
    assert rel_err(o, o_ref) <= TOL[torch.bfloat16] and rel_err(lse, lse_ref) <= TOL[torch.bfloat16]


# Own rows of 144 MiB at most, one row more; private cartridges: one each, two requests on one, up to 144 MiB with the own rows and past
# them, half of the requests without, several on one beside others of their own, more requests than one look at the others' numbers takes
@pytest.mark.parametrize("lens,pool_p,ids", [((20000, 1, 16863), 0, ()), ((20000, 1, 16864), 0, ()), ((20000, 1, 16864), 90, (1, -1, 0)), ((5,) * 20, 2048, range(20)),
                                             ((5,) * 20, 2048, (*range(19), 0)), ((600,) * 40, 321, range(40)), ((600,) * 40, 322, range(40)), ((5,) * 36, 1019, range(36)), ((4,) * 36, 1020, range(36)), ((5,) * 36, 1020, range(36)),
                                             ((30,) * 40, 2048, [i // 2 if i % 2 else -1 for i in range(40)]), ((7,) * 64, 1100, [i if i % 3 else i % 4 for i in range(64)]),
                                             ((1, 3, 2) * 100, 160, [i if i % 5 else 299 - i // 9 for i in range(300)])])
def test_decode_rows_that_are_not_kept_in_caches(lens, pool_p, ids):
    Hq, Hkv, B = 16, 8, len(lens)
    n_pool = max(ids, default=-1) + 1
    g = torch.Generator(device=DEV).manual_seed(sum(lens) + n_pool)
    rn = lambda *sz: (0.6 * torch.randn(*sz, generator=g, device=DEV)).to(torch.bfloat16)
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32, device=DEV)
    q, k, v, shared = rn(B, Hq, 128), rn(sum(lens), Hkv, 128), rn(sum(lens), Hkv, 128), [(rn(Hkv, 70, 128), rn(Hkv, 70, 128))]
    pk = pv = cid = None
    if pool_p:
        pk, pv, cid = rn(n_pool, Hkv, pool_p, 128), rn(n_pool, Hkv, pool_p, 128), torch.tensor(list(ids), device=DEV, dtype=torch.int32)
    o, lse = cb.cart_decode_composed(q, shared, pk, pv, cid, k, v, cu, max(lens))
    torch.cuda.synchronize()
    z = lambda t: None if t is None else f64(t)
    o_ref, lse_ref = orc.decode_composed(f64(q), [(f64(a), f64(b)) for a, b in shared], z(pk), z(pv),
                                         None if cid is None else cid.cpu().numpy(), f64(k), f64(v), cu.cpu().numpy())
    assert rel_err(o, o_ref) <= TOL[torch.bfloat16] and rel_err(lse, lse_ref) <= TOL[torch.bfloat16]


# Cartridges that many requests read are kept in caches however many others the pool holds (us, a pool of 4 / of 132: 97 / 97; 97 / 147 when the size of
# the pool decided)
def test_decode_time_of_a_few_cartridges_of_many():
    B, Hq, Hkv, pool_p = 128, 32, 8, 2048
    g = torch.Generator(device=DEV).manual_seed(1)
    rn = lambda *sz: (0.1 * torch.randn(*sz, generator=g, device=DEV)).to(torch.bfloat16)
    lens = torch.randint(1, 101, (B,), generator=torch.Generator().manual_seed(2))
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lens.numpy())]), dtype=torch.int32, device=DEV)
    T, cid = int(cu[-1]), torch.arange(B, device=DEV, dtype=torch.int32) % 4
    q, k, v, shared, pk, pv = rn(B, Hq, 128), rn(T, Hkv, 128), rn(T, Hkv, 128), [(rn(Hkv, 2048, 128), rn(Hkv, 2048, 128))], rn(132, Hkv, pool_p, 128), rn(132, Hkv, pool_p, 128)
    us = [best_us(lambda: cb.cart_decode_composed(q, shared, pk[:n], pv[:n], cid, k, v, cu, int(lens.max()))) for n in (4, 132)]
    assert us[1] < 1.2 * us[0], us


# The last turn of a row has one to four vectors a thread, for some of the threads; rows that are not kept in caches (more than 144 MiB)
@pytest.mark.parametrize("dtype,N,V", [(torch.bfloat16, 3, 8 * n + r) for n, r in ((1, 0), (255, 7), (256, 1), (257, 0), (1023, 0), (1024, 0), (1025, 3), (1792, 0))] +
                         [(torch.float32, 3, 4 * n + r) for n, r in ((1, 0), (511, 3), (1025, 1), (4097, 0), (6145, 2), (12289, 0))] +
                         [(torch.bfloat16, 599, 128256), (torch.float32, 1181, 32003), (torch.bfloat16, 1901, 40001), (torch.bfloat16, 3803, 20003),
                          (torch.float32, 2401, 16003), (torch.float32, 301, 128257)])
def test_topk_last_turns(dtype, N, V):
    K = min(20, V)
    g = torch.Generator(device=DEV).manual_seed(V)
    x = (3.0 * torch.randn(N, V, generator=g, device=DEV)).to(dtype)
    x[0, -3:] = 40.0                                           # winners among the last elements
    idx, lp = cb.cart_teacher_topk(x, K)
    v, ref = (t[:, :K] for t in torch.sort(x.float(), dim=1, descending=True, stable=True))
    assert torch.equal(idx.long(), ref)
    want = v.double() - torch.logsumexp(x.double(), 1, keepdim=True)
    # (the log-sum-exp's rounding, 2^-23 of at most 64, and its sum's, a few 2^-24)
    assert (lp.double() - want).abs().max().item() <= 1e-5


# Launches of more than 2^32 threads (8.4 million rows in workgroups of 512): every row is computed.
def test_topk_of_millions_of_rows():
    N, V, K = 8_400_000, 136, 130
    x = torch.empty(N, V, dtype=torch.bfloat16, device=DEV)
    g = torch.Generator(device=DEV).manual_seed(1)
    for c in x.split(2 ** 20):
        c.copy_(torch.randn(c.shape, generator=g, device=DEV))
    idx = torch.full((N, K), -1, dtype=torch.int32, device=DEV)
    cb.cart_teacher_topk(x, K, teacher_idx=idx)
    for c, i in zip(x.split(2 ** 20), idx.split(2 ** 20)):
        ref = torch.sort(c.float(), dim=1, descending=True, stable=True)[1][:, :K]
        assert torch.equal(i.long(), ref)


def test_attention_vector_of_millions_of_workgroups():
    B, H, D, P = 270_000, 32, 64, 2
    g = torch.Generator(device=DEV).manual_seed(2)
    q, k, v, do = (torch.randn(B, 1, H, D, generator=g, device=DEV) for _ in range(4))
    zk, zv = (torch.randn(H, P, D, generator=g, device=DEV) for _ in range(2))
    outs = [torch.full_like(q, float("nan")) for _ in range(4)]
    lse = torch.full((B, H, 1), float("nan"), device=DEV)
    cb.cart_attn_fwd(q, k, v, zk, zv, o=outs[0], lse=lse)
    cb.cart_attn_bwd(q, k, v, zk, zv, outs[0], lse, do, d_q=outs[1], d_k_own=outs[2], d_v_own=outs[3])
    torch.cuda.synchronize()
    assert all(torch.isfinite(t).all() for t in outs + [lse])
    for b in (0, B // 2, B - 1):
        n = [f64(t[b:b + 1]) for t in (q, k, v)] + [f64(zk), f64(zv), f64(do[b:b + 1])]
        ref = [*orc.attn_fwd(*n[:5]), *orc.attn_bwd(*n)[:3]]
        for x, r in zip([outs[0][b:b + 1], lse[b:b + 1]] + [t[b:b + 1] for t in outs[1:]], ref):
            assert rel_err(x, r) <= TOL[torch.float32]


# Events of a backward call, in either form the planner takes and of the fp32 kernels: what stands in front of the
# gradients' sums is dQ, dK + dV, or the row statistics, all three gradients, or all three and nothing.
@pytest.mark.parametrize("cfg,first_share", [((1, 128, 32, 8, 128, 1024, "bf16"), (0.0, 0.6)), ((13, 267, 8, 2, 128, 2990, "bf16"), (0.15, 0.8)),
                                             ((2, 128, 8, 2, 64, 256, "f32"), (0.5, 1.0)), ((2, 304, 16, 16, 128, 67, "f32"), (0.9, 1.0)),
                                             ((2, 304, 16, 16, 96, 67, "f32"), (0.1, 0.8))], ids=["one", "two", "f32", "f32_128", "f32_two"])
def test_events_of_a_backward_call(cfg, first_share):
    B, S, Hq, Hkv, D, P, dt = cfg
    t = synth.attn_inputs(synth.AttnConfig("", 5, B, S, Hq, Hkv, D, P, dt, 1.0, 1.0, 0.1), DEV)
    a = (t["q"], t["k_own"], t["v_own"], t["z_k"], t["z_v"])
    o, lse = cb.cart_attn_fwd(*a)
    tr = cb.KernelTrace(4)
    shares = []
    for _ in range(6):
        with tr:
            cb.cart_attn_bwd(*a, o, lse, t["d_o"])
        torch.cuda.synchronize()
        x, y, z = tr.intervals_ms()
        assert min(x, y, z) >= 0.0
        shares.append(x / (x + y))
    tr.close()
    assert first_share[0] <= sorted(shares)[3] <= first_share[1], shares
