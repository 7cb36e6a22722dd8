"""One workspace kept for a program's largest call has to serve its smaller ones (host only)."""
import ctypes as C
import math
import random

import pytest

from paper_2506_06266_amd import binding as cb

HEADS = [(32, 8), (24, 8), (8, 2), (4, 1), (16, 16), (64, 8)]


@pytest.fixture(scope="module")
def lib():
    return cb.load()


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _batched(lib, B, S, Hq, Hkv, P):
    d = cb.AttnDesc(B, S, Hq, Hkv, 128, P, cb.CART_BF16, 0.0, 0, 0, cb.IMPL_AUTO)
    return lib.cart_attn_fwd_workspace(C.byref(d)), lib.cart_attn_bwd_workspace(C.byref(d))


def _packed(lib, T, B, most, Hq, Hkv, P):
    d = cb.AttnVarlenDesc(T, B, most, Hq, Hkv, 128, P, cb.CART_BF16, 0.0, 0, 0)
    return lib.cart_attn_varlen_fwd_workspace(C.byref(d)), lib.cart_attn_varlen_bwd_workspace(C.byref(d))


def _covers(big, small, what):
    assert min(big + small) >= 0 and all(b >= s for b, s in zip(big, small)), (what, big, small)


def test_the_training_batch_covers_a_short_last_batch(lib):
    _covers(_batched(lib, 16, 2048, 32, 8, 4096), _batched(lib, 1, 700, 32, 8, 4096), "16 x 2048, 1 x 700")


# (allocating a workspace that is never used is a tenth of the smallest calls' time)
@pytest.mark.parametrize("B,S,Hq,Hkv,P", [(5, 9, 48, 4, 0), (1, 64, 32, 8, 0), (4, 64, 8, 2, 33), (1, 128, 32, 8, 64)])
def test_the_smallest_forward_calls_need_no_workspace(lib, B, S, Hq, Hkv, P):
    assert _batched(lib, B, S, Hq, Hkv, P)[0] == 0


@pytest.mark.parametrize("seed", range(4))
def test_attention_workspace_never_grows_towards_smaller_problems(lib, seed):
    rng = random.Random(seed)
    for _ in range(500):
        Hq, Hkv = rng.choice(HEADS)
        P = rng.choice([0, _log(rng, 1, 16384)])
        P2 = rng.choice([P, rng.randint(0, P)])
        B, S = _log(rng, 1, 64), _log(rng, 1, 4096)
        B2, S2 = rng.choice([B, rng.randint(1, B)]), rng.choice([S, rng.randint(1, S)])
        _covers(_batched(lib, B, S, Hq, Hkv, P), _batched(lib, B2, S2, Hq, Hkv, P2), (B, S, Hq, Hkv, P, B2, S2, P2))
        T = rng.randint(S, B * S)
        T2 = rng.randint(S2, T) if rng.random() < 0.5 else T
        if T2 >= B2:
            _covers(_packed(lib, T, B, S, Hq, Hkv, P), _packed(lib, T2, B2, S2, Hq, Hkv, P2), (T, B, S, Hq, Hkv, P, T2, B2, S2, P2))


# (fp32, and bf16 at other head_dims: delta, and the sums of prefix blocks split over the token rows)
@pytest.mark.parametrize("dtype", [cb.CART_F32, cb.CART_BF16])
def test_vector_workspace_never_grows_towards_smaller_problems(lib, dtype):
    rng = random.Random(11 + dtype)

    def need(B, S, Hq, Hkv, D, P):
        d = cb.AttnDesc(B, S, Hq, Hkv, D, P, dtype, 0.0, 0, 0, cb.IMPL_VECTOR)
        return lib.cart_attn_fwd_workspace(C.byref(d)), lib.cart_attn_bwd_workspace(C.byref(d))

    for _ in range(1500):
        Hq, Hkv = rng.choice(HEADS + [(2, 1), (28, 4)])
        big = (_log(rng, 1, 64), _log(rng, 1, 2048), Hq, Hkv, _log(rng, 1, 256), rng.choice([0, _log(rng, 1, 8192)]))
        small = [rng.choice([x, rng.randint(min(x, 1), x)]) for x in big]
        small[2:4] = Hq, Hkv
        _covers(need(*big), need(*small), (big, small))


# (every split the rule may take: 2 sums of one part, at most eight parts and as many prefix blocks as CUs)
@pytest.mark.parametrize("B,S,Hq,Hkv,D,P", [(4, 128, 8, 2, 128, 128), (2, 64, 4, 2, 200, 64), (1, 32, 2, 1, 64, 16), (4, 256, 8, 2, 64, 4096)])
def test_vector_workspace_holds_the_split_sums(lib, B, S, Hq, Hkv, D, P):
    d = cb.AttnDesc(B, S, Hq, Hkv, D, P, cb.CART_F32, 0.0, 0, 0, cb.IMPL_AUTO)
    delta = (4 * B * Hq * S + 255) // 256 * 256
    blocks = -(-P // 16) * Hkv
    parts = max(s for s in range(1, 9) if s == 1 or blocks * s <= 256)        # (256 CUs are assumed where there is no GPU)
    assert lib.cart_attn_bwd_workspace(C.byref(d)) >= delta + (parts * 2 * Hkv * P * D * 4 if parts > 1 else 0)


# (the partials of a problem and those of a smaller one: as long as neither exceeds the static array)
@pytest.mark.parametrize("seed", range(4))
def test_decode_workspace_never_grows_towards_smaller_problems(lib, seed):
    rng = random.Random(seed)
    cap = lib.cart_decode_static_capacity()
    for _ in range(800):
        Hq, Hkv = rng.choice(HEADS)
        B, most, P, pool = _log(rng, 1, 256), _log(rng, 1, 16384), rng.choice([0, _log(rng, 1, 8192)]), rng.choice([0, _log(rng, 1, 4096)])
        B2, most2, P2 = (rng.choice([x, rng.randint(min(x, 1), x)]) for x in (B, most, P))
        T = rng.randint(max(B, most), B * most) if B * most > max(B, most) else max(B, most)
        T2 = min(T, rng.randint(max(B2, most2), max(B2 * most2, B2, most2)))
        need = []
        for b, t, m, p in ((B, T, most, P), (B2, T2, most2, P2)):
            d = cb.DecodeDesc(b, Hq, Hkv, 128, p, t, m, cb.CART_BF16, 0.0, cb.IMPL_AUTO)
            seg = (cb.Segment * 1)(cb.Segment(0x1000, 0x1000, p))
            c = cb.DecodeComposedDesc(b, Hq, Hkv, 128, 1, b if pool else 0, pool, t, m, cb.CART_BF16, 0.0)
            need.append((lib.cart_decode_workspace(C.byref(d)), lib.cart_decode_composed_workspace(C.byref(c), seg)))
        for big, small in zip(*need):
            assert 0 < small and (small <= big or max(small, big) > cap), (B, Hq, Hkv, P, pool, T, most, B2, T2, most2, P2, big, small)


# Partials beyond cart_decode_static's 32 MiB are cut again only where that makes them fit, and never where a
# caller's workspace is the only one there is (private cartridges).  B, Hq, Hkv, slots, longest, own rows -> most MB
@pytest.mark.parametrize("B,Hq,Hkv,P,most,T,mb", [(32, 32, 8, 8192, 16384, 30000, 41.8), (128, 32, 8, 512, 9000, 568051, 33.6)])
def test_decode_is_cut_again_only_where_that_fits(lib, B, Hq, Hkv, P, most, T, mb):
    d = cb.DecodeDesc(B, Hq, Hkv, 128, P, T, most, cb.CART_BF16, 0.0, cb.IMPL_AUTO)
    assert lib.cart_decode_workspace(C.byref(d)) <= mb * 1e6


def test_decode_with_private_cartridges_keeps_the_estimated_cut(lib):
    seg = (cb.Segment * 1)(cb.Segment(0x1000, 0x1000, 47))
    d = cb.DecodeComposedDesc(208, 64, 8, 128, 1, 208, 786, 3973, 40, cb.CART_BF16, 0.0)
    assert 0 < lib.cart_decode_composed_workspace(C.byref(d), seg) <= 34.4e6
