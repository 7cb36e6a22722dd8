"""Which backward calls take dQ, dK and dV in one launch, and that its cuts fit the workspace (host only; the planner is
called directly, a call to an entry point would need a GPU)."""
import ctypes as C
import math
import random

import pytest

from paper_2506_06266_amd import binding as cb

CUS = 256           # (assumed where there is no GPU)


class _Plan(C.Structure):
    _fields_ = [("chunk", C.c_int32), ("n_part", C.c_int32), ("head_parts", C.c_int32), ("e_full", C.c_int32),
                ("n_blocks", C.c_int32), ("n_parts", C.c_int32), ("part", C.c_uint32 * 256), ("first", C.c_uint32 * 256),
                ("one_launch", C.c_bool), ("kv_front", C.c_int32)]


def plan(B, S, Hq, Hkv, P, T=0):
    f = C.CDLL(cb.LIB_PATH)["_ZN4cart8plan_bwdERK14cart_attn_desci"]
    f.argtypes, f.restype = [C.c_void_p, C.c_int], C.POINTER(_Plan)
    d = cb.AttnDesc(B, S, Hq, Hkv, 128, P, cb.CART_BF16, 0.0, 0, 0, cb.IMPL_AUTO)
    return _Plan.from_buffer_copy(f(C.addressof(d), T).contents)


# us a call in two launches, in one: 52 -> 37, 41 -> 26, 194 -> 175, 88 -> 66, packed 61 -> 42, 309 -> 263
@pytest.mark.parametrize("B,S,Hq,Hkv,P,T", [(1, 128, 32, 8, 1024, 0), (1, 300, 24, 8, 0, 0), (2, 333, 32, 8, 4096, 0), (1, 2048, 8, 2, 256, 0),
                                            (4, 272, 8, 2, 1000, 602), (8, 638, 32, 8, 1501, 2628)])
def test_one_launch_where_two_leave_the_chip_idle(B, S, Hq, Hkv, P, T):
    assert plan(B, S, Hq, Hkv, P, T).one_launch


# many rounds of blocks: the statistics' own launch costs more than the ends of two launches
@pytest.mark.parametrize("B,S,Hq,Hkv,P,T", [(16, 2048, 32, 8, 4096, 0), (32, 1024, 24, 8, 2048, 0), (64, 1024, 32, 8, 4096, 37251)])
def test_two_launches_of_many_rounds(B, S, Hq, Hkv, P, T):
    assert not plan(B, S, Hq, Hkv, P, T).one_launch


# long blocks of somewhat more than a round, prefix blocks many of them: the last ones start late.  us a call in two launches,
# in one: 206 -> 226, packed 138 -> 147, 141 -> 152, 263 -> 290
@pytest.mark.parametrize("B,S,Hq,Hkv,P,T", [(13, 267, 8, 2, 2990, 0), (11, 230, 8, 2, 5629, 1415), (16, 71, 8, 2, 6672, 0), (21, 213, 8, 2, 3561, 0)])
def test_two_launches_where_one_starts_its_last_blocks_late(B, S, Hq, Hkv, P, T):
    assert not plan(B, S, Hq, Hkv, P, T).one_launch


# ... and no more than that is refused: 222 -> 198, 220 -> 197, packed 130 -> 118, 114 -> 104
@pytest.mark.parametrize("B,S,Hq,Hkv,P,T", [(1, 567, 32, 8, 5785, 0), (17, 177, 32, 8, 931, 0), (10, 361, 24, 8, 1065, 1694), (9, 313, 8, 2, 2113, 0)])
def test_one_launch_of_somewhat_more_or_less_than_a_round(B, S, Hq, Hkv, P, T):
    assert plan(B, S, Hq, Hkv, P, T).one_launch


@pytest.mark.parametrize("seed", range(3))
def test_cuts_of_one_launch(seed):
    rng = random.Random(seed)
    log = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    for _ in range(300):
        Hq, Hkv = rng.choice([(32, 8), (24, 8), (8, 2), (4, 1), (16, 16), (7, 1), (64, 8)])
        B, S, P = log(1, 40), log(1, 3000), rng.choice([0, log(1, 9000)])
        T = rng.choice([0, 0, rng.randint(S, B * S)])
        p, G = plan(B, S, Hq, Hkv, P, T), Hq // Hkv
        tokens = T or B * S
        blocks = -(-(-(-(T if T and P else S) // 64) * G) // 4) * (1 if T and P else B)
        assert p.e_full + p.n_blocks == blocks
        assert p.n_parts <= max(1, CUS // Hkv) and G % p.head_parts == 0
        assert p.n_part == -(-tokens // p.chunk) and p.chunk % 64 == 0 and (P or p.n_part == 1)
        # every part of every split block once, in order
        seen = [(w & 255, (w >> 8) & 255, w >> 16) for w in p.part[:p.n_parts]]
        assert seen == [(b, i, n) for b, n in sorted({(b, n) for b, _, n in seen}) for i in range(n)]
        assert [p.first[b] for b in range(p.n_blocks)] == [seen.index((b, 0, n)) for b, n in sorted({(b, n) for b, _, n in seen})]
        if p.one_launch:
            pre, per_kb = -(-P // 128) * p.n_part if P else 0, B * p.head_parts
            assert (p.kv_front - pre) % per_kb == 0 and 0 <= (p.kv_front - pre) // per_kb <= -(-S // 128)


def _up(n):
    return (n + 255) // 256 * 256


# What a call lays out one behind the other -- the row statistics, the partials of dZ, of split query blocks, of own keys,
# the packed rows' first rows -- ends inside what the query returns: an overrun would be a write no check sees.
@pytest.mark.parametrize("seed", range(4))
def test_every_plan_fits_the_workspace(seed):
    lib, rng = cb.load(), random.Random(100 + seed)
    log = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    forms = [0, 0]
    for _ in range(600):
        Hq, Hkv = rng.choice([(32, 8), (24, 8), (8, 2), (4, 1), (16, 16), (7, 1), (64, 8), (48, 4), (6, 3)])
        B, S, P = log(1, 64), log(1, 4096), rng.choice([0, log(1, 16384)])
        T = rng.choice([0, rng.randint(S, B * S)])
        p = plan(B, S, Hq, Hkv, P, T)
        forms[p.one_launch] += 1
        tokens = T or B * S
        laid = (2 * _up(4 * tokens * Hq) + 2 * _up(p.n_part * Hkv * P * 128 * 4) + p.n_parts * Hkv * 256 * 128 * 4 +
                (2 * _up(p.head_parts * tokens * Hkv * 128 * 4) if p.head_parts > 1 else 0) + (_up(4 * T) if T and P else 0))
        if T:
            d = cb.AttnVarlenDesc(T, B, S, Hq, Hkv, 128, P, cb.CART_BF16, 0.0, 0, 0)
            most = lib.cart_attn_varlen_bwd_workspace(C.byref(d))
        else:
            d = cb.AttnDesc(B, S, Hq, Hkv, 128, P, cb.CART_BF16, 0.0, 0, 0, cb.IMPL_AUTO)
            most = lib.cart_attn_bwd_workspace(C.byref(d))
        assert laid <= most, (B, S, Hq, Hkv, P, T, laid, most)
    assert min(forms) > 50          # (both forms were looked at)
