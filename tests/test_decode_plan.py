"""How the decode step cuts its shared segments and own rows, and that it fits the workspace (host only; the planner is called
directly, a call to an entry point would need a GPU)."""
import ctypes as C
import math
import random

import pytest

from paper_2506_06266_amd import binding as cb

SEG = 8


class _Table(C.Structure):
    _fields_ = [("zk", C.c_void_p * SEG), ("zv", C.c_void_p * SEG), ("p", C.c_int32 * SEG), ("tiles", C.c_int32 * SEG), ("n_ps", C.c_int32 * SEG),
                ("slot0", C.c_int32 * SEG), ("blk0", C.c_int32 * (SEG + 1)), ("n_seg", C.c_int32)]


class _Plan(C.Structure):
    _fields_ = [("tab", _Table)] + [(n, C.c_int32) for n in ("G", "n_rb", "n_ps", "share", "pool_share", "n_oc", "n_cc", "pool_r0", "n_own_wg")] + [
        ("part_o_bytes", C.c_size_t), ("part_l_bytes", C.c_size_t)]


def plan(B, Hq, Hkv, max_own, T, segs, pool_p=0):
    f = C.CDLL(cb.LIB_PATH)["_ZN4cart11decode_planEiiiiiPKiii"]
    f.argtypes, f.restype = [C.c_int] * 5 + [C.c_void_p, C.c_int, C.c_int], _Plan
    p = (C.c_int32 * SEG)(*segs)
    return f(B, Hq, Hkv, max_own, T, C.addressof(p), len(segs), pool_p)


def _drawn(rng, most_rows):
    log = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    while True:
        Hq, Hkv = rng.choice([(32, 8), (24, 8), (8, 2), (4, 1), (16, 16), (28, 4)])
        B, most, n = log(1, 256), log(1, 8192), rng.choice([2, 3, 4, 8])
        segs = [log(1, 9000) for _ in range(n)] if rng.random() < 0.5 else [log(1, 4000)] * n
        if B * Hq <= most_rows:
            return B, Hq, Hkv, most, max(B, rng.randint(B, B * most), most), segs


# Each of several segments: parts of one length, together the segment, at most a quarter longer than one cartridge of as many tiles
# would be cut (a tile, where that is more), and never more of them.
@pytest.mark.parametrize("seed", range(4))
def test_segments_are_cut_in_parts_of_one_length(seed):
    rng = random.Random(seed)
    longer = 0
    for _ in range(1500):
        B, Hq, Hkv, most, T, segs = _drawn(rng, 500)       # (no plan of so few rows is a lean one)
        tiles = [-(-s // 32) for s in segs]
        p, tps = plan(B, Hq, Hkv, most, T, segs), plan(B, Hq, Hkv, most, T, [32 * sum(tiles)]).tab.tiles[0]
        assert p.tab.n_seg == len(segs)
        slot = blk = 0
        for k, n in enumerate(tiles):
            size, parts = p.tab.tiles[k], p.tab.n_ps[k]
            assert (p.tab.p[k], p.tab.slot0[k], p.tab.blk0[k]) == (segs[k], slot, blk)
            assert (parts - 1) * size < n <= parts * size and parts <= -(-n // tps), (B, Hq, Hkv, most, T, segs)
            assert size <= max(tps * 5 // 4, tps + 1 if tps <= 3 else 0), (B, Hq, Hkv, most, T, segs, tps, size)
            assert size == -(-n // parts)
            longer += size > tps
            slot += parts
            blk += Hkv * p.n_rb * parts
        assert (p.n_ps, p.tab.blk0[len(segs)]) == (slot, blk)
    assert longer > 100


# One segment beside empty ones is cut as it is alone.
def test_one_segment_among_empty_ones():
    for B, P in ((1, 31), (4, 2048), (128, 8192), (40, 5000)):
        a, b = plan(B, 32, 8, 500, 250 * B, [P]), plan(B, 32, 8, 500, 250 * B, [0, P, 0])
        assert (a.tab.tiles[0], a.n_ps, a.share, a.n_own_wg) == (b.tab.tiles[0], b.n_ps, b.share, b.n_own_wg)


# Whether own ranges get longer for CUs that are not shared is decided by the longest part there is: us a call, by the
# estimate's / by that one 43.8 -> 32.8, 31.9 -> 25.5, 45.4 -> 40.2
@pytest.mark.parametrize("B,Hq,Hkv,most,T,segs,share", [(184, 8, 2, 365, 33438, (39, 517, 34, 36, 7457, 6106, 1104, 76), 352),
                                                        (136, 8, 2, 451, 29531, (222, 216, 206, 1737, 6314, 193, 345, 1131), 224),
                                                        (124, 32, 8, 195, 13061, (151, 30, 7139), 416)])
def test_own_ranges_beside_longer_parts(B, Hq, Hkv, most, T, segs, share):
    assert plan(B, Hq, Hkv, most, T, segs).share == share


# Partials of every slot, and their log-sum-exps, inside what the query returns (which reads no segment: any address will do).
@pytest.mark.parametrize("seed", range(2))
def test_every_plan_fits_the_workspace(seed):
    lib, rng = cb.load(), random.Random(50 + seed)
    for _ in range(1000):
        B, Hq, Hkv, most, T, segs = _drawn(rng, 1 << 20)
        pool_p = rng.choice([0, 0, rng.randint(1, 3000)])
        p = plan(B, Hq, Hkv, most, T, segs, pool_p)
        assert p.part_o_bytes >= (p.n_ps + p.n_cc + p.n_oc) * B * Hq * 128 * 4 and p.part_l_bytes >= (p.n_ps + p.n_cc + p.n_oc) * B * Hq * 4
        d = cb.DecodeComposedDesc(B, Hq, Hkv, 128, len(segs), B if pool_p else 0, pool_p, T, most, cb.CART_BF16, 0.0)
        shared = (cb.Segment * len(segs))(*[cb.Segment(256, 256, s) for s in segs])
        assert p.part_o_bytes + p.part_l_bytes <= lib.cart_decode_composed_workspace(C.byref(d), shared)
