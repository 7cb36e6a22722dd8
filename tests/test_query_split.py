"""How query blocks are split along their key tiles (host only; the planner is called directly, a call to an entry
point would need a GPU)."""
import ctypes as C

import pytest

from paper_2506_06266_amd import binding as cb


def _parts(B, S, Hq, Hkv, P, T=0, kind=0):
    """(blocks per KV head that run whole, split blocks, their parts)"""
    lib = C.CDLL(cb.LIB_PATH)
    split = lib["_ZN4cart16attn_query_splitERNS_4mfma10QuerySplitERK14cart_attn_desciNS0_11QueryKernelE"]
    split.argtypes, split.restype = [C.c_void_p, C.c_void_p, C.c_int, C.c_int], None
    out = (C.c_int32 * 4096)()
    d = cb.AttnDesc(B, S, Hq, Hkv, 128, P, cb.CART_BF16, 0.0, 0, 0, cb.IMPL_AUTO)
    split(C.addressof(out), C.addressof(d), T, kind)
    return tuple(out[:3])


# Forward launches that are slower in parts (us whole, as they were split): too few tiles to gain what the parts cost
# (1 x 256, 512 slots 23.1, 27.6; 1 x 32, 8 / 8 heads 13.9, 20.5; 6 x 90 24.4, 29.8; 2 x 333 17.5, 24.8), or tiles that
# cannot be divided (sequences of 700, 1, 90 packed 40.6, 52.3; 4000, 10, 500 146.8, 153.9; 100, 60, 200 26.7, 30.6).
@pytest.mark.parametrize("B,S,Hq,Hkv,P,T", [(1, 256, 32, 8, 512, 0), (1, 32, 8, 8, 300, 0), (6, 90, 16, 4, 700, 0), (2, 333, 3, 3, 31, 0),
                                            (3, 700, 32, 8, 300, 791), (3, 4000, 8, 8, 128, 4510), (3, 200, 32, 8, 500, 360)])
def test_forward_runs_whole_where_parts_cost_more(B, S, Hq, Hkv, P, T):
    assert _parts(B, S, Hq, Hkv, P, T)[1:] == (0, 0)


# ... and those that are faster in parts (whole, split): 1 x 700 41.9, 38.5; 1 x 64 48.6, 26.3; 1 x 1024 28.4, 23.8;
# 8 x 512 206, 190 (its last half round); four sequences of 300 packed 42.7, 36.2
@pytest.mark.parametrize("B,S,Hq,Hkv,P,T,least", [(1, 700, 32, 8, 1000, 0, 3), (1, 64, 32, 8, 2000, 0, 5), (1, 1024, 8, 2, 0, 0, 3),
                                                  (8, 512, 24, 8, 4096, 0, 2), (4, 300, 8, 2, 1000, 1200, 3)])
def test_forward_is_split_where_that_is_faster(B, S, Hq, Hkv, P, T, least):
    whole, blocks, parts = _parts(B, S, Hq, Hkv, P, T)
    assert blocks > 0 and parts > (least - 1) * blocks


# (the packed launch of whole and split blocks that the GPU tests run)
def test_packed_launch_of_whole_and_split_blocks():
    for kind in (0, 1):
        whole, blocks, parts = _parts(8, 640, 32, 8, 1501, 2240, kind)
        assert (whole, blocks) == (32, 3) and parts > blocks
