"""The layers of a training step ask for the same two query splits in turn, the forward's and dQ's: neither may
evict the other's (host only; the planner is called directly, a call to an entry point would need a GPU)."""
import ctypes as C
import time

from paper_2506_06266_amd import binding as cb


def test_forward_and_dq_splits_are_both_kept():
    lib = C.CDLL(cb.LIB_PATH)
    split = lib["_ZN4cart16attn_query_splitERNS_4mfma10QuerySplitERK14cart_attn_desciNS0_11QueryKernelE"]
    split.argtypes, split.restype = [C.c_void_p, C.c_void_p, C.c_int, C.c_int], None
    out = (C.c_uint32 * 4096)()
    d = cb.AttnDesc(32, 516, 8, 2, 128, 1024, cb.CART_BF16, 0.0, 0, 0, cb.IMPL_AUTO)
    o, p = C.addressof(out), C.addressof(d)

    def us(kinds):
        best = float("inf")
        for _ in range(20):
            t0 = time.perf_counter()
            for _ in range(200):
                for k in kinds:
                    split(o, p, 0, k)
            best = min(best, (time.perf_counter() - t0) / 400)
        return best

    alone, in_turn = max(us([0, 0]), us([1, 1])), us([0, 1])
    assert in_turn < 2.0 * alone, (in_turn, alone)     # (planned afresh each time: 10 x and more)
