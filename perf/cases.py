"""What this library is timed on: one pass of each public entry point a training or a serving
program calls, over the range of sizes, layouts, data types and options such programs use.

A training step of a cartridge calls the attention forward and backward of every layer (batched,
or packed when the conversations differ in length) and the distillation loss; the teacher's
records are produced by the top-k entry point while it generates; a server calls the decode step.
Shapes come from the library's own configurations (`synth.py`) and lie around them.
"""
from __future__ import annotations

import math
import random

import torch

from paper_2506_06266_amd import binding as cart
from paper_2506_06266_amd import synth

STD = 1.0 / math.sqrt(128.0)      # Q, K, V and dO of the layer-shaped configurations
Z_STD = 0.02                      # the trainable prefix


def _train(name, B, S, Hq, Hkv, P, n_frozen=0, dtype="bf16", D=128):
    return {"name": name, "kind": "train", "B": B, "S": S, "Hq": Hq, "Hkv": Hkv, "D": D, "P": P,
            "n_frozen": n_frozen, "dtype": dtype}


def _packed(name, n_seq, min_len, max_len, Hq, Hkv, P, len_seed, n_frozen=0):
    return {"name": name, "kind": "packed", "n_seq": n_seq, "min_len": min_len, "max_len": max_len, "Hq": Hq,
            "Hkv": Hkv, "D": 128, "P": P, "len_seed": len_seed, "n_frozen": n_frozen, "dtype": "bf16"}


def _loss(name, N, V, K, dtype, mode):
    return {"name": name, "kind": "loss", "N": N, "V": V, "K": K, "dtype": dtype, "mode": mode}


def _topk(name, N, V, K, dtype):
    return {"name": name, "kind": "topk", "N": N, "V": V, "K": K, "dtype": dtype}


def _decode(name, B, Hq, Hkv, P, n_shared, pool_p, min_len, max_len, len_seed):
    return {"name": name, "kind": "decode", "B": B, "Hq": Hq, "Hkv": Hkv, "D": 128, "P": P, "n_shared": n_shared,
            "pool_p": pool_p, "min_len": min_len, "max_len": max_len, "len_seed": len_seed, "dtype": "bf16"}


def listed():
    return [
        # ---- attention of one layer, forward and backward ---------------------------------------
        # the full training batch of the two model shapes (one layer each)
        _train("train_8b", 16, 2048, 32, 8, 4096),
        _train("train_3b", 32, 1024, 24, 8, 2048),
        # the same training on a packed batch: 64 conversations of 64 .. 1024 tokens
        _packed("train_packed", 64, 64, 1024, 32, 8, 4096, 3101),
        # one conversation of odd length on an odd-sized cartridge with a frozen sink slot: a
        # micro-batch of one, as gradient accumulation and small GPUs' settings run it
        _train("train_one_sequence", 1, 700, 32, 8, 1000, n_frozen=1),
        # the fp32 problem gradient checks are run on
        _train("train_f32_tiny", 2, 64, 2, 1, 32, dtype="f32", D=64),
        # ---- distillation loss with its gradient ------------------------------------------------
        # a full batch's logits
        _loss("loss_full", 16384, 128256, 20, "bf16", "topk"),
        # a vocabulary whose rows are not 16-byte multiples, a micro-batch of positions
        _loss("loss_odd_vocab", 1024, 50257, 20, "bf16", "topk"),
        # logits a model head hands over in fp32, rest-bucket reading
        _loss("loss_f32_rest", 2048, 128256, 20, "f32", "rest"),
        # ---- teacher records --------------------------------------------------------------------
        _topk("teacher_topk", 16384, 128256, 20, "bf16"),
        # ---- decode -----------------------------------------------------------------------------
        # a full server: 128 requests share one cartridge
        _decode("decode_shared", 128, 32, 8, 8192, 1, 0, 1, 1024, 5001),
        # every request brings its own cartridge behind a small shared one
        _decode("decode_private", 128, 32, 8, 2048, 1, 2048, 1, 1024, 5001),
        # a nearly idle server: four requests, latency is what counts
        _decode("decode_few", 4, 32, 8, 2048, 1, 0, 1, 150, 5003),
    ]


HEADS = [(32, 8), (32, 8), (24, 8), (8, 2)]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    u = rng.random()
    if u < 0.25:
        # batches of 1 .. 32 sequences of 64 .. 2048 tokens, cartridges of 128 .. 8192 slots or none
        while True:
            Hq, Hkv = rng.choice(HEADS)
            c = _train("", _log(rng, 1, 32), _log(rng, 64, 2048), Hq, Hkv,
                       0 if rng.random() < 0.1 else _log(rng, 128, 8192))
            c["n_frozen"] = 1 if c["P"] and rng.random() < 0.5 else 0
            if work(c)["flops"] <= work(listed()[0])["flops"]:
                break
    elif u < 0.38:
        while True:
            Hq, Hkv = rng.choice(HEADS)
            hi = _log(rng, 128, 1024)
            c = _packed("", _log(rng, 4, 64), _log(rng, 1, hi), hi, Hq, Hkv, _log(rng, 128, 8192), rng.randrange(10000))
            c["n_frozen"] = rng.randrange(2)
            if work(c)["flops"] <= work(listed()[0])["flops"]:
                break
    elif u < 0.44:
        Hq, Hkv = rng.choice([(2, 1), (4, 2), (8, 2)])
        c = _train("", rng.randint(1, 4), _log(rng, 32, 256), Hq, Hkv, rng.choice([0, _log(rng, 16, 256)]), dtype="f32",
                   D=rng.choice([64, 128]))
    elif u < 0.68:
        # positions from a few sequences' tail to a full batch; vocabularies of any size
        while True:
            mode = rng.choice(["topk", "topk", "rest", "ntp"])
            c = _loss("", _log(rng, 32, 16384), _vocab(rng), 1 if mode == "ntp" else rng.randint(5, 64),
                      rng.choice(["bf16", "bf16", "f32"]), mode)
            if work(c)["bytes"] <= work(listed()[5])["bytes"]:
                break
    elif u < 0.80:
        # (the fp32 ones up to what a teacher's generation step hands over at once)
        dtype = rng.choice(["bf16", "bf16", "f32"])
        c = _topk("", _log(rng, 32, 16384 if dtype == "bf16" else 2048), _vocab(rng), rng.randint(5, 64), dtype)
    else:
        # one request to a full server; no, one or several shared cartridges, some with one per
        # request; short and long histories
        while True:
            Hq, Hkv = rng.choice(HEADS)
            n_shared = rng.choice([0, 1, 1, 1, 3])
            B = _log(rng, 1, 128)
            hi = _log(rng, 16, 16384)
            c = _decode("", B, Hq, Hkv, _log(rng, 128, 8192) if n_shared else 0, n_shared,
                        _log(rng, 128, 2048) if rng.random() < 0.25 else 0, 1, hi, rng.randrange(10000))
            if work(c)["bytes"] <= 5.0e9:
                break
    del c["name"]
    return c


def _vocab(rng):
    return rng.choice([128256, 50257, 32000, _log(rng, 4096, 131072), _log(rng, 4096, 131072)])


# ---- inputs -------------------------------------------------------------------------------------
def _lengths(case, n, seed=None):
    """The case's lengths; a seed deals them out in another order (their sum stays)."""
    g = torch.Generator().manual_seed(case["len_seed"])
    lens = torch.randint(case["min_len"], case["max_len"] + 1, (n,), generator=g)
    if seed is None:
        return lens
    return lens[torch.randperm(n, generator=torch.Generator().manual_seed(seed))]


def _offsets(lens):
    cu = torch.zeros(lens.numel() + 1, dtype=torch.int32)
    cu[1:] = torch.cumsum(lens, 0).to(torch.int32)
    return cu.cuda()


def prepare(case, seed):
    kind, dev = case["kind"], "cuda"
    if kind == "train":
        f32 = case["dtype"] == "f32"
        cfg = synth.AttnConfig("", seed, case["B"], case["S"], case["Hq"], case["Hkv"], case["D"], case["P"], case["dtype"],
                               1.0 if f32 else STD, 1.0 if f32 else STD, 1.0 / 8.0 if f32 else Z_STD)
        t = synth.attn_inputs(cfg, dev)
        if case["P"] == 0:
            t["z_k"] = t["z_v"] = None
        return {"case": case, **t}
    if kind == "packed":
        lens = _lengths(case, case["n_seq"], seed)
        T, Hq, Hkv, P = int(lens.sum()), case["Hq"], case["Hkv"], case["P"]
        g = torch.Generator(device=dev).manual_seed(seed)
        rn = lambda *sz, std: synth._normal(sz, std, torch.bfloat16, g, dev)
        return {"case": case, "q": rn(T, Hq, 128, std=STD), "k_own": rn(T, Hkv, 128, std=STD), "v_own": rn(T, Hkv, 128, std=STD),
                "z_k": rn(Hkv, P, 128, std=Z_STD), "z_v": rn(Hkv, P, 128, std=Z_STD), "d_o": rn(T, Hq, 128, std=STD),
                "cu": _offsets(lens), "max_len": int(lens.max())}
    if kind in ("loss", "topk"):
        if kind == "topk":
            g = torch.Generator(device=dev).manual_seed(seed)
            return {"case": case, "logits": synth._normal((case["N"], case["V"]), 3.0, synth.torch_dtype(case["dtype"]), g, dev)}
        t = synth.kl_inputs(synth.KLConfig("", seed, case["N"], case["V"], case["K"], case["dtype"], 3.0, 3.0, 0.95), dev)
        if case["mode"] == "ntp":
            t["teacher_logp"] = None
        return {"case": case, **t}
    lens = _lengths(case, case["B"], seed)
    T, B, Hq, Hkv, P = int(lens.sum()), case["B"], case["Hq"], case["Hkv"], case["P"]
    g = torch.Generator(device=dev).manual_seed(seed)
    rn = lambda *sz, std: synth._normal(sz, std, torch.bfloat16, g, dev)
    n = case["n_shared"]
    cuts = [P * i // n for i in range(n + 1)] if n else [0]
    st = {"case": case, "q": rn(B, Hq, 128, std=STD),
          "shared": [(rn(Hkv, b - a, 128, std=Z_STD), rn(Hkv, b - a, 128, std=Z_STD)) for a, b in zip(cuts, cuts[1:])],
          "k_own": rn(T, Hkv, 128, std=STD), "v_own": rn(T, Hkv, 128, std=STD), "cu": _offsets(lens), "max_len": int(lens.max())}
    if case["pool_p"]:
        st["pool_k"] = rn(B, Hkv, case["pool_p"], 128, std=Z_STD)
        st["pool_v"] = rn(B, Hkv, case["pool_p"], 128, std=Z_STD)
        st["cart_id"] = torch.randperm(B, generator=g, device=dev).to(torch.int32)
    return st


# ---- one pass -----------------------------------------------------------------------------------
def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "train":
        a = (st["q"], st["k_own"], st["v_own"], st["z_k"], st["z_v"])
        o, lse = cart.cart_attn_fwd(*a)
        return (o, lse) + tuple(cart.cart_attn_bwd(*a, o, lse, st["d_o"], n_frozen=case["n_frozen"]))
    if kind == "packed":
        a = (st["q"], st["k_own"], st["v_own"], st["z_k"], st["z_v"], st["cu"], st["max_len"])
        o, lse = cart.cart_attn_varlen_fwd(*a)
        return (o, lse) + tuple(cart.cart_attn_varlen_bwd(*a, o, lse, st["d_o"], n_frozen=case["n_frozen"]))
    if kind == "loss":
        mode = cart.KL_REST if case["mode"] == "rest" else cart.KL_TOPK
        return cart.cart_distill_kl_fwd_bwd(st["logits"], st["teacher_idx"], st["teacher_logp"], 1.0 / case["N"], mode=mode)
    if kind == "topk":
        return cart.cart_teacher_topk(st["logits"], case["K"])
    own = (st["k_own"], st["v_own"], st["cu"], st["max_len"])
    if len(st["shared"]) <= 1 and not case["pool_p"]:
        z_k, z_v = st["shared"][0] if st["shared"] else (None, None)
        return cart.cart_decode(st["q"], z_k, z_v, *own)
    return cart.cart_decode_composed(st["q"], st["shared"], st.get("pool_k"), st.get("pool_v"), st.get("cart_id"), *own)


# ---- what a pass cannot do without, and how close another correct program comes -----------------
def work(case):
    kind, es = case["kind"], 4 if case["dtype"] == "f32" else 2
    if kind in ("train", "packed"):
        Hq, Hkv, D, P = case["Hq"], case["Hkv"], case["D"], case["P"]
        lens = [case["S"]] * case["B"] if kind == "train" else _lengths(case, case["n_seq"]).tolist()
        T = sum(lens)
        pairs = Hq * sum(n * P + n * (n + 1) // 2 for n in lens)
        # in: q, dO, own K and V, Z; out: O, LSE, dQ, dK, dV, dZ (fp32)
        return {"bytes": es * (4 * T * Hq * D + 4 * T * Hkv * D + 2 * Hkv * P * D) + 4 * T * Hq + 8 * Hkv * P * D,
                "flops": 14 * D * pairs}        # 2 contractions forward, 5 backward
    if kind == "loss":
        N, V, K = case["N"], case["V"], case["K"]
        return {"bytes": 2 * es * N * V + 8 * N * K, "flops": 6 * N * V}
    if kind == "topk":
        N, V, K = case["N"], case["V"], case["K"]
        return {"bytes": es * N * V + 8 * N * K, "flops": 3 * N * V}
    B, Hq, Hkv, D = case["B"], case["Hq"], case["Hkv"], case["D"]
    T = int(_lengths(case, B).sum())
    keys = T + B * (case["P"] + case["pool_p"])
    return {"bytes": es * (2 * B * Hq * D + 2 * T * Hkv * D + 2 * Hkv * case["P"] * D + 2 * B * Hkv * case["pool_p"] * D) + 4 * B * Hq,
            "flops": 4 * D * keys * Hq}


def tolerance(case):
    """About four times the distance of each entry point from the same computation in 64 bits
    (2-norm, and the largest difference over the larger of the value and the tensor's rms)."""
    if case["kind"] == "topk":
        # seen: 1.7e-7, 4.2e-7; the indices are exact (comparisons of stored values)
        return {"rel": 1e-6, "max": 2e-6, "differ": 0.0}
    if case["kind"] == "loss":
        # fp32, seen: 1.1e-7, 1.6e-6; bf16, one rounding (2^-9) of every gradient: 1.65e-3, 3.9e-3
        return {"rel": 1e-6, "max": 1e-5} if case["dtype"] == "f32" else {"rel": 6e-3, "max": 1.6e-2}
    if case["dtype"] == "f32":
        # seen: 1.1e-6, 5.6e-6 (dZ of 4 x 200 rows)
        return {"rel": 5e-6, "max": 3e-5}
    # bf16 P and dS as operands, one rounding of every output; seen: 2.8e-3, 1.3e-2
    return {"rel": 1.1e-2, "max": 6e-2}
