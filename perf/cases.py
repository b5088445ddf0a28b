"""The work that a program has this library do, as cases to be timed.

Every case goes through the public entry points of
``paper_1902_05320_amd.kbatch`` with inputs resident on the GPU, as the
library takes them (the server's requests are host arrays, as it takes
those).  Sizes follow the repository's own workloads (the uniform 2^24 x 64 B
batch, the uneven mixed batch, the 1 GiB tree, the serving stream, the
latency shapes) and spread around them; inputs are uniform random bytes,
lengths are equal or log-uniform, and messages are packed back to back.

Kinds: ``batch`` (one variant), ``mixed`` (a variant per message), ``xof``,
``merkle``, ``keccak_p``, ``graph`` (a captured batch, replayed) and
``serve`` (a burst of requests to the server).
"""

from __future__ import annotations

import hashlib
import math

import numpy as np
import torch

from paper_1902_05320_amd import kbatch

# 32-bit operations of one Keccak-f[1600] with three-input logic operations:
# theta 80, rho 48 and chi 50 a round, iota 37 in all
OPS = 24 * 178 + 37
RATE = (144, 136, 104, 72)
DIGEST = (28, 32, 48, 64)


def listed():
    return [
        # one file's digest: a single chain of permutations, pure latency
        {"name": "single_1MiB", "kind": "batch", "variant": 1, "n": 1, "len": 1 << 20,
         "spread": False, "checked": True},
        # a handful of records of two to three blocks through the default
        # call: launches, argument checks and the host are the cost
        {"name": "tiny_17x200B", "kind": "batch", "variant": 3, "n": 17, "len": 200,
         "spread": False, "checked": True},
        # a program's own small batch of short messages, captured once and
        # replayed: what the launches themselves cost
        {"name": "graph_4096x64B", "kind": "graph", "variant": 1, "n": 4096, "len": 64,
         "spread": False},
        # the headline batch: many short equal messages, into a kept output
        {"name": "uniform_16M_64B", "kind": "batch", "variant": 1, "n": 1 << 24, "len": 64,
         "spread": False, "checked": False},
        # pages of one size, fewer than the chip has lanes
        {"name": "pages_32768x4KiB", "kind": "batch", "variant": 1, "n": 32768, "len": 4096,
         "spread": False, "checked": False},
        # records of an odd size at odd addresses, the default call, SHA3-384
        {"name": "records_100003x1001B", "kind": "batch", "variant": 2, "n": 100003, "len": 1001,
         "spread": False, "checked": True},
        # a large batch of everything: lengths over four decades, a variant
        # per message
        {"name": "uneven_mixed_1M", "kind": "mixed", "n": 1 << 20, "len": 16384},
        # seeds expanded to a kilobyte of output each with SHAKE128
        {"name": "xof_65537x33B_1000B", "kind": "xof", "security": 128, "n": 65537, "len": 33,
         "out_len": 1000},
        # the hash tree of a large buffer of pages
        {"name": "merkle_1GiB_4KiB", "kind": "merkle", "variant": 1, "len": 1 << 30, "leaf": 4096},
        # the hash tree of a small file in odd pieces
        {"name": "merkle_5MB_odd", "kind": "merkle", "variant": 1, "len": 5000001, "leaf": 1000},
        # the bare permutation over a set of states, in place
        {"name": "keccak_p1600_1M", "kind": "keccak_p", "b": 1600, "rounds": 24, "n": 1 << 20},
        # a burst of requests at the server, as the serving stream draws them
        {"name": "serve_6_requests", "kind": "serve", "requests": 6, "max_msgs": 4096,
         "len": 65536},
    ]


def _logint(rng, lo, hi):
    return min(hi, max(lo, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def draw(rng):
    kind = rng.choice(("batch", "batch", "batch", "mixed", "xof", "merkle", "keccak_p", "graph",
                       "serve"))
    if kind == "batch":
        n = _logint(rng, 1, 1 << 24)
        variant = rng.randrange(4)
        # at most 2^30 bytes and 12 M blocks in all, messages to 1 MiB
        most = max(1, min(1 << 20, (1 << 30) // n, (12_000_000 // n) * RATE[variant]))
        return {"kind": "batch", "variant": variant, "n": n, "len": _logint(rng, 1, most),
                "spread": n > 16 and rng.random() < 0.5, "checked": rng.random() < 0.5}
    if kind == "mixed":
        return {"kind": "mixed", "n": _logint(rng, 16, 1 << 19), "len": _logint(rng, 32, 16384)}
    if kind == "xof":
        n = _logint(rng, 1, 1 << 17)
        return {"kind": "xof", "security": rng.choice((128, 256)), "n": n,
                "len": _logint(rng, 1, 2000), "out_len": _logint(rng, 16, 4000)}
    if kind == "merkle":
        total = _logint(rng, 1, 1 << 29)
        leaf = _logint(rng, 64, 1 << 16)
        if rng.random() < 0.5:  # pages of whole words
            leaf -= leaf % 64
            total -= total % 8
        return {"kind": "merkle", "variant": rng.randrange(4), "len": max(total, 1), "leaf": leaf}
    if kind == "keccak_p":
        b = rng.choice((200, 400, 800, 1600, 1600))
        return {"kind": "keccak_p", "b": b, "rounds": rng.choice((12, 24, 12 + 2 * int(math.log2(b // 25)))),
                "n": _logint(rng, 1, 1 << 20)}
    if kind == "graph":
        n = _logint(rng, 1, 1 << 17)
        return {"kind": "graph", "variant": rng.randrange(4), "n": n, "len": _logint(rng, 1, 2000),
                "spread": n > 16 and rng.random() < 0.5}
    return {"kind": "serve", "requests": rng.randint(1, 6), "max_msgs": _logint(rng, 16, 4096),
            "len": _logint(rng, 64, 65536)}


# --------------------------------------------------------------------------
# Inputs, from the seed alone
# --------------------------------------------------------------------------

def _lengths(gen, n, length, spread):
    """n lengths: all `length`, or log-uniform in [0, length]."""
    if not spread:
        return torch.full((n,), length, dtype=torch.int64)
    u = torch.rand(n, generator=gen, dtype=torch.float64)
    return (float(length + 2) ** u).floor().to(torch.int64).sub_(1).clamp_(0, length)


def _spread(case):
    return case["kind"] in ("mixed", "serve") or bool(case.get("spread"))


def _batch_lengths(case, seed):
    """(lengths, variants) of a batch, on the host."""
    gen = torch.Generator().manual_seed(int(seed) * 3 + 1)
    lens = _lengths(gen, case["n"], case["len"], _spread(case))
    var = torch.randint(0, 4, (case["n"],), generator=gen, dtype=torch.uint8)
    return lens, var


def _bytes(nbytes, seed):
    gen = torch.Generator(device="cuda").manual_seed(int(seed) * 3 + 2)
    words = torch.randint(-(1 << 63), (1 << 63) - 1, ((max(nbytes, 1) + 7) // 8,), generator=gen,
                          device="cuda")
    return words.view(torch.uint8)[:nbytes]


def _requests(case, seed):
    """(variant, offsets, lengths) of each request, host arrays, and the pool's size."""
    rng = np.random.Generator(np.random.PCG64(int(seed)))
    pool = 1 << 26
    out = []
    for q in range(case["requests"]):  # sizes spread over 1 .. max_msgs
        k = max(1, case["max_msgs"] * (2 * q + 1) // (2 * case["requests"]))
        lens = np.floor(np.power(float(case["len"] + 2), rng.random(k))).astype(np.int64) - 1
        lens = np.clip(lens, 0, case["len"])
        offs = rng.integers(0, pool - case["len"], size=k, dtype=np.int64)
        out.append((1 if rng.random() < 0.5 else 3, offs, lens))
    return out, pool


def prepare(case, seed):
    kind = case["kind"]
    st = {"case": case}
    if kind == "merkle":
        st["data"] = _bytes(case["len"], seed)
        return st
    if kind == "keccak_p":
        nb = (case["b"] + 7) // 8
        st["states"] = _bytes(case["n"] * nb, seed).reshape(case["n"], nb)
        return st
    if kind == "serve":
        st["requests"], pool = _requests(case, seed)
        st["pool"] = _bytes(pool, seed)
        st["server"] = kbatch.Server(st["pool"], max_step_msgs=1 << 16, steps_in_flight=3)
        return st
    lens, var = _batch_lengths(case, seed)
    offs = torch.cumsum(lens, 0) - lens
    st["data"] = _bytes(int(lens.sum()), seed)
    if st["data"].numel() == 0:
        st["data"] = torch.zeros(1, dtype=torch.uint8, device="cuda")
    st["offsets"], st["lengths"] = offs.cuda(), lens.cuda()
    if kind == "mixed":
        st["variants"] = var.cuda()
        st["out"] = torch.empty((case["n"], 64), dtype=torch.uint8, device="cuda")
    elif kind == "graph" or not case.get("checked", True):
        st["out"] = torch.empty((case["n"], DIGEST[case["variant"]]), dtype=torch.uint8, device="cuda")
    if kind == "graph":
        st["graph"] = kbatch.graph_batch(case["variant"], st["data"], st["offsets"], st["lengths"],
                                         st["out"])
    return st


# --------------------------------------------------------------------------
# One pass
# --------------------------------------------------------------------------

def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "batch":
        if case["checked"]:  # the default call: bounds checked, a new output
            return kbatch.keccak_batch(case["variant"], st["data"], st["offsets"], st["lengths"])
        return kbatch.keccak_batch(case["variant"], st["data"], st["offsets"], st["lengths"],
                                   out=st["out"], check_bounds=False)
    if kind == "mixed":
        return kbatch.keccak_batch_mixed(st["variants"], st["data"], st["offsets"], st["lengths"],
                                         out=st["out"], check_bounds=False)
    if kind == "xof":
        return kbatch.keccak_batch_xof(case["security"], st["data"], st["offsets"], st["lengths"],
                                       case["out_len"])
    if kind == "merkle":
        return kbatch.merkle_root(case["variant"], st["data"], case["leaf"])
    if kind == "keccak_p":
        return kbatch.keccak_p_batch(case["b"], case["rounds"], st["states"])
    if kind == "graph":
        st["graph"].replay()
        return st["out"]
    server = st["server"]
    sizes = {}
    for variant, offs, lens in st["requests"]:
        sizes[server.submit(variant, offs, lens)] = offs.size
    got = {}
    while len(got) < len(sizes):
        for rid in server.poll(wait_ms=100):
            got[rid] = server.result(rid, sizes[rid])[0]
    return [got[rid] for rid in sizes]


# --------------------------------------------------------------------------
# What a pass cannot do without
# --------------------------------------------------------------------------

def _blocks(lens, rate):
    return int((lens // rate + 1).sum())


def _tree_nodes(leaves):
    """Node pairs hashed above `leaves` leaves (an unpaired last node is carried up)."""
    pairs = 0
    while leaves > 1:
        pairs += leaves // 2
        leaves = (leaves + 1) // 2
    return pairs


def work(case):
    kind = case["kind"]
    if kind == "keccak_p":
        w = case["b"] // 25
        nb = (case["b"] + 7) // 8
        return {"bytes": 2 * nb * case["n"],
                "flops": case["n"] * case["rounds"] * 178 * (1.0 if w == 64 else 0.5)}
    if kind == "merkle":
        v = case["variant"]
        leaves = -(-case["len"] // case["leaf"])
        last = case["len"] - (leaves - 1) * case["leaf"]
        perms = (leaves - 1) * (case["leaf"] // RATE[v] + 1) + last // RATE[v] + 1
        perms += _tree_nodes(leaves) * (2 * DIGEST[v] // RATE[v] + 1)
        return {"bytes": case["len"] + DIGEST[v], "flops": perms * OPS}
    if kind == "serve":
        reqs, _ = _requests(case, 1)
        perms = sum(_blocks(lens, RATE[v]) for v, _, lens in reqs)
        total = sum(int(lens.sum()) + 80 * lens.size for _, _, lens in reqs)
        return {"bytes": total, "flops": perms * OPS}
    lens, var = _batch_lengths(case, 1)
    total, n = int(lens.sum()), case["n"]
    if kind == "mixed":
        perms = sum(_blocks(lens[var == v], RATE[v]) for v in range(4))
        return {"bytes": total + 17 * n + 64 * n, "flops": perms * OPS}
    if kind == "xof":
        rate = 168 if case["security"] == 128 else 136
        perms = _blocks(lens, rate) + n * ((case["out_len"] - 1) // rate)
        return {"bytes": total + 16 * n + case["out_len"] * n, "flops": perms * OPS}
    v = case["variant"]
    return {"bytes": total + 16 * n + DIGEST[v] * n, "flops": _blocks(lens, RATE[v]) * OPS}


# --------------------------------------------------------------------------
# The same results from Python's hashlib
# --------------------------------------------------------------------------

_SHA3 = (hashlib.sha3_224, hashlib.sha3_256, hashlib.sha3_384, hashlib.sha3_512)


def _digests(data, offs, lens, hash_of, width):
    buf = memoryview(data)
    out = np.zeros((len(offs), width), dtype=np.uint8)
    for i, (o, n) in enumerate(zip(offs.tolist(), lens.tolist())):
        d = hash_of(i, buf[o:o + n])
        out[i, :len(d)] = np.frombuffer(d, dtype=np.uint8)
    return out


def exact(case, seed):
    """What run() returns, from hashlib; None where that takes too long (or, for the bare
    permutation, where it has no such function)."""
    kind = case["kind"]
    if kind == "keccak_p" or work(case)["flops"] > 3e6 * OPS:
        return None
    if kind == "merkle":
        h = _SHA3[case["variant"]]
        data = memoryview(_bytes(case["len"], seed).cpu().numpy())
        level = [h(data[i:i + case["leaf"]]).digest() for i in range(0, case["len"], case["leaf"])]
        while len(level) > 1:
            up = [h(level[i] + level[i + 1]).digest() for i in range(0, len(level) - 1, 2)]
            level = up + level[len(level) - len(level) % 2:]
        return np.frombuffer(level[0], dtype=np.uint8)
    if kind == "serve":
        reqs, pool = _requests(case, seed)
        data = _bytes(pool, seed).cpu().numpy()
        return [_digests(data, offs, lens, lambda i, m, h=_SHA3[v]: h(m).digest(), 64)
                for v, offs, lens in reqs]
    lens, var = _batch_lengths(case, seed)
    offs = (torch.cumsum(lens, 0) - lens).numpy()
    data = _bytes(int(lens.sum()), seed).cpu().numpy()
    if kind == "mixed":
        return _digests(data, offs, lens.numpy(), lambda i, m: _SHA3[var[i]](m).digest(), 64)
    if kind == "xof":
        h = hashlib.shake_128 if case["security"] == 128 else hashlib.shake_256
        k = case["out_len"]
        return _digests(data, offs, lens.numpy(), lambda i, m: h(m).digest(k), k)
    h = _SHA3[case["variant"]]
    return _digests(data, offs, lens.numpy(), lambda i, m: h(m).digest(), DIGEST[case["variant"]])
