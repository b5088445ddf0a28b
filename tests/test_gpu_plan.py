"""What the plan of a bucketed batch decides on the device: which messages go to
the wide split tail, which to the pair form, and which waves take them.  Every
case is compared with the CPU oracle, byte for byte.  Needs an MI355X; run
with -m gpu."""

import time

import numpy as np
import pytest

from paper_1902_05320_amd import workloads as wl

pytestmark = pytest.mark.gpu

DIGEST = (28, 32, 48, 64)


@pytest.fixture(scope="module")
def kb():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1902_05320_amd import kbatch
    kbatch.load_library()
    return kbatch


def _say(*a):
    print("[case]", *a, flush=True)


def _dev(b):
    import torch
    return (torch.from_numpy(b.data).cuda(), torch.from_numpy(b.offsets.astype(np.int64)).cuda(),
            torch.from_numpy(b.lengths.astype(np.int64)).cuda(),
            torch.from_numpy(b.variants.astype(np.uint8)).cuda())


def _check(kb, o2, b, variants=(-1, 1, 3), tile=None):
    import torch
    data, offs, lens, var = _dev(b)
    for v in variants:
        if v < 0:
            got = kb.keccak_batch_mixed(var, data, offs, lens, tile=tile)
            want = o2.sha3_batch_mixed(b.variants, b.data, b.offsets, b.lengths)
        else:
            got = kb.keccak_batch(v, data, offs, lens, tile=tile)
            want = o2.sha3_batch(8 * DIGEST[v], b.data, b.offsets, b.lengths)
        torch.cuda.synchronize()
        assert np.array_equal(got.cpu().numpy(), want), v


LONG = {
    # two waves per SIMD take the split tail (nothing after it is long)
    "tail_then_short": lambda r: np.concatenate([r.integers(15_000, 17_000, 3000), r.integers(0, 900, 60_000)]),
    # a second wave starts on the long messages beside the tail
    "tail_then_long": lambda r: np.concatenate([r.integers(9_000, 17_000, 9000), r.integers(0, 900, 60_000)]),
    # everything past the tail in pairs at its bounds: 32 messages on each wave
    # that takes no split items (1024 of the mixed kernel's)
    "pairs_34815": lambda r: np.concatenate([r.integers(9_000, 17_000, 2048), r.integers(0, 400, 32_767)]),
    "pairs_34817": lambda r: np.concatenate([r.integers(9_000, 17_000, 2048), r.integers(0, 400, 32_769)]),
    # more messages than that: pairs by the length of the chain alone
    "log_uniform_70001": lambda r: wl.log_uniform_lengths(r, 70_001, 9_000),
    "linear_70001": lambda r: r.integers(0, 3_000, 70_001),
    "log_uniform_300001": lambda r: wl.log_uniform_lengths(r, 300_001, 3_000),
}


@pytest.mark.parametrize("case", list(LONG))
def test_long_messages_past_the_split_tail(kb, o2, case):
    rng = np.random.Generator(np.random.PCG64(130))
    lens = LONG[case](rng)
    rng.shuffle(lens)
    b = wl.explicit(lens, seed=131, variant=rng.integers(0, 4, lens.size).astype(np.uint8), gap=1, lead=3)
    _say("plan", case, b.n)
    _check(kb, o2, b)


@pytest.mark.parametrize("security", [128, 256])
@pytest.mark.parametrize("n,out_len", [(5_000, 700), (40_000, 100), (40_000, 700), (70_001, 700)])
def test_xof_plan_counts_the_squeezes(kb, o2, security, n, out_len):
    # chains of one to ten blocks and none or several more permutations for the
    # output: pairs whole, by the shortest chain, by the mean chain
    import torch
    rng = np.random.Generator(np.random.PCG64(136))
    b = wl.explicit(wl.log_uniform_lengths(rng, n, 1300), seed=137, gap=1, lead=3)
    data, offs, lens, _ = _dev(b)
    _say("xof plan", security, n, out_len)
    got = kb.keccak_batch_xof(security, data, offs, lens, out_len)
    torch.cuda.synchronize()
    got = got.cpu().numpy()
    for i in range(0, n, 7):
        m = b.data[b.offsets[i]:b.offsets[i] + b.lengths[i]].tobytes()
        assert got[i].tobytes() == o2.shake(security, m, out_len), i


@pytest.mark.parametrize("n", [5_000, 32_768, 32_769, 65_536, 65_537])
@pytest.mark.parametrize("steps", [0, 1, 7])
def test_short_messages_in_items_of_their_own(kb, o2, n, steps):
    # one to six blocks: pairs of one message each up to 32768, from five blocks
    # on up to 65536, then several messages to an item; a tile's steps hold
    # whatever the batch
    rng = np.random.Generator(np.random.PCG64(134))
    lens = rng.choice([40, 71, 72, 143, 144, 150, 287, 288, 360, 431], n)
    lens[::64] = 600  # no chunk of one-block messages
    b = wl.explicit(lens, seed=135, variant=rng.integers(0, 4, n).astype(np.uint8), gap=1, lead=3)
    t = None
    if steps:
        t = kb.Tile()
        t.steps_per_item = steps
    _say("short messages", n, "steps", steps)
    _check(kb, o2, b, variants=(-1, 0, 3), tile=t)


def test_short_uneven_batch_keeps_its_time(kb):
    # 10^4 SHA3-224 messages of one block or two, against the same with the four
    # steps per item of a tile: 0.68 of the time, 1.0 when the plan took four too
    import torch
    rng = np.random.Generator(np.random.PCG64(6))
    n = 10_000
    lens = wl.log_uniform_lengths(rng, n, 200)
    offs = np.cumsum(lens) - lens
    data = torch.randint(0, 256, (int(lens.sum()),), dtype=torch.uint8, device="cuda")
    o, l = torch.from_numpy(offs).cuda(), torch.from_numpy(lens).cuda()
    out = torch.empty((n, 28), dtype=torch.uint8, device="cuda")
    four = kb.Tile()
    four.steps_per_item = 4
    best = {}
    for tile in (None, four) * 10:
        torch.cuda.synchronize()
        t = time.perf_counter()
        for _ in range(10):
            kb.keccak_batch(0, data, o, l, out=out, tile=tile, check_bounds=False)
        torch.cuda.synchronize()
        best[tile is None] = min(best.get(tile is None, 1e9), time.perf_counter() - t)
    _say("short uneven 10000", {k: round(1e5 * v) for k, v in best.items()})
    assert best[True] < 0.85 * best[False]


@pytest.mark.parametrize("waves", [1, 2])
def test_split_tail_with_few_waves(kb, o2, waves):
    # with one wave per SIMD none is left beside the split tail
    rng = np.random.Generator(np.random.PCG64(132))
    lens = LONG["tail_then_long"](rng)
    b = wl.explicit(lens, seed=133, variant=rng.integers(0, 4, lens.size).astype(np.uint8), gap=1, lead=1)
    t = kb.Tile()
    t.waves_per_simd = waves
    _say("split tail, waves per SIMD", waves)
    _check(kb, o2, b, tile=t)


def test_uneven_batch_of_few_waves_keeps_its_time(kb):
    # 10^5 mixed messages of up to 16 KiB, log-uniform, against one thread per
    # message: 0.34 of its time; 0.50 when the messages after the split tail
    # waited for it.  (Best of several runs of either; the bound lies halfway.)
    import torch
    rng = np.random.Generator(np.random.PCG64(5))
    n = 100_000
    lens = wl.log_uniform_lengths(rng, n, 16384)
    offs = np.cumsum(lens) - lens
    data = torch.randint(0, 256, (int(lens.sum()),), dtype=torch.uint8, device="cuda")
    var = torch.from_numpy(rng.integers(0, 4, n).astype(np.uint8)).cuda()
    o, l = torch.from_numpy(offs).cuda(), torch.from_numpy(lens).cuda()
    out = torch.empty((n, 64), dtype=torch.uint8, device="cuda")
    best = {}
    for mode in ("persistent", "plain") * 12:
        torch.cuda.synchronize()
        t = time.perf_counter()
        kb.keccak_batch_mixed(var, data, o, l, out=out, mode=mode, check_bounds=False)
        torch.cuda.synchronize()
        best[mode] = min(best.get(mode, 1e9), time.perf_counter() - t)
    _say("uneven 100000", {k: round(1e6 * v) for k, v in best.items()})
    assert best["persistent"] < 0.42 * best["plain"]
