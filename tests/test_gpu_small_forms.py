"""The kernels that a batch of more than four messages per SIMD (4096 on 1024
SIMDs) reaches, at the edges of their blocks: below that number a batch with no
tile is hashed in the wide form alone.  Byte for byte against the CPU oracle.
Needs an MI355X; run with -m gpu."""

import numpy as np
import pytest

from paper_1902_05320_amd import workloads as wl

pytestmark = pytest.mark.gpu

RATES = (144, 136, 104, 72)
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


def _at_offsets(lens, mod16, variants, seed, step):
    """Message i at byte step * i + mod16[i] of one buffer, which ends with the
    last message (step a multiple of 16 that holds one)."""
    rng = np.random.Generator(np.random.PCG64(seed))
    offs = step * np.arange(lens.size, dtype=np.int64) + mod16
    data = rng.integers(0, 256, int((offs + lens).max()), dtype=np.uint8)
    return wl.Batch(data, offs, lens.astype(np.int64), variants.astype(np.uint8), seed, "offsets")


def _dev(b):
    import torch
    return (torch.from_numpy(b.data).cuda(), torch.from_numpy(b.offsets).cuda(),
            torch.from_numpy(b.lengths).cuda(), torch.from_numpy(b.variants).cuda())


def _mixed_want(o2, b):
    good = b.variants < 4
    want = o2.sha3_batch_mixed(np.where(good, b.variants, 0).astype(np.uint8), b.data, b.offsets, b.lengths)
    return np.where(good[:, None], want, 0).astype(np.uint8)


def _compare(kb, o2, v, b, **kw):
    import torch
    data, offs, lens, var = _dev(b)
    if v < 0:
        got, want = kb.keccak_batch_mixed(var, data, offs, lens, **kw), _mixed_want(o2, b)
    else:
        got = kb.keccak_batch(v, data, offs, lens, **kw)
        want = o2.sha3_batch(8 * DIGEST[v], b.data, b.offsets, b.lengths)
    torch.cuda.synchronize()
    bad = np.nonzero((got.cpu().numpy() != want).any(axis=1))[0]
    assert bad.size == 0, (bad[:10].tolist(), b.lengths[bad[:10]].tolist(), b.offsets[bad[:10]].tolist())


@pytest.mark.parametrize("v", [-1, 0, 1, 2, 3])
def test_one_block_chunks_at_every_length_and_offset(kb, o2, v):
    # every length of one block, 0 to R - 1 (of the message's own variant in the
    # mixed form), at every address mod 16: chunks that the first pass hashes
    n = 4 * 16 * max(RATES)
    i = np.arange(n)
    var = i % 4 if v < 0 else np.full(n, v)
    rate = np.asarray(RATES)[var]
    i = i // 4 if v < 0 else i
    b = _at_offsets(i % rate, i // rate % 16, var, 161, 160)
    assert len(set(zip(b.variants.tolist(), b.lengths.tolist(), (b.offsets % 16).tolist()))) == \
        16 * (sum(RATES) if v < 0 else RATES[v])
    _say("one-block chunks", v)
    _compare(kb, o2, v, b)


@pytest.mark.parametrize("security", [128, 256])
def test_xof_one_block_chunks_at_every_length_and_offset(kb, o2, security):
    import torch
    R = 168 if security == 128 else 136
    n = 32 * R
    i = np.arange(n)
    b = _at_offsets(i % R, i // R % 16, np.zeros(n), 162, 192)
    data, offs, lns, _ = _dev(b)
    _say("xof one-block chunks", security)
    for out_len in (33, R + 2):
        got = kb.keccak_batch_xof(security, data, offs, lns, out_len)
        torch.cuda.synchronize()
        got = got.cpu().numpy()
        for i in range(n):
            m = b.data[b.offsets[i]:b.offsets[i] + b.lengths[i]].tobytes()
            assert got[i].tobytes() == o2.shake(security, m, out_len), (out_len, i)


@pytest.mark.parametrize("n", [7_000, 70_001])
@pytest.mark.parametrize("v", [-1, 0, 1, 2, 3])
def test_deferred_chunks_at_every_length_and_offset(kb, o2, v, n):
    # up to three blocks, at every address mod 16: all in the pair form, and
    # (more than 65536) one thread per message with the longest in pairs
    R = max(RATES) if v < 0 else RATES[v]
    rng = np.random.Generator(np.random.PCG64(163))
    i = np.arange(n)
    b = _at_offsets(i % (3 * R + 2), i // (3 * R + 2) % 16, rng.integers(0, 4, n), 164, 448)
    _say("deferred chunks", v, n)
    _compare(kb, o2, v, b)


@pytest.mark.parametrize("n,longest", [(5_000, 71), (5_000, 500), (66_000, 71), (66_000, 500), (66_000, 9_000)])
def test_invalid_variants_give_zero_slots_in_every_form(kb, o2, n, longest):
    # variant bytes of 4 and more in chunks of one block, in pair items and in
    # one-thread items; in the last case long messages with invalid variants
    # lie among those of the split tail
    rng = np.random.Generator(np.random.PCG64(165))
    lens = rng.integers(0, longest + 1, n) if longest < 9_000 else wl.log_uniform_lengths(rng, n, longest)
    var = rng.integers(0, 4, n)
    var[::3] = rng.integers(4, 256, var[::3].size)
    b = wl.explicit(lens, seed=166, variant=var.astype(np.uint8), gap=1, lead=3)
    _say("invalid variants", n, longest)
    _compare(kb, o2, -1, b)


@pytest.mark.parametrize("n", [1, 300, 3000, 4096])
def test_small_batches_through_the_two_passes(kb, o2, n):
    # a tile keeps a small batch in the two passes: few messages, all long (all
    # of them split items, up to twice the usual number of those), short, equal
    rng = np.random.Generator(np.random.PCG64(167))
    t = kb.Tile()
    t.steps_per_item = 4
    for name, lens in (("long", rng.integers(6_000, 9_000, n)), ("short", rng.integers(0, 300, n)),
                       ("empty", np.zeros(n, np.int64)), ("equal", np.full(n, 64))):
        b = wl.explicit(lens, seed=168, variant=rng.integers(0, 4, n).astype(np.uint8), gap=1, lead=3)
        _say("two passes", n, name)
        for v in (-1, 1, 3):
            if b.data.size:
                _compare(kb, o2, v, b, tile=t)


def test_slices_that_end_with_the_buffer(kb, o2):
    # most of 5000 overlapping slices end within two bytes of the end
    rng = np.random.Generator(np.random.PCG64(169))
    n = 5_000
    data = rng.integers(0, 256, 5000, dtype=np.uint8)
    for most in (60, 400):
        lens = rng.integers(0, most, n)
        offs = np.maximum(data.size - lens - rng.integers(0, 3, n), 0)
        b = wl.Batch(data, offs.astype(np.int64), lens.astype(np.int64), rng.integers(0, 4, n).astype(np.uint8), 8, "ov")
        _say("slices at the end", most)
        for v in (-1, 0, 1, 2, 3):
            _compare(kb, o2, v, b)
