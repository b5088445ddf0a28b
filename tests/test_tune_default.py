"""The library's own choice as a tuning result: stored, it takes the place of
earlier choices; looked up, a batch call runs as with no tile; and the autotuner
returns it where it is the fastest (a small batch, one wide launch)."""

import json

import numpy as np
import pytest

from paper_1902_05320_amd import workloads as wl


@pytest.fixture(scope="module")
def kb():
    from paper_1902_05320_amd import kbatch
    kbatch.load_library()
    return kbatch


def test_stored_default_removes_the_class_choices(kb, tmp_path):
    path = str(tmp_path / "tune.json")
    key = dict(arch="gfx950", rocm="7.2")
    t = kb.Tile()
    t.waves_per_simd = 2
    t.class_threads[7], t.class_steps[1] = 32, 4
    kb.tune_store(path, 1, 300, t, **key)
    kb.tune_store(path, 1, 5000, t, **key)  # another batch class
    kb.tune_store(path, 2, 300, t, **key)  # another variant
    kb.tune_store(path, 1, 400, kb.Tile(), **key)  # 300's batch class
    got = kb.tune_lookup(1, 300, path=path, **key)
    assert got is not None and got.as_dict() == kb.Tile().as_dict()
    assert kb.tune_lookup(1, 5000, path=path, **key).as_dict() == t.as_dict()
    assert kb.tune_lookup(2, 300, path=path, **key).as_dict() == t.as_dict()
    assert len(json.load(open(path))["entries"]) == 3 + 3 + 1
    kb.tune_store(path, 1, 300, t, **key)  # and a choice the place of the default
    assert kb.tune_lookup(1, 300, path=path, **key).as_dict() == t.as_dict()


def _batch(n, length, seed):
    import torch
    b = wl.uniform(n, length, seed=seed)
    return b, (torch.from_numpy(b.data).cuda(), torch.from_numpy(b.offsets.astype(np.int64)).cuda(),
               torch.from_numpy(b.lengths.astype(np.int64)).cuda())


def _launches(kb, fn):
    import torch
    kb.timing_enable(True)
    out = fn()
    torch.cuda.synchronize()
    n = kb.timing_read()[1]
    kb.timing_enable(False)
    return out, n


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1, 300, 2048, 2049, 4096, 4097])
def test_cached_default_runs_as_no_tile(kb, o2, n, tmp_path, monkeypatch):
    b, dev = _batch(n, 200, 140)
    path = str(tmp_path / "tune.json")
    kb.tune_store(path, 1, n, kb.Tile())
    want, launches = _launches(kb, lambda: kb.keccak_batch(1, *dev))
    monkeypatch.setenv("KBATCH_TUNE", path)
    print("[case] cached default", n, launches, flush=True)
    got, cached_launches = _launches(kb, lambda: kb.keccak_batch(1, *dev))
    used, cached = kb.last_tile()
    assert cached and used.as_dict() == kb.Tile().as_dict()
    assert cached_launches == launches
    _, given_launches = _launches(kb, lambda: kb.keccak_batch(1, *dev, tile=kb.Tile()))
    assert given_launches == launches
    assert np.array_equal(got.cpu().numpy(), want.cpu().numpy())
    assert np.array_equal(got.cpu().numpy(), o2.sha3_batch(256, b.data, b.offsets, b.lengths))


@pytest.mark.gpu
def test_autotune_of_a_small_batch_returns_the_default(kb, tmp_path, monkeypatch):
    # one wide launch of about 10 us against four launches of about 70
    b, dev = _batch(300, 200, 141)
    path = str(tmp_path / "tune.json")
    print("[case] autotune 300 x 200 B", flush=True)
    tile, ms, rejected = kb.autotune(1, *dev, reps=5, cache=path)
    print("[case] best", ms, tile.as_dict(), flush=True)
    assert rejected == 0 and tile.as_dict() == kb.Tile().as_dict()
    monkeypatch.setenv("KBATCH_TUNE", path)
    assert _launches(kb, lambda: kb.keccak_batch(1, *dev))[1] == 1
