"""Which kind a batch call's launches are timed as.  Needs an MI355X; run with
-m gpu."""

import numpy as np
import pytest

from paper_1902_05320_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 300, 2048, 2049, 4096, 4097])
def test_arrival_order_pass_is_timed_as_the_first_pass(n):
    # whatever form hashes it; the explicit wide mode has a kind of its own
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1902_05320_amd import kbatch as kb
    b = wl.uneven(n, 300, seed=150)
    data = torch.from_numpy(b.data).cuda() if b.data.size else torch.zeros(1, dtype=torch.uint8, device="cuda")
    offs, lens = torch.from_numpy(b.offsets.astype(np.int64)).cuda(), torch.from_numpy(b.lengths.astype(np.int64)).cuda()
    print("[case] timing kinds", n, flush=True)
    for mode, kind in (("persistent", "first_pass"), ("wide", "wide")):
        kb.timing_enable(True, kinds=["first_pass", "wide"])
        kb.keccak_batch(1, data, offs, lens, mode=mode)
        torch.cuda.synchronize()
        ms, launches = kb.timing_read(kind)
        total = kb.timing_read()[1]
        kb.timing_enable(False)
        assert launches == total == 1 and ms > 0.0, (mode, launches, total)
