"""Requests of the larger classes that come together share a batch; one that
comes alone, or while others keep coming, still runs."""
import time

import numpy as np
import pytest
import torch

from paper_2001_06111_amd import binding, synth
from tests.gpu_util import oracle_all, upload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,gap", [(1, 0.0), (6, 0.0), (12, 0.0004)])
def test_medium_requests(n, gap):
    gs = [synth.scaled_chunglu(17000 + 500 * i, seed=50 + i) for i in range(n)]
    ds = [upload(g) for g in gs]
    torch.cuda.synchronize()
    eng = binding.BtEngine(slots=2)
    for i, d in enumerate(ds):
        eng.bt_engine_submit(d, i)
        time.sleep(gap)
    eng.bt_engine_drain()
    done = eng.bt_engine_poll()
    st = eng.bt_engine_stats()
    eng.bt_engine_destroy()
    assert sorted(r for r, _ in done) == list(range(n)) and all(s == binding.BT_OK for _, s in done)
    assert 1 <= st["batches"] <= n and st["admitted"] == n
    for i, g in enumerate(gs):
        assert np.array_equal(eng.results[i][2].cpu().numpy(), oracle_all(g)[2])
