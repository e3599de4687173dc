"""The serving engine's memory budget where it is tight: no slot's workspace
holds more than the budget, whichever way its batch ends."""
import numpy as np
import pytest
import torch

from paper_2001_06111_amd import binding, synth
from tests.gpu_util import oracle_all, upload

pytestmark = pytest.mark.gpu


def estimate(g):
    """What bt_engine_submit reserves: the wedge bound of Lemma 6 (68 bytes
    each), 250 bytes an edge, 40 a vertex and 1 MiB."""
    u, v = g.edges()
    du, dv = np.bincount(u, minlength=g.n_upper), np.bincount(v, minlength=g.n_lower)
    return 68 * int(np.minimum(du[u], dv[v]).sum()) + 250 * g.m + 40 * (g.n_upper + g.n_lower) + (1 << 20)


def test_batch_with_a_request_that_fails():
    """A request whose graph turns malformed after it was submitted fails its
    batch; the others are run again one by one within the same budget."""
    bad, good = synth.uniform(1200, 1800, 16500, 1), synth.scaled_chunglu(150_000, seed=41)
    budget = estimate(bad) + estimate(good)
    eng = binding.BtEngine(hbm_budget=budget, slots=-1)
    try:
        ds = [upload(bad), upload(good)]
        for i, d in enumerate(ds):
            eng.bt_engine_submit(d, i)
        ds[0].col.fill_(-1)
        torch.cuda.synchronize()
        assert eng.bt_engine_step() == 2
        done, mem = dict(eng.bt_engine_poll()), eng.bt_engine_memory()
    finally:
        eng.bt_engine_destroy()
    assert done == {0: binding.BT_EINVAL, 1: binding.BT_OK}
    assert np.array_equal(eng.results[1][2].cpu().numpy(), oracle_all(good)[2])
    assert mem["peak_held"] <= budget and mem["peak_committed"] <= budget, mem


@pytest.mark.parametrize("g", [synth.uniform(1200, 1800, 16500, 1), synth.scaled_chunglu(17000, seed=1),
                               synth.uniform(5000, 7000, 117248, 2), synth.complete(150, 150),
                               synth.scaled_chunglu(60000, seed=1)], ids=lambda g: g.name)
def test_budget_of_one_request(g):
    """A budget of just the estimate admits the request and holds it."""
    budget = estimate(g)
    eng = binding.BtEngine(hbm_budget=budget, slots=-1)
    try:
        d = upload(g)
        eng.bt_engine_submit(d, 0)
        assert eng.bt_engine_step() == 1
        done, mem = dict(eng.bt_engine_poll()), eng.bt_engine_memory()
    finally:
        eng.bt_engine_destroy()
    assert done == {0: binding.BT_OK}
    assert np.array_equal(eng.results[0][2].cpu().numpy(), oracle_all(g)[2])
    assert mem["peak_held"] <= budget and mem["peak_committed"] <= budget, mem
