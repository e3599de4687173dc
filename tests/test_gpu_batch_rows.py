"""Batches whose rows list their ids in any order: every batch takes them,
whatever its graphs' sizes, with results in the caller's edge order, and
refuses an id that a row holds twice."""
import numpy as np
import pytest

from paper_2001_06111_amd import binding, synth
from tests.gpu_util import oracle_all, upload

pytestmark = pytest.mark.gpu


def _any_order(g, seed):
    """g with each row's ids shuffled, and where each of its edges went."""
    rng = np.random.default_rng(seed)
    at = np.concatenate([lo + rng.permutation(hi - lo)
                         for lo, hi in zip(g.row_ptr[:-1], g.row_ptr[1:])]).astype(np.int64)
    return synth.Graph(g.n_upper, g.n_lower, g.row_ptr, g.col[at], g.name), at


@pytest.mark.parametrize("sizes", [(3000,), (3000, 9000), (3500, 16383, 4000), (3000, 20000)])
def test_rows_in_any_order(sizes):
    gs = [synth.scaled_chunglu(m, seed=m) for m in sizes]
    want = [oracle_all(g) for g in gs]
    mixed = [_any_order(g, i) for i, g in enumerate(gs)]
    sups, phis, _ = binding.bt_decompose_batch([upload(g) for g, _ in mixed])
    for (osup, _, ophi), (_, at), s, p in zip(want, mixed, sups, phis):
        assert np.array_equal(s.cpu().numpy(), osup[at]) and np.array_equal(p.cpu().numpy(), ophi[at])
    twice = mixed[0][0]
    i = int(np.flatnonzero(np.diff(twice.row_ptr) > 1)[0])
    twice.col[twice.row_ptr[i] + 1] = twice.col[twice.row_ptr[i]]
    with pytest.raises(binding.BtError) as ei:
        binding.bt_decompose_batch([upload(twice)] + [upload(g) for g, _ in mixed[1:]])
    assert ei.value.status == binding.BT_EINVAL
