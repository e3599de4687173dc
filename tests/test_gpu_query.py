"""GPU parity of the k-bitruss components (bt_bitruss_components) against the
oracle's breadth-first search: labels must match exactly (components are
numbered by smallest edge id, so the labelling is unique)."""
import numpy as np
import pytest
import torch

from oracle.query import bitruss_components
from paper_2001_06111_amd import binding, synth
from tests import graphs
from tests.gpu_util import upload

pytestmark = pytest.mark.gpu


def _check(g, ks):
    dg = upload(g)
    _, phi, _ = binding.bt_decompose(dg)
    ph = phi.cpu().numpy()
    for k in ks:
        comp, c = binding.bt_bitruss_components(dg, phi, k)
        torch.cuda.synchronize()
        ocomp, oc = bitruss_components(g.n_upper, g.n_lower, g.row_ptr, g.col, ph, k)
        assert c == oc, f"{g.name} k={k}"
        assert np.array_equal(comp.cpu().numpy(), ocomp), f"{g.name} k={k}"


def test_components_small_graphs():
    for grey in (True, False):
        g, _, _ = graphs.worked_example(grey)
        _check(g, [0, 1, 2, 3])
    for g in [graphs.k2_1001(), synth.complete(5, 6), graphs.star(30), graphs.cycle(6),
              graphs.disjoint_union(graphs.disjoint_union(synth.complete(3, 3), synth.complete(2, 4)),
                                    graphs.star(5))]:
        _check(g, [-1, 0, 1, 3, 4, 100])


@pytest.mark.parametrize("seed", range(3))
def test_components_random(seed):
    rng = np.random.default_rng(700 + seed)
    g = graphs.random_dense(int(rng.integers(20, 60)), int(rng.integers(20, 60)), 0.1, seed)
    _check(g, [0, 1, 2, 5])


def test_components_chunglu():
    g = synth.scaled_chunglu(20_000, seed=5)
    _, phi, _ = binding.bt_decompose(upload(g))
    ph = phi.cpu().numpy()
    ks = sorted({0, 1, int(np.median(ph)), int(np.percentile(ph, 90)), int(ph.max())})
    _check(g, ks)


def test_components_empty_and_invalid():
    g = synth.from_edges(3, 4, [])
    dg = upload(g)
    comp, c = binding.bt_bitruss_components(dg, torch.empty(0, dtype=torch.int64, device="cuda"), 1)
    assert c == 0 and comp.numel() == 0
    bad = synth.uniform(10, 10, 30, 1)
    col = bad.col.copy()
    col[2] = 99
    d = binding.DeviceGraph(bad.n_upper, bad.n_lower, torch.from_numpy(bad.row_ptr).cuda(),
                            torch.from_numpy(col).cuda())
    with pytest.raises(binding.BtError) as ei:
        binding.bt_bitruss_components(d, torch.zeros(bad.m, dtype=torch.int64, device="cuda"), 1)
    assert ei.value.status == binding.BT_EINVAL


@pytest.mark.parametrize("seed", range(4))
def test_components_rows_of_wave_lengths(seed):
    """Rows of 0 to 200 edges with arbitrary numbers, so that a row's first
    edge of the k-bitruss lies in any of its 64-edge pieces or in none."""
    rng = np.random.default_rng(900 + seed)
    lens = [0, 1, 63, 64, 65, 127, 128, 129, 200, 0, 3]
    edges = [(i, int(j)) for i, n in enumerate(lens) for j in rng.choice(220, n, replace=False)]
    g = synth.from_edges(len(lens), 220, edges)
    ph = np.where(rng.random(g.m) < (0.5, 0.05, 0.01, 0.9)[seed], rng.integers(0, 9, g.m), 0)
    dg = upload(g)
    phi = torch.from_numpy(ph.astype(np.int64)).cuda()
    for k in (-1, 0, 1, 4, 9):
        comp, c = binding.bt_bitruss_components(dg, phi, k)
        ocomp, oc = bitruss_components(g.n_upper, g.n_lower, g.row_ptr, g.col, ph, k)
        assert c == oc and np.array_equal(comp.cpu().numpy(), ocomp), k
