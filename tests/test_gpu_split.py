"""The peel that splits graphs of 2^14 edges and more into ranges of bitruss
numbers, at its edges: graphs around the sizes that one workgroup takes
(2^14 edges whole, 28,672 as a part), dense cores that no level splits,
unions whose graphs differ in size and in depth, the level-by-level form and
the two-kernel rounds.  Bit-exact against the oracle."""
import numpy as np
import pytest
import torch

from paper_2001_06111_amd import binding, synth
from tests import graphs
from tests.gpu_util import oracle_all, upload

pytestmark = pytest.mark.gpu
MODES = [None, "plain", "graph"]


def _cl(m, seed=0):
    return synth.chung_lu(max(20, m // 20), max(30, m // 12), m, 2.2, 2.2, m / 4, m / 4, m + seed)


def _set(monkeypatch, mode):
    if mode:
        monkeypatch.setenv("BT_PEEL_MODE", mode)


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("m", [1, 65, 16384, 28671, 28672, 28673, 60000, 150001])
def test_sizes(m, mode, monkeypatch):
    g = _cl(m) if m > 65 else synth.uniform(20, 30, m, m)
    osup, obf, ophi = oracle_all(g)
    _set(monkeypatch, mode)
    sup, phi, st = binding.bt_decompose(upload(g), stats=True)
    assert np.array_equal(sup.cpu().numpy(), osup) and np.array_equal(phi.cpu().numpy(), ophi)
    assert st["butterflies"] == obf and st["max_phi"] == int(ophi.max())
    assert st["levels"] == np.unique(ophi).size


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("g", [synth.complete(160, 180), synth.complete(2, 20000),
                               synth.complete(128, 129),
                               graphs.random_dense(220, 210, 0.8, 5),
                               graphs.random_dense(3000, 12, 0.9, 6),
                               graphs.disjoint_union(_cl(30000), synth.complete(170, 170))],
                         ids=lambda g: g.name)
def test_dense(g, mode, monkeypatch):
    osup, _, ophi = oracle_all(g)
    _set(monkeypatch, mode)
    for variant in (binding.BT_PEEL_BATCH_BLOOM, binding.BT_PEEL_BATCH_EDGE):
        sup, phi, _ = binding.bt_decompose_variant(upload(g), variant)
        assert np.array_equal(sup.cpu().numpy(), osup) and np.array_equal(phi.cpu().numpy(), ophi)
    _, phi, _ = binding.bt_decompose_pc(upload(g), tau=0.3)
    assert np.array_equal(phi.cpu().numpy(), ophi)


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("union", ["0", "1"])
def test_union_of_mixed_sizes(mode, union, monkeypatch):
    gs = [_cl(m, i) for i, m in enumerate((90000, 16384, 28672, 28673, 17000, 50000))]
    gs += [graphs.random_dense(220, 210, 0.8, 5), graphs.star(20000), synth.complete(3, 9000)]
    if mode:  # the sweeps then take small graphs as well
        gs += [synth.from_edges(3, 3, []), synth.uniform(20, 30, 64, 1), _cl(300)]
    _set(monkeypatch, mode)
    if union == "1":
        monkeypatch.setenv("BT_BATCH_PEEL", "union")
    sups, phis, _ = binding.bt_decompose_batch([upload(g) for g in gs])
    for g, s, p in zip(gs, sups, phis):
        osup, _, ophi = oracle_all(g)
        assert np.array_equal(s.cpu().numpy(), osup) and np.array_equal(p.cpu().numpy(), ophi)


@pytest.mark.parametrize("unit", [False, True])
def test_leaves_beside_deeper_sweeps(unit):
    """Graphs of two sweeps and more, whose first leaves start beside the second."""
    for g in (synth.scaled_chunglu(500000, seed=31),
              synth.chung_lu(2000, 40000, 300000, 1.8, 2.3, 3000, 3000, 3)):
        _, _, ophi = oracle_all(g)
        variant = binding.BT_PEEL_BATCH_EDGE if unit else binding.BT_PEEL_BATCH_BLOOM
        for _ in range(2):
            _, phi, _ = binding.bt_decompose_variant(upload(g), variant, want_sup=False)
            assert np.array_equal(phi.cpu().numpy(), ophi)


@pytest.mark.parametrize("m", [20000, 60000, 150001])
def test_launches_that_end_in_their_first_round(m, monkeypatch):
    """Every launch of a sweep yields after 16 rounds, so many launches begin
    with little left to do, the last ones with a job's last decision."""
    g = _cl(m)
    _, phi0, _ = binding.bt_decompose(upload(g), want_sup=False)
    monkeypatch.setenv("BT_PEEL_YIELD", "1")
    for tau in (0.1, 0.3):
        _, phi, st = binding.bt_decompose_pc(upload(g), tau=tau, want_sup=False, stats=True)
        assert st["peel_yields"] >= 1
        assert np.array_equal(phi.cpu().numpy(), phi0.cpu().numpy())


@pytest.mark.parametrize("mode", ["plain", "graph"])
def test_listed_gathers(mode, monkeypatch):
    """Ranges long enough that level-by-level gathers list what remains."""
    gs = [_cl(140000, 1), _cl(200000, 2), _cl(3000, 3)]
    want = [oracle_all(g)[2] for g in gs]
    monkeypatch.setenv("BT_PEEL_MODE", mode)
    phis = binding.bt_decompose_batch([upload(g) for g in gs])[1]
    for w, phi in zip(want, phis):
        assert np.array_equal(phi.cpu().numpy(), w)


@pytest.mark.parametrize("mode", [None, "split", "graph"])
@pytest.mark.parametrize("m", [16400, 117248, 300000])
def test_few_levels(m, mode, monkeypatch):
    """Uniform graphs, whose few levels are peeled one by one (or split)."""
    f = (m / 10000) ** 0.5
    g = synth.uniform(round(1000 * f), round(1500 * f), m, m)
    osup, _, ophi = oracle_all(g)
    _set(monkeypatch, mode)
    sup, phi, st = binding.bt_decompose(upload(g), stats=True)
    assert np.array_equal(sup.cpu().numpy(), osup) and np.array_equal(phi.cpu().numpy(), ophi)
    assert st["max_phi"] == int(ophi.max()) and st["levels"] == np.unique(ophi).size
    _, phi, _ = binding.bt_decompose_pc(upload(g), 0.05)
    assert np.array_equal(phi.cpu().numpy(), ophi)


@pytest.mark.parametrize("log2", ["0", "6", "11", "15"])
@pytest.mark.parametrize("g", [_cl(30000), _cl(60000), synth.complete(170, 180),
                               graphs.random_dense(220, 210, 0.8, 5),
                               graphs.disjoint_union(_cl(20000), synth.complete(130, 140))],
                         ids=lambda g: g.name)
def test_leaves_of_bounded_wedges(g, log2, monkeypatch):
    """Parts of more wedges than a leaf may hold go on to the next sweep,
    whatever their edges and depth, down to parts of one level."""
    ophi = oracle_all(g)[2]
    monkeypatch.setenv("BT_LEAF_WEDGES_LOG2", log2)
    monkeypatch.setenv("BT_PEEL_MODE", "split")
    phi = binding.bt_decompose(upload(g))[1]
    assert np.array_equal(phi.cpu().numpy(), ophi)
    phi = binding.bt_decompose_pc(upload(g), tau=0.3)[1]
    assert np.array_equal(phi.cpu().numpy(), ophi)


def test_few_edges_of_many_wedges(monkeypatch):
    """2,500 hubs on 20 common lower vertices (and 5,000 of their own each)
    and 2,800 upper vertices on ten of them: 28,000 edges, fewer than a leaf
    takes, that hold 7.0e7 wedges and stay together at the next depth."""
    hubs, own, common, small, ten = 2500, 5000, 20, 2800, 10
    lower = np.concatenate([np.broadcast_to(np.arange(common), (hubs, common)),
                            common + own * np.arange(hubs)[:, None] + np.arange(own)], axis=1)
    some = np.sort(np.argsort(np.random.default_rng(7).random((small, 12)), axis=1)[:, :ten], axis=1)
    row_ptr = np.concatenate([np.arange(hubs + 1) * (common + own),
                              hubs * (common + own) + ten * np.arange(1, small + 1)])
    g = synth.Graph(hubs + small, common + own * hubs, row_ptr.astype(np.int64),
                    np.concatenate([lower.ravel(), some.ravel()]).astype(np.int32), "hubs")
    d = upload(g)
    sup, phi, st = binding.bt_decompose(d, stats=True)
    monkeypatch.setenv("BT_PEEL_MODE", "plain")
    sup0, phi0, st0 = binding.bt_decompose(d, stats=True)
    assert torch.equal(phi, phi0) and torch.equal(sup, sup0)
    for k in ("butterflies", "max_phi", "levels", "bloom_wedges"):
        assert st[k] == st0[k], k


@pytest.mark.parametrize("unit", [False, True])
@pytest.mark.parametrize("mode", ["plain", "graph"])
def test_thresholds_of_long_ranges(mode, unit, monkeypatch):
    """Ranges of 2^18 edges and more, whose level-by-level gathers scan a list of
    the edges below a threshold: alone, beside others, and resumed after
    yields; with batch bloom processing and without."""
    g = synth.chung_lu(6000, 40000, 300001, 2.0, 2.3, 4000, 4000, 7)
    ophi = oracle_all(g)[2]
    d = upload(g)
    monkeypatch.setenv("BT_PEEL_MODE", mode)
    variant = binding.BT_PEEL_BATCH_EDGE if unit else binding.BT_PEEL_BATCH_BLOOM
    _, phi, st = binding.bt_decompose_variant(d, variant, stats=True)
    assert np.array_equal(phi.cpu().numpy(), ophi)
    assert mode == "graph" or st["levels"] == np.unique(ophi).size
    if mode == "plain":
        monkeypatch.setenv("BT_PEEL_YIELD", "1")
        _, phi, st1 = binding.bt_decompose_variant(d, variant, stats=True)
        assert st1["peel_yields"] >= 1 and st1["rounds"] == st["rounds"]
        assert np.array_equal(phi.cpu().numpy(), ophi)
        monkeypatch.delenv("BT_PEEL_YIELD")
    if not unit:
        h = _cl(280000, 5)
        phis = binding.bt_decompose_batch([d, upload(h), upload(_cl(20000))])[1]
        assert np.array_equal(phis[0].cpu().numpy(), ophi)
        assert np.array_equal(phis[1].cpu().numpy(), oracle_all(h)[2])
