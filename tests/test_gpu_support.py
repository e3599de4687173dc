"""Support counting at the edges of its walks: starts of each tier (a wave,
256, 512 and 1,024 threads; cut into parts above 2^18 wedges), hash and dense
tables, windows of ids, rows longer than a workgroup's step, and counts above
8 and 16 bits.  Bit-exact against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2001_06111_amd import binding, synth
from tests import graphs
from tests.gpu_util import oracle_all, upload

pytestmark = pytest.mark.gpu


def _skewed(n_light, n_mid, deg_mid, n_x, name):
    """A start whose wedges all lie in one share of the degrees.  Lower ids:
    x, n_x vertices that share two middles with it, n_light of degree one,
    and n_mid of degree deg_mid that hold most of the degrees."""
    xs = 0
    z = 1 + np.arange(n_x)
    light = 1 + n_x + np.arange(n_light)
    mid = 1 + n_x + n_light + np.arange(n_mid)
    nl = 1 + n_x + n_light + n_mid
    own = n_x + 10  # middles of x alone, so that its priority is the highest
    u, l = [], []

    def add(uu, ll):
        uu, ll = np.broadcast_arrays(uu, ll)
        u.append(uu.ravel())
        l.append(ll.ravel())

    for y in (0, 1):
        add(y, z)
        add(y, xs)
    add(2 + np.arange(own), xs)
    far = 2 + own
    add(far + np.arange(n_light) // 100, light)
    blk = far + (n_light + 99) // 100
    add(blk + np.arange(deg_mid)[:, None], mid[None, :])
    nu = blk + deg_mid
    keys = np.sort(np.concatenate(u).astype(np.int64) * nl + np.concatenate(l))
    return synth._csr_from_keys(nu, nl, keys, name)


CASES = [
    synth.uniform(3, 5, 9, 0),
    synth.complete(2, 2),
    synth.complete(16, 17),       # starts of up to 256 wedges
    synth.complete(16, 129),
    synth.complete(45, 46),       # 2,048
    synth.complete(128, 129),     # 16,384
    synth.complete(500, 530),     # above 2^18: parts
    synth.complete(2, 70001),     # more rows than a 16-bit count holds
    synth.complete(3, 65536),
    synth.complete(255, 300),     # counts of a byte, and above
    synth.complete(256, 300),
    synth.complete(257, 300),
    synth.chung_lu(3000, 200000, 400000, 1.9, 2.2, 20000, 20000, 11),
    synth.chung_lu(90000, 150000, 500000, 2.1, 2.3, 30000, 30000, 12),
    synth.chung_lu(300000, 400, 600000, 2.0, 2.0, 400, 30000, 13),
    graphs.star(5000),
]


@pytest.mark.parametrize("g", CASES, ids=lambda g: g.name)
def test_support(g):
    osup, obf, _ = oracle.support(g.n_upper, g.n_lower, g.row_ptr, g.col)
    sup, bf = binding.bt_support(upload(g))
    assert np.array_equal(sup.cpu().numpy(), osup) and bf == obf


@pytest.mark.parametrize("shape", [(200000, 400, 1000, 2500), (1000000, 400, 3000, 6000),
                                   (40000, 100, 500, 1000)])
def test_wedges_in_one_share_of_the_degrees(shape):
    test_support(_skewed(*shape, "skewed"))


@pytest.mark.parametrize("m", [1, 1023, 1024, 1025, 65536, 65537, 262143, 262145])
def test_sizes_of_the_sorts(m):
    f = max(1, m // 10)
    test_support(synth.chung_lu(max(3, f // 2), max(3, f), m, 2.1, 2.4, f, f, m)
                 if m > 1 else synth.uniform(3, 4, 1, 0))


@pytest.mark.parametrize("where", [0, 1, 4999, 9997, 9998])
def test_order_inside_and_between_rows(where):
    """Lower ids may start over at a row's beginning only, empty rows or not."""
    row_ptr = np.array([0, 0, 5000, 5000, 5000, 10000, 10000])
    col = np.concatenate([np.arange(5000), np.arange(5000)]).astype(np.int32)
    g = synth.Graph(6, 5000, row_ptr, col, "two rows")
    test_support(g)
    bad = col.copy()
    bad[where + 1 if where != 4999 else 5001] = bad[where if where != 4999 else 5000]
    with pytest.raises(binding.BtError) as ei:
        binding.bt_support(upload(synth.Graph(6, 5000, row_ptr, bad, "bad")))
    assert ei.value.status == binding.BT_EINVAL
    for r in (row_ptr + 1, row_ptr[::-1].copy(), np.array([0, 0, 5000, 4000, 5000, 10000, 9999])):
        with pytest.raises(binding.BtError) as ei:
            binding.bt_support(upload(synth.Graph(6, 5000, r, col, "bad rows")))
        assert ei.value.status == binding.BT_EINVAL


@pytest.mark.parametrize("shape", [(200000, 100, 500, 2500), (60000, 60, 300, 1500)])
def test_index_of_wedges_in_one_share_of_the_degrees(shape):
    """The index's sweep over shares of the degrees: one share holds more
    wedges than its hash table, the others next to none."""
    g = _skewed(*shape, "skewed")
    osup, obf, _ = oracle.support(g.n_upper, g.n_lower, g.row_ptr, g.col)
    ophi, _ = oracle.bitruss(g.n_upper, g.n_lower, g.row_ptr, g.col, sup=osup)
    sup, phi, st = binding.bt_decompose(upload(g), stats=True)
    assert np.array_equal(sup.cpu().numpy(), osup) and st["butterflies"] == obf
    assert np.array_equal(phi.cpu().numpy(), ophi)


@pytest.mark.parametrize("nu,nl", [(1, 1), (1, 2), (2, 1022), (500, 524), (500, 525), (1, 8191),
                                   (8191, 1), (4096, 4096), (3000, 5192), (3000, 5193), (1, 8192)])
def test_orders_by_one_workgroup(nu, nl):
    """Vertex counts around a wave's rows, one block's and the most that one
    workgroup ranks (8,192); degrees up to the whole other layer."""
    m = min(nu * nl, max(nl, 6 * (nu + nl)))
    g = synth.complete(nu, nl) if m == nu * nl else synth.uniform(nu, nl, m, nu + nl)
    osup, obf, ophi = oracle_all(g)
    got, phi, st = binding.bt_decompose(upload(g), stats=True)
    assert np.array_equal(got.cpu().numpy(), osup) and np.array_equal(phi.cpu().numpy(), ophi)
    assert st["butterflies"] == obf
    assert np.array_equal(binding.bt_support(upload(g))[0].cpu().numpy(), osup)


def test_side_streams_go_with_the_workspace():
    """Walks of several tiers and leaves of several sizes, whose launches run
    beside each other, before and after the workspace is given back."""
    g = synth.chung_lu(9000, 15000, 100000, 2.1, 2.3, 9000, 9000, 12)
    osup, obf, ophi = oracle_all(g)
    d = upload(g)
    for _ in range(3):
        sup, bf = binding.bt_support(d)
        assert np.array_equal(sup.cpu().numpy(), osup) and bf == obf
        assert np.array_equal(binding.bt_decompose(d)[1].cpu().numpy(), ophi)
        binding.bt_release_workspace()


@pytest.mark.parametrize("a,b", [(760, 790), (1100, 500)])
def test_starts_cut_into_parts(a, b):
    """Starts of more than 2^19 wedges, which several workgroups share (closed
    form: an edge of K(a, b) lies in (a - 1)(b - 1) butterflies)."""
    sup, bf = binding.bt_support(upload(synth.complete(a, b)))
    assert bool((sup == (a - 1) * (b - 1)).all()) and bf == a * (a - 1) // 2 * (b * (b - 1) // 2)
