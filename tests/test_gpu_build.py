"""Connectivity of networks large enough to be built through bins of sources,
bit-exact against the oracle: groups one short of, at and one over the sizes of
the group sort (64, 128, .. 1,024 keys of a wave, 16,384 of a block), sources
far more densely connected than others, and listed connections that crowd onto
one source (a bin overflows and the device atomics build the network)."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2007_14236_amd import workloads as W
from test_gpu_rules import assert_same, canonical

pytestmark = pytest.mark.gpu

SYN = 1 << 20
LIF = dict(tau_m=20.0, C_m=250.0, E_L=0.0, V_th=20.0, V_reset=10.0, t_ref=2.0)


@pytest.fixture(scope="module")
def snn():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2007_14236_amd import snn as S
    S.lib()
    return S


def pop(name, n):
    return dict(name=name, model="lif_delta", n=n, ports=1, params=dict(LIF), V0=None, I_e=0.0)


def check(snn, spec):
    assert W.count_synapses(spec) >= SYN
    g = snn.Net(spec)
    assert_same(canonical(g.synapses()), canonical(O.OracleNet(spec).synapses()))


@pytest.mark.parametrize("length", [2, 63, 64, 65, 128, 129, 255, 257, 512, 513, 1024, 1025, 16384, 16385])
def test_group_lengths(snn, length):
    ns = SYN // length + 1
    pr = dict(src="S", tgt="T", rule="all_to_all", weight=1.0, delay=("const", 0.5, 0.0), port=0,
              weight_dist=dict(kind="uniform", low=0.0, high=1.0, levels=7))
    check(snn, dict(name="len", dt=0.1, seed=3, dmax=8, populations=[pop("S", ns), pop("T", length)], projections=[pr],
                    poisson=[]))


@pytest.mark.parametrize("k", [1, 40, 3000])
def test_uneven_sources(snn, k):
    """k synapses a target from 7 neurons, 250 from 5,000; delays up to 63 steps."""
    d = ("uniform", 0.1, 6.4)
    projs = [dict(src="A", tgt="B", K=k, weight=1.0, delay=d, port=0),
             dict(src="B", tgt="B", K=250, weight=-1.0, delay=d, port=0),
             dict(src="B", tgt="A", rule="fixed_outdegree", K=3, weight=2.0, delay=d, port=0)]
    check(snn, dict(name="uneven", dt=0.1, seed=4, dmax=63, populations=[pop("A", 7), pop("B", 5000)],
                    projections=projs, poisson=[]))


@pytest.mark.parametrize("crowd", [0.0, 0.9])
def test_listed_connections(snn, crowd):
    r = np.random.default_rng(5)
    n, m = 4000, SYN + 77
    src = np.where(r.random(m) < crowd, 17, r.integers(0, n, m))
    pr = dict(rule="list", src_gids=src, tgt_gids=r.integers(0, n, m), delays_ms=r.integers(1, 30, m) * 0.1,
              weights=r.choice([0.5, 1.0, -2.0], m), port=0)
    check(snn, dict(name="list", dt=0.1, seed=4, dmax=40, populations=[pop("A", n)], projections=[pr], poisson=[]))


@pytest.mark.parametrize("length", [255, 256, 4096, 4097, 8192, 8193, 16384, 16385])
@pytest.mark.parametrize("dmax", [1, 40])
def test_row_lengths(snn, length, dmax):
    """Rows of one length, at the edges of what a block sorts at once, beside
    sources of a few synapses."""
    ns = SYN // length + 1
    d = ("uniform", 0.1, 0.1 * dmax) if dmax > 1 else ("const", 0.1, 0.0)
    projs = [dict(src="S", tgt="T", rule="fixed_outdegree", K=length, weight=1.0, delay=d, port=0,
                  weight_dist=dict(kind="uniform", low=0.0, high=1.0, levels=5)),
             dict(src="F", tgt="T", rule="fixed_outdegree", K=2, weight=-1.0, delay=d, port=0)]
    spec = dict(name="rows", dt=0.1, seed=6, dmax=dmax, populations=[pop("F", 3), pop("S", ns), pop("T", 3000)],
                projections=projs, poisson=[])
    check(snn, spec)


@pytest.mark.parametrize("na,ka,nb,kb", [(1295, 146, 927, 270), (508, 198, 2324, 168)])
def test_targets_behind_two_kinds_of_sources(snn, na, ka, nb, kb):
    """6,000 neurons without synapses of their own behind populations whose
    expected out-degrees do not cancel exactly: bins of such neurons alone."""
    projs = [dict(src=s, tgt="T", K=k, weight=1.0, delay=("uniform", 0.1, 6.4), port=0) for s, k in (("A", ka), ("B", kb))]
    check(snn, dict(name="behind", dt=0.1, seed=4, dmax=63, populations=[pop("A", na), pop("B", nb), pop("T", 6000)],
                    projections=projs, poisson=[]))


@pytest.mark.parametrize("k", [7, 9])
def test_few_synapses_a_neuron(snn, k):
    """160,000 sources of 7 synapses (drawn by device atomics) and of 9 (through bins)."""
    pr = dict(src="S", tgt="T", rule="fixed_outdegree", K=k, weight=1.0, delay=("uniform", 0.1, 1.5), port=0)
    check(snn, dict(name="few", dt=0.1, seed=4, dmax=15, populations=[pop("S", 160_000), pop("T", 100)], projections=[pr],
                    poisson=[]))
