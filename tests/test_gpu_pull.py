"""GPU parity of pulled delivery (LIF networks whose connection groups put
many synapses on each target tile): a tile's block counts the runs of its
instance's spikes instead of reading a bin.  Sizes where it can go wrong: one
slice, several, and several tiles; a tile in several parts; runs of a few
synapses and of thousands; one delay and many; two ports and four weight
classes; multiplicities above one; rasters and pending inputs bit-exact against
the oracle.  Snapshots pass between a pulling network and one that delivers the
same through bins."""
import sys

import numpy as np
import pytest

from oracle import oracle as O
from paper_2007_14236_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _name(request):
    print(f"\n[gpu-case] {request.node.nodeid}", flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def snn():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2007_14236_amd import snn as S
    S.lib()
    return S


def brunel(n, k, seed, delay, dmax=25):
    return W.brunel_lif(n=n, k=k, seed=seed, delay=delay, dmax=dmax, nu_ext=260.0)


def two_ports(seed=5):
    lif = dict(tau_m=10.0, C_m=250.0, E_L=-65.0, V_th=-50.0, V_reset=-65.0, t_ref=1.0, tau_syn=[0.5, 2.0])
    pops = [dict(name=q, model="lif_exp", n=n, ports=2, params=dict(lif), V0=W.initial_v(seed, n, -65.0, -50.0), I_e=420.0)
            for q, n in (("A", 900), ("B", 357))]
    projs = [dict(src=s, tgt=t, K=k, weight=w, delay=("uniform", 0.1, 0.6), port=p)
             for s, w, p, k in (("A", 20.0, 0, 120), ("B", -45.0, 1, 60), ("A", 9.0, 1, 50), ("B", -11.0, 0, 40))
             for t in ("A", "B")]
    return dict(name="two_ports", dt=0.1, seed=seed, dmax=8, populations=pops, projections=projs, poisson=[])


def multiplicity(seed=6):
    times = [[0.5, 0.5, 0.5, 2.0, 7.1], [1.0, 3.0, 3.0], [4.0] * 31]
    lif = dict(tau_m=20.0, C_m=250.0, E_L=0.0, V_th=20.0, V_reset=10.0, t_ref=2.0)
    pops = [dict(name="G", model="spike_generator", n=3, ports=1, params={}, spike_times=times),
            dict(name="R", model="parrot_neuron", n=3, ports=1, params={}),
            dict(name="L", model="lif_delta", n=1200, ports=1, params=lif, V0=np.linspace(0.0, 19.5, 1200), I_e=250.0)]
    projs = [dict(src="G", tgt="R", rule="one_to_one", weight=1.0, delay=("const", 0.3, 0.0), port=0),
             dict(src="R", tgt="L", rule="fixed_indegree", K=9, weight=0.05, delay=("uniform", 0.1, 1.5), port=0),
             dict(src="L", tgt="L", rule="fixed_indegree", K=40, weight=-0.2, delay=("const", 1.0, 0.0), port=0)]
    return dict(name="mult", dt=0.1, seed=seed, dmax=20, populations=pops, projections=projs, poisson=[])


NETS = {
    # ten instances of 300 to 1,533 neurons
    "shared_tiles": (lambda: [brunel(300 + 137 * i, 90 + 30 * i, 40 + i, ("uniform", 0.1, 0.5)) for i in range(10)], 256),
    "one_net_one_delay": (lambda: [brunel(2500, 300, 21, ("const", 0.8, 0.0))], 256),
    "long_runs": (lambda: [brunel(1025, 1025, 3, ("const", 0.1, 0.0), 1), brunel(513, 500, 4, ("const", 0.1, 0.0), 1)], 512),
    "many_delays": (lambda: [brunel(1500, 1500, 8, ("uniform", 0.1, 6.4), 63)], 512),
    "slices": (lambda: [brunel(9001, 200, 9, ("uniform", 0.1, 0.4)), brunel(4097, 150, 10, ("const", 0.2, 0.0))], 0),
    "tiles": (lambda: [brunel(16385, 250, 11, ("const", 0.3, 0.0)), brunel(700, 90, 12, ("const", 0.1, 0.0))], 0),
    "parts": (lambda: [W.brunel_lif(n=4100, k=4000, g=3.0, seed=13, delay=("uniform", 0.1, 0.8), dmax=9, nu_ext=300.0)], 0),
    "library_tile": (lambda: [brunel(600 + i, 60, 60 + i, ("uniform", 0.1, 0.4)) for i in range(3)], 0),
    "two_ports": (lambda: [two_ports()], 256),
    "multiplicity": (lambda: [multiplicity(), multiplicity(7)], 256),
}


@pytest.mark.parametrize("name", sorted(NETS))
def test_pulled_delivery_bit_exact(snn, name):
    make, tile = NETS[name]
    specs, steps, probe = make(), 150, (0, 40, 111)
    g = snn.Net(specs, delivery="binned", tile_neurons=tile)
    c = g.counters()
    assert c["tile_runs"] == 1 and c["tile_window"] == 1
    recs, events, pairs = [], 0, 0
    for sp in specs:
        o = O.OracleNet(sp, O.FP32SO)
        rec = o.record_input(steps + 1)
        o.simulate(steps + 1)
        recs.append((o.spikes(), rec))
    done = 0
    for n in probe:  # the input of step n + 1 after n + 1 steps, read twice
        g.simulate(n + 1 - done)
        done = n + 1
        for port in range(recs[0][1].shape[2]):
            inp = g.get_input(port)
            assert np.array_equal(inp, g.get_input_noalloc(port))
            for inst, (_, rec) in zip(g.instances, recs):
                assert np.array_equal(inp[inst["first"]:inst["first"] + inst["n"]], rec[n + 1][:, port]), (n, port)
    g.simulate(steps - done)
    gs, gg, gm = g.spikes()
    for inst, ((os_, og, om), _) in zip(g.instances, recs):
        sel = (gg >= inst["first"]) & (gg < inst["first"] + inst["n"])
        keep = os_ < steps
        assert np.array_equal(gs[sel], os_[keep]) and np.array_equal(gg[sel] - inst["first"], og[keep])
        assert np.array_equal(gm[sel], om[keep])
    assert len(gs) > 50
    a, d = g.counters(), snn.Net(specs, delivery="direct")
    d.simulate(steps)
    for k in ("spikes", "events", "pairs", "overflow"):
        assert a[k] == d.counters()[k], k


@pytest.mark.parametrize("src,dst", [(0, 0), (0, 1 << 20), (1 << 20, 0)])
def test_snapshots_between_pull_and_bins(snn, src, dst):
    """A bin capacity that was asked for keeps the bins.  Tiles of at most
    2^14 synapses (256 neurons, in-degree 60) have bins of their in-degree at
    the library's capacity and at a large one, so both networks hold the same
    arrays."""
    specs = [brunel(300 + 137 * i, 60, 40 + i, ("uniform", 0.1, 0.3)) for i in range(4)]
    a = snn.Net(specs, delivery="binned", tile_neurons=256, bin_capacity=src)
    b = snn.Net(specs, delivery="binned", tile_neurons=256, bin_capacity=dst)
    a.simulate(87)
    b.simulate(6)
    b.restore(a.snapshot())
    for x in (a, b):
        x.simulate(101)
    assert np.array_equal(a.get_input(0), b.get_input(0))
    for x, y in zip(a.spikes(87, 188), b.spikes(87, 188)):
        assert np.array_equal(x, y) and len(x) > 0
    assert np.array_equal(a.get_state("V_m"), b.get_state("V_m"))
    ca, cb = a.counters(), b.counters()
    assert all(ca[k] == cb[k] for k in ("steps", "spikes", "events", "pairs", "spill_events"))
