"""GPU parity of nearest-neighbour STDP (Sec. 2.1, after Morrison et al.
2008), through the C ABI, against the oracle (whose rule is pinned by closed
forms and a plain-Python replay in test_oracle_stdp.py):

- single pre/post pairs of spike generators at known time differences, both
  orders, same and adjacent steps, bounds and multiplicity, additive and
  multiplicative: the final fixed-point weight equals the oracle's;
- recurrent LIF networks with plastic projections beside static ones
  (all-to-all and fixed in-degree, delta and exponential PSCs): rasters,
  potentials, per-step inputs and every synaptic weight bit-exact, in both
  delivery modes and as members of a batch;
- a snapshot taken mid-run continues with the same weights.
"""
import sys

import numpy as np
import pytest

from oracle import oracle as O
from paper_2007_14236_amd import workloads as W
from test_oracle_stdp import pair_spec

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


PAIRS = [
    ([1.0], [3.0], {}), ([3.0], [1.0], {}), ([1.0], [3.0], dict(mu_plus=1)), ([3.0], [1.0], dict(mu_minus=1)),
    ([1.0, 1.5], [3.0], {}), ([3.0], [1.0, 1.5], {}), ([1.0], [2.0, 3.0], dict(mu_plus=1)),
    ([1.0], [1.4], {}), ([1.0], [1.3], {}), ([1.0], [1.3], dict(lambda_=1.0, alpha=1.0)),
    ([1.0], [1.2], dict(lambda_=1.0, alpha=1.0)), ([2.0, 2.0, 2.0], [1.0], dict(mu_minus=1)),
    ([0.5, 1.7, 2.9, 4.0], [1.0, 1.8, 4.0, 6.5], dict(mu_plus=1, mu_minus=1)),
]


@pytest.mark.parametrize("delivery", ["direct", "binned"])
def test_single_pairs_equal_the_oracle(snn, delivery):
    for pre, post, kw in PAIRS:
        spec, _ = pair_spec(pre, post, **kw)
        o = O.OracleNet(spec)
        o.simulate(120)
        g = snn.Net(spec, delivery=delivery)
        try:
            g.simulate(120)
            w_gpu, w_orc = g.weights(), o.synapses()["wq"]
            assert np.array_equal(w_gpu, w_orc), (pre, post, kw, w_gpu, w_orc)
        finally:
            g.close()


def plastic_brunel(seed=21, n=10, k=4, nu=1000.0):
    spec = W.brunel_lif(n=n, k=k, nu_ext=nu, seed=seed, delay=("uniform", 0.1, 0.45), dmax=8)
    spec["projections"].append(dict(src="E", tgt="E", rule="all_to_all", weight=0.4, port=0,
                                    delay=("uniform", 0.1, 0.45),
                                    stdp=dict(tau_plus=5.0, tau_minus=7.0, alpha=1.1, mu_plus=1, mu_minus=0,
                                              w_max=2.0, **{"lambda": 0.2})))
    return spec


def plastic_mc(seed=3):
    """Small microcircuit stand-in (exponential PSCs) whose L2/3E -> L2/3E and
    L4E -> L2/3E projections are plastic (additive and multiplicative)."""
    spec = W.microcircuit(scale=0.05, k_scale=0.25, k_ext=3500, seed=seed)
    for pr in spec["projections"]:
        if pr["tgt"] == "L23E" and pr["src"] == "L23E":
            pr["stdp"] = dict(tau_plus=15.0, tau_minus=30.0, alpha=0.9, mu_plus=1, mu_minus=1, w_max=200.0,
                              **{"lambda": 0.05})
        if pr["tgt"] == "L23E" and pr["src"] == "L4E":
            pr["stdp"] = dict(tau_plus=20.0, tau_minus=20.0, alpha=1.0, mu_plus=0, mu_minus=0, w_max=300.0,
                              **{"lambda": 0.02})
    return spec


def plastic_brunel_big(seed=8):
    spec = W.brunel_lif(n=800, k=80, nu_ext=300.0, seed=seed, delay=("uniform", 0.1, 2.0), dmax=25)
    for pr in spec["projections"]:
        if pr["src"] == "E":
            pr["stdp"] = dict(tau_plus=16.8, tau_minus=33.7, alpha=1.0, mu_plus=1, mu_minus=1, w_max=0.3,
                              **{"lambda": 0.03})
    return spec


NETS = {"brunel10": plastic_brunel, "brunel800": plastic_brunel_big, "mc": plastic_mc}


@pytest.mark.parametrize("name", sorted(NETS))
@pytest.mark.parametrize("delivery", ["direct", "binned"])
def test_plastic_networks_bit_exact(snn, name, delivery):
    spec = NETS[name]()
    steps = 600
    o = O.OracleNet(spec, O.FP32SO)
    w0 = o.synapses()["wq"]
    o.simulate(steps)
    g = snn.Net(spec, delivery=delivery)
    try:
        assert np.array_equal(g.weights(), w0)
        g.simulate(steps)
        gs, gg, gm = g.spikes()
        os_, og, om = o.spikes()
        assert len(os_) > 50
        assert np.array_equal(gs, os_) and np.array_equal(gg, og) and np.array_equal(gm, om)
        assert np.array_equal(g.get_state("V_m").astype(np.float32), o.get_state("V_m").astype(np.float32))
        w1 = o.synapses()["wq"]
        assert np.count_nonzero(w1 != w0) > 0, "the rule never acted"
        assert np.array_equal(g.weights(), w1)
    finally:
        g.close()


def test_plastic_inputs_per_step(snn):
    """Every step's delivered integer input (plastic weights as they were at
    delivery) equals the oracle's recording."""
    spec = plastic_brunel_big()
    steps = 200
    o = O.OracleNet(spec, O.FP32SO)
    rec = o.record_input(steps + 1)
    o.simulate(steps + 1)
    g = snn.Net(spec, delivery="direct")
    try:
        for n in range(steps):
            g.simulate(1)
            assert np.array_equal(g.get_input(0), rec[n + 1][:, 0]), n
    finally:
        g.close()


def test_plastic_batch_members_equal_the_oracle(snn):
    specs = [plastic_brunel_big(seed=8), plastic_brunel(seed=22), plastic_brunel_big(seed=9)]
    for sp in specs:
        sp["dmax"] = 25
    steps = 400
    g = snn.Net(specs, delivery="binned")
    try:
        g.simulate(steps)
        st, gid, _ = g.spikes()
        wg = g.weights()
        syn = g.synapses()
        for k, sp in enumerate(specs):
            lo, n = g.instances[k]["first"], g.instances[k]["n"]
            o = O.OracleNet(sp, O.FP32SO)
            o.simulate(steps)
            os_, og, _ = o.spikes()
            sel = (gid >= lo) & (gid < lo + n)
            assert np.array_equal(st[sel], os_) and np.array_equal(gid[sel] - lo, og), k
            mine = (syn["src"] >= lo) & (syn["src"] < lo + n)
            assert np.array_equal(wg[mine], o.synapses()["wq"]), k
    finally:
        g.close()


def test_plastic_snapshot_continues(snn):
    spec = plastic_brunel_big()
    a = snn.Net(spec)
    try:
        a.simulate(150)
        blob = a.snapshot()
        a.simulate(150)
        b = snn.Net(spec)
        try:
            b.restore(blob)
            b.simulate(150)
            assert np.array_equal(a.weights(), b.weights())
            sa, sb = a.spikes(150), b.spikes(150)
            assert all(np.array_equal(x, y) for x, y in zip(sa, sb))
        finally:
            b.close()
    finally:
        a.close()


@pytest.mark.parametrize("delivery", ["direct", "binned"])
@pytest.mark.parametrize("n_tgt", [1, 63, 64, 65, 257, 1025])
def test_arrival_list_places(snn, n_tgt, delivery):
    """A few generators onto n_tgt neurons through a plastic and a static
    projection: a step's arrivals fill a wave, a block and a round of the flat
    scan exactly, fall one short or one over, and mix plastic with static
    synapses; every weight equals the oracle's."""
    lif = dict(tau_m=10.0, C_m=250.0, E_L=0.0, V_th=15.0, V_reset=0.0, t_ref=1.0)
    times = [[1.0, 3.3, 6.0], [1.0, 4.1], [2.5, 6.0, 6.1]]
    stdp = dict(tau_plus=10.0, tau_minus=12.0, alpha=1.0, mu_plus=1, mu_minus=1, w_max=9.0, **{"lambda": 0.1})
    pops = [dict(name="G", model="spike_generator", n=3, ports=1, params={}, spike_times=times),
            dict(name="T", model="lif_delta", n=n_tgt, ports=1, params=lif, V0=np.linspace(0.0, 14.5, n_tgt), I_e=0.0)]
    projs = [dict(src="G", tgt="T", rule="all_to_all", weight=4.0, delay=("const", 0.5, 0.0), port=0, stdp=stdp),
             dict(src="G", tgt="T", rule="all_to_all", weight=1.5, delay=("const", 0.5, 0.0), port=0)]
    spec = dict(name="places", dt=0.1, seed=3, dmax=8, populations=pops, projections=projs, poisson=[])
    o = O.OracleNet(spec, O.FP32SO)
    o.simulate(100)
    g = snn.Net(spec, delivery=delivery)
    try:
        g.simulate(100)
        assert np.array_equal(g.spikes()[1], o.spikes()[1])
        assert np.array_equal(g.weights(), o.synapses()["wq"])
    finally:
        g.close()
