"""Strips at the edges of their rules: half a wave's neurons a strip and a whole
one's, a last strip of one neuron, few targets that take all the events of a step,
lists that overflow; rasters, inputs, state and counters bit-exact against the
oracle and against delivery by device atomics."""
import sys

import numpy as np
import pytest

import test_gpu_strip as TT
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


def check(snn, monkeypatch, specs, **kw):
    net = snn.Net(specs, **kw)
    assert net.step_kernel() == "k_step_strip"
    net.close()
    monkeypatch.setitem(TT.NETS, "here", lambda: (specs, kw))
    TT.test_strips_bit_exact(snn, "here")


@pytest.mark.parametrize("n", [2080, 8192, 8193])
def test_strips_of_half_a_wave_and_of_one(snn, monkeypatch, n):
    check(snn, monkeypatch, [TT.brunel(n, 60)])


@pytest.mark.parametrize("targets", [1, 33, 500])
def test_generators_onto_few_neurons(snn, monkeypatch, targets):
    """300 generators, a third of them in each step, 60,000 synapses."""
    times = [[0.1 * (1 + s) for s in range(i % 3, 200, 3)] for i in range(300)]
    lif = dict(tau_m=20.0, C_m=250.0, E_L=0.0, V_th=20.0, V_reset=10.0, t_ref=2.0)
    pops = [dict(name="G", model="spike_generator", n=300, ports=1, params={}, spike_times=times),
            dict(name="L", model="lif_delta", n=targets, ports=1, params=lif, V0=np.linspace(0.0, 19.0, targets), I_e=100.0)]
    projs = [dict(src="G", tgt="L", rule="fixed_outdegree", K=200, weight=0.02 * targets / 500, delay=("uniform", 0.1, 2.0), port=0)]
    check(snn, monkeypatch, [dict(name="few", dt=0.1, seed=3, dmax=25, populations=pops, projections=projs, poisson=[])])


@pytest.mark.parametrize("delay", [("uniform", 0.1, 2.5), ("const", 0.1, 0.0), ("const", 0.7, 0.0)], ids=["many", "first", "one"])
def test_rows_beyond_a_block(snn, monkeypatch, delay):
    """Sources of 8,191, 8,192 and 8,193 synapses and of some 20,000, which are brought
    to their strips in two ways; each source fires."""
    lif = dict(tau_m=20.0, C_m=250.0, E_L=0.0, V_th=20.0, V_reset=10.0, t_ref=2.0)
    pops = [dict(name=f"S{k}", model="lif_delta", n=3, ports=1, params=dict(lif), V0=np.array([3.0, 15.0, 19.9]), I_e=400.0)
            for k in (8191, 8192, 8193, 20011)]
    pops.append(dict(name="T", model="lif_delta", n=2501, ports=1, params=dict(lif), V0=np.linspace(0.0, 19.9, 2501), I_e=200.0))
    projs = [dict(src=p["name"], tgt="T", rule="fixed_outdegree", K=int(p["name"][1:]), weight=w, delay=delay, port=0)
             for p, w in zip(pops, (0.11, -0.07, 0.05, 0.02))]
    check(snn, monkeypatch, [dict(name="rows", dt=0.1, seed=5, dmax=30, populations=pops, projections=projs, poisson=[])])
