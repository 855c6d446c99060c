"""Which kernel steps a network: the networks of the parity tests of the
one-block, strip and pulled steps run those kernels (and forced delivery or an
asked-for bin size the others), so that what these tests compare is what they are
about; and networks at the edges of the rules."""
import sys

import numpy as np
import pytest

import test_gpu_pull as TP
import test_gpu_small as TS
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


def kernel(snn, specs, **kw):
    net = snn.Net(specs, **kw)
    try:
        return net.step_kernel()
    finally:
        net.close()


# networks of the small tests that one block does not step: more than four weight classes onto a neuron; 4,200 synapses
# drawn onto 300 neurons from parrots of up to 31 spikes a step, which 16 bits need not count
NOT_SMALL = ("many_classes", "devices")


@pytest.mark.parametrize("name", sorted(TS.NETS))
def test_small_networks(snn, name):
    assert kernel(snn, TS.NETS[name]()) == ("k_step_strip" if name in NOT_SMALL else "k_small")
    assert kernel(snn, TS.NETS[name](), delivery="direct") == "k_step"


@pytest.mark.parametrize("name", sorted(TT.NETS))
def test_strips(snn, name):
    specs, kw = TT.NETS[name]()
    assert kernel(snn, specs, **kw) == "k_step_strip"
    assert kernel(snn, specs, delivery="direct", **kw) == "k_step"


@pytest.mark.parametrize("name", sorted(TP.NETS))
def test_pulled_networks(snn, name):
    make, tile = TP.NETS[name]
    tile = 1024 if tile else 0
    assert kernel(snn, make(), delivery="binned", tile_neurons=tile) == "k_pull"
    assert kernel(snn, make(), delivery="binned", tile_neurons=tile, bin_capacity=1 << 20) == "k_step_binned_runs"


def test_devices_in_one_block(snn, monkeypatch):
    """The devices of the small tests with few enough synapses for 16-bit counts."""
    sp = TS.devices()
    sp["projections"][1]["K"] = 25
    assert kernel(snn, sp) == "k_small"
    monkeypatch.setitem(TS.NETS, "few_from_devices", lambda: [sp])
    TS.test_small_networks_bit_exact(snn, "few_from_devices")
    for src, dst in (("auto", "auto"), ("auto", "direct"), ("direct", "auto")):
        TS.test_small_snapshots(snn, "few_from_devices", src, dst)


def test_edges_of_the_rules(snn):
    b = lambda n, k: W.brunel_lif(n=n, k=k, nu_ext=260.0, delay=("uniform", 0.1, 0.4), dmax=5)
    assert kernel(snn, b(2045, 50)) == "k_small" and kernel(snn, b(2050, 50)) == "k_step_strip"
    meter = dict(b(500, 50), multimeters=[dict(var="V_m", gids=[0, 3], interval=5)])
    assert kernel(snn, meter) == "k_step_strip"
    stdp = b(500, 50)
    stdp["projections"][0]["stdp"] = dict(w_max=1.0)
    assert kernel(snn, stdp) == "k_step"
    assert kernel(snn, W.adex_balanced(n=2000, k=100)) == "k_step_binned"
    assert kernel(snn, W.adex_balanced(n=2000, k=100), delivery="direct") == "k_step"
    net = snn.Net(b(500, 50), build=False)
    assert net.step_kernel() == ""
    net.build()
    net.simulate(3)
    net._check(net.L.snn_release(net.h))
    assert net.step_kernel() == "k_small"
    net.close()
