"""Poisson counts, drawn eight thresholds at a time: means about and far beyond a
round of eight, several tables; as read back, and as the kernels of every kind of
network use them (potentials against the oracle)."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2007_14236_amd import workloads as W

pytestmark = pytest.mark.gpu

LIF = dict(tau_m=20.0, C_m=250.0, E_L=0.0, V_th=20.0, V_reset=10.0, t_ref=2.0)


@pytest.fixture(scope="module")
def snn():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2007_14236_amd import snn as S
    S.lib()
    return S


def spec(n, means):
    pops = [dict(name=f"P{k}", model="lif_delta", n=n + k, ports=1, params=dict(LIF), V0=None, I_e=0.0)
            for k in range(len(means))]
    projs = [dict(src="P0", tgt="P0", K=3, weight=0.01, delay=("const", 0.2, 0.0), port=0)]
    pois = [dict(tgt=f"P{k}", rate=m * 100.0, n_inputs=100, weight=0.02, port=0) for k, m in enumerate(means)]
    return dict(name="poisson", dt=0.1, seed=5, dmax=4, populations=pops, projections=projs, poisson=pois)


@pytest.mark.parametrize("delivery", ["auto", "direct", "binned"])
@pytest.mark.parametrize("n", [300, 1100])
def test_poisson_counts_over_means(snn, n, delivery):
    sp = spec(n, (0.02, 1.0, 7.5, 8.5, 16.0, 40.0, 60.0))
    g, o = snn.Net(sp, delivery=delivery), O.OracleNet(sp, O.FP32SO)
    some = np.arange(0, g.N, 37)
    for step in (0, 12345):
        assert np.array_equal(g.poisson_counts(step)[some], [o.poisson_count(int(i), step) for i in some])
    g.simulate(25)
    o.simulate(25)
    assert np.array_equal(g.get_state("V_m").astype(np.float32), o.get_state("V_m").astype(np.float32))
    for x, y in zip(g.spikes(), o.spikes()):
        assert np.array_equal(x.astype(np.int64), y.astype(np.int64))
