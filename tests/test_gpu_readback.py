"""Readback through the C ABI: a raster read in windows equals the raster read
once (windows that end where a drain was started among them), in every way of
delivery; per-port state written and read back by ranges."""
import numpy as np
import pytest

from paper_2007_14236_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def snn():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2007_14236_amd import snn as S
    S.lib()
    return S


NETS = {
    "direct": lambda: (W.brunel_lif(n=1000, k=100, seed=3, nu_ext=260.0), dict(delivery="direct")),
    "tiles": lambda: (W.brunel_lif(n=3000, k=60, seed=4, nu_ext=260.0, delay=("uniform", 0.1, 2.0)),
                      dict(delivery="binned", tile_neurons=256)),
    "adex": lambda: (W.adex_balanced(n=2000, k=100, seed=5), dict()),
    "pulled": lambda: ([W.brunel_lif(n=5000 + 777 * i, k=300, seed=6 + i, nu_ext=260.0) for i in range(2)],
                       dict(delivery="binned")),
}


@pytest.mark.parametrize("name", sorted(NETS))
@pytest.mark.parametrize("steps", [[1000], [100, 900, 1000], [999, 1, 1, 1000, 37]])
def test_raster_windows(snn, name, steps):
    spec, cfg = NETS[name]()
    a, b = snn.Net(spec, **cfg), snn.Net(spec, **cfg)
    got, t = [], 0
    for n in steps:
        a.simulate(n)
        got.append(a.spikes(t, t + n))
        t += n
    b.simulate(t)
    want = b.spikes()
    assert len(want[0]) > 100
    for k in range(3):
        assert np.array_equal(np.concatenate([x[k] for x in got]), want[k])
    key = want[0].astype(np.int64) * (1 << 32) + want[1]
    assert np.all(np.diff(key) > 0)  # by step, then gid
    assert len(want[0]) == b.counters()["spikes"]


@pytest.mark.parametrize("first,n", [(0, 1), (0, 700), (3, 5), (699, 1), (100, 600)])
def test_port_state_ranges(snn, first, n):
    spec = W.adex_balanced(n=700, k=20, seed=2)
    net = snn.Net(spec)
    base = [np.linspace(0.0, 3.0, 700).astype(np.float32) + p for p in (0, 1)]
    for p in (0, 1):
        net.set_state("g", 0, base[p], port=p)
    new = np.arange(n, dtype=np.float32) + 50
    net.set_state("g", first, new, port=1)
    base[1][first:first + n] = new
    for p in (0, 1):
        assert np.array_equal(net.get_state("g", port=p), base[p])
        assert np.array_equal(net.get_state("g", first, n, port=p), base[p][first:first + n])
    net.set_state("V_m", first, [-61.5], n=n)
    assert np.all(net.get_state("V_m", first, n) == -61.5)
    ref = [net.get_input(p) for p in (0, 1)]
    net.simulate(7)
    for p in (0, 1):
        assert np.array_equal(net.get_input(p, first, n), net.get_input_noalloc(p, first, n))
    assert len(ref[0]) == 700
