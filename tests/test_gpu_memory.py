"""Builds, restores and served requests when device memory runs out: what is
allocated only for speed may be refused at any point, by allocators that leave
HIP's error behind as a failed hipMalloc does, and a restore asks for none."""
import ctypes as C
import sys

import numpy as np
import pytest

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


def brunel(n, k, seed=3, delay=("uniform", 0.1, 1.4), dmax=25):
    return W.brunel_lif(n=n, k=k, seed=seed, delay=delay, dmax=dmax, nu_ext=260.0)


def budget_allocator(snn, limit):
    """At most `limit` bytes; what is beyond is refused after a hipMalloc that fails."""
    hip_malloc = snn.lib().hipMalloc
    hip_malloc.restype, hip_malloc.argtypes = C.c_int, [C.POINTER(C.c_void_p), C.c_size_t]

    class Budget(snn.TorchAllocator):
        def __init__(self):
            super().__init__()
            self.limit, self.held, self.peak, self.sizes = limit, 0, 0, {}

        def _a(self, nbytes, user):
            if self.held + nbytes > self.limit:
                assert hip_malloc(C.byref(C.c_void_p()), 1 << 60) != 0
                return None
            p = super()._a(nbytes, user)
            if p:
                self.sizes[p] = nbytes
                self.held += nbytes
                self.peak = max(self.peak, self.held)
            return p

        def _f(self, ptr, user):
            self.held -= self.sizes.pop(ptr, 0)
            super()._f(ptr, user)

    return Budget()


NETS = {
    "strips": (lambda: [brunel(2100, 600)], dict(delivery="auto"), dict(delivery="direct")),
    "small": (lambda: [brunel(1500, 100)], dict(delivery="auto"), dict(delivery="direct")),
    "pull": (lambda: [brunel(5000, 300), brunel(700, 300, seed=4)], dict(delivery="binned"),
             dict(delivery="binned", bin_capacity=1 << 30)),
}


@pytest.mark.parametrize("name", sorted(NETS))
def test_a_refusal_that_leaves_an_error_behind(snn, name):
    """Budgets from what the plain network needs to what it takes with all that
    makes it faster: each builds, and gives the same raster."""
    make, kw, plain_kw = NETS[name]

    def run(limit, kw):
        al = budget_allocator(snn, limit)
        net = snn.Net(make(), allocator=al, **kw)
        net.simulate(60)
        sp, peak = net.spikes(), al.peak
        net.close()
        return sp, peak

    ref, plain = run(1 << 40, plain_kw)
    _, full = run(1 << 40, kw)
    assert len(ref[0]) > 0
    for limit in np.linspace(plain, full, 9).astype(np.int64):
        sp, _ = run(int(limit), kw)
        assert all(np.array_equal(a, b) for a, b in zip(ref, sp)), limit


def test_restore_allocates_nothing(snn):
    """A pulled network whose allocator gives nothing after the build."""
    al = budget_allocator(snn, 1 << 40)
    make, kw, _ = NETS["pull"]
    a, b = snn.Net(make(), **kw), snn.Net(make(), allocator=al, **kw)
    a.simulate(47)
    b.simulate(30)
    snap = a.snapshot()
    al.limit = al.held
    b.restore(snap)
    for x in (a, b):
        x.simulate(40)
    for x, y in zip(a.spikes(47, 87), b.spikes(47, 87)):
        assert len(x) > 0 and np.array_equal(x, y)
    assert np.array_equal(a.get_state("V_m"), b.get_state("V_m"))
    assert all(a.counters()[k] == b.counters()[k] for k in ("steps", "spikes", "events", "pairs"))


class Server:
    """The library's request server, one request at a time."""

    def __init__(self, snn, budget, slots):
        self.S, self.L, self.h = snn, snn.lib(), C.c_void_p()
        assert self.L.snn_server_create(int(budget), slots, C.byref(self.h)) == 0

    def submit(self, net, steps):
        t = C.c_uint64()
        assert self.L.snn_server_submit(self.h, net.h, steps, C.byref(t)) == 0
        return t.value

    def result(self, ticket, timeout=60.0):
        out, info = C.c_void_p(), self.S.JobInfo()
        assert self.L.snn_server_wait(self.h, ticket, timeout) == 0
        self.L.snn_server_result(self.h, ticket, C.byref(out), C.byref(info))
        return info

    def close(self):
        self.L.snn_server_destroy(self.h)


def test_served_network_without_device_memory_fails_as_such(snn):
    """The budget refuses the bins' scratch (12 10^6 synapses), then the device
    has no room for the raster ring (32 MiB): that is the failure, once."""
    class NoRing(snn.TorchAllocator):
        def _a(self, nbytes, user):
            return None if nbytes == 32 << 20 else super()._a(nbytes, user)

    net = snn.Net(brunel(4000, 3000), allocator=NoRing(), build=False)
    srv = Server(snn, 120 << 20, 1)
    try:
        info = srv.result(srv.submit(net, 20))
        assert info.status == -2 and info.attempts == 1, (info.status, info.attempts, info.error)
    finally:
        srv.close()
        net.close()


def test_extra_memory_keeps_no_request_waiting(snn):
    """A budget for two networks without their strips: each is built at once."""
    spec = lambda: [brunel(2100, 400)]
    al = budget_allocator(snn, 1 << 40)
    snn.Net(spec(), allocator=al, delivery="direct").close()
    nets = [snn.Net(spec(), build=False) for _ in range(2)]
    srv = Server(snn, 2 * al.peak + (1 << 20), 2)
    try:
        tickets = [srv.submit(net, 20000) for net in nets]
        for net, t in zip(nets, tickets):
            info = srv.result(t)
            assert info.status == 0 and info.attempts == 1
        assert all(np.array_equal(a, b) for a, b in zip(nets[0].spikes(), nets[1].spikes()))
    finally:
        srv.close()
        for net in nets:
            net.close()


def test_pulled_network_keeps_no_bins(snn):
    """bins_total of a snapshot's header: 8 bytes each, two buffers, in the binned
    network; the pulled one holds no such array."""
    def sizes(**kw):
        al = budget_allocator(snn, 1 << 40)
        net = snn.Net(NETS["pull"][0](), allocator=al, delivery="binned", **kw)
        total = int(net.snapshot()[32:40].view(np.uint64)[0])
        out = net.step_kernel(), (8 * total + 255) // 256 * 256 in al.sizes.values()
        net.close()
        return out

    assert sizes() == ("k_pull", False)
    assert sizes(bin_capacity=100_000) == ("k_step_binned_runs", True)
