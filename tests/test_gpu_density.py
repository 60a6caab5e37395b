"""The density pass at the sizes where its tiles of 2048 points and its two ways to sum them
(the last of up to 256 blocks, or a second launch) change over: rho against the sum of the
returned n, the copies of n to device and host memory, and the same bits from every way to
call it.  The sum of n is exact to a rounding per addition: 1e-14 relative, as elsewhere.
"""
import math

import numpy as np
import pytest

from paper_1607_03062_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(1, 1), (23, 89), (32, 64), (683, 3), (1024, 512), (1025, 512)])
@pytest.mark.parametrize("scheme,precision", [("strang", "fp64"), ("strang", "fp32"), ("midpoint", "fp64")])
def test_density_and_snapshot(gpu, nx, ny, scheme, precision):
    import torch

    g = {"nx": nx, "ny": ny, "px": (-1.3, 1.2), "py": (-1.1, 1.4)}
    s = gpu.Solver.for_grid(g, precision, scheme).set_field(wl.sin2(0.3, 0.6, 2), 200)
    scale = 4 * (2.5 / nx) * (2.5 / ny) / (4 * math.pi ** 2)
    st = torch.cuda.Stream()

    def both(call):
        """rho and n of a call with n to the device and with n to the host; they agree."""
        dev, host = torch.empty(nx * ny, dtype=torch.float64, device="cuda"), np.empty(nx * ny)
        rho = call(dev, st)
        assert call(host, st) == rho and call(None, st) == rho
        st.synchronize()
        assert np.array_equal(dev.cpu().numpy(), host)
        want = scale * math.fsum(host)
        assert abs(rho - want) <= 1e-14 * want
        return rho, host

    s.propagate(90, stream=st)
    both(lambda n, t: s.snapshot(n_out=n, stream=t))
    s.propagate(-1, stream=st)
    end = both(lambda n, t: s.density(n_out=n, stream=t))
    static = both(lambda n, t: s.density_static(n_out=n, stream=t))
    last = both(lambda n, t: s.snapshot(n_out=n, stream=t))
    for other in (static, last):
        assert other[0] == end[0] and np.array_equal(other[1], end[1])
    only_n = torch.empty(nx * ny, dtype=torch.float64, device="cuda")
    assert s.density(n_out=only_n, want_rho=False, stream=st) is None
    st.synchronize()
    assert np.array_equal(only_n.cpu().numpy(), end[1])
    s.close()


def test_first_density_of_new_handles_on_a_stream_that_waits_for_nothing(gpu):
    """What a first pd_set_field clears is cleared when it returns: the first density of each
    of many new handles, on a stream without any order to the default one."""
    import torch

    st = torch.cuda.Stream()
    g, f = wl.grid(40, 1.5), wl.sin2(0.2, 0.6, 2)
    got = []
    for _ in range(40):
        s = gpu.Solver.for_grid(g, "fp64").set_field(f, 64)
        got.append(s.propagate(-1, stream=st).density(stream=st))
        got.append(s.density(stream=st))
        s.close()
    assert got[0] > 0 and got.count(got[0]) == len(got)


def test_overlapping_static_densities_leave_later_calls_alone(gpu):
    """Two threads call pd_density_static on handles of 4 and of 10 tiles at the same time, each
    on its own stream: those calls share the device's scratch and may be wrong, what comes
    after them may not."""
    import threading

    import torch

    f, made = wl.sin2(0.3, 0.6, 2), []
    for n in (90, 140):
        s = gpu.Solver.for_grid(wl.grid(n, 1.5), "fp64").set_field(f, 150)
        st = torch.cuda.Stream()
        s.propagate(-1, stream=st)
        made.append((s, st, s.density(stream=st)))

    def call(s, st):
        for _ in range(300):
            s.density_static(stream=st)

    threads = [threading.Thread(target=call, args=(s, st)) for s, st, _ in made]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for s, st, rho in made + made[::-1]:
        assert s.density_static(stream=st) == rho and s.density(stream=st) == rho
        assert s.snapshot(stream=st) == rho
    for s, _, _ in made:
        s.close()


def test_n_to_memory_that_only_a_copy_reaches(gpu):
    """n_out_on_device = 1 with an address that is no memory of the handle's device (here
    page-locked host memory), and one that is not a multiple of 8: what the copy engine
    reaches, the call serves, from pd_density, pd_density_static and pd_snapshot."""
    import ctypes

    import torch

    from paper_1607_03062_amd import _lib

    m = 60 * 50
    s = gpu.Solver.for_grid({"nx": 60, "ny": 50, "px": (-1.3, 1.2), "py": (-1.1, 1.4)}, "fp64")
    s.set_field(wl.sin2(0.3, 0.6, 2), 300)
    pinned = torch.zeros(m, dtype=torch.float64, pin_memory=True)
    raw = torch.zeros(8 * m + 8, dtype=torch.uint8, device="cuda")
    lib, st = _lib.load(), torch.cuda.Stream()
    for name in ("pd_snapshot", "pd_density", "pd_density_static"):
        if name != "pd_density_static":
            s.propagate(150, stream=st)
        want = np.empty(m)
        rho_want = (s.snapshot if name == "pd_snapshot" else s.density)(n_out=want, stream=st)
        for address in (pinned.data_ptr(), raw.data_ptr() + 4):
            rho = ctypes.c_double()
            assert getattr(lib, name)(s.handle, address, 1, ctypes.byref(rho), _lib.stream_handle(st)) == 0
            st.synchronize()
            got = pinned.numpy() if address == pinned.data_ptr() else raw[4:4 + 8 * m].cpu().numpy().view(np.float64)
            assert rho.value == rho_want and np.array_equal(got, want), name
            pinned.zero_()
            raw.zero_()
            torch.cuda.synchronize()
    s.close()


def test_captured_pass_with_its_sum(gpu):
    """A density pass, sum included, in a graph of the caller's (a snapshot on the way), replayed
    between eager work of the same and of other handles: n bit for bit each time, and the
    handle's later sums as before."""
    import torch

    g, f = wl.grid(150, 2.0), wl.sin2(0.15, 0.5, 4)
    s = gpu.Solver.for_grid(g, "fp64").set_field(f, 800)
    want = np.empty(150 * 150)
    rho = s.propagate(300).snapshot(n_out=want)
    s.rewind()
    n, cap, graph = torch.zeros(150 * 150, dtype=torch.float64, device="cuda"), torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=cap, capture_error_mode="thread_local"):
        s.propagate(300, stream=cap)
        s.snapshot(n_out=n, want_rho=False, stream=cap)
    torch.cuda.synchronize()
    for _ in range(5):
        n.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(n.cpu().numpy(), want)
        assert s.snapshot() == rho
        gpu.Solver.for_grid(wl.grid(40, 1.5), "fp64").set_field(f, 100).solve()
    del graph
    s.close()
