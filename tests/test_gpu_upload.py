"""Descriptor tables and host spots on their way to the GPU: pieces of up to
256 KiB are read by a kernel from pinned memory, up to 16 pieces per launch,
larger ones go by copy commands.  Whichever way they take, the results are
those of spots that lie on the GPU already, bit for bit.
"""
import numpy as np
import pytest

import paper_2003_05293_amd as hg
from workload import Grid, OPTICS, spot_cloud

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    import torch
    assert torch.cuda.is_available()
    hg.load()
    yield
    torch.cuda.synchronize()


def on_gpu(s):
    import torch
    return torch.tensor(np.stack([s.x_mm, s.y_mm, s.z_mm, s.amp]), dtype=torch.float64,
                        device="cuda")


@pytest.mark.parametrize("N", [1, 3, 257, 4096])
def test_host_spots_equal_device_spots(N):
    print("[case] upload, host spots", N, flush=True)
    g = Grid(64, 48)
    s = spot_cloud(N, N, g)
    for seed in (1, 2, 3):  # the same staging, refilled while the last call may run
        a = hg.cswgs(g, OPTICS, s, 2, 0.5, seed)
        b = hg.cswgs_device(g, OPTICS, on_gpu(s), 2, 0.5, seed)
        assert np.array_equal(a.cpu().numpy(), b.cpu().numpy())


@pytest.mark.parametrize("count", [15, 16, 17, 33])
def test_requests_of_one_step(count):
    """count arrays of spots and the tables in one step of the engine."""
    import torch
    print("[case] upload, engine", count, flush=True)
    g = Grid(96, 80)
    spots = [spot_cloud(50 + k, 3 + 5 * (k % 7), g) for k in range(count)]
    e = hg.Engine(1 << 28, count)
    st = torch.cuda.Stream()
    phis = [torch.empty(g.M, dtype=torch.float32, device="cuda") for _ in spots]
    tickets = [e.submit(g, OPTICS, s, 3, 0.5, k, p) for k, (s, p) in enumerate(zip(spots, phis))]
    for _ in range(20):
        e.step(stream=st)
        if all([e.poll(t) for t in tickets]):
            break
    st.synchronize()
    e.close()
    for k, (s, p) in enumerate(zip(spots, phis)):
        ref = hg.cswgs_device(g, OPTICS, on_gpu(s), 3, 0.5, k)
        assert np.array_equal(p.cpu().numpy(), ref.cpu().numpy()), k


@pytest.mark.parametrize("count", [8, 96])
def test_tables_of_a_batch(count):
    """The tables of 8 holograms (a kernel reads them) and of 96 (a copy)."""
    import torch
    print("[case] upload, batch", count, flush=True)
    g = Grid(64, 64)
    spots = [spot_cloud(k, 4 + k % 5, g) for k in range(count)]
    jobs = [hg.DeviceJob.from_spots(g, OPTICS, s, 12, 0.25, k) for k, s in enumerate(spots)]
    hg.cswgs_batch(jobs)
    torch.cuda.synchronize()
    for k in (0, count - 1):
        ref = hg.cswgs_device(g, OPTICS, on_gpu(spots[k]), 12, 0.25, k)
        assert np.array_equal(jobs[k].phi.cpu().numpy(), ref.cpu().numpy())


def test_capture_by_the_caller_stays_refused():
    """A replay would read the staging area as later calls have left it."""
    import torch
    print("[case] upload, captured stream", flush=True)
    g = Grid(64, 48)
    s = on_gpu(spot_cloud(1, 20, g))
    st = torch.cuda.Stream()
    phi = torch.empty(g.M, dtype=torch.float32, device="cuda")
    with torch.cuda.stream(st):
        hg.cswgs_device(g, OPTICS, s, 3, 0.25, 1, phi=phi, stream=st)
    torch.cuda.synchronize()
    ref = phi.clone()
    with pytest.raises(Exception):
        with torch.cuda.graph(torch.cuda.CUDAGraph(), stream=st):
            hg.cswgs_device(g, OPTICS, s, 3, 0.25, 1, phi=phi, stream=st)
    phi.zero_()
    torch.cuda.synchronize()
    with torch.cuda.stream(st):
        hg.cswgs_device(g, OPTICS, s, 3, 0.25, 1, phi=phi, stream=st)
    torch.cuda.synchronize()
    assert torch.equal(phi, ref)


@pytest.mark.parametrize("entry", ["single", "batch"])
def test_every_capture_by_the_caller_is_refused(entry):
    """Also where the attempts follow each other without an ordinary call
    between them, and again after one.  (An engine's step waits for its own
    events first, which HIP refuses on a captured stream.)"""
    import torch
    print("[case] upload, captures in a row", entry, flush=True)
    g = Grid(64, 48)
    spots = spot_cloud(1, 20, g)
    s = on_gpu(spots)
    st = torch.cuda.Stream()
    phi = torch.empty(g.M, dtype=torch.float32, device="cuda")
    job = hg.DeviceJob.from_spots(g, OPTICS, spots, 3, 0.25, 1)
    torch.cuda.synchronize()

    def call():
        if entry == "single":
            hg.cswgs_device(g, OPTICS, s, 3, 0.25, 1, phi=phi, stream=st)
        else:
            hg.cswgs_batch([job], stream=st)

    with torch.cuda.stream(st):
        call()
    torch.cuda.synchronize()
    for attempts in (3, 2):
        for k in range(attempts):
            with pytest.raises(hg.HGError, match="HG_EDEVICE"):
                with torch.cuda.graph(torch.cuda.CUDAGraph(), stream=st):
                    call()
        torch.cuda.synchronize()
        with torch.cuda.stream(st):
            call()
        torch.cuda.synchronize()
