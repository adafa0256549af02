"""The limits of fixed scratch (the static area, an engine's budget).

What a hologram counts for does not follow the operand tables that the kernels
happen to use (on grids wider than high they take more than they count for,
from a reserve behind the limit), so the largest number of spots that is
accepted is part of the interface: it runs and equals the same hologram with
memory of its own, and one spot more is refused.
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


@pytest.mark.parametrize("W,H,I,c,precision,N", [
    (1920, 1152, 2, 1 / 16, "fp32", 944),
    (1920, 1152, 0, 1.0, "fp32", 1104),
    (1152, 1920, 2, 1 / 16, "fp32", 864),
    (1152, 1152, 2, 1 / 16, "fp32", 1280),
    (8192, 64, 2, 1 / 4, "fp32", 464),
    (1920, 1152, 2, 1 / 16, "mixed", 1280),
])
def test_largest_static_hologram(W, H, I, c, precision, N):
    import torch
    print("[case] scratch limit", W, H, I, precision, N, flush=True)
    g = Grid(W, H)
    phi = torch.empty(g.M, dtype=torch.float32, device="cuda")
    s = on_gpu(spot_cloud(1, N, g))
    hg.cswgs_static(g, OPTICS, s, I, c, 1, phi, precision=precision)
    ref = hg.cswgs_device(g, OPTICS, s, I, c, 1, precision=precision)
    torch.cuda.synchronize()
    assert np.array_equal(phi.cpu().numpy(), ref.cpu().numpy())
    with pytest.raises(hg.HGError, match="HG_ENOMEM"):
        hg.cswgs_static(g, OPTICS, on_gpu(spot_cloud(1, N + 1, g)), I, c, 1, phi,
                        precision=precision)


def test_engine_budget():
    """Two requests, each of almost the whole budget, are served one after the
    other; 1152 spots count for 72 x 64 lanes x 32 bytes x (2 x 120 + 3 x 72
    blocks), more than the budget.  (The random order is shared: it does not
    count here.)"""
    import torch
    print("[case] scratch limit, engine", flush=True)
    g, N = Grid(1920, 1152), 1072
    spots = [spot_cloud(k, N, g) for k in range(2)]
    e = hg.Engine((63 << 20) - 256, 4)
    st = torch.cuda.Stream()
    phis = [torch.empty(g.M, dtype=torch.float32, device="cuda") for _ in spots]
    tickets = [e.submit(g, OPTICS, s, 2, 1 / 16, k, p) for k, (s, p) in enumerate(zip(spots, phis))]
    for _ in range(50):
        e.step(stream=st)
        st.synchronize()
        if all([e.poll(t) for t in tickets]):
            break
    with pytest.raises(hg.HGError, match="HG_ENOMEM"):
        e.submit(g, OPTICS, spot_cloud(3, 1152, g), 2, 1 / 16, 1, phis[0])
    e.close()
    for k, (s, p) in enumerate(zip(spots, phis)):
        ref = hg.cswgs_device(g, OPTICS, on_gpu(s), 2, 1 / 16, k)
        assert np.array_equal(p.cpu().numpy(), ref.cpu().numpy()), k
