"""Jobs whose scratch comes out of a limit that the caller set (an engine's
budget, the static area): the limit bounds the device memory that is taken, and
the full-grid iteration pass, which does without the forward product's own
operand table there, gives the same bits.
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


@pytest.mark.parametrize("budget_mib", [64, 512, 2048])
def test_engine_takes_no_more_than_its_budget(budget_mib):
    """The pool is allocated at creation; 8 MiB cover the allocator's granules
    and the small buffers beside it."""
    import torch
    print("[case] fixed scratch, engine memory", budget_mib, flush=True)
    hg.Engine(1 << 20, 1).close()  # what the first engine of a process sets up
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    e = hg.Engine(budget_mib << 20, 4)
    torch.cuda.synchronize()
    taken = before - torch.cuda.mem_get_info()[0]
    e.close()
    assert taken <= (budget_mib + 8) << 20, taken / 2 ** 20


# one block of 16 spots, remainders of the groups of four blocks, more than the
# waves bring together at a time (128), and both tile edges ragged
@pytest.mark.parametrize("W,H", [(33, 65), (130, 67), (64, 192)])
@pytest.mark.parametrize("N", [1, 16, 17, 33, 49, 64, 65, 128, 129, 260, 513])
def test_static_area_gives_the_same_bits(W, H, N):
    import torch
    print("[case] fixed scratch, static area", W, H, N, flush=True)
    g = Grid(W, H)
    s = on_gpu(spot_cloud(N, N, g))
    for I, c in ((1, 0.5), (3, 0.5)):
        phi = torch.empty(g.M, dtype=torch.float32, device="cuda")
        hg.cswgs_static(g, OPTICS, s, I, c, 2, phi)
        ref = hg.cswgs_device(g, OPTICS, s, I, c, 2)
        torch.cuda.synchronize()
        assert np.array_equal(phi.cpu().numpy(), ref.cpu().numpy()), I


def test_engine_requests_of_several_widths():
    """FP32 requests on wide, square and tall grids in the same steps."""
    import torch
    print("[case] fixed scratch, engine widths", flush=True)
    shapes = [(300, 90, 20), (128, 128, 100), (90, 300, 70), (257, 130, 300)]
    st = torch.cuda.Stream()
    e = hg.Engine(64 << 20, 4)
    phis, tickets = [], []
    for k, (W, H, N) in enumerate(shapes):
        g = Grid(W, H)
        phis.append(torch.empty(g.M, dtype=torch.float32, device="cuda"))
        tickets.append(e.submit(g, OPTICS, spot_cloud(k, N, g), 4, 0.25, k, phis[-1]))
    for _ in range(20):
        e.step(stream=st)
        st.synchronize()
        if all([e.poll(t) for t in tickets]):
            break
    e.close()
    for k, (W, H, N) in enumerate(shapes):
        g = Grid(W, H)
        ref = hg.cswgs(g, OPTICS, spot_cloud(k, N, g), 4, 0.25, k)
        assert np.array_equal(phis[k].cpu().numpy(), ref.cpu().numpy()), k
