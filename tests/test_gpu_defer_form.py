"""The compressed pass that takes and leaves deferred updates (k_pass_defer),
at the edges of its dispatch.

The pass keeps the arithmetic and summation order of the per-pixel pass, so
the bar is bit identity with what still runs that pass: up to 256 spots the
chained launch (N at the edges of every spot-lane layout, a window whose last
tile is ragged, fewer blocks than tiles, and tiles of two 64-pixel parts, for
windows of more than 8192 x 64 pixels), above 256 spots (two spot units per
wave) the wide per-pixel pass of direct=True.
"""
import numpy as np
import pytest

import paper_2003_05293_amd as hg
from workload import Grid, OPTICS, PUPIL_OPTICS, spot_cloud

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    import torch
    assert torch.cuda.is_available()
    hg.load()
    yield
    torch.cuda.synchronize()


def run(g, optics, s, I, c, seed, **tune):
    phi, V = hg.cswgs(g, optics, s, I, c, seed, trace=True, tune=tune)
    return phi.cpu().numpy(), np.asarray(V)


@pytest.mark.parametrize("N", [1, 8, 9, 16, 17, 32, 33, 64, 65, 128, 129, 192, 193, 256])
@pytest.mark.parametrize("optics", [OPTICS, PUPIL_OPTICS], ids=["uniform", "pupil"])
def test_equals_chained(N, optics):
    print("[case] defer form vs chained", N, flush=True)
    g = Grid(131, 97)
    s = spot_cloud(N, N, g)
    phi, V = run(g, optics, s, 4, 0.3, 7)
    phi_c, V_c = run(g, optics, s, 4, 0.3, 7, chain_passes=1)
    assert np.array_equal(phi, phi_c) and np.array_equal(V, V_c)
    phi_b, V_b = run(g, optics, s, 4, 0.3, 7, subset_block_cap=5)
    assert np.array_equal(phi, phi_b) and np.array_equal(V, V_b)


def test_two_parts_per_tile_equals_chained():
    print("[case] defer form, two parts per tile", flush=True)
    g = Grid(1100, 1000)  # 550,000 window pixels
    s = spot_cloud(3, 21, g)
    phi, V = run(g, OPTICS, s, 3, 0.5, 1, subset_block_cap=700)
    phi_c, V_c = run(g, OPTICS, s, 3, 0.5, 1, subset_block_cap=700, chain_passes=1)
    assert np.array_equal(phi, phi_c) and np.array_equal(V, V_c)


@pytest.mark.parametrize("N", [257, 320, 321, 512, 513])
def test_many_spots_equal_per_pixel_pass(N):
    """Two spot units per wave: the fields of every compressed iteration
    against the wide per-pixel pass (which direct=True keeps)."""
    print("[case] defer form, many spots", N, flush=True)
    g, I = Grid(131, 97), 4
    s = spot_cloud(N, N, g)
    phi, V = run(g, OPTICS, s, I, 0.4, 5)
    _, V_d = hg.cswgs(g, OPTICS, s, I, 0.4, 5, trace=True, direct=True)
    assert np.array_equal(V[:I - 1], np.asarray(V_d)[:I - 1])
    phi_b, V_b = run(g, OPTICS, s, I, 0.4, 5, subset_block_cap=5)
    assert np.array_equal(phi, phi_b) and np.array_equal(V, V_b)


@pytest.mark.parametrize("precision", ["fp32", "mixed"])
def test_large_launch_equals_alone(precision):
    """A launch of several tiles per block (forward sums by chains from 33
    spots on) against each hologram alone (by units)."""
    import torch
    g, I, c = Grid(641, 509), 3, 0.3
    counts = [32, 33, 40, 64, 65, 100, 127, 128, 129, 150, 192, 200, 255, 256]
    jobs = [hg.DeviceJob.from_spots(g, OPTICS, spot_cloud(n, n, g), I, c, n, precision=precision)
            for n in counts]
    print("[case] defer form, large launch", precision, flush=True)
    hg.cswgs_batch(jobs)
    torch.cuda.synchronize()
    for n, job in zip(counts, jobs):
        phi = hg.cswgs(g, OPTICS, spot_cloud(n, n, g), I, c, n, precision=precision)
        assert np.array_equal(phi.cpu().numpy(), job.phi.cpu().numpy()), n


@pytest.mark.parametrize("N", [20, 100])
def test_more_tiles_than_resident_blocks(N):
    """One pass of more than 2048 tiles (some blocks take two) against the
    chained launch, and three passes of 6600 tiles together against each
    alone."""
    import torch
    g, I, c = Grid(641, 509), 3, 0.43  # 140,292 window pixels
    spots = [spot_cloud(N + k, N + k, g) for k in range(3)]
    print("[case] defer form, more tiles than resident blocks", N, flush=True)
    alone = []
    for s in spots:
        phi, V = run(g, OPTICS, s, I, c, 3)
        phi_c, V_c = run(g, OPTICS, s, I, c, 3, chain_passes=1)
        assert np.array_equal(phi, phi_c) and np.array_equal(V, V_c)
        alone.append(phi)
    jobs = [hg.DeviceJob.from_spots(g, OPTICS, s, I, c, 3) for s in spots]
    hg.cswgs_batch(jobs)
    torch.cuda.synchronize()
    for phi, job in zip(alone, jobs):
        assert np.array_equal(phi, job.phi.cpu().numpy())
