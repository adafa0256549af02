"""Compressed holograms on grids of one column (and of one row) in the passes
that take and leave deferred updates.

Mixed precision, every iteration against the FP64 oracle with the state that
the fields of the iterations before it give (so no iteration's rounding is
amplified by the next): V is the mean over the m pixels of the iteration's set
of terms whose operands carry FP16 roundings, 8 2^-11 / sqrt(m) where these are
independent from pixel to pixel (the bar of the mixed forward pass); on one
line a spot's coefficient or amplitude, and its factor along the line's normal,
are rounded once for all pixels, at most 2^-11 per component for each of the
four operands of the two products, in line with V_n: 8 2^-11 |V_n| more.  The
same for the fields of the final hologram.  FP32: bit identity with the chained launch, which hands its
state over inside one launch and defers nothing.
"""
import math

import numpy as np
import pytest

import oracle
import paper_2003_05293_amd as hg
from oracle import sampler
from workload import Grid, OPTICS, spot_cloud

pytestmark = pytest.mark.gpu

SIZES = [(1, 1), (1, 4099), (1, 8192), (4099, 1)]


@pytest.fixture(scope="module", autouse=True)
def gpu():
    import torch
    assert torch.cuda.is_available()
    hg.load()
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("W,H", SIZES[1:])
@pytest.mark.parametrize("N", [1, 16, 256])
@pytest.mark.parametrize("I", [2, 3, 4])
def test_mixed_fields_of_every_iteration(W, H, N, I):
    print("[case] one column, mixed", W, H, N, I, flush=True)
    g, c, seed = Grid(W, H), 0.5, 5
    s = spot_cloud(N, N, g)
    phi, V = hg.cswgs(g, OPTICS, s, I, c, seed, trace=True, precision="mixed")
    w, th = np.ones(N), oracle.theta0(seed, N)
    everything = np.arange(g.M)

    def bar(want, m):
        return 8 * 2.0 ** -11 * (1 / math.sqrt(m) + np.abs(want))

    for j in range(1, I + 1):
        p = sampler.subset(g.M, sampler.ORDER_KEY, j, c) if j < I else everything
        want = oracle.forward(g, OPTICS, s, oracle.backward(g, OPTICS, s, w, th, p), p)
        err = np.abs(V[j - 1] - want)
        print("one column, iteration", j, "err / bar", float((err / bar(want, p.size)).max()))
        assert np.all(err <= bar(want, p.size)), j
        w, th = oracle.update(w, V[j - 1])
    got = oracle.forward(g, OPTICS, s, phi.cpu().numpy().astype(np.float64))
    want = oracle.forward(g, OPTICS, s, oracle.backward(g, OPTICS, s, w, th))
    assert np.all(np.abs(got - want) <= bar(want, g.M))


@pytest.mark.parametrize("W,H", SIZES)
@pytest.mark.parametrize("N", [1, 16, 256])
def test_fp32_equals_chained(W, H, N):
    print("[case] one column, FP32", W, H, N, flush=True)
    g = Grid(W, H)
    s = spot_cloud(N, N, g)
    phi, V = hg.cswgs(g, OPTICS, s, 4, 0.4, 7, trace=True)
    phi_c, V_c = hg.cswgs(g, OPTICS, s, 4, 0.4, 7, trace=True, tune={"chain_passes": 1})
    assert np.array_equal(phi.cpu().numpy(), phi_c.cpu().numpy()) and np.array_equal(V, V_c)
