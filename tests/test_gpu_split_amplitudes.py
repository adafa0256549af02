"""The full-grid iteration pass on split FP16 operands with target amplitudes
spread over decades within one hologram: one pass with (w, theta) held fixed,
every spot's field against the FP64 oracle and against the per-pixel FP32 form
(direct=True).

Bar, on |V_n - V_n(oracle)|, with sum A_n^2 = 1:
- errors of S that are independent from pixel to pixel, as for equal
  amplitudes, 4 2^-21 / sqrt(M): S errs by a fraction of its rms, whatever the
  amplitude of spot n;
- errors of an operand that are a function of the row or the column alone (a
  table entry's or a coefficient's rounding, 2^-23 of a spot's amplitude): their
  mean over the W or H values is below 4 2^-23 / sqrt(W or H), and they reach
  spot n through the overlap of the two spots' factors along the other axis,
  o_mn = |mean conj(G_n) G_m|, weighted with A_m;
- roundings in line with spot n's own field, 2^-21 |V_n| (at most eight of 2^-24).
Nothing in it grows with the ratio of the amplitudes: a unit that drops the low
bits of a weak spot's terms beside a strong one's (2^-24 of the strong amplitude,
always towards zero) misses it, since those errors add up over the pixels.
The per-pixel form forms phases of up to 2^7 turns in FP32 and takes sines to
2^-20: 4 2^-14 / sqrt(M) + 2^-18 |V_n| more.
"""
import math

import numpy as np
import pytest

import oracle
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


def factors(s, n, lat, pitch_mm):
    """e^{i phi} of every spot along one axis, (n, N)."""
    off = (np.arange(n) - 0.5 * (n - 1)) * pitch_mm
    lf = OPTICS.lambda_mm * OPTICS.focal_mm
    t = lat[None] * off[:, None] / lf + s.z_mm[None] * (off[:, None] ** 2) / (lf * OPTICS.focal_mm)
    return np.exp(2j * np.pi * (t - np.rint(t)))


def check(g, s, w, th):
    s.amp = s.amp / np.linalg.norm(w * s.amp)
    A = w * s.amp
    V = hg.step(g, OPTICS, s, w, th)
    V_direct = hg.step(g, OPTICS, s, w, th, direct=True)
    Vo = oracle.forward(g, OPTICS, s, oracle.backward(g, OPTICS, s, w, th))
    F, G = factors(s, g.W, s.x_mm, g.pitch_mm), factors(s, g.H, s.y_mm, g.pitch_mm)
    ox = np.sqrt((np.abs(F.conj().T @ F / g.W) ** 2) @ A ** 2)
    oy = np.sqrt((np.abs(G.conj().T @ G / g.H) ** 2) @ A ** 2)
    bar = (4 * 2.0 ** -21 / math.sqrt(g.M) +
           4 * 2.0 ** -23 * (oy / math.sqrt(g.W) + ox / math.sqrt(g.H)) + 2.0 ** -21 * np.abs(Vo))
    err = np.abs(V - Vo)
    print("err / bar", float((err / bar).max()), "|V|", float(np.abs(Vo).min()),
          float(np.abs(Vo).max()))
    assert np.all(err <= bar)
    bar_d = bar + 4 * 2.0 ** -14 / math.sqrt(g.M) + 2.0 ** -18 * np.abs(Vo)
    assert np.all(np.abs(V - V_direct) <= bar_d)


@pytest.mark.parametrize("W,H", [(640, 480), (333, 259)])
@pytest.mark.parametrize("N", [5, 17, 60])
@pytest.mark.parametrize("decades", [1, 3, 5])
def test_spread_amplitudes(W, H, N, decades):
    print("[case] split pass, spread amplitudes", W, H, N, decades, flush=True)
    g = Grid(W, H)
    s = spot_cloud(N, N, g)
    rng = np.random.Generator(np.random.PCG64(10 * N + decades))
    s.amp = 10.0 ** -rng.uniform(0, decades, N)
    check(g, s, rng.uniform(0.7, 1.4, N), rng.uniform(0, 2 * math.pi, N))
