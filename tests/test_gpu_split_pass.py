"""The full-grid iteration pass with split FP16 operands at the edges of its
tiling, one pass with (w, theta) held fixed against the FP64 oracle.

Bar, on |V_n - V_n(oracle)|: an operand's two halves leave at most 2^-22 of it,
the dropped product of the two small halves at most 2^-22 of a term, and the
FP32 sums round by 2^-24 per added group, all independent from term to term; a
term of S has magnitude A_n with sum A_n^2 about 1, so S errs by less than
2^-21 of its rms, u by that over |S|, and a mean of M such terms by less than
4 2^-21 / sqrt(M) (the factor covers weak pixels, whose mean-square phase error
grows with the logarithm of M); V_n itself is rounded to FP32 in the sums of a
tile, 2^-23 |V_n|.  N covers one 16-spot block, remainders of the groups of
four blocks, and more spots than the waves bring together at a time (128).
"""
import math

import numpy as np
import pytest

import oracle
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


CASES = [(1, 1, 1), (33, 65, 2), (32, 64, 16), (97, 61, 17), (130, 67, 33), (64, 129, 49),
         (65, 63, 64), (96, 128, 65), (100, 90, 128), (70, 75, 129), (61, 97, 260), (48, 80, 513)]


@pytest.mark.parametrize("W,H,N", CASES)
@pytest.mark.parametrize("optics", [OPTICS, PUPIL_OPTICS], ids=["uniform", "pupil"])
@pytest.mark.parametrize("amp", [1.0, 1e-12, 1e9], ids=["unit", "tiny", "huge"])
def test_step_split(W, H, N, optics, amp):
    print("[case] split pass", W, H, N, amp, flush=True)
    g = Grid(W, H)
    s = spot_cloud(N, N, g)
    s.amp = s.amp * amp  # the pass scales its operands: any amplitude
    rng = np.random.Generator(np.random.PCG64(N))
    w, th = rng.uniform(0.5, 2.0, N), rng.uniform(0, 2 * math.pi, N)
    V = hg.step(g, optics, s, w, th)
    p = oracle.pupil_pixels(g, optics)
    Vo = oracle.forward(g, optics, s, oracle.backward(g, optics, s, w, th, p), p)
    err = np.abs(V - Vo)
    bar = 4 * 2.0 ** -21 / math.sqrt(p.size) + 2.0 ** -23 * np.abs(Vo)
    print("split pass", W, H, N, "err / bar", float((err / bar).max()))
    assert np.all(err <= bar)
