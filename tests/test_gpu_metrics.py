"""FP64 metrics (matrix-core product over tiles of 64 rows) at the edges of
their tiling: columns beyond the last quad and the last split, rows beyond the
last group, every remainder of 16-spot blocks, and blocks that take their
columns in several chunks.

Bar: e, u and the intensities within 1e-12 of the oracle's on the same Phi.
Each field is a mean of M unit terms whose phases (up to |t| = 500 turns) carry
2 pi |t| 2^-53 = 4e-13 rad at most, independent from term to term, so a field
errs by less than 4e-13 and an intensity (at most 1) by twice that.
"""
import numpy as np
import pytest

import oracle
import paper_2003_05293_amd as hg
from workload import Grid, OPTICS, PUPIL_OPTICS, spot_cloud

pytestmark = pytest.mark.gpu

CASES = [(1, 1, 1), (3, 2, 15), (66, 65, 16), (67, 63, 17), (130, 64, 48), (97, 129, 49),
         (64, 40, 64), (61, 70, 65), (90, 50, 112), (700, 4200, 5)]


@pytest.mark.parametrize("W,H,N", CASES)
@pytest.mark.parametrize("optics", [OPTICS, PUPIL_OPTICS], ids=["uniform", "pupil"])
def test_metrics_tiling_edges(W, H, N, optics):
    import torch
    print("[case] metrics", W, H, N, flush=True)
    g = Grid(W, H)
    s = spot_cloud(N, N, g)
    rng = np.random.Generator(np.random.PCG64(W * H + N))
    phi = rng.uniform(-np.pi, np.pi, g.M).astype(np.float32)
    e, u, inten = hg.metrics(g, optics, s, torch.as_tensor(phi, device="cuda"))
    eo, uo, io = oracle.metrics(g, optics, s, phi.astype(np.float64))
    print("errors", abs(e - eo), abs(u - uo), np.abs(inten - io).max())
    assert abs(e - eo) <= 1e-12 * N and np.abs(inten - io).max() <= 1e-12
    # u = 2 lo / (hi + lo): the error of the intensities over their size
    assert abs(u - uo) <= 4e-12 / io.max()
