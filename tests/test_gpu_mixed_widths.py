"""Passes of up to 256 and of more spots in one round: joined in one launch or,
beyond 20480 blocks of narrow passes, in two.  Either way every hologram has the
bits that it has alone, whatever the order of the jobs.
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


# narrow tiles in the round: 2 x 400, 7 x 2925 = 20475, 8 x 2925 = 23400
@pytest.mark.parametrize("W,H,c,narrow", [(320, 160, 0.5, 2), (720, 520, 0.5, 7), (720, 520, 0.5, 8)])
@pytest.mark.parametrize("wide", [[257], [300, 512]])
def test_narrow_beside_wide(W, H, c, narrow, wide):
    import torch
    print("[case] mixed widths", W, H, narrow, wide, flush=True)
    g, I = Grid(W, H), 4
    counts = [20 + 33 * k % 237 for k in range(narrow)]
    counts = counts[:narrow // 2] + wide + counts[narrow // 2:]
    spots = [spot_cloud(k, n, g) for k, n in enumerate(counts)]
    jobs = [hg.DeviceJob.from_spots(g, OPTICS, s, I, c, k) for k, s in enumerate(spots)]
    hg.cswgs_batch(jobs)
    torch.cuda.synchronize()
    for k, (s, job) in enumerate(zip(spots, jobs)):
        ref = hg.cswgs(g, OPTICS, s, I, c, k)
        assert np.array_equal(job.phi.cpu().numpy(), ref.cpu().numpy()), counts[k]
