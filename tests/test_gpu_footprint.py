"""Screen smoothing at the edges of its kernel's ranges, against the oracle:
1e-12 relative (FP64 on both sides, sums of at most 4225 positive terms)."""
import numpy as np
import pytest
import torch

import paper_2604_23305_amd as g
from oracle import inputs as oin
from tests.gpu_util import new_ctx

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = new_ctx(workspace_bytes=64 << 20)
    yield c
    g.free(c)


@pytest.mark.parametrize("ny,nx,dx,dy,r", [
    (1, 1, 0.2, 0.2, 5.0),        # one cell
    (3, 257, 1.0, 1.0, 0.5),      # footprint of one cell
    (5, 256, 0.5, 0.9, 1.0),      # cells on the rim are outside
    (17, 255, 0.25, 0.25, 2.1),   # 8 rows: the largest of its kernel
    (33, 300, 0.3, 0.25, 2.3),    # 9 rows
    (40, 513, 0.2, 0.2, 3.3),     # 16
    (70, 70, 0.1, 0.2, 3.21),     # 32 columns
    (1100, 40, 0.2, 0.2, 5.1),    # 25 rows, several strips
    (90, 300, 0.2, 0.2, 5.3),     # 26
    (90, 300, 0.3, 0.1, 3.25),    # 32 rows, the largest
])
@pytest.mark.parametrize("taper", [-10.0, 6.0])
def test_footprint_sizes_match_oracle(ctx, ny, nx, dx, dy, r, taper):
    scr = np.random.default_rng([ny, nx]).uniform(0.5, 1.5, (ny, nx))
    got = g.convolve_screen(ctx, torch.from_numpy(scr).cuda(), dx, dy, r,
                            taper).cpu().numpy()
    ref = oin.convolve_screen(scr, dx, dy, r, taper)
    assert (np.abs(got - ref) / np.abs(ref)).max() <= 1e-12


def test_a_nan_cell_reaches_its_footprint_only(ctx):
    scr = np.ones((80, 300))
    scr[40, 150] = np.nan
    got = g.convolve_screen(ctx, torch.from_numpy(scr).cuda(), 0.2, 0.2, 3.0,
                            -10.0).cpu().numpy()
    ref = oin.convolve_screen(scr, 0.2, 0.2, 3.0, -10.0)
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.isnan(got).sum() > 600
