"""Footprints of up to 16 cells on either side of the line between the kernel
that sums cell by cell in tiles and the one that works down strips: screens of
every tile remainder, narrow and tall ones, oblong cells.  Both against the
oracle's weighted mean, FP64 with its cells summed in another order: (number of
cells + 8) 2^-53 relative, all terms being positive."""
import numpy as np
import pytest
import torch

import paper_2604_23305_amd as g
from oracle import inputs as oin
from tests.gpu_util import new_ctx

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = new_ctx(workspace_bytes=1 << 20)
    yield c
    g.free(c)


def mean(scr, dx, dy, r_tel, t_edge):
    rx, ry = int(r_tel // dx), int(r_tel // dy)
    y, x = np.mgrid[-ry:ry + 1, -rx:rx + 1]
    r = np.hypot(x * dx, y * dy)
    w = np.where(r < r_tel, 10.0 ** (t_edge * (r / r_tel) ** 2 / 20.0), 0.0)
    w /= w.sum()
    pad = np.pad(scr, ((ry, ry), (rx, rx)), mode="edge")
    out = np.zeros(scr.shape)
    for j in range(2 * ry + 1):
        for i in range(2 * rx + 1):
            out += w[j, i] * pad[j:j + scr.shape[0], i:i + scr.shape[1]]
    return out, w.size


@pytest.mark.parametrize("ny,nx", [(1, 1), (31, 63), (32, 64), (33, 65), (70, 300),
                                   (3000, 64), (2, 700)])
@pytest.mark.parametrize("n", [0, 1, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 16])
@pytest.mark.parametrize("aspect", [1.0, 0.6])
def test_tiles_and_strips(ctx, ny, nx, n, aspect):
    scr = np.random.default_rng([ny, nx, n]).uniform(0.5, 2.0, (ny, nx))
    dx, dy = 5.0 / (n + 0.5), 5.0 / (n + 0.5) / aspect
    got = g.convolve_screen(ctx, torch.from_numpy(scr).cuda(), dx, dy, 5.0, -10.0)
    ref, cells = mean(scr, dx, dy, 5.0, -10.0)
    assert (np.abs(got.cpu().numpy() - ref) <= (cells + 8) * 2.0 ** -53 * 2 * ref).all()


@pytest.mark.parametrize("n", [2, 6, 9])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_a_bad_cell_reaches_its_footprint_only(ctx, n, bad):
    scr = np.ones((60, 200))
    scr[30, 100] = bad
    d = 5.0 / (n + 0.5)
    got = g.convolve_screen(ctx, torch.from_numpy(scr).cuda(), d, d, 5.0, -10.0).cpu().numpy()
    y, x = np.mgrid[:60, :200]
    inside = np.hypot((x - 100) * d, (y - 30) * d) < 5.0
    assert not np.isfinite(got[inside]).any()
    assert np.abs(got[~inside] - 1.0).max() <= 1e-13
