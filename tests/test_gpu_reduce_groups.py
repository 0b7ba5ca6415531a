"""Reductions whose workspace holds fewer channels than there are: the scratch
of the sorted gridding is taken where at least 8 channels (or all) fit beside
it, and left out where not.  Same oracle and bars as the other
reduction tests; T* has the same bits on every route."""
import numpy as np
import pytest
import torch

import paper_2604_23305_amd as g
from tests.gpu_util import new_ctx
from tests.test_gpu_reduce import check_tstar
from tests.test_gpu_reduce_paths import ARC, check_maps, fields, scenario

pytestmark = pytest.mark.gpu


def up(x):
    return -(-x // 256) * 256


@pytest.mark.parametrize("T,K,n", [(6200, 19, 9), (8192, 9, 21), (12289, 17, 9)])
def test_groups_of_every_size(T, K, n):
    P = 7
    sc = scenario("daisy", T, K)
    t_b, d = fields(sc, T, T)
    tiles = -(-T // 2048)
    extra = (2 * up(P * T * 8) + P * tiles * 2048 * 6 + up(P * tiles * 4) + 2048)
    per = up(T * 8) + P * n * n * 16
    fixed = up(T * 16) + up(K * 8) + 256
    got = []
    # beside the scratch: nothing, one channel, 7, 8, 15, 16, all but one, all
    for beside in (-1, 1, 7, 8, 15, 16, K - 1, K):
        panel = fixed + 256 + (extra + beside * per if beside > 0 else 3 * per)
        ctx = new_ctx(workspace_bytes=(panel + 64) * 4 // 3 + 512)
        try:
            run = g.ScenarioRun(ctx, sc)
            ts = torch.zeros_like(d)
            mp = torch.zeros((K, n, n), dtype=torch.float64, device="cuda")
            wt = torch.zeros_like(mp)
            g.reduce(ctx, run.reduce_desc(d, 30 * ARC, t_star=ts, maps=(mp, wt), map_n=n,
                                          map_half_rad=150 * ARC, pwv_mean_mm=1.1, T=T))
            ts = ts.cpu().numpy()
            if not got:
                ref, scale = check_tstar(sc, ts, t_b, 1.1, 30 * ARC)
            check_maps(sc, ref, scale, mp, wt, 150 * ARC, n)
            got.append(ts)
        finally:
            g.free(ctx)
    assert all(np.array_equal(got[0], x) for x in got[1:])
