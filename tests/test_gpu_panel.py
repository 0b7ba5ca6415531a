"""The two orders the panel takes its rows in.

A job with a source and at least 12288 rows sorts them by source cell; the
same rows in smaller windows come in their own order.  The arithmetic of a
row is the same, so the outputs agree bit for bit, and the range counters
count the same events.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2604_23305_amd as g
from tests.gpu_util import new_ctx, rel_err
from tests.test_oracle_pins import tiny_scenario
from workloads.scenario import Source

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("F,pitch,offset", [
    (3, 3, 0),          # fewer bins than a lane takes
    (5, 8, 1),          # a lane across the end; rows of odd alignment
    (30, 31, 3),
    (1030, 1030, 0),    # two passes of bins, the second of two lanes
    (1026, 1029, 2),
])
def test_sorted_rows_match_rows_in_order(F, pitch, offset):
    P, K, T = 7, 2, 1800
    sc = tiny_scenario(F=F, K=K, P=P, T=T, filt="matrix")
    s = sc.source
    cube = s.cube * np.float32(2e4)        # some elements beyond P / 8
    sc.source = Source(cube=cube, az0=s.az0, daz=s.daz, el0=s.el0, del_=s.del_)
    # the same cube at a pitch and an offset of its own, NaN between rows
    buf = torch.full((s.n_el * s.n_az * pitch + 4,), float("nan"), device="cuda")
    rows = buf[offset:offset + s.n_el * s.n_az * pitch].view(s.n_el, s.n_az, pitch)
    rows[:, :, :F] = torch.from_numpy(cube).cuda()
    # bring the last row to the end of its allocation
    last = buf[: offset + (s.n_el * s.n_az - 1) * pitch + F].clone()

    def job(run, out, a, b):
        j = run.signal_job(out, a, b)
        j.cube, j.cube_ld = last.data_ptr() + 4 * offset, pitch
        return j

    got = []
    for step in (T, 896):
        ctx = new_ctx()
        try:
            run = g.ScenarioRun(ctx, sc)
            out = run.alloc(with_p_kid=True, with_sigma=True, with_pwv=True)
            g.simulate_tod(ctx, [job(run, out, a, min(a + step, T))
                                 for a in range(0, T, step)])
            torch.cuda.synchronize()
            got.append((out, g.counters(ctx)))
        finally:
            g.free(ctx)
    (x, cx), (y, cy) = got
    for name in ("tod", "p_kid", "sigma", "pwv"):
        assert torch.equal(getattr(x, name), getattr(y, name)), name
    assert cx == cy and cx[3] > 0
    ref = oracle.tod.simulate(sc)
    # far from the reference the bound is that of an FP32 sum of F terms
    e = rel_err(x.p_kid.cpu().numpy(), ref["p_kid"])
    assert e.max() <= max(1e-6, (F + 8) * 2.0 ** -24)


@pytest.mark.parametrize("T,window", [
    (4680, 1792), (4700, 1792), (9340, 1792), (9380, 1792), (18720, 1792),
    (700, 512), (500, 128),   # 4 and 2 rows per workgroup in the windows
])
def test_every_spread_of_the_rows_gives_the_same_outputs(T, window):
    """7 pixels on either side of 32768, 65536 and 131072 panel rows, and
    below 4096 and 1024, two passes of bins, in one window and in several."""
    sc = tiny_scenario(F=1030, K=2, P=7, T=T, filt="matrix")
    got = []
    for step in (T, window):
        ctx = new_ctx()
        try:
            run = g.ScenarioRun(ctx, sc)
            out = run.alloc(with_p_kid=True, with_sigma=True, with_pwv=True)
            g.simulate_tod(ctx, [run.signal_job(out, a, min(a + step, T))
                                 for a in range(0, T, step)])
            torch.cuda.synchronize()
            got.append((out, g.counters(ctx)))
        finally:
            g.free(ctx)
    (x, cx), (y, cy) = got
    for name in ("tod", "p_kid", "sigma", "pwv"):
        assert torch.equal(getattr(x, name), getattr(y, name)), name
    assert cx == cy
