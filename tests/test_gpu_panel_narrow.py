"""Panels of up to 512 bins, whose rows are spread over the waves of a workgroup:
one wave a row up to 256 bins, two up to 512, four beyond.  In their own order
and sorted, in launches of 2, 4, 8 and 32 rows per workgroup."""
import numpy as np
import pytest
import torch

import oracle
import paper_2604_23305_amd as g
from tests.gpu_util import new_ctx, rel_err
from tests.test_oracle_pins import tiny_scenario
from workloads.scenario import Scan
from workloads import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("F", [1, 64, 255, 256, 257, 500, 512, 513])
@pytest.mark.parametrize("scan", ["daisy", "traj"])
def test_narrow_panels(F, scan):
    P, K, T = 7, 2, 4700
    sc = tiny_scenario(F=F, K=K, P=P, T=T, filt="matrix")
    if scan == "traj":
        t = np.arange(T) / sc.f_sample_hz
        traj = 40 * gen.ARCSEC * np.stack([np.cos(9 * t), np.sin(7 * t)], axis=1)
        sc.scan = Scan("traj", theta0=sc.scan.theta0, traj=np.ascontiguousarray(traj))
    got = []
    # sorted in one launch; windows of 896, 512, 128 and 64 samples in order
    for step in (T, 896, 512, 128, 64):
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
    x, cx = got[0]
    for y, cy in got[1:]:
        for name in ("tod", "p_kid", "sigma", "pwv"):
            assert torch.equal(getattr(x, name), getattr(y, name)), name
        assert cx == cy
    ref = oracle.tod.simulate(sc)
    e = rel_err(x.p_kid.cpu().numpy(), ref["p_kid"])
    assert e.max() <= max(1e-6, (F + 8) * 2.0 ** -24)
