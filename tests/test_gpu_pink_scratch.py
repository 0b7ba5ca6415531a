"""1/f series whose scratch is the whole 1/f area of the workspace."""
import numpy as np
import pytest
import torch

import paper_2604_23305_amd as g
from tests.gpu_util import new_ctx
from tests.test_oracle_pins import tiny_scenario

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,ws", [(1 << 18, 4 << 20), (1 << 14, 4096)])
def test_series_as_long_as_the_workspace(T, ws):
    """A quarter of the workspace, or 64 KiB, holds one series at a time of 4
    bytes a sample; the next length is refused."""
    sc = tiny_scenario(F=16, K=3, P=1, T=T, source=False)
    sc.pink_alpha = np.array([1.0, 0.5, 2.0])
    got = []
    for w in (ws, 64 << 20):
        ctx = new_ctx(workspace_bytes=w)
        try:
            run = g.ScenarioRun(ctx, sc)
            x = torch.zeros((1, 3, T), device="cuda")
            g.simulate_tod(ctx, [run.pink_job(x, accumulate=False)])
            torch.cuda.synchronize()
            got.append(x.cpu())
            if w == ws:
                j = run.pink_job(torch.zeros((1, 3, 2 * T), device="cuda"))
                j.t_total = 2 * T
                with pytest.raises(g.GtodError):
                    g.simulate_tod(ctx, [j])
        finally:
            g.free(ctx)
    assert torch.isfinite(got[0]).all() and torch.equal(got[0], got[1])
