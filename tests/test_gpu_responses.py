"""Responses that are not finite (an FP32 job then takes 32 channels with FP32
operands): what they do to their own channel, and that nothing else depends on
the launch a row is in."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle
import paper_2604_23305_amd as g
from tests.gpu_util import new_ctx, rel_err, run_signal
from tests.test_oracle_pins import tiny_scenario
from workloads.scenario import Filters

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [g.PREC_FP32, g.PREC_SPLIT_BF16])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("F,K,P,T,channel", [
    (40, 200, 5, 6300, 37),       # 256 x 128 tiles, 64 x 64 in the windows
    (40, 130, 1, 300, 129),       # 64 x 32 tiles
    (33, 64, 5, 4990, 3),
])
def test_responses_that_are_not_finite(F, K, P, T, channel, bad, prec):
    sc = tiny_scenario(F=F, K=K, P=P, T=T, filt="matrix", uniform=1.02)
    m = sc.spectral.filters.matrix.copy()
    m[5, channel] = bad
    sc.spectral = dataclasses.replace(sc.spectral, filters=Filters("matrix", matrix=m))
    ctx = new_ctx()
    try:
        run, out = run_signal(ctx, sc, precision=prec)
        part = run.alloc(with_p_kid=True, with_sigma=True)
        g.simulate_tod(ctx, [run.signal_job(part, a, min(a + 448, T), precision=prec)
                             for a in range(0, T, 448)])
        torch.cuda.synchronize()
        whole = [getattr(out, n).cpu().numpy() for n in ("tod", "p_kid", "sigma")]
        parts = [getattr(part, n).cpu().numpy() for n in ("tod", "p_kid", "sigma")]
    finally:
        g.free(ctx)
    others = np.arange(K) != channel
    for name, x, y in zip(("tod", "p_kid", "sigma"), whole, parts):
        if name != "sigma":               # a NEP^2 that is NaN counts as 0
            assert not np.isfinite(x[:, channel]).any()
        assert np.isfinite(x[:, others]).all(), name
        assert np.array_equal(x, y, equal_nan=True), name
    m[5, channel] = 0.0
    ref = oracle.tod.simulate(dataclasses.replace(sc, t_total=64), photon_noise=False)
    e = rel_err(whole[1][:, others, :64], ref["p_kid"][:, others])
    assert e.max() <= 1e-6
