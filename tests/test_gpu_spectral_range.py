"""Setups whose reference power spans many decades over the bins, or vanishes.

P_KID within 1e-6 of the oracle and sigma within 1e-5, the bars of the parity
tests, channel by channel: a channel whose response lies in the faintest bins
alone is as accurate as the others.  Without any reference power every sum is
of terms of one sign and bounded by the rounding of F of them: (F + 8) 2^-24.
"""
import dataclasses

import numpy as np
import pytest

import oracle
import paper_2604_23305_amd as g
from tests.gpu_util import new_ctx, rel_err, report, run_signal
from tests.test_oracle_pins import tiny_scenario
from workloads.scenario import Filters, Stage

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,uniform", [
    (g.PREC_FP32, 1.02), (g.PREC_FP32, None),
    (g.PREC_SPLIT_BF16, 1.02),           # near the reference, where its bars hold
])
@pytest.mark.parametrize("decades", [3, 9, 15])
def test_channels_in_faint_bins(prec, uniform, decades):
    """A cold filter in front of the detectors passes less and less from bin
    to bin; half of the channels see one bin each, the others all."""
    F = 64
    sc = tiny_scenario(F=F, K=2 * F, P=2, T=200, filt="matrix", uniform=uniform)
    eta = 10.0 ** (-decades * np.arange(F) / (F - 1))
    m = np.concatenate([0.3 * np.eye(F), sc.spectral.filters.matrix[:, F:]], axis=1)
    sc.spectral = dataclasses.replace(sc.spectral, filters=Filters("matrix", matrix=m),
                                      stages=[Stage("reflect", eta=eta, t_K=0.05)])
    with np.errstate(over="ignore"):
        ref = oracle.tod.simulate(sc)
    c = new_ctx()
    try:
        _, out = run_signal(c, sc, precision=prec)
        if prec == g.PREC_SPLIT_BF16:
            assert g.counters(c)[3] == 0
        for name, tol in (("p_kid", 1e-6), ("sigma", 1e-5)):
            e = rel_err(getattr(out, name).cpu().numpy(), ref[name])
            report(name, e)
            assert e.max() <= tol, name
    finally:
        g.free(c)


@pytest.mark.parametrize("prec", [g.PREC_FP32, g.PREC_SPLIT_BF16])
@pytest.mark.parametrize("temperature", [1e-3, 0.2])
def test_a_sky_that_emits_nothing(prec, temperature):
    """Sky and background too cold to emit in these bins: all power is the
    source's, at a reference spectrum of (1 mK) nothing at all or (0.2 K) less
    than FP32 holds in some bins."""
    F, K, T = 40, 7, 300
    sc = tiny_scenario(F=F, K=K, P=2, T=T, filt="matrix")
    sc.spectral = dataclasses.replace(sc.spectral, t_atm_K=temperature, stages=[])
    sc.t_cmb_K = temperature
    with np.errstate(over="ignore"):
        ref = oracle.tod.simulate(sc, photon_noise=False)
    c = new_ctx(t_cmb_K=temperature)
    try:
        _, out = run_signal(c, sc, precision=prec, photon_noise=False)
        for name in ("p_kid", "tod"):
            got, want = getattr(out, name).cpu().numpy().astype(float), ref[name]
            lit = want > 1e-3 * want.max()     # rows inside the source grid
            assert lit.any()
            e = np.abs(got - want)[lit] / want[lit]
            report(name, e)
            tol = (F + 8) * 2.0 ** (-24 if prec == g.PREC_FP32 else -16)
            assert e.max() <= tol, name
    finally:
        g.free(c)
