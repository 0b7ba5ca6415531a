"""Rows of a user trajectory at elevations without an airmass.

The spectral power of such a row is the formula's, evaluated in FP32: xi =
-expm1(-tau / sin(el)), which for a negative sine falls without bound and
overflows to -inf from tau / |sin(el)| = 88.8 on.  With a response that sees
one bin per channel P_KID shows it bin by bin."""
import dataclasses

import numpy as np
import pytest

import oracle
import paper_2604_23305_amd as g
from tests.gpu_util import new_ctx, run_signal
from tests.test_oracle_pins import tiny_scenario
from workloads.scenario import Filters, Scan

pytestmark = pytest.mark.gpu
T0 = np.pi / 3


def scenario(F, elevations):
    """One channel per bin, no source, a stare-like trajectory that visits the
    elevations one after another."""
    T = len(elevations)
    sc = tiny_scenario(F=F, K=F, P=1, T=T, filt="matrix", source=False, uniform=1.0)
    sc.dtheta = np.zeros(1)
    traj = np.zeros((T, 2))
    traj[:, 1] = np.asarray(elevations) - T0
    sc.scan = Scan("traj", theta0=T0, traj=traj)
    sc.spectral = dataclasses.replace(sc.spectral, filters=Filters("matrix", matrix=np.eye(F)))
    return sc


@pytest.mark.parametrize("F", [16, 40, 1100])
@pytest.mark.parametrize("prec", [g.PREC_FP32, g.PREC_SPLIT_BF16])
def test_below_the_horizon(F, prec):
    """Elevations from just below 0 to -pi/2 and beyond pi: opaque bins come out
    infinite or NaN, never like an ordinary opaque sky."""
    el = np.concatenate([-np.geomspace(1e-5, np.pi / 2, 60), [T0], np.pi + np.linspace(0.01, 0.5, 9)])
    sc = scenario(F, el)
    c = new_ctx()
    try:
        _, out = run_signal(c, sc, precision=prec, photon_noise=False)
        got = out.p_kid.cpu().numpy()[0].astype(np.float64)       # [bin][row]
        assert g.counters(c)[2] == len(el) - 1
    finally:
        g.free(c)
    with np.errstate(all="ignore"):
        ref = oracle.tod.simulate(sc, photon_noise=False)["p_kid"][0]
        ez, _ = oracle.tod.lut_transmission(sc.spectral, np.ones(1))
        x = -np.log(ez[0])[:, None] / np.sin(el)[None, :]
    # FP32 rounds x = tau / sin(el) by a few 2^-24 of itself, P by e^-x times that
    tame = (x > -1.0) & (x < 0)
    assert tame.any()
    assert (np.abs(got - ref)[tame] <= 1e-4 * np.abs(ref)[tame]).all()
    lost = x < -89.0
    assert lost.any() and not np.isfinite(got[lost]).any()
    up = np.sin(el) > 0
    assert (np.abs(got - ref)[:, up] <= 1e-6 * ref[:, up]).all()


@pytest.mark.parametrize("F", [33, 40, 64])
@pytest.mark.parametrize("prec", [g.PREC_FP32, g.PREC_SPLIT_BF16])
def test_on_the_horizon(F, prec):
    """Elevation 0 exactly: the airmass is infinite and every bin opaque.  The
    padding of the frequency axis, which has no optical depth, adds nothing.
    Single bins, off by a few roundings of the operands: 2^-20, 16-bit ones
    2^-13."""
    sc = scenario(F, np.array([T0, 0.0, T0]))
    c = new_ctx()
    try:
        _, out = run_signal(c, sc, precision=prec, photon_noise=False)
        got = out.p_kid.cpu().numpy()[0].astype(np.float64)
    finally:
        g.free(c)
    with np.errstate(all="ignore"):
        ref = oracle.tod.simulate(sc, photon_noise=False)["p_kid"][0]
    assert np.isfinite(ref).all()
    tol = 2.0 ** (-20 if prec == g.PREC_FP32 else -13)
    assert (np.abs(got - ref) <= tol * ref).all()
