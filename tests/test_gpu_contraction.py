"""Tile shapes of the contraction and rows beyond its FP16 range.

Against the FP64 oracle: P_KID and the TOD within 1e-6 relative and sigma
within 1e-5 while the spectra stay near the reference (the bars of the
parity tests); F + 8 FP32 roundings, (F + 8) 2^-24, where a source outshines
it, since the sums are then of terms of one sign without the reference part.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2604_23305_amd as g
from tests.gpu_util import new_ctx, rel_err, report, run_signal
from tests.test_oracle_pins import tiny_scenario
from workloads.scenario import Source

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = new_ctx()
    yield c
    g.free(c)


def _near_reference(sc):
    """[P][T]: rows whose every bin deviates from the reference spectrum by
    at most P / 8, the range the split path's bars are stated for."""
    spec = sc.spectral
    eta_z, _ = oracle.tod.lut_transmission(spec, np.array([spec.ref_pwv_mm]))
    pref = oracle.tod.cascade(sc, eta_z ** (1.0 / np.sin(spec.ref_el_rad)),
                              None)[0]
    near = np.zeros((sc.n_pix, sc.t_total), dtype=bool)
    for p in range(sc.n_pix):
        geo = oracle.tod.row_geometry(sc, p, np.arange(sc.t_total))
        ez, _ = oracle.tod.lut_transmission(spec, geo["pwv"])
        P = oracle.tod.cascade(sc, ez ** geo["csc"][:, None],
                               oracle.tod.source_power(sc.source, geo["az"],
                                                       geo["el"]))
        near[p] = (np.abs(P - pref) <= P / 8).all(axis=1)
    return near


@pytest.mark.parametrize("prec", [g.PREC_FP32, g.PREC_SPLIT_BF16])
@pytest.mark.parametrize("F,K,P,T", [
    (33, 130, 2, 6300),    # 256 x 128 tiles, a last group of one 32-tile
    (40, 90, 5, 4990),     # three live 32-tiles, a last half tile of rows
    (64, 64, 5, 4990),     # 256 x 64 tiles
    (96, 31, 5, 4990),     # the same with one live 32-tile
    (40, 129, 5, 500),     # 64 x 64 tiles
    (40, 129, 1, 65),      # 64 x 32 tiles, the last of padding rows
    (48, 33, 1, 200),      # the same, both halves of a response group
    (200, 64, 3, 63),
])
def test_tile_shapes_match_oracle_and_each_other(ctx, F, K, P, T, prec):
    """Every tile shape against the oracle; the same rows computed in
    windows of 448 samples, which take the small shape, bit for bit."""
    sc = tiny_scenario(F=F, K=K, P=P, T=T, filt="matrix")
    ref = oracle.tod.simulate(sc)
    run, out = run_signal(ctx, sc, precision=prec)
    rows = np.ones((P, 1, T), dtype=bool)
    if prec == g.PREC_SPLIT_BF16:
        rows = _near_reference(sc)[:, None, :]
        assert rows.mean() > 0.01
    for name, tol in (("p_kid", 1e-6), ("tod", 1e-6), ("sigma", 1e-5)):
        e = rel_err(getattr(out, name).cpu().numpy(), ref[name]) * rows
        report(name, e)
        assert e.max() <= tol, name
    part = run.alloc(with_p_kid=True, with_sigma=True)
    g.simulate_tod(ctx, [run.signal_job(part, a, min(a + 448, T), precision=prec)
                         for a in range(0, T, 448)])
    torch.cuda.synchronize()
    for name in ("tod", "p_kid", "sigma"):
        assert torch.equal(getattr(out, name), getattr(part, name)), name


@pytest.mark.parametrize("F,K,P,T", [(40, 70, 7, 600), (40, 130, 7, 1900)])
def test_rows_beyond_the_half_precision_range(ctx, F, K, P, T):
    """A source a million times brighter than the sky calls for more than
    the FP16 halves hold in some rows; those are as accurate as the others.
    With a huge spectral line in place of it they come out infinite, and the
    other rows bit for bit as without it."""
    sc = tiny_scenario(F=F, K=K, P=P, T=T, filt="matrix")
    s = sc.source
    sc.source = Source(cube=s.cube * np.float32(1e6), az0=s.az0, daz=s.daz,
                       el0=s.el0, del_=s.del_)
    ref = oracle.tod.simulate(sc)
    faint = tiny_scenario(F=F, K=K, P=P, T=T, filt="matrix")
    dark = oracle.tod.simulate(faint, photon_noise=False)
    ratio = ref["p_kid"].max(axis=1) / dark["p_kid"].max(axis=1)
    assert (ratio > 200).any() and (ratio < 20).any()
    _, out = run_signal(ctx, sc)
    for name in ("p_kid", "tod", "sigma"):
        e = rel_err(getattr(out, name).cpu().numpy(), ref[name])
        report(name, e)
        assert e.max() <= (F + 8) * 2.0 ** -24, name

    _, base = run_signal(ctx, faint)
    cube = s.cube.copy()
    cube[4, 4, 7] = np.inf
    faint.source = Source(cube=cube, az0=s.az0, daz=s.daz, el0=s.el0, del_=s.del_)
    _, out = run_signal(ctx, faint)
    got, was = out.tod.cpu().numpy(), base.tod.cpu().numpy()
    hit = ~np.isfinite(got)
    assert hit.any() and not hit.all()
    assert np.array_equal(hit, np.broadcast_to(hit[:, :1], hit.shape))
    assert np.isposinf(out.p_kid.cpu().numpy()[hit]).any()
    assert np.array_equal(got[~hit], was[~hit])
