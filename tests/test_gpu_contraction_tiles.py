"""Every tile of the contraction, with one to four live 32-channel tiles in the
last channel group, and rows beyond the FP16 range in the largest one.  Each
case names the tile that it is for, and checks that the launch takes it.

Bars as in the other contraction tests: P_KID and TOD 1e-6, sigma 1e-5 near the
reference; (F + 8) 2^-24 where a source outshines it."""
import numpy as np
import pytest
import torch

import oracle
import paper_2604_23305_amd as g
from paper_2604_23305_amd import binding
from tests.gpu_util import new_ctx, rel_err, report, run_signal
from tests.test_gpu_contraction import _near_reference
from tests.test_oracle_pins import tiny_scenario
from workloads import gen
from workloads.scenario import Source

gpu = pytest.mark.gpu
NAMES = ("tod", "p_kid", "sigma")


def scenario(F, K, P, T):
    sc = tiny_scenario(F=F, K=K, P=7, T=T, filt="matrix", uniform=1.02)
    sc.dphi, sc.dtheta = (x[:P] for x in gen.hex_spaxels(2, 12 * gen.ARCSEC))
    return sc


def tile(prec, P, T, K):
    return binding.contraction_tile(prec, P * (-(-T // 128) * 128), K)


@pytest.mark.parametrize("prec", [g.PREC_FP32, g.PREC_SPLIT_BF16])
def test_the_tile_does_not_grow_with_fewer_rows(prec):
    """The rule, on the host: tiles from 64 x 32 to 256 x 128, never the widest
    for up to 64 channels, and errors for what is no launch."""
    for K in (1, 31, 64, 65, 130, 347, 720):
        seen = [binding.contraction_tile(prec, rows, K) for rows in (128, 2560, 10240, 1 << 20)]
        assert all(t in {(64, 32), (64, 64), (128, 64), (256, 64), (256, 128)} for t in seen)
        assert seen[0][0] == 64 and seen[-1][0] == 256
        assert K > 64 or all(t[1] <= 64 for t in seen)
    for bad in ((2, 128, 1), (prec, 0, 1), (prec, 128, 0)):
        with pytest.raises(g.GtodError):
            binding.contraction_tile(*bad)


@pytest.fixture(scope="module")
def ctx():
    c = new_ctx()
    yield c
    g.free(c)


CASES = [
    # F, K, P, T, tile in FP32 and split
    (40, 130, 5, 5000, (256, 128), (256, 128)),   # last group: one live tile
    (33, 190, 5, 5000, (256, 128), (256, 128)),   # two
    (64, 90, 12, 5000, (256, 128), (256, 128)),   # three, one group
    (40, 224, 5, 5000, (256, 128), (256, 128)),   # three
    (96, 256, 5, 4990, (256, 128), (256, 128)),   # four, a half tile of rows last
    (40, 64, 12, 5000, (256, 64), (256, 64)),
    (40, 31, 12, 5000, (256, 64), (256, 64)),     # one live tile
    (64, 64, 5, 5000, (128, 64), (128, 64)),
    (40, 129, 5, 500, (64, 64), (64, 64)),
    (48, 33, 1, 200, (64, 32), (64, 32)),
]


@gpu
@pytest.mark.parametrize("prec", [g.PREC_FP32, g.PREC_SPLIT_BF16])
@pytest.mark.parametrize("F,K,P,T,t32,tsplit", CASES)
def test_tiles_against_the_oracle_and_small_launches(ctx, F, K, P, T, t32, tsplit, prec):
    assert tile(prec, P, T, K) == (t32 if prec == g.PREC_FP32 else tsplit)
    sc = scenario(F, K, P, T)
    ref = oracle.tod.simulate(sc)
    run, out = run_signal(ctx, sc, precision=prec)
    rows = np.ones((P, 1, T), dtype=bool)
    if prec == g.PREC_SPLIT_BF16:
        rows = _near_reference(sc)[:, None, :]
        assert rows.mean() > 0.5
    for name, tol in (("p_kid", 1e-6), ("tod", 1e-6), ("sigma", 1e-5)):
        e = rel_err(getattr(out, name).cpu().numpy(), ref[name]) * rows
        report(name, e)
        assert e.max() <= tol, name
    part = run.alloc(with_p_kid=True, with_sigma=True)
    g.simulate_tod(ctx, [run.signal_job(part, a, min(a + 256, T), precision=prec)
                         for a in range(0, T, 256)])
    torch.cuda.synchronize()
    for name in NAMES:
        assert torch.equal(getattr(out, name), getattr(part, name)), name


@gpu
@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("F,K,P,T", [
    (40, 130, 5, 5000), (40, 190, 5, 5000), (64, 90, 12, 5000), (40, 256, 5, 5000)])
def test_rows_beyond_half_precision_in_the_largest_tile(ctx, F, K, P, T, accumulate):
    """A source a million times brighter: rows taken again with FP32 operands by
    the 256 x 128 tiles, with one to four live tiles, are as accurate as the
    others and the same bits as in small launches, also when added to a TOD."""
    assert tile(g.PREC_FP32, P, T, K) == (256, 128)
    sc = scenario(F, K, P, T)
    s = sc.source
    sc.source = Source(cube=s.cube * np.float32(1e6), az0=s.az0, daz=s.daz, el0=s.el0,
                       del_=s.del_)
    ref = oracle.tod.simulate(sc, photon_noise=False)
    r = ref["p_kid"].max(axis=1) / ref["p_kid"].max(axis=1).min()
    assert (r > 200).any() and (r < 20).any()
    run = g.ScenarioRun(ctx, sc)
    base = torch.randn((sc.n_pix, K, T), device="cuda",
                       generator=torch.Generator("cuda").manual_seed(K)) * 1e-13
    got = []
    for step in (T, 256):
        out = run.alloc(with_p_kid=True, with_sigma=True)
        out.tod.copy_(base)
        g.simulate_tod(ctx, [run.signal_job(out, a, min(a + step, T), photon_noise=False,
                                            accumulate=accumulate)
                             for a in range(0, T, step)])
        torch.cuda.synchronize()
        got.append(out)
    for name in ("p_kid", "sigma"):
        e = rel_err(getattr(got[0], name).cpu().numpy(), ref[name])
        report(name, e)
        assert e.max() <= (F + 8) * 2.0 ** -24, name
    want = base + got[0].p_kid if accumulate else got[0].p_kid
    assert torch.equal(got[0].tod, want)
    for name in NAMES:
        assert torch.equal(getattr(got[0], name), getattr(got[1], name)), name
