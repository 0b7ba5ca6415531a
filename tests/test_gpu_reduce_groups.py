"""The routes of a reduction: by its length, its channels and the workspace.

Reductions whose workspace holds fewer channels than there are: the scratch
of the sorted gridding is taken where at least 8 channels (or all) fit beside
it, and left out where not.  Same oracle and bars as the other
reduction tests; T* has the same bits on every route."""
import numpy as np
import pytest
import torch

import paper_2604_23305_amd as g
from oracle import reduce as orr
from tests.gpu_util import new_ctx
from tests.test_gpu_reduce import check_tstar
from tests.test_gpu_reduce_paths import ARC, fields, scenario

pytestmark = pytest.mark.gpu


def check_maps(sc, ref, scale, mp, wt, half, n):
    """A variance formed in FP64 as (S2 - S1^2 / m) / (m - 1), of T* with errors
    up to e = 16 roundings of the terms it is made of, is off by at most dvar:
    cells whose few samples nearly coincide are allowed that much in their
    spaxel's weight m / var, and whether they count at all where it reaches
    var / 2."""
    eps = 2.0 ** -52
    count, mean, var = orr.spaxel_maps(sc, ref, half, n)
    m_o, w_o = orr.combine(count, mean, var)
    m_g, w_g = (x.cpu().numpy().reshape(sc.K, -1) for x in (mp, wt))
    m = np.maximum(count, 2.0)[:, None, :]
    e = 16 * eps * scale.max()
    spread = (ref.max(axis=2) - ref.min(axis=2))[:, :, None] ** 2
    v = np.where(np.isfinite(var), var, np.inf)
    dvar = 4 * e * np.sqrt(v * m / (m - 1)) + 4 * e * e + 8 * eps * spread * m / (m - 1)
    dvar = np.where(np.isfinite(var), dvar, 0.0)
    sure = (np.isnan(var) | (dvar < v / 2)).all(axis=0)
    assert sure.mean() > 0.9
    w = np.where(np.isfinite(var), m / v, 0.0)
    dw = np.where(sure, 2 * w * dvar / v, 0.0)
    live = (w_o > 0) & sure
    assert live.any()
    assert np.array_equal((w_g > 0)[sure], (w_o > 0)[sure])
    assert np.array_equal(np.isnan(m_g)[sure], np.isnan(m_o)[sure])
    assert (np.abs(w_g - w_o)[live] <= (dw.sum(axis=0) + 1e-10 * w_o)[live]).all()
    off = np.where(dw > 0, dw * np.abs(np.nan_to_num(mean) - np.nan_to_num(m_o)), 0.0)
    off = 2 * off.sum(axis=0) / np.where(w_o > 0, w_o, 1.0)
    assert (np.abs(m_g - m_o)[live] <= (off + 1e-9 * scale.max())[live]).all()


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


@pytest.mark.parametrize("scan,half", [("stare", 150 * ARC), ("daisy", 150 * ARC),
                                       ("wide", 0.08)])
@pytest.mark.parametrize("T,K,n,pad", [
    (4799, 4, 15, 1), (4800, 4, 15, 0),        # the first sorted length
    (6143, 5, 31, 0), (6145, 7, 48, 3),        # a tile of one sample; an odd channel
    (7999, 3, 21, 1), (8000, 2, 21, 2), (15999, 1, 9, 0), (16000, 1, 9, 1),
    (1500, 160, 48, 0),                        # more blocks than the card holds
])
def test_sorted_and_unsorted_maps(scan, half, T, K, n, pad):
    sc = scenario(scan, T, K)
    t_b, d = fields(sc, T, T + pad)
    ctx = new_ctx(workspace_bytes=64 << 20)
    try:
        run = g.ScenarioRun(ctx, sc)
        ts = torch.zeros_like(d)
        mp = torch.zeros((K, n, n), dtype=torch.float64, device="cuda")
        wt = torch.zeros_like(mp)
        g.reduce(ctx, run.reduce_desc(d, 30 * ARC, t_star=ts, maps=(mp, wt), map_n=n,
                                      map_half_rad=half, pwv_mean_mm=1.1, T=T))
        ts = ts.cpu().numpy()
        assert (ts[:, :, T:] == 0).all()
        ref, scale = check_tstar(sc, ts[:, :, :T], t_b, 1.1, 30 * ARC)
        check_maps(sc, ref, scale, mp, wt, half, n)
    finally:
        g.free(ctx)


@pytest.mark.parametrize("K", [1, 2, 3, 4, 5, 8, 9, 17])
@pytest.mark.parametrize("T", [3, 16384, 16385])
def test_common_mode_of_few_channels(T, K):
    """Without maps: with and without the table of cosecants, threads of one to
    eight channels."""
    sc = scenario("daisy", T, K)
    t_b, d = fields(sc, T, T)
    ctx = new_ctx(workspace_bytes=16 << 20)
    try:
        run = g.ScenarioRun(ctx, sc)
        ts = torch.zeros_like(d)
        g.reduce(ctx, run.reduce_desc(d, 30 * ARC, t_star=ts, pwv_mean_mm=1.1, T=T))
        check_tstar(sc, ts.cpu().numpy(), t_b, 1.1, 30 * ARC)
    finally:
        g.free(ctx)
