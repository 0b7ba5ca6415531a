"""Common mode and maps at the edges of their kernels' ranges: tiles and tails
of time, an odd channel left over, rows at any alignment, cells of one run and
of many, narrow and wide elevation ranges, workspaces with and without room for
the run lists.

Tolerances: T* within 2^-23 of itself (FP32 storage) + 1e-10 of the terms that
cancel; maps within 1e-9 of those, weights 1e-8 relative (FP64 throughout)."""
import numpy as np
import pytest
import torch

import paper_2604_23305_amd as g
from oracle import reduce as orr
from tests.gpu_util import new_ctx
from tests.test_gpu_reduce import check_tstar, hex_scenario
from workloads import gen
from workloads.scenario import Scan

pytestmark = pytest.mark.gpu
ARC = gen.ARCSEC


def scenario(scan, T, K):
    sc = hex_scenario(T=max(T, 8), F=200, K=K)
    if scan == "stare":
        sc.scan = Scan("stare", theta0=sc.scan.theta0)
    elif scan == "wide":          # several degrees
        t = np.arange(max(T, 8)) / sc.f_sample_hz
        traj = np.stack([0.08 * np.cos(3 * t), 0.08 * np.sin(5 * t)], axis=1)
        sc.scan = Scan("traj", theta0=sc.scan.theta0, traj=np.ascontiguousarray(traj))
    return sc


def fields(sc, T, ld):
    r = np.random.default_rng([T, sc.K])
    t_b = (200.0 + r.standard_normal((sc.n_pix, sc.K, T))).astype(np.float32)
    d = torch.full((sc.n_pix, sc.K, ld), float("nan"), device="cuda")
    d[:, :, :T] = torch.from_numpy(t_b).cuda()
    return t_b, d


def check_maps(sc, ref, scale, mp, wt, half, n):
    m_o, w_o = orr.combine(*orr.spaxel_maps(sc, ref, half, n))
    m_g, w_g = (x.cpu().numpy().reshape(sc.K, -1) for x in (mp, wt))
    live = w_o > 0
    assert live.any() and np.array_equal(w_g > 0, live)
    assert np.array_equal(np.isnan(m_g), np.isnan(m_o))
    assert np.abs(m_g[live] - m_o[live]).max() <= 1e-9 * scale.max()
    assert (np.abs(w_g[live] - w_o[live]) / w_o[live]).max() <= 1e-8


@pytest.mark.parametrize("scan,half", [("stare", 150 * ARC), ("daisy", 150 * ARC),
                                       ("wide", 0.08)])
@pytest.mark.parametrize("T,K,n,pad", [
    (2, 1, 2, 0),
    (5, 3, 9, 1),            # rows at every alignment
    (2047, 4, 15, 0),
    (2048, 5, 31, 0),
    (2049, 2, 48, 3),        # a tile of one sample; the largest map
    (4101, 7, 21, 2),
])
@pytest.mark.parametrize("room", [True, False])
def test_maps_and_common_mode(scan, half, T, K, n, pad, room):
    sc = scenario(scan, T, K)
    # one channel's rows and statistics (three quarters of the workspace hold
    # them), and nothing else
    tight = 24 * T + 8 * K + sc.n_pix * n * n * 16 + 2048
    ctx = new_ctx(workspace_bytes=8 << 20 if room else tight * 4 // 3)
    try:
        run = g.ScenarioRun(ctx, sc)
        t_b, d = fields(sc, T, T + pad)
        ts = torch.zeros_like(d)
        mp = torch.zeros((K, n, n), dtype=torch.float64, device="cuda")
        wt = torch.zeros_like(mp)
        g.reduce(ctx, run.reduce_desc(d, 30 * ARC, t_star=ts, maps=(mp, wt), map_n=n,
                                      map_half_rad=half, pwv_mean_mm=1.1, T=T))
        ts = ts.cpu().numpy()
        assert (ts[:, :, T:] == 0).all()
        ref, scale = check_tstar(sc, ts[:, :, :T], t_b, 1.1, 30 * ARC)
        check_maps(sc, ref, scale, mp, wt, half, n)
        # without maps; into the TOD itself
        g.reduce(ctx, run.reduce_desc(d, 30 * ARC, t_star=d, pwv_mean_mm=1.1, T=T))
        check_tstar(sc, d.cpu().numpy()[:, :, :T], t_b, 1.1, 30 * ARC)
    finally:
        g.free(ctx)


@pytest.mark.parametrize("length,pad", [(1, 0), (40, 3), (9362, 1), (9363, 0), (30001, 7)])
def test_mean_pwv_of_the_partial_sums(length, pad):
    """7 rows of PWV around one tile of the partial sums (65536 values) and
    over several, contiguous and pitched: the same bits as summed by one block,
    where the workspace has no room for the partial sums."""
    sc = scenario("daisy", 64, 3)
    r = np.random.default_rng(length)
    pwv = torch.full((7, length + pad), float("nan"), device="cuda")
    pwv[:, :length] = torch.from_numpy(r.uniform(0.8, 1.3, (7, length)).astype(np.float32))
    got = []
    for ws in (8 << 20, 4096):
        ctx = new_ctx(workspace_bytes=ws)
        try:
            run = g.ScenarioRun(ctx, sc)
            _, d = fields(sc, 64, 64)
            ts = torch.zeros_like(d)
            desc = run.reduce_desc(d, 30 * ARC, t_star=ts, pwv=pwv)
            desc.pwv_len = length
            g.reduce(ctx, desc)
            got.append(ts.cpu())
        finally:
            g.free(ctx)
    assert torch.isfinite(got[0]).all() and torch.equal(got[0], got[1])
