"""1/f series at every number of pass-1 columns of the two-pass transform (1 to
512), against the oracle's FP64 series: the bound of the other 1/f tests, 1e-5
of the series' rms.  Accumulated into a TOD, whatever the rows' alignment, they
are the written series added with one FP32 rounding: the same bits."""
import numpy as np
import pytest
import torch

import oracle
import paper_2604_23305_amd as g
from oracle import pink as opk
from tests.gpu_util import new_ctx
from tests.test_gpu_parity import TOL_PINK, tiny_scenario

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = new_ctx(workspace_bytes=64 << 20)
    yield c
    g.free(c)


@pytest.mark.parametrize("lg", range(12, 22))     # N = 2^lg: 2^(lg - 12) columns
@pytest.mark.parametrize("odd", [0, 1])
def test_every_column_count(ctx, lg, odd):
    T = (1 << lg) - (1 << (lg - 2)) + odd
    sc = tiny_scenario(F=16, K=2, P=2, T=T)
    sc.pink_alpha = np.array([1.0, 1.7])
    run = g.ScenarioRun(ctx, sc)
    tod = torch.full((sc.n_pix, sc.K, T), 7.0, device="cuda")
    g.simulate_tod(ctx, [run.pink_job(tod, accumulate=False)])
    got = tod.cpu().numpy()
    A = opk.amplitude(oracle.tod.reference_nep2(sc), sc.pink_alpha, 1.0)
    for p, k in ((0, 0), (1, 1)):
        ref = opk.series(sc.seed, p, k, A[k], sc.pink_alpha[k], T, 160.0)
        assert np.abs(got[p, k] - ref).max() <= TOL_PINK * ref.std()
    base = torch.randn(sc.n_pix * sc.K * T + 1, device="cuda",
                       generator=torch.Generator("cuda").manual_seed(lg)) * got.std()
    for offset in (0, 1):
        into = base.clone()[offset:offset + got.size].reshape(got.shape)
        want = (into + tod).cpu()
        g.simulate_tod(ctx, [run.pink_job(into, accumulate=True)])
        assert torch.equal(into.cpu(), want)
