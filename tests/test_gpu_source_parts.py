"""Outputs of the transformed source convolution that are summed directly, by one
workgroup per frequency or by several: a lone bright node, whose far sidelobes
lie below the transforms' error.  7.5e-8 relative, as for all outputs."""
import numpy as np
import pytest
import torch

import paper_2604_23305_amd as g
from tests.gpu_util import new_ctx
from tests.test_gpu_source import D, plane

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_az,n_el", [(30, 31), (41, 50), (60, 90), (200, 99)])
@pytest.mark.parametrize("n_f", [1, 20, 130, 300])
def test_few_and_many_frequencies(n_az, n_el, n_f):
    nu = np.linspace(210e9, 457e9, n_f)
    I = plane("node", n_el, n_az).astype(np.float32)
    cube = torch.from_numpy(I).cuda()[:, :, None].repeat(1, 1, n_f).contiguous()
    c = new_ctx(workspace_bytes=1 << 30)
    try:
        got = g.convolve_source(c, cube, nu, D, 0.9, D, 5.0, -10.0)[:, :, [0, n_f - 1]]
        F = g.far_field(c, nu, n_az, n_el, D, D, 5.0, -10.0)[[0, n_f - 1]].cpu().numpy()
        got = got.cpu().numpy().astype(np.float64)
    finally:
        g.free(c)
    j, i = np.argwhere(I)[0]
    w = np.float64(np.float32(np.cos(0.9 + D * j)))
    for f in range(2):
        ref = np.pi * 25.0 * D * D * w * F[f].astype(np.float64)[
            np.abs(np.arange(n_el) - j)][:, np.abs(np.arange(n_az) - i)]
        assert (np.abs(got[..., f] - ref) <= 7.5e-8 * ref).all()
