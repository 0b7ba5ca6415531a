"""Input preparation in a workspace smaller than its fixed scratch (quadrature
nodes, footprint factors): the same results as in a large one, and nothing
written beyond the workspace's own allocation."""
import numpy as np
import pytest
import torch

import paper_2604_23305_amd as g
from tests.gpu_util import new_ctx

pytestmark = pytest.mark.gpu
D = 2.5 * np.pi / 180 / 3600


def test_a_workspace_of_256_bytes():
    nu = np.array([457e9])
    scr = torch.from_numpy(np.random.default_rng(1).uniform(0, 2, (70, 300))).cuda()
    got = []
    for ws in (256, 64 << 20):
        ctx = new_ctx(workspace_bytes=ws)
        try:
            # 58.9 kB of nodes for 300 entries by quadrature, the most there can be
            far = g.far_field(ctx, nu, 300, 1, 5990.0 / 2 / np.pi / 5.0 * 299792458.0 / 457e9 / 299,
                              D, 5.0, -10.0)
            small = g.convolve_screen(ctx, scr, 0.2, 0.2, 5.0, -10.0)
            torch.cuda.synchronize()
            got.append((far.cpu(), small.cpu()))
            assert g.memory(ctx)[0] >= 64 << 10
        finally:
            g.free(ctx)
    assert torch.equal(got[0][0], got[1][0])
    assert torch.equal(got[0][1], got[1][1])
