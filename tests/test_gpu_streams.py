"""Calls that run at the same time: on two streams of one context, and in two
host threads with a context each.  Every output has the bits it has alone."""
import threading

import numpy as np
import pytest
import torch

import paper_2604_23305_amd as g
from paper_2604_23305_amd import binding
from tests.gpu_util import new_ctx
from tests.test_oracle_pins import tiny_scenario
from workloads import gen

pytestmark = pytest.mark.gpu
ARC = gen.ARCSEC


class Work:
    """A signal job in each precision with 1/f noise added, a reduction of its
    TOD (common mode alone: maps are summed by atomics), a source convolution and
    a screen."""

    def __init__(self, ctx, seed, F, K, T, n):
        self.ctx, self.seed = ctx, seed
        sc = tiny_scenario(F=F, K=K, P=7, T=T, filt="matrix", seed=seed)
        sc.pink_alpha = np.linspace(0.8, 1.2, K)
        sc.dphi, sc.dtheta = gen.hex_spaxels(1, 12 * ARC)
        self.run = g.ScenarioRun(ctx, sc)
        r = torch.Generator("cuda").manual_seed(seed)
        self.cube = torch.rand((n, n + 3, 9), generator=r, device="cuda")
        self.screen = torch.rand((90, 700), generator=r, device="cuda", dtype=torch.float64)
        self.tod = torch.rand((7, K, T), generator=r, device="cuda") + 200.0
        self.out = [self.run.alloc(with_p_kid=True, with_sigma=True) for _ in range(2)]
        self.star = torch.zeros_like(self.tod)
        self.made = []

    def enqueue(self, stream):
        with torch.cuda.stream(stream):
            for prec in (0, 1):
                o = self.out[prec]
                g.simulate_tod(self.ctx, [
                    self.run.pink_job(o.tod, accumulate=False),
                    self.run.signal_job(o, precision=prec, accumulate=True)])
            g.reduce(self.ctx, self.run.reduce_desc(self.tod, 6 * ARC, t_star=self.star,
                                                    pwv_mean_mm=1.0))
            d = 2.5 * ARC
            self.made = [
                binding.convolve_source(self.ctx, self.cube, np.linspace(2e11, 4e11, 9), d, 0.9,
                                        d, 5.0, -10.0),
                binding.convolve_screen(self.ctx, self.screen, 0.2, 0.2, 5.0, -10.0),
                binding.convolve_screen(self.ctx, self.screen, 2.0, 2.0, 5.0, -10.0)]

    def results(self):
        o = [getattr(x, n) for x in self.out for n in ("tod", "p_kid", "sigma")]
        return [x.cpu() for x in o + [self.star] + self.made]


# two of every kind of launch: small tiles and large, in order and sorted rows
SIZES = [(1, 64, 70, 3000, 40), (2, 1100, 3, 300, 30)]


def alone():
    want = []
    for size in SIZES:
        ctx = new_ctx()
        try:
            w = Work(ctx, *size)
            torch.cuda.synchronize()
            w.enqueue(torch.cuda.current_stream())
            torch.cuda.synchronize()
            want.append(w.results())
        finally:
            g.free(ctx)
    return want


def check(want, got):
    for a, b in zip(want, got):
        assert len(a) == len(b)
        for x, y in zip(a, b):
            assert torch.equal(x, y)


def test_two_streams_of_one_context():
    want = alone()
    ctx = new_ctx(workspace_bytes=256 << 20)
    try:
        work = [Work(ctx, *size) for size in SIZES]
        streams = [torch.cuda.Stream() for _ in work]
        torch.cuda.synchronize()
        for _ in range(3):
            for w, s in zip(work, streams):
                w.enqueue(s)
        torch.cuda.synchronize()
        check(want, [w.results() for w in work])
    finally:
        g.free(ctx)


def test_two_threads_with_a_context_each():
    want = alone()
    got, errors = [None, None], []

    def body(i):
        try:
            ctx = new_ctx(workspace_bytes=256 << 20)
            try:
                s = torch.cuda.Stream()
                with torch.cuda.stream(s):
                    w = Work(ctx, *SIZES[i])
                    for _ in range(3):
                        w.enqueue(s)
                    s.synchronize()
                    got[i] = w.results()
            finally:
                g.free(ctx)
        except Exception as e:     # reported by the test's own thread
            errors.append(e)

    threads = [threading.Thread(target=body, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    check(want, got)
