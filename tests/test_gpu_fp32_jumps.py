"""FP32 paths with kicks and flips at any rate: rings that are never filled, that wrap and
that cut blocks short, and on the jump-adapted grid steps with more kicks than a ring.  The
path precision has code of its own for these (rings of nine slots, the first piece of a step
selected in every lane), so the FP64 tests do not cover it."""
from __future__ import annotations

import numpy as np
import pytest

from helpers import oracle_paths, say
from paper_1409_4923_amd import bmotor as B
from paper_1409_4923_amd import workloads as W

pytestmark = pytest.mark.gpu
SHORT, LONG = 60, 400


def workload(noise, rate_dt, **kw):
    w = W.C2.with_(prec=W.F32, noise=noise, n_paths=130, n_steps=LONG, n_window=133, Fa=0.3, Fb=0.6, point=4)
    rate = rate_dt / w.step()
    return w.with_(lam=rate, zeta=0.05, mua=0.5 * rate, mub=rate, **kw)


def final(w, cuts, tune=None):
    e = B.Ensemble(*W.to_c(w), tune=tune)
    for c in cuts:
        e.integrate(c)
    return e.read()


@pytest.mark.parametrize("extra", [0, W.DICH, W.JUMP_GRID, W.DICH | W.JUMP_GRID],
                         ids=["kicks", "kicks+flips", "jump-grid", "jump-grid+flips"])
@pytest.mark.parametrize("gauss", [W.GAUSS, W.NORMAL], ids=["three-point", "normal"])
@pytest.mark.parametrize("rate_dt", [1e-6, 0.016, 0.11, 0.6, 3.0, 9.0])
def test_fp32_jumps_at_any_rate(rate_dt, gauss, extra):
    """Every jump at its step as in FP64; the positions of the FP64 oracle over a stretch too
    short for the dynamics to amplify the roundings; and the same bits whatever the cuts, the
    launch shape and the paths that share a wave (which decide when a block is cut short and
    which lanes take a step with a full ring of their neighbour's)."""
    w = workload(gauss | W.POISSON | extra, rate_dt)
    say("fp32 jumps", rate_dt, gauss, extra)
    # 60 steps: about 3 roundings of 2.4e-7 per step in v, amplified by at most
    # exp(sqrt(4 pi^2) 60 dt) = 3.4
    x, v, noise, _ = oracle_paths(w, 0, w.n_paths, SHORT)
    got = final(w, [SHORT])
    assert np.array_equal(got.noise.numpy(), noise)
    for a, b in ((got.x.numpy(), x), (got.v.numpy(), v)):
        assert np.max(np.abs(a - b) / np.maximum(1.0, np.abs(b))) <= 5e-4
    one = final(w, [LONG])
    assert np.array_equal(one.noise.numpy(), oracle_paths(w, 0, w.n_paths, LONG)[2])
    for n, cuts, tune in ((130, [3, 16, 114, 1, 266], B.make_tune(1, 64)), (130, [77, 323], B.make_tune(2, 128)),
                          (1, [LONG], None), (70, [50, 350], None)):
        got = final(w.with_(n_paths=n), cuts, tune)
        for a, b in ((one.x, got.x), (one.v, got.v), (one.noise, got.noise), (one.vp, got.vp)):
            assert np.array_equal(a.numpy()[:n], b.numpy()), (n, cuts)
