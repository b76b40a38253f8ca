"""Edges of the step loop's per-wave LDS tables and jump queues: waves with few paths,
horizons and cuts that are no multiple of a block of steps."""
from __future__ import annotations

import numpy as np
import pytest

from helpers import oracle_paths, say
from paper_1409_4923_amd import bmotor as B
from paper_1409_4923_amd import workloads as W

pytestmark = pytest.mark.gpu
BASE = {"gauss": W.C2.with_(noise=W.GAUSS), "poisson": W.C2, "dich": W.C3,
        "jump-grid": W.C2.with_(noise=W.GAUSS | W.POISSON | W.JUMP_GRID)}


def final(w, cuts, tune=None):
    e = B.Ensemble(*W.to_c(w), tune=tune)
    for c in cuts:
        e.integrate(c)
    return e.read()


@pytest.mark.parametrize("n", [1, 64, 65, 1024, 1025, 2048, 2049])
def test_statistics_in_one_launch_or_two(n):
    """Up to 2048 paths the velocities and their reduction are one launch: the same bits
    as a scan point, whose reduction runs on its own."""
    w = W.C1.with_(n_paths=n, n_steps=80, n_window=33, point=5)
    say("statistics", n)
    m, r = W.to_c(w)
    e = B.Ensemble(m, r)
    e.integrate(80)
    sc = B.Scan([m], [r])
    sc.launch()
    assert bytes(memoryview(e.stats())) == bytes(memoryview(sc.stats()[0]))


@pytest.mark.parametrize("prec", [W.F32, W.F64], ids=["f32", "f64"])
@pytest.mark.parametrize("model", sorted(BASE))
@pytest.mark.parametrize("n", [1, 20, 35, 36, 37, 64 + 3])
def test_few_paths_in_a_wave(model, prec, n):
    """A path does not depend on how many lanes of its wave hold a path."""
    w = BASE[model].with_(prec=prec, n_steps=77, n_window=19)
    say("few paths", model, prec, n)
    ref = final(w.with_(n_paths=192), [77])
    got = final(w.with_(n_paths=n), [5, 16, 56])
    for a, b in ((ref.x, got.x), (ref.v, got.v), (ref.noise, got.noise), (ref.vp, got.vp)):
        assert np.array_equal(a.numpy()[:n], b.numpy())


@pytest.mark.parametrize("rate", [0.1, 2.0, 20.0, 300.0])
def test_flips_at_any_rate(rate):
    """Dichotomous noise from flips in few blocks of steps to several in every four
    (windows with a look ahead, without one, and cut short by a full queue): every flip
    at its step, against the FP64 oracle."""
    w = W.C3.with_(prec=W.F64, mua=rate, mub=2.0 * rate, n_paths=130, n_steps=1100, n_window=333)
    say("flips", rate)
    got = final(w, [7, 500, 593])
    x, _, noise, _ = oracle_paths(w, 0, w.n_paths, w.n_steps)
    assert np.array_equal(got.noise.numpy(), noise)
    assert np.max(np.abs(got.x.numpy() - x) / np.maximum(1.0, np.abs(x))) <= 1e-9


@pytest.mark.parametrize("extra", [0, W.DICH, W.JUMP_GRID, W.DICH | W.JUMP_GRID],
                         ids=["kicks", "kicks+flips", "jump-grid", "jump-grid+flips"])
@pytest.mark.parametrize("rate_dt", [1e-6, 0.016, 0.09, 0.11, 0.6, 3.0])
def test_kicks_at_any_rate(rate_dt, extra):
    """Jump rings that are never filled, that wrap, that cut blocks short, of either size,
    and steps with more kicks than a ring: every kick at its step, against the FP64 oracle;
    the same bits from one call and from several."""
    w = W.C2.with_(prec=W.F64, noise=W.GAUSS | W.POISSON | extra, n_paths=130, n_steps=400, n_window=133,
                   Fa=0.3, Fb=0.6, point=4)
    rate = rate_dt / w.step()
    w = w.with_(lam=rate, zeta=0.05 / max(1.0, rate / 5.0), mua=0.5 * rate, mub=rate)
    say("kicks", rate_dt, extra)
    one = final(w, [400])
    got = final(w, [3, 16, 114, 1, 266], B.make_tune(1, 64))
    assert np.array_equal(one.x.numpy(), got.x.numpy()) and np.array_equal(one.noise.numpy(), got.noise.numpy())
    x, v, noise, _ = oracle_paths(w, 0, w.n_paths, w.n_steps)
    assert np.array_equal(got.noise.numpy(), noise)
    for a, b in ((got.x.numpy(), x), (got.v.numpy(), v)):
        assert np.max(np.abs(a - b) / np.maximum(1.0, np.abs(b))) <= 1e-9


@pytest.mark.parametrize("prec", [W.F32, W.F64], ids=["f32", "f64"])
@pytest.mark.parametrize("spp", [1, 7, 408, 409, 832, 833, 1500, 3400])
def test_forcing_tables_of_any_length(spp, prec):
    """Tables that go with one launch's arguments, with several, and by a copy: the same
    bits as a scan point, whose table a kernel forms; also through a resume."""
    w = W.C1.with_(prec=prec, spp=spp, n_paths=70, n_steps=2 * spp + 40, n_window=spp // 2, point=2)
    m, r = W.to_c(w)
    say("table", spp, prec)
    sc = B.Scan([m], [r])
    sc.launch()
    e = B.Ensemble(m, r)
    e.integrate(spp)
    f = B.Ensemble(m, r, checkpoint=e.checkpoint())
    for x in (e, f):
        x.integrate(w.n_steps - spp)
        assert bytes(memoryview(x.stats())) == bytes(memoryview(sc.stats()[0]))
