"""The FP64 kernels' periodic force (argument in turns, one polynomial) through one step
of Algorithm 1 without noise, from positions where its reduction can go wrong: quarter
and half turns, the ends of a period, tiny, negative, unfolded and huge positions."""
from __future__ import annotations

import numpy as np
import pytest

from helpers import say
from paper_1409_4923_amd import bmotor as B
from paper_1409_4923_amd import workloads as W

pytestmark = pytest.mark.gpu
PI = np.longdouble("3.14159265358979323846264338327950288")


def positions():
    q = np.array([0.0, 0.125, 0.25, 0.375, 0.5, 0.75, 1.0])
    near = np.concatenate([np.nextafter(q, -9.0), q, np.nextafter(q, 9.0)])
    rng = np.random.default_rng(1)
    return np.concatenate([near, -near, [1e-300, 1e-17, 2.0 ** -30, 3.0 ** 9, -1e5 / 3, 2.0 ** 30 + 0.375,
                                         2.0 ** 51 + 0.5, 2.0 ** 53, 1e300], rng.uniform(-3, 3, 200),
                           rng.uniform(-1e6, 1e6, 200)])


def cos_turns(x):
    """cos 2 pi x in extended precision: the reduction by whole turns is exact."""
    r = np.abs(x - np.rint(x))
    return np.where(r <= 0.125, np.cos(2 * PI * r), np.sin(2 * PI * (np.longdouble(0.25) - r)))


@pytest.mark.parametrize("pot", [W.POT_SIN, W.POT_RATCHET], ids=["sin", "ratchet"])
def test_force_over_the_whole_line(pot):
    h, F = 2.0 ** -6, 0.3
    x0 = positions()
    w = W.C3.with_(pot=pot, noise=0, prec=W.F64, n_paths=len(x0), n_steps=1, n_window=0, dt=h, F=F)
    say("fp64 force", w.name, pot, len(x0))
    e = B.Ensemble(*W.to_c(w))
    rec = B.records(e.read_state()).copy()
    rec["x"], rec["periods"] = x0, 0
    e.write_state(rec)
    e.integrate(1)
    got = e.read().x.numpy()

    def force(x):
        c = cos_turns(x)
        return (-2 * PI * c if pot == W.POT_SIN else 2 * PI * c + PI * (2 * c * c - 1)) + np.longdouble(F)

    x = x0.astype(np.longdouble)
    f1 = force(x)
    f2 = force((x + f1 * h).astype(np.float64).astype(np.longdouble))
    xp = x + (f1 + f2) * (h / 2)
    want = x + (f1 + force(xp.astype(np.float64).astype(np.longdouble))) * (h / 2)
    # one evaluation is within 4e-15 (the roundings of values below 4 pi); the stages
    # evaluate at positions a few ulp apart, where the force changes by at most 8 pi^2
    # times that; the step weighs the forces with h, and x itself is rounded four times
    ulp = np.spacing(np.maximum(np.abs(x0), 1.0))
    tol = 4.0 * ulp + h * (4e-15 + 2.0 * 79.0 * 2.0 * ulp)
    err = np.abs((got.astype(np.longdouble) - want).astype(np.float64))
    assert np.all(np.isfinite(got)) and np.all(err <= tol), (x0[np.argmax(err / tol)], err.max())
