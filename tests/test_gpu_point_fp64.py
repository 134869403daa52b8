"""FP64 points on both sides of the evaluation's dividing lines, against the
oracle: the one-step solution of Kepler's equation (|axn| + |ayn| up to 3e-3) and
Newton's iteration, wavefronts that mix the two, short-period rotations below
1.25e-3, below 0.05 and beyond (orbits inside the Earth), and times so far from
epoch that the secular angles are reduced first.

Bars: both sides round a handful of sums of the angles' size, so the mean anomaly
may differ by 32 half-ulps of |n t| + 20 rad; that moves the position by at most
a sqrt((1 + e) / (1 - e)) and the velocity by n a / (1 - e)^2 per radian.  Inside
the Earth the secular rates of the node and perigee are of the mean motion's
size: four times that.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2603_27830_amd as sg

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")
RADIUS = 6378.135


def elements(a, e, seed):
    """Rows: mean motion (rad/min), eccentricity, inclination, angles, drag, epoch."""
    rng = np.random.default_rng(seed)
    n = len(a)
    ang = lambda: rng.uniform(0.0, 2.0 * np.pi, n)  # noqa: E731
    return np.stack([oracle.ke() * a ** -1.5, e, rng.uniform(0.1, 3.0, n), ang(), ang(), ang(), np.zeros(n), np.zeros(n)])


def bars(el, t, factor=1.0):
    n, e = el[0][:, None], el[1][:, None]
    a = RADIUS * (n / oracle.ke()) ** (-2.0 / 3.0)
    dphi = factor * 32.0 * 2.0 ** -53 * (np.abs(n * t[None]) + 20.0)
    return dphi * a * np.sqrt((1.0 + e) / (1.0 - e)), dphi * n / 60.0 * a / (1.0 - e) ** 2


@pytest.mark.parametrize("T", [1, 3, 64, 100])
@pytest.mark.parametrize("kind", ["one_step", "newton", "mixed"])
def test_kepler_both_sides_of_the_bound(kind, T):
    small = [0.0, 1e-7, 1e-5, 5e-4, 1.5e-3, 2.5e-3, 2.9e-3]
    large = [3.1e-3, 5e-3, 1e-2, 3e-2, 0.1, 0.3]
    e = np.array({"one_step": small, "newton": large, "mixed": small + large}[kind] * 10)
    a = 1.08 / (1.0 - e) + np.linspace(0.0, 0.3, e.size)
    el = elements(a, e, e.size)
    el[6] = 1e-5
    t = np.linspace(-1440.0, 10080.0, T) if T > 1 else np.array([4321.0])
    r0, v0, c0 = oracle.propagate(el, t)[:3]
    r, v, c = (x.cpu().numpy() for x in sg.propagate(sg.init(torch.from_numpy(el).to(DEV)), torch.from_numpy(t).to(DEV), "fp64"))
    print(f"[gpu] point fp64 {kind} T={T}", flush=True)
    assert np.array_equal(c, c0)
    br, bv = bars(el, t)
    assert (np.abs(r - r0) <= br).all() and (np.abs(v - v0) <= bv).all()


@pytest.mark.parametrize("a", [0.95, 0.8, 0.7, 0.5, 0.3, 0.15])
def test_rotations_inside_the_earth(a):
    el = elements(np.full(70, a), np.linspace(0.0, 0.02, 70), 3)
    t = np.linspace(0.0, 30.0, 65)
    r0, v0, c0 = oracle.propagate(el, t)[:3]
    r, v, c = (x.cpu().numpy() for x in sg.propagate(sg.init(torch.from_numpy(el).to(DEV)), torch.from_numpy(t).to(DEV), "fp64"))
    print(f"[gpu] point fp64 a={a}", flush=True)
    assert np.array_equal(c, c0) and (c == 6).all()
    br, bv = bars(el, t, 4.0)
    assert (np.abs(r - r0) <= br).all() and (np.abs(v - v0) <= bv).all()


@pytest.mark.parametrize("t", [2.0e12, -3.0e14, 1.0e18])
def test_far_times_stay_on_the_orbit(t):
    el = elements(np.linspace(1.1, 1.4, 64), np.full(64, 1e-3), 5)
    for tt in (torch.full((1,), t), torch.full((64,), t)):
        r, _, c = sg.propagate(sg.init(torch.from_numpy(el).to(DEV)), tt.to(DEV, torch.float64), "fp64")
        print(f"[gpu] point fp64 t={t}", flush=True)
        d = r.norm(dim=0).cpu().numpy() / (RADIUS * np.linspace(1.1, 1.4, 64))[:, None]
        assert (c == 0).all() and (abs(d - 1.0) < 0.01).all()
