"""Mixed-precision points on both sides of the evaluation's dividing lines, dense
and in ragged lists, against the oracle: |axn| + |ayn| below 4.5e-3 (one Newton
step, series in e_L^2) and above, short-period rotations below 1.25e-3, below 0.05
and beyond (orbits inside the Earth).

Bars: the mixed path's 5 m and 5 mm/s, the velocity's in proportion to the orbit's
speed.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2603_27830_amd as sg
from test_gpu_point_fp64 import elements

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")


def check(el, t):
    r0, v0, c0 = oracle.propagate(el, t)[:3]
    rec = sg.init(torch.from_numpy(el).to(DEV))
    tt = torch.from_numpy(t).to(DEV)
    n, T = el.shape[1], t.size
    bar = 5e-6 * np.maximum(1.0, np.cbrt(el[0] / oracle.ke()))[:, None]
    r, v, c = (x.cpu().numpy() for x in sg.propagate(rec, tt, "mixed"))
    assert np.array_equal(c, c0)
    assert (np.abs(r - r0) <= 5e-3).all() and (np.abs(v - v0) <= bar).all()
    off = torch.arange(n + 1, dtype=torch.int64, device=DEV) * T
    r, v, c = (x.cpu().numpy().reshape(x.shape[:-1] + (n, T)) for x in sg.propagate_ragged(rec, off, tt.repeat(n), "mixed"))
    assert np.array_equal(c, c0)
    assert (np.abs(r - r0) <= 5e-3).all() and (np.abs(v - v0) <= bar).all()


@pytest.mark.parametrize("T", [1, 64, 100])
@pytest.mark.parametrize("kind", ["one_step", "newton", "mixed"])
def test_kepler_both_sides_of_the_bound(kind, T):
    small = [0.0, 1e-7, 1e-4, 1.5e-3, 3e-3, 4.4e-3]
    large = [4.7e-3, 8e-3, 3e-2, 0.1]
    e = np.array({"one_step": small, "newton": large, "mixed": small + large}[kind] * 10)
    el = elements(1.1 / (1.0 - e) + np.linspace(0.0, 0.1, e.size), e, e.size)
    el[6] = 1e-5
    print(f"[gpu] point mixed {kind} T={T}", flush=True)
    check(el, np.linspace(-720.0, 4320.0, T) if T > 1 else np.array([1234.0]))


@pytest.mark.parametrize("a", [0.95, 0.7, 0.3, 0.15])
def test_rotations_inside_the_earth(a):
    print(f"[gpu] point mixed a={a}", flush=True)
    check(elements(np.full(70, a), np.linspace(0.0, 0.02, 70), 3), np.linspace(0.0, 30.0, 65))
