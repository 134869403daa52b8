"""Angles of any size: elements whose node, argument or anomaly is far beyond the
range of the sine table, and drag polynomials long after a decay.

Bars: an element angle X stands for X mod 2 pi exactly, so the record's sin M0
is that of the reduced angle to 1e-15 (an ulp or so of 1, twice), and states with
the node at X are those with the reduced node up to the node's own rounding
(half an ulp of X, as X plus the node's drift is rounded) and 1e-9 km.  Sines and cosines are bounded: a state
is never further out than twice the semi-major axis a0 A(t)^2 (e < 1).
"""
from decimal import Decimal, getcontext

import numpy as np
import pytest
import torch

import oracle
import paper_2603_27830_amd as sg
import synth

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")
LARGE = np.array([3.0e11, 2.0e12, -1.0e13, 6.9e13, 7.1e13, 1.2e14, -3.0e14, 1.0e15, 4.0e15])


def reduced(x):
    """x mod 2 pi by decimal arithmetic, the double nearest."""
    getcontext().prec = 60
    turn = 2 * Decimal("3.14159265358979323846264338327950288419716939937510582097494459")
    return float(Decimal(float(x)) % turn)


def states(el, t):
    rec = sg.init(torch.from_numpy(el).to(DEV))
    r, v, c = sg.propagate(rec, torch.from_numpy(t).to(DEV), "fp64")
    return rec, r.cpu().numpy(), v.cpu().numpy(), c.cpu().numpy()


def slots(rec):
    """The record's doubles: 64 of the header, then 64 per satellite."""
    return rec.consts.cpu().numpy().view(np.float64)[64:64 + 64 * rec.n].reshape(rec.n, 64)


def test_sines_of_large_element_angles():
    el = synth.shell_elements(LARGE.size, 4)
    el[5] = LARGE
    rec, *_ = states(el, np.zeros(1))
    want = np.array([np.sin(reduced(x)) for x in LARGE])
    print("[gpu] angles: sin M0", flush=True)
    assert np.abs(slots(rec)[:, 18] - want).max() <= 1e-15


def test_states_with_a_large_node():
    el = synth.shell_elements(LARGE.size, 4)
    t = np.array([0.0, 700.0, -2000.0])
    el[3] = [reduced(x) for x in LARGE]
    _, r0, v0, c0 = states(el, t)
    el[3] = LARGE
    rec, r, v, c = states(el, t)
    print("[gpu] angles: large node", flush=True)
    assert np.array_equal(c, c0) and (c == 0).all()
    far = np.linalg.norm(r0, axis=0)
    assert (np.linalg.norm(r - r0, axis=0) <= 1e-9 + far * np.spacing(np.abs(LARGE))[:, None]).all()
    # the node turns the state about the pole: its third component and its size stay
    assert np.abs(r[2] - r0[2]).max() <= 1e-9
    assert np.abs(np.linalg.norm(r, axis=0) - far).max() <= 1e-9
    jac = sg.jacobian(rec, torch.from_numpy(t).to(DEV)).cpu().numpy()
    # (its node sum rounds by itself: the horizontal distance is what both share)
    assert np.abs(np.hypot(jac[0, 3], jac[1, 3]) - np.hypot(r[0], r[1])).max() <= 1e-8


@pytest.mark.parametrize("row", [3, 4])
def test_deep_space_terms_with_large_angles(row):
    """The lunar-solar rates and coefficients: those of the reduced angle, their
    sums of a few dozen products to 1e-12 of the largest of each kind."""
    el = synth.deep_elements(LARGE.size, 5)
    n = LARGE.size
    terms = []
    for angles in ([reduced(x) for x in LARGE], LARGE):
        el[row] = angles
        rec, *_ = states(el, np.zeros(1))
        terms.append(rec.consts.cpu().numpy().view(np.float64)[64 + 64 * n:].reshape(n, 64)[:, :31])
    print(f"[gpu] angles: deep-space terms, row {row}", flush=True)
    assert (np.abs(terms[1] - terms[0]) <= 1e-12 * np.abs(terms[0]).max(axis=0)).all()


@pytest.mark.parametrize("row", [3, 4, 5])
def test_deep_space_states_with_large_angles_are_bounded(row):
    el = synth.deep_elements(8 * LARGE.size, 4)
    el[row] = np.tile(LARGE, 8)
    _, r, _, c = states(el, np.array([0.0, 700.0, -2000.0]))
    a = 6378.135 * (oracle.ke() / el[0]) ** (2.0 / 3.0)
    ok = (c == 0) | (c == 6)
    print(f"[gpu] angles: deep space, row {row}: {int(ok.sum())} states", flush=True)
    assert ok.sum() > ok.size // 2
    assert (np.linalg.norm(r, axis=0)[ok] <= np.broadcast_to(2.1 * a[:, None], ok.shape)[ok]).all()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_states_long_after_a_decay_are_bounded(prec):
    n = 400
    el = synth.shell_elements(n, 6)
    rng = np.random.default_rng(6)
    el[6] = 10.0 ** rng.uniform(-6.0, -1.0, n) * rng.choice([-1.0, 1.0], n)
    t = np.array([1e5, 1e6, 1e7, -1e7, 1e8, 1e9, -1e10, 1e11])
    rec = sg.init(torch.from_numpy(el).to(DEV))
    r, _, c = (x.cpu().numpy().astype(float) for x in sg.propagate(rec, torch.from_numpy(t).to(DEV), prec))
    d = slots(rec)
    C1, D2, D3, D4, a0 = d[:, 30], d[:, 32], d[:, 33], d[:, 34], d[:, 38]
    dt = t[None] - d[:, 12:13]
    A = 1.0 - dt * (C1[:, None] + dt * (D2[:, None] + dt * (D3[:, None] + dt * D4[:, None])))
    a = a0[:, None] * A * A * 6378.135
    ok = ((c == 0) | (c == 6)) & (a > 1e4) & (a < 1e30)
    print(f"[gpu] angles: long after decay, {prec}: {int(ok.sum())} states", flush=True)
    assert ok[:, 4:].sum() > 100
    far = np.linalg.norm(r, axis=0)
    assert (far[ok] <= 2.1 * a[ok]).all()
