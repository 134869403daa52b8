"""Conjunction screening by column sets: sizes at the edges of the tables and of
the four-point class words, point sets that overflow a table, distances from
far below to far above the spacing, and coordinates far from the origin.

Bars as for every screening test: the events identical to the brute-force
oracle's, distances equal to 1e-15 relative (the same operations on the same
stored positions).
"""
import numpy as np
import pytest
import torch

import paper_2603_27830_amd as sg
from oracle import screen as osc

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")


def shell(n, T, seed, radius=6900.0):
    rng = np.random.default_rng(seed)
    v = rng.normal(size=(3, n, T))
    v *= (radius + rng.uniform(-20.0, 20.0, (n, T))) / np.linalg.norm(v, axis=0)
    for _ in range(min(60, n // 2)):
        i, j = rng.choice(n, 2, replace=False)
        k = rng.integers(0, T)
        v[:, j, k] = v[:, i, k] + rng.normal(size=3) * rng.uniform(0.0, 15.0)
    return v


def matches(r, D, err=None):
    cap = 1 << 21
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)  # noqa: E731
    pairs, dist, total = sg.screen(dev(r), D, None if err is None else dev(err), capacity=cap)
    p, d = pairs.cpu().numpy().astype(np.int64), dist.cpu().numpy()
    order = np.lexsort((p[:, 1], p[:, 0], p[:, 2]))
    want, far = osc.screen(r, D, err=err)
    print(f"[gpu] screen columns {r.shape} {r.dtype} D={D}: {total} events", flush=True)
    assert total == len(want) <= cap
    assert np.array_equal(p[order], want)
    assert np.allclose(d[order], far, rtol=1e-15, atol=0.0)
    return total


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("n,T", [(2, 1), (5, 70), (3071, 3), (3072, 2), (3073, 3), (6146, 2), (12289, 1)])
def test_table_and_word_edges(n, T, dtype):
    matches(shell(n, T, n).astype(dtype), 12.0)


@pytest.mark.parametrize("D", [1e-3, 0.7, 60.0, 900.0])
def test_distances_around_the_spacing(D):
    r = shell(3500, 2, 11)
    r[:, 1] = r[:, 0] + 0.4 * min(D, 1.0)
    assert matches(r, D) > 0


@pytest.mark.parametrize("kind", ["plane", "line", "point"])
def test_points_that_overflow_a_table(kind):
    """All x in one column: one set holds every point and works in runs."""
    rng = np.random.default_rng(5)
    n, T = 7001, 1
    r = np.zeros((3, n, T))
    r[0] = 6900.0 + rng.uniform(0.0, 0.5, (n, T))
    if kind != "point":
        r[1] = rng.uniform(-7000.0, 7000.0, (n, T))
    if kind == "plane":
        r[2] = rng.uniform(-7000.0, 7000.0, (n, T))
    if kind == "point":
        r += rng.normal(size=r.shape) * 40.0
    assert matches(r, 4.0 if kind == "point" else 20.0 if kind == "plane" else 1.5) > 0


@pytest.mark.parametrize("scale,D", [(1e-3, 1e-6), (1.0, 1e-2), (1e6, 5.0), (1e30, 1e28)])
def test_ratios_of_distance_to_coordinate(scale, D):
    """Distances down to the float rounding of the coordinates and below it."""
    r = shell(4000, 2, 8) * scale
    r[:, 7] = r[:, 3]
    r[0, 7] += 0.5 * D
    assert matches(r, D) > 0


def test_invalid_and_overflowing_points_are_left_out():
    r = shell(5000, 66, 21)[:, :, :66]
    rng = np.random.default_rng(2)
    err = np.zeros(r.shape[1:], np.uint8)
    err[rng.random(err.shape) < 0.2] = 1
    err[rng.random(err.shape) < 0.1] = 6
    r[:, rng.random(5000) < 0.05, :] = np.nan
    r[0, 17, :] = np.inf
    matches(r[:, :, [0, 1, 63, 64, 65]], 20.0, err[:, [0, 1, 63, 64, 65]])
