"""Screening with points far from the others: finite double positions beyond
float's range, and single satellites far outside the rest's radius.

Bars as for every screening test: events identical to the brute-force oracle's
or to the device-memory path's, distances equal to 1e-15 relative.
"""
import numpy as np
import pytest

from test_gpu_screen import check, gpu_events, shell_points

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [0, 2])
@pytest.mark.parametrize("n", [40, 3500])
def test_heights_beyond_float_range(n, mode):
    """Pairs at z = +-1e39 and 3e300 km: as valid as any other."""
    r = shell_points(n, 2, seed=n, planted=10)
    z = [1e39, 1e39, -1e39, 1e39, 3e300, 3e300]
    r[2, : len(z)] = np.array(z)[:, None]
    r[:2, : len(z)] = 100.0 + np.arange(len(z))[:, None]
    print(f"[gpu] screen heights beyond float: n={n} mode={mode}", flush=True)
    assert check(r, 12.0, mode=mode) > 6  # (0, 1), (0, 3), (1, 3) and (4, 5) at both times, and planted ones


def orbit(T, radius, seed):
    """One satellite's track at a radius: [3, T]."""
    a = np.random.default_rng(seed).uniform(0.0, 6.28) + np.linspace(0.0, 2.0, T)
    return radius * np.array([np.cos(a), np.sin(a) * 0.8, np.sin(a) * 0.6])


def catalogue(kind, n, T):
    """Low satellites with others far out, pairs among both."""
    r = shell_points(n, T, seed=n + T, planted=60)
    rng = np.random.default_rng(n)
    if kind in ("geo", "half"):
        m = n // 20 if kind == "geo" else n // 2
        a = rng.uniform(0.0, 6.28, (m, 1)) + np.linspace(0.0, 0.3, T)
        r[:, :m] = np.array([42164.0 * np.cos(a), 42164.0 * np.sin(a), rng.normal(size=(m, T)) * 20.0])
    else:
        r[:, 7] = orbit(T, float(kind), 1)
        r[:, 9] = r[:, 7] + 3.0
    return r


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("kind", ["42164", "120000", "4e6", "1e9", "geo", "half"])
def test_far_satellites_match_oracle(kind, dtype):
    r = catalogue(kind, 7000, 2).astype(dtype)
    print(f"[gpu] screen far satellites: {kind} {np.dtype(dtype).name}", flush=True)
    assert check(r, 11.0) > 20


def both_paths(r, D, err=None):
    ev, d, total = gpu_events(r, D, err, cap=1 << 22)
    ev2, d2, total2 = gpu_events(r, D, err, cap=1 << 22, mode=2)
    assert total == total2 == len(ev) and np.array_equal(ev, ev2) and np.array_equal(d, d2)
    return total


@pytest.mark.parametrize("kind", ["42164", "120000", "geo"])
@pytest.mark.parametrize("n,T", [(3073, 66), (16_384, 3), (16_385, 3), (40_003, 2), (200_000, 1), (200_001, 1)])
def test_far_satellites_match_the_device_memory_path(kind, n, T):
    """Satellite counts at the edges of one set, of counting every point, and of the
    column path."""
    print(f"[gpu] screen paths: {kind} n={n} T={T}", flush=True)
    assert both_paths(catalogue(kind, n, T).astype(np.float32), 9.0) > 20


def test_codes_and_invalid_points_over_more_than_one_time_tile():
    r = catalogue("42164", 5000, 66)
    rng = np.random.default_rng(2)
    err = np.zeros(r.shape[1:], np.uint8)
    err[rng.random(err.shape) < 0.2] = 1
    err[rng.random(err.shape) < 0.1] = 6
    r[:, rng.random(5000) < 0.05, :] = np.nan
    r[0, 17, :] = np.inf
    print("[gpu] screen: codes over 66 times", flush=True)
    assert both_paths(r, 20.0, err) > 100
    assert check(r, 20.0, err, times=[0, 1, 63, 64, 65]) > 10


def test_times_of_different_extent():
    """A time whose points all lie in one column beside ordinary ones."""
    r = shell_points(6000, 3, seed=3, planted=30)
    r[0, :, 1] = 6900.0 + 0.01 * np.arange(6000) / 6000.0
    r[:, :, 2] *= 40.0
    print("[gpu] screen: extents", flush=True)
    assert check(r, 9.0) > 20


@pytest.mark.parametrize("mode", [0, 2])
def test_twenty_thousand_match_oracle(mode):
    r = shell_points(20_000, 2, seed=78, planted=200).astype(np.float32)
    print(f"[gpu] screen n=20000 mode={mode}", flush=True)
    assert check(r, 15.0, mode=mode) > 100
