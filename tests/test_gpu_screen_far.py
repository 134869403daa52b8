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
