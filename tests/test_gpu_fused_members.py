"""The fused elements-to-states launch by its members: deep-space satellites alone,
singly and among others, on both widths of the launch and beyond what its on-chip
memory holds at a time (66,000 x 3), against the two-stage path.

Bars: codes, satellite flags and the places of NaN states equal for every member;
near-Earth states to rounding, as for the fused call everywhere (FP64 1e-8 km and
1e-11 km/s, the float paths 5 m and 5 mm/s); deep-space states FP64 1e-6 km and
1e-9 km/s, mixed the deep-space bar of the mixed path against FP64 (10 m and 1e-2
m/s times (|r| / 7,000 km) / (1 - e0)).
"""
import numpy as np
import pytest
import torch

import paper_2603_27830_amd as sg
import synth
from test_gpu_deep import check_mixed
from test_gpu_fused_groups import DEV, TOL, mixture

pytestmark = pytest.mark.gpu


def members(kind, n, seed):
    if kind == "mixture":
        return mixture(n, seed)
    el = synth.shell_elements(n, seed)
    deep = np.ones(n, bool) if kind == "deep" else np.arange(n) % 997 == (n - 1) % 997
    el[:, deep] = synth.deep_elements(max(n, 64), seed)[:, :n][:, deep]
    return el, deep


@pytest.mark.parametrize("prec", ["fp64", "mixed", "fp32"])
@pytest.mark.parametrize("kind,n,T", [
    ("deep", 1, 2), ("deep", 64, 2), ("deep", 65, 8), ("deep", 129, 33), ("deep", 1000, 32), ("deep", 70, 300),
    ("deep", 40_000, 9), ("deep", 66_000, 3), ("deep", 200, 1), ("one", 64, 5), ("one", 3000, 1), ("one", 30_000, 19),
    ("mixture", 33_000, 9), ("mixture", 32_769, 17), ("mixture", 20_001, 19), ("mixture", 600, 700),
    ("mixture", 70_001, 8), ("mixture", 3000, 1)])
def test_members_match_two_stage_path(kind, n, T, prec):
    el, deep = members(kind, n, n + T)
    t = np.sort(np.random.default_rng(T).uniform(-600.0, 4000.0, T))
    e, dt = torch.from_numpy(el).to(DEV), torch.from_numpy(t).to(DEV)
    rec = sg.init(e, ref_jd=synth.DEEP_REF_JD)
    r0, v0, c0 = (x.cpu().numpy() for x in sg.propagate(rec, dt, prec))
    flags = torch.full((n,), 255, dtype=torch.uint8, device=DEV)
    r, v, c = (x.cpu().numpy() for x in sg.propagate_elements(e, dt, prec, flags=flags, ref_jd=synth.DEEP_REF_JD))
    print(f"[gpu] fused members {kind} n={n} T={T} {prec} deep={int(deep.sum())}", flush=True)
    assert np.array_equal(c, c0)
    assert np.array_equal(flags.cpu().numpy(), rec.flags.cpu().numpy())
    assert np.array_equal(np.isnan(r), np.isnan(r0)) and np.array_equal(np.isnan(v), np.isnan(v0))
    tr, tv = TOL[prec]
    near = ~deep
    assert np.nanmax(np.abs(r[:, near] - r0[:, near]), initial=0.0) <= tr
    assert np.nanmax(np.abs(v[:, near] - v0[:, near]), initial=0.0) <= tv
    if prec == "fp64":
        assert np.nanmax(np.abs(r[:, deep] - r0[:, deep]), initial=0.0) <= 1e-6
        assert np.nanmax(np.abs(v[:, deep] - v0[:, deep]), initial=0.0) <= 1e-9
    elif prec == "mixed" and deep.any():
        rd, vd, cd = (x.cpu().numpy() for x in sg.propagate(rec, dt, "fp64"))
        check_mixed(r[:, deep], v[:, deep], c[deep], rd[:, deep], vd[:, deep], cd[deep], el[1, deep][:, None])
