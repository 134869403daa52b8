"""The fused elements-to-states launch over its workgroups: satellites at the
edges of 64, times split over the grid's second extent, and deep-space,
simplified-drag and invalid members among near-Earth ones (the deep-space ones
are propagated apart from the others), against the two-stage path.

Bars: codes and satellite flags equal; states to rounding, as for the fused call
everywhere (FP64 1e-8 km and 1e-11 km/s, the float paths 5 m and 5 mm/s), and
for the deep-space members the float paths' accuracy of 10 m and 1e-2 m/s.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2603_27830_amd as sg
import synth

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")
TOL = {"fp64": (1e-8, 1e-11), "mixed": (5e-3, 5e-6), "fp32": (5e-3, 5e-6)}


def mixture(n, seed):
    el = synth.shell_elements(n, seed)
    rng = np.random.default_rng(seed)
    kind = rng.integers(0, 8, n)
    deep = kind == 0
    el[:, deep] = synth.config5(max(n, 64), 1).elem[:, :n][:, deep]
    el[0, kind == 1] = oracle.ke() * ((6378.135 + 200.0) / 6378.135) ** -1.5
    el[1, kind == 2] = 1.25
    el[0, kind == 3] *= -1.0 if seed % 2 else 1.0
    return el, deep


@pytest.mark.parametrize("n,T", [(1, 2), (63, 3), (64, 19), (65, 32), (129, 7), (1000, 2), (5, 1300), (70, 300),
                                 (66_000, 3)])
@pytest.mark.parametrize("prec", ["fp64", "mixed", "fp32"])
def test_fused_groups_match_two_stage_path(n, T, prec):
    el, deep = mixture(n, n + T)
    t = np.sort(np.random.default_rng(T).uniform(-600.0, 4000.0, T))
    e, dt = torch.from_numpy(el).to(DEV), torch.from_numpy(t).to(DEV)
    rec = sg.init(e, ref_jd=synth.DEEP_REF_JD)
    r0, v0, c0 = (x.cpu().numpy() for x in sg.propagate(rec, dt, prec))
    flags = torch.full((n,), 255, dtype=torch.uint8, device=DEV)
    r, v, c = (x.cpu().numpy() for x in sg.propagate_elements(e, dt, prec, flags=flags, ref_jd=synth.DEEP_REF_JD))
    print(f"[gpu] fused groups n={n} T={T} {prec} deep={int(deep.sum())}", flush=True)
    assert np.array_equal(c, c0)
    assert np.array_equal(flags.cpu().numpy(), rec.flags.cpu().numpy())
    assert np.array_equal(np.isnan(r), np.isnan(r0)) and np.array_equal(np.isnan(v), np.isnan(v0))
    tr, tv = TOL[prec]
    near = ~deep
    assert np.nanmax(np.abs(r[:, near] - r0[:, near]), initial=0.0) <= tr
    assert np.nanmax(np.abs(v[:, near] - v0[:, near]), initial=0.0) <= tv
    if deep.any() and prec != "fp32":
        tr, tv = (1e-6, 1e-9) if prec == "fp64" else (1e-2, 1e-5)
        assert np.nanmax(np.abs(r[:, deep] - r0[:, deep]), initial=0.0) <= tr
        assert np.nanmax(np.abs(v[:, deep] - v0[:, deep]), initial=0.0) <= tv
