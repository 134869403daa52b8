"""The flat ragged kernel with one chunk per wavefront (a grid that covers every
chunk) and with its loop (a plan held to one wavefront per compute unit), at
edges of the 64-point chunk and the four-wavefront workgroup, against the
oracle: FP64 within 1e-8 km and 1e-11 km/s, mixed within 5 m and 5 mm/s (the
bars of ragged propagation everywhere)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2603_27830_amd as sg
import synth

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")
TOL = {"fp64": (1e-8, 1e-11), "mixed": (5e-3, 5e-6)}


@pytest.mark.parametrize("nnz", [1, 63, 64, 65, 255, 256, 257, 1025, 70_001])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_once_and_loop_match_the_oracle(nnz, prec):
    n = max(1, nnz // 50)
    rng = np.random.default_rng(nnz)
    el = synth.shell_elements(n, nnz)
    cuts = np.sort(rng.integers(0, nnz + 1, n - 1))  # empty lists among them
    off = np.concatenate([[0], cuts, [nnz]]).astype(np.int64)
    t = rng.uniform(0.0, 1440.0, nnz)
    r0, v0, c0 = oracle.propagate_ragged(el, off, t)[:3]
    rec = sg.init(torch.from_numpy(el).to(DEV))
    do, dt = torch.from_numpy(off).to(DEV), torch.from_numpy(t).to(DEV)
    plan = sg.RaggedPlan(rec, do, dt, prec, autotune=False, graph=False, config=(1, 256, 1))
    print(f"[gpu] flat once/loop nnz={nnz} {prec}", flush=True)
    for r, v, c in (sg.propagate_ragged(rec, do, dt, prec), plan.launch()):
        assert np.array_equal(c.cpu().numpy(), c0)
        assert np.abs(r.cpu().numpy() - r0).max() <= TOL[prec][0]
        assert np.abs(v.cpu().numpy() - v0).max() <= TOL[prec][1]
