"""FP64 VJP and Jacobian over lists of very different lengths: long ones side by
side, at the end, and alone among empty ones, in batches whose groups hold several
satellites.

Bars as for the grouped calls: 1e-8 relative per satellite for the VJP and 1e-8 of
each column's scale for the Jacobian against the oracle's dual numbers.
"""
import numpy as np
import pytest

import oracle
import paper_2603_27830_amd as sg
import synth
from test_gpu_grad_groups import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,first,count,length,rest", [(9341, 100, 16, 700, 3), (8193, 8189, 4, 500, 1), (2049, 0, 1, 3000, 0),
                                                       (16_385, 5000, 9, 200, 0), (3000, 2998, 2, 1, 0)])
def test_long_lists_side_by_side(n, first, count, length, rest):
    el = synth.shell_elements(n, n)
    lens = np.full(n, rest)
    lens[first:first + count] = length
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    rng = np.random.default_rng(n)
    t = rng.uniform(-500.0, 3000.0, off[-1])
    gr, gv = rng.normal(size=(3, t.size)), rng.normal(size=(3, t.size)) * 1e3
    rec = sg.init(dev(el))
    got = sg.vjp_ragged(rec, dev(off), dev(t), dev(gr), dev(gv), "fp64").cpu().numpy()
    J = sg.jacobian_ragged(rec, dev(off), dev(t), "fp64").cpu().numpy()
    print(f"[gpu] lists n={n}: {count} of {length}", flush=True)
    assert np.all(got[:, lens == 0] == 0.0) and np.isfinite(got).all() and np.isfinite(J).all()
    # what the Jacobian says the VJP is, for every satellite
    per = np.einsum("rmp,rp->mp", J, np.concatenate([gr, gv]))
    owner = np.repeat(np.arange(n), lens)
    want = np.array([np.bincount(owner, w, minlength=n) for w in per])
    size = np.array([np.bincount(owner, np.abs(w), minlength=n) for w in per])
    assert (np.abs(got - want) <= 1e-9 * size + 1e-300).all()
    sample = np.unique(np.concatenate([np.arange(first, first + count)[:3], [0, n - 1, min(first + count, n - 1)]]))
    pick = np.concatenate([np.arange(off[i], off[i + 1]) for i in sample])
    o = np.concatenate([[0], np.cumsum(lens[sample])]).astype(np.int64)
    ref = oracle.vjp_ragged(el[:, sample], o, t[pick], gr[:, pick], gv[:, pick])
    use = lens[sample] > 0
    a, b = got[:, sample][:, use], ref[:, use]
    scale = np.median(np.abs(b), axis=1, keepdims=True)
    assert np.max(np.linalg.norm((a - b) / scale, axis=0) / np.linalg.norm(b / scale, axis=0)) <= 1e-8
