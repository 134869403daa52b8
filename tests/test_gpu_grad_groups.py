"""FP64 VJP and Jacobian over groups of satellites: list lengths at the edges of
the 64-point chunks, group sizes from one to eight with a partial last group,
and deep-space, simplified-drag, invalid and empty members inside a group.

Bars (as for the same calls on small batches): 1e-8 relative per satellite for
the VJP and 1e-8 of each column's scale for the Jacobian against the oracle's
dual numbers, on a sample of satellites that holds every list length, every
special member and the whole last group.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2603_27830_amd as sg
import synth

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")
LENGTHS = np.array([0, 1, 2, 63, 64, 65, 127, 128, 129, 7, 192, 193, 31])


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def batch(n, longest, seed):
    el = synth.config1(n, 1).elem.copy()
    rng = np.random.default_rng(seed)
    lens = LENGTHS[LENGTHS <= longest][rng.integers(0, (LENGTHS <= longest).sum(), n)]
    lens[:LENGTHS.size] = np.minimum(LENGTHS, longest)
    deep = rng.choice(n, 5, replace=False)
    el[:, deep] = synth.config5(64, 1).elem[:, :5]
    el[7, deep] = 0.0
    simple = np.setdiff1d(rng.choice(n, 6, replace=False), deep)
    el[0, simple] = oracle.ke() * ((6378.135 + 200.0) / 6378.135) ** -1.5
    invalid = np.setdiff1d(rng.choice(n, 3, replace=False), np.union1d(deep, simple))
    el[1, invalid] = 1.5
    offsets = np.zeros(n + 1, np.int64)
    offsets[1:] = np.cumsum(lens)
    t = np.concatenate([np.sort(rng.uniform(-500.0, 3000.0, L)) for L in lens])
    sample = np.unique(np.concatenate([np.arange(LENGTHS.size), deep, simple, invalid, np.arange(n - 9, n)]))
    return el, lens, offsets, t, deep, invalid, sample, rng


# (satellites, longest list): groups of one, two, four and eight
CASES = [(40, 193), (2051, 193), (5003, 129), (8201, 31), (9001, 2)]


@pytest.mark.parametrize("n,longest", CASES)
def test_grouped_vjp_matches_dual_oracle(n, longest):
    el, lens, offsets, t, deep, invalid, sample, rng = batch(n, longest, n)
    gr, gv = rng.normal(size=(3, t.size)), rng.normal(size=(3, t.size)) * 1e3
    rec = sg.init(dev(el))
    got = sg.vjp_ragged(rec, dev(offsets), dev(t), dev(gr), dev(gv), "fp64").cpu().numpy()
    assert np.all(np.isnan(got[:, deep]))
    assert np.all(got[:, invalid] == 0.0)
    assert np.all(got[:, np.setdiff1d(np.flatnonzero(lens == 0), deep)] == 0.0)
    pick = np.concatenate([np.arange(offsets[i], offsets[i + 1]) for i in sample])
    off = np.zeros(sample.size + 1, np.int64)
    off[1:] = np.cumsum(lens[sample])
    want = oracle.vjp_ragged(el[:, sample], off, t[pick], gr[:, pick], gv[:, pick])
    use = ~np.isin(sample, np.union1d(deep, invalid)) & (lens[sample] > 0)
    a, b = got[:, sample][:, use], want[:, use]
    scale = np.median(np.abs(b), axis=1, keepdims=True)
    worst = np.max(np.linalg.norm((a - b) / scale, axis=0) / np.linalg.norm(b / scale, axis=0))
    print(f"[gpu] grouped vjp n={n} longest={longest}: {worst:.2e}", flush=True)
    assert worst <= 1e-8
    again = sg.vjp_ragged(rec, dev(offsets), dev(t), dev(gr), dev(gv), "fp64").cpu().numpy()
    assert np.array_equal(got, again, equal_nan=True)


@pytest.mark.parametrize("n,longest", CASES)
def test_grouped_jacobian_matches_dual_oracle(n, longest):
    el, lens, offsets, t, deep, invalid, sample, rng = batch(n, longest, n + 1)
    rec = sg.init(dev(el))
    J = sg.jacobian_ragged(rec, dev(offsets), dev(t), "fp64").cpu().numpy()
    owner = np.repeat(np.arange(n), lens)
    lost = np.isin(owner, np.union1d(deep, invalid))
    assert np.all(np.isnan(J[:, :, lost])) and np.all(np.isfinite(J[:, :, ~lost]))
    pick = np.flatnonzero(np.isin(owner, sample) & ~lost)
    ref, _, _, err = oracle.jacobian_points(el, owner[pick], t[pick])
    assert np.all((err == 0) | (err == 6))
    ref = np.transpose(ref, (1, 2, 0))
    worst = (np.abs(J[:, :, pick] - ref).max(axis=2) / (np.abs(ref).max(axis=2) + 1e-300)).max()
    print(f"[gpu] grouped jacobian n={n} longest={longest}: {worst:.2e}", flush=True)
    assert worst <= 1e-8


@pytest.mark.parametrize("n,T", [(2051, 64), (2051, 65), (4099, 1), (1023, 257)])
def test_dense_grid_as_lists_is_the_grid_bit_for_bit(n, T):
    d = synth.config1(n, T)
    rng = np.random.default_rng(T)
    g = dev(rng.normal(size=(3, n, T)))
    rec, off, tt = sg.init(dev(d.elem)), dev(np.arange(n + 1, dtype=np.int64) * T), dev(np.tile(d.t, n))
    assert torch.equal(sg.vjp(rec, dev(d.t), g, None, "fp64"), sg.vjp_ragged(rec, off, tt, g.reshape(3, -1), None, "fp64"))
    assert torch.equal(sg.jacobian(rec, dev(d.t), "fp64").reshape(6, 7, -1), sg.jacobian_ragged(rec, off, tt, "fp64"))
