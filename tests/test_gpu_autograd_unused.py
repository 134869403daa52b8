"""Autograd with one of the two outputs unused: its cotangent is absent, not
zeros.  The gradients of r alone and of v alone add up to that of both; the
kernels sum in the same order, so each component agrees to 64 half-ulps of the
parts' magnitudes (fewer than 64 points per satellite, one addition each)."""
import pytest
import torch

import paper_2603_27830_amd as sg
import synth

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("ragged", [False, True])
def test_gradients_of_the_parts_add_up(ragged):
    n, T = 37, 20
    el = torch.from_numpy(synth.shell_elements(n, 4)).to(DEV).requires_grad_()
    t = torch.linspace(0.0, 300.0, T, dtype=torch.float64, device=DEV)
    gen = torch.Generator(device=DEV).manual_seed(1)

    def call():
        if ragged:
            off = torch.arange(n + 1, dtype=torch.int64, device=DEV) * T
            return sg.SGP4RaggedFunction.apply(el, off, t.repeat(n), "fp64")
        return sg.SGP4Function.apply(el, t, "fp64")

    r, v, _ = call()
    wr, wv = (torch.randn(x.shape, dtype=x.dtype, device=DEV, generator=gen) for x in (r, v))
    gr, = torch.autograd.grad((r * wr).sum(), el)
    r, v, _ = call()
    gv, = torch.autograd.grad((v * wv).sum(), el)
    r, v, _ = call()
    both, = torch.autograd.grad((r * wr).sum() + (v * wv).sum(), el)
    assert gr.shape == (8, n) and (gr[7] == 0).all() and (gv[7] == 0).all() and gv[:7].abs().sum() > 0
    rec = sg.init(el.detach())
    scale = 0.0
    for k in range(3):  # magnitude of the parts, summed without cancellation
        for w, i in ((wr, 0), (wv, 3)):
            j = sg.jacobian(rec, t)[i + k] * w[k].reshape(n, T)
            scale = scale + j.abs().sum(-1)
    assert ((gr + gv - both).abs()[:7] <= 64 * 2.0 ** -53 * scale).all()
