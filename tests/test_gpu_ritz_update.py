"""The block eigensolver's one-pass update (up to 16 vectors) and the separate one (more): after four
steps, with and without kept search directions, the returned residual norms come from F X carried
along by the update, so they equal those of the oracle's operator on the returned vectors.

Bars: FP64, 4 steps of sums over at most 64 vectors whose coefficients reach 10 (Cholesky form) give
below 1e-9 of |F| ~ 40; FP32 with one rounding of 2^-24 per stored value and step, 64 terms: 1e-3."""

import numpy as np
import pytest
import torch

import synth
from oracle import scf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("k", [1, 7, 8, 9, 15, 16, 17, 21, 22])
def test_residuals_are_those_of_the_vectors(k, prec):
    import paper_2405_01522_amd as ace
    n, h = 12, 0.5
    dt = torch.float64 if prec == "fp64" else torch.float32
    rng = np.random.default_rng(k)
    x = synth.coords(n, h)
    v = 0.5 * (x[:, None, None] ** 2 + 1.2 * x[None, :, None] ** 2 + 1.5 * x[None, None, :] ** 2)
    phi = torch.from_numpy(synth.mgs(rng.normal(size=(k, n, n, n)), h ** 3)).to("cuda", dt)
    ctx = ace.AceContext(n, h, dt)
    opts = ace.eig_opts(max_steps=4, tol=0.0, precond="kinetic", shift=1.0, sweeps=4)
    ev, rn, steps = ctx.fock_lowest_states(torch.from_numpy(v[None]).to("cuda", dt), phi, opts=opts)
    assert steps == 4
    p = phi.cpu().numpy().astype(np.float64)
    bar = 4e-8 if prec == "fp64" else 1e-3
    for i in range(k):
        r = scf.kinetic(p[i], h) + v * p[i] - ev[i] * p[i]
        assert abs(np.sqrt(np.sum(r * r) * h ** 3) - rn[i]) < bar
