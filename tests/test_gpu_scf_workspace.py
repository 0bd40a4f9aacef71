"""The SCF pieces share a workspace that a context keeps: what a call returns does not depend on
the calls before it, their sizes, or the stream they ran on (equal to the bit)."""

import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_calls_do_not_depend_on_earlier_ones(prec):
    import paper_2405_01522_amd as ace
    n, h = 16, 0.5
    dt = torch.float64 if prec == "fp64" else torch.float32
    rng = np.random.default_rng(5)
    x = synth.coords(n, h)
    v = torch.from_numpy(0.5 * (x[:, None, None] ** 2 + 1.3 * x[None, :, None] ** 2
                                + 1.7 * x[None, None, :] ** 2)[None]).to("cuda", dt)
    phi = torch.from_numpy(synth.mgs(rng.normal(size=(12, n, n, n)), h ** 3)).to("cuda", dt)
    opts = ace.eig_opts(max_steps=5, tol=0.0, precond="kinetic", shift=1.0, sweeps=4)

    def calls(ctx, k):
        p = phi[:k].clone()
        ev, rn, _ = ctx.fock_lowest_states(v, p, opts=opts)
        z = ctx.kinetic_precondition(phi[:k])
        vh = ctx.hartree_potential(ctx.scf_density(phi[:k]))
        return [ev, rn] + [t.cpu().numpy() for t in (p, z, vh)]

    fresh = {k: calls(ace.AceContext(n, h, dt), k) for k in (1, 6, 12)}
    used = ace.AceContext(n, h, dt)
    other = torch.cuda.Stream()
    for k in (6, 1, 12, 6):
        for a, b in zip(calls(used, k), fresh[k]):
            assert np.array_equal(a, b)
        other.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(other):
            got = calls(used, k)
        torch.cuda.current_stream().wait_stream(other)
        for a, b in zip(got, fresh[k]):
            assert np.array_equal(a, b)
