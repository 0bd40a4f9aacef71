"""FP32 coupling blocks whose contractions have more (tile, chunk) items than the device has CUs, so
that a workgroup works several in turn: chunks of one whole step, and the last one partial (15^3
points: 53 steps, the last of 47 points), against the oracle.

Bar: as for blocks of one item each, 2^-15 of the largest entry (operands split into two BF16 parts,
the product of the low parts left out, sums of magnitudes within 4 times the largest entry)."""

import numpy as np
import pytest
import torch

import synth
from oracle import tda

pytestmark = pytest.mark.gpu


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda", torch.float32)


@pytest.mark.parametrize("n,no,nv", [(16, 8, 32), (15, 8, 32), (15, 3, 43)])
def test_coupling_blocks(n, no, nv):
    import paper_2405_01522_amd as ace
    h = 0.4
    m = synth.small_real(11 * n + no, n, h, no, nv)
    ctx = ace.AceContext(n, h, torch.float32)
    c, b = ctx.tdhf_coupling(_t(m.phi), _t(m.phi_virt), 2)
    cr = tda.coupling_block(m.phi, m.phi_virt, h, 2)
    br = tda.b_block(m.phi, m.phi_virt, h, 2)
    bar = 2.0 ** -15 * max(np.abs(cr).max(), np.abs(br).max())
    assert np.abs(c.cpu().numpy() - cr).max() < bar
    assert np.abs(b.cpu().numpy() - br).max() < bar


def test_uhf_blocks():
    import paper_2405_01522_amd as ace
    n, h = 15, 0.4
    a, b = synth.small_real(31, n, h, 3, 43), synth.small_real(32, n, h, 4, 32)
    ctx = ace.AceContext(n, h, torch.float32)
    c, bb = ctx.uhf_coupling(_t(a.phi), _t(a.phi_virt), _t(b.phi), _t(b.phi_virt))
    cr, br = tda.uhf_blocks(a.phi, a.phi_virt, b.phi, b.phi_virt, h)
    bar = 2.0 ** -15 * max(np.abs(cr).max(), np.abs(br).max())
    assert np.abs(c.cpu().numpy() - cr).max() < bar
    assert np.abs(bb.cpu().numpy() - br).max() < bar
