"""FP32 coupling blocks at the edges of the contraction's tiles (128 rows, pieces of 32 and 16 rows,
steps of 64 points), against the oracle.

Grids: 9^3 (single loads, the last of 12 steps holds 25 points) and 10^3 (16-byte loads, the last
of 16 steps holds 40 points).  Bar: the operands are split into two BF16 parts whose lowest product,
below 2^-17 of the product, is dropped; sums of magnitudes are within 4 times the largest entry
here, so 2^-15 of that covers them and the FP32 sums."""

import numpy as np
import pytest
import torch

import synth
from oracle import tda

pytestmark = pytest.mark.gpu


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda", torch.float32)


# rows and columns of the two contractions: no nv squared, no (no + 1) / 2 by nv (nv + 1) / 2
@pytest.mark.parametrize("n", [9, 10])
@pytest.mark.parametrize("no,nv", [(1, 1), (2, 15), (4, 32), (3, 43), (16, 2)])
def test_coupling_blocks(n, no, nv):
    import paper_2405_01522_amd as ace
    h = 0.5
    m = synth.small_real(7 * n + no, n, h, no, nv)
    ctx = ace.AceContext(n, h, torch.float32)
    c, b = ctx.tdhf_coupling(_t(m.phi), _t(m.phi_virt), 2)
    cr = tda.coupling_block(m.phi, m.phi_virt, h, 2)
    br = tda.b_block(m.phi, m.phi_virt, h, 2)
    bar = 2.0 ** -15 * max(np.abs(cr).max(), np.abs(br).max())
    assert np.abs(c.cpu().numpy() - cr).max() < bar
    assert np.abs(b.cpu().numpy() - br).max() < bar


@pytest.mark.parametrize("n", [9, 10])
def test_uhf_blocks(n):
    import paper_2405_01522_amd as ace
    h = 0.5
    a, b = synth.small_real(3 * n, n, h, 3, 43), synth.small_real(5 * n, n, h, 2, 12)
    ctx = ace.AceContext(n, h, torch.float32)
    c, bb = ctx.uhf_coupling(_t(a.phi), _t(a.phi_virt), _t(b.phi), _t(b.phi_virt))
    cr, br = tda.uhf_blocks(a.phi, a.phi_virt, b.phi, b.phi_virt, h)
    bar = 2.0 ** -15 * max(np.abs(cr).max(), np.abs(br).max())
    assert np.abs(c.cpu().numpy() - cr).max() < bar
    assert np.abs(bb.cpu().numpy() - br).max() < bar
