"""The XY pass of launches with at most one plane per CU (whole planes) gives the bits of larger ones
(planes by halves), at the edges with both forms, on both sides of the rule: pair potentials from a
short list equal those of the same pairs at the head of a longer one, and the oracle's.

Bars: as for the halves themselves, 1e-13 and 5e-6 of the largest value in a transform (six
transforms of length P: about 40 roundings)."""

import numpy as np
import pytest
import torch

from oracle import poisson

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,dtype", [
    (56, torch.complex64), (64, torch.complex64), (56, torch.float32), (64, torch.float32),
    (40, torch.complex128), (48, torch.complex128), (40, torch.float64), (48, torch.float64),
    (56, torch.float64), (64, torch.complex128)])
def test_short_lists_give_the_bits_of_long_ones(n, dtype):
    import paper_2405_01522_amd as ace
    h = 0.25
    rng = np.random.default_rng(800 + n)
    a = rng.normal(size=(3, n, n, n))
    if dtype.is_complex:
        a = a + 1j * rng.normal(size=a.shape)
    phi = torch.from_numpy(a).to("cuda", dtype)
    ctx = ace.AceContext(n, h, dtype)
    pairs = [[j, i] for j in range(3) for i in range(3)] * 2
    long = ctx.pair_poisson_batched(phi, phi, pairs)
    # 1 to 4 transforms; real storage packs two pairs into one
    for count in ((1, 2, 3, 4) if dtype.is_complex else (2, 4, 6, 8)):
        assert torch.equal(ctx.pair_poisson_batched(phi, phi, pairs[:count]), long[:count]), count
    ref_phi = phi.cpu().numpy().astype(np.complex128 if dtype.is_complex else np.float64)
    khat = poisson.kernel_hat(n, h)
    refs = [poisson.fft(np.conj(ref_phi[j]) * ref_phi[i], h, khat) for j, i in pairs[:2]]
    got = long[:2].cpu().numpy()
    tol = (1e-13 if dtype in (torch.complex128, torch.float64) else 5e-6) * np.abs(refs).max()
    assert np.abs(got - np.array(refs)).max() < tol
    ctx.close()
