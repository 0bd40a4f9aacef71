"""Pair potentials at the box edges whose XY pass works a plane by halves (FP32 storage from
edge 56, FP64 from edge 40) and at the edges on either side of that rule, against the FP64
oracle, with an odd number of pairs so that real storage leaves one pair without a partner.

Bars (max-norm relative): a convolution is six transforms of length P, i.e. about
6 log2(P) ~ 40 roundings on any path, which accumulate like their square root for random data:
~1e-15 in FP64 and ~4e-7 in FP32 against the largest value in the transform, which for real
storage is that of the two potentials that share it (pairs 0 and 1 here, the second one 100 times
larger).  The bars leave a factor of about ten on the worst element: 1e-13 and 5e-6.
"""

import numpy as np
import pytest
import torch

from oracle import poisson

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,dtype", [
    (48, torch.complex64), (56, torch.complex64), (64, torch.complex64),
    (48, torch.float32), (56, torch.float32), (64, torch.float32),
    (32, torch.complex128), (40, torch.complex128), (48, torch.complex128),
    (56, torch.complex128), (64, torch.complex128),
    (32, torch.float64), (40, torch.float64), (48, torch.float64), (56, torch.float64),
    (64, torch.float64)])
def test_pair_potentials(n, dtype):
    import paper_2405_01522_amd as ace
    h = 0.25
    rng = np.random.default_rng(700 + n)
    a = rng.normal(size=(2, n, n, n))
    if dtype.is_complex:
        a = a + 1j * rng.normal(size=a.shape)
    phi = torch.from_numpy(a).to("cuda", dtype)
    ref_phi = phi.cpu().numpy().astype(np.complex128 if dtype.is_complex else np.float64)
    ctx = ace.AceContext(n, h, dtype)
    pairs = [[0, 1], [1, 1], [1, 0]]
    v = ctx.pair_poisson_batched(phi, phi, pairs).cpu().numpy()
    khat = poisson.kernel_hat(n, h)
    tol = 1e-13 if dtype in (torch.complex128, torch.float64) else 5e-6
    refs = [poisson.fft(np.conj(ref_phi[j]) * ref_phi[i], h, khat) for j, i in pairs]
    scale = [np.max(np.abs(r)) for r in refs]
    if not dtype.is_complex:
        scale[0] = scale[1] = max(scale[0], scale[1])
    for p, ref in enumerate(refs):
        err = np.max(np.abs(v[p] - ref)) / scale[p]
        assert err < tol, (n, dtype, p, err)
    ctx.close()
