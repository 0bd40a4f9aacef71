"""The one-workgroup symmetric eigensolver over its orders (1 to 64: odd ones carry a padding
index; block counts on both sides of whole wavefronts), spectra and magnitudes, against numpy.

Bar: every sweep passes each entry through n - 1 rotations of a few roundings each; 10 sweeps of
n rounds with 4 eps give a backward error and a loss of orthogonality below 40 n eps."""

import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _spectrum(kind, n, rng):
    if kind == "random":
        return rng.normal(size=n)
    if kind == "clusters":
        return 1.0 + np.arange(n) // 3 + 1e-13 * (np.arange(n) % 3)
    return 10.0 ** (-12.0 * np.arange(n) / n)  # graded


@pytest.mark.parametrize("kind", ["random", "clusters", "graded"])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 11, 15, 16, 17, 22, 23, 31, 32, 33, 47, 48, 49, 63, 64])
def test_against_numpy(n, kind):
    from paper_2405_01522_amd._lib import lib
    rng = np.random.default_rng(17 * n + len(kind))
    q, _ = np.linalg.qr(rng.normal(size=(n, n)))
    a = (q * _spectrum(kind, n, rng)) @ q.T
    a = 0.5 * (a + a.T)
    lda, ldv = n + 1, n + 2
    bar = 40 * n * 2.0 ** -52
    fn = lib().sym_eig_small
    for scale in (1.0, 1e145, 1e-145):  # the last two: outside the squares' safe range
        buf = torch.full((n, lda), float("nan"), dtype=torch.float64)
        buf[:, :n] = torch.from_numpy(a * scale)
        A = buf.cuda()
        w = torch.empty(n, dtype=torch.float64, device="cuda")
        V = torch.full((n, ldv), 7.0, dtype=torch.float64, device="cuda")
        p = ctypes.c_void_p
        assert fn(n, p(A.data_ptr()), lda, p(w.data_ptr()), p(V.data_ptr()), ldv, None) == 0
        torch.cuda.synchronize()
        ev, vec = w.cpu().numpy() / scale, V.cpu().numpy()
        assert np.all(vec[:, n:] == 7.0)
        vec = vec[:, :n]
        norm = np.abs(np.linalg.eigvalsh(a)).max()
        assert np.all(np.diff(ev) >= 0)
        assert np.abs(ev - np.linalg.eigvalsh(a)).max() <= bar * norm
        assert np.linalg.norm(a @ vec - vec * ev, 2) <= bar * norm
        assert np.linalg.norm(vec.T @ vec - np.eye(n), 2) <= bar
