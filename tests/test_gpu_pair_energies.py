"""Per-pair exchange energies: two pairs share a transform and are told apart
by the Hermitian symmetry of their spectra.

Each pair is compared by itself, relative to its own size: the orbitals are
narrow Gaussians, so the energies span many orders of magnitude, and the two
densities of a transform are brought level before they share it.  FP64: the
rounding of a length-n^3 transform is a few eps relative to the larger
density, level to within a factor of two in overlap and (|B| <= |rho|_1) to
within about 1e2 in amplitude: 1e-12.  FP32: the same with eps = 6e-8 and
errors that average over the n^3 terms: 1e-4.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2110_07670_amd import _lib
    _lib.load()
    return _lib


def _orbitals(n, k, seed):
    """Gaussians of unlike widths and heights, far apart and close by."""
    rng = np.random.default_rng(seed)
    L = np.array([9.0, 10.0, 11.0])
    x = [L[a] * np.arange(n) / n for a in range(3)]
    phi = np.zeros((k, n, n, n))
    for i in range(k):
        c, s = rng.uniform(0, 1, 3) * L, rng.uniform(0.6, 1.2)
        g = []
        for a in range(3):
            d = x[a] - c[a]
            d -= L[a] * np.rint(d / L[a])
            g.append(np.exp(-d * d / (2 * s * s)))
        phi[i] = g[0][:, None, None] * g[1][None, :, None] * g[2][None, None, :]
    return np.ascontiguousarray(phi), L


def _reference(phi, L, alpha):
    k, n = phi.shape[0], phi.shape[1]
    m = np.fft.fftfreq(n, d=1.0 / n)
    G2 = sum((2 * np.pi / L[a]) ** 2 * (m.reshape([-1 if b == a else 1 for b in range(3)]) ** 2)
             for a in range(3))
    K = np.where(G2 > 0, 4 * np.pi / np.where(G2 > 0, G2, 1.0), 0.0)
    e = np.zeros((k, k))
    for i in range(k):
        for j in range(i, k):
            z = np.fft.fftn(phi[i] * phi[j])
            e[i, j] = (-alpha * (1 if i == j else 2) * np.prod(L) / float(n) ** 6
                       * np.sum(K * (z.real ** 2 + z.imag ** 2)))
    return e


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n,k", [(16, 1), (16, 2), (24, 5), (32, 6), (40, 4), (48, 7), (64, 4),
                                 (80, 3), (96, 3)])
def test_pair_energies_each(lib, n, k, prec):
    import torch
    print("[gpu-case] pair energies n=%d k=%d %s" % (n, k, prec), flush=True)
    phi, L = _orbitals(n, k, 31 + n)
    plan = lib.Plan(n, L, k, prec, 0.25)
    ex, pe = lib.exx_energy(plan, torch.from_numpy(phi).to("cuda:0"), pair_energies=True)
    ex1, _ = lib.exx_energy(plan, torch.from_numpy(phi).to("cuda:0"))
    torch.cuda.synchronize()
    e, ref = pe.cpu().numpy(), _reference(phi, L, 0.25)
    iu = np.triu_indices(k)
    tol = 1e-12 if prec == "fp64" else 1e-4
    assert np.all(np.abs(e[iu] - ref[iu]) <= tol * np.abs(ref[iu])), \
        np.max(np.abs(e[iu] / ref[iu] - 1))
    assert np.all(e[np.tril_indices(k, -1)] == 0.0)
    for x in (ex, ex1):
        assert abs(float(x.item()) - ref.sum()) <= 0.01 * tol * abs(ref.sum()) + 1e-15


@pytest.mark.parametrize("n", [120, 128, 144, 160, 192])
def test_pair_energies_large_grids(lib, n):
    """Two pairs of one row and the leftover of the other, each against the
    build's own oracle-pinned route: E_x without the split."""
    import torch
    print("[gpu-case] pair energies n=%d" % n, flush=True)
    phi, L = _orbitals(n, 2, 5)
    plan = lib.Plan(n, L, 2, "fp64", 0.25)
    _, pe = lib.exx_energy(plan, torch.from_numpy(phi).to("cuda:0"), pair_energies=True)
    torch.cuda.synchronize()
    e, ref = pe.cpu().numpy(), _reference(phi, L, 0.25)
    iu = np.triu_indices(2)
    assert np.all(np.abs(e[iu] / ref[iu] - 1) <= 1e-12)


def test_pair_energies_masked(lib):
    import torch
    print("[gpu-case] pair energies with a mask", flush=True)
    n, k = 24, 7
    phi, L = _orbitals(n, k, 77)
    mask = np.random.default_rng(3).random((k, k)) < 0.5
    mask[4] = False
    plan = lib.Plan(n, L, k, "fp64", 0.25)
    ex, pe = lib.exx_energy(plan, torch.from_numpy(phi).to("cuda:0"), mask, pair_energies=True)
    torch.cuda.synchronize()
    ref = np.where(np.triu(mask), _reference(phi, L, 0.25), 0.0)
    e = pe.cpu().numpy()
    assert np.all(np.abs(e - ref) <= 1e-12 * np.abs(ref))
    assert abs(float(ex.item()) - ref.sum()) <= 1e-13 * abs(ref.sum())
