"""SCDM at the edges of its kernels' shapes: orbital counts around the 64
values of a column that a lane row holds, fewer columns than workgroups, and
a polar iteration that does not end within the launched iterations.

Orbitals are seeded normal fields (orthonormalised, or scaled row by row), so
no two residual norms tie; the pivots must be the oracle's.  phi_loc = U^T Phi
with U the polar factor: FP64 rounding of the factor is amplified by at most
the condition number of A_C (a normal matrix of k columns: below 1e4 here, so
1e-10 as elsewhere; the scaled case 1e6, so 1e6 x eps x 100 = 2e-8).
"""
import numpy as np
import pytest

from oracle import scdm_oracle as SO

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2110_07670_amd import _lib
    _lib.load()
    return _lib


def _run(lib, phi, points=None):
    import torch
    k, n = phi.shape[0], phi.shape[1]
    plan = lib.Plan(n, (8.0,) * 3, k)
    pts = None if points is None else torch.from_numpy(points.astype(np.int32)).to("cuda:0")
    piv, loc, info = lib.scdm_localize(plan, torch.from_numpy(phi).to("cuda:0"), pts)
    torch.cuda.synchronize()
    return piv.cpu().numpy().astype(np.int64), loc.cpu().numpy(), int(info.item())


def _field(k, n, seed):
    x = np.random.default_rng(seed).standard_normal((n ** 3, k))
    q, _ = np.linalg.qr(x)
    return np.ascontiguousarray(q.T).reshape(k, n, n, n)


@pytest.mark.parametrize("k,m", [(1, 1), (1, 700), (3, 7), (63, 4096), (64, 100), (65, 65),
                                 (130, 901), (257, 4096), (300, 321)])
def test_scdm_orbital_counts(lib, k, m):
    print("[gpu-case] scdm k=%d points=%d" % (k, m), flush=True)
    n = 16
    phi = _field(k, n, 100 + k)
    pts = np.sort(np.random.default_rng(k).permutation(n ** 3)[:m])
    piv, loc, info = _run(lib, phi, None if m == n ** 3 else pts)
    assert info == 0
    ref, U, loc_ref = SO.scdm(phi, pts)
    assert np.array_equal(piv, ref)
    assert np.linalg.norm(loc - loc_ref) / np.linalg.norm(loc_ref) < 1e-10


def test_scdm_slow_polar_iteration(lib):
    print("[gpu-case] scdm with a condition number of 1e6", flush=True)
    k, n = 12, 16
    phi = _field(k, n, 7) * (10.0 ** (-6.0 * np.arange(k) / (k - 1)))[:, None, None, None]
    pts = np.arange(n ** 3)
    piv, loc, info = _run(lib, phi)
    assert info == 0
    ref, U, loc_ref = SO.scdm(phi, pts)
    assert np.array_equal(piv, ref)
    assert np.linalg.norm(loc - loc_ref) / np.linalg.norm(loc_ref) < 2e-8
