"""The FP64 matrix products behind ace_apply and the overlap integrals, at the
edges of their tile shapes, against numpy.

Tolerance: every output is a sum of at most N k products of order-one normals
in FP64; the normwise relative error of such sums in any order is below
sqrt(N + k) eps times a small constant, 4096 points and 512 orbitals: 2e-14.
The bound here is 1e-12.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
TOL = 1e-12


@pytest.fixture(scope="module")
def lib():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2110_07670_amd import _lib
    _lib.load()
    return _lib


def _normal(shape, seed, shift):
    """Normals on the device; shift: the tensor starts 8 bytes past an
    allocation (contiguous, but only 8-byte aligned)."""
    import torch
    x = np.random.default_rng(seed).standard_normal(shape)
    buf = torch.empty(x.size + 1, dtype=torch.float64, device="cuda:0")
    t = buf[1:].view(shape) if shift else buf[:-1].view(shape)
    t.copy_(torch.from_numpy(x))
    return x.reshape(shape[0], -1), t


def _rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("shift", [False, True], ids=["aligned", "8_byte_aligned"])
@pytest.mark.parametrize("k,n_vec", [(1, 1), (5, 16), (16, 17), (17, 3), (32, 33), (40, 64),
                                     (64, 65), (65, 40), (100, 130), (128, 9), (129, 128),
                                     (200, 31), (257, 20), (300, 70), (512, 5)])
def test_apply_product_shapes(lib, k, n_vec, shift):
    import torch
    print("[gpu-case] apply k=%d n_vec=%d shift=%s" % (k, n_vec, shift), flush=True)
    n = 16
    plan = lib.Plan(n, (7.0, 8.0, 9.0), k)
    xi, xi_d = _normal((k, n, n, n), 1, shift)
    psi, psi_d = _normal((n_vec, n, n, n), 2, shift)
    _, out = _normal((n_vec, n, n, n), 3, shift)
    ws = lib.workspace(plan.apply_workspace_bytes(n_vec))
    lib.apply_into(plan, xi_d, psi_d, out, ws)
    torch.cuda.synchronize()
    dV = 7.0 * 8.0 * 9.0 / n ** 3
    ref = -(dV * (psi @ xi.T)) @ xi
    assert _rel(out.cpu().numpy().reshape(n_vec, -1), ref) < TOL


@pytest.mark.parametrize("shift", [False, True], ids=["aligned", "8_byte_aligned"])
@pytest.mark.parametrize("k", [1, 16, 33, 64, 100, 130, 260])
def test_overlap_integral_shapes(lib, k, shift):
    import torch
    print("[gpu-case] overlaps k=%d shift=%s" % (k, shift), flush=True)
    n = 16
    plan = lib.Plan(n, (7.0, 8.0, 9.0), k)
    phi, phi_d = _normal((k, n, n, n), 4, shift)
    S = lib.overlap_integrals(plan, phi_d)
    torch.cuda.synchronize()
    S = S.cpu().numpy()
    ref = (7.0 * 8.0 * 9.0 / n ** 3) * (np.abs(phi) @ np.abs(phi).T)
    assert _rel(S, ref) < TOL
    assert np.array_equal(S, S.T) or _rel(S, S.T) < 1e-15
