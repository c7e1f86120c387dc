"""The polar iteration on matrices that need more steps than the usual 20 or
30, with several 16 x 16 tiles: the part that one workgroup does alone (up to
128 orbitals) and the part that is launched step by step.

Orbitals are orthonormal fields scaled down row by row to 1e-6 (no two
residual norms tie, so the pivots must be the oracle's).  phi_loc = U^T Phi
with U the polar factor, whose FP64 rounding is amplified by the condition
number at most: 1e6 x eps x 100 = 2e-8.
"""
import numpy as np
import pytest

from oracle import scdm_oracle as SO
from tests.test_gpu_scdm_shapes import _field, _run, lib  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [40, 64, 70, 128, 140, 260])
def test_slow_polar_iteration(lib, k):  # noqa: F811
    print("[gpu-case] scdm of %d orbitals, condition number 1e6" % k, flush=True)
    n = 16
    phi = _field(k, n, 7) * (10.0 ** (-6.0 * np.arange(k) / (k - 1)))[:, None, None, None]
    piv, loc, info = _run(lib, phi)
    assert info == 0
    ref, U, loc_ref = SO.scdm(phi, np.arange(n ** 3))
    assert np.array_equal(piv, ref)
    assert np.linalg.norm(loc - loc_ref) / np.linalg.norm(loc_ref) < 2e-8
