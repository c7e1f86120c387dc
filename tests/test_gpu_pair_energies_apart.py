"""FP64 per-pair energies where the two pairs of a transform must not show in
each other: a NaN or an infinity in one orbital, densities that vanish or are
far smaller; and pairs that go alone where sharing does not pay.

Every pair is what it is by itself: NaN where its own density is not finite,
exactly zero where its density is, and elsewhere numpy's value to 1e-12 (the
bound of the ordinary pairs: a few eps of a transform whose two densities are
level).
"""
import numpy as np
import pytest

from tests.test_gpu_pair_energies import _orbitals, _reference, lib  # noqa: F401

pytestmark = pytest.mark.gpu


def _pairs(lib, phi, L):
    import torch
    plan = lib.Plan(phi.shape[1], L, phi.shape[0], "fp64", 0.25)
    _, pe = lib.exx_energy(plan, torch.from_numpy(phi).to("cuda:0"), pair_energies=True)
    torch.cuda.synchronize()
    return pe.cpu().numpy()


@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("k,where", [(5, 3), (6, 0), (24, 7)])
def test_not_finite_orbital(lib, k, where, bad):  # noqa: F811
    print("[gpu-case] pair energies with %s in orbital %d of %d" % (bad, where, k), flush=True)
    phi, L = _orbitals(32, k, 9)
    ref = _reference(phi, L, 0.25)
    phi[where, 1, 2, 3] = bad
    e = _pairs(lib, phi, L)
    own = np.zeros((k, k), dtype=bool)
    own[where] = own[:, where] = True
    iu = np.triu_indices(k)
    assert np.all(np.isnan(e[iu]) == own[iu])
    ok = np.triu(~own)
    assert np.all(np.abs(e[ok] - ref[ok]) <= 1e-12 * np.abs(ref[ok]))


def test_vanishing_densities(lib):  # noqa: F811
    """Orbitals on slabs that do not meet: their pairs' energies are zero."""
    print("[gpu-case] pair energies of orbitals that do not meet", flush=True)
    n, k = 32, 24
    phi, L = _orbitals(n, k, 4)
    for i in range(k):
        keep = np.zeros(n, dtype=bool)
        keep[np.arange(8) + 8 * (i % 4)] = True
        phi[i, ~keep] = 0.0
    e, ref = _pairs(lib, phi, L), _reference(phi, L, 0.25)
    iu = np.triu_indices(k)
    apart = (iu[0] % 4) != (iu[1] % 4)
    assert np.all(e[iu][apart] == 0.0)
    assert np.all(np.abs(e[iu][~apart] - ref[iu][~apart]) <= 1e-12 * np.abs(ref[iu][~apart]))


def test_far_smaller_pairs(lib):  # noqa: F811
    """Narrow orbitals along a line: overlaps from 1 down to 1e-140, energies
    down to 1e-280, each to 1e-12 of itself."""
    print("[gpu-case] pair energies down to 1e-280", flush=True)
    n, k, width = 48, 12, 0.75
    L = np.array([90.0, 18.0, 18.0])
    x = [L[a] * np.arange(n) / n for a in range(3)]
    phi = np.zeros((k, n, n, n))
    # neighbours in the list share a transform: 0.3 of the cell apart at most, so
    # that the images lie farther
    for i, place in enumerate((0, 4, 1, 3, 2, 2.5, 0.5, 3.5, 1.5, 0.25, 3.75, 2.25)):
        c = np.array([0.075 * place * L[0], 9.0, 9.0])
        g = [np.exp(-((x[a] - c[a] - L[a] * np.rint((x[a] - c[a]) / L[a])) / width) ** 2 / 2)
             for a in range(3)]
        phi[i] = g[0][:, None, None] * g[1][None, :, None] * g[2][None, None, :]
    e, ref = _pairs(lib, phi, L), _reference(phi, L, 0.25)
    iu = np.triu_indices(k)
    assert np.abs(ref[iu]).min() < 1e-270 and np.all(ref[iu] != 0.0)
    assert np.all(np.abs(e[iu] - ref[iu]) <= 1e-12 * np.abs(ref[iu])), e[iu] / ref[iu] - 1


@pytest.mark.parametrize("n,k", [(16, 54), (24, 30), (32, 20), (40, 16), (48, 12), (64, 9),
                                 (80, 7), (96, 6), (120, 5), (128, 5), (144, 4), (160, 4),
                                 (192, 4)])
def test_shared_transforms(lib, n, k):  # noqa: F811
    """Two pairs per transform on every grid (rows of even and odd length)."""
    print("[gpu-case] shared pair energies n=%d k=%d" % (n, k), flush=True)
    phi, L = _orbitals(n, k, 100 + n)
    plan = lib.Plan(n, L, k, "fp64", 0.25)
    assert _stage_counts(lib, plan, phi)[7] == 3
    e, ref = _pairs(lib, phi, L), _reference(phi, L, 0.25)
    iu = np.triu_indices(k)
    assert np.all(np.abs(e[iu] - ref[iu]) <= 1e-12 * np.abs(ref[iu]))


def _stage_counts(lib, plan, phi, mask=None):
    import torch
    plan.set_profiling(True)
    lib.exx_energy(plan, torch.from_numpy(phi).to("cuda:0"), mask, pair_energies=True)
    plan.set_profiling(False)
    return [count for _, count in plan.profile_read().values()]


@pytest.mark.parametrize("kind", ["few_orbitals", "diagonal", "few_pairs"])
def test_alone_where_sharing_does_not_pay(lib, kind):  # noqa: F811
    """No overlap integrals (a third stage-7 entry beside the tables and the
    sum) where few or no transforms would be saved."""
    print("[gpu-case] pair energies alone: %s" % kind, flush=True)
    n, k = (48, 3) if kind == "few_orbitals" else (48, 24)
    phi, L = _orbitals(n, k, 12)
    mask = None
    if kind == "diagonal":
        mask = np.eye(k, dtype=bool)
    if kind == "few_pairs":
        mask = np.zeros((k, k), dtype=bool)
        mask[2, 5:9] = mask[7, 11:14] = True
    plan = lib.Plan(n, L, k, "fp64", 0.25)
    assert _stage_counts(lib, plan, phi, mask)[7] == 2
    import torch
    _, pe = lib.exx_energy(plan, torch.from_numpy(phi).to("cuda:0"), mask, pair_energies=True)
    torch.cuda.synchronize()
    e = pe.cpu().numpy()
    ref = _reference(phi, L, 0.25)
    ref = np.where(np.triu(np.ones((k, k)) if mask is None else mask), ref, 0.0)
    assert np.all(np.abs(e - ref) <= 1e-12 * np.abs(ref))
