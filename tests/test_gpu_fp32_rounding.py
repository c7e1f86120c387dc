"""FP32 transforms round alike wherever they run: the potentials that the fused
inverse-z/W pass folds off the diagonal are, bit for bit, those of the
four-pass schedule, so the W rows differ only by the order of their FP64 sums.

The off-diagonal tile's share is W of 32 orbitals less W of the 16 orbitals of
each block alone, on either schedule.  Each row is a sum of 32 FP64 products,
so two orders agree to 32 eps of the largest, 7e-15; the difference of two
builds loses no more than that again: 1e-13 of the largest W.  A single FP32
rounding of a potential (6e-8 of it) shows at 1e-10 and above.

The grids are those whose passes before the inverse z transform round alike on
both schedules; at 24, 32 and 120 the two forms of the x pass fuse the Coulomb
product differently.
"""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2110_07670_amd import _lib
    _lib.load()
    return _lib


def _w(lib, phi, four_pass):
    plan = lib.Plan(phi.shape[1], (7.0, 8.0, 9.0), phi.shape[0], "fp32", 0.25)
    plan.set_tiling(16)
    plan.set_schedule(four_pass)
    return lib.ace_build(plan, phi)["W"]


@pytest.mark.parametrize("n", [40, 48, 64, 80, 96, 128, 144, 160])
def test_off_diagonal_potentials(lib, n):
    import torch
    print("[gpu-case] FP32 rounding off the diagonal n=%d" % n, flush=True)
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(n)
    phi = torch.randn((32, n, n, n), generator=gen, dtype=torch.float64, device="cuda:0")
    phi /= n ** 1.5
    off, top = [], 0.0
    for four in (False, True):
        W = _w(lib, phi, four)
        top = max(top, float(W.abs().max()))
        for b in (0, 16):
            W[b:b + 16] -= _w(lib, phi[b:b + 16].contiguous(), four)
        off.append(W)
    assert float((off[0] - off[1]).abs().max()) <= 1e-13 * top
