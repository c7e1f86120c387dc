"""FP32 builds whose last block of orbitals is ragged and meets several full
blocks: those tiles become one, of several row blocks, on the fused pass.

Against the four-pass schedule.  From 64^3 on (four-step lengths of 4 and 8
along the last step) both round every potential alike, so W differs by the
order of FP64 sums alone: 40 terms, 1e-14 normwise, and 1e-12 asked; at 48^3
diagonal tiles round otherwise, so FP32's 1e-6 there.  One case is compared
with the oracle too.
"""
import numpy as np
import pytest

from oracle import ace_oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2110_07670_amd import _lib
    _lib.load()
    return _lib


def _fields(n, k):
    import torch
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(n + k)
    phi = torch.randn((k, n, n, n), generator=gen, dtype=torch.float64, device="cuda:0")
    return phi / n ** 1.5


def _w(lib, phi, block, four_pass):
    plan = lib.Plan(phi.shape[1], (7.0, 8.0, 9.0), phi.shape[0], "fp32", 0.25)
    plan.set_tiling(block)
    plan.set_schedule(four_pass)
    return lib.ace_build(plan, phi)["W"]


@pytest.mark.parametrize("k,block", [(20, 8), (28, 8), (40, 16)])
@pytest.mark.parametrize("n", [48, 64, 80, 96, 128])
def test_merged_ragged_tiles(lib, n, k, block):
    print("[gpu-case] merged ragged tiles n=%d k=%d block=%d" % (n, k, block), flush=True)
    phi = _fields(n, k)
    a, b = _w(lib, phi, block, False), _w(lib, phi, block, True)
    assert float((a - b).norm() / b.norm()) < (1e-6 if n == 48 else 1e-12)


def test_merged_ragged_tiles_oracle(lib):
    print("[gpu-case] merged ragged tiles against the oracle", flush=True)
    phi = _fields(40, 20)
    W = _w(lib, phi, 8, False).cpu().numpy()
    ref = O.apply_vx(phi.cpu().numpy(), np.diag([7.0, 8.0, 9.0]), 0.25)
    assert O.rel_err(W, ref) < 1e-6
